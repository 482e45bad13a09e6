"""Closure training at the edges of its launches: groups smaller than, equal to
and one past a tile of 16 rows, groups that share tiles, more tiles than one
look-ahead of a chain, row counts that leave a partial last tile, and no steps.

Tolerance: the oracle rounds to BF16 where the device does, so a step differs
by FP32 sums of a few hundred terms (2e-5 of a gradient) and by hidden values
that round to the other BF16 neighbour (0.4% of one term of a gradient); Adam
moves a parameter by about the learning rate, 1e-3, so five steps stay far
within 1e-4 of parameters of order 0.25.
"""
import numpy as np
import pytest

import oracle.closure as cl

pytestmark = pytest.mark.gpu

SIZES = [[1], [5], [16], [17], [15, 1, 33], [29, 29, 29, 29], [61, 3, 40, 7], [1] * 40, [300], [61] * 20, [13] * 90]


@pytest.fixture(scope="module")
def pk():
    import torch
    import paper_2509_25840_amd as pk
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    return pk


def flat(p):
    return np.concatenate([p["W1"].ravel(), p["b1"], p["W2"], [p["b2"]]]).astype(np.float32)


@pytest.mark.parametrize("sizes", SIZES, ids=lambda v: f"{len(v)}x{max(v)}")
def test_training_steps_match_the_oracle(pk, sizes):
    rng = np.random.default_rng(len(sizes) + max(sizes))
    start = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    rows = int(start[-1])
    feat = rng.normal(size=(rows, 16)).astype(np.float32)
    feat = cl.bf16(feat).astype(np.float32)
    G, b, ct, groups = [], [], [], []
    for q, P in enumerate(sizes):
        x = rng.normal(size=(P + 4, P))
        r = x @ rng.normal(size=P) * 0.05 + 0.02 * rng.normal(size=P + 4)
        G.append(x.T @ x)
        b.append(x.T @ r)
        ct.append([r @ r, 2.0 * (r @ r)])
        groups.append((np.arange(start[q], start[q + 1]), G[-1], b[-1], *ct[-1]))
    p = cl.init_params(3)
    p["b1"], p["b2"] = rng.normal(0, 0.1, cl.NHID), 0.02
    prm = flat(p)
    p = {"W1": prm[:512].reshape(16, 32).astype(np.float64), "b1": prm[512:544].astype(np.float64),
         "W2": prm[544:576].astype(np.float64), "b2": float(prm[576])}
    tr = pk.ClosureTrainer(prm)
    args = feat, start, np.concatenate([g.ravel() for g in G]), np.concatenate(b), np.array(ct)
    tr.train(*args, n_steps=0, lr=1e-3)
    assert np.array_equal(tr.prm, prm) and not tr.m.any() and not tr.v.any()
    # two calls: the second starts from the first's moments and step count
    loss = np.concatenate([tr.train(*args, n_steps=3, lr=1e-3), tr.train(*args, n_steps=2, lr=1e-3)])
    ref, st = [], {}
    for _ in range(5):
        s, cache = cl.forward(p, feat.astype(np.float64))
        L, gs = cl.loss_grad(s, groups)
        ref.append(L)
        cl.adam_step(p, cl.backward(p, cache, np.float32(gs).astype(np.float64)), st, 1e-3)
    err = np.linalg.norm(tr.prm - flat(p)) / np.linalg.norm(flat(p))
    print(f"[train] {len(sizes)} groups, {rows} rows: parameters {err:.2e}", flush=True)
    assert np.allclose(loss, ref, rtol=1e-4)
    assert err < 1e-4


def test_rows_of_g_are_read_as_rows(pk):
    """G need not be symmetric: the gradient of a row takes that row of G."""
    rng = np.random.default_rng(4)
    sizes = [17, 5, 30, 1, 150]  # (150 x 150: two workgroups transpose it)
    start = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    feat = cl.bf16(rng.normal(size=(int(start[-1]), 16))).astype(np.float32)
    groups = [(np.arange(start[q], start[q + 1]), rng.normal(size=(P, P)), rng.normal(size=P), 1.0, 2.0)
              for q, P in enumerate(sizes)]
    p = cl.init_params(5)
    prm = flat(p)
    p = {"W1": prm[:512].reshape(16, 32).astype(np.float64), "b1": prm[512:544].astype(np.float64),
         "W2": prm[544:576].astype(np.float64), "b2": float(prm[576])}
    tr = pk.ClosureTrainer(prm)
    loss = tr.train(feat, start, np.concatenate([g[1].ravel() for g in groups]), np.concatenate([g[2] for g in groups]),
                    np.array([g[3:] for g in groups]), n_steps=3, lr=1e-3)
    ref, st = [], {}
    for _ in range(3):
        s, cache = cl.forward(p, feat.astype(np.float64))
        L, gs = cl.loss_grad(s, groups)
        ref.append(L)
        cl.adam_step(p, cl.backward(p, cache, np.float32(gs).astype(np.float64)), st, 1e-3)
    assert np.allclose(loss, ref, rtol=1e-4)
    assert np.linalg.norm(tr.prm - flat(p)) / np.linalg.norm(flat(p)) < 1e-4


def test_training_holds_one_copy_of_g(pk):
    """Device memory taken by a call whose G has 0.8 GB, watched while it runs."""
    import threading
    import torch
    P = 10000
    feat = np.random.default_rng(6).normal(size=(P, 16)).astype(np.float32)
    G = np.eye(P)
    net = cl.init_params(7)
    tr = pk.ClosureTrainer(flat(net))
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    least, done = [free], threading.Event()

    def watch():
        while not done.wait(0.002):
            least[0] = min(least[0], torch.cuda.mem_get_info()[0])

    t = threading.Thread(target=watch)
    t.start()
    try:
        loss = tr.train(feat, [0, P], G.ravel(), np.zeros(P), [0.0, 1.0], n_steps=2, lr=1e-3)
    finally:
        done.set()
        t.join()
    taken = free - least[0]
    s, _ = cl.forward(net, feat.astype(np.float64))
    print(f"[train] one group of {P}: {taken / 1e6:.0f} MB", flush=True)
    assert np.allclose(loss[0], np.sum(s * s), rtol=1e-2)
    assert G.nbytes <= taken < 1.5 * G.nbytes
