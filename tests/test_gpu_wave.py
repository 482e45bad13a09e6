"""The wave-plane kernels (k_pwave, k_pwave2, k_hwave) at the edges of their shapes:
cubes of every line bucket, ragged blocks whose planes just fill or just pass
the vectors per lane of a variant, one- and two-plane remainders, and the
shortest axes, against the FP64 oracles.

Tolerance: a right-hand side, an excitation and two RK4 steps are sums of a
few hundred products per value, so FP64 rounding is a few 1e-16 relative L2;
1e-13 is the bar the other parity tests use.
"""
import sys

import numpy as np
import pytest

import oracle as orc
import oracle.hermite as oh
import workloads as wl

pytestmark = pytest.mark.gpu

TOL = 1e-13


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def rel_l2(a, b):
    a, b = np.asarray(a, dtype=np.float64).ravel(), np.asarray(b, dtype=np.float64).ravel()
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.fixture(scope="module")
def pk():
    import torch
    import paper_2509_25840_amd as pk
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    return pk


# (p axes, K): planes N2 x N3 of 64, 128, 255, 256, 384 and 408 points meet
# the vector counts 1, 2, 4, 6 and 9; N1 leaves part of the last wave idle
PWAVE = [((8, 8, 8), 2), ((5, 8, 8), 1), ((7, 5, 6), 2), ((12, 12, 12), 2), ((9, 12, 11), 1), ((16, 16, 16), 2),
         ((13, 8, 16), 1), ((16, 9, 15), 2), ((5, 16, 16), 1), ((24, 24, 24), 1), ((17, 15, 17), 1), ((5, 16, 24), 1),
         ((23, 24, 17), 1), ((24, 5, 5), 1)]
X3 = {"lin": [1.0, -0.7, 0.4], "quad": [[0.2, 0.05, -0.03], [0.05, -0.1, 0.02], [-0.03, 0.02, 0.3]]}


@pytest.mark.parametrize("Np,K", PWAVE, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else f"k{v}")
def test_pwave_matches_the_oracle(pk, Np, K):
    w = wl.workload("three_mode_24", Nq=[5, 6, 5], Np=list(Np), K=K)
    say(f"[k_pwave] p {Np} K {K}")
    env = orc.boltzmann(w)[0]
    sm = wl.smooth_state(w, seed=3)
    W = env[None] * (1.0 + 0.3 * sm / np.abs(sm).max() + 0.05 * wl.noise_state(w, seed=4))
    with pk.Solver(pk.params_from_workload(w)) as s:
        assert s.tile_config()["pcube_stream"] == 1
        s.set_state(W)
        s.rhs()
        e_rhs = rel_l2(s.get_state(), orc.rhs(w, W))
        s.set_state(W)
        s.propagate(2, 0.002)
        e_rk4 = rel_l2(s.get_state(), orc.rk4(w, W, 2, 0.002))
        s.set_state(W)
        s.perturb(X3)
        e_x = rel_l2(s.get_state(), orc.perturb(w, X3, W))
    say(f"    rhs {e_rhs:.2e} rk4 {e_rk4:.2e} perturb {e_x:.2e}")
    assert e_rhs < TOL and e_rk4 < TOL and e_x < TOL


# (p axes, K): squares of every line bucket; planes N1 x N2 that just fill or just
# pass 64 values per lane slot; task counts that are no multiple of a
# workgroup's four
PWAVE2 = [((8, 8), 2), ((12, 12), 1), ((16, 16), 3), ((24, 24), 0), ((32, 32), 1), ((5, 8), 1), ((7, 6), 0), ((9, 12), 2),
          ((16, 12), 0), ((13, 16), 1), ((24, 16), 1), ((17, 23), 2), ((32, 20), 1), ((25, 26), 0), ((31, 32), 1),
          ((5, 32), 2), ((29, 5), 1)]


@pytest.mark.parametrize("Np,K", PWAVE2, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else f"k{v}")
def test_pwave2_matches_the_oracle_and_k_pblock(pk, monkeypatch, Np, K):
    """k_pwave2 (two modes, p axes of up to 32 points): the oracle's right-hand
    side, RK4 steps and excitation, and k_pblock's FP32 branches
    (CHFPE_PWAVE2=0)."""
    w = wl.workload("two_mode_32", Nq=[5, 7], Np=list(Np), K=K)
    say(f"[k_pwave2] p {Np} K {K}")
    env = orc.boltzmann(w)[0]
    sm = wl.smooth_state(w, seed=3)
    W = env[None] * (1.0 + 0.3 * sm / np.abs(sm).max() + 0.05 * wl.noise_state(w, seed=4))
    X2 = {"lin": X3["lin"][:2], "quad": [r[:2] for r in X3["quad"][:2]]}
    R = {}
    for on in ("1", "0"):
        monkeypatch.setenv("CHFPE_PWAVE2", on)
        with pk.Solver(pk.params_from_workload(w)) as s:
            s.set_state(W)
            s.rhs()
            e_rhs = rel_l2(s.get_state(), orc.rhs(w, W))
            s.set_state(W)
            s.propagate(2, 0.002)
            e_rk4 = rel_l2(s.get_state(), orc.rk4(w, W, 2, 0.002))
            s.set_state(W)
            s.perturb(X2)
            e_x = rel_l2(s.get_state(), orc.perturb(w, X2, W))
        say(f"    rhs {e_rhs:.2e} rk4 {e_rk4:.2e} perturb {e_x:.2e}")
        assert e_rhs < TOL and e_rk4 < TOL and e_x < TOL
        with pk.Solver(pk.params_from_workload(w, precision=pk.CHFPE_FP32, batch=3)) as s:
            s.equilibrate(4, 0.004)
            R[on] = s.response_2d(w["A"], w["B"], w["C"], 4, 4, 1, 2, 0.004)
    say(f"    FP32 branches {rel_l2(R['1'], R['0']):.2e}")
    assert rel_l2(R["1"], R["0"]) < 1e-4


# (q axes, Hermite functions, K): as above; two modes take planes N1 x N2 by
# four tasks per workgroup (task counts that are no multiple of four)
HWAVE = [((8, 8, 8), (3, 2, 3), 2), ((12, 12, 12), (2, 3, 2), 2), ((16, 16, 16), (2, 2, 3), 1), ((24, 24, 24), (2, 3, 2), 1),
         ((5, 16, 24), (2, 2, 2), 2), ((23, 24, 17), (2, 2, 2), 1), ((7, 9, 16), (2, 3, 2), 2), ((5, 6, 7), (3, 3, 3), 1),
         ((32, 32), (4, 3), 3), ((24, 24), (3, 3), 2), ((16, 16), (5, 3), 1), ((12, 12), (3, 4), 2), ((8, 8), (3, 5), 3),
         ((31, 20), (3, 3), 2), ((5, 32), (3, 3), 1), ((16, 24), (3, 5), 0), ((25, 16), (3, 3), 1)]


@pytest.mark.parametrize("Nq,Nh,K", HWAVE, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else f"k{v}")
def test_hwave_matches_the_oracle(pk, Nq, Nh, K):
    M = len(Nq)
    w = wl.workload({2: "two_mode_32", 3: "three_mode_24"}[M], Nq=list(Nq), Np=list(Nh), K=K, basis="hermite")
    say(f"[k_hwave] q {Nq} functions {Nh} K {K}")
    rng = np.random.default_rng(8)
    qs = np.meshgrid(*[oh.q_grid(w, s) for s in range(M)], indexing="ij")
    env = np.exp(-0.35 * sum((w["omega"][s] * qs[s]) ** 2 for s in range(M)))
    C = rng.normal(size=oh.shape(w)[:1 + M] + (1,) * M) * env * (1.0 + 0.1 * rng.normal(size=oh.shape(w)))
    T = oh.tables(w)
    with pk.Solver(pk.params_from_workload(w)) as s:
        s.set_state(C)
        s.rhs()
        e_rhs = rel_l2(s.get_state(), oh.rhs(w, C, T))
        s.set_state(C)
        s.propagate(2, 0.002)
        e_rk4 = rel_l2(s.get_state(), oh.rk4(w, C, 2, 0.002, T))
    say(f"    rhs {e_rhs:.2e} rk4 {e_rk4:.2e}")
    assert e_rhs < TOL and e_rk4 < TOL


@pytest.mark.parametrize("N", [8, 12, 16])
@pytest.mark.parametrize("Np", [(8, 8, 8), (6, 7, 10), (5, 5, 12)])
def test_qcube_matches_the_oracle_and_the_two_passes(pk, monkeypatch, N, Np):
    """k_qcube (q cubes of 8, 12 and 16 points) with p blocks that end in a
    whole and in a partial run of 64 bytes: the oracle's right-hand side and RK4
    steps, and the (q_2, q_3) and q_1 passes' FP32 branches (CHFPE_QCUBE=0)."""
    w = wl.workload("three_mode_24", Nq=[N] * 3, Np=list(Np), K=1)
    say(f"[k_qcube] q {N} p {Np}")
    env = orc.boltzmann(w)[0]
    sm = wl.smooth_state(w, seed=5)
    W = env[None] * (1.0 + 0.3 * sm / np.abs(sm).max() + 0.05 * wl.noise_state(w, seed=6))
    R = {}
    for on in ("1", "0"):
        monkeypatch.setenv("CHFPE_QCUBE", on)
        with pk.Solver(pk.params_from_workload(w)) as s:
            s.set_state(W)
            s.rhs()
            e_rhs = rel_l2(s.get_state(), orc.rhs(w, W))
            s.set_state(W)
            s.propagate(2, 0.002)
            e_rk4 = rel_l2(s.get_state(), orc.rk4(w, W, 2, 0.002))
        assert e_rhs < TOL and e_rk4 < TOL
        with pk.Solver(pk.params_from_workload(w, precision=pk.CHFPE_FP32, batch=2)) as s:
            s.equilibrate(4, 0.004)
            R[on] = s.response_2d(w["A"], w["B"], w["C"], 3, 4, 1, 2, 0.004)
    say(f"    rhs {e_rhs:.2e} rk4 {e_rk4:.2e} FP32 branches {rel_l2(R['1'], R['0']):.2e}")
    assert rel_l2(R["1"], R["0"]) < 1e-4
