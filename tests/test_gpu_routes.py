"""Results on either side of the lines between kernels of the same work: the
shapes of test_plan.py, whose kernels that file asserts, against the oracles,
and waves of branches against the FP64 responses of single states.

Tolerances: FP64 as in the other parity tests (a few hundred products per value
and two RK4 steps: 1e-13; 200 steps of a bounded propagation by another
kernel: 1e-11).  FP32 branches round every value four times a step, 6e-8 each:
at most 5e-5 after the 200 steps of a branch here, below the FP32 bar of 1e-4.
(The times are long enough for R to develop: at t near 0 it is a difference of
far larger terms.)
"""
import numpy as np
import pytest

import oracle as orc
import oracle.closure as cl
import oracle.hermite as oh
import test_plan
import workloads as wl

pytestmark = pytest.mark.gpu

TOL = 1e-13
X3 = {"lin": [1.0, -0.7, 0.4], "quad": [[0.2, 0.05, -0.03], [0.05, -0.1, 0.02], [-0.03, 0.02, 0.3]]}


def rel_l2(a, b):
    a, b = np.asarray(a, dtype=np.float64).ravel(), np.asarray(b, dtype=np.float64).ravel()
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def ops(M):
    return {"lin": X3["lin"][:M], "quad": [r[:M] for r in X3["quad"][:M]]}


def grid_state(w, seed):
    sm = wl.smooth_state(w, seed=seed)
    return orc.boltzmann(w)[0][None] * (1.0 + 0.3 * sm / np.abs(sm).max() + 0.05 * wl.noise_state(w, seed=seed + 1))


@pytest.fixture(scope="module")
def pk():
    import torch
    import paper_2509_25840_amd as pk
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    return pk


def check_waves(pk, w, batch=2, n_t1=3, prec=1):
    """Branch waves (the last one ragged) against the response of single states."""
    M = w["M"]
    A, B = ops(M), wl.optical(M, lin=[0.5, 0.8, -0.3][:M])
    R = {}
    for key, kw in (("one", {}), ("wave", {"precision": prec, "batch": batch})):
        with pk.Solver(pk.params_from_workload(w, **kw)) as s:
            s.equilibrate(20, 0.005)
            R[key] = s.response_2d(A, B, A, n_t1, 6, 40 // n_t1 + 1, 40, 0.005)
    e = rel_l2(R["wave"], R["one"])
    print(f"    waves {e:.2e} of {np.abs(R['one']).max():.1e}", flush=True)
    assert e < (1e-4 if prec else 1e-11)


@pytest.mark.parametrize("Np", [c[0] for c in test_plan.THREE], ids=str)
def test_three_modes(pk, Np):
    print(f"[three modes] p {Np}", flush=True)
    w = wl.workload("three_mode_24", Nq=[5, 6, 5], Np=list(Np), K=1)
    W = grid_state(w, 3)
    with pk.Solver(pk.params_from_workload(w)) as s:
        s.set_state(W)
        s.rhs()
        e_rhs = rel_l2(s.get_state(), orc.rhs(w, W))
        s.set_state(W)
        s.propagate(2, 0.002)
        e_rk4 = rel_l2(s.get_state(), orc.rk4(w, W, 2, 0.002))
        s.set_state(W)
        s.perturb(X3)
        e_x = rel_l2(s.get_state(), orc.perturb(w, X3, W))
    print(f"    rhs {e_rhs:.2e} rk4 {e_rk4:.2e} perturb {e_x:.2e}", flush=True)
    assert e_rhs < TOL and e_rk4 < TOL and e_x < TOL
    check_waves(pk, w)


@pytest.mark.parametrize("Np", [c[0] for c in test_plan.THREE if c[3]], ids=str)
def test_three_modes_with_a_closure(pk, Np):
    print(f"[closure] p {Np}", flush=True)
    w = wl.workload("three_mode_24", Nq=[5, 6, 5], Np=list(Np), K=1)
    sv = np.random.default_rng(9).normal(0, 0.02, len(cl.features(w)))
    W = grid_state(w, 5)
    with pk.Solver(pk.params_from_workload(w)) as s:
        s.set_closure(sv)
        s.set_state(W)
        s.propagate(2, 0.002)
        e_rk4 = rel_l2(s.get_state(), cl.propagate(w, W, 2, 0.002, sv))
        s.set_state(W)
        s.perturb(X3)
        e_x = rel_l2(s.get_state(), cl.perturb(w, X3, W, sv))
    print(f"    rk4 {e_rk4:.2e} perturb {e_x:.2e}", flush=True)
    assert e_rk4 < TOL and e_x < TOL


@pytest.mark.parametrize("Nq", [c[0] for c in test_plan.HERMITE], ids=str)
def test_hermite_basis(pk, Nq):
    M = len(Nq)
    print(f"[hermite] q {Nq}", flush=True)
    w = wl.workload({1: "one_mode_48", 2: "two_mode_32", 3: "three_mode_24"}[M], Nq=list(Nq), Np=[3, 2, 2][:M], K=2,
                    basis="hermite")
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
    print(f"    rhs {e_rhs:.2e} rk4 {e_rk4:.2e}", flush=True)
    assert e_rhs < TOL and e_rk4 < TOL
    check_waves(pk, w)


# planes of one, three and five vectors a lane, and waves of more and fewer states
# than k_pblock takes over at
@pytest.mark.parametrize("Np,batch,prec", [((9, 5), 2, 1), ((20, 5), 2, 1), ((24, 8), 2, 1), ((32, 5), 2, 1),
                                           ((32, 8), 2, 1), ((25, 12), 2, 0), ((27, 17), 2, 1), ((8, 8), 24, 0),
                                           ((8, 8), 24, 1), ((5, 5), 24, 0), ((25, 5), 12, 0), ((20, 6), 12, 0)], ids=str)
def test_two_modes(pk, Np, batch, prec):
    print(f"[two modes] p {Np}, {batch} states", flush=True)
    w = wl.workload("two_mode_32", Nq=[9, 9], Np=list(Np), K=3)
    W = grid_state(w, 3)
    with pk.Solver(pk.params_from_workload(w)) as s:
        s.set_state(W)
        s.propagate(2, 0.002)
        e_rk4 = rel_l2(s.get_state(), orc.rk4(w, W, 2, 0.002))
        s.set_state(W)
        s.perturb(ops(2))
        e_x = rel_l2(s.get_state(), orc.perturb(w, ops(2), W))
    print(f"    rk4 {e_rk4:.2e} perturb {e_x:.2e}", flush=True)
    assert e_rk4 < TOL and e_x < TOL
    check_waves(pk, w, batch=batch, n_t1=batch + 1, prec=prec)


# FP32 branches by every form of the wave-plane kernels: cubes (16-byte vectors)
# of each line bucket, and the vector counts of ragged planes
PWAVE32 = [(8, 8, 8), (12, 12, 12), (16, 16, 16), (24, 24, 24), (7, 5, 6), (9, 12, 11), (13, 8, 16), (9, 15, 16),
           (12, 7, 20), (5, 16, 24), (23, 24, 17)]
HWAVE32 = [(8, 8, 8), (12, 12, 12), (16, 16, 16), (24, 24, 24), (5, 6, 7), (9, 12, 11), (7, 9, 16), (5, 16, 24),
           (23, 24, 17), (8, 8), (12, 12), (16, 16), (24, 24), (32, 32), (5, 7), (9, 11), (13, 16), (20, 17), (25, 15),
           (31, 20)]


@pytest.mark.parametrize("Np", PWAVE32, ids=str)
def test_fp32_waves_of_k_pwave(pk, Np):
    print(f"[k_pwave FP32] p {Np}", flush=True)
    w = wl.workload("three_mode_24", Nq=[5, 6, 5], Np=list(Np), K=1)
    plan = pk.kernel_plan(pk.params_from_workload(w, precision=1, batch=2))
    assert plan["branches"] == "k_pwave"
    check_waves(pk, w)


@pytest.mark.parametrize("Nq", HWAVE32, ids=str)
def test_fp32_waves_of_k_hwave(pk, Nq):
    print(f"[k_hwave FP32] q {Nq}", flush=True)
    M = len(Nq)
    w = wl.workload({2: "two_mode_32", 3: "three_mode_24"}[M], Nq=list(Nq), Np=[3, 2, 2][:M], K=2, basis="hermite")
    plan = pk.kernel_plan(pk.params_from_workload(w, precision=1, batch=2))
    assert plan["branches"] == "k_hwave"
    check_waves(pk, w)


# k_pblock for one mode (k_one switched off), with its line solves by lane pairs and by lanes
@pytest.mark.parametrize("split", ["0", "1"])
@pytest.mark.parametrize("Nq,Np", [(9, 12), (12, 24), (10, 48), (7, 31)])
def test_one_mode_k_pblock(pk, monkeypatch, Nq, Np, split):
    monkeypatch.setenv("CHFPE_ONE", "0")
    monkeypatch.setenv("CHFPE_TUNE_PB_SPLIT", split)
    print(f"[k_pblock] one mode {Nq} x {Np} split {split}", flush=True)
    w = wl.workload("one_mode_48", Nq=[Nq], Np=[Np], K=2)
    p = pk.params_from_workload(w)
    assert pk.kernel_plan(p)["state"] == "k_pblock" and not pk.kernel_plan(p)["one"]
    W = grid_state(w, 7)
    with pk.Solver(p) as s:
        s.set_state(W)
        s.propagate(2, 0.002)
        e_rk4 = rel_l2(s.get_state(), orc.rk4(w, W, 2, 0.002))
        s.set_state(W)
        s.perturb(ops(1))
        e_x = rel_l2(s.get_state(), orc.perturb(w, ops(1), W))
    print(f"    rk4 {e_rk4:.2e} perturb {e_x:.2e}", flush=True)
    assert e_rk4 < TOL and e_x < TOL


# q cubes whose planes fill the rounds of k_qcube and leave a partial last one, with
# p blocks that end in a whole and in a partial run of 64 bytes
@pytest.mark.parametrize("Np", [(8, 8, 8), (6, 7, 10)], ids=str)
@pytest.mark.parametrize("N", range(5, 16))
def test_q_cubes(pk, N, Np):
    print(f"[k_qcube] q {N} p {Np}", flush=True)
    w = wl.workload("three_mode_24", Nq=[N] * 3, Np=list(Np), K=1)
    p = pk.params_from_workload(w)
    assert pk.kernel_plan(p)["q"] == "k_qcube"
    W = grid_state(w, 5)
    with pk.Solver(p) as s:
        s.set_state(W)
        s.rhs()
        e_rhs = rel_l2(s.get_state(), orc.rhs(w, W))
        s.set_state(W)
        s.propagate(2, 0.002)
        e_rk4 = rel_l2(s.get_state(), orc.rk4(w, W, 2, 0.002))
    print(f"    rhs {e_rhs:.2e} rk4 {e_rk4:.2e}", flush=True)
    assert e_rhs < TOL and e_rk4 < TOL
    check_waves(pk, w)
