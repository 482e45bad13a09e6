"""k_one (whole one-mode propagations by one workgroup per state) at the edges
of its line buckets, element counts and launch splits, against the FP64 oracle
and against the launches per pass (CHFPE_ONE=0).

Tolerances: FP64 rounding of two RK4 steps is a few 1e-16 relative L2, 1e-13
is the bar of the other parity tests; the two device paths differ by rounding
alone, which 300 steps of a bounded propagation let grow to below 1e-11; FP32
branches agree to the 1e-4 of the FP32 bar.
"""
import numpy as np
import pytest

import oracle as orc
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pk():
    import torch
    import paper_2509_25840_amd as pk
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    return pk


def rel_l2(a, b):
    a, b = np.asarray(a, dtype=np.float64).ravel(), np.asarray(b, dtype=np.float64).ravel()
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("Nq,Np,K", [(5, 5, 0), (16, 16, 3), (16, 15, 6), (17, 9, 1), (32, 32, 4), (31, 32, 6), (33, 48, 3),
                                     (48, 48, 0), (48, 48, 3), (7, 48, 2), (48, 6, 3), (40, 41, 5)])
def test_steps_and_response_match_the_oracle(pk, Nq, Np, K):
    print(f"[k_one] {Nq} x {Np} depth {K}", flush=True)
    w = wl.workload("one_mode_48", Nq=[Nq], Np=[Np], K=K)
    sm = wl.smooth_state(w, seed=2)
    W = orc.boltzmann(w)[0][None] * (1.0 + 0.3 * sm / np.abs(sm).max() + 0.05 * wl.noise_state(w, seed=3))
    with pk.Solver(pk.params_from_workload(w)) as s:
        s.set_state(W)
        s.propagate(2, 0.002)
        e = rel_l2(s.get_state(), orc.rk4(w, W, 2, 0.002))
        Weq = orc.equilibrate(w, 6, 0.004)
        s.equilibrate(6, 0.004)
        r = rel_l2(s.response_1d(w["A"], 9, 2, 0.004), orc.response_1d(w, w["A"], Weq, 9, 2, 0.004))
    print(f"    rk4 {e:.2e} response {r:.2e}", flush=True)
    assert e < 1e-13 and r < 1e-10


@pytest.mark.parametrize("batch,prec,tol", [(0, "f64", 1e-11), (3, "f64", 1e-11), (3, "f32", 1e-4)])
def test_long_and_batched_runs_match_the_launches_per_pass(pk, monkeypatch, batch, prec, tol):
    """Propagations over a launch's step limit (300 steps, and a stride of
    260), and waves of branches with a ragged last one."""
    w = wl.workload("one_mode_48", Nq=[20], Np=[18], K=3)
    P = wl.optical(1, lin=[1.0], quad=[[0.1]])
    out = {}
    for one in ("0", "1"):
        monkeypatch.setenv("CHFPE_ONE", one)
        with pk.Solver(pk.params_from_workload(w, precision=pk.CHFPE_FP32 if prec == "f32" else pk.CHFPE_FP64,
                                               batch=batch)) as s:
            s.equilibrate(300, 0.004)
            out[one] = [s.get_state(), s.response_1d(w["A"], 3, 260, 0.004),
                        s.response_2d(w["A"], P, w["A"], 5, 4, 3, 2, 0.004),
                        s.response_3d(w["A"], P, P, w["A"], 2, 5, 3, 1, 2, 0.004)]
    for a, b in zip(out["1"], out["0"]):
        print(f"    {rel_l2(a, b):.2e}", flush=True)
        assert rel_l2(a, b) < tol
