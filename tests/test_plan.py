"""Which kernels a context runs (chfpe_kernel_plan; host only): the shapes that
the GPU tests of one kernel use do run it, and CHFPE_* switches leave it."""
import ctypes

import pytest

import test_gpu_one
import test_gpu_wave
import workloads as wl

SWITCHES = ("CHFPE_PWAVE", "CHFPE_PWAVE2", "CHFPE_HWAVE", "CHFPE_QCUBE", "CHFPE_ONE", "CHFPE_PCUBE",
            "CHFPE_TUNE_PC_STREAM", "CHFPE_TUNE_PB_NB", "CHFPE_TUNE_PB_SPLIT", "CHFPE_TUNE_PB_RUN", "CHFPE_TUNE_Q_PC")


@pytest.fixture
def plan(monkeypatch):
    import paper_2509_25840_amd as pk
    for v in SWITCHES:
        monkeypatch.delenv(v, raising=False)

    def of(M, Nq, Np, K=1, precision=0, batch=0, basis=None, **env):
        w = wl.workload({1: "one_mode_48", 2: "two_mode_32", 3: "three_mode_24"}[M], Nq=list(Nq), Np=list(Np), K=K,
                        **({"basis": basis} if basis else {}))
        with monkeypatch.context() as m:
            for k, v in env.items():
                m.setenv(k, str(v))
            return pk.kernel_plan(pk.params_from_workload(w, precision=precision, batch=batch))
    return of


@pytest.mark.parametrize("Np,K", test_gpu_wave.PWAVE2)
def test_two_modes(plan, Np, K):
    assert plan(2, (5, 7), Np, K)["state"] == "k_pwave2"
    got = plan(2, (5, 7), Np, K, precision=1, batch=3)
    assert got["state"] == got["branches"] == "k_pwave2" and got["q"] == "k_qpass"
    assert plan(2, (5, 7), Np, K, CHFPE_PWAVE2=0)["state"] in ("k_pblock", "k_pcube")


@pytest.mark.parametrize("N", range(5, 17))
def test_three_mode_q_cubes(plan, N):
    for Np, prec in (((8, 8, 8), 0), ((6, 7, 10), 1), ((5, 5, 12), 1)):
        got = plan(3, [N] * 3, Np, precision=prec, batch=2)
        assert got["q"] == "k_qcube" and got["q_closure"] == ("" if prec else "k_qpass")
        assert plan(3, [N] * 3, Np, precision=prec, batch=2, CHFPE_QCUBE=0)["q"] == "k_qpass"
    assert plan(3, [N] * 3, (5, 5, 7))["q"] == "k_qpass"  # 175 p points: no whole 16-byte vectors
    assert plan(3, [N, N, N + 1], (8, 8, 8))["q"] == "k_qpass"
    assert plan(3, [17] * 3, (8, 8, 8))["q"] == "k_qpass"


# (p axes, FP64 state, FP32 branches, FP64 state with a closure): planes on either
# side of each line between k_pwave and k_pcube, and axes that only k_pcube_s takes
THREE = [((24, 5, 5), "k_pcube", "k_pcube", ""), ((24, 12, 12), "k_pcube", "k_pwave", ""),
         ((24, 9, 18), "k_pwave", "k_pwave", ""), ((17, 12, 10), "k_pcube", "k_pcube", ""),
         ((20, 13, 17), "k_pcube", "k_pwave", ""), ((20, 13, 18), "k_pwave", "k_pwave", ""),
         ((16, 15, 17), "k_pcube_s", "k_pcube_s", ""), ((16, 16, 17), "k_pwave", "k_pcube_s", ""),
         ((10, 10, 17), "k_pcube_s", "k_pwave", ""), ((8, 16, 17), "k_pwave", "k_pwave", ""),
         ((5, 6, 20), "k_pcube_s", "k_pwave", ""), ((5, 5, 18), "k_pcube_s", "k_pcube_s", ""),
         ((5, 7, 20), "k_pwave", "k_pwave", ""), ((16, 8, 8), "k_pcube_s", "k_pcube_s", "k_pcube"),
         ((16, 9, 9), "k_pcube_s", "k_pwave", "k_pwave"), ((13, 11, 11), "k_pwave", "k_pwave", "k_pwave"),
         ((12, 8, 8), "k_pcube_s", "k_pcube_s", "k_pcube"), ((12, 10, 10), "k_pcube_s", "k_pwave", "k_pcube"),
         ((12, 11, 11), "k_pwave", "k_pwave", "k_pwave"), ((14, 9, 11), "k_pwave", "k_pwave", "k_pwave"),
         ((5, 5, 13), "k_pwave", "k_pwave", "k_pcube"), ((5, 5, 9), "k_pcube_s", "k_pcube_s", "k_pcube"),
         ((5, 6, 9), "k_pwave", "k_pwave", "k_pcube"), ((8, 5, 5), "k_pwave", "k_pwave", "k_pwave"),
         ((12, 12, 12), "k_pwave", "k_pwave", "k_pwave"), ((8, 5, 26), "k_pcube_s", "k_pcube_s", ""),
         ((16, 26, 9), "k_pcube_s", "k_pcube_s", ""), ((20, 7, 25), "k_pcube", "k_pcube", "")]


@pytest.mark.parametrize("Np,f64,f32,clos", THREE)
def test_three_modes(plan, Np, f64, f32, clos):
    got = plan(3, (5, 6, 5), Np, precision=1, batch=2)
    assert (got["state"], got["branches"]) == (f64, f32)
    got = plan(3, (5, 6, 5), Np)
    assert (got["state"], got["branches"], got["closure"]) == (f64, "", clos)
    left = plan(3, (5, 6, 5), Np, precision=1, batch=2, CHFPE_PWAVE=0)
    assert left["state"] == left["branches"] == ("k_pcube_s" if Np[0] <= 16 else "k_pcube")


# (q axes, FP64 state, FP32 branches): as above for k_hwave and k_hcube
HERMITE = [((24, 5, 5), "k_hcube", "k_hcube"), ((24, 13, 13), "k_hcube", "k_hwave"), ((24, 11, 18), "k_hwave", "k_hwave"),
           ((17, 14, 14), "k_hwave", "k_hcube"), ((17, 16, 17), "k_hwave", "k_hwave"), ((16, 15, 17), "k_hcube", "k_hcube"),
           ((16, 16, 17), "k_hwave", "k_hwave"), ((12, 10, 20), "k_hcube", "k_hwave"), ((10, 9, 18), "k_hcube", "k_hcube"),
           ((10, 12, 18), "k_hcube", "k_hwave"), ((5, 13, 20), "k_hwave", "k_hwave"), ((16, 7, 7), "k_hwave", "k_hcube"),
           ((16, 6, 6), "k_hcube", "k_hcube"), ((13, 8, 8), "k_hcube", "k_hcube"), ((13, 9, 9), "k_hwave", "k_hwave"),
           ((12, 5, 5), "k_hwave", "k_hcube"), ((12, 8, 8), "k_hwave", "k_hwave"), ((8, 5, 5), "k_hwave", "k_hwave"),
           ((32, 8, 9), "k_hcube", "k_hcube"), ((6, 27, 7), "k_hcube", "k_hcube"), ((40, 20), "k_hcube", "k_hcube"),
           ((33, 9), "k_hcube", "k_hcube"), ((5, 5), "k_hwave", "k_hwave"), ((32, 5), "k_hwave", "k_hwave"),
           ((31,), "k_hcube", "k_hcube")]


@pytest.mark.parametrize("Nq,f64,f32", HERMITE)
def test_hermite_basis(plan, Nq, f64, f32):
    got = plan(len(Nq), Nq, (3, 2, 2)[:len(Nq)], precision=1, batch=2, basis="hermite")
    assert (got["state"], got["branches"], got["q"]) == (f64, f32, "")
    left = plan(len(Nq), Nq, (3, 2, 2)[:len(Nq)], precision=1, batch=2, basis="hermite", CHFPE_HWAVE=0)
    assert left["state"] == left["branches"] == "k_hcube"


@pytest.mark.parametrize("Np,prec,batch,branches", [
    ((8, 8), 0, 9, "k_pwave2"), ((8, 8), 0, 64, "k_pblock"), ((8, 8), 1, 64, "k_pblock"), ((5, 5), 0, 64, "k_pwave2"),
    ((13, 5), 0, 64, "k_pwave2"), ((25, 5), 0, 16, "k_pblock"), ((25, 5), 1, 16, "k_pwave2"), ((24, 6), 0, 16, "k_pwave2"),
    ((20, 6), 0, 16, "k_pblock"), ((32, 6), 0, 16, "k_pblock"), ((28, 8), 0, 16, "k_pwave2"), ((32, 5), 0, 3, "k_pwave2")])
def test_two_mode_waves_of_small_planes(plan, Np, prec, batch, branches):
    got = plan(2, (20, 24), Np, precision=prec, batch=batch)
    assert (got["state"], got["branches"]) == ("k_pwave2", branches)


@pytest.mark.parametrize("Nq,Np,K,prec,batch,positions", [
    ((30, 30), (16, 16), 3, 0, 0, 16), ((30, 30), (10, 10), 3, 0, 0, 8), ((30, 30), (24, 24), 3, 0, 0, 8),
    ((18, 22), (16, 16), 3, 0, 16, 8), ((32, 32), (16, 16), 3, 0, 0, 16), ((32, 32), (24, 24), 3, 0, 0, 8),
    ((32, 32), (16, 16), 3, 0, 64, 16), ((13, 15), (10, 10), 3, 0, 0, 16), ((24, 24), (24, 24), 3, 0, 0, 8),
    ((8, 18, 17), (8, 8, 8), 1, 1, 2, 8), ((8, 12, 12), (16, 16, 16), 1, 1, 4, 16)])
def test_width_of_two_axis_q_tiles(plan, Nq, Np, K, prec, batch, positions):
    assert plan(len(Nq), Nq, Np, K, precision=prec, batch=batch)["q_positions"] == positions


def test_one_mode(plan):
    cases = next(m for m in test_gpu_one.test_steps_and_response_match_the_oracle.pytestmark if m.name == "parametrize")
    for Nq, Np, K in cases.args[1]:
        # both derivative arrays of K + 1 elements fit the LDS
        fits = (Nq, Np, K) != (40, 41, 5)
        assert plan(1, [Nq], [Np], K)["one"] == fits, (Nq, Np, K)
        assert not plan(1, [Nq], [Np], K, CHFPE_ONE=0)["one"]
    assert plan(1, [20], [18], 3)["one"]


@pytest.mark.parametrize("Nq,K,batch", [((5, 17), 11, 1024), ((5, 17), 12, 900), ((17, 5), 11, 1024), ((5, 26), 10, 900),
                                        ((5, 18), 12, 900)])
def test_half_width_q_tiles_refuse_no_batch(plan, Nq, K, batch):
    """FP32 waves of 251 to 286 GB whose (q_1, q_2) launch fits one dispatch (2^32
    work-items) with tiles of 16 positions, and would not with 8."""
    assert plan(2, Nq, (48, 48), K, precision=1, batch=batch)["branches"] == "k_pcube"
    assert plan(2, Nq, (48, 48), K, precision=1, batch=batch, CHFPE_TUNE_Q_PC=16)["branches"] == "k_pcube"


def test_the_plan_is_refused_where_setup_refuses(plan):
    import paper_2509_25840_amd as pk
    with pytest.raises(pk.ChfpeError):
        plan(2, (5, 49), (8, 8))
    out = (ctypes.c_int32 * 6)()
    assert pk.lib().chfpe_kernel_plan(None, out, 6) == pk.CHFPE_EINVAL
    p = pk.params_from_workload(wl.workload("one_mode_48"))
    assert pk.lib().chfpe_kernel_plan(ctypes.byref(p), None, 6) == pk.CHFPE_EINVAL
    assert pk.lib().chfpe_kernel_plan(ctypes.byref(p), out, 2) == 2
