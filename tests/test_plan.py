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


@pytest.mark.parametrize("N", [8, 12, 16])
def test_three_mode_q_cubes(plan, N):
    for Np, prec in (((8, 8, 8), 0), ((6, 7, 10), 1), ((5, 5, 12), 1)):
        got = plan(3, [N] * 3, Np, precision=prec, batch=2)
        assert got["q"] == "k_qcube" and got["q_closure"] == ("" if prec else "k_qpass")
        assert plan(3, [N] * 3, Np, precision=prec, batch=2, CHFPE_QCUBE=0)["q"] == "k_qpass"
    assert plan(3, [N] * 3, (5, 5, 7))["q"] == "k_qpass"  # 175 p points: no whole 16-byte vectors


def test_one_mode(plan):
    cases = next(m for m in test_gpu_one.test_steps_and_response_match_the_oracle.pytestmark if m.name == "parametrize")
    for Nq, Np, K in cases.args[1]:
        # both derivative arrays of K + 1 elements fit the LDS
        fits = (Nq, Np, K) != (40, 41, 5)
        assert plan(1, [Nq], [Np], K)["one"] == fits, (Nq, Np, K)
        assert not plan(1, [Nq], [Np], K, CHFPE_ONE=0)["one"]
    assert plan(1, [20], [18], 3)["one"]


def test_the_plan_is_refused_where_setup_refuses(plan):
    import paper_2509_25840_amd as pk
    with pytest.raises(pk.ChfpeError):
        plan(2, (5, 49), (8, 8))
    out = (ctypes.c_int32 * 6)()
    assert pk.lib().chfpe_kernel_plan(None, out, 6) == pk.CHFPE_EINVAL
    p = pk.params_from_workload(wl.workload("one_mode_48"))
    assert pk.lib().chfpe_kernel_plan(ctypes.byref(p), None, 6) == pk.CHFPE_EINVAL
    assert pk.lib().chfpe_kernel_plan(ctypes.byref(p), out, 2) == 2
