"""Kernel timing reports the launches that an untimed run makes: one-mode
propagations stay in k_one, with the same results."""
import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,prec", [(0, 0), (3, 0), (3, 1)])
def test_timing_changes_no_launch_of_one_mode(batch, prec):
    import paper_2509_25840_amd as pk
    w = wl.workload("one_mode_48", Nq=[20], Np=[18], K=3)
    P = wl.optical(1, lin=[1.0], quad=[[0.1]])
    out, times = {}, {}
    for every in (0, 1, 100):
        with pk.Solver(pk.params_from_workload(w, precision=prec, batch=batch)) as s:
            s.set_kernel_timing(every)
            s.equilibrate(300, 0.004)  # launches of 256 and 44 steps
            out[every] = [s.get_state(), s.response_1d(w["A"], 3, 260, 0.004), s.response_2d(w["A"], P, w["A"], 5, 4, 3, 2, 0.004)]
            times[every] = {k: v for k, v in s.kernel_times().items() if v[0] > 0}
        print(f"[timing] every {every}: {times[every]}", flush=True)
        for a, b in zip(out[every], out[0]):
            assert np.array_equal(a, b)
    assert not times[0]
    for every in (1, 100):
        assert not any("pblock" in k or "qpass" in k for k in times[every])
        n, ms, by = times[every]["one_propagation"]
        assert ms > 0 and by == 2 * 8 * 4 * 20 * 18
    # of steps 0 .. 819 of the first two calls, in launches of 256, 44, 256, 4, 256 and
    # 4, and the at most 42 of the third, only those of 256 hold multiples of 100
    assert times[100]["one_propagation"][0] == 3
    assert times[1]["one_propagation"][0] > times[100]["one_propagation"][0]
    assert ("batch_one_propagation" in times[1]) == (batch > 1)
