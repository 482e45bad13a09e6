"""Whole states in and out through the ring of pinned chunks (states of more
than 32 MiB): every value comes back as it went in.  Coefficients of the Hermite
basis are copied as they are, so equality is exact.
"""
import threading

import numpy as np
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pk():
    import torch
    import paper_2509_25840_amd as pk
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    return pk


def solver(pk, Nq, Nh, K):
    return pk.Solver(pk.params_from_workload(wl.workload("two_mode_32", Nq=Nq, Np=Nh, K=K, basis="hermite")))


# 31.99 MiB (one copy), 32.2 MiB, a last chunk of a few values, many rounds of the ring
@pytest.mark.parametrize("Nq,Nh,K", [([32, 32], [13, 15], 5), ([32, 32], [14, 14], 5), ([48, 47], [11, 13], 5),
                                     ([32, 32], [32, 32], 6)])
def test_states_come_back_as_they_went_in(pk, Nq, Nh, K):
    with solver(pk, Nq, Nh, K) as s:
        for seed in (0, 1):
            W = np.random.default_rng(seed).normal(size=s.count)
            s.set_state(W)
            assert np.array_equal(s.get_state(), W)


def test_two_threads_with_a_solver_each(pk):
    bad = []

    def run(seed):
        with solver(pk, [32, 32], [24, 16], 5) as s:
            for k in range(3):
                W = np.random.default_rng(10 * seed + k).normal(size=s.count)
                s.set_state(W)
                if not np.array_equal(s.get_state(), W):
                    bad.append((seed, k))

    t = [threading.Thread(target=run, args=(i,)) for i in range(2)]
    for x in t:
        x.start()
    for x in t:
        x.join()
    assert not bad


def test_pinned_arrays_come_back_as_they_went_in(pk):
    """Arrays that the caller has pinned go over the link directly."""
    import torch
    with solver(pk, [32, 32], [24, 16], 5) as s:
        a = torch.empty(s.count, dtype=torch.float64, pin_memory=True).numpy()
        b = torch.empty(s.count, dtype=torch.float64, pin_memory=True).numpy()
        for seed in (0, 1):
            a[:] = np.random.default_rng(seed).normal(size=s.count)
            s.set_state(a)
            s._check(pk.lib().chfpe_get_state(s._ctx, pk._dptr(b)))
            assert np.array_equal(a, b) and np.array_equal(s.get_state(), a)
