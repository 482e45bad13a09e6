"""chfpe_autotune keeps no request that it could not measure: where the kernels
of a step do not depend on a shape, the request stays automatic, in the context
and for later ones, and with a closure set afterwards."""
import pytest

import workloads as wl

pytestmark = pytest.mark.gpu

KEYS = ("request_pblock_blocks", "request_split", "request_qpass_positions", "request_pblock_run")
AUTO = (0, -1, 0, 0)


@pytest.fixture(scope="module")
def pk():
    import torch
    import paper_2509_25840_amd as pk
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    return pk


def requests(cfg):
    return tuple(cfg[k] for k in KEYS)


# q cubes by k_qcube with p blocks by k_pwave, k_pcube_s and (q width 1) k_pwave
@pytest.mark.parametrize("Nq,Np,K", [((8, 8, 8), (8, 8, 8), 1), ((12, 12, 12), (6, 7, 10), 0), ((8, 8, 8), (12, 6, 6), 1),
                                     ((16, 16, 16), (5, 5, 8), 0)], ids=str)
def test_three_modes_with_one_shape_stay_automatic(pk, Nq, Np, K):
    p = pk.params_from_workload(wl.workload("three_mode_24", Nq=list(Nq), Np=list(Np), K=K))
    with pk.Solver(p) as s:
        before = s.tile_config()
        print(f"[autotune] {Nq} {Np}: {requests(s.autotune(1))}", flush=True)
        assert s.tile_config() == before and requests(before) == AUTO
    with pk.Solver(p) as s:
        assert s.tile_config() == before


@pytest.mark.parametrize("N,K,batch", [(20, 3, 0), (32, 1, 5), (48, 0, 0)])
def test_one_mode_stays_automatic(pk, N, K, batch):
    p = pk.params_from_workload(wl.workload("one_mode_48", Nq=[N], Np=[N - 2], K=K), batch=batch)
    with pk.Solver(p) as s:
        print(f"[autotune] one mode {N}: {requests(s.autotune(1))}", flush=True)
        assert requests(s.tile_config()) == AUTO
