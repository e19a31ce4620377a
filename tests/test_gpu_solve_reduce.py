"""The squared residuals of the entering state, added up inside the one-lane solve or by a launch
of their own: few rows with few and with many gather items per block of the solve, rows that do
not fill a block, and time bins of both kinds (the chain's two passes).

Bar: RMSE within 1e-5 of the fp64 oracle's, the half-sweeps' own."""
import numpy as np
import pytest

import oracle
import workload
from tests.test_gpu_bptf import check_chain
from tests.test_gpu_parity import dev, make_als

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,M,D", [(1, 5000, 10), (3, 200_000, 10), (40, 20_000, 20),
                                   (64, 3000, 4), (65, 30_000, 20), (300, 2000, 16)])
def test_entering_rmse_of_few_rows(N, M, D):
    deg = np.full(M, min(N, 3))
    deg[::11] = 0
    ptr, col, val = workload.make_custom(M, N, deg, seed=N + D)
    U0, V0 = workload.init_factors(M, N, D, seed=5 + N)
    want = oracle.rmse(ptr, col, val.astype(np.float64), U0, V0)
    for chunk in (24, 0):  # up to 9000 chunks per block, and the automatic split
        print(f"few rows N={N} M={M} D={D} chunk={chunk}", flush=True)
        tuning = dict(hub_threshold=48, chunk=chunk) if chunk else None
        with make_als(M, N, ptr, col, val, D, tuning) as als:
            for _ in range(2):  # the ticket is back at zero
                als.half_sweep("items", dev(U0), 0.065, dev(V0))
                assert abs(als.rmse_in() - want) <= 1e-5


@pytest.mark.parametrize("chunk", [8, 200])
def test_chain_of_few_bins(chunk):
    check_chain(400, 300, 8, 12, 2780 + chunk, tuning=dict(hub_threshold=256, chunk=chunk),
                empty_bins=(2,), deg=(10, 40), label="reduce")
