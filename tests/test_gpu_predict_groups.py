"""Predictions at the widths where the load width and the lanes per pair change (one, four or
eight lanes; float, float2 or float4 loads), with pair counts that leave a partial group and
block, pairs outside the tables, and the validation RMSE through the same kernels.

Tolerance: the derived per-pair bound of test_gpu_predict (the group's shorter chains and its
shuffle tree round each product at most D times, as one chain does)."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_predict import RMSE_TOL, dev_f, dev_i, pred_bound, small_ctx

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("D", [3, 5, 23, 25, 6, 10, 46, 50, 12, 20, 92, 96, 89, 126])
def test_group_edges(D):
    M, N = 301, 203
    rng = np.random.default_rng(D)
    U = rng.standard_normal((M, D), dtype=np.float32)
    V = rng.standard_normal((N, D), dtype=np.float32)
    print(f"predict groups D={D}", flush=True)
    with small_ctx(M, N, D) as als:
        for n in (1, 31, 33, 2051):
            users = rng.integers(0, M, n).astype(np.int32)
            items = rng.integers(0, N, n).astype(np.int32)
            want = oracle.predict(users, items, U, V)
            bound = pred_bound(U, V, users, items)
            bad_u, bad_i = users.copy(), items.copy()
            bad_u[::7], bad_i[3::7] = M, -1
            got = als.predict(dev_f(U), dev_f(V), dev_i(bad_u), dev_i(bad_i)).cpu().numpy()
            outside = (bad_u != users) | (bad_i != items)
            assert np.isnan(got[outside]).all()
            assert np.all(np.abs(got - want)[~outside] <= bound[~outside])
            r = rng.integers(0, 101, n).astype(np.uint8)
            als.set_holdout(users, items, r)
            rmse = als.holdout_rmse(dev_f(U), dev_f(V))
            assert abs(rmse - np.sqrt(np.mean((r - want) ** 2))) <= min(
                RMSE_TOL, np.sqrt(np.mean(bound ** 2)) + 1e-12)


def test_more_pairs_than_one_grid():
    """Eight lanes per pair: 2^32 threads are passed at 537M pairs, which repeat every 4096."""
    M, N, D, n = 301, 203, 50, 2 ** 29 + 8192
    rng = np.random.default_rng(D)
    U = rng.standard_normal((M, D), dtype=np.float32)
    V = rng.standard_normal((N, D), dtype=np.float32)
    users = dev_i(rng.integers(0, M, 4096).astype(np.int32)).repeat(n // 4096)
    items = dev_i(rng.integers(0, N, 4096).astype(np.int32)).repeat(n // 4096)
    print(f"predict D={D} pairs={n}", flush=True)
    with small_ctx(M, N, D) as als:
        got = als.predict(dev_f(U), dev_f(V), users, items).view(-1, 4096)
        assert torch.equal(got, got[:1].expand_as(got))
        one = als.predict(dev_f(U), dev_f(V), users[:4096].clone(), items[:4096].clone())
        assert torch.equal(one, got[-1])
