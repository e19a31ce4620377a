"""The automatic split of long rows (no tuning given): rows at the edges of its threshold and
chunks, slot counts with every remainder of the four summing waves, ALS and Gibbs draws with
and without the augmented column; a workspace too small for the fine split, which falls back
to the coarse one instead of being refused; and chunks cut and ordered by windows of a large
fixed table.

Bar: the half-sweep's own, relative row error 1e-4 against the fp64 oracle."""
import numpy as np
import pytest

import oracle
import workload
from tests.test_gpu_parity import check_first_half_sweeps, dev, rel_rows, ROW_TOL

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def edge_matrix(D):
    """Users around multiples of the finest split's chunk (256 ratings up to D = 20, 512
    above; rows of over two chunks split), among ordinary ones."""
    c = 256 if D <= 20 else 512
    N = 9 * c
    deg = [2 * c - 1, 2 * c, 2 * c + 1, 3 * c - 1, 3 * c, 3 * c + 1, 4 * c, 4 * c + 1, 5 * c + 7,
           8 * c, 8 * c + 64, 0, 1, 3 * c + 63] + [c // 4] * 50
    ptr, col, val = workload.make_custom(len(deg), N, np.array(deg), seed=7 + D)
    return len(deg), N, ptr, col, val, c, np.array(deg)


@pytest.mark.parametrize("D", [1, 10, 16, 17, 20, 21, 32, 33, 48, 64, 100, 112, 128])
def test_automatic_split(D):
    from paper_1108_2580_amd import ALS

    M, N, ptr, col, val, c, deg = edge_matrix(D)
    U0, V0 = workload.init_factors(M, N, D, seed=5 + D)
    with ALS(M, N, ptr, col, val, D) as als:
        st = als.plan_stats("users")
    assert st["split_rows"] == int((deg > 2 * c).sum())
    assert st["chunks"] == int((-(-deg[deg > 2 * c] // c)).sum())
    check_first_half_sweeps(M, N, ptr, col, val, D, 0.065, U0, V0, label=f"auto{D}")
    # two slots fit: the plan takes the coarse split, under which no row here is split
    with ALS(M, N, ptr, col, val, D, tuning=dict(workspace_bytes=2 * st["slot_bytes"])) as als:
        assert als.plan_stats("users")["split_rows"] == 0
    check_first_half_sweeps(M, N, ptr, col, val, D, 0.065, U0, V0, label=f"small{D}",
                            tuning=dict(workspace_bytes=2 * st["slot_bytes"]))


@pytest.mark.parametrize("D", [20, 33, 48, 100, 128])
def test_gibbs_draw_of_split_rows(D):
    from paper_1108_2580_amd import ALS

    M, N, ptr, col, val, c, deg = edge_matrix(D)
    U0, V0 = workload.init_factors(M, N, D, seed=9 + D)
    rng = np.random.default_rng(D)
    A = rng.normal(size=(D, D))
    Lam, mu = A @ A.T / D + np.eye(D), rng.normal(size=D)
    z = rng.standard_normal((M, D), dtype=np.float32)
    d64 = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    alpha = 0.0625
    print(f"gibbs split D={D}", flush=True)
    with ALS(M, N, ptr, col, val, D) as als:
        assert als.plan_stats("users")["split_rows"] > 0
        out = dev(U0)
        als.gibbs_half_sweep("users", dev(V0), alpha, d64(Lam), d64(mu), dev(z), out)
        got = out.cpu().numpy()
    want, _ = oracle.gibbs_rows(ptr, col, val.astype(np.float64), V0, alpha, Lam, mu, z, U0)
    assert rel_rows(got, want).max() <= ROW_TOL


def long_items(D, M, N=60):
    """Items of hundreds to hundreds of thousands of ratings on a users' table of over 24 MB
    (only items of under 1800 ratings get shorter chunks by it than without)."""
    deg = np.full(M, 3)
    deg[::50] = 0
    deg[7] = N
    return workload.make_custom(M, N, deg, seed=11 + D,
                                item_weights=np.r_[np.arange(1, N) ** -2.5, 0.0])


def windowed_chunks(d, D, M):
    """The chunks that windows of 4 MB of the table cut rows of d > 512 ratings into."""
    windows = M * (16 if D <= 16 else 32) * 4 >> 22
    assert windows >= 6
    d = d[d > 512]
    chunk = np.minimum(256, np.maximum(128, -(-(d // windows) // 64) * 64))
    return int((-(-d // chunk)).sum())


@pytest.mark.parametrize("D,M", [(10, 450_000), (20, 250_000)])
def test_windowed_chunks(D, M):
    """The items' fixed table is over 24 MB: the long items' chunks follow windows of it, the
    users' side keeps the plain split."""
    from paper_1108_2580_amd import ALS

    N = 60
    ptr, col, val = long_items(D, M)
    U0, V0 = workload.init_factors(M, N, D, seed=13 + D)
    with ALS(M, N, ptr, col, val, D) as als:
        st, whole = als.plan_stats("items"), als.plan_stats("users")
    d = np.bincount(col, minlength=N)
    assert whole["split_rows"] == 0 and st["split_rows"] == int((d > 512).sum()) > 10
    assert st["chunks"] == windowed_chunks(d, D, M) > int((-(-d // 256))[d > 512].sum())
    check_first_half_sweeps(M, N, ptr, col, val, D, 0.065, U0, V0, label=f"windows{D}")


@pytest.mark.parametrize("D,M", [(10, 450_000), (20, 250_000)])
@pytest.mark.parametrize("method", ["weighted", "gibbs", "tensor", "bptf"])
def test_windowed_chunks_of_other_methods(method, D, M):
    """Weights, second indices, the prior image and the time plan, whose indices repeat within a
    row, beside windowed chunks (a plan with windows is one batch)."""
    from tests import test_gpu_bayes, test_gpu_bptf, test_gpu_tensor

    N, bins = 60, 12
    ptr, col, val = long_items(D, M)
    print(f"windows {method} D={D}", flush=True)
    if method == "weighted":
        U0, V0 = workload.init_factors(M, N, D, seed=13 + D)
        check_first_half_sweeps(M, N, ptr, col, val, D, 0.065, U0, V0, label=f"windows{D}",
                                weights=workload.rating_weights(col.size, seed=17 + D))
    elif method == "gibbs":
        test_gpu_bayes.check_gibbs_both_sides(M, N, ptr, col, val, D, 0.05, 19 + D,
                                              label=f"windows{D}")
    elif method == "tensor":
        rng = np.random.default_rng(23 + D)
        t = rng.integers(0, bins - 1, size=col.size).astype(np.int32)
        U, V, T = (rng.normal(m, s, size=(n, D)).astype(np.float32)
                   for m, s, n in ((0, 0.5, M), (0, 0.5, N), (1, 0.3, bins)))
        test_gpu_tensor.check_modes(M, N, bins, ptr, col, val, t, U, V, T, D, 0.065,
                                    label=f"windows{D}")
    else:
        test_gpu_bptf.check_chain(M, N, bins, D, 29 + D, deg=(2, 4), empty_bins=(2,),
                                  label=f"windows{D}")
