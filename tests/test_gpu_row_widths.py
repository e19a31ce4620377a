"""Rows, chunks and split rows of the fused row kernel at the widths without an augmented
column (their last tile has no padding block to carry the right-hand side), by method: each
has an instance of its own. Split rows come in several batches, whole rows beside them.

Bars: those of the methods' own tests (relative row error 1e-4 against the fp64 oracle)."""
import pytest

import workload
from tests import test_gpu_bayes, test_gpu_bptf, test_gpu_parity, test_gpu_split, test_gpu_tensor
from tests.test_gpu_split import test_gibbs_draw_of_split_rows as gibbs_draw

pytestmark = pytest.mark.gpu

WIDTHS = [48, 64, 80, 96, 112, 128]  # and 109, 125: the narrowest of the two widest


def split_tuning(D, slots=25):
    t = (D + 15) // 16
    return dict(hub_threshold=256, chunk=200,
                workspace_bytes=slots * 4 * (t * (t + 1) // 2 * 256 + 16 * t))


@pytest.mark.parametrize("D", [*WIDTHS, 109, 125])
def test_bptf_chain(D):
    # room for 25 slots: the bins of one parity take several batches; the second chain is whole
    test_gpu_bptf.check_chain(400, 300, 8, D, 1780 + D, tuning=split_tuning(D), empty_bins=(2,),
                              deg=(10, 40), label="split")
    test_gpu_bptf.check_chain(300, 200, 30, D, 1700 + D, label="whole")


@pytest.mark.parametrize("D", [*WIDTHS, 109, 125])
def test_gibbs(D):
    gibbs_draw(D)
    ptr, col, val = test_gpu_bayes.small_matrix(300, 200, 60 + D)
    test_gpu_bayes.check_gibbs_both_sides(300, 200, ptr, col, val, D, 0.05, 70 + D,
                                          label=f"whole{D}")


@pytest.mark.parametrize("D", WIDTHS)
def test_als(D):
    test_gpu_parity.test_widths_with_split_rows_and_batches(D)
    test_gpu_split.test_automatic_split(D)


@pytest.mark.parametrize("D", WIDTHS)
def test_weighted(D):
    test_gpu_parity.test_weighted_widths_with_split_rows(D)
    M, N, ptr, col, val, _, _ = test_gpu_split.edge_matrix(D)
    U0, V0 = workload.init_factors(M, N, D, seed=5 + D)
    test_gpu_parity.check_first_half_sweeps(
        M, N, ptr, col, val, D, 0.065, U0, V0, label=f"wauto{D}",
        weights=workload.rating_weights(col.size, seed=3 + D))


@pytest.mark.parametrize("D", WIDTHS)
def test_tensor(D):
    test_gpu_tensor.test_tensor_split_rows_and_batches(D)
    test_gpu_tensor.test_tensor_modes_match_oracle(D)
