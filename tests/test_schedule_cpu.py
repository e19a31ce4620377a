"""The order in which a half-sweep's gather items start, on the host alone."""
import ctypes

import numpy as np
import pytest

import paper_1108_2580_amd as pkg

ITEM = np.dtype([("start", "<i8"), ("slot", "<i8"), ("len", "<i4"), ("row", "<i4")])


def library(name, *argtypes):
    fn = getattr(ctypes.CDLL(pkg.LIB_PATH), name)
    fn.restype = ctypes.c_int64
    fn.argtypes = argtypes
    return fn


def order_items(items, ptr, n_chunks):
    fn = library("_ZN3als11order_itemsEPNS_8WorkItemEPKlll", ctypes.c_void_p, ctypes.c_void_p,
                 ctypes.c_int64, ctypes.c_int64)
    out = items.copy()
    return fn(out.ctypes.data, ptr.ctypes.data, n_chunks, len(out)), out


@pytest.mark.parametrize("chunk_lens,row_lens", [
    ([], [9, 5, 1]), ([4, 4, 2], []), ([4, 4, 2], [8, 6, 5, 4, 3, 1]), ([4, 3], [4, 2]),
    ([256] * 9, [500, 257, 256, 0]), ([1], [3, 2, 1]), ([4, 4], [8, 5, 4, 4, 4, 3]),
    ([4, 4], [8, 4]), ([4, 4], [8, 4, 2]), ([4], [])])
def test_largest_work_starts_first(chunk_lens, row_lens):
    n = len(chunk_lens)
    items = np.zeros(n + len(row_lens), ITEM)
    items["len"] = chunk_lens + row_lens
    items["slot"] = list(range(n)) + [~k for k in range(len(row_lens))]
    items["row"] = np.arange(len(items))
    items["start"] = np.arange(len(items)) * 1000
    lead, out = order_items(items, items["start"].astype(np.int64), n)
    assert sorted(map(tuple, out)) == sorted(map(tuple, items))
    whole = out["slot"] < 0
    longest = max(chunk_lens, default=0)
    # no whole row longer than the chunks is left behind them unless shorter ones hold more than
    # a quarter of the ratings; the rows keep their order
    behind = sum(k for k in row_lens if k <= longest)
    few = n > 0 and 4 * behind <= sum(chunk_lens) + sum(row_lens)
    assert lead == (sum(k > longest for k in row_lens) if few else 0)
    assert whole[:lead].all() and not whole[lead:lead + n].any() and whole[lead + n:].all()
    assert out["len"][whole].tolist() == row_lens


@pytest.mark.parametrize("degrees,chunk", [([700], 256), ([3000, 2100, 600, 513], 256),
                                           ([9001, 8193, 8193], 4096), ([1153] * 7, 576)])
def test_chunks_are_even_and_go_by_depth(degrees, chunk):
    even = library("_ZN3als10even_chunkEll", ctypes.c_int64, ctypes.c_int64)
    ptr = np.concatenate([[0], np.cumsum(degrees)]).astype(np.int64)
    items = []
    for row, d in enumerate(degrees):
        c = even(d, chunk)
        # as many chunks as before, none longer, each but the last of the same whole groups
        assert c % 64 == 0 and c <= chunk and -(-d // c) == -(-d // chunk)
        assert -(-d // c) * 64 > -(-d // c) * c - d  # the last is short by less than 64 a chunk
        for q in range(-(-d // c)):
            items.append((ptr[row] + q * c, len(items), min(c, d - q * c), row))
    items = np.array(items, ITEM)
    lead, out = order_items(items, ptr, len(items))
    assert lead == 0 and sorted(map(tuple, out)) == sorted(map(tuple, items))
    depth = out["start"] - ptr[out["row"]]
    assert (np.diff(depth) >= 0).all()


@pytest.mark.parametrize("rows,residuals,fused", [
    (1, 512, True), (50, 513, False), (50, 10_000, False), (64, 512, True), (65, 1024, True),
    (65, 1025, False), (4096, 64 * 512, True), (4096, 64 * 512 + 1, False), (4097, 4097, False)])
def test_the_solve_adds_up_bounded_runs_of_residuals(rows, residuals, fused):
    fn = library("_ZN3als13solve_reducesEll", ctypes.c_int64, ctypes.c_int64)
    fn.restype = ctypes.c_bool
    assert fn(rows, residuals) == fused


@pytest.mark.parametrize("n", [*range(1, 41), 1000, 4099])
def test_interleaved_runs(n):
    """Each position once, and the members on one XCD are consecutive and in order."""
    fn = library("_ZN3als11interleavedEll", ctypes.c_int64, ctypes.c_int64)
    at = np.array([fn(r, n) for r in range(n)])
    assert sorted(at) == list(range(n))
    for xcd in range(8):
        members = [r for r in range(n) if at[r] % 8 == xcd]
        assert (np.diff(members) == 1).all() and (np.diff(at[members]) == 8).all()
