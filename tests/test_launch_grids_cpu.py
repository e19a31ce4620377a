"""Launches of more threads than one HIP grid holds (2^32 - 1) go in slices that cover the work
once. No GPU: a stand-in for HIP's launch calls records what the library would launch."""
import os
import subprocess
import sys

import pytest

import paper_1108_2580_amd as pkg

HERE = os.path.dirname(os.path.abspath(__file__))
LIMIT = 2 ** 32

CALL = """
import ctypes, sys
ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
fn = getattr(ctypes.CDLL(sys.argv[2]), sys.argv[3])
types = dict(i=ctypes.c_int, l=ctypes.c_int64, f=ctypes.c_float, p=ctypes.c_void_p)
empty = ctypes.create_string_buffer(256)  # a zeroed RowPrior or Hadamard
args = [a.split(":") for a in sys.argv[4:]]
fn.argtypes = [types[t[0]] for t, _ in args]
sys.exit(fn(*[ctypes.addressof(empty) if v == "empty" else float(v) if t == "f" else int(v)
              for t, v in args]))
"""


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    lib = str(tmp_path_factory.mktemp("recorder") / "librecorder.so")
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", "-o", lib,
                           os.path.join(HERE, "launch_recorder.c")])

    def run(name, n_args, *args):
        r = subprocess.run([sys.executable, "-c", CALL, lib, pkg.LIB_PATH, name, *args],
                           capture_output=True, text=True,
                           env=dict(os.environ, RECORDED_ARGS=str(n_args)))
        assert r.returncode == 0, r.stderr
        out = [[int(w) for w in line.split()] for line in r.stdout.splitlines()]
        assert all(threads * blocks < LIMIT for threads, blocks, *_ in out)
        return out

    return run


# rows of two chunks each; at D = 100 a split row's sum takes 28 blocks of 256 threads
@pytest.mark.parametrize("D,DP,parts", [(100, 112, 28), (128, 128, 37), (33, 48, 6)])
@pytest.mark.parametrize("n", [1000, 600_000, 5_600_000])
def test_sums_of_split_rows(launches, D, DP, parts, n):
    out = launches("_ZN3als16launch_sum_slotsEiiPKNS_7RowTaskElfPfRKNS_8RowPriorEP12ihipStream_t", 1,
                   f"i:{DP}", f"i:{D}", "p:4096", f"l:{n}", "f:0.1", "p:8192", "p:empty", "p:0")
    assert len(out) == -(-n // ((LIMIT - 1) // 256 // parts))
    at = 4096  # RowTask records of 24 bytes
    for threads, blocks, rows, *_ in out:
        assert threads == 256 and blocks % parts == 0 and rows == at
        at += blocks // parts * 24
    assert at == 4096 + 24 * n


# one, four and eight lanes per pair, with float, float2 and float4 loads
@pytest.mark.parametrize("D,lanes", [(3, 1), (10, 4), (50, 8), (33, 8), (20, 4), (100, 8)])
@pytest.mark.parametrize("n", [1000, 600_000_000, 5_000_000_000])
@pytest.mark.parametrize("sse", [False, True])
def test_predictions(launches, D, lanes, n, sse):
    pred, r, blocks_out = (0, 1 << 36, 1 << 37) if sse else (1 << 35, 0, 0)
    out = launches("_ZN3als14launch_predictEPKfS1_llilPKiS3_PKhPfPdP12ihipStream_t", 11,
                   "p:4096", "p:8192", "l:1000", "l:900", f"i:{D}", f"l:{n}", f"p:{1 << 33}",
                   f"p:{1 << 34}", f"p:{r}", f"p:{pred}", f"p:{blocks_out}", "p:0")
    first = block = 0
    for threads, blocks, U, V, M, N, _, k, users, items, rk, pk, bk in out:
        assert threads == 256 and blocks == -(-k * lanes // 256)
        assert (users, items) == ((1 << 33) + 4 * first, (1 << 34) + 4 * first)
        assert (rk, pk) == ((r + first, 0) if sse else (0, pred + 4 * first))
        assert bk == (blocks_out + 8 * block if sse else 0)
        first, block = first + k, block + blocks
    assert first == n and block == -(-n * lanes // 256)


ITEMS = [1000, 70_000_000, 200_000_000]


def check_slices(out, n, at, *strides):
    """Every launch starts where the one before ended, in each of the arrays at `at`."""
    first = 0
    for threads, blocks, *args in out:
        assert threads == 64
        for (k, base), stride in zip(at, strides):
            assert args[k] == base + stride * first
        first += blocks
    assert first == n and len(out) == -(-n // ((LIMIT - 1) // 64))


@pytest.mark.parametrize("D,DP", [(33, 48), (100, 112), (128, 128)])
@pytest.mark.parametrize("n", ITEMS)
@pytest.mark.parametrize("split_rows", [False, True])
def test_rows(launches, D, DP, n, split_rows):
    items, rows = (0, 1 << 33) if split_rows else (1 << 33, 0)
    out = launches("_ZN3als11launch_rowsEiPKNS_8WorkItemEPKNS_7RowTaskElPKiPKhPKfSB_lPfifSC_PdPiSD"
                   "_SD_RKNS_8RowPriorERKNS_8HadamardEP12ihipStream_t", 13,
                   f"i:{DP}", f"p:{items}", f"p:{rows}", f"l:{n}", "p:64", "p:64", "p:0", "p:64",
                   "l:1000", "p:64", f"i:{D}", "f:0.1", "p:64", f"p:{1 << 35}", "p:64", "p:0",
                   "p:0", "p:empty", "p:empty", "p:0")
    check_slices(out, n, [(split_rows, 1 << 33), (11, 1 << 35)], 24, 8)


@pytest.mark.parametrize("D", [10, 20])
@pytest.mark.parametrize("n", ITEMS)
def test_narrow_grams(launches, D, n):
    out = launches("_ZN3als14launch_gram_neEiPKNS_8WorkItemElPKiPKhPKfS8_lS8_PfS9_PdRKNS_8Hadamard"
                   "EP12ihipStream_t", 11,
                   f"i:{D}", f"p:{1 << 33}", f"l:{n}", "p:64", "p:64", "p:0", "p:64", "l:1000",
                   "p:64", "p:64", "p:64", f"p:{1 << 35}", "p:empty", "p:0")
    check_slices(out, n, [(0, 1 << 33), (10, 1 << 35)], 24, 8)


@pytest.mark.parametrize("DP", [16, 48])
@pytest.mark.parametrize("n", ITEMS)
def test_residuals(launches, DP, n):
    out = launches("_ZN3als12launch_residEiPKNS_8WorkItemElPKiPKhPKflS8_iPdRKNS_8HadamardEP12ihip"
                   "Stream_t", 8, f"i:{DP}", f"p:{1 << 33}", f"l:{n}", "p:64", "p:64", "p:64",
                   "l:1000", "p:64", f"i:{DP}", f"p:{1 << 35}", "p:empty", "p:0")
    check_slices(out, n, [(0, 1 << 33), (7, 1 << 35)], 24, 8)


@pytest.mark.parametrize("D", [10, 20])
@pytest.mark.parametrize("n", [1000, 20_000_000])
def test_sums_of_split_records(launches, D, n):
    out = launches("_ZN3als17launch_solve_laneEiPKNS_7RowTaskElllPKfPffS5_PiRKNS_8RowPriorERKNS_11"
                   "SolveReduceEP12ihipStream_t", 4, f"i:{D}", f"p:{1 << 33}", f"l:{n}", f"l:{n}",
                   "l:7", "p:64", "p:64", "f:0.1", "p:64", "p:64", "p:empty", "p:empty", "p:0")
    first = 0
    for threads, blocks, rows, base, *_ in out[:-1]:
        assert threads == 256 and rows == (1 << 33) + 24 * first and base == 7 + first
        first += blocks
    assert first == n and out[-1][:2] == [64, -(-n // 64)]
