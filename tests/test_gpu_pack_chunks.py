"""The finishing pass of the storage builder's sort at the edges of its paths, against the CPU checker, bit for bit: chunks that
just fit a block, that just do not, that just fit the large block, and that just do not; keys crowded into one interval of the
cut by value; distances inside a chunk that need 32 bits and more."""
import numpy as np
import pytest

import oracle
import paper_2202_04305_amd as sp
from gen import prng
from gpu_util import say, gpu_pack, assert_storage_equal

pytestmark = pytest.mark.gpu
SEED = 20220305


@pytest.fixture
def msd_first():
    sp.sp_pack_sort_mode(2)
    yield
    sp.sp_pack_sort_mode(0)


def check(shape, coords, dtype, what):
    p = prng.permutation(SEED, 5, coords[0].size)
    coords = [np.ascontiguousarray(c[p]) for c in coords]
    v = prng.uniform_pm1(SEED, 6, p.size, dtype)
    say("case", what, "shape", shape, "entries", p.size)
    lt, order = (1,) * len(shape), tuple(range(len(shape)))
    assert_storage_equal(gpu_pack(lt, order, shape, coords, v, 64, 64), oracle.pack(lt, order, shape, coords, v, 64, 64))


def distinct(stream, count, bound):
    c = np.unique(prng.below(SEED, stream, count + count // 4 + 64, bound))
    return c[prng.permutation(SEED, stream + 1, c.size)][:count].astype(np.int64)


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("length", [2047, 2048, 2049, 8191, 8192, 8193])
@pytest.mark.parametrize("spread", ["even", "crowded"])
def test_one_row_per_chunk(msd_first, dtype, length, spread):
    """Rows far apart, so that each is a chunk; crowded: all columns but one side by side at the far end of the row."""
    m, n = 1 << 20, 1 << 20
    rows = [3, m // 2, m - 1]
    cols = [distinct(10 + 2 * i, length, n) if spread == "even" else np.append(np.arange(n - length + 1, n), 7) for i in range(len(rows))]
    check((m, n), [np.repeat(np.array(rows, dtype=np.int64), length), np.concatenate(cols)], dtype, "%s rows of %d" % (spread, length))


@pytest.mark.parametrize("bits", [47, 48, 49, 62])
def test_distances_around_32_bits_and_runs_of_neighbours(msd_first, bits):
    """Two passes take the top 16 bits of the key, so chunks span bits - 16 and a little more; groups of 2 to 60 neighbouring keys
    share an interval however fine the cut (one interval holds up to 48 keys before the chunk is sorted digit by digit)."""
    n = 1 << (bits // 2)
    m = 1 << (bits - bits // 2)
    base_r, base_c = prng.below(SEED, 20, 3000, m), prng.below(SEED, 21, 3000, n - 64)
    runs = 2 + prng.below(SEED, 22, 3000, 59)
    r = np.repeat(base_r, runs)
    c = np.repeat(base_c, runs) + (np.arange(r.size) - np.repeat(np.cumsum(runs) - runs, runs))
    lin = np.unique(r.astype(np.int64) * n + c)
    check((m, n), [lin // n, lin % n], np.float64, "key of %d bits" % bits)


@pytest.mark.parametrize("per_row,col_bits", [(1500, 24), (3000, 24), (3000, 26), (5200, 26)])
def test_every_sub_bucket_larger_than_a_chunk(per_row, col_bits):
    """The sort as the builder chooses it, a million entries and more in few of the 65536 sub-buckets: each alone in its chunk, in
    the finishing kernel, the larger one, or left to the other sort."""
    rows = (1 << 20) // per_row + 20
    r = np.repeat(np.arange(rows, dtype=np.int64) * 3, per_row)
    c = prng.below(SEED, 30, r.size, 1 << col_bits).astype(np.int64)
    lin = np.unique((r << col_bits) + c)
    check((1 << 16, 1 << col_bits), [lin >> col_bits, lin & ((1 << col_bits) - 1)], np.float64, "rows of %d, %d bits" % (per_row, 16 + col_bits))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_every_chunk_crowded(msd_first, dtype):
    """A band of 64 columns: nearly every chunk spans several rows and has each row's columns in one interval; more such chunks than
    the kernel that sorts them digit by digit has blocks, some rows long enough for the large block."""
    m, n, per = 22000, 1 << 20, 64
    r = np.repeat(np.arange(m, dtype=np.int64), per)
    c = np.repeat((np.arange(m, dtype=np.int64) * 47) % (n - 4096), per) + np.tile(np.arange(per, dtype=np.int64), m)
    extra = np.arange(3000, dtype=np.int64)
    rows = np.concatenate([r, np.full(3000, 5000), np.full(3000, 15000)])
    cols = np.concatenate([c, n - 3100 + extra, n - 3100 + extra])
    check((m, n), [rows, cols], dtype, "band of 64 columns")
