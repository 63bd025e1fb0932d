"""The storage builder's sort by buckets against the CPU checker, bit for bit, at the sizes where its choices change: one bucket and
several, one partition and two, keys of 32 bits, cut at multiples of 2^32, of 64 bits; rows that fill buckets by themselves,
columns that crowd, a sample that misleads (the build is done again by the stable sorts), entries given twice."""
import numpy as np
import pytest

import oracle
import paper_2202_04305_amd as sp
from gen import prng
from gpu_util import say, gpu_pack, assert_storage_equal

pytestmark = pytest.mark.gpu
SEED = 7250311
CSR, CSC, DCSR, CDR = ((0, 1), (0, 1)), ((0, 1), (1, 0)), ((1, 1), (0, 1)), ((1, 0), (0, 1))
TWO = 2048 * 512                       # up to here one partition


def distinct(shape, nnz, seed):
    total = int(np.prod([int(s) for s in shape], dtype=object))
    lin = np.unique(prng.below(seed, 1, int(nnz * 1.2) + 16, total))
    while lin.size < nnz:
        lin = np.unique(np.concatenate([lin, prng.below(seed + lin.size, 1, nnz, total)]))
    return shuffled(lin, nnz, shape, seed)


def shuffled(lin, nnz, shape, seed):
    lin = lin[prng.permutation(seed, 2, lin.size)][:nnz]
    out = []
    for s in reversed(shape[1:]):
        out.append((lin % s).astype(np.int64))
        lin = lin // s
    return [lin.astype(np.int64)] + out[::-1]


def check(fmt, shape, coords, dtype=np.float64, widths=(32, 32)):
    n = len(coords[0])
    say("case", fmt, "shape", shape, "entries", n, dtype.__name__, widths)
    v = prng.uniform_pm1(SEED + n, 3, n, dtype)
    ref = oracle.pack(*fmt, shape, coords, v, *widths)
    assert_storage_equal(gpu_pack(*fmt, shape, coords, v, *widths), ref)


@pytest.mark.parametrize("fmt", [CSR, CSC, DCSR, CDR])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_sizes_where_the_number_of_buckets_changes(fmt, dtype):
    for n in (1, 2, 255, 256, 2047, 2048, 2049, 4095, 4096, 4097, 12289, 100003):
        shape = (300, 401) if n <= 12289 else (3001, 2003)
        check(fmt, shape, distinct(shape, n, SEED + n), dtype, (32, 64) if n % 2 else (64, 32))


@pytest.mark.parametrize("shape", [(65537, 65521), (1 << 16, 1 << 16), (1 << 20, 1 << 20), ((1 << 22) + 3, (1 << 20) + 7), (1 << 23, 1 << 23), (1 << 24, 1 << 24)])
def test_keys_around_and_beyond_32_bits(shape):
    """Multiples of 2^32 inside the key range: none, none, 255, 1024, more than are split at (64-bit keys), and 48 key bits."""
    for n in (1500, 70001, 700001):
        coords = distinct(shape, n, SEED + 5 * n)
        check(CSR if n > 60000 or shape[0] < 1 << 21 else DCSR, shape, coords)
        if n == 70001:
            check(DCSR, shape, coords, np.float32)


@pytest.mark.parametrize("n", [TWO, TWO + 1, 2 * TWO + 3])
@pytest.mark.parametrize("shape", [(70001, 65521), (1 << 18, 1 << 21), (1 << 23, 1 << 22)])
def test_one_partition_and_two(n, shape):
    check(CSR, shape, distinct(shape, n, SEED + n))


def test_ranks():
    for fmt, shape, n in [(((1,), (0,)), (1 << 22,), 50001), (((0, 1, 1), (0, 2, 1)), (400, 500, 601), 60001), (((0, 0, 1), (2, 0, 1)), (40, 50, 60), 30001),
                          (((1, 1, 1), (0, 1, 2)), (1200, 900, 2900), TWO + 77), (((1, 0, 1, 1), (0, 1, 3, 2)), (30, 5, 70, 80), 40001),
                          (((1,) * 5, (4, 3, 2, 1, 0)), (30, 31, 32, 33, 34), 200003)]:
        check(fmt, shape, distinct(shape, n, SEED + n))


@pytest.mark.parametrize("n_rest", [60000, TWO])
def test_rows_that_fill_buckets_and_columns_that_crowd(n_rest):
    m, n = 1 << 17, 1 << 20
    lin = [np.arange(20000, dtype=np.int64) * 37 + 11 * n, np.arange(9000, dtype=np.int64) + 4000 * n + 777,          # a long row, a full stretch of one
           np.arange(100000, dtype=np.int64) + (m - 1) * n]
    r = np.arange(1000, dtype=np.int64)
    lin += [(20000 + r)[:, None].repeat(128, 1).ravel() * n + (r[:, None] * 3 + np.arange(128)).ravel(),               # a band
            ((50000 + r)[:, None] * n + (r[:, None] // 64 * 64 + np.arange(64))).ravel()]                             # blocks
    lin.append(prng.below(SEED, 9, n_rest, m * n))
    lin = np.unique(np.concatenate(lin))
    coords = shuffled(lin, lin.size, (m, n), SEED)
    for fmt in (CSR, DCSR):
        check(fmt, (m, n), coords)
    check(CSC, (n, m), coords[::-1])


def sampled_positions(n):
    """Where the builder looks: one entry per stretch of n / S, at a scrambled place in it."""
    if n > TWO:
        first = min(max(n // 128, 16384), 131072)
        Q, share = max(min(-(-n // first), 512), -(-n // (2 * 131072))), 32
    else:
        Q, share = -(-n // 2048), 48
    S = min(-(-share * Q // 1024) * 1024, 32768)
    i = np.arange(S, dtype=np.uint64)
    x = i ^ (i >> np.uint64(16))
    x = (x * np.uint64(0x7feb352d)) & np.uint64(0xffffffff)
    x ^= x >> np.uint64(15)
    x = (x * np.uint64(0x846ca68b)) & np.uint64(0xffffffff)
    x ^= x >> np.uint64(16)
    return np.minimum(((i.astype(np.float64) + x.astype(np.float64) * 2.0 ** -32) * (float(n) / float(S))).astype(np.int64), n - 1)


@pytest.mark.parametrize("fmt", [CSR, DCSR])
@pytest.mark.parametrize("n", [200000, TWO + 100000])
def test_a_sample_that_misleads(fmt, n):
    """The sampled entries are spread over the matrix, all others lie in one corner: a bucket gets more than it has room for."""
    m = 1 << 16
    at = np.unique(sampled_positions(n))
    corner = prng.permutation(SEED, 4, 4 * n)[: n - at.size]
    side = int(np.ceil(np.sqrt(4 * n)))
    rows, cols = np.empty(n, np.int64), np.empty(n, np.int64)
    rest = np.ones(n, bool)
    rest[at] = False
    rows[rest], cols[rest] = corner // side, corner % side
    spread = np.unique(prng.below(SEED, 5, 2 * at.size, m * m))
    spread = spread[spread // m > side]
    spread = spread[prng.permutation(SEED, 6, spread.size)][: at.size]
    assert spread.size == at.size
    rows[at], cols[at] = spread // m, spread % m
    check(fmt, (m, m), [rows, cols])


@pytest.mark.parametrize("fmt", [CSR, DCSR])
@pytest.mark.parametrize("n", [3000, 50000, TWO + 1])
def test_entries_given_twice_and_coordinates_out_of_range(fmt, n):
    shape = (5000, 4000)
    coords = distinct(shape, n, SEED + 3)
    v = np.ones(n)
    for change, code in [("one twice", 7), ("all the same", 7), ("out of range", 6)]:
        c = [x.copy() for x in coords]
        if change == "one twice":
            c[0][n - 1], c[1][n - 1] = c[0][n // 3], c[1][n // 3]
        elif change == "all the same":
            c[0][:], c[1][:] = 17, 23
        else:
            c[1][n // 2] = shape[1]
        say("case", fmt, n, change)
        with pytest.raises(sp.SpError) as e:
            gpu_pack(*fmt, shape, c, v, 32, 32)
        assert e.value.code == code


@pytest.mark.parametrize("fmt", [CSR, CSC, DCSR])
def test_input_that_is_sorted_already(fmt):
    """A bucket that gets 256 entries or more of a tile (1024 entries; 12288 from 1,572,864 entries on) gets them in a mixed order: every
    place exactly once, whatever the number is."""
    for n in (255, 256, 257, 511, 512, 767, 1023, 1024, 1025, 2048 + 255, 2048 + 256, 100003, TWO + 1, 1572863, 1572864, 1600001):
        shape = (300, 401) if n < 4096 else (40009, 30011)
        coords = distinct(shape, n, SEED + 7 * n)
        key = coords[0] * shape[1] + coords[1] if fmt != CSC else coords[1] * shape[0] + coords[0]
        order = np.argsort(key)
        check(fmt, shape, [c[order] for c in coords], np.float64 if n % 2 else np.float32)
        if n > 100000:
            check(fmt, shape, [c[order[::-1]] for c in coords])


def test_bands_and_blocks_that_are_sorted_already():
    r = np.arange(1600000 // 64 + 1, dtype=np.int64)
    m = r.size
    band = [r.repeat(64), (r[:, None] + np.arange(64)).ravel() % m]
    order = np.argsort(band[0] * m + band[1])
    for fmt in (CSR, DCSR, CSC):
        check(fmt, (m, m), [c[order] for c in band])
    b = np.arange(1600000 // 4096 + 1, dtype=np.int64)
    i, j = np.divmod(np.arange(4096), 64)
    rows, cols = (b[:, None] * 64 + i).ravel(), (b[:, None] * 64 + j).ravel()
    order = np.argsort(rows * (64 * b.size) + cols)
    for fmt in (CSR, CSC):
        check(fmt, (64 * b.size, 64 * b.size), [rows[order], cols[order]], np.float32)


@pytest.mark.parametrize("widths", [(32, 32), (64, 64)])
@pytest.mark.parametrize("n,columns", [(3000, 50), (40000, 1 << 20), (70000, 1 << 31), (TWO + 5, 1 << 26)])
def test_many_rows_that_begin_in_one_bucket(n, columns, widths):
    """Rows of a bucket beyond 2048 are counted 4096 at a time: entries only before, only behind and only at the edges of such stretches, and
    anywhere in them; the last rows empty."""
    m = min(4 * n, 1 << 20) - 5
    for where in ("anywhere", "first rows", "last rows", "edges", "two ends"):
        rows = prng.below(SEED + n, 11, 2 * n, m)
        if where == "first rows":
            rows = rows % max(n // 30, 60)
        elif where == "last rows":
            rows = m - 1 - rows % max(n // 30, 60)
        elif where == "edges":
            rows = np.minimum(rows // 2048 * 2048 + rows % 3, m - 1)
        elif where == "two ends":
            rows = np.where(rows % 2 == 0, rows % 500, m - 1 - rows % 500)
        lin = np.unique(rows * columns + prng.below(SEED + n, 12, 2 * n, columns))
        check(CSR, (m, columns), shuffled(lin, n, (m, columns), SEED), np.float32, widths if columns < 1 << 31 else (widths[0], 64))
