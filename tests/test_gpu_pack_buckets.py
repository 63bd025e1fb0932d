"""The storage builder's sort by buckets against the CPU checker, bit for bit, at the sizes where its choices change: one bucket and
several, one partition and two, keys of 32 bits, cut at multiples of 2^32, of 64 bits; rows that fill buckets by themselves,
columns that crowd, buckets that overflow (the build is done again by the stable sorts), entries given twice."""
import ctypes

import numpy as np
import pytest

import oracle
import paper_2202_04305_amd as sp
from paper_2202_04305_amd import binding
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


@pytest.mark.parametrize("columns", [1 << 20, 1 << 31, 1 << 44])
def test_keys_that_crowd_at_every_scale(columns):
    """Columns spread evenly over their logarithm: cutting an interval again leaves one part with most of its keys, and the merge sort has
    them.  Runs of one key, of an odd and an even number, and of 17; up to 4096 entries in one bucket, more in several."""
    for n in (150, 255, 256, 257, 300, 511, 513, 1000, 2047, 2304, 3839, 3841, 4095, 4096, 9000, 70000, TWO + 9):
        c = np.exp2(prng.uniform_pm1(SEED + n, 17, 3 * n, np.float64) * 0.5 * np.log2(columns) + 0.5 * np.log2(columns)).astype(np.int64) % columns
        m = 1 if n < 300 else min(n // 300 + 1, 1 << (48 - int(columns).bit_length()))
        lin = np.unique((prng.below(SEED + n, 18, 3 * n, m) ** 2 // m) * columns + c)
        n = min(n, lin.size)
        check(DCSR if n % 2 else CSR, (m, columns), shuffled(lin, n, (m, columns), SEED), np.float64 if n % 3 else np.float32, (32, 32) if columns < 1 << 31 else (32, 64))


def sampled_positions(n):
    """Where the builder looks: one entry per stretch of n / S, at a scrambled place in it (the mixer is Chris Wellons' lowbias32)."""
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


class overflows:
    """The builds inside that were done again, by where a bucket overflowed: [in the first partition, later]."""

    def __enter__(self):
        self.counters = (ctypes.c_int * 2).in_dll(binding.load_library(), "g_pack_overflows")
        self.before = list(self.counters)
        return self

    def __exit__(self, *exc):
        self.counts = [a - b for a, b in zip(self.counters, self.before)]


def unravel(lin, shape):
    out = []
    for s in reversed(shape[1:]):
        out.append(lin % s)
        lin = lin // s
    return [lin] + out[::-1]


FEW, WIDE = 1 << 23, 1 << 24           # rows: far more than entries; with as many columns 48-bit keys
OUTPUTS = [(CSR, (1 << 16, 1 << 16)),                                   # crd and pos from the buckets
           (DCSR, (1 << 16, 1 << 16)),                                  # distances, then all levels
           (((0, 1, 1), (0, 1, 2)), (40, 1 << 13, 1 << 12)),            # the same under a dense level
           (CDR, (1 << 17, 40)), (CSR, (FEW, 1 << 9)),                  # sorted keys
           (DCSR, (WIDE, WIDE))]                                        # sorted keys of 64 bits


@pytest.mark.parametrize("fmt,shape", OUTPUTS)
@pytest.mark.parametrize("n", [200000, TWO + 100000])
def test_a_sample_that_misleads(fmt, shape, n):
    """The sampled entries are spread over the upper half of the key range, all others lie at its beginning: the first bucket gets more
    than it has room for, and the stable sorts build the tensor."""
    total = int(np.prod([int(s) for s in shape], dtype=object))
    at = np.unique(sampled_positions(n))
    lin = np.empty(n, np.int64)
    rest = np.ones(n, bool)
    rest[at] = False
    lin[rest] = prng.permutation(SEED, 4, n + n // 4)[: n - at.size]
    spread = np.unique(prng.below(SEED, 5, 2 * at.size, total // 2)) + total // 2
    lin[at] = spread[prng.permutation(SEED, 6, spread.size)][: at.size]
    for dtype in (np.float64, np.float32):
        with overflows() as o:
            check(fmt, shape, unravel(lin, shape), dtype)
        assert o.counts == [1, 0]


@pytest.mark.parametrize("fmt", [CSC, ((1, 1), (1, 0))])
@pytest.mark.parametrize("n", [200000, TWO + 100000])
def test_a_sample_that_misleads_a_conversion(fmt, n):
    """One entry per row, so that the source keeps their order; the sampled ones in the last columns, all others in the first sixteen."""
    N = 1 << 16
    at = np.unique(sampled_positions(n))
    cols = prng.below(SEED, 7, n, 16)
    cols[at] = N // 2 + prng.below(SEED, 8, at.size, N // 2)
    coords, v = [np.arange(n, dtype=np.int64), cols], prng.uniform_pm1(SEED, 9, n, np.float32)
    A = gpu_pack(*CSR, (n, N), coords, v)
    with overflows() as o:
        B = sp.sp_convert(A, sp.sp_encode(*fmt, 32, 32))
    say("case", fmt, n, "overflows", o.counts)
    assert o.counts == [1, 0]
    assert_storage_equal(B, oracle.pack(*fmt, (n, N), coords, v, 32, 32))


@pytest.mark.parametrize("fmt,shape", [(CSR, (1 << 16, 1 << 16)), (DCSR, (1 << 16, 1 << 16)), (CSR, (FEW, 1 << 9))])
def test_a_bucket_with_more_entries_than_a_block_sorts(fmt, shape):
    """One partition: a bucket has 4144 entries, its room is 4192, the finishing kernel takes 4096."""
    n = 200000
    at = sampled_positions(n)
    S, Q = at.size, -(-n // 2048)
    assert np.unique(at).size == S
    step = (1 << 32) // S
    i0, i1 = 40 * S // Q, 41 * S // Q                        # the samples of the 40th bucket; between two samples it has `more` others
    more = np.zeros(S, np.int64)
    more[i0:i1] = (4144 - (i1 - i0)) // (i1 - i0)
    more[i0: i0 + (4144 - (i1 - i0)) % (i1 - i0)] += 1
    elsewhere = np.flatnonzero((np.arange(S) < i0) | (np.arange(S) >= i1))
    left = n - S - int(more.sum())
    more[elsewhere] = left // elsewhere.size
    more[elsewhere[: left % elsewhere.size]] += 1
    i = np.repeat(np.arange(S), more)
    others = i * step + 8 + 997 * (np.arange(i.size) - np.repeat(np.cumsum(more) - more, more))
    lin = np.empty(n, np.int64)
    rest = np.ones(n, bool)
    rest[at] = False
    lin[at] = np.arange(S) * step + 7
    lin[rest] = others[prng.permutation(SEED, 10, others.size)]
    assert np.unique(lin).size == n and lin.max() < 1 << 32
    with overflows() as o:
        check(fmt, shape, unravel(lin, shape))
    assert o.counts == [0, 1]


def test_a_part_with_more_entries_than_its_room():
    """Two partitions, 48-bit keys: the last bucket spans a third of the key range or more, so that its sample, cut to 32 bits, cannot tell
    8000 neighbouring keys apart."""
    body = np.unique(prng.below(SEED, 11, 1100000, 1 << 44))
    sparse = (1 << 44) + np.unique(prng.below(SEED, 12, 9000, int(0.7 * 2 ** 48) - (1 << 44)))
    crowd = 3 * (1 << 46) + np.arange(8000)
    behind = crowd[-1] + 1 + np.unique(prng.below(SEED, 13, 1000, (1 << 46) - 16000))
    lin = np.concatenate([body, sparse, crowd, behind])
    lin = lin[prng.permutation(SEED, 14, lin.size)]
    with overflows() as o:
        check(DCSR, (WIDE, WIDE), unravel(lin, (WIDE, WIDE)))
    assert o.counts == [0, 1]


@pytest.mark.parametrize("fmt,shape", OUTPUTS)
def test_an_entry_given_six_thousand_times(fmt, shape):
    """They fill a part of the second partition by themselves; the stable sorts report them."""
    coords = distinct(shape, TWO, SEED + 15)
    coords = [np.concatenate([c, np.full(6000, c[17])]) for c in coords]
    order = prng.permutation(SEED, 16, coords[0].size)
    with overflows() as o, pytest.raises(sp.SpError) as e:
        gpu_pack(*fmt, shape, [c[order] for c in coords], np.ones(order.size, np.float32))
    say("case", fmt, shape, "overflows", o.counts)
    assert e.value.code == 7 and o.counts == [0, 1]


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
