"""The levels that the storage builder writes, around the edges of the level sweep's tiles of 1024 sorted entries, for every mix of
level types of rank 1 to 4 (by the sweep, after a sort that leaves keys, and by the builder's own choice, which writes the levels of
many formats from its buckets), against the CPU checker, bit for bit; level sizes that are and are not powers of two; keys above and below 2^52
(where the division of a key by a stride changes its method)."""
import itertools

import numpy as np
import pytest

import oracle
import paper_2202_04305_amd as sp
from gen import prng
from gpu_util import say, gpu_pack, assert_storage_equal

pytestmark = pytest.mark.gpu
SEED = 20220417


@pytest.fixture(params=[0, 1], ids=["sort chosen", "level sweep"])
def sort_mode(request):
    sp.sp_pack_sort_mode(request.param)
    yield request.param
    sp.sp_pack_sort_mode(0)


def entries(shape, nnz, stream):
    total = int(np.prod([int(s) for s in shape], dtype=object))
    lin = np.unique(prng.below(SEED, stream, nnz + nnz // 8 + 16, min(total, 1 << 52)))
    if total > 1 << 52:                                    # spread over the whole range of the key
        lin = np.unique(lin.astype(object) * (total >> 52)).astype(np.int64)
    lin = lin[prng.permutation(SEED, stream + 1, lin.size)][:nnz]
    coords = []
    for s in reversed(shape):
        coords.append(lin % s)
        lin = lin // s
    return coords[::-1]


@pytest.mark.parametrize("nnz", [1, 63, 1023, 1024, 1025, 4097])
@pytest.mark.parametrize("rank", [1, 2, 3, 4])
def test_every_mix_of_level_types(nnz, rank, sort_mode):
    sides = [(9000,), (64, 150), (16, 25, 22), (8, 11, 10, 9)][rank - 1]
    coords = entries(sides, nnz, 10 * rank)
    for i, lt in enumerate(itertools.product((0, 1), repeat=rank)):
        order = tuple(np.roll(np.arange(rank), i % rank))
        v = prng.uniform_pm1(SEED, 3, coords[0].size, np.float32 if i % 2 else np.float64)
        pw, cw = [(32, 32), (64, 32), (32, 64), (64, 64)][i % 4]
        say("case rank", rank, "levels", lt, "order", order, "entries", v.size, "widths", pw, cw)
        assert_storage_equal(gpu_pack(lt, order, sides, coords, v, pw, cw), oracle.pack(lt, order, sides, coords, v, pw, cw))


@pytest.mark.parametrize("lt", [(1, 1, 1), (0, 1, 1), (1, 0, 1)])
@pytest.mark.parametrize("sides", [(37, 1 << 20, 100003), (37, (1 << 29) - 3, (1 << 28) + 1), (5, 1 << 29, 1 << 28)])
def test_wide_keys(lt, sides):
    if lt[1] == 0:
        sides = (sides[0], 1000, sides[2])
    coords = entries(sides, 20000, 90)
    v = prng.uniform_pm1(SEED, 4, coords[0].size, np.float64)
    say("case wide keys", lt, sides)
    assert_storage_equal(gpu_pack(lt, (0, 1, 2), sides, coords, v, 64, 64), oracle.pack(lt, (0, 1, 2), sides, coords, v, 64, 64))
