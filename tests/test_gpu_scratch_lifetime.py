"""Scratch that a handle keeps between products: what a recorded product was recorded with stays until sp_tensor_free, whatever
other products make the scratch larger in between; and products of a width that is no multiple of 16 bytes may overlap on
different streams, and with replays.

The allocator keeps count of the blocks the library holds, so a block that goes back too early is seen before anything is
replayed.  Tolerance: the products' own."""
import numpy as np
import pytest
import torch

import oracle
import paper_2202_04305_amd as sp
from paper_2202_04305_amd import binding
from gen import workloads as W, prng
from gpu_util import say, dev, assert_product_close, DEV

pytestmark = pytest.mark.gpu


def _matrix(dtype=np.float64):
    w = W.cfg2_powerlaw_csr(6000, 5000, mean=30.0, sigma=1.5, cap=3000)
    w.vals = w.vals.astype(dtype)
    return w


def _pack(w, lt=(0, 1)):
    alloc = binding._TorchAllocator(DEV)
    return sp.sp_pack(sp.sp_encode(lt, (0, 1), 32, 32), w.shape, [dev(w.rows), dev(w.cols)], dev(w.vals), allocator=alloc), alloc


def _record(call):
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    return graph


def _check_replays(graph, out, ref, mag, dtype, between):
    for replay in range(3):
        out.fill_(float("nan"))
        between()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert_product_close(out, ref, mag, dtype, "replay %d" % replay)


@pytest.mark.parametrize("dtype,N,more", [(np.float64, 33, 65), (np.float64, 32, 64), (np.float32, 7, 31), (np.float64, 33, 64), (np.float64, 32, 33)])
def test_recorded_spmm_outlives_a_wider_product(dtype, N, more):
    w = _matrix(dtype)
    A, alloc = _pack(w)
    B = prng.uniform_pm1(7, 1, w.shape[1] * more, dtype=dtype).reshape(-1, more)
    ref, mag = oracle.matmul_coo(w.shape, w.rows, w.cols, w.vals, B)
    Bn, Bw = dev(np.ascontiguousarray(B[:, :N])), dev(B)
    Cn, Cw = torch.empty((w.shape[0], N), dtype=A.dtype, device=DEV), torch.empty((w.shape[0], more), dtype=A.dtype, device=DEV)
    sp.sp_prepare(A, N)
    say("case recorded spmm", dtype.__name__, N, "then", more)
    graph = _record(lambda: sp.sp_matmul(A, Bn, Cn))
    held, bytes_held = set(alloc.live), sp.sp_tensor_info(A).derivedBytes
    sp.sp_matmul(A, Bw, Cw)
    torch.cuda.synchronize()
    assert held <= set(alloc.live), "scratch that the graph uses went back to the allocator"
    assert sp.sp_tensor_info(A).derivedBytes > bytes_held
    _check_replays(graph, Cn, ref[:, :N], mag[:, :N], dtype, lambda: sp.sp_matmul(A, Bw, Cw))
    assert_product_close(Cw, ref, mag, dtype, "the wider product")
    del graph
    A.free()
    assert not alloc.live


def test_scratch_nothing_was_recorded_with_goes_back():
    w = _matrix()
    A, alloc = _pack(w)
    for N in (8, 16, 17, 33):
        B, C = torch.ones((w.shape[1], N), dtype=A.dtype, device=DEV), torch.empty((w.shape[0], N), dtype=A.dtype, device=DEV)
        sp.sp_matmul(A, B, C)
        count = len(alloc.live) if N == 8 else count
        assert len(alloc.live) == count


@pytest.mark.parametrize("J,more", [(42, 58), (43, 59)])
def test_recorded_mttkrp_outlives_a_wider_product(J, more):
    """A factor large enough, and gathered from often enough, for its padded copy to be part of the scratch."""
    t = W.tensor3_slices(I=50, K=300, L=40000, nnz=2000000, k_mean=200, l_mean=20000, sigma=0.3, J=more)
    C, D = t.factors()
    ref, mag = oracle.mttkrp_coo(t.shape, t.ci, t.ck, t.cl, t.vals, C, D)
    alloc = binding._TorchAllocator(DEV)
    T = sp.sp_pack(sp.sp_encode((0, 1, 1), (0, 1, 2), 32, 32), t.shape, [dev(x) for x in (t.ci, t.ck, t.cl)], dev(t.vals), allocator=alloc)
    Cn, Dn = [dev(np.ascontiguousarray(f[:, :J])) for f in (C, D)]
    An, Aw = [torch.empty((t.shape[0], j), dtype=torch.float64, device=DEV) for j in (J, more)]
    say("case recorded mttkrp", J, "then", more)
    sp.sp_mttkrp(T, Cn, Dn, A=An)                          # makes what the recording may not make
    graph = _record(lambda: sp.sp_mttkrp(T, Cn, Dn, A=An))
    held = set(alloc.live)
    assert sp.sp_tensor_info(T).derivedBytes >= 40000 * 384, "no padded copy: the test does not reach it"
    sp.sp_mttkrp(T, dev(C), dev(D), A=Aw)
    torch.cuda.synchronize()
    assert held <= set(alloc.live), "scratch that the graph uses went back to the allocator"
    _check_replays(graph, An, ref[:, :J], mag[:, :J], np.float64, lambda: sp.sp_mttkrp(T, dev(C), dev(D), A=Aw))


def test_recorded_sddmm_outlives_a_wider_product():
    w = _matrix()
    S, alloc = _pack(w)
    order = np.lexsort((w.cols, w.rows))
    K, more = 16, 40
    A, B = prng.uniform_pm1(8, 1, w.shape[0] * more).reshape(-1, more), prng.uniform_pm1(8, 2, w.shape[1] * more).reshape(more, -1)
    ref, mag = oracle.sddmm_coo(w.shape, w.rows, w.cols, w.vals, np.ascontiguousarray(A[:, :K]), np.ascontiguousarray(B[:K]))
    An, Bn, X = dev(np.ascontiguousarray(A[:, :K])), dev(np.ascontiguousarray(B[:K])), torch.empty(w.nnz, dtype=torch.float64, device=DEV)
    sp.sp_sddmm(S, An, Bn, X)
    say("case recorded sddmm", K, "then", more)
    graph = _record(lambda: sp.sp_sddmm(S, An, Bn, X))
    held = set(alloc.live)
    sp.sp_sddmm(S, dev(A), dev(B))
    torch.cuda.synchronize()
    assert held <= set(alloc.live), "scratch that the graph uses went back to the allocator"
    _check_replays(graph, X, ref[order], mag[order], np.float64, lambda: sp.sp_sddmm(S, dev(A), dev(B)))


@pytest.mark.parametrize("lt", [(0, 1), (1, 1)])
def test_odd_widths_overlap_on_streams_and_with_replays(lt):
    """One tensor, three streams, products of 33 and 17 columns in flight at once and a recorded one of 9: every result is its own."""
    w = W.cfg2_powerlaw_csr(40000, 30000, mean=24.0, sigma=1.5, cap=20000)
    A, _ = _pack(w, lt)
    sp.sp_prepare(A, 33)
    widths = (33, 17, 33)
    B = prng.uniform_pm1(7, 1, w.shape[1] * 33).reshape(-1, 33)
    ref, mag = oracle.matmul_coo(w.shape, w.rows, w.cols, w.vals, B)
    say("case overlapping streams", lt)
    streams = [torch.cuda.Stream() for _ in widths]
    Bs = [dev(np.ascontiguousarray(B[:, :n])) for n in widths]
    Cs = [[torch.empty((w.shape[0], n), dtype=torch.float64, device=DEV) for _ in range(6)] for n in widths]
    Bg, Cg = dev(np.ascontiguousarray(B[:, :9])), torch.empty((w.shape[0], 9), dtype=torch.float64, device=DEV)
    graph = _record(lambda: sp.sp_matmul(A, Bg, Cg))
    torch.cuda.synchronize()
    for call in range(6):
        for s, b, c in zip(streams, Bs, Cs):
            with torch.cuda.stream(s):
                sp.sp_matmul(A, b, c[call])
        graph.replay()
    torch.cuda.synchronize()
    for n, c in zip(widths, Cs):
        for call in range(6):
            assert_product_close(c[call], ref[:, :n], mag[:, :n], np.float64, "stream with %d columns, call %d" % (n, call))
    assert_product_close(Cg, ref[:, :9], mag[:, :9], np.float64, "replay among the streams")
    # once its stream has nothing left to do the scratch goes to the next one, which gets the same bits
    again = torch.empty_like(Cs[0][0])
    sp.sp_matmul(A, Bs[0], again)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        more = torch.empty_like(again)
        sp.sp_matmul(A, Bs[0], more)
    torch.cuda.synchronize()
    assert torch.equal(again, more) and sp.sp_tensor_info(A).lazyPrepares == 0
