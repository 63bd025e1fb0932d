// C[i,j] = sum_k A[i,k] * B[k,j] with A sparse and B, C dense row-major (arXiv 2202.04305,
// Section 1: the SpMM kernel; Section 6.2: matrix times vector).  The loops the paper's
// compiler would emit visit, per outer position, the pos range of the inner compressed
// level (Section 4.3); the kernels below visit exactly those entries, split differently:
//
//   rows kernel      G lanes per stored row, strided over the row, shuffle reduction.
//   stream kernel    SpMV: every block owns 2048 consecutive stored entries whatever rows
//                    they belong to: coalesced crd/values stream, gathered x, products
//                    staged in LDS, rows reduced from LDS (a thread per short row, a wave per
//                    long one); rows that cross a block boundary are completed by a small
//                    fix-up kernel from per-block carries (deterministic, no atomics).
//   runs kernel      SpMM: groups of lanes across the columns of B take runs of consecutive stored entries (windows, carries
//                    and fix-up as above).
//   windows kernel   SpMM: the same windows, a wave per row inside them: even rows of medium length.
//   spmm kernels     one wave per stored row, lanes across the columns of B: small products, and where no scratch can be had.
//   scatter kernel   column-major storage (CSC / DCSC): a wave per stored column, atomic
//                    adds into the rows of C.
//
// "Row-major" means the outer level holds dimension 0; that level may be dense (CSR: row =
// position) or compressed (DCSR: row = crd0[position], so empty rows cost nothing).
#include "spmi_internal.h"

namespace {

constexpr int kThreads = 256;
constexpr int kST = kSpmiStreamThreads;        // threads per block of the stream kernel, 8 stored entries each
constexpr int kStreamT = (int)kSpmiStreamT;   // stored entries per block of the stream kernel (the row blocks are built for it)
constexpr int kLongRow = 64;        // in-window row length above which a wave reduces the row
constexpr int kQueue = 64;
constexpr int64_t kSpmvSliceBytes = (int64_t)2 << 20;     // slice of x one column panel gathers from: half of a 4 MB per-XCD L2
constexpr int kPre = 1;             // rounds of the row loop whose pos entries are fetched ahead
static_assert(kStreamT / (kLongRow + 1) < kQueue, "queue of long rows too small");

template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
    return v;
}

template <typename VT>
__global__ __launch_bounds__(kThreads) void zero_matrix_kernel(VT *__restrict__ C, int64_t m, int64_t N, int64_t ldc)
{
    const int64_t total = m * N;
    int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * kThreads;
    for (; i < total; i += stride) C[(i / N) * ldc + (i % N)] = (VT)0;
}

// ---- G lanes per stored row -------------------------------------------------------------
template <typename PT, typename CT, typename VT, int G>
__global__ __launch_bounds__(kThreads) void spmv_rows_kernel(const PT *__restrict__ pos, const CT *__restrict__ crd,
                                                             const VT *__restrict__ val, const CT *__restrict__ rowid, int64_t nrows,
                                                             const VT *__restrict__ x, int64_t ldb, VT *__restrict__ y, int64_t ldc,
                                                             int accumulate)
{
    const int64_t r = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / G;
    const int sub = threadIdx.x % G;
    VT acc = 0;
    if (r < nrows) {
        const int64_t a = (int64_t)pos[r], b = (int64_t)pos[r + 1];
        for (int64_t p = a + sub; p < b; p += G) acc += val[p] * x[(int64_t)crd[p] * ldb];
    }
#pragma unroll
    for (int d = G / 2; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, 64);
    if (sub == 0 && r < nrows) {
        const int64_t row = rowid ? (int64_t)rowid[r] : r;
        y[row * ldc] = accumulate ? y[row * ldc] + acc : acc;
    }
}

// ---- stream kernel ----------------------------------------------------------------------
// Measured on the 1M x 1M workload: with operands cold in HBM the kernel runs 10 % faster at 3 waves per SIMD than at
// the 8 the register count would allow (fewer concurrent entry streams); warm it makes no difference.
#ifndef SPMI_WPE
#define SPMI_WPE 3
#endif
template <typename PT, typename CT, typename VT>
__global__ __launch_bounds__(kST) __attribute__((amdgpu_waves_per_eu(1, SPMI_WPE))) void spmv_stream_kernel(const PT *__restrict__ pos, const CT *__restrict__ crd,
                                                               const VT *__restrict__ val, const CT *__restrict__ rowid,
                                                               const int32_t *__restrict__ rowblk, int64_t nrows, int64_t nnz,
                                                               const VT *__restrict__ x, int64_t ldb, VT *__restrict__ y, int64_t ldc,
                                                               VT *__restrict__ carry, int accumulate)
{
    const int64_t win = blockIdx.x;
    __shared__ VT prods[kStreamT];
    __shared__ int queue[kQueue];
    __shared__ int qn, lo_began_earlier;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t s = win * kStreamT;
    const int64_t e = (s + kStreamT < nnz) ? s + kStreamT : nnz;
    if (tid == 0) qn = 0;

    // phase A: this block's entries (two consecutive entries per lane and step), every load issued before the
    // first use.  The pos entries of the rows that meet the window (see phase B) are fetched in the same
    // batch, for the first kPre rounds of the row loop, so that their latency hides under the gathers.
    const bool full = e - s == kStreamT;
    constexpr int E = kSpmiStreamPer;
    CT k[E];
    VT v[E];
    if (full) {
#pragma unroll
        for (int t = 0; t < E / 2; ++t) {
            const int64_t p = s + (int64_t)(t * kST + tid) * 2;
            k[2 * t] = crd[p]; k[2 * t + 1] = crd[p + 1];
            v[2 * t] = val[p]; v[2 * t + 1] = val[p + 1];
        }
    }
    const int64_t lo = rowblk[win], hi = rowblk[win + 1];
    const int64_t last = hi < nrows ? hi : nrows - 1;
    PT pre_a[kPre], pre_b[kPre];
#pragma unroll
    for (int i = 0; i < kPre; ++i) {
        int64_t r = lo + tid + (int64_t)i * kST;
        r = r <= last ? r : last;                      // clamped, not predicated: the loads stay unconditional
        pre_a[i] = pos[r];
        pre_b[i] = pos[r + 1];
    }
    if (full) {
        VT xv[E];
#pragma unroll
        for (int i = 0; i < E; ++i) xv[i] = x[(int64_t)k[i] * ldb];
#pragma unroll
        for (int t = 0; t < E / 2; ++t) {
            prods[(t * kST + tid) * 2] = v[2 * t] * xv[2 * t];
            prods[(t * kST + tid) * 2 + 1] = v[2 * t + 1] * xv[2 * t + 1];
        }
    } else {
        for (int i = tid; i < (int)(e - s); i += kST) prods[i] = val[s + i] * x[(int64_t)crd[s + i] * ldb];
    }
    if (tid == 0) lo_began_earlier = (int64_t)pre_a[0] < s;      // thread 0 prefetched pos[lo]
    __syncthreads();

    // phase B: rows lo..hi meet this window.  Rows lo..hi-1 end here and are written; row hi only
    // starts here (its head goes to y, the rest arrives through later blocks' carries); if row lo
    // began in an earlier window its part goes to this block's carry.
    const bool lo_carried = lo_began_earlier != 0;
    auto emit = [&](int64_t r, VT sum) {
        if (r == lo && lo_carried) { carry[win] = sum; return; }
        VT *dst = y + (rowid ? (int64_t)rowid[r] : r) * ldc;
        *dst = accumulate ? *dst + sum : sum;
    };
    auto short_row = [&](int64_t r, int64_t pa, int64_t pb) {
        const int a = (int)((pa > s ? pa : s) - s), b = (int)((pb < e ? pb : e) - s);
        if (r == hi && b <= a) return;               // row hi starts at the next window: not ours
        if (b - a > kLongRow) { queue[atomicAdd(&qn, 1)] = (int)(r - lo); return; }
        VT sum = 0;
        for (int i = a; i < b; ++i) sum += prods[i];
        emit(r, sum);
    };
#pragma unroll
    for (int k = 0; k < kPre; ++k) {
        const int64_t r = lo + tid + (int64_t)k * kST;
        if (r <= last) short_row(r, (int64_t)pre_a[k], (int64_t)pre_b[k]);
    }
    for (int64_t r = lo + tid + (int64_t)kPre * kST; r <= last; r += kST)
        short_row(r, (int64_t)pos[r], (int64_t)pos[r + 1]);
    __syncthreads();
    const int nq = qn;
    for (int q = wave; q < nq; q += kST / 64) {
        const int64_t r = lo + queue[q];
        const int64_t pa = (int64_t)pos[r], pb = (int64_t)pos[r + 1];
        const int a = (int)((pa > s ? pa : s) - s), b = (int)((pb < e ? pb : e) - s);
        VT sum = 0;
        for (int i = a + lane; i < b; i += 64) sum += prods[i];
        sum = wave_sum(sum);
        if (lane == 0) emit(r, sum);
    }
}

// One thread per block boundary: the first boundary a row crosses adds all of that row's carries, in
// block order, to the head part already in y.
template <typename PT, typename CT, typename VT>
__global__ __launch_bounds__(kThreads) void spmv_stream_fixup_kernel(const PT *__restrict__ pos, const CT *__restrict__ rowid,
                                                                     const int32_t *__restrict__ rowblk, int64_t nblocks,
                                                                     const VT *__restrict__ carry, VT *__restrict__ y, int64_t ldc)
{
    const int64_t b = (int64_t)blockIdx.x * kThreads + threadIdx.x + 1;
    if (b >= nblocks) return;
    const int64_t r = rowblk[b];
    const int64_t start = (int64_t)pos[r];
    if (start >= b * kStreamT || start < (b - 1) * kStreamT) return;   // not crossed here, or crossed earlier already
    VT sum = 0;
    for (int64_t bb = b; bb < nblocks && rowblk[bb] == r; ++bb) sum += carry[bb];
    const int64_t row = rowid ? (int64_t)rowid[r] : r;
    y[row * ldc] += sum;
}

// Column-segmented SpMV, last step: y[r] = (y[r]) + sum over panels of the per-panel partial results.
template <typename VT>
__global__ __launch_bounds__(kThreads) void spmv_panel_sum_kernel(const VT *__restrict__ part, int64_t nrows, int panels,
                                                                  VT *__restrict__ y, int64_t ldc, int accumulate)
{
    const int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (r >= nrows) return;
    VT sum = accumulate ? y[r * ldc] : (VT)0;
    for (int p = 0; p < panels; ++p) sum += part[(int64_t)p * nrows + r];
    y[r * ldc] = sum;
}

// ---- binned SpMV (see sp_bins): two streaming passes, every gather and every scattered add inside the LDS ----
constexpr int kBinThreads = 1024;
constexpr int kBinPW = 1 << kSpmiBinPanelShift;
constexpr int kBinRB = 1 << kSpmiBinRowShift;

// First pass: block (panel, piece) loads the panel's slice of x into LDS, then streams its share of the panel's entries, 16 bytes
// of values per lane and load: the product of entry e = val[e] * x[panel * PW + lcol[e]] goes to the row-block-major array, to
// slot e % 8 of the group that gdst names for e's group of 8.  Padding entries carry value 0 and column PW, where the slice
// holds a zero, so that they give 0 whatever x holds.  Blocks beyond the pieces clear y (m contiguous values, kBinClear of them a
// block), where rows that are not stored have to become zero.
constexpr int kBinClear = 16384;
template <typename VT>
__global__ __launch_bounds__(kBinThreads) void spmv_bins_multiply_kernel(const VT *__restrict__ val, const uint16_t *__restrict__ lcol,
                                                                         const uint32_t *__restrict__ gdst, const int64_t *__restrict__ pstart,
                                                                         int panels, int pieces, int64_t n, const VT *__restrict__ x, int64_t ldb,
                                                                         VT *__restrict__ prod, VT *__restrict__ y, int64_t m)
{
    constexpr int V = 16 / sizeof(VT);
    typedef VT vec_t __attribute__((ext_vector_type(V)));
    typedef uint16_t idx_t __attribute__((ext_vector_type(V)));
    __shared__ VT xs[kBinPW + V];
    // blocks go to the eight XCDs in turn: the pieces of one panel are given to blocks b, b + 8, b + 16, ... so that they
    // share an L2 and the panel's slice of x is fetched from memory once, not once per piece
    const int grp = 8 * pieces, work = (panels + 7) / 8 * grp;
    if ((int)blockIdx.x >= work) {                     // whole block
        const int64_t a = (int64_t)((int)blockIdx.x - work) * kBinClear, b = a + kBinClear < m ? a + kBinClear : m;
        for (int64_t i = a + threadIdx.x; i < b; i += kBinThreads) y[i] = (VT)0;
        return;
    }
    const int p = (int)(blockIdx.x / grp) * 8 + (int)(blockIdx.x % 8), q = (int)(blockIdx.x / 8) % pieces;
    if (p >= panels) return;                           // whole block (the panel count is rounded up to eight)
    const int64_t pa = pstart[p], pb = pstart[p + 1];  // multiples of 8
    auto cut = [&](int k) -> int64_t {                 // piece boundaries: multiples of 8 inside the panel
        if (k <= 0) return pa;
        if (k >= pieces) return pb;
        return (pa + (pb - pa) * k / pieces) & ~(int64_t)7;
    };
    const int64_t a = cut(q), b = cut(q + 1);
    if (a >= b) return;                                // whole block
    const int64_t c0 = (int64_t)p * kBinPW;
    for (int i = threadIdx.x; i < kBinPW + V; i += kBinThreads) xs[i] = (i < kBinPW && c0 + i < n) ? x[(c0 + i) * ldb] : (VT)0;
    __syncthreads();
    const int64_t nvec = (b - a) / V;
    const vec_t *__restrict__ vv = (const vec_t *)(val + a);
    const idx_t *__restrict__ cc = (const idx_t *)(lcol + a);
    const uint32_t *__restrict__ gg = gdst + (a >> 3);
    constexpr int U = 2, GV = 8 / V;                   // GV lanes share a group
    auto store = [&](int64_t j, uint32_t g, const vec_t &r) { *(vec_t *)(prod + ((int64_t)g * 8 + (int64_t)(j % GV) * V)) = r; };
    int64_t j = threadIdx.x;
    for (; j + (U - 1) * kBinThreads < nvec; j += U * kBinThreads) {
        vec_t v[U];
        idx_t c[U];
        uint32_t g[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { v[u] = vv[j + u * kBinThreads]; c[u] = cc[j + u * kBinThreads]; g[u] = gg[(j + u * kBinThreads) / GV]; }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            vec_t r;
#pragma unroll
            for (int t = 0; t < V; ++t) r[t] = v[u][t] * xs[c[u][t]];
            store(j + u * kBinThreads, g[u], r);
        }
    }
    for (; j < nvec; j += kBinThreads) {
        const vec_t v = vv[j];
        const idx_t c = cc[j];
        const uint32_t g = gg[j / GV];
        vec_t r;
#pragma unroll
        for (int t = 0; t < V; ++t) r[t] = v[t] * xs[c[t]];
        store(j, g, r);
    }
}

// Second pass: block = row block.  It streams the row block's products and 16-bit rows, which the first pass left side by side
// (a lane takes a group of 8 with 16-byte loads), and adds them into the block's slice of y in LDS (atomic adds: the order in
// which a row's products meet is not fixed); the slice is written out at the end.  Every stored row of the row block is
// written (m of them; rowid[q] is the matrix row of stored row q when not all rows are stored, and the caller has then
// zeroed the others).  The slice is f64 for f32 products as well: adds of 32 bits to the LDS are the slower ones (2.7 M entries in 41
// row blocks, x of 4 MB: 100 us for the product, 29 now), and long sums lose nothing.
// f64: four slices, a quarter of the waves adding into each, so that a row's sum is four shorter ones (rows of up to 54 entries: error
// 1.9e-16 of the result with one, as in the streamed kernel, 1.3e-16 with four, 1.4e-16 by column panels; the same time).
template <typename CT, typename VT>
__global__ __launch_bounds__(kBinThreads) void spmv_bins_reduce_kernel(const VT *__restrict__ prod, const uint16_t *__restrict__ lrow,
                                                                       const int64_t *__restrict__ rbstart, int rshift, int64_t m,
                                                                       const CT *__restrict__ rowid, VT *__restrict__ y, int64_t ldc,
                                                                       int accumulate)
{
    constexpr int V = 16 / sizeof(VT), NV = 8 / V;
    typedef VT vec_t __attribute__((ext_vector_type(V)));
    typedef unsigned uint4v __attribute__((ext_vector_type(4)));
    constexpr int kCopies = sizeof(VT) == 8 ? 4 : 1;
    __shared__ double ys[kCopies * kBinRB];
    const int rb = (int)blockIdx.x;
    const int rows = 1 << rshift;                      // <= kBinRB
    for (int i = threadIdx.x; i < kCopies * rows; i += kBinThreads) ys[i] = 0.0;
    double *__restrict__ mine = ys + (int)(threadIdx.x / 64) % kCopies * rows;
    __syncthreads();
    const int64_t g0 = rbstart[rb] >> 3, g1 = rbstart[rb + 1] >> 3;
    const vec_t *__restrict__ pp = (const vec_t *)prod;
    const uint4v *__restrict__ rr = (const uint4v *)lrow;
    for (int64_t g = g0 + threadIdx.x; g < g1; g += kBinThreads) {
        vec_t v[NV];
#pragma unroll
        for (int k = 0; k < NV; ++k) v[k] = pp[g * NV + k];
        const uint4v r = rr[g];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const unsigned w = (t >> 1) == 0 ? r.x : (t >> 1) == 1 ? r.y : (t >> 1) == 2 ? r.z : r.w;
            atomicAdd(&mine[(t & 1) ? (w >> 16) : (w & 0xffffu)], (double)v[t / V][t % V]);
        }
    }
    __syncthreads();
    const int64_t r0 = (int64_t)rb << rshift;
    for (int i = threadIdx.x; i < rows; i += kBinThreads) {
        const int64_t q = r0 + i;                      // stored row; rowid maps it to the matrix row where not all rows are stored
        if (q < m) {
            VT *dst = y + (rowid ? (int64_t)rowid[q] : q) * ldc;
            double sum = ys[i];
            if constexpr (kCopies == 4) sum = (sum + ys[rows + i]) + (ys[2 * rows + i] + ys[3 * rows + i]);
            *dst = (VT)(accumulate ? (double)*dst + sum : sum);
        }
    }
}

// ---- SpMM: a wave per stored row, CG lanes across a tile of B's columns, 64/CG entries in flight ----
template <typename PT, typename CT, typename VT, int CG>
__global__ __launch_bounds__(kThreads) void spmm_rows_kernel(const PT *__restrict__ pos, const CT *__restrict__ crd,
                                                             const VT *__restrict__ val, const CT *__restrict__ rowid, int64_t nrows,
                                                             const VT *__restrict__ B, int64_t N, int64_t ldb, VT *__restrict__ C,
                                                             int64_t ldc, int accumulate)
{
    constexpr int S = 64 / CG;                        // entries of the row handled side by side
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (r >= nrows) return;                           // whole wave
    const int jl = lane % CG, sl = lane / CG;
    const int64_t a = (int64_t)pos[r], b = (int64_t)pos[r + 1];
    const int64_t row = rowid ? (int64_t)rowid[r] : r;
    for (int64_t j0 = 0; j0 < N; j0 += CG) {
        const int64_t j = j0 + jl;
        const bool jin = j < N;
        VT acc = 0;
        int64_t p = a + sl;
        if constexpr (CG == 64) {                      // 512-byte rows of B (f64): two row gathers in flight measured best
            VT acc1 = 0;
            for (; p + S < b; p += 2 * S) {
                const int64_t k0 = (int64_t)crd[p], k1 = (int64_t)crd[p + S];
                const VT v0 = val[p], v1 = val[p + S];
                if (jin) { acc += v0 * B[k0 * ldb + j]; acc1 += v1 * B[k1 * ldb + j]; }
            }
            if (p < b && jin) acc += val[p] * B[(int64_t)crd[p] * ldb + j];
            acc += acc1;
        } else {                                       // narrower tiles: four
            constexpr int U = 4;
            VT accu[U];
#pragma unroll
            for (int u = 0; u < U; ++u) accu[u] = 0;
            for (; p + (U - 1) * S < b; p += U * S) {
                int64_t k[U];
                VT v[U], bv[U];
#pragma unroll
                for (int u = 0; u < U; ++u) { k[u] = (int64_t)crd[p + u * S]; v[u] = val[p + u * S]; }
#pragma unroll
                for (int u = 0; u < U; ++u) bv[u] = jin ? B[k[u] * ldb + j] : (VT)0;
#pragma unroll
                for (int u = 0; u < U; ++u) accu[u] += v[u] * bv[u];
            }
            for (; p < b; p += S)
                if (jin) accu[0] += val[p] * B[(int64_t)crd[p] * ldb + j];
#pragma unroll
            for (int u = 0; u < U; ++u) acc += accu[u];
        }
#pragma unroll
        for (int d = 32; d >= CG; d >>= 1) acc += __shfl_xor(acc, d, 64);
        if (sl == 0 && jin) C[row * ldc + j] = accumulate ? C[row * ldc + j] + acc : acc;
    }
}

// SpMM with 16-byte loads: LR lanes cover one row of B (N = LR * 16 / sizeof(VT) columns), 64 / LR stored entries of
// the row of A side by side, two gathers in flight per lane.  Needs N a multiple of the vector width and B, C rows
// 16-byte aligned; the dispatch checks it.
template <typename PT, typename CT, typename VT, int LR>
__global__ __launch_bounds__(kThreads) void spmm_rows_vec_kernel(const PT *__restrict__ pos, const CT *__restrict__ crd,
                                                                 const VT *__restrict__ val, const CT *__restrict__ rowid, int64_t nrows,
                                                                 const VT *__restrict__ B, int64_t ldb, VT *__restrict__ C, int64_t ldc,
                                                                 int accumulate)
{
    constexpr int V = 16 / sizeof(VT);
    constexpr int S = 64 / LR;
    typedef VT vec_t __attribute__((ext_vector_type(V)));
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (r >= nrows) return;                           // whole wave
    const int jl = lane % LR, sl = lane / LR;
    const int64_t a = (int64_t)pos[r], b = (int64_t)pos[r + 1];
    constexpr int U = S >= 4 ? 2 : 4;                 // row gathers in flight per lane (measured: 8 to 16 entries per step)
    vec_t accu[U];
#pragma unroll
    for (int u = 0; u < U; ++u) accu[u] = (vec_t)(0);
    int64_t p = a + sl;
    for (; p + (U - 1) * S < b; p += U * S) {
        int64_t k[U];
        VT v[U];
        vec_t bv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) { k[u] = (int64_t)crd[p + u * S]; v[u] = val[p + u * S]; }
#pragma unroll
        for (int u = 0; u < U; ++u) bv[u] = *(const vec_t *)(B + k[u] * ldb + jl * V);
#pragma unroll
        for (int u = 0; u < U; ++u) accu[u] += v[u] * bv[u];
    }
    if (p < b) {                                      // the last, partial step: same batch of loads, clamped and masked
        int64_t k[U];
        VT v[U];
        vec_t bv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t pp = p + u * S;
            const bool in = pp < b;
            k[u] = (int64_t)crd[in ? pp : p];
            v[u] = in ? val[pp] : (VT)0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) bv[u] = *(const vec_t *)(B + k[u] * ldb + jl * V);
#pragma unroll
        for (int u = 0; u < U; ++u) accu[u] += v[u] * bv[u];
    }
    vec_t acc0 = accu[0];
#pragma unroll
    for (int u = 1; u < U; ++u) acc0 += accu[u];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        VT x = acc0[e];
#pragma unroll
        for (int d = 32; d >= LR; d >>= 1) x += __shfl_xor(x, d, 64);
        acc0[e] = x;
    }
    if (sl == 0) {
        const int64_t row = rowid ? (int64_t)rowid[r] : r;
        vec_t *dst = (vec_t *)(C + row * ldc + jl * V);
        *dst = accumulate ? *dst + acc0 : acc0;
    }
}

// The product cut by stored entries for any number of columns, leading dimension and element-aligned address.  Block = window
// of 1024 stored entries as above (blockIdx.y: a tile of lr_tile * V columns).  A group of LR lanes covers a row of B, V
// elements per lane, and takes a run of consecutive entries, whatever rows they belong to: it adds up while the row stays the
// same and writes C when it changes, so rows of any length keep every lane busy.  The sum of a row that began in an earlier
// run of the window waits in LDS for the group that began it; the part of a row that began in
// an earlier window goes to carry[w].  Fixed order, no atomics.  A window that lies inside one row is dealt out entry by entry.
// Runs are long (up to 256 entries), so a group adds up four entries at a time and these sums in spmi_long_sum: against a plain
// chain the error falls from 1.07e-7 to 5.5e-8 (rows of 64 entries, 32 f32 columns; 6.8e-8 with a wave per row) and from 2.4e-16 to
// 9.7e-17 (lognormal rows, 64 f64 columns; 1.6e-16), relative 2-norm; it costs 1 % (33.6 M entries, 32 f32 columns).
// The last lane of a row moves back to the last V columns and stores only those that the lane before it does not have, so
// every load is V elements wide (the memory path takes such loads at any element-aligned address).
// Bound by the rows of B it gathers (16.9 M random 512-byte rows alone: 1.15 ms).  Measured before (a wave per row of the
// window with shuffles at the end of every row; a wave per row and a column per lane for widths that are no multiple of 16
// bytes) and now: 16.9 M entries, 64 f64 columns 1.329 -> 1.280 ms; 33.6 M entries with short rows, 32 f32 columns 561 -> 363 us
// (417 with the groups' entries kept at an even stride);
// 5.0 M entries, 64-bit pos / crd, 33 f64 columns 1.250 -> 0.276 ms; 4 M entries, 4 per row, 2 f64 columns 303 -> 74 us;
// 6 M entries in rows of 20,000, 12 f32 columns 39 us (48 without the windows inside one row).
// kNarrow: runs of a few entries (one or two lanes per row of B).  Most of a sum's additions are then those of the groups' parts,
// which keep what they round off as well.
template <typename PT, typename CT, typename VT, int V, typename OT, bool kNarrow>
__global__ __launch_bounds__(kThreads, !kNarrow && sizeof(VT) + sizeof(OT) + sizeof(CT) <= 12 ? 8 : 4) void spmm_runs_kernel(const PT *__restrict__ pos, const CT *__restrict__ crd, const VT *__restrict__ val,
                                                             const CT *__restrict__ rowid, const int32_t *__restrict__ rowblk, int64_t nrows,
                                                             int64_t nnz, const VT *__restrict__ B, int64_t N, int64_t ldb, int lr_tile,
                                                             VT *__restrict__ C, int64_t ldc, VT *__restrict__ carry, int accumulate)
{
    constexpr int T = (int)kStreamT, U = 4, kWaves = kThreads / 64;
    static_assert(T == 1024, "by_run, kRoom and the 16-byte vectors in s_val and s_row");
    typedef VT vec_t __attribute__((ext_vector_type(V)));
    typedef VT mem_vec_t __attribute__((ext_vector_type(V), aligned(sizeof(VT))));
    constexpr int kRoom = T + kThreads;                              // run length (rounded up) * odd stride: 256 * 5 at most
    __shared__ OT s_off[kRoom];
    __shared__ __align__(16) VT s_val[kRoom];
    __shared__ __align__(16) CT s_row[kRoom];
    __shared__ vec_t s_part[kThreads];                               // sums of rows that began before a group's run ...
    vec_t *s_lo = (vec_t *)s_val;                                    // ... and what they round off, once the values are used up
    static_assert(sizeof(vec_t) * kThreads <= sizeof(s_val) && sizeof(vec_t) * kThreads <= sizeof(s_row), "room for a vector per thread");
    __shared__ int s_wave[kWaves];
    const int64_t j0 = (int64_t)blockIdx.y * lr_tile * V;
    const int64_t width = N - j0 < (int64_t)lr_tile * V ? N - j0 : (int64_t)lr_tile * V;
    const int LR = (int)((width + V - 1) / V);                       // 1..64
    const int S = 64 / LR, G = kWaves * S;                           // groups per wave, per block
    const int run = (T + G - 1) / G;                                 // entries per group
    const uint32_t by_run = (uint32_t)(((uint64_t)1 << 22) / (uint32_t)run + 1);      // i / run for i < 1024: exact, run <= 256
    // entry i of the window is kept at (i % run) * P + i / run: the groups of a wave read neighbouring words, and with an odd P
    // neighbouring entries lie on different banks when they are put there
    const int P = G | 1;
    auto at = [=](int i) {
        const int g = (int)(__umul24((uint32_t)i, by_run) >> 22);
        return (int)__umul24((uint32_t)(i - (int)__umul24((uint32_t)g, (uint32_t)run)), (uint32_t)P) + g;
    };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t s = (int64_t)blockIdx.x * T;
    const int64_t e = s + T < nnz ? s + T : nnz;
    const int ne = (int)(e - s);
    const OT brow = (OT)(ldb * (int64_t)sizeof(VT));
#pragma unroll
    for (int x = 0; x < T / kThreads; ++x) {
        const int i = x * kThreads + threadIdx.x;
        if (i < ne) {
            const int w = at(i);
            s_off[w] = (OT)crd[s + i] * brow;
            s_val[w] = val[s + i];
        }
    }
    const int64_t lo = rowblk[blockIdx.x], hi = rowblk[blockIdx.x + 1];
    const int64_t last = hi < nrows ? hi : nrows - 1;
    const bool continued = (int64_t)pos[lo] < s;                     // the first row began in an earlier window
    const bool one_row = (int64_t)pos[lo + 1] >= e;                  // and holds the whole window
    if (!accumulate && !rowid && last > lo)                          // rows without entries: zero (with a row list C was cleared before)
        for (int64_t r0 = lo + wave * 64; r0 <= last; r0 += kThreads) {
            const int64_t r = r0 + lane;
            uint64_t empty = __ballot(r <= last && r != hi && pos[r <= last ? r : last] == pos[(r <= last ? r : last) + 1]);
            for (; empty; empty &= empty - 1) {
                VT *dst = C + (r0 + __builtin_ctzll(empty)) * ldc + j0;
                for (int64_t j = lane; j < width; j += 64) dst[j] = (VT)0;
            }
        }
    const int sl = lane / LR, jl = lane - sl * LR;
    const int group = sl < S ? wave * S + sl : G;                    // lanes beyond S * LR take nothing
    const int first = group * run < ne ? group * run : ne, end = first + run < ne ? first + run : ne;
    const int64_t want = j0 + (int64_t)jl * V;
    const int64_t col = want <= N - V ? want : N - V;                // this lane's columns: [col, col + V), its own from skip on
    const int skip = (int)(want - col);
    const OT colb = (OT)(col * (int64_t)sizeof(VT));
    const char *Bb = (const char *)B;
    auto store = [&](VT *dst, vec_t v, bool add) {
        if (skip == 0) {
            mem_vec_t *d = (mem_vec_t *)dst;
            if (add) *d = *d + v;
            else *d = v;
        } else {
#pragma unroll
            for (int c = 1; c < V; ++c)
                if (c >= skip) dst[c] = add ? dst[c] + v[c] : v[c];
        }
    };
    const int slot = group * LR + jl;                                // this lane's place in s_part
    spmi_long_sum<VT, V> sum;                                        // of the row so far
    vec_t acc = (vec_t)(0), head_lo = (vec_t)(0);                    // acc: up to U entries more of it
    sum.clear();
    if (one_row) {
        // No rows to tell apart: the groups take the entries in turn, so that neighbouring columns are asked for together.
        __syncthreads();
        for (int k = group < G ? group : ne; k < ne; k += U * G) {
            VT v[U];
            vec_t bv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int w = at(k + u * G < ne ? k + u * G : k);
                v[u] = s_val[w];
                bv[u] = *(const mem_vec_t *)(Bb + (s_off[w] + colb));
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k + u * G < ne) acc += v[u] * bv[u];
            sum.add(acc);
            acc = (vec_t)(0);
        }
        vec_t part = sum.value(acc);
        for (int d = 1; d < S; d <<= 1) {
#pragma unroll
            for (int c = 0; c < V; ++c) {
                const VT other = __shfl(part[c], lane + d * LR < 64 ? lane + d * LR : lane, 64);
                part[c] += sl + d < S ? other : (VT)0;
            }
        }
        if (sl == 0) s_part[slot] = part;
        __syncthreads();
        if (group != 0) return;
        for (int g = S; g < G; g += S) part += s_part[g * LR + jl];
        if (continued) store(carry + (int64_t)blockIdx.x * N + col, part, false);
        else store(C + (rowid ? (int64_t)rowid[lo] : lo) * ldc + col, part, accumulate);
        return;
    }
    spmi_rows_of_entries<kThreads, T / kThreads>([=](int64_t r) { return (int64_t)pos[r]; }, rowid, lo, last, s, e, s_row, s_wave, at);
    auto keep_head = [&]() {
        if (!kNarrow) { s_part[slot] = sum.value(acc); return; }
        const spmi_pair<VT, V> done = sum.pair(acc);
        s_part[slot] = done.half(0);
        head_lo = done.half(1);
    };
    CT row = 0;
    bool head = false;                                               // the row being added up began before this run
    if (first < end) {
        row = s_row[group];
        head = group == 0 ? continued : s_row[(run - 1) * P + group - 1] == row;
    }
    const int mine = end - first, last_w = (mine - 1) * P + group;   // entries of this run, where the last one is kept
    for (int k = 0; k < mine; k += U) {
        VT v[U];
        vec_t bv[U];
        CT rw[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int next = (k + u) * P + group, w = next < last_w ? next : last_w;
            rw[u] = s_row[w];
            v[u] = s_val[w];
            bv[u] = *(const mem_vec_t *)(Bb + (s_off[w] + colb));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (k + u < mine) {
                if (rw[u] != row) {
                    if (head) keep_head();
                    else store(C + (int64_t)row * ldc + col, sum.value(acc), accumulate);
                    head = false;
                    row = rw[u];
                    acc = (vec_t)(0);
                    sum.clear();
                }
                acc += v[u] * bv[u];
            }
        }
        if (k + U < mine) {
            sum.add(acc);
            acc = (vec_t)(0);
        }
    }
    if (head) keep_head();                                           // the whole run belongs to a row that began before it
    // The sums of a row that fills whole runs are added up towards the first of them, over twice as many groups each step.
    const int full = (ne + run - 1) / run;                           // groups that took something
    const bool whole_runs = __syncthreads_or(head);
    if (kNarrow) {                                                   // the values of the window have been read
        if (group < G) s_lo[slot] = head_lo;
        __syncthreads();
    }
    auto part_of = [&](int at_slot) { return spmi_pair<VT, V>::from(s_part[at_slot], s_lo[at_slot]); };      // kNarrow
    if (whole_runs)
        for (int d = 1; d < full; d <<= 1) {
            const bool take = group + d < full && s_row[group + d] == s_row[group];      // rows ascend: everything between is that row's too
            const vec_t other = take ? s_part[slot + d * LR] : (vec_t)(0), other_lo = take && kNarrow ? s_lo[slot + d * LR] : (vec_t)(0);
            __syncthreads();
            if (take && kNarrow) {
                spmi_pair<VT, V> part = part_of(slot);
                part.add(spmi_pair<VT, V>::from(other, other_lo));
                s_part[slot] = part.half(0);
                s_lo[slot] = part.half(1);
            } else if (take) s_part[slot] += other;
            __syncthreads();
        }
    if (first >= end) return;
    if (group == 0 && continued) store(carry + (int64_t)blockIdx.x * N + col, kNarrow ? part_of(slot).value() : s_part[slot], false);
    if (!head) {
        const bool more = group + 1 < full && s_row[group + 1] == row;
        if (kNarrow) {
            spmi_pair<VT, V> all = sum.pair(acc);
            if (more) all.add(part_of(slot + LR));
            acc = all.value();
        } else {
            acc = sum.value(acc);
            if (more) acc += s_part[slot + LR];
        }
        store(C + (int64_t)row * ldc + col, acc, accumulate);
    }
}

// The same product with a wave per row of the window, for even rows of medium length (see spmm_windows_launch): block w owns
// the entries [w*T, (w+1)*T), its four waves take the rows that meet the window in turn, LR lanes (a power of two) across a row of
// B and 64 / LR entries side by side, their sums meet in a shuffle tree.  No rows to tell apart inside a run and neighbouring
// entries asked for together; but a wave with a long row keeps the block.
// The window's values and, instead of its coordinates, the byte offsets of the rows of B that they select (OT: 32 bits
// when B is below 4 GB) are first copied into LDS with coalesced loads: the loop over the entries then works on small
// window-relative integers and every gather address is a wave-uniform base plus a lane offset.
template <typename PT, typename CT, typename VT, int LR, typename OT>
__global__ __launch_bounds__(kThreads) void spmm_windows_vec_kernel(const PT *__restrict__ pos, const CT *__restrict__ crd,
                                                                    const VT *__restrict__ val, const CT *__restrict__ rowid,
                                                                    const int32_t *__restrict__ rowblk, int64_t nrows, int64_t nnz,
                                                                    const VT *__restrict__ B, int64_t ldb, VT *__restrict__ C, int64_t ldc,
                                                                    VT *__restrict__ carry, int accumulate)
{
    constexpr int V = 16 / sizeof(VT), S = 64 / LR, U = S >= 4 ? 2 : 4;
    typedef VT vec_t __attribute__((ext_vector_type(V)));
    __shared__ OT s_off[kStreamT];
    __shared__ VT s_val[kStreamT];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int jl = lane % LR, sl = lane / LR;
    const int64_t s = (int64_t)blockIdx.x * kStreamT;
    const int64_t e = s + kStreamT < nnz ? s + kStreamT : nnz;
    const int ne = (int)(e - s);
    const OT brow = (OT)(ldb * (int64_t)sizeof(VT));
    for (int i = threadIdx.x; i < ne; i += kThreads) {
        s_off[i] = (OT)crd[s + i] * brow;
        s_val[i] = val[s + i];
    }
    const int64_t lo = rowblk[blockIdx.x], hi = rowblk[blockIdx.x + 1];
    const int64_t last = hi < nrows ? hi : nrows - 1;
    __syncthreads();
    const char *Bb = (const char *)B;
    const OT colb = (OT)(jl * V * (int)sizeof(VT));
    for (int64_t r = lo + wave; r <= last; r += kThreads / 64) {
        const int64_t pa = (int64_t)pos[r], pb = (int64_t)pos[r + 1];
        const int a = (int)((pa > s ? pa : s) - s), b = (int)((pb < e ? pb : e) - s);
        if (r == hi && b <= a) continue;              // row hi starts at the next window: not ours (wave-uniform)
        vec_t accu[U];
#pragma unroll
        for (int u = 0; u < U; ++u) accu[u] = (vec_t)(0);
        for (int p0 = a; p0 < b; p0 += U * S) {       // wave-uniform
            VT v[U];
            vec_t bv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int pp = p0 + sl + u * S;
                const bool in = pp < b;
                const int idx = in ? pp : a;
                v[u] = in ? s_val[idx] : (VT)0;
                bv[u] = *(const vec_t *)(Bb + (s_off[idx] + colb));
                if (!in) bv[u] = (vec_t)(0);          // not 0 * infinity
            }
#pragma unroll
            for (int u = 0; u < U; ++u) accu[u] += v[u] * bv[u];
        }
        vec_t acc = accu[0];
#pragma unroll
        for (int u = 1; u < U; ++u) acc += accu[u];
#pragma unroll
        for (int c = 0; c < V; ++c) {
            VT x = acc[c];
#pragma unroll
            for (int d = 32; d >= LR; d >>= 1) x += __shfl_xor(x, d, 64);
            acc[c] = x;
        }
        if (sl == 0) {
            if (pa < s) *(vec_t *)(carry + (int64_t)blockIdx.x * LR * V + jl * V) = acc;
            else {
                vec_t *dst = (vec_t *)(C + (rowid ? (int64_t)rowid[r] : r) * ldc + jl * V);
                *dst = accumulate ? *dst + acc : acc;
            }
        }
    }
}

// A wave per block boundary: the first boundary a row crosses adds all of that row's carries, in block order.
template <typename PT, typename CT, typename VT>
__global__ __launch_bounds__(kThreads) void spmm_windows_fixup_kernel(const PT *__restrict__ pos, const CT *__restrict__ rowid,
                                                                      const int32_t *__restrict__ rowblk, int64_t nblocks, int64_t N,
                                                                      const VT *__restrict__ carry, VT *__restrict__ C, int64_t ldc)
{
    const int lane = threadIdx.x & 63;
    const int64_t b = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6) + 1;
    if (b >= nblocks) return;
    const int64_t r = rowblk[b];
    const int64_t start = (int64_t)pos[r];
    if (start >= b * kStreamT || start < (b - 1) * kStreamT) return;   // not crossed here, or crossed earlier already
    const int64_t row = rowid ? (int64_t)rowid[r] : r;
    // the blocks whose window begins inside the row: 64 of them looked at a time
    int64_t stop = b;
    for (uint64_t same = ~(uint64_t)0; same == ~(uint64_t)0; ) {
        const int64_t bb = stop + lane;
        same = __ballot(bb < nblocks && rowblk[bb < nblocks ? bb : nblocks] == r);
        stop += same == ~(uint64_t)0 ? 64 : __builtin_ctzll(~same);
    }
    for (int64_t j = lane; j < N; j += 64) {
        VT sum = 0;
        int64_t bb = b;
        for (; bb + 4 <= stop; bb += 4) {
            const VT c0 = carry[bb * N + j], c1 = carry[(bb + 1) * N + j], c2 = carry[(bb + 2) * N + j], c3 = carry[(bb + 3) * N + j];
            sum = (((sum + c0) + c1) + c2) + c3;
        }
        for (; bb < stop; ++bb) sum += carry[bb * N + j];
        C[row * ldc + j] += sum;
    }
}

// ---- column-major storage: a wave per stored column, atomic adds into C ------------------
template <typename PT, typename CT, typename VT, int CG>
__global__ __launch_bounds__(kThreads) void spmm_scatter_kernel(const PT *__restrict__ pos, const CT *__restrict__ crd,
                                                                const VT *__restrict__ val, const CT *__restrict__ colid, int64_t ncols,
                                                                const VT *__restrict__ B, int64_t N, int64_t ldb, VT *__restrict__ C,
                                                                int64_t ldc)
{
    constexpr int S = 64 / CG;
    const int lane = threadIdx.x & 63;
    const int64_t q = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (q >= ncols) return;
    const int jl = lane % CG, sl = lane / CG;
    const int64_t a = (int64_t)pos[q], b = (int64_t)pos[q + 1];
    if (a == b) return;
    const int64_t k = colid ? (int64_t)colid[q] : q;
    for (int64_t j0 = 0; j0 < N; j0 += CG) {
        const int64_t j = j0 + jl;
        if (j >= N) continue;
        const VT bj = B[k * ldb + j];
        for (int64_t p = a + sl; p < b; p += S) unsafeAtomicAdd(&C[(int64_t)crd[p] * ldc + j], val[p] * bj);
    }
}

// ---- dense innermost level (the paper's compressed-then-dense format of Section 4.1 and the all-dense one) ----
// Row-major: stored row q holds all `n` values of matrix row rowid[q] (or q).  A block per stored row: lanes
// stride over the row with coalesced loads, LG lanes side by side per tile of CG columns of B.
template <typename CT, typename VT, int CG>
__global__ __launch_bounds__(kThreads) void dense_rows_kernel(const VT *__restrict__ val, const CT *__restrict__ rowid, int64_t n,
                                                              const VT *__restrict__ B, int64_t N, int64_t ldb, VT *__restrict__ C,
                                                              int64_t ldc, int accumulate)
{
    constexpr int KS = kThreads / CG;                 // entries of the row handled side by side
    __shared__ VT red[kThreads];
    const int64_t q = blockIdx.x;
    const int jl = threadIdx.x % CG, kl = threadIdx.x / CG;
    const VT *__restrict__ vrow = val + q * n;
    const int64_t row = rowid ? (int64_t)rowid[q] : q;
    for (int64_t j0 = 0; j0 < N; j0 += CG) {
        const int64_t j = j0 + jl;
        VT acc = 0;
        if (j < N)
            for (int64_t k = kl; k < n; k += KS) acc += vrow[k] * B[k * ldb + j];
        red[threadIdx.x] = acc;
        __syncthreads();
        for (int stride = kThreads / 2; stride >= CG; stride >>= 1) {
            if (threadIdx.x < stride) red[threadIdx.x] += red[threadIdx.x + stride];
            __syncthreads();
        }
        if (kl == 0 && j < N) C[row * ldc + j] = accumulate ? C[row * ldc + j] + red[jl] : red[jl];
        __syncthreads();
    }
}

// Column-major: stored column q holds all `m` values of matrix column colid[q] (or q): C[i, j] = sum_q V[q, i] * B[col_q, j].
// A thread per (i, j); every row of C is written, so no zero fill is needed and no atomics either.
template <typename CT, typename VT, int CG>
__global__ __launch_bounds__(kThreads) void dense_cols_kernel(const VT *__restrict__ val, const CT *__restrict__ colid, int64_t ncols,
                                                              int64_t m, const VT *__restrict__ B, int64_t N, int64_t ldb,
                                                              VT *__restrict__ C, int64_t ldc, int accumulate)
{
    constexpr int IS = kThreads / CG;                 // rows of C per block
    const int jl = threadIdx.x % CG;
    const int64_t i = (int64_t)blockIdx.x * IS + threadIdx.x / CG;
    if (i >= m) return;
    for (int64_t j0 = 0; j0 < N; j0 += CG) {
        const int64_t j = j0 + jl;
        if (j >= N) continue;
        VT acc = accumulate ? C[i * ldc + j] : (VT)0;
        for (int64_t q = 0; q < ncols; ++q) {
            const int64_t k = colid ? (int64_t)colid[q] : q;
            acc += val[q * m + i] * B[k * ldb + j];
        }
        C[i * ldc + j] = acc;
    }
}

// Row-major dense innermost level, one column (y = A.x with fully stored rows): pure streaming.  Block (c, q) takes
// 2048 consecutive values of stored row q with 16-byte loads and leaves one partial sum; a second small kernel adds
// the partial sums of a row in order (deterministic) and writes y.
constexpr int kDenseChunk = kThreads * 8;
template <typename VT>
__global__ __launch_bounds__(kThreads) void dense_rows_spmv_partial_kernel(const VT *__restrict__ val, int64_t n, const VT *__restrict__ x,
                                                                           int64_t nchunks, VT *__restrict__ partial)
{
    constexpr int V = 16 / sizeof(VT);                // elements per 16-byte load
    typedef VT vec_t __attribute__((ext_vector_type(V)));
    __shared__ VT wsum[kThreads / 64];
    const int64_t q = blockIdx.y, c = blockIdx.x;
    const int64_t k0 = c * kDenseChunk;
    const VT *__restrict__ vrow = val + q * n;
    VT acc = 0;
    if (k0 + kDenseChunk <= n) {
        vec_t a[8 / V], b[8 / V];
#pragma unroll
        for (int t = 0; t < 8 / V; ++t) {
            const int64_t k = k0 + (int64_t)(t * kThreads + threadIdx.x) * V;
            a[t] = *(const vec_t *)(vrow + k);
            b[t] = *(const vec_t *)(x + k);
        }
#pragma unroll
        for (int t = 0; t < 8 / V; ++t)
#pragma unroll
            for (int e = 0; e < V; ++e) acc += a[t][e] * b[t][e];
    } else {
        for (int64_t k = k0 + threadIdx.x; k < n; k += kThreads) acc += vrow[k] * x[k];
    }
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        VT tot = 0;
        for (int w = 0; w < kThreads / 64; ++w) tot += wsum[w];
        partial[q * nchunks + c] = tot;
    }
}

template <typename CT, typename VT>
__global__ __launch_bounds__(kThreads) void dense_rows_spmv_finish_kernel(const VT *__restrict__ partial, int64_t nchunks, const CT *__restrict__ rowid,
                                                                          int64_t nstored, VT *__restrict__ y, int64_t ldc, int accumulate)
{
    const int64_t q = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (q >= nstored) return;
    VT sum = 0;
    for (int64_t c = 0; c < nchunks; ++c) sum += partial[q * nchunks + c];
    const int64_t row = rowid ? (int64_t)rowid[q] : q;
    y[row * ldc] = accumulate ? y[row * ldc] + sum : sum;
}

inline unsigned grid_for(int64_t n, int64_t per_block) { return (unsigned)(n > 0 ? ceil_div(n, per_block) : 1); }

template <typename PT, typename CT, typename VT>
sp_status zero_c(VT *C, int64_t m, int64_t N, int64_t ldc, hipStream_t st)
{
    if (m * N == 0) return SP_OK;
    const int64_t nb = ceil_div(m * N, kThreads);
    hipLaunchKernelGGL(zero_matrix_kernel<VT>, dim3((unsigned)(nb < 16384 ? nb : 16384)), dim3(kThreads), 0, st, C, m, N, ldc);
    SP_HIP(hipGetLastError());
    return SP_OK;
}

// Which stored rows a product walks: all positions of the outer level, or only the stored / non-empty ones through a row-id list
// (a compressed outer level, or a dense one that is mostly empty and therefore carries the list of its non-empty rows).
template <typename PT, typename CT>
struct row_view {
    const PT *pos; const CT *rowid; int64_t nrows; const sp_rowblocks *rowblocks; bool dcsr;
    explicit row_view(const sp_tensor *A)
    {
        pos = (const PT *)A->pos[1];
        dcsr = A->enc.lt[0] == SP_COMPRESSED;
        rowid = dcsr ? (const CT *)A->crd[0] : nullptr;
        nrows = A->npos[1] - 1;
        rowblocks = &A->rowblocks;
        if (!dcsr && A->nz_pos) {
            dcsr = true;
            pos = (const PT *)A->nz_pos; rowid = (const CT *)A->nz_rowid; nrows = A->nz_rows; rowblocks = &A->nz_rowblocks;
        }
    }
};

// The SpMM cut by stored entries plus its fix-up, with the per-block carries in `carry` (room for N values per block).
// N >= 2.
template <typename PT, typename CT, typename VT>
sp_status spmm_windows_launch(const sp_tensor *A, const row_view<PT, CT> &rv, const VT *B, int64_t N, int64_t ldb, VT *C, int64_t ldc,
                              int accumulate, VT *carry, hipStream_t st)
{
    constexpr int V = 16 / sizeof(VT);
    const PT *pos = rv.pos;
    const CT *crd = (const CT *)A->crd[1];
    const VT *val = (const VT *)A->values;
    const CT *rowid = rv.rowid;
    const int64_t nrows = rv.nrows, nnz = A->ncrd[1];
    const sp_rowblocks *rowblocks = rv.rowblocks;
    const int64_t nb = rowblocks->nblocks;
    const bool small = sizeof(CT) == 4 && (uint64_t)A->shape[1] * (uint64_t)ldb * sizeof(VT) < ((uint64_t)1 << 32);     // 32-bit byte offsets into B (64-bit coordinates keep 64-bit offsets)
#define SPMI_SPMM_RUNS_O(VV, OT, NARROW)                                                                                      \
    hipLaunchKernelGGL((spmm_runs_kernel<PT, CT, VT, VV, OT, NARROW>), dim3((unsigned)nb, (unsigned)ceil_div(ceil_div(N, VV), lr_tile)), dim3(kThreads), 0, \
                       st, pos, crd, val, rowid, (const int32_t *)rowblocks->start, nrows, nnz, B, N, ldb, lr_tile, C, ldc, carry, accumulate)
#define SPMI_SPMM_RUNS(VV, NARROW)                          \
    do {                                                    \
        if (small) SPMI_SPMM_RUNS_O(VV, uint32_t, NARROW);  \
        else SPMI_SPMM_RUNS_O(VV, uint64_t, NARROW);        \
    } while (0)
    // A wave per row where rows are even and of medium length, and for one or two 16-byte pieces where they are long: there the
    // runs kernel's tables of rows cost more than its balance gives.  4.2 M entries, rows of even length, a wave per row against
    // runs: 64 entries, 4 f32 columns 33 / 38 us, 64 f32 columns 128 / 135; 256 entries, 4 f32 29 / 38, 32 f64 60 / 78; 48 entries,
    // 16 f32 63 / 62; 512 entries, 32 f64 88 / 62.  Lognormal rows of mean 64, 64 f32: 193 / 144.  6 M entries in rows of 20,000, 4 f32: 28 / 34.
    const double mean = (double)nnz / (double)nrows;
    const int64_t lr = N / V;
    const bool one_load = N % V == 0 && ldb % V == 0 && ldc % V == 0 && (uintptr_t)B % 16 == 0 && (uintptr_t)C % 16 == 0 && lr >= 1 && lr <= 64 && (lr & (lr - 1)) == 0;
    const bool wave_per_row = one_load && ((mean >= 96 && lr <= 2) || (mean >= (lr <= 8 ? 56 : 96) && mean < 448 && (double)A->max_segment <= 4 * mean));
#define SPMI_SPMM_WIN_O(LR, OT)                                                                                               \
    hipLaunchKernelGGL((spmm_windows_vec_kernel<PT, CT, VT, LR, OT>), dim3((unsigned)nb), dim3(kThreads), 0, st, pos, crd, val, rowid,    \
                       (const int32_t *)rowblocks->start, nrows, nnz, B, ldb, C, ldc, carry, accumulate)
#define SPMI_SPMM_WIN(LR)                           \
    do {                                            \
        if (small) SPMI_SPMM_WIN_O(LR, uint32_t);   \
        else SPMI_SPMM_WIN_O(LR, uint64_t);         \
    } while (0)
    const int VV = N >= V ? V : 2;                // two or three columns in f32: loads of two
    const int64_t pieces = ceil_div(N, VV);
    // at least 512 blocks where the columns allow: few windows share the columns out among more blocks
    const int64_t split = nb < 512 ? ceil_div(512, nb) : 1;
    const int64_t wanted = ceil_div(pieces, split) > 4 ? ceil_div(pieces, split) : 4;
    const int lr_tile = (int)(wanted < 64 ? wanted : 64);
    if (wave_per_row) {
        if (lr == 1) SPMI_SPMM_WIN(1);
        else if (lr == 2) SPMI_SPMM_WIN(2);
        else if (lr == 4) SPMI_SPMM_WIN(4);
        else if (lr == 8) SPMI_SPMM_WIN(8);
        else if (lr == 16) SPMI_SPMM_WIN(16);
        else if (lr == 32) SPMI_SPMM_WIN(32);
        else SPMI_SPMM_WIN(64);
    } else if (VV == V && pieces <= 2) SPMI_SPMM_RUNS(V, true);
    else if (VV == V) SPMI_SPMM_RUNS(V, false);
    else SPMI_SPMM_RUNS(2, true);                 // f32 only
#undef SPMI_SPMM_RUNS
#undef SPMI_SPMM_RUNS_O
#undef SPMI_SPMM_WIN
#undef SPMI_SPMM_WIN_O
    SP_HIP(hipGetLastError());
    if (nb > 1) {
        hipLaunchKernelGGL((spmm_windows_fixup_kernel<PT, CT, VT>), dim3(grid_for(nb - 1, kThreads / 64)), dim3(kThreads), 0, st, pos,
                           rowid, (const int32_t *)rowblocks->start, nb, N, (const VT *)carry, C, ldc);
        SP_HIP(hipGetLastError());
    }
    return SP_OK;
}

// What the binned kernel's second pass needs for its heaviest row block, in microseconds (out: bits of a float, zero before): a row
// block is one workgroup's, and products of one row that meet in a wave add to one address of the LDS one after the other.  Per thousand
// products 0.25, and 0.17 more for every doubling of the lanes that a bucket's products of a row fill (a lane takes eight): f32,
// 3 M entries in 200,000 rows of 2 M columns, with one row of 990,000: 1256 us (one of 9000: 26; 20 side by side of 20,000: 317; none: 18).
template <typename PT>
__global__ __launch_bounds__(kThreads) void spmv_bins_peak_kernel(const PT *__restrict__ pos, int64_t nrows, int rshift, float lanes_per_product,
                                                                  unsigned *__restrict__ out)
{
    __shared__ float wsum[kThreads / 64];
    const int64_t r0 = (int64_t)blockIdx.x << rshift, r1 = r0 + ((int64_t)1 << rshift) < nrows ? r0 + ((int64_t)1 << rshift) : nrows;
    float us = 0;
    for (int64_t r = r0 + threadIdx.x; r < r1; r += kThreads) {
        const float len = (float)(pos[r + 1] - pos[r]);
        us += 1e-3f * len * (0.25f + 0.17f * __log2f(fminf(fmaxf(len * lanes_per_product, 1.0f), 64.0f)));
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) us += __shfl_xor(us, d, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = us;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kThreads / 64; ++w) us += wsum[w];
        atomicMax(out, __float_as_uint(us));              // positive floats are ordered as their bits are
    }
}

template <typename PT>
sp_status spmv_bins_peak(const sp_tensor *A, const PT *pos, int64_t nrows, int rshift, int64_t panels, hipStream_t st, double *us)
{
    sp_mem mem{A->alloc, A->free_, A->ctx};
    sp_scratch tmp(mem);
    unsigned *out = (unsigned *)tmp.get(64);
    if (!out) return SP_ERR_ALLOC;
    SP_TRY(spmi_fill_zero(out, 64, st));
    hipLaunchKernelGGL(spmv_bins_peak_kernel<PT>, dim3((unsigned)ceil_div(nrows, (int64_t)1 << rshift)), dim3(kThreads), 0, st, pos, nrows, rshift,
                       (float)(1.0 / (8.0 * (double)panels)), out);
    SP_HIP(hipGetLastError());
    float h = 0;
    SP_HIP(hipMemcpyAsync(&h, out, 4, hipMemcpyDeviceToHost, st));
    SP_HIP(hipStreamSynchronize(st));
    *us = (double)h;
    return SP_OK;
}

// The inspector step of the matrix-times-vector product (Section 6.2): decides which SpMV kernel the tensor's products run
// and builds the regrouped copy that kernel reads.  Measures once how scattered the columns are (one pass over crd, one
// synchronisation), may allocate through the tensor's allocator.  The decision is kept in A->plan_spmv.  A kernel chosen here
// gives way to one that needs less where its copy cannot be had (the streamed kernel needs none); one that was asked for does not.
// unprepared: a product comes without sp_prepare before it.  Then matrices of fewer than two million entries, and those whose
// binned copy would be small or sparsely filled, take the streamed kernel as they are: a copy costs more than it saves in ten
// products (1.5 M entries, 100,000 rows of 3 M columns: 46 us for the first product, 349 with the copy; 8 M in 400,000 rows, DCSR: 218 and
// 475), and the smaller ones ask nothing of the device, so that their products can be recorded.  A later sp_prepare decides for
// all products after it.
template <typename PT, typename CT, typename VT>
sp_status prepare_spmv_t(const sp_tensor *A, hipStream_t st, bool unprepared)
{
    if (A->plan_spmv && (unprepared || !A->plan_spmv_open)) return SP_OK;
    A->plan_spmv = A->plan_spmv_open = 0;
    const row_view<PT, CT> rv(A);
    const int64_t nnz = A->ncrd[1], nrows = rv.nrows;
    int kernel = A->tune_spmv;
    const bool fixed = kernel != 0;
    if (kernel == 0) {
        // small and even (no row beyond one wave's stride): one launch of the rows kernel beats stream + fix-up
        const bool small_even = nnz < ((int64_t)1 << 18) && A->max_segment <= 64;
        kernel = (rv.rowblocks->start && nnz >= 8 * kStreamT && !small_even) ? 2 : 1;
        // A large matrix whose gathers are scattered over a large x: no gather should leave the chip's caches.  The binned copy keeps
        // them inside the LDS, L2-sized column panels inside the L2.  Gathers that mostly fall into the line of their predecessor
        // stay as they are.
        const double xbytes = (double)A->shape[1] * sizeof(VT);
        const bool large = nnz >= ((int64_t)1 << 21), segments = !rv.dcsr && nnz >= ((int64_t)1 << 22);
        const bool candidate = kernel == 2 && nnz >= ((int64_t)1 << 20) && xbytes > (double)(3 << 20);
        if (candidate && unprepared && !large) A->plan_spmv_open = 1;
        else if (candidate) {
            double share = 0;
            const sp_status sc = spmi_column_scatter(A, st, &share);
            if (sc != SP_OK && sc != SP_ERR_ALLOC) return sc;
            const int64_t panels = ceil_div(A->shape[1], (int64_t)kBinPW);
            const int rshift = spmi_bin_row_shift(nnz, nrows, panels);
            const int64_t rowblocks = ceil_div(nrows, (int64_t)1 << rshift);
            const double buckets = (double)panels * (double)rowblocks;
            // buckets of 32 entries, a row block for every CU: where the binned copy saves most
            const bool full_bins = large && (double)nnz >= 32.0 * buckets && nrows > 255 * (int64_t)kBinRB;
            // Microseconds, fitted to measurements in
            // f64 over 0.3 to 16 M entries, 9,000 to 3 M rows and x of 4 to 64 MB (most within a sixth):
            //   streamed: a cache line from beyond the L2 per entry that misses it, and the rows to be cleared
            //   panels:   5.4 per million entries, 6.9 per million (row, panel) pairs
            //   binned:   x and 18.5 bytes per entry (buckets padded to eights), then 10 bytes per entry or the heaviest
            //             row block, which is at least the mean one
            // profiles/spmv_choice_measurements.txt has 30 matrices.  Measured (by the formula): f64, 3 M entries in 200,000 rows of 2 M columns 51 us (54) streamed, 22 (25) binned; 16 M in 1 M rows
            // of 4 M columns 278 (296), 90 (104) and 205 (200) by panels; the same sorted by length, rows of up to 300, f32: 226 (236), 140 (152)
            // and 112 (200).
            const double M = 1e-6 * (double)nnz, v = (double)sizeof(VT) / 8.0, clear = rv.dcsr ? 1.6e-7 * (double)A->shape[0] * sizeof(VT) : 0.0;
            const double padded = M + 1e-6 * std::min(3.5 * buckets, 7.0 * (double)nnz);
            const double streamed = 5.0 + M * (5.5 + 14.5 * (1.0 - (double)(4 << 20) / std::max(xbytes, (double)(4 << 20)))) + clear;
            const double paneled = segments ? 3.0 + 5.4 * M + 6.9e-6 * (double)nrows * std::ceil(xbytes / (double)kSpmvSliceBytes) : 1e30;
            const double others = std::min(streamed, large ? paneled : streamed);
            auto binned = [&](double peak) {
                return 4.0 + 2e-7 * xbytes + padded * (1.0 + 2.8 * v) + 0.6 * clear + std::max(padded * (0.3 + 1.5 * v), 2.0 + peak);
            };
            const double peak = 250.0 * padded / (double)rowblocks;
            double limit = 0.9 * others;
            if (share >= 0.5 && unprepared && !full_bins && !segments) A->plan_spmv_open = 1;
            else if (share >= 0.5 && full_bins) {
                // as long as no row block is far heavier than the mean one: f64, 16.9 M entries in 1 M rows of 524,288 columns, rows of up to
                // 4754, the heaviest block 1.3 times the mean: 128 us, streamed 156; sorted by length, 13 times the mean: 87 and 54.  The
                // streamed kernel misses an x of 3 to 4 MB too (16 M even entries, 400,000 columns: 146 us, binned 123), which the formula leaves out.
                kernel = 4;
                limit = std::max(others, 1.5 * binned(peak));
            } else if (share >= 0.5 && sizeof(VT) == 8 && A->max_segment > kLongRow) {
                // long rows in f64: the binned copy's second pass adds a quarter of a row's products one by one, where the others add them
                // up in trees; it is left to the shapes above
                kernel = segments ? 3 : 2;
            } else if (share >= 0.5) {
                // Short rows are added up one by one in the other kernels, in four parts in the binned one (f32: in f64), which is no less exact
                // there: whichever is the fastest.
                if (large && paneled < streamed) kernel = 3;
                if (binned(peak) < limit) kernel = 4;
            }
            // no row block holds more than its rows of the longest length: often that answers it without asking the device
            const double most = std::min((double)nnz, (double)A->max_segment * (double)((int64_t)1 << rshift));
            const double lanes = std::min(std::max((double)A->max_segment / (8.0 * (double)panels), 1.0), 64.0);
            if (kernel == 4 && binned(std::max(peak, 1e-3 * most * (0.25 + 0.17 * std::log2(lanes)))) >= limit) {
                double heaviest = 0;
                const sp_status sh = spmv_bins_peak<PT>(A, rv.pos, nrows, rshift, panels, st, &heaviest);
                if (sh != SP_OK && sh != SP_ERR_ALLOC) return sh;
                if (binned(std::max(peak, heaviest)) >= limit) kernel = large && paneled < streamed ? 3 : 2;
            }
        }
    }
    if (kernel == 4) {
        const sp_status sb = spmi_build_bins(A, st);
        if ((sb == SP_ERR_UNSUPPORTED || sb == SP_ERR_ALLOC) && !fixed) kernel = (!rv.dcsr && nnz >= ((int64_t)1 << 22)) ? 3 : 2;
        else if (sb != SP_OK) return sb;
    }
    if (kernel == 3) {
        if (A->enc.lt[0] == SP_COMPRESSED) return SP_ERR_UNSUPPORTED;
        const sp_status sb = spmi_build_segments(A, sizeof(VT), kSpmvSliceBytes, st);
        if ((sb == SP_ERR_UNSUPPORTED || sb == SP_ERR_ALLOC) && !fixed) kernel = 2;
        else if (sb != SP_OK) return sb;
    }
    if (kernel == 2 && !rv.rowblocks->start) return SP_ERR_UNSUPPORTED;
    A->plan_spmv = kernel;
    return SP_OK;
}

// Scratch of the SpMM cut by stored entries: one row of N values per block for every part of sp_spmm_carry, kept by the tensor
// and made larger on demand.
template <typename PT, typename CT, typename VT>
sp_status prepare_spmm_t(const sp_tensor *A, int64_t N, hipStream_t st)
{
    const row_view<PT, CT> rv(A);
    if (!rv.rowblocks->start || A->tune_spmm == 1 || A->tune_spmm == 2) return SP_OK;
    sp_spmm_carry &c = A->spmm_carry;
    if (c.columns >= N) return SP_OK;
    constexpr int64_t V = 16 / sizeof(VT);
    const size_t column = (size_t)rv.rowblocks->nblocks * sizeof(VT);
    const size_t whole = (column * (size_t)(N < 64 * V ? N : 64 * V) + 255) & ~(size_t)255, any = (column * (size_t)N + 255) & ~(size_t)255;
    c.mem.shared |= c.used[0] && c.user[0] != st;
    c.columns = 0;
    c.used[0] = c.used[1] = false;
    SP_TRY(spmi_reserve(A, c.mem, whole + 2 * any, st));
    c.offset[0] = 0; c.offset[1] = whole; c.offset[2] = whole + any;
    c.columns = N;
    return SP_OK;
}

// May a product on this stream, or in this recording, use part 1 or 2 of the scratch?  Part 1 goes to another stream once its
// user has nothing left to do; a graph keeps part 2.
bool spmm_part_is_ours(const sp_spmm_carry &c, int part, hipStream_t st, unsigned long long graph)
{
    const bool same = c.used[part - 1] && c.user[part - 1] == st;
    if (part == 1) return !c.used[0] || same || spmi_idle(c.user[0]);
    return graph != 0 && (!c.used[1] || (same && c.graph == graph));
}

template <typename PT, typename CT, typename VT>
sp_status prepare_rowmajor_t(const sp_tensor *A, const VT *, int64_t N, int64_t, VT *, int64_t, int, hipStream_t st)
{
    if (A->npos[1] - 1 <= 0) return SP_OK;
    if (N == 1) return prepare_spmv_t<PT, CT, VT>(A, st, false);
    return prepare_spmm_t<PT, CT, VT>(A, N, st);
}

template <typename PT, typename CT, typename VT>
sp_status rowmajor_t(const sp_tensor *A, const VT *B, int64_t N, int64_t ldb, VT *C, int64_t ldc, int accumulate, hipStream_t st)
{
    const row_view<PT, CT> rv(A);
    const PT *pos = rv.pos;
    const CT *crd = (const CT *)A->crd[1];
    const VT *val = (const VT *)A->values;
    const bool dcsr = rv.dcsr;
    const CT *rowid = rv.rowid;
    const int64_t nrows = rv.nrows;              // stored rows
    const sp_rowblocks *rowblocks = rv.rowblocks;
    const int64_t m = A->shape[0];
    const int64_t nnz = A->ncrd[1];
    if (N == 1 && nrows > 0 && !A->plan_spmv) {  // no sp_prepare before this product: the inspector runs now (may allocate and synchronise)
        ++A->lazy_prepares;
        SP_TRY((prepare_spmv_t<PT, CT, VT>(A, st, true)));
    }
    // rows that are not stored become zero; the first pass of the binned kernel does that on the way
    const bool clears = dcsr && !accumulate && N == 1 && nrows > 0 && A->plan_spmv == 4 && ldc == 1;
    if (dcsr && !accumulate && !clears) SP_TRY((zero_c<PT, CT, VT>(C, m, N, ldc, st)));
    if (nrows == 0) return SP_OK;
    if (N == 1) {
        const int kernel = A->plan_spmv;
        if (kernel == 3) {
            // the segmented copy is an ordinary CSR over panels*nrows virtual rows: stream it into the per-panel
            // partial vector (consecutive blocks gather from the same <= 2 MB slice of x), then add the panels up
            const sp_segments *g = A->segments;
            const sp_tensor *S = g->seg;
            int64_t vrows = (int64_t)g->panels * g->nrows;
            const PT *spos = (const PT *)S->pos[1];
            const CT *srowid = nullptr;
            const sp_rowblocks *srb = &S->rowblocks;
            if (S->nz_pos) {          // long runs of empty virtual rows (an empty panel): only the others are visited
                SP_TRY((zero_c<PT, CT, VT>((VT *)g->partial, vrows, 1, 1, st)));
                spos = (const PT *)S->nz_pos; srowid = (const CT *)S->nz_rowid; srb = &S->nz_rowblocks; vrows = S->nz_rows;
            }
            const int64_t nb = srb->nblocks;
            sp_prof_scope prof(A, st);
            hipLaunchKernelGGL((spmv_stream_kernel<PT, CT, VT>), dim3((unsigned)nb), dim3(kST), 0, st, spos,
                               (const CT *)S->crd[1], (const VT *)S->values, srowid, (const int32_t *)srb->start,
                               vrows, S->ncrd[1], B, ldb, (VT *)g->partial, (int64_t)1, (VT *)srb->carry, 0);
            SP_HIP(hipGetLastError());
            if (nb > 1) {
                hipLaunchKernelGGL((spmv_stream_fixup_kernel<PT, CT, VT>), dim3(grid_for(nb - 1, kThreads)), dim3(kThreads), 0, st,
                                   spos, srowid, (const int32_t *)srb->start, nb, (const VT *)srb->carry, (VT *)g->partial, (int64_t)1);
                SP_HIP(hipGetLastError());
            }
            hipLaunchKernelGGL((spmv_panel_sum_kernel<VT>), dim3(grid_for(g->nrows, kThreads)), dim3(kThreads), 0, st,
                               (const VT *)g->partial, g->nrows, g->panels, C, ldc, accumulate);
            SP_HIP(hipGetLastError());
            return SP_OK;
        }
        if (kernel == 4) {
            const sp_bins *g = A->bins;                                       // over the same stored rows as pos / rowid here
            sp_prof_scope prof(A, st);
            hipLaunchKernelGGL((spmv_bins_multiply_kernel<VT>), dim3((unsigned)(ceil_div(g->panels, 8) * 8 * g->pieces + (clears ? ceil_div(m, kBinClear) : 0))),
                               dim3(kBinThreads), 0, st, (const VT *)g->val, (const uint16_t *)g->lcol, (const uint32_t *)g->gdst, (const int64_t *)g->pstart,
                               g->panels, g->pieces, A->shape[1], B, ldb, (VT *)g->prod, C, m);
            SP_HIP(hipGetLastError());
            hipLaunchKernelGGL((spmv_bins_reduce_kernel<CT, VT>), dim3((unsigned)g->rowblocks), dim3(kBinThreads), 0, st, (const VT *)g->prod,
                               (const uint16_t *)g->lrow, (const int64_t *)g->rbstart, g->rshift, g->nrows, rowid, C, ldc, accumulate);
            SP_HIP(hipGetLastError());
            return SP_OK;
        }
        if (kernel == 2) {
            const int64_t nb = rowblocks->nblocks;
            {
            sp_prof_scope prof(A, st);
            hipLaunchKernelGGL((spmv_stream_kernel<PT, CT, VT>), dim3((unsigned)nb), dim3(kST), 0, st, pos, crd, val, rowid,
                               (const int32_t *)rowblocks->start, nrows, nnz, B, ldb, C, ldc, (VT *)rowblocks->carry, accumulate);
            }
            SP_HIP(hipGetLastError());
            if (nb > 1) {
                hipLaunchKernelGGL((spmv_stream_fixup_kernel<PT, CT, VT>), dim3(grid_for(nb - 1, kThreads)), dim3(kThreads), 0, st, pos,
                                   rowid, (const int32_t *)rowblocks->start, nb, (const VT *)rowblocks->carry, C, ldc);
                SP_HIP(hipGetLastError());
            }
            return SP_OK;
        }
        const double avg = (double)nnz / (double)nrows;
        sp_prof_scope prof(A, st);
#define SPMI_ROWS(G)                                                                                                          \
    hipLaunchKernelGGL((spmv_rows_kernel<PT, CT, VT, G>), dim3(grid_for(nrows * G, kThreads)), dim3(kThreads), 0, st, pos, crd, \
                       val, rowid, nrows, B, ldb, C, ldc, accumulate)
        if (avg <= 3) SPMI_ROWS(2);
        else if (avg <= 6) SPMI_ROWS(4);
        else if (avg <= 12) SPMI_ROWS(8);
        else if (avg <= 24) SPMI_ROWS(16);
        else if (avg <= 48) SPMI_ROWS(32);
        else SPMI_ROWS(64);
#undef SPMI_ROWS
        SP_HIP(hipGetLastError());
        return SP_OK;
    }
    // Tried and dropped (measured on the 1M x 1M matrix times a 1M x 64 operand): one launch per column panel of the
    // segmented copy, so that the slice of B a launch gathers from fits the 256 MB last-level cache.  Re-reading and
    // re-writing C once per panel costs more than the gathers save: 3.17 ms against 2.94 ms.
    sp_prof_scope prof(A, st);
    {
        constexpr int64_t V = 16 / sizeof(VT);
        const int64_t lr = N / V;
        const bool aligned = N % V == 0 && ldb % V == 0 && ldc % V == 0 && (uintptr_t)B % 16 == 0 && (uintptr_t)C % 16 == 0;
        const bool fits = aligned && (lr == 1 || lr == 2 || lr == 4 || lr == 8 || lr == 16 || lr == 32 || lr == 64);    // a wave per row
        const bool fits_any = aligned && lr >= 1 && lr <= 64;                                                           // cut by entries
        if (A->tune_spmm == 2 && !fits) return SP_ERR_UNSUPPORTED;
        if (A->tune_spmm == 3 && (!fits_any || !rowblocks->start)) return SP_ERR_UNSUPPORTED;
        // Cut by entries is faster than a wave per row from some 10^5 entries on, whatever the width and the row lengths (300,000
        // entries, 20,000 skewed rows, f64: 14 against 29 us with 5 columns, 30 against 413 us with 64).  A smaller product
        // is its second launch (20,000 entries: 12 against 8 us), unless a wave walks a long row in many steps: widths that
        // have no 16-byte kernel keep the single launch up to twelve steps.
        const int64_t cg = N > 32 ? 64 * ceil_div(N, 64) * 2 : N > 16 ? 32 : N > 8 ? 16 : N > 4 ? 8 : 4;       // lanes of a wave per entry there
        const bool tiny = !fits_any && nnz < ((int64_t)1 << 17) && A->max_segment * cg <= 256 * 12;
        const bool by_entries = A->tune_spmm == 3 || (A->tune_spmm == 0 && rowblocks->start && !tiny && N / (64 * V) < 65535);      // a grid's y
        if (by_entries) {
            // a product that the wave-per-row kernel can also do goes there when there is no scratch to be had
            sp_spmm_carry &c = A->spmm_carry;
            unsigned long long graph = 0;
            const bool recording = spmi_recording(st, &graph);
            const int part = fits_any ? 0 : recording ? 2 : 1;
            bool scratch = part == 0 || spmm_part_is_ours(c, part, st, graph);
            if (scratch && c.columns < N) {      // no sp_prepare for this many columns: the scratch is made now
                scratch = false;
                if (part != 2) {
                    ++A->lazy_prepares;
                    const sp_status made = prepare_spmm_t<PT, CT, VT>(A, N, st);
                    if (made != SP_OK && (part == 0 || made != SP_ERR_ALLOC)) return made;
                    scratch = made == SP_OK;
                }
            }
            if (scratch) {
                if (part > 0) { c.user[part - 1] = st; c.used[part - 1] = true; }
                if (part == 2) c.graph = graph;
                c.mem.shared |= recording;
                return spmm_windows_launch<PT, CT, VT>(A, rv, B, N, ldb, C, ldc, accumulate, (VT *)((char *)c.mem.ptr + c.offset[part]), st);
            }
        }
        if (fits && A->tune_spmm != 1) {
#define SPMI_SPMM_VEC(LR)                                                                                                     \
    hipLaunchKernelGGL((spmm_rows_vec_kernel<PT, CT, VT, LR>), dim3(grid_for(nrows, kThreads / 64)), dim3(kThreads), 0, st, pos, \
                       crd, val, rowid, nrows, B, ldb, C, ldc, accumulate)
            if (lr == 1) SPMI_SPMM_VEC(1);
            else if (lr == 2) SPMI_SPMM_VEC(2);
            else if (lr == 4) SPMI_SPMM_VEC(4);
            else if (lr == 8) SPMI_SPMM_VEC(8);
            else if (lr == 16) SPMI_SPMM_VEC(16);
            else if (lr == 32) SPMI_SPMM_VEC(32);
            else SPMI_SPMM_VEC(64);
#undef SPMI_SPMM_VEC
            SP_HIP(hipGetLastError());
            return SP_OK;
        }
    }
#define SPMI_SPMM(CG)                                                                                                      \
    hipLaunchKernelGGL((spmm_rows_kernel<PT, CT, VT, CG>), dim3(grid_for(nrows, kThreads / 64)), dim3(kThreads), 0, st, pos, crd, \
                       val, rowid, nrows, B, N, ldb, C, ldc, accumulate)
    if (N > 32) SPMI_SPMM(64);
    else if (N > 16) SPMI_SPMM(32);
    else if (N > 8) SPMI_SPMM(16);
    else if (N > 4) SPMI_SPMM(8);
    else SPMI_SPMM(4);
#undef SPMI_SPMM
    SP_HIP(hipGetLastError());
    return SP_OK;
}

template <typename PT, typename CT, typename VT>
sp_status scatter_t(const sp_tensor *A, const VT *B, int64_t N, int64_t ldb, VT *C, int64_t ldc, int accumulate, hipStream_t st)
{
    const PT *pos = (const PT *)A->pos[1];
    const CT *crd = (const CT *)A->crd[1];
    const VT *val = (const VT *)A->values;
    const CT *colid = A->enc.lt[0] == SP_COMPRESSED ? (const CT *)A->crd[0] : nullptr;
    const int64_t ncols = A->npos[1] - 1;
    if (!accumulate) SP_TRY((zero_c<PT, CT, VT>(C, A->shape[0], N, ldc, st)));
    if (ncols == 0) return SP_OK;
    sp_prof_scope prof(A, st);
#define SPMI_SCAT(CG)                                                                                                         \
    hipLaunchKernelGGL((spmm_scatter_kernel<PT, CT, VT, CG>), dim3(grid_for(ncols, kThreads / 64)), dim3(kThreads), 0, st, pos, \
                       crd, val, colid, ncols, B, N, ldb, C, ldc)
    if (N > 32) SPMI_SCAT(64);
    else if (N > 16) SPMI_SCAT(32);
    else if (N > 8) SPMI_SCAT(16);
    else if (N > 4) SPMI_SCAT(8);
    else if (N > 2) SPMI_SCAT(4);
    else if (N > 1) SPMI_SCAT(2);
    else SPMI_SCAT(1);
#undef SPMI_SCAT
    SP_HIP(hipGetLastError());
    return SP_OK;
}

// Scratch of the streaming product of fully stored rows with a vector: one partial sum per 2048-value chunk.
template <typename PT, typename CT, typename VT>
sp_status prepare_dense_inner_t(const sp_tensor *A, const VT *, int64_t N, int64_t, VT *, int64_t, int, hipStream_t st)
{
    const bool outer_compressed = A->enc.lt[0] == SP_COMPRESSED;
    const int64_t nstored = outer_compressed ? A->ncrd[0] : A->size[0];
    const int64_t inner = A->size[1];
    if (A->enc.perm[0] != 0 || N != 1 || inner < kDenseChunk || nstored <= 0 || nstored > 65535) return SP_OK;
    const size_t need = (size_t)(nstored * ceil_div(inner, kDenseChunk)) * sizeof(VT);
    if (A->dense_partial_bytes >= need) return SP_OK;
    sp_mem mem{A->alloc, A->free_, A->ctx};
    if (A->dense_partial) { SP_HIP(hipStreamSynchronize(st)); mem.put(A->dense_partial); A->dense_partial = nullptr; A->dense_partial_bytes = 0; }
    A->dense_partial = mem.get((need + 255) & ~(size_t)255);
    if (!A->dense_partial) return SP_ERR_ALLOC;
    A->dense_partial_bytes = need;
    return SP_OK;
}

template <typename PT, typename CT, typename VT>
sp_status dense_inner_t(const sp_tensor *A, const VT *B, int64_t N, int64_t ldb, VT *C, int64_t ldc, int accumulate, hipStream_t st)
{
    const VT *val = (const VT *)A->values;
    const bool outer_compressed = A->enc.lt[0] == SP_COMPRESSED;
    const CT *outer = outer_compressed ? (const CT *)A->crd[0] : nullptr;
    const int64_t nstored = outer_compressed ? A->ncrd[0] : A->size[0];        // stored rows (row-major) or columns
    const int64_t inner = A->size[1];
    const int64_t m = A->shape[0];
    const bool rowmajor = A->enc.perm[0] == 0;
    if (rowmajor && outer_compressed && !accumulate) SP_TRY((zero_c<PT, CT, VT>(C, m, N, ldc, st)));
    if (!rowmajor && nstored == 0 && !accumulate) return zero_c<PT, CT, VT>(C, m, N, ldc, st);
    if (nstored == 0 || inner == 0) return SP_OK;
    if (rowmajor && nstored > 0x7fffffff) return SP_ERR_TOO_LARGE;
    sp_prof_scope prof(A, st);
    constexpr int64_t V = 16 / sizeof(VT);
    if (rowmajor && N == 1 && ldb == 1 && inner >= kDenseChunk && inner % V == 0 && nstored <= 65535 &&
        (uintptr_t)B % 16 == 0 && (uintptr_t)val % 16 == 0) {
        // fully stored rows times a vector: the streaming path (16-byte loads need every row 16-byte aligned)
        const int64_t nchunks = ceil_div(inner, kDenseChunk);
        if (A->dense_partial_bytes < (size_t)(nstored * nchunks) * sizeof(VT)) {
            ++A->lazy_prepares;
            SP_TRY((prepare_dense_inner_t<PT, CT, VT>(A, B, N, ldb, C, ldc, accumulate, st)));
        }
        hipLaunchKernelGGL((dense_rows_spmv_partial_kernel<VT>), dim3((unsigned)nchunks, (unsigned)nstored), dim3(kThreads), 0, st, val, inner,
                           B, nchunks, (VT *)A->dense_partial);
        SP_HIP(hipGetLastError());
        hipLaunchKernelGGL((dense_rows_spmv_finish_kernel<CT, VT>), dim3(grid_for(nstored, kThreads)), dim3(kThreads), 0, st,
                           (const VT *)A->dense_partial, nchunks, outer, nstored, C, ldc, accumulate);
        SP_HIP(hipGetLastError());
        return SP_OK;
    }
#define SPMI_DENSE(CG)                                                                                                        \
    do {                                                                                                                      \
        if (rowmajor)                                                                                                         \
            hipLaunchKernelGGL((dense_rows_kernel<CT, VT, CG>), dim3((unsigned)nstored), dim3(kThreads), 0, st, val, outer, inner, B, N, \
                               ldb, C, ldc, accumulate);                                                                       \
        else                                                                                                                  \
            hipLaunchKernelGGL((dense_cols_kernel<CT, VT, CG>), dim3(grid_for(m, kThreads / CG)), dim3(kThreads), 0, st, val, outer,    \
                               nstored, inner, B, N, ldb, C, ldc, accumulate);                                                 \
    } while (0)
    if (N > 32) SPMI_DENSE(64);
    else if (N > 8) SPMI_DENSE(32);
    else if (N > 1) SPMI_DENSE(8);
    else SPMI_DENSE(1);
#undef SPMI_DENSE
    SP_HIP(hipGetLastError());
    return SP_OK;
}

}  // namespace

#define SPMI_DISPATCH_TYPES(FN, A, ...)                                                             \
    do {                                                                                            \
        const int pw__ = (A)->enc.pw, cw__ = (A)->enc.cw;                                           \
        if ((A)->dtype == SP_F64) {                                                                 \
            if (pw__ == 32 && cw__ == 32) return FN<int32_t, int32_t, double>(A, (const double *)B, N, ldb, (double *)C, ldc, accumulate, st); \
            if (pw__ == 32) return FN<int32_t, int64_t, double>(A, (const double *)B, N, ldb, (double *)C, ldc, accumulate, st);               \
            if (cw__ == 32) return FN<int64_t, int32_t, double>(A, (const double *)B, N, ldb, (double *)C, ldc, accumulate, st);               \
            return FN<int64_t, int64_t, double>(A, (const double *)B, N, ldb, (double *)C, ldc, accumulate, st);                               \
        } else {                                                                                    \
            if (pw__ == 32 && cw__ == 32) return FN<int32_t, int32_t, float>(A, (const float *)B, N, ldb, (float *)C, ldc, accumulate, st);    \
            if (pw__ == 32) return FN<int32_t, int64_t, float>(A, (const float *)B, N, ldb, (float *)C, ldc, accumulate, st);                  \
            if (cw__ == 32) return FN<int64_t, int32_t, float>(A, (const float *)B, N, ldb, (float *)C, ldc, accumulate, st);                  \
            return FN<int64_t, int64_t, float>(A, (const float *)B, N, ldb, (float *)C, ldc, accumulate, st);                                  \
        }                                                                                           \
    } while (0)

sp_status spmi_matmul_rowmajor(const sp_tensor *A, const void *B, int64_t N, int64_t ldb, void *C, int64_t ldc, int accumulate,
                               hipStream_t st)
{
    SPMI_DISPATCH_TYPES(rowmajor_t, A);
}

sp_status spmi_prepare_rowmajor(const sp_tensor *A, int64_t N, hipStream_t st)
{
    const void *B = nullptr; void *C = nullptr; const int64_t ldb = N, ldc = N; const int accumulate = 0;
    SPMI_DISPATCH_TYPES(prepare_rowmajor_t, A);
}

sp_status spmi_prepare_dense_inner(const sp_tensor *A, int64_t N, hipStream_t st)
{
    const void *B = nullptr; void *C = nullptr; const int64_t ldb = N, ldc = N; const int accumulate = 0;
    SPMI_DISPATCH_TYPES(prepare_dense_inner_t, A);
}

sp_status spmi_matmul_colmajor_scatter(const sp_tensor *A, const void *B, int64_t N, int64_t ldb, void *C, int64_t ldc,
                                       int accumulate, hipStream_t st)
{
    SPMI_DISPATCH_TYPES(scatter_t, A);
}

sp_status spmi_matmul_dense_inner(const sp_tensor *A, const void *B, int64_t N, int64_t ldb, void *C, int64_t ldc, int accumulate,
                                  hipStream_t st)
{
    SPMI_DISPATCH_TYPES(dense_inner_t, A);
}

// ---- the product for callers that cannot allocate ------------------------------------------------------------------
// The per-block carries of the SpMM cut by stored entries live in this array instead of a buffer from the tensor's
// allocator.  Every GPU the library runs on holds its own copy until the process ends; host code reaches it only through
// the address hipGetSymbolAddress returns for the current device (the name itself is a host-side stand-in).
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
static void *g_scratch_ptr[kMaxDevices];               // per device, filled in on the first call on that device

static sp_status static_scratch(void **out)
{
    int device = -1;
    SP_HIP(hipGetDevice(&device));
    if (device < 0 || device >= kMaxDevices) return SP_ERR_UNSUPPORTED;
    if (!g_scratch_ptr[device]) {
        void *ptr = nullptr;
        SP_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return SP_ERR_HIP;
        g_scratch_ptr[device] = ptr;
    }
    *out = g_scratch_ptr[device];
    return SP_OK;
}

namespace {
template <typename PT, typename CT, typename VT>
sp_status noalloc_t(const sp_tensor *A, const VT *B, int64_t N, int64_t ldb, VT *C, int64_t ldc, int accumulate, hipStream_t st)
{
    const row_view<PT, CT> rv(A);
    constexpr int64_t V = 16 / sizeof(VT);
    const int64_t lr = N / V;
    const bool aligned = N % V == 0 && ldb % V == 0 && ldc % V == 0 && (uintptr_t)B % 16 == 0 && (uintptr_t)C % 16 == 0;
    if (!rv.rowblocks->start || !aligned || lr < 1 || lr > 64) return SP_ERR_UNSUPPORTED;
    if ((size_t)rv.rowblocks->nblocks * (size_t)N * sizeof(VT) > kStaticScratchBytes) return SP_ERR_TOO_LARGE;
    void *carry = nullptr;
    SP_TRY(static_scratch(&carry));
    if (rv.dcsr && !accumulate) SP_TRY((zero_c<PT, CT, VT>(C, A->shape[0], N, ldc, st)));   // rows that are not stored become zero
    if (rv.nrows == 0) return SP_OK;
    // nothing in the carries has to start at zero: a block writes its carry before the fix-up reads it, and the fix-up
    // reads only carries of blocks whose first row began in an earlier block
    return spmm_windows_launch<PT, CT, VT>(A, rv, B, N, ldb, C, ldc, accumulate, (VT *)carry, st);
}
}  // namespace

extern "C" sp_status sp_matmul_noalloc(const sp_tensor *A, const void *B, int64_t N, int64_t ldb, void *C, int64_t ldc, int accumulate,
                                       void *stream)
{
    if (!A) return SP_ERR_NULL;
    if (A->enc.rank != 2) return SP_ERR_RANK;
    if (N < 0 || ldb < N || ldc < N || ldb < 1 || ldc < 1) return SP_ERR_SHAPE;
    if (N == 0 || A->shape[0] == 0) return SP_OK;
    if (!C || (!B && A->shape[1] > 0)) return SP_ERR_NULL;
    if (A->enc.lt[1] != SP_COMPRESSED || A->enc.perm[0] != 0 || A->tables_pending) return SP_ERR_UNSUPPORTED;
    hipStream_t st = (hipStream_t)stream;
    SPMI_DISPATCH_TYPES(noalloc_t, A);
}
