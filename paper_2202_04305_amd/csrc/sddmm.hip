// Sampled dense-dense product X[i,j] = S[i,j] * sum_k A[i,k] * B[k,j] (arXiv 2202.04305, Section 6.2: the kernel of
// the state-space search experiment).  X has S's sparsity pattern, so the result is one value per stored position
// of S, in storage order: no insertion into a sparse output is needed.
//
// Per stored entry (i, j) the kernel needs row i of A and column j of B.  B is K x n row-major in the paper's
// formula, so a column is a stride-n walk; it is transposed once per call into an n x K scratch (unless the caller
// already holds it that way), after which every entry reads one contiguous row of K values, exactly as the SpMM
// kernel reads rows of its dense operand.  Groups of lanes take runs of stored entries: the row of A sits in registers,
// the row of the transposed B comes in 16-byte loads, and a short shuffle reduction finishes each dot product.
#include "spmi_internal.h"

namespace {

constexpr int kThreads = 256;

template <typename VT>
__global__ __launch_bounds__(256) void transpose_kernel(const VT *__restrict__ B, int64_t K, int64_t n, int64_t ldb,
                                                        VT *__restrict__ Bt, int64_t ldt)
{
    __shared__ VT tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;          // 32 x 8 threads
    const int64_t j0 = (int64_t)blockIdx.x * 32, k0 = (int64_t)blockIdx.y * 32;
#pragma unroll
    for (int r = ty; r < 32; r += 8)
        if (k0 + r < K && j0 + tx < n) tile[r][tx] = B[(k0 + r) * ldb + j0 + tx];
    __syncthreads();
#pragma unroll
    for (int r = ty; r < 32; r += 8)
        if (j0 + r < n && k0 + tx < K) Bt[(j0 + r) * ldt + k0 + tx] = tile[tx][r];
}

// Work is cut by stored entries: block w owns the entries [w*T, (w+1)*T) (T and the table `rowblk` of the row holding
// every T-th entry are the stream SpMV's), or, where there are too few such windows to fill the chip, the block's share
// of `parts` equal shares of one.  A group of LR lanes takes a run of consecutive entries, one dot product at a time:
// lane jl holds vectors jl, jl + LR, ... (NV of them, 16 bytes each) of the row of A, which it loads again only when the
// run reaches another row, and loads the same pieces of the row of the transposed B.  No row of S is too short to fill a
// wave and none is walked by one wave alone.  The window's values of S, the byte offsets of the rows of the transposed
// B (OT: 32 bits when the matrix is below 4 GB) and the row of every entry are made in LDS first; the results replace
// the values there and leave with coalesced stores.
//
// The pieces of a lane are added up one by one and then together (sum_of_parts): one chain over all of them, up to 32 products, had
// 1.04 to 1.43 times the error of a wave's 64 lanes (f32, K = 256: 1.17e-7 against 8.2e-8, now 7.2e-8).
//
// Any K of one to 64 16-byte pieces (V <= K <= 64 V) and any leading dimension: the lane that holds the end of a row moves back to its last V columns and clears
// those that another lane has, so every load is 16 bytes wide (the memory path takes them at any element-aligned address).
//
// The rows of the transposed B set the pace (16.9 M random rows of 512 bytes: 1.15 ms).  Measured before (a wave per row of
// the window; any K that is not a power of two of 16-byte pieces: a lane per column and a wave per row) and now, whole product:
// 16.9 M entries, K = 64 f64 1.564 -> 1.497 ms; 5.0 M entries, K = 33 f64 3.51 -> 0.33 ms, K = 100 5.08 -> 0.78 ms; 20,000 entries,
// K = 64 65 -> 12 us.
template <typename VT>
struct sddmm_vec {
    static constexpr int V = 16 / sizeof(VT);
    typedef VT type __attribute__((ext_vector_type(V)));
    typedef VT in_memory __attribute__((ext_vector_type(V), aligned(sizeof(VT))));
};

// A lane's pieces of a dot product, each added up by itself: in a tree, or in f64 where f32 has more than two.
template <typename VT, int NV>
__device__ __forceinline__ VT sum_of_parts(VT (&part)[NV])
{
    if (sizeof(VT) == 4 && NV > 2) {
        double sum = 0;
#pragma unroll
        for (int v = 0; v < NV; ++v) sum += (double)part[v];
        return (VT)sum;
    }
#pragma unroll
    for (int w = 1; w < NV; w <<= 1)
#pragma unroll
        for (int v = 0; v + w < NV; v += 2 * w) part[v] += part[v + w];
    return part[0];
}

template <typename PT, typename CT, typename VT, int LR, int NV, typename OT>
__global__ __launch_bounds__(kThreads) void sddmm_entries_kernel(const PT *__restrict__ pos, const CT *__restrict__ crd,
                                                                 const VT *__restrict__ sval, const CT *__restrict__ rowid,
                                                                 const int32_t *__restrict__ rowblk, int64_t nrows, int64_t nnz, int parts,
                                                                 const VT *__restrict__ A, int64_t lda, const VT *__restrict__ Bt,
                                                                 int64_t ldt, int64_t K, VT *__restrict__ X)
{
    constexpr int V = sddmm_vec<VT>::V;
    constexpr int T = (int)kSpmiStreamT;
    constexpr int U = NV <= 2 ? 4 : NV <= 4 ? 2 : 1;                 // entries of a group in flight
    typedef typename sddmm_vec<VT>::type vec_t;
    typedef typename sddmm_vec<VT>::in_memory mem_vec_t;
    constexpr int kPad = T + T / 32;                                 // groups read 32 entries apart: kept off each other's bank
    __shared__ OT s_off[kPad];
    __shared__ VT s_val[kPad];
    __shared__ CT s_row[kPad];
    __shared__ int s_wave[kThreads / 64];
    auto at = [](int i) { return i + (i >> 5); };
    const int64_t win = blockIdx.x / parts;
    const int share = T / parts;
    const int64_t s = win * T + (int64_t)(blockIdx.x % parts) * share;
    if (s >= nnz) return;                                            // the whole block
    const int64_t e = s + share < nnz ? s + share : nnz;
    const int ne = (int)(e - s);
    const OT brow = (OT)(ldt * (int64_t)sizeof(VT));
    for (int i = threadIdx.x; i < ne; i += kThreads) {
        s_off[at(i)] = (OT)crd[s + i] * brow;
        s_val[at(i)] = sval[s + i];
    }
    const int64_t lo = rowblk[win], hi = rowblk[win + 1];
    const int64_t last = hi < nrows ? hi : nrows - 1;
    spmi_rows_of_entries<kThreads, T / kThreads>([=](int64_t r) { return (int64_t)pos[r]; }, rowid, lo, last, s, e, s_row, s_wave, at);
    const int jl = threadIdx.x % LR, group = threadIdx.x / LR;
    const int run_len = share * LR / kThreads;                       // entries of a group: 4 * LR, or LR
    const int64_t want = (int64_t)(jl + (NV - 1) * LR) * V;          // only the last piece of a row can reach past its end
    const int64_t tail = want <= K - V ? want : K - V;
    const int skip = want - tail < V ? (int)(want - tail) : V;       // columns of the last piece that another lane has
    const OT colb = (OT)(jl * V * (int)sizeof(VT)), tailb = (OT)(tail * (int64_t)sizeof(VT));
    const char *Bb = (const char *)Bt;
    vec_t av[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) av[v] = (vec_t)(0);
    CT row = (CT)-1;
    for (int k = 0; k < run_len; k += U) {
        int idx[U];
        vec_t bv[U][NV];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = group * run_len + k + u;
            idx[u] = i < ne ? i : ne - 1;                            // past the end: loaded, not stored
            const OT off = s_off[at(idx[u])];
#pragma unroll
            for (int v = 0; v < NV; ++v)
                bv[u][v] = *(const mem_vec_t *)(Bb + (off + (v < NV - 1 ? colb + (OT)(v * LR * 16) : tailb)));
        }
        VT dot[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const CT mine = s_row[at(idx[u])];
            if (mine != row) {
                row = mine;
                const char *Ab = (const char *)(A + (int64_t)row * lda);
#pragma unroll
                for (int v = 0; v < NV; ++v) av[v] = *(const mem_vec_t *)(Ab + (v < NV - 1 ? colb + (OT)(v * LR * 16) : tailb));
#pragma unroll
                for (int c = 0; c < V; ++c) if (c < skip) av[NV - 1][c] = (VT)0;
            }
#pragma unroll
            for (int c = 0; c < V; ++c) if (c < skip) bv[u][NV - 1][c] = (VT)0;      // not 0 * infinity
            VT part[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                part[v] = 0;
#pragma unroll
                for (int c = 0; c < V; ++c) part[v] += av[v][c] * bv[u][v][c];
            }
            dot[u] = sum_of_parts(part);
        }
        if (LR >= U && U > 1) {
            // The U sums are reduced together: each of the first log2(U) exchange steps halves the number of sums a lane
            // carries (a lane keeps the half its bit selects and hands the other half over), the remaining steps finish the
            // one sum left: sum u ends complete in the lanes whose top bits of jl are u.
            int m = LR / 2;
#pragma unroll
            for (int n = U; n > 1; n >>= 1) {
                const bool upper = (jl & m) != 0;
#pragma unroll
                for (int q = 0; q < n / 2; ++q) {
                    const VT send = upper ? dot[q] : dot[q + n / 2];
                    const VT keep = upper ? dot[q + n / 2] : dot[q];
                    dot[q] = keep + __shfl_xor(send, m, 64);
                }
                m >>= 1;
            }
#pragma unroll
            for (; m >= 1; m >>= 1) dot[0] += __shfl_xor(dot[0], m, 64);
            constexpr int D = LR / U > 0 ? LR / U : 1;               // lanes that end with the same sum
            const int u = jl / D;
            const int i = group * run_len + k + u;
            if (jl % D == 0 && k + u < run_len && i < ne) s_val[at(i)] *= dot[0];
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int d = LR / 2; d >= 1; d >>= 1) dot[u] += __shfl_xor(dot[u], d, 64);
                const int i = group * run_len + k + u;
                if (jl == 0 && k + u < run_len && i < ne) s_val[at(i)] *= dot[u];
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < ne; i += kThreads) X[s + i] = s_val[at(i)];
}

// any K: CG lanes per entry, each striding over k
template <typename PT, typename CT, typename VT, int CG>
__global__ __launch_bounds__(kThreads) void sddmm_rows_kernel(const PT *__restrict__ pos, const CT *__restrict__ crd,
                                                              const VT *__restrict__ sval, const CT *__restrict__ rowid, int64_t nrows,
                                                              const VT *__restrict__ A, int64_t lda, const VT *__restrict__ Bt,
                                                              int64_t ldt, int64_t K, VT *__restrict__ X)
{
    constexpr int S = 64 / CG;
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * (kThreads / 64) + (threadIdx.x >> 6);
    if (r >= nrows) return;
    const int jl = lane % CG, sl = lane / CG;
    const int64_t a = (int64_t)pos[r], b = (int64_t)pos[r + 1];
    if (a == b) return;
    const int64_t i = rowid ? (int64_t)rowid[r] : r;
    const int64_t steps = (b - a + S - 1) / S;
    for (int64_t t = 0; t < steps; ++t) {
        const int64_t p = a + t * S + sl;
        const int64_t pc = p < b ? p : b - 1;
        const int64_t j = (int64_t)crd[pc];
        VT dot = 0;
        for (int64_t k = jl; k < K; k += CG) dot += A[i * lda + k] * Bt[j * ldt + k];
#pragma unroll
        for (int d = CG / 2; d >= 1; d >>= 1) dot += __shfl_xor(dot, d, 64);
        if (jl == 0 && p < b) X[p] = sval[p] * dot;
    }
}

inline unsigned grid_for(int64_t n, int64_t per_block) { return (unsigned)(n > 0 ? ceil_div(n, per_block) : 1); }

template <typename PT, typename CT, typename VT>
sp_status sddmm_t(const sp_tensor *S, const VT *A, int64_t lda, const VT *B, int64_t ldb, int b_is_transposed, int64_t K, VT *X,
                  hipStream_t st)
{
    const PT *pos = (const PT *)S->pos[1];
    const CT *crd = (const CT *)S->crd[1];
    const VT *sval = (const VT *)S->values;
    const CT *rowid = S->enc.lt[0] == SP_COMPRESSED ? (const CT *)S->crd[0] : nullptr;
    int64_t nrows = S->npos[1] - 1;
    const sp_rowblocks *rowblocks = &S->rowblocks;
    if (!rowid && S->nz_pos) { pos = (const PT *)S->nz_pos; rowid = (const CT *)S->nz_rowid; nrows = S->nz_rows; rowblocks = &S->nz_rowblocks; }
    const int64_t n = S->shape[1];
    if (S->nvalues == 0 || nrows == 0) return SP_OK;
    if (K == 0) return spmi_fill_zero(X, (size_t)S->nvalues * sizeof(VT), st);   // X was allocated by the caller: exact size, 4-byte multiple

    constexpr int64_t V = 16 / sizeof(VT);
    const VT *Bt = B;
    int64_t ldt = ldb;
    if (!b_is_transposed) {
        ldt = (K + V - 1) / V * V;                         // rows of the scratch start 16-byte aligned
        // the transposed operand lives in scratch the tensor keeps and grows on demand: only a call that needs more than any
        // call before it allocates (and then waits for the stream, since the old block may still be read)
        const size_t need = (size_t)(n > 0 ? n : 1) * ldt * sizeof(VT);
        SP_TRY(spmi_reserve(S, S->sddmm_bt, need, st));
        S->sddmm_bt.shared |= spmi_recording(st);
        VT *scratch = (VT *)S->sddmm_bt.ptr;
        hipLaunchKernelGGL(transpose_kernel<VT>, dim3(grid_for(n, 32), grid_for(K, 32)), dim3(256), 0, st, B, K, n, ldb, scratch, ldt);
        SP_HIP(hipGetLastError());
        Bt = scratch;
    }
    {
        sp_prof_scope prof(S, st);
        const int64_t nvec = ceil_div(K, V);                        // 16-byte pieces of a row
        const bool vec = rowblocks->start && K >= V && nvec <= 64;
        const bool small = sizeof(CT) == 4 && (uint64_t)n * (uint64_t)ldt * sizeof(VT) < ((uint64_t)1 << 32);      // 32-bit byte offsets into the transposed B (64-bit coordinates keep 64-bit offsets)
        const dim3 grid(grid_for(nrows, kThreads / 64));
        if (vec) {
            // fewer windows than four per CU: a block takes a quarter of one
            const int parts = rowblocks->nblocks < 1024 ? 4 : 1;
            const dim3 blocks((unsigned)(rowblocks->nblocks * parts));
#define SPMI_SDDMM_VEC_O(LR, NV, OT)                                                                                          \
    hipLaunchKernelGGL((sddmm_entries_kernel<PT, CT, VT, LR, NV, OT>), blocks, dim3(kThreads), 0, st, pos, crd, sval, rowid,  \
                       (const int32_t *)rowblocks->start, nrows, S->ncrd[1], parts, A, lda, Bt, ldt, K, X)
#define SPMI_SDDMM_VEC(LR, NV)                              \
    do {                                                    \
        if (sizeof(CT) == 4 && small) SPMI_SDDMM_VEC_O(LR, NV, uint32_t);      \
        else SPMI_SDDMM_VEC_O(LR, NV, uint64_t);            \
    } while (0)
            if (nvec == 1) SPMI_SDDMM_VEC(1, 1);
            else if (nvec == 2) SPMI_SDDMM_VEC(2, 1);
            else if (nvec <= 4) SPMI_SDDMM_VEC(4, 1);
            else if (nvec <= 8) SPMI_SDDMM_VEC(8, 1);
            else if (nvec <= 16) SPMI_SDDMM_VEC(8, 2);
            else if (nvec <= 24) SPMI_SDDMM_VEC(8, 3);
            else if (nvec <= 32) SPMI_SDDMM_VEC(8, 4);
            else if (nvec <= 40) SPMI_SDDMM_VEC(8, 5);
            else if (nvec <= 48) SPMI_SDDMM_VEC(8, 6);
            else if (nvec <= 56) SPMI_SDDMM_VEC(8, 7);
            else SPMI_SDDMM_VEC(8, 8);
#undef SPMI_SDDMM_VEC
#undef SPMI_SDDMM_VEC_O
        } else {
#define SPMI_SDDMM(CG)                                                                                                        \
    hipLaunchKernelGGL((sddmm_rows_kernel<PT, CT, VT, CG>), grid, dim3(kThreads), 0, st, pos, crd, sval, rowid, nrows, A, lda, Bt, ldt, \
                       K, X)
            if (K > 32) SPMI_SDDMM(64);
            else if (K > 8) SPMI_SDDMM(32);
            else if (K > 2) SPMI_SDDMM(8);
            else SPMI_SDDMM(2);
#undef SPMI_SDDMM
        }
        SP_HIP(hipGetLastError());
    }
    return SP_OK;
}

}  // namespace

extern "C" sp_status sp_sddmm(const sp_tensor *S, const void *A, int64_t lda, const void *B, int64_t ldb, int b_is_transposed,
                              int64_t K, void *X, void *stream)
{
    if (!S) return SP_ERR_NULL;
    if (S->enc.rank != 2) return SP_ERR_RANK;
    const int64_t n = S->shape[1];
    if (K < 0 || lda < K || (b_is_transposed ? ldb < K : ldb < n)) return SP_ERR_SHAPE;
    if (S->nvalues > 0 && (!X || (K > 0 && (!A || !B)))) return SP_ERR_NULL;
    if (S->enc.perm[0] != 0 || S->enc.lt[1] != SP_COMPRESSED) return SP_ERR_UNSUPPORTED;   // row-major with a compressed inner level
    hipStream_t st = (hipStream_t)stream;
    SP_TRY(spmi_ensure_tables(S, st));
    const int pw = S->enc.pw, cw = S->enc.cw;
#define SPMI_GO(PT, CT)                                                                                                       \
    return S->dtype == SP_F64 ? sddmm_t<PT, CT, double>(S, (const double *)A, lda, (const double *)B, ldb, b_is_transposed, K, (double *)X, st) \
                              : sddmm_t<PT, CT, float>(S, (const float *)A, lda, (const float *)B, ldb, b_is_transposed, K, (float *)X, st)
    if (pw == 32 && cw == 32) SPMI_GO(int32_t, int32_t);
    if (pw == 32) SPMI_GO(int32_t, int64_t);
    if (cw == 32) SPMI_GO(int64_t, int32_t);
    SPMI_GO(int64_t, int64_t);
#undef SPMI_GO
}
