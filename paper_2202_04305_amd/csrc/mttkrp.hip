// Matricized tensor times Khatri-Rao product A[i,j] = sum_{k,l} B[i,k,l] * D[l,j] * C[k,j] (arXiv 2202.04305,
// Section 6.3) for a packed rank-3 tensor B whose outermost level stores dimension i (dense or compressed) and whose
// two inner levels are compressed, in either order of k and l (the two formats of the paper's experiment).
//
// Call "mid" the factor matrix indexed by the level-1 coordinate and "inner" the one indexed by the level-2
// coordinate.  For a level-1 fibre f (one pair of level-0 position and level-1 coordinate m) the sum factors as
//     A[i,:] += mid[m,:] .* sum_{p in fibre f} values[p] * inner[crd2[p],:]
// so the hot loop is the SpMM loop over the entries of a fibre (a gather of rows of `inner`), one elementwise product
// per fibre, and a running sum per slice i.  Both factor matrices are small next to B (megabytes) and live in cache;
// B's crd2 / values stream from HBM once.
//
// Work is cut by stored entries: a block owns the entries [w*TW, (w+1)*TW), a group of LR lanes covers the J columns (16-byte
// loads) and takes a run of consecutive entries, whatever fibres and slices they belong to: it adds up a fibre, takes the
// fibre's row of `mid` in when the fibre ends, and writes A when the slice does.  Parts of a slice that began in an earlier run
// meet in LDS, the part that began in an earlier window goes to carry[w] (J values); a second kernel adds a slice's carries to
// A in a fixed pattern; everything else is written to A directly.  No atomics: results are bit-reproducible.
#include "spmi_internal.h"

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
// Stored entries per block.  20 M entries, 42 f64 columns: 256 -> 682 us, 512 -> 523, 1024 -> 461 (every block makes its tables once;
// larger ones leave too few blocks on a CU for the LDS).
constexpr int64_t kTW = 1024;

__global__ __launch_bounds__(kThreads) void zero_rows_kernel(char *__restrict__ A, int64_t rows, int64_t row_bytes, int64_t ld_bytes)
{
    const int64_t words = row_bytes / 4;      // element sizes are 4 or 8
    const int64_t total = rows * words;
    for (int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x; t < total; t += (int64_t)gridDim.x * kThreads)
        *(uint32_t *)(A + (t / words) * ld_bytes + (t % words) * 4) = 0u;
}

// dst[r, 0..cols) = src[r, 0..cols) for a row-major matrix with other leading dimensions, in pieces of type W
template <typename W>
__global__ __launch_bounds__(kThreads) void repitch_rows_kernel(const char *__restrict__ src, int64_t src_ld_bytes, int64_t rows,
                                                                int64_t row_bytes, char *__restrict__ dst, int64_t dst_ld_bytes)
{
    const int64_t pieces = row_bytes / (int64_t)sizeof(W);
    const int64_t total = rows * pieces;
    for (int64_t t = (int64_t)blockIdx.x * kThreads + threadIdx.x; t < total; t += (int64_t)gridDim.x * kThreads) {
        const int64_t r = t / pieces, c = t % pieces;
        *(W *)(dst + r * dst_ld_bytes + c * (int64_t)sizeof(W)) = *(const W *)(src + r * src_ld_bytes + c * (int64_t)sizeof(W));
    }
}

// wfib[w] = level-1 fibre holding entry w*TW, wslc[w] = level-0 position holding that fibre (largest index whose
// pos entry is <= the target: empty slices are skipped by construction).  A window boundary w that is the first one
// its slice crosses (the slice begins inside window w - 1) is appended to `cross` (count in cross[-1]); the order of
// that list does not matter, every entry is an independent piece of work for the fix-up kernel.  An entry is the
// pair (w, last window that begins inside the same slice).
template <typename PT>
__global__ __launch_bounds__(kThreads) void mttkrp_windows_table_kernel(const PT *__restrict__ pos1, int64_t nslc,
                                                                        const PT *__restrict__ pos2, int64_t nfib, int64_t nwin,
                                                                        int32_t *__restrict__ wfib, int32_t *__restrict__ wslc,
                                                                        int32_t *__restrict__ cross)
{
    const int64_t w = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    if (w >= nwin) return;
    const int64_t s = w * kTW;
    int64_t lo = 0, hi = nfib - 1;            // pos2[lo] <= s always (pos2[0] = 0)
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if ((int64_t)pos2[mid] <= s) lo = mid; else hi = mid - 1;
    }
    const int64_t f = lo;
    lo = 0; hi = nslc - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if ((int64_t)pos1[mid] <= f) lo = mid; else hi = mid - 1;
    }
    wfib[w] = (int32_t)f;
    wslc[w] = (int32_t)lo;
    if (w >= 1) {
        const int64_t start = (int64_t)pos2[(int64_t)pos1[lo]];
        if (start < s && start >= s - kTW) {
            const int64_t end = (int64_t)pos2[(int64_t)pos1[lo + 1]];      // first entry past the slice
            const int64_t a = (end - 1) / kTW;                             // last window that begins inside the slice
            const int at = atomicAdd(&cross[-1], 1);
            cross[2 * at] = (int32_t)w;
            cross[2 * at + 1] = (int32_t)a;
        }
    }
}

template <typename VT, int V>
struct vec_of {
    typedef VT type __attribute__((ext_vector_type(V)));
    typedef VT in_memory __attribute__((ext_vector_type(V), aligned(sizeof(VT))));
};

// grid = (windows rounded up to a multiple of 8, column tiles of lr_tile * V columns).  The block first makes in LDS, for every
// entry of its window, the value, the byte offset of the row of the inner factor (OT: 32 bits when both factor matrices are
// below 4 GB), the row of the mid factor and the slice.  Any J >= V, leading dimension and element-aligned address: the last
// lane of a row moves back to the last V columns and stores only those that the lane before it does not have.
// The entries are added up four at a time, these sums eight at a time: one chain for all of a run's had up to 1.3 times the error
// on wide rows (2,000 slices of 750 entries, 100 f64 columns 4.5e-16 -> 1.8e-16 relative 2-norm).  A window that one
// slice fills ends in shuffles instead of the search for equal slices.
// Bound by the rows of the inner factor that it gathers.  Measured before (a wave per 128 entries that walked their fibres one
// after the other; a column per lane for widths that are no multiple of 16 bytes) and now: 76.9 M entries, 42 f64 columns
// 1.870 -> 1.825 ms; 20 M entries in fibres of one to four, 16 columns 577 -> 290 us; 20 M entries in 40 slices, 16 f64 columns
// 203 -> 199 us, 64 f64 columns 450 -> 457, 32 f32 columns 180 -> 198, 64 f32 columns 245 -> 279 (without the windows of one slice 219,
// 458, 218, 299); 30,000 entries in fibres of one or two, 42 columns 56 -> 20 us.
template <typename PT, typename CT, typename VT, int V, typename OT>
__global__ __launch_bounds__(kThreads) void mttkrp_runs_kernel(const PT *__restrict__ pos1, const CT *__restrict__ crd0, const CT *__restrict__ crd1,
                                                               const PT *__restrict__ pos2, const CT *__restrict__ crd2, const VT *__restrict__ val,
                                                               const int32_t *__restrict__ wfib, const int32_t *__restrict__ wslc, int64_t nwin,
                                                               int64_t nfib, int64_t nslc, int64_t nnz, const VT *__restrict__ M, int64_t ldm,
                                                               const VT *__restrict__ X, int64_t ldx, VT *__restrict__ A, int64_t lda,
                                                               VT *__restrict__ carry, int64_t J, int lr_tile, int accumulate)
{
    constexpr int T = (int)kTW, U = 4, PER = T / kThreads;
    static_assert(T == 1024, "a whole number of entries per thread; by_run, kRoom");
    typedef typename vec_of<VT, V>::type vec_t;
    typedef typename vec_of<VT, V>::in_memory mem_vec_t;
    constexpr int kRoom = T + kThreads;                            // run length (rounded up) * odd stride: 256 * 5 at most
    __shared__ OT s_xoff[kRoom];
    __shared__ VT s_val[kRoom];
    __shared__ CT s_mid[kRoom], s_slc[kRoom];
    __shared__ vec_t s_part[kThreads];
    __shared__ int s_wave[kWaves];
    // Workgroups go to the 8 XCDs in turn, each with an L2 of its own.  Block b therefore takes the (b / 8)-th window of
    // the (b % 8)-th eighth of the windows: an XCD walks a contiguous range of entries, so the rows of the factor
    // matrices that a slice keeps coming back to are found in that XCD's L2.  (Only the mapping depends on this.)
    const int64_t w = (int64_t)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
    if (w >= nwin) return;                                         // the whole block
    const int64_t j0 = (int64_t)blockIdx.y * lr_tile * V;
    const int64_t width = J - j0 < (int64_t)lr_tile * V ? J - j0 : (int64_t)lr_tile * V;
    const int LR = (int)((width + V - 1) / V);                     // 1..64
    const int S = 64 / LR, G = kWaves * S;                         // groups per wave, per block
    const int run = (T + G - 1) / G;                               // entries per group
    const uint32_t by_run = (uint32_t)(((uint64_t)1 << 21) / (uint32_t)run + 1);      // i / run for i < 1024: exact, run <= 256
    // entry i of the window is kept at (i % run) * P + i / run: the groups of a wave read neighbouring words, and with an odd P
    // neighbouring entries lie on different banks when they are put there
    const int P = G | 1;
    auto at = [=](int i) {
        const int g = (int)(__umul24((uint32_t)i, by_run) >> 21);
        return (int)__umul24((uint32_t)(i - (int)__umul24((uint32_t)g, (uint32_t)run)), (uint32_t)P) + g;
    };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t s = w * T;
    const int64_t e = s + T < nnz ? s + T : nnz;
    const int ne = (int)(e - s);
    const OT xrow = (OT)(ldx * (int64_t)sizeof(VT)), mrow = (OT)(ldm * (int64_t)sizeof(VT));
#pragma unroll
    for (int x = 0; x < PER; ++x) {
        const int i = x * kThreads + threadIdx.x;
        if (i < ne) {
            s_xoff[at(i)] = (OT)crd2[s + i] * xrow;
            s_val[at(i)] = val[s + i];
        }
    }
    const int64_t f0 = wfib[w], f1 = w + 1 < nwin ? (int64_t)wfib[w + 1] : nfib - 1;
    const int64_t q0 = wslc[w], q1 = w + 1 < nwin ? (int64_t)wslc[w + 1] : nslc - 1;
    spmi_rows_of_entries<kThreads, PER>([=](int64_t f) { return (int64_t)pos2[f]; }, crd1, f0, f1, s, e, s_mid, s_wave, at);
    spmi_rows_of_entries<kThreads, PER>([=](int64_t q) { return (int64_t)pos2[(int64_t)pos1[q]]; }, crd0, q0, q1, s, e, s_slc, s_wave, at);
    const bool continued = (int64_t)pos2[(int64_t)pos1[q0]] < s;   // the first slice began in an earlier window
    const bool one_slice = (int64_t)pos2[(int64_t)pos1[q0 + 1]] >= e;   // and holds the whole window
    const int sl = lane / LR, jl = lane - sl * LR;
    const int group = sl < S ? wave * S + sl : G;                  // lanes beyond S * LR take nothing
    const int first = group * run < ne ? group * run : ne, end = first + run < ne ? first + run : ne;
    const int64_t want = j0 + (int64_t)jl * V;
    const int64_t col = want <= J - V ? want : J - V;              // this lane's columns: [col, col + V), its own from skip on
    const int skip = (int)(want - col);
    const OT colb = (OT)(col * (int64_t)sizeof(VT));
    const char *Xb = (const char *)X, *Mb = (const char *)M;
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
    const int slot = group * LR + jl;                              // this lane's place in s_part
    // The slice's sum, of some eight times U entries more, of U entries more; of the running fibre among these, and its row of mid.
    vec_t sum = (vec_t)(0), mid_sum = (vec_t)(0), acc = (vec_t)(0), t = (vec_t)(0), c = (vec_t)(0);
    CT slice = 0, mid = 0;
    bool head = false;                                             // the slice being added up began before this run
    if (first < end) {
        slice = s_slc[group];
        mid = s_mid[group];
        head = group == 0 ? continued : s_slc[(run - 1) * P + group - 1] == slice;
        c = *(const mem_vec_t *)(Mb + ((OT)mid * mrow + colb));
    }
    CT mid_ahead = mid, slice_ahead = slice;                       // of the last entry requested
    const int mine = end - first, last_x = (mine - 1) * P + group; // entries of this run, where the last one is kept
    for (int k = 0; k < mine; k += U) {
        VT v[U];
        vec_t bv[U], mv[U];
        CT qs[U];
        bool fresh[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int next = (k + u) * P + group, x = next < last_x ? next : last_x;
            const CT m = s_mid[x];
            qs[u] = s_slc[x];
            v[u] = s_val[x];
            bv[u] = *(const mem_vec_t *)(Xb + (s_xoff[x] + colb));
            fresh[u] = m != mid_ahead || qs[u] != slice_ahead;     // a new fibre
            mid_ahead = m;
            slice_ahead = qs[u];
            if (fresh[u]) mv[u] = *(const mem_vec_t *)(Mb + ((OT)m * mrow + colb));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (k + u < mine) {
                if (fresh[u]) {
                    if (u > 0) acc += c * t;                       // at u = 0 the entries before have been taken in (t is zero, c may be infinite)
                    t = (vec_t)(0);
                    c = mv[u];
                    if (qs[u] != slice) {
                        acc = sum + (mid_sum + acc);
                        if (head) s_part[slot] = acc;
                        else store(A + (int64_t)slice * lda + col, acc, accumulate);
                        head = false;
                        slice = qs[u];
                        acc = mid_sum = sum = (vec_t)(0);
                    }
                }
                t += v[u] * bv[u];
            }
        }
        mid_sum += acc + c * t;
        acc = t = (vec_t)(0);
        if (k % (8 * U) == 7 * U) { sum += mid_sum; mid_sum = (vec_t)(0); }
    }
    acc = sum + mid_sum;
    if (one_slice) {
        // every group has a part of one sum: towards the first group of each wave, then over the waves
        for (int d = 1; d < S; d <<= 1) {
#pragma unroll
            for (int x = 0; x < V; ++x) {
                const VT other = __shfl(acc[x], lane + d * LR < 64 ? lane + d * LR : lane, 64);
                acc[x] += sl + d < S ? other : (VT)0;
            }
        }
        if (sl == 0) s_part[slot] = acc;
        __syncthreads();
        if (group != 0) return;
        for (int g = S; g < G; g += S) acc += s_part[g * LR + jl];
        if (continued) store(carry + w * J + col, acc, false);
        else store(A + (int64_t)slice * lda + col, acc, accumulate);
        return;
    }
    if (head) s_part[slot] = acc;                                  // the whole run belongs to a slice that began before it
    // The sums of a slice that fills whole runs are added up towards the first of them, over twice as many groups each step.
    const int full = (ne + run - 1) / run;                         // groups that took something
    if (__syncthreads_or(head))
        for (int d = 1; d < full; d <<= 1) {
            const bool take = group + d < full && s_slc[group + d] == s_slc[group];      // slices ascend: everything between is that slice's too
            const vec_t other = take ? s_part[slot + d * LR] : (vec_t)(0);
            __syncthreads();
            if (take) s_part[slot] += other;
            __syncthreads();
        }
    if (first >= end) return;
    if (group == 0 && continued) store(carry + w * J + col, s_part[slot], false);
    if (!head) {
        if (group + 1 < full && s_slc[group + 1] == slice) acc += s_part[slot + LR];
        store(A + (int64_t)slice * lda + col, acc, accumulate);
    }
}

// A block per listed window boundary (the first one a slice crosses): adds all of that slice's carries to A.  The
// carries are summed in a fixed pattern (four strided partial sums per column, combined in order), so the result is
// the same on every call.
template <typename CT, typename VT, int kFixThreads>
__global__ __launch_bounds__(kFixThreads) void mttkrp_fixup_kernel(const CT *__restrict__ crd0, const int32_t *__restrict__ wslc,
                                                                   const int32_t *__restrict__ cross, int64_t nwin, int64_t J,
                                                                   const VT *__restrict__ carry, VT *__restrict__ A, int64_t lda)
{
    constexpr int kFixGroups = kFixThreads / 64;
    __shared__ VT part[kFixGroups][64];
    if ((int)blockIdx.x >= cross[-1]) return;                      // block-uniform
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int64_t b = cross[2 * blockIdx.x], last = cross[2 * blockIdx.x + 1];
    const int32_t q = wslc[b];
    const int64_t i = crd0 ? (int64_t)crd0[q] : (int64_t)q;
    for (int64_t jb = 0; jb < J; jb += 64) {                       // block-uniform
        const int64_t j = jb + lane;
        VT s0 = 0, s1 = 0, s2 = 0, s3 = 0;
        if (j < J) {
            int64_t bb = b + g;
            for (; bb + 3 * kFixGroups <= last; bb += 4 * kFixGroups) {
                s0 += carry[bb * J + j];
                s1 += carry[(bb + kFixGroups) * J + j];
                s2 += carry[(bb + 2 * kFixGroups) * J + j];
                s3 += carry[(bb + 3 * kFixGroups) * J + j];
            }
            for (; bb <= last; bb += kFixGroups) s0 += carry[bb * J + j];
        }
        part[g][lane] = (s0 + s1) + (s2 + s3);
        __syncthreads();
        if (g == 0 && j < J) {
            VT tot = part[0][lane];
#pragma unroll
            for (int k = 1; k < kFixGroups; ++k) tot += part[k][lane];
            A[i * lda + j] += tot;
        }
        __syncthreads();
    }
}

// Is a copy of a factor matrix with rows padded to whole lines made up for by the lines that the gathers then leave out?  The copy
// costs its bytes, read and written; a gather saves the lines its row touches beyond the padded ones, over all the places
// in a line where rows begin.  The line is where measured times cross (42 and 60 f64 columns, 60,000 to 1 M rows: 24 to 36
// gathers per row; 60 f32 columns 10 to 16; 33 f64 columns, which save nothing: never), at 3.5 times the bytes saved.  1 M rows,
// 42 f64 columns: 8 gathers per row 619 us with the copy, 510 without; 64 per row, 200,000 rows 696 and 758; 20,000 rows (6.7 MB),
// 2000 per row 1119 and 1055; 28,818 rows (9.7 MB), 2668 per row 1826 and 1943.
bool padding_pays(uintptr_t first, int64_t rows, int64_t row_bytes, int64_t ld_bytes, int64_t gathers)
{
    const int64_t padded = (row_bytes + 127) / 128;
    if (rows * row_bytes <= ((int64_t)8 << 20)) return false;
    int64_t touched = 0;                                             // by rows 0..127: their places in a line repeat after that
    for (int64_t r = 0; r < 128; ++r) touched += ((int64_t)((first + (uint64_t)r * (uint64_t)ld_bytes) % 128) + row_bytes + 127) / 128;
    const double saved = (double)touched / 128 - (double)padded;     // lines per gather
    return (double)gathers * saved * 128 >= 3.5 * (double)rows * (double)(row_bytes + padded * 128);
}

template <typename PT, typename CT, typename VT>
sp_status mttkrp_t(const sp_tensor *B, const VT *M, int64_t ldm, const VT *X, int64_t ldx, int64_t J, VT *A, int64_t lda,
                   int accumulate, hipStream_t st)
{
    const int64_t I = B->shape[0];
    if (I == 0 || J == 0) return SP_OK;
    if (!accumulate) {
        hipLaunchKernelGGL(zero_rows_kernel, dim3((unsigned)(ceil_div(I * J, kThreads) < 2048 ? ceil_div(I * J, kThreads) : 2048)),
                           dim3(kThreads), 0, st, (char *)A, I, J * (int64_t)sizeof(VT), lda * (int64_t)sizeof(VT));
        SP_HIP(hipGetLastError());
    }
    const int64_t nnz = B->nvalues;
    if (nnz == 0) return SP_OK;
    const PT *pos1 = (const PT *)B->pos[1], *pos2 = (const PT *)B->pos[2];
    const CT *crd0 = (const CT *)B->crd[0], *crd1 = (const CT *)B->crd[1], *crd2 = (const CT *)B->crd[2];
    const int64_t nslc = B->npos[1] - 1, nfib = B->npos[2] - 1;
    const int64_t nwin = ceil_div(nnz, kTW);
    const sp_tensor *Bt = B;                    // the handle's scratch and tables are its cache (mutable members)
    sp_mem mem{B->alloc, B->free_, B->ctx};
    const int64_t ncross = nslc < nwin - 1 ? nslc : nwin - 1;        // a slice has at most one first crossing
    const size_t table_bytes = (size_t)(2 * nwin + 4 + (ncross > 0 ? 2 * ncross : 0)) * 4;
    if (!Bt->mttkrp_windows) {
        // the handle takes the table only once its build has been enqueued: a failure on the way leaves no half-built table behind
        void *table = mem.get(table_bytes);
        if (!table) return SP_ERR_ALLOC;
        int32_t *wfib = (int32_t *)table, *wslc = wfib + nwin, *cross = wslc + nwin + 4;
        sp_status built = spmi_fill_zero(wslc + nwin, 16, st);     // cross[-1] = 0: the length of the list
        if (built == SP_OK) {
            hipLaunchKernelGGL(mttkrp_windows_table_kernel<PT>, dim3((unsigned)ceil_div(nwin, kThreads)), dim3(kThreads), 0, st, pos1, nslc,
                               pos2, nfib, nwin, wfib, wslc, cross);
            if (hipGetLastError() != hipSuccess) built = SP_ERR_HIP;
        }
        if (built != SP_OK) { (void)hipStreamSynchronize(st); mem.put(table); return built; }
        Bt->mttkrp_windows = table;
    }
    const bool recording = spmi_recording(st);
    SP_TRY(spmi_reserve(B, Bt->mttkrp_carry, (size_t)nwin * J * sizeof(VT), st));
    Bt->mttkrp_carry.shared |= recording;
    VT *carry = (VT *)Bt->mttkrp_carry.ptr;
    const int32_t *wfib = (const int32_t *)B->mttkrp_windows, *wslc = wfib + nwin, *cross = wslc + nwin + 4;
    constexpr int VV = 16 / sizeof(VT);
    // rows that can be copied 16 bytes at a time
    const bool pieces16 = J % VV == 0 && ldm % VV == 0 && ldx % VV == 0 && lda % VV == 0 && (uintptr_t)M % 16 == 0 && (uintptr_t)X % 16 == 0 &&
                          (uintptr_t)A % 16 == 0;
    const int64_t K = B->shape[1], L = B->shape[2];
    const int64_t rows_m = B->enc.perm[1] == 1 ? K : L, rows_x = B->enc.perm[1] == 1 ? L : K;
    // The inner factor is gathered a row per stored entry, the mid factor a row per fibre.  Where such a matrix is larger
    // than two L2 caches and enough gathers save a line each, a copy with rows padded to whole 128-byte lines is
    // gathered from instead (a 336-byte row then touches 3 lines, not 3.5 on average); the copy is made on every call
    // into a buffer the tensor keeps.  Rows of an odd size go without the copy where that buffer cannot be had.
    const int64_t row_bytes = J * (int64_t)sizeof(VT);
    for (int which = 0; which < 2; ++which) {
        const VT *&F = which == 0 ? X : M;
        int64_t &ldf = which == 0 ? ldx : ldm;
        const int64_t rows_f = which == 0 ? rows_x : rows_m;
        if (!(J >= VV && padding_pays((uintptr_t)F, rows_f, row_bytes, ldf * (int64_t)sizeof(VT), which == 0 ? nnz : nfib))) continue;
        const int64_t ldp_bytes = (row_bytes + 127) / 128 * 128;
        const size_t want = (size_t)rows_f * (size_t)ldp_bytes;
        sp_kept &pad = Bt->mttkrp_pad[which];
        if (!pieces16 && recording && pad.bytes < want) continue;
        const sp_status room = spmi_reserve(B, pad, want, st);
        if (room == SP_ERR_ALLOC && !pieces16) continue;
        SP_TRY(room);
        pad.shared |= recording;
        const int64_t pieces = rows_f * (pieces16 ? row_bytes / 16 : J);
        const dim3 copy_grid((unsigned)(ceil_div(pieces, kThreads) < 4096 ? ceil_div(pieces, kThreads) : 4096));
        if (pieces16)
            hipLaunchKernelGGL(repitch_rows_kernel<uint4>, copy_grid, dim3(kThreads), 0, st, (const char *)F, ldf * (int64_t)sizeof(VT), rows_f,
                               row_bytes, (char *)pad.ptr, ldp_bytes);
        else
            hipLaunchKernelGGL(repitch_rows_kernel<VT>, copy_grid, dim3(kThreads), 0, st, (const char *)F, ldf * (int64_t)sizeof(VT), rows_f,
                               row_bytes, (char *)pad.ptr, ldp_bytes);
        SP_HIP(hipGetLastError());
        F = (const VT *)pad.ptr;
        ldf = ldp_bytes / (int64_t)sizeof(VT);
    }
    // byte offsets into the factor matrices fit 32 bits when both are below 4 GB
    const bool small = sizeof(CT) == 4 && (uint64_t)rows_m * (uint64_t)ldm * sizeof(VT) < ((uint64_t)1 << 32) &&
                       (uint64_t)rows_x * (uint64_t)ldx * sizeof(VT) < ((uint64_t)1 << 32);      // 64-bit coordinates keep 64-bit offsets
    {
        sp_prof_scope prof(B, st);
        const unsigned gx = (unsigned)(ceil_div(nwin, 8) * 8);                     // a multiple of 8: see the block mapping in the kernel
        const int V = J >= VV ? VV : J >= 2 ? 2 : 1;                              // fewer columns than a load holds: shorter loads
        const int64_t pieces = ceil_div(J, V);
        // at least 512 blocks where the columns allow: few windows share the columns out among more blocks
        const int64_t split = nwin < 512 ? ceil_div(512, nwin) : 1;
        const int64_t wanted = ceil_div(pieces, split) > 4 ? ceil_div(pieces, split) : 4;
        const int lr_tile = (int)(wanted < 64 ? wanted : 64);
#define SPMI_MTTKRP(V, OT)                                                                                                             \
    hipLaunchKernelGGL((mttkrp_runs_kernel<PT, CT, VT, V, OT>), dim3(gx, (unsigned)ceil_div(pieces, lr_tile)), dim3(kThreads), 0, st, pos1, crd0, \
                       crd1, pos2, crd2, (const VT *)B->values, wfib, wslc, nwin, nfib, nslc, nnz, M, ldm, X, ldx, A, lda,              \
                       carry, J, lr_tile, accumulate)
#define SPMI_MTTKRP_V(V)                            \
    do {                                            \
        if (small) SPMI_MTTKRP(V, uint32_t);        \
        else SPMI_MTTKRP(V, uint64_t);              \
    } while (0)
        if (V == VV) SPMI_MTTKRP_V(VV);
        else if (V == 2) SPMI_MTTKRP_V(2);
        else SPMI_MTTKRP_V(1);
#undef SPMI_MTTKRP_V
#undef SPMI_MTTKRP
        SP_HIP(hipGetLastError());
    }
    if (ncross > 0) {
        // sixteen waves where slices fill many windows, four where a few carries per slice leave most of them idle (12,092 slices of
        // six windows: 46 us with sixteen, 20 with four)
        if (nwin > 32 * ncross)
            hipLaunchKernelGGL((mttkrp_fixup_kernel<CT, VT, 1024>), dim3((unsigned)ncross), dim3(1024), 0, st, crd0, wslc, cross, nwin, J,
                               (const VT *)carry, A, lda);
        else
            hipLaunchKernelGGL((mttkrp_fixup_kernel<CT, VT, 256>), dim3((unsigned)ncross), dim3(256), 0, st, crd0, wslc, cross, nwin, J,
                               (const VT *)carry, A, lda);
        SP_HIP(hipGetLastError());
    }
    return SP_OK;
}

}  // namespace

extern "C" sp_status sp_mttkrp(const sp_tensor *B, const void *C, int64_t ldc, const void *D, int64_t ldd, int64_t J, void *A,
                               int64_t lda, int accumulate, void *stream)
{
    if (!B) return SP_ERR_NULL;
    if (B->enc.rank != 3) return SP_ERR_RANK;
    if (J < 0 || ldc < J || ldd < J || lda < J) return SP_ERR_SHAPE;
    if (J > 0 && B->shape[0] > 0 && !A) return SP_ERR_NULL;
    if (J > 0 && B->nvalues > 0 && (!C || !D)) return SP_ERR_NULL;
    // dimension i outermost, both inner levels compressed; anything else: convert first
    if (B->enc.perm[0] != 0 || B->enc.lt[1] != SP_COMPRESSED || B->enc.lt[2] != SP_COMPRESSED) return SP_ERR_UNSUPPORTED;
    const bool k_first = B->enc.perm[1] == 1;
    const void *M = k_first ? C : D, *X = k_first ? D : C;
    const int64_t ldm = k_first ? ldc : ldd, ldx = k_first ? ldd : ldc;
    hipStream_t st = (hipStream_t)stream;
    const int pw = B->enc.pw, cw = B->enc.cw;
#define SPMI_GO(PT, CT)                                                                                                            \
    return B->dtype == SP_F64 ? mttkrp_t<PT, CT, double>(B, (const double *)M, ldm, (const double *)X, ldx, J, (double *)A, lda, accumulate, st) \
                              : mttkrp_t<PT, CT, float>(B, (const float *)M, ldm, (const float *)X, ldx, J, (float *)A, lda, accumulate, st)
    if (pw == 32 && cw == 32) SPMI_GO(int32_t, int32_t);
    if (pw == 32) SPMI_GO(int32_t, int64_t);
    if (cw == 32) SPMI_GO(int64_t, int32_t);
    SPMI_GO(int64_t, int64_t);
#undef SPMI_GO
}
