// Internal declarations shared by the library's translation units (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <string.h>
#include <type_traits>
#include <atomic>
#include <vector>
#include "spmi.h"
#include "spmi_bench.h"

struct sp_encoding {
    int rank;
    int lt[SP_MAX_RANK];
    int perm[SP_MAX_RANK];   // perm[l] = dimension stored at level l
    int pw, cw;              // widths the kernels work on: 32 or 64
    int pw_store, cw_store;  // widths asked for (8, 16, 32, 64): what sp_pos / sp_crd hand out
};

// Row blocks of the streaming SpMV: block b covers rows [rowblk[b], rowblk[b+1]) of the
// outer level; built once at pack time from pos of the innermost level.
struct sp_rowblocks {
    void *start = nullptr;   // DEVICE int32[nblocks + 1]
    void *carry = nullptr;   // DEVICE value-typed[nblocks]: partial sums of rows that cross block boundaries
    int64_t nblocks = 0;
};

// Column-segmented copy for SpMV with a large x: the stored entries regrouped by column panel
// (panel = column >> shift), each panel a CSR over all rows, so that the x slice a panel gathers
// from stays in the per-XCD L2.  `seg` is a CSR tensor over panels*nrows virtual rows.
struct sp_segments {
    sp_tensor *seg = nullptr;
    int panels = 0, shift = 0;
    int64_t nrows = 0;
    void *partial = nullptr;          // DEVICE value-typed[panels * nrows]: per-panel results before they are added up
};

// Binned copy for SpMV with a large x and scattered columns: the stored entries regrouped into buckets (column panel
// of 2^pshift columns, row block of 2^rshift stored rows), panel-major, rows ascending inside a bucket.  Every entry keeps
// its value, its column inside the panel and its row inside the row block in 16 bits each.  The product runs in two
// streaming passes: one multiplies a panel's entries by the panel's slice of x held in LDS and writes the products in
// place (`prod`), the other adds a row block's products up in slices of y in the LDS.  No gather ever leaves the LDS.
struct sp_bins {
    // Entries regrouped into buckets (column panel, row block), every bucket padded to a multiple of 8 entries (np in all).
    // Panel-major arrays (buckets of a panel side by side, rows ascending inside a bucket):
    void *val = nullptr;              // DEVICE value-typed[np]; padding 0
    uint16_t *lcol = nullptr;         // DEVICE [np]: column - panel * 2^pshift; padding 2^pshift
    uint32_t *gdst = nullptr;         // DEVICE [np / 8]: group of 8 entries -> its group in the row-block-major arrays
    int64_t *pstart = nullptr;        // DEVICE [panels + 1]: first entry of each panel
    // Row-block-major arrays (buckets of a row block side by side):
    void *prod = nullptr;             // DEVICE value-typed[np]: the products of the running call
    uint16_t *lrow = nullptr;         // DEVICE [np]: stored row - rowblock * 2^rshift; padding 0
    int64_t *rbstart = nullptr;       // DEVICE [rowblocks + 1]: first entry of each row block
    int64_t nnz = 0, np = 0, nrows = 0;   // entries, entries with padding, stored rows
    int panels = 0, rowblocks = 0, pieces = 0, rshift = 0;
};


// Scratch that a handle keeps between products and makes larger on demand (spmi_reserve).
struct sp_kept {
    void *ptr;                        // DEVICE
    size_t bytes;
    bool shared;                      // something besides the calling stream may still use it: see spmi_reserve
};

// The per-block carries of the SpMM cut by stored entries: one block of scratch in three parts, each with room for `columns`
// values (part 0: for as many of them as its products have) per block.
//   0  products that have no other kernel of their speed (rows of 16-byte pieces): shared by all streams, the caller keeps
//      products of one tensor on different streams apart
//   1  products of any other width, which a kernel without scratch can do as well: used by one stream at a time, so that
//      such products may overlap on different streams
//   2  the same, recorded into one graph from one stream: its replays may overlap with anything else
struct sp_spmm_carry {
    sp_kept mem;
    int64_t columns;
    size_t offset[3];
    hipStream_t user[2];              // the stream that uses part 1 / part 2
    bool used[2];
    unsigned long long graph;         // the recording that uses part 2
};

struct sp_tensor {
    sp_encoding enc;
    int dtype;
    int64_t shape[SP_MAX_RANK];
    int64_t size[SP_MAX_RANK];       // by level
    void *pos[SP_MAX_RANK];          // DEVICE, nullptr for dense levels
    int64_t npos[SP_MAX_RANK];
    void *crd[SP_MAX_RANK];
    int64_t ncrd[SP_MAX_RANK];
    void *pos_narrow[SP_MAX_RANK];   // DEVICE copies in 8 or 16 bits when such a width was asked for, else nullptr
    void *crd_narrow[SP_MAX_RANK];
    void *values;
    int64_t nvalues;
    int64_t nnz;
    int64_t max_segment;
    sp_alloc_fn alloc;
    sp_free_fn free_;
    void *ctx;
    // Derived state: tables, regrouped copies and scratch that the product kernels use.  None of it is part of the paper's
    // storage; sp_pack builds some of it, sp_prepare (or, lazily, the first product that needs it) the rest.  It is a cache
    // in the C++ sense, hence `mutable`: a product takes the handle as const and may still fill it in.
    mutable sp_rowblocks rowblocks;
    // a dense outer level whose segments are mostly empty: ids and pos entries of the non-empty ones (else nullptr)
    mutable void *nz_rowid, *nz_pos;
    mutable int64_t nz_rows;
    mutable sp_rowblocks nz_rowblocks;
    mutable sp_tensor *transposed;           // CSC/DCSC viewed through a row-major copy (owned)
    mutable sp_segments *segments;           // owned, built on first use
    mutable sp_bins *bins;                   // owned, built on first use
    mutable double scatter;                  // share of stored entries whose successor lies in another 128-byte line of x; < 0: not measured yet
    mutable void *dense_partial;             // DEVICE scratch of the dense-row SpMV (per-chunk partial sums)
    mutable size_t dense_partial_bytes;
    mutable sp_spmm_carry spmm_carry;
    mutable sp_kept sddmm_bt;                // scratch of the SDDMM: the transposed dense operand (n x K)
    mutable void *mttkrp_windows;            // DEVICE int32[2 * windows]: fibre and slice holding the first entry of each window (rank 3)
    mutable sp_kept mttkrp_carry;            // scratch of the MTTKRP (J values per window)
    mutable sp_kept mttkrp_pad[2];           // scratch of the MTTKRP: inner / mid factor matrix with rows padded to whole cache lines
    mutable std::vector<void *> *outgrown;   // scratch that was outgrown while it was shared, owned
    mutable size_t outgrown_bytes;
    mutable int tables_pending;              // rowblocks / non-empty rows not built yet (a result of sp_spgemm): built on first use by a product
    mutable int plan_spmv;                   // SpMV kernel a product with one column runs (1..4); 0 = not decided yet (sp_prepare or the first product decides)
    mutable int plan_spmv_open;              // plan_spmv was taken by a product without sp_prepare, which may still decide otherwise
    mutable int lazy_prepares;               // how many products had to build, allocate or decide something first (none after sp_prepare)
    int tune_spmv, tune_csc, tune_spmm, tune_spgemm;
    int profile;
    std::vector<hipEvent_t> *prof_events;   // start/stop pairs, owned
};

extern thread_local int g_last_hip_error;

#define SP_HIP(call)                                            \
    do {                                                        \
        hipError_t e__ = (call);                                \
        if (e__ != hipSuccess) {                                \
            g_last_hip_error = (int)e__;                        \
            return SP_ERR_HIP;                                  \
        }                                                       \
    } while (0)

#define SP_TRY(call)                                            \
    do {                                                        \
        sp_status s__ = (call);                                 \
        if (s__ != SP_OK) return s__;                           \
    } while (0)

// Brackets the main kernel of a product with events when profiling is on.
struct sp_prof_scope {
    const sp_tensor *t; hipStream_t st; hipEvent_t stop = nullptr;
    sp_prof_scope(const sp_tensor *t_, hipStream_t st_) : t(t_), st(st_) {
        if (!t->profile || !t->prof_events) return;
        hipEvent_t a = nullptr;
        if (hipEventCreate(&a) != hipSuccess) return;
        if (hipEventCreate(&stop) != hipSuccess) { (void)hipEventDestroy(a); stop = nullptr; return; }
        (void)hipEventRecord(a, st);
        t->prof_events->push_back(a);
        t->prof_events->push_back(stop);
    }
    ~sp_prof_scope() { if (stop) (void)hipEventRecord(stop, st); }
};

static inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Device memory through the caller's allocator (or hipMalloc when none was given).
struct sp_mem {
    sp_alloc_fn alloc; sp_free_fn free_; void *ctx;
    void *get(size_t bytes) const;
    void put(void *p) const;
};

// Is work on this stream being recorded instead of run?  (An error counts as yes: what may not be asked now may not allocate
// either.)  graph (may be null): the number of the recording, 0 when it is not known.
bool spmi_recording(hipStream_t st, unsigned long long *graph = nullptr);
// Has everything enqueued on this stream been done?  (No while it is being recorded.)
bool spmi_idle(hipStream_t st);
// Room for `need` bytes in scratch the handle keeps; the contents do not survive.  A block that becomes too small is given back
// once `st` has done its work, unless it is shared: a graph recorded with it, or another stream, may use it at any time, so it
// stays with the handle (t->outgrown) until sp_tensor_free.
sp_status spmi_reserve(const sp_tensor *t, sp_kept &k, size_t need, hipStream_t st);

// A scope that frees its temporaries on exit.
struct sp_scratch {
    const sp_mem &mem;
    std::vector<void *> ptrs;
    explicit sp_scratch(const sp_mem &m) : mem(m) {}
    ~sp_scratch() { for (void *p : ptrs) mem.put(p); }
    void *get(size_t bytes) {
        void *p = mem.get(bytes ? bytes : 16);
        if (p) ptrs.push_back(p);
        return p;
    }
    // Takes a temporary out of the scope (its new owner frees it through the same allocator); false when p is not one.
    bool release(void *p) {
        for (size_t i = 0; i < ptrs.size(); ++i)
            if (ptrs[i] == p) { ptrs.erase(ptrs.begin() + (long)i); return true; }
        return false;
    }
};

// ---- device helpers shared by the sources ---------------------------------------------------
template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T v, int lane)
{
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        T o = __shfl_up(v, d, 64);
        if (lane >= d) v += o;
    }
    return v;
}

// Lanes of the wave that hold the same 8-bit digit as this lane (among lanes with valid set).  Per bit: the lanes that agree
// with this one are ~(ballot ^ mine), `mine` being all ones or all zeros; m & ~(ballot ^ mine) is one three-input bit
// operation per 32-bit half (truth table 0x90 with m as the first input), five vector instructions per bit in all.
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool valid)
{
    const uint64_t v = __builtin_amdgcn_ballot_w64(valid);
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const int mine = __builtin_amdgcn_sbfe((int)d, b, 1);
        const uint64_t bb = __builtin_amdgcn_ballot_w64(mine != 0);
        lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)bb, (uint32_t)mine, 0x90);
        hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(bb >> 32), (uint32_t)mine, 0x90);
    }
    return ((uint64_t)hi << 32) | lo;
}

// The row of every stored entry of a stretch [s, e) of a compressed innermost level (at most kThreads * PER entries), made by a
// whole block in LDS: row[at(i)] = the row of entry s + i, mapped through rowid where there is one.  pos(r) is where row r
// begins; lo..last are the rows that can meet the stretch, lo among those that begin at or before it.  Each row marks its first
// entry, the marks' running maximum is every entry's row.  waves: LDS, one int per wave.  The block meets at a barrier on the
// way in and out.
template <int kThreads, int PER, typename POS, typename CT, typename AT>
__device__ __forceinline__ void spmi_rows_of_entries(POS pos, const CT *__restrict__ rowid, int64_t lo, int64_t last, int64_t s,
                                                     int64_t e, CT *row, int *waves, AT at)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = (int)(e - s);
    if (pos(lo + 1) >= e) {                                        // one row holds them all (block-uniform)
        const CT only = rowid ? rowid[lo] : (CT)lo;
        for (int i = tid; i < n; i += kThreads) row[at(i)] = only;
        __syncthreads();
        return;
    }
    for (int i = tid; i < n; i += kThreads) row[at(i)] = 0;
    __syncthreads();
    for (int64_t r = lo + tid; r <= last; r += kThreads) {
        const int64_t pa = pos(r), pb = pos(r + 1);
        const int64_t a = pa > s ? pa : s, b = pb < e ? pb : e;
        if (a < b) row[at((int)(a - s))] = (CT)(r - lo);
    }
    __syncthreads();
    int run = 0, mark[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int x = tid * PER + i;
        mark[i] = x < n ? (int)row[at(x)] : 0;
        run = mark[i] > run ? mark[i] : run;
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) { const int v = __shfl_up(run, d, 64); if (lane >= d && v > run) run = v; }
    if (lane == 63) waves[wave] = run;
    int before = __shfl_up(run, 1, 64);
    if (lane == 0) before = 0;
    __syncthreads();
    for (int w = 0; w < wave; ++w) before = waves[w] > before ? waves[w] : before;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int x = tid * PER + i;
        before = mark[i] > before ? mark[i] : before;
        if (x < n) row[at(x)] = rowid ? rowid[lo + before] : (CT)(lo + before);
    }
    __syncthreads();
}

// Sums whose rounding error hardly grows with the number of terms.  f64: held as hi + lo, hi rounded and lo collecting what the
// additions to hi round off (Knuth's two-sum, exact for any two numbers); an infinity stays one, although lo is not a number
// then.  f32: held in f64.  half(i) / from(): the two vectors that a sum takes in memory.
template <typename VT, int V>
struct spmi_pair {
    typedef VT vec_t __attribute__((ext_vector_type(V)));
    vec_t hi, lo;
    __device__ __forceinline__ vec_t half(int i) const { return i ? lo : hi; }
    static __device__ __forceinline__ spmi_pair from(vec_t a, vec_t b) { spmi_pair p; p.hi = a; p.lo = b; return p; }
    __device__ __forceinline__ void add(const spmi_pair &o)
    {
        const vec_t s = hi + o.hi, b = s - hi;
        lo += o.lo + ((hi - (s - b)) + (o.hi - b));
        hi = s;
    }
    __device__ __forceinline__ vec_t value() const
    {
        vec_t r = hi + lo;
#pragma unroll
        for (int c = 0; c < V; ++c) r[c] = r[c] == r[c] ? r[c] : hi[c];
        return r;
    }
};
template <int V>
struct spmi_pair<float, V> {
    typedef float vec_t __attribute__((ext_vector_type(V)));
    typedef double sum_t __attribute__((ext_vector_type(V)));
    sum_t sum;
    __device__ __forceinline__ vec_t half(int i) const
    {
        vec_t h[2];
        __builtin_memcpy(h, &sum, sizeof(sum));
        return h[i];
    }
    static __device__ __forceinline__ spmi_pair from(vec_t a, vec_t b)
    {
        const vec_t h[2] = {a, b};
        spmi_pair p;
        __builtin_memcpy(&p.sum, h, sizeof(p.sum));
        return p;
    }
    __device__ __forceinline__ void add(const spmi_pair &o) { sum += o.sum; }
    __device__ __forceinline__ vec_t value() const
    {
        vec_t r;
#pragma unroll
        for (int c = 0; c < V; ++c) r[c] = (float)sum[c];
        return r;
    }
};
// One lane's long sum, which gets a few terms at a time, added up in VT before.  value(t), pair(t): with the last of them.
// f64: with a cheaper addition that is exact where hi is the larger one (Dekker's; only the first few terms are not smaller).
template <typename VT, int V>
struct spmi_long_sum {
    typedef typename spmi_pair<VT, V>::vec_t vec_t;
    spmi_pair<VT, V> p;
    __device__ __forceinline__ void clear() { p.hi = (vec_t)(0); p.lo = (vec_t)(0); }
    __device__ __forceinline__ void add(vec_t t)
    {
        const vec_t s = p.hi + t;
        p.lo += t - (s - p.hi);
        p.hi = s;
    }
    __device__ __forceinline__ vec_t value(vec_t t) const
    {
        vec_t r = p.hi + (p.lo + t);
#pragma unroll
        for (int c = 0; c < V; ++c) r[c] = r[c] == r[c] ? r[c] : p.hi[c] + t[c];
        return r;
    }
    __device__ __forceinline__ spmi_pair<VT, V> pair(vec_t t) const
    {
        spmi_pair<VT, V> q = p;
        q.add(spmi_pair<VT, V>::from(t, (vec_t)(0)));
        return q;
    }
};
template <int V>
struct spmi_long_sum<float, V> {
    typedef typename spmi_pair<float, V>::vec_t vec_t;
    spmi_pair<float, V> p;
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int c = 0; c < V; ++c) p.sum[c] = 0;
    }
    __device__ __forceinline__ void add(vec_t t)
    {
#pragma unroll
        for (int c = 0; c < V; ++c) p.sum[c] += (double)t[c];
    }
    __device__ __forceinline__ spmi_pair<float, V> pair(vec_t t) const
    {
        spmi_pair<float, V> q = p;
#pragma unroll
        for (int c = 0; c < V; ++c) q.sum[c] += (double)t[c];
        return q;
    }
    __device__ __forceinline__ vec_t value(vec_t t) const { return pair(t).value(); }
};

// Of 64 entries the sort's sampled histogram takes one, at a place that changes from group to group: entries often come in
// order, and with rows of 64 a fixed place would be the same one of every row (a full last column would never be seen).
__device__ __forceinline__ uint32_t spmi_sampled_place(uint32_t group) { return (group * 2654435761u) >> 26; }

// Division of a key by a level's stride or size, which the host knows when it launches: a shift when the divisor is a
// power of two, a multiplication by the reciprocal in double plus a one-step correction while the dividend is below
// 2^52 (the estimate is then within one of the quotient), the hardware's 64-bit division otherwise.
struct spmi_divisor {
    uint64_t d;
    double inv;
    int shift;          // >= 0: d == 1 << shift
};

static inline spmi_divisor spmi_make_divisor(uint64_t d)
{
    spmi_divisor v;
    v.d = d;
    v.inv = 1.0 / (double)d;
    v.shift = -1;
    if ((d & (d - 1)) == 0) { v.shift = 0; while (((uint64_t)1 << v.shift) != d) ++v.shift; }
    return v;
}

__device__ inline uint64_t spmi_div_by(uint64_t x, const spmi_divisor &v)
{
    if (v.shift >= 0) return x >> v.shift;
    if (x < ((uint64_t)1 << 52)) {
        uint64_t q = (uint64_t)((double)x * v.inv);
        const int64_t r = (int64_t)(x - q * v.d);
        if (r < 0) --q;
        else if ((uint64_t)r >= v.d) ++q;
        return q;
    }
    return x / v.d;
}

// ---- levels.hip ----
// First half of the level sweep over n sorted keys: *counts = what the second half needs (a temporary of `tmp`; null when no
// compressed level lies above the innermost one), totals[0..] (DEVICE, one per such level from the outermost on) = their sizes.
sp_status spmi_sweep_count(const sp_tensor *t, const uint64_t *keys, int64_t n, sp_scratch &tmp, hipStream_t st, unsigned long long *totals,
                           uint32_t **counts);
// Second half: writes crd and pos of every compressed level of t (allocated by the caller; pos under a dense level is left as
// counts to be scanned, and arrives zeroed), and, where the innermost level is dense (vout not null), every value to its position.
// dup_flags (may be null): dup_flags[1] is set when a key occurs twice.
sp_status spmi_sweep_emit(const sp_tensor *t, const uint64_t *keys, int64_t n, const uint32_t *counts, const void *vals, void *vout, int *dup_flags,
                          hipStream_t st);

// ---- pack.hip ----------------------------------------------------------------------------
// In-place exclusive prefix sum of n elements of width `bits` (32 or 64); data[n-1] afterwards
// holds the sum of the first n-1 inputs.
sp_status spmi_exclusive_scan(void *data, int64_t n, int bits, sp_scratch &tmp, hipStream_t st);
sp_status spmi_fill_zero(void *p, size_t bytes, hipStream_t st);
// ---- sort.hip ----
// Stable radix sort, least significant digit first, of (key, payload) pairs on the low `key_bits` bits taken as whole 8-bit
// digits (so ceil(key_bits / 8) * 8 bits decide), payload of 4 or 8 bytes.  keys: a temporary of `tmp`, overwritten; vals: only
// read.  *keys_out / *vals_out: where the sorted arrays are (temporaries of `tmp`, or the inputs themselves when there was
// nothing to sort).
sp_status spmi_radix_sort_pairs(uint64_t *keys, const void *vals, int payload_bytes, int64_t n, int key_bits, sp_scratch &tmp,
                                hipStream_t st, uint64_t **keys_out, const void **vals_out);
// The same sort (same arguments, same stability) with the most significant digits first: two passes over device memory, the
// rest inside the LDS.  Only for inputs that spmi_msd_sort_suits() accepted: enough entries, keys wide enough, and (from a
// sampled histogram of the top 16 key bits, samp_ready when the caller has it already; synchronises the stream) either few
// entries in groups of equal top 16 key bits too large for the LDS, none of them huge, or all groups of about a size that
// the larger finishing kernel holds.
//
// Whoever makes the keys can fill in, on the way, what the first pass would otherwise read them for (sp_msd_plan, empty when
// this sort is out of the question): for the tile e / kSpmiMsdTile of entry e, ctr[digit * tiles + tile] counts the entries
// whose digit is (key >> digit_shift) & 255 (every word written, zero included), and samp[(key >> samp_shift) & 0xffff]
// counts one entry of 64 (entry e with e % 64 == spmi_sampled_place(e / 64); samp arrives zeroed).
#ifndef SPMI_SORT_T
#define SPMI_SORT_T 256
#endif
constexpr int kSpmiMsdTile = SPMI_SORT_T * 16;
struct sp_msd_plan { uint32_t *ctr, *samp; uint32_t tiles; int digit_shift, samp_shift; };
sp_status spmi_msd_plan(int64_t n, int key_bits, sp_scratch &tmp, hipStream_t st, sp_msd_plan *plan);
sp_status spmi_msd_sort_suits(const uint64_t *keys, int64_t n, int key_bits, sp_scratch &tmp, hipStream_t st, uint32_t *samp_ready, bool *suits);
sp_status spmi_msd_sort_pairs(uint64_t *keys, const void *vals, int payload_bytes, int64_t n, int key_bits, sp_scratch &tmp, hipStream_t st,
                              uint32_t *ctr_ready, uint64_t **keys_out, const void **vals_out);
// Whichever of the two suits (or the one that sp_pack_sort_mode() of the bench header forces); plan: null, or what
// spmi_msd_plan() handed out and the maker of the keys filled in.
sp_status spmi_sort_pairs(uint64_t *keys, const void *vals, int payload_bytes, int64_t n, int key_bits, sp_scratch &tmp, hipStream_t st,
                          const sp_msd_plan *plan, uint64_t **keys_out, const void **vals_out);
extern std::atomic<int> g_pack_sort_mode;
// ---- buckets.hip ----
// The builder's sort for entries with distinct keys (equal ones are reported, not ordered).  spmi_bucket_plan_for() says whether
// n entries with keys below `total` suit it and how they will be cut; rows: as in spmi_bucket_out, 0 where anything else leaves.
// The caller fills in a job; spmi_bucket_begin() takes scratch and enqueues the sample and the partitions, spmi_bucket_end() the
// finishing pass (so that the arrays it writes are allocated while the GPU is busy).
// Entries come as coordinates by level (checked against the sizes: flags[0]) or as keys; neither they nor vals are changed.  What
// leaves is one of
//   the sorted keys and values;
//   crd, pos and values of an innermost compressed level of size `inner` under `rows` positions of dense ones, and, where rowblk is
//   given, the row of every kSpmiStreamT-th entry;
//   dist (32-bit keys only) and values: then flags + 16 has the sizes of the levels (64 bits each, from the second on; job.levels,
//   counted from the innermost outwards), and spmi_bucket_levels() writes crd and pos of them all.  pos of the outermost
//   one arrives zeroed and is left as counts to be scanned where dense levels lie above it.
// flags (job.flags, zeroed by spmi_bucket_begin), once the stream is done: [0] a coordinate was out of range, [1] a key occurs
// twice, [2] or [3] a bucket overflowed: the outputs are of no use then (keys stay below total, dist and heads must not be
// used) and the stable sorts have to do it.
constexpr size_t kSpmiFlagBytes = 64 + 8 * SP_MAX_RANK;              // the flags of a build: 64 bytes of them, then the sizes of levels
struct spmi_bucket_source {
    const int64_t *coord[SP_MAX_RANK];   // by level, or
    const uint64_t *keys;                // the keys themselves (coord unused)
    int64_t size[SP_MAX_RANK];
    int rank;
};
struct spmi_levels { int count; spmi_divisor size[SP_MAX_RANK]; };   // compressed levels from the innermost outwards (0: not wanted)
// buckets by sample, multiples of 2^fbits, sampled keys; compressed levels above the innermost; two partitions, 64-bit keys
struct spmi_bucket_plan { uint32_t Q, F, S; int fbits, slots; bool two, wide; };
struct spmi_bucket_job {
    spmi_bucket_source src;
    spmi_bucket_plan plan;
    spmi_levels levels;
    int64_t n;
    uint64_t total;
    int key_bits, payload_bytes;
    void *tab;
    int *flags;                          // DEVICE, kSpmiFlagBytes
};
struct spmi_bucket_out { uint64_t *keys; uint32_t *dist; void *values, *crd, *pos; int32_t *rowblk; int64_t rows; uint64_t inner; int pw, cw; };
bool spmi_bucket_plan_for(int64_t n, uint64_t total, int key_bits, int64_t rows, spmi_bucket_plan *plan);
sp_status spmi_bucket_begin(spmi_bucket_job *job, const void *vals, int payload_bytes, sp_scratch &tmp, hipStream_t st);
sp_status spmi_bucket_end(const spmi_bucket_job &job, const spmi_bucket_out &out, sp_scratch &tmp, hipStream_t st);
sp_status spmi_bucket_levels(const spmi_bucket_job &job, const uint32_t *dist, void *const *crd, void *const *pos, bool dense_above, int pw, int cw, hipStream_t st);
// ---- pack.hip ----
// The storage of a tensor whose n entries are given as linearised keys (level order, mixed radix over the level sizes)
// with the value bits as payload, both temporaries of `tmp`; entries with equal keys are added up in the order given.
sp_status spmi_pack_keys(const sp_encoding *enc, const int64_t *shape, sp_dtype dt, sp_alloc_fn alloc, sp_free_fn free_, void *ctx,
                         int64_t n, uint64_t *keys, void *payload, sp_scratch &tmp, hipStream_t st, sp_tensor **out);
// Every stored position of `from` packed under another encoding of the same rank; synchronises.
sp_status spmi_repack(const sp_tensor *from, const sp_encoding *enc, hipStream_t st, sp_tensor **out);
sp_status spmi_build_rowblocks(const sp_tensor *t, hipStream_t st);
sp_status spmi_build_segments(const sp_tensor *A, int64_t row_bytes, int64_t slice_bytes, hipStream_t st);
#ifndef SPMI_BIN_PSHIFT
#define SPMI_BIN_PSHIFT 13
#endif
#ifndef SPMI_BIN_RSHIFT
#define SPMI_BIN_RSHIFT 11
#endif
constexpr int kSpmiBinPanelShift = SPMI_BIN_PSHIFT;          // columns per panel of the binned copy: 8192 (a 64 KB slice of an f64 x)
constexpr int kSpmiBinRowShift = SPMI_BIN_RSHIFT;            // most rows per row block: 2048 (16 KB per slice of y: four slices for f64, one of f64 sums for f32)
// Rows per row block (a power of two) of the binned copy of nnz entries in m stored rows: 2048, or fewer where these would leave
// CUs without a row block in the second pass, as long as a bucket keeps 24 entries (padding to eights stays near a seventh).
// 2.7 M entries in 83,886 rows, x of 4 MB: 37 us a product in 41 row blocks of 2048, 29 in 164 of 512.
static inline int spmi_bin_row_shift(int64_t nnz, int64_t m, int64_t panels)
{
    int shift = kSpmiBinRowShift;
    while (shift > 8 && ceil_div(m, (int64_t)1 << shift) < 128 && (double)nnz >= 24.0 * (double)panels * (double)ceil_div(m, (int64_t)1 << (shift - 1))) --shift;
    return shift;
}
sp_status spmi_build_bins(const sp_tensor *A, hipStream_t st);
// How scattered the gathers of a product are: the share of stored entries of the innermost level whose successor is 16 or
// more coordinates away (or belongs to the next segment).  Measured once per tensor, then cached; synchronises the first time.
sp_status spmi_column_scatter(const sp_tensor *A, hipStream_t st, double *share);
#ifndef SPMI_ST
#define SPMI_ST 128
#endif
#ifndef SPMI_PER
#define SPMI_PER 8
#endif
constexpr int kSpmiStreamThreads = SPMI_ST;                  // threads per block of the stream kernel
constexpr int kSpmiStreamPer = SPMI_PER;                     // stored entries per thread (even)
constexpr int64_t kSpmiStreamT = kSpmiStreamThreads * kSpmiStreamPer;     // stored entries per block

// keys[e] = linearised key, in the level order of `shaped` (a tensor handle whose enc and size[] are set), of the entry
// with coordinates coords[d][e]; flags[0] != 0 afterwards on the device when a coordinate was out of range.
sp_status spmi_make_keys(const sp_tensor *shaped, const int64_t *const *coords, int64_t n, uint64_t *keys, int *flags, hipStream_t st);
// A new tensor handle with shape, sizes by level and the key width worked out (SP_ERR_TOO_LARGE, SP_ERR_WIDTH as sp_pack
// documents; `entries_in_an_empty_dimension` turns into SP_ERR_COORD_RANGE at its place in that order).
sp_status spmi_new_tensor(const sp_encoding *enc, const int64_t *shape, sp_dtype dt, sp_alloc_fn alloc, sp_free_fn free_, void *ctx,
                          bool entries_in_an_empty_dimension, sp_tensor **out, int *key_bits_out);
// The derived tables of a finished storage (see pack.hip); flags: 64 device bytes, the second half zero; input_flags: HOST
// int[2] that receives flags[0..1] (nothing more is built when one is set), or null.
sp_status spmi_finish_tensor(sp_tensor *t, int *flags, sp_scratch &tmp, hipStream_t st, int *input_flags);
// *out (DEVICE, zero before the call) = the longest of the nseg segments of a pos array of width pw; enqueued only.
sp_status spmi_max_segment_async(const void *pos, int pw, int64_t nseg, unsigned long long *out, hipStream_t st);
// Builds the tables a product kernel reads (row blocks, non-empty rows) when the tensor still lacks them; synchronises then.
sp_status spmi_ensure_tables(const sp_tensor *t, hipStream_t st);
// Hands the tensor out on SP_OK, releases everything it holds otherwise.
sp_status spmi_finish_pack(sp_tensor *t, sp_status status, hipStream_t st, sp_tensor **out);

// ---- api.hip -----------------------------------------------------------------------------
// Builds and keeps the row-major copy of a column-major tensor (A->transposed); no-op when it exists.
sp_status spmi_build_transposed(const sp_tensor *A, hipStream_t st);

// ---- matmul.hip --------------------------------------------------------------------------
sp_status spmi_matmul_rowmajor(const sp_tensor *A, const void *B, int64_t N, int64_t ldb,
                               void *C, int64_t ldc, int accumulate, hipStream_t st);
// Everything a product of a row-major tensor (compressed / dense innermost level) with N columns would otherwise build on
// first use: the kernel choice, regrouped copies, scratch.  May allocate and synchronise; a no-op when nothing is missing.
sp_status spmi_prepare_rowmajor(const sp_tensor *A, int64_t N, hipStream_t st);
sp_status spmi_prepare_dense_inner(const sp_tensor *A, int64_t N, hipStream_t st);
sp_status spmi_matmul_dense_inner(const sp_tensor *A, const void *B, int64_t N, int64_t ldb, void *C, int64_t ldc,
                                  int accumulate, hipStream_t st);
sp_status spmi_matmul_colmajor_scatter(const sp_tensor *A, const void *B, int64_t N, int64_t ldb,
                                       void *C, int64_t ldc, int accumulate, hipStream_t st);
