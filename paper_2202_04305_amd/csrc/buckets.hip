// The storage builder's sort by buckets (arXiv 2202.04305, Section 4.2: the entries of the coordinate scheme are brought into the
// level order of the target format before its arrays are built).  For entries with distinct keys: the order of equal keys is not
// kept, they are only reported (sort.hip has the stable sorts).
//
// The key range is cut into buckets by splitters taken from a sorted sample, so that buckets hold about the same number of
// entries whatever the pattern is; entries are moved straight from where the caller has them (coordinates, or keys made from
// another encoding) into their buckets; a block then sorts one bucket in the LDS and writes the finished arrays.
//
//   sample      up to 32768 keys, sorted in runs of 1024, ranked against each other: the splitters
//   partition   a block takes a tile of entries, finds every entry's bucket, reserves room in each bucket with one atomic add, orders
//               the tile by bucket in the LDS and writes runs.  No counting pass: a bucket's room is what the sample says
//               plus six standard deviations.  Keys shrink to 32 bits where no bucket spans more (multiples of 2^32 are
//               splitters too): 12 bytes per entry from here on.
//   second partition, above a million entries: the same inside each bucket, its splitters from a count of its keys by equal intervals
//               (a sample again where one interval holds too much)
//   finish      a block per bucket: sorted by value in the LDS; then crd, pos and values leave (levels above the innermost all dense), or
//               32-bit distances from which bucket_levels_kernel writes every level (compressed levels inside dense ones), or the
//               sorted keys (any other format: the level sweep does the rest)
//
// Should a bucket get more entries than its room (a sample that misleads, or many equal keys), nothing is written out of
// bounds, the build is marked and the caller builds again with the stable sorts.
//
// What bounds it: memory; in the finishing kernel vector instructions (issued in 53 % of the busy cycles; bank conflicts of the LDS 17 %).  Per entry of a CSR matrix in f64: 24 bytes read and 12
// written, 4 read, 12 and 12, 12 and 12.  16.9 M entries of a 1M x 1M lognormal matrix, kernel by kernel: sample and its ranks
// 26 us, first partition 155 to 165 (3.8 TB/s), cutting the buckets 45, second partition 102 (4.0), finish 144 (2.8); the whole call
// 841 us with the stable sorts, 575 now.  76.9 M entries of rank 3, all levels compressed: 960, 132, 415 (4.4), 535 and
// levels 350; 3490 us, 2665 now.
// Reserving room instead of counting first, 16.9 M entries into 256 buckets: 128 us for all of it, against 70 for a counting pass, 25
// to scan its table and 90 to move.  One partition into thousands of buckets instead of two: runs of two entries (8192 buckets:
// 2.3 TB/s); no LDS staging, each entry written where it belongs: 1.2 to 1.6 times as long.
#include <algorithm>
#include <cmath>
#include "spmi_internal.h"

namespace {

constexpr int kMaxBuckets = 3072;             // of the first partition
constexpr int kCells = 2048;                  // equal parts of the key range, each knowing which buckets it meets
constexpr int kRun = 1024;                    // sampled keys a block sorts
constexpr int kMaxSample = 32 * kRun;
constexpr int kSubSample = 8192;              // most keys sampled inside one bucket
constexpr int kShare = 48;                    // sampled keys per final bucket
constexpr int kOnePartition = 512;             // final buckets up to which one partition makes them (1.39 M entries: 205 us with one, 1.4 M 179 with two; 1 M: 156)
constexpr int kShareFirst = 32;               // sampled keys per bucket that is partitioned again
constexpr int kPR = 12;                       // partition: entries per thread
constexpr int kPT = 512, kWideT = 1024;       // its threads: the second partition and small inputs, the first one
constexpr int kSmallR = 2;                    // entries per thread where larger tiles would leave most of the chip idle
constexpr int kFT = 256, kFE = 16;            // finishing kernel: threads, entries per thread
constexpr int kCap = kFT * kFE;               // entries a block sorts in the LDS
constexpr int kTarget = 2048;                 // entries per final bucket where a sample cuts them
constexpr int kExact = 3456;                  // the same where they are counted first
constexpr int kPartCells = 16384;             // equal intervals of a bucket whose entries are counted
constexpr int kHeavy = 512;                   // more entries than this in one of them: a sample cuts the bucket (kExact + kHeavy < kCap)
constexpr int kFirstLeast = 16384, kFirst = 131072;         // entries per bucket of the first of two partitions: n / 128 between these
constexpr int kCells1 = 4 * kFT;              // equal intervals of a final bucket, each then cut by what it holds
constexpr int kSpread = 24;                   // more keys than this in one interval: a second attempt at spreading them
constexpr int kCrowd = 32;                    // more keys than this in one interval then: left to a merge sort (R-MAT, 48-bit keys, 2.5 M entries: 414 us a call, 435 with 96)

typedef spmi_bucket_source source;

// key of entry e; a coordinate out of range sets bad and makes the key 0
__device__ __forceinline__ uint64_t key_of(const source &s, int64_t e, bool &bad)
{
    if (s.keys) return s.keys[e];
    uint64_t key = 0;
    bool b = false;
    for (int l = 0; l < s.rank; ++l) {
        const int64_t c = s.coord[l][e];
        b |= (c < 0) | (c >= s.size[l]);
        key = key * (uint64_t)s.size[l] + (uint64_t)c;
    }
    bad |= b;
    return b ? 0 : key;
}

// A published 32-bit mixer: lowbias32, found by Chris Wellons' hash-prospector.
__device__ __forceinline__ uint32_t scramble(uint32_t x)
{
    x ^= x >> 16; x *= 0x7feb352du;
    x ^= x >> 15; x *= 0x846ca68bu;
    return x ^ (x >> 16);
}

// position of sample i of S among n entries: one per stretch of n / S, at a scrambled place in it (entries often come in an order
// with a period)
__device__ __forceinline__ int64_t sampled_position(uint32_t i, uint32_t S, int64_t n)
{
    const int64_t at = (int64_t)(((double)i + (double)scramble(i) * 0x1p-32) * ((double)n / (double)S));
    return at < n ? at : n - 1;
}

// Bitonic sort of S numbers (a power of two, 1024 * E at most) by a block of 1024 threads: thread t holds numbers t, t + 1024, ...  Steps
// between lanes of a wave are shuffles, steps of 1024 and more stay in the thread, the others go through the LDS.  Sorted numbers
// are left in key.
template <int E>
__device__ __forceinline__ void block_sort(uint32_t (&x)[E], uint32_t S, uint32_t *key)
{
    const uint32_t tid = threadIdx.x;
#pragma unroll 1
    for (uint32_t size = 2; size <= S; size *= 2) {
#pragma unroll 1
        for (uint32_t half = size / 2; half > 0; half /= 2) {
            if (half >= 1024) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
#pragma unroll
                    for (int h = 1; h < E; h *= 2) {
                        if ((e & h) == 0 && half == (uint32_t)h * 1024u && (uint32_t)(e | h) * 1024u < S) {
                            const bool up = ((tid + (uint32_t)e * 1024u) & size) == 0;
                            const uint32_t a = x[e], c = x[e | h];
                            x[e] = (a < c) == up ? a : c;
                            x[e | h] = (a < c) == up ? c : a;
                        }
                    }
                }
                continue;
            }
            if (half >= 64) {
                __syncthreads();
#pragma unroll
                for (int e = 0; e < E; ++e)
                    if (tid + (uint32_t)e * 1024u < S) key[tid + e * 1024] = x[e];
                __syncthreads();
            }
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const uint32_t i = tid + (uint32_t)e * 1024u;
                if ((uint32_t)e * 1024u < S) {
                    const uint32_t o = half >= 64 ? key[(i ^ half) < S ? i ^ half : 0u] : (uint32_t)__shfl_xor((int)x[e], (int)half, 64);
                    const bool keep_less = ((i & half) == 0) == ((i & size) == 0);
                    x[e] = (x[e] < o) == keep_less ? x[e] : o;
                }
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (tid + (uint32_t)e * 1024u < S) key[tid + e * 1024] = x[e];
    __syncthreads();
}

// A block sorts kRun sampled keys (their upper 32 bits).
__global__ __launch_bounds__(kRun) void sample_runs_kernel(source s, int64_t n, uint32_t S, int shift, uint32_t *__restrict__ runs)
{
    __shared__ uint32_t key[kRun];
    const uint32_t i = blockIdx.x * kRun + threadIdx.x;
    bool bad = false;
    uint32_t x[1] = {(uint32_t)(key_of(s, sampled_position(i, S, n), bad) >> shift)};
    block_sort<1>(x, kRun, key);
    runs[i] = key[threadIdx.x];
}

// Every sampled key's place among all of them, from a binary search in each of the other runs (all runs in the LDS); those whose
// place begins a share of S / Q become splitters.  The multiples of 2^32 get their places the same way.
constexpr int kRankT = 256;
__global__ __launch_bounds__(kRankT) void sample_ranks_kernel(const uint32_t *__restrict__ runs, uint32_t S, int shift, uint32_t Q, uint32_t F,
                                                              uint32_t *__restrict__ splitter, uint32_t *__restrict__ forced_rank, int fbits)
{
    extern __shared__ __align__(16) uint32_t key[];
    for (uint32_t i = threadIdx.x; i < S / 4; i += kRankT) ((uint4 *)key)[i] = ((const uint4 *)runs)[i];
    __syncthreads();
    const uint32_t i = blockIdx.x * kRankT + threadIdx.x, nruns = S / kRun;
    if (i >= S + F) return;
    const uint32_t mine = i < S ? key[i] : (uint32_t)(((uint64_t)(i - S + 1) << fbits) >> shift);
    const uint32_t own = i < S ? i / kRun : nruns;
    uint32_t rank = i < S ? i % kRun : 0;
    for (uint32_t r0 = 0; r0 < nruns; r0 += 4) {
        uint32_t at[4] = {0, 0, 0, 0};                       // keys of the run that come before mine: equal ones of an earlier run do
#pragma unroll
        for (uint32_t w = kRun / 2; w > 0; w >>= 1) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t r = r0 + j < nruns ? r0 + j : r0;
                const uint32_t o = key[r * kRun + at[j] + w - 1];
                if (o < mine || (o == mine && r < own && i < S)) at[j] += w;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t r = r0 + j;
            if (r < nruns && r != own) {
                const uint32_t o = key[r * kRun + at[j]];    // at <= kRun - 1 so far: one more step
                rank += at[j] + ((o < mine || (o == mine && r < own && i < S)) ? 1u : 0u);
            }
        }
    }
    if (i >= S) { forced_rank[i - S] = rank; return; }
    const uint32_t j = (uint32_t)(((uint64_t)rank * Q + S - 1) / S);
    if (j >= 1 && j < Q && (uint32_t)(((uint64_t)j * S) / Q) == rank) splitter[j - 1] = mine;
}

// Room for a bucket that d of S sampled keys fell into: its share of n plus six standard deviations and a little.
__host__ __device__ inline uint64_t room_for(double d, double S, double n)
{
    const double r = n / S * (d + 6.0 * sqrt(d + 4.0) + 10.0);
    return ((uint64_t)(r < n ? r : n) + 31u) & ~(uint64_t)15u;
}

struct level1 {
    uint64_t *lo;             // [B + 1] smallest key of each bucket; lo[B] = the end of the key range
    uint32_t *start, *end;    // [B] room of each bucket
    uint32_t *cur;            // [B] where the next entry goes (beyond end: overflow)
    uint16_t *lut;            // [kCells + 1] bucket of the first key of each cell
    uint32_t *out;            // [B + 1] where the bucket's entries end up in the sorted order
    uint32_t *sub0;           // [B + 1] first part of each bucket (two partitions)
    uint32_t *tile0;          // [B + 1] first tile of each bucket
    uint32_t *room2;          // [B] where the room of its parts begins
    uint32_t *used;           // [B] how many parts it has (those after them stay empty)
    int B;
};

__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t *wsum, uint32_t &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const uint32_t incl = wave_inclusive_scan(v, lane);
    __syncthreads();
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t before = incl - v;
    total = 0;
    for (int w = 0; w < waves; ++w) { before += w < wave ? wsum[w] : 0u; total += wsum[w]; }
    return before;
}

// One block: the splitters and the multiples of 2^32 merged into the buckets' lower ends, room for each of them, the cells' table.
__global__ __launch_bounds__(1024) void buckets_kernel(const uint32_t *__restrict__ splitter, const uint32_t *__restrict__ forced_rank, uint32_t S,
                                                       int shift, uint32_t Q, uint32_t F, int fbits, uint64_t total, int cell_shift, int64_t n, level1 t, int *__restrict__ flags)
{
    __shared__ uint64_t lo[kMaxBuckets + 1];
    __shared__ uint32_t rank[kMaxBuckets + 1];
    __shared__ uint32_t wsum[16];
    const int tid = threadIdx.x;
    const uint32_t B = Q + F;
    if (tid < (int)(kSpmiFlagBytes / 4)) flags[tid] = 0;
    if (tid == 0) { lo[0] = 0; rank[0] = 0; lo[B] = total; rank[B] = S; }
    for (uint32_t i = tid; i + 1 < Q; i += 1024) {
        const uint64_t v = (uint64_t)splitter[i] << shift;
        const uint32_t f = (uint32_t)((v >> fbits) < F ? (v >> fbits) : F);
        lo[1 + i + f] = v;
        rank[1 + i + f] = (uint32_t)(((uint64_t)(i + 1) * S) / Q);
    }
    for (uint32_t j = tid; j < F; j += 1024) {
        const uint64_t v = (uint64_t)(j + 1) << fbits;
        uint32_t a = 0, z = Q - 1;                               // splitters below v
        while (a < z) {
            const uint32_t mid = (a + z) / 2;
            if (((uint64_t)splitter[mid] << shift) < v) a = mid + 1;
            else z = mid;
        }
        lo[1 + j + a] = v;
        rank[1 + j + a] = forced_rank[j];
    }
    __syncthreads();
    uint32_t run = 0;
    for (uint32_t b0 = 0; b0 < B; b0 += 1024) {
        const uint32_t b = b0 + tid;
        uint32_t room = 0;
        if (b < B) {
            const uint32_t d = rank[b + 1] > rank[b] ? rank[b + 1] - rank[b] : 0u;
            room = S ? (uint32_t)room_for((double)d, (double)S, (double)n) : (uint32_t)((n + 31) & ~(int64_t)15);
        }
        uint32_t all;
        const uint32_t at = run + block_exclusive_scan(room, wsum, all);
        run += all;
        if (b < B) { t.lo[b] = lo[b]; t.start[b] = at; t.end[b] = at + room; t.cur[b] = at; }
    }
    if (tid == 0) t.lo[B] = total;
    for (int c = tid; c <= kCells; c += 1024) {
        const uint64_t first = (uint64_t)c << cell_shift;
        uint32_t a = 0, z = B - 1;                               // last bucket that begins at or before the cell
        while (a < z) {
            const uint32_t mid = (a + z + 1) / 2;
            if (lo[mid] <= first) a = mid;
            else z = mid - 1;
        }
        t.lut[c] = (uint16_t)a;
    }
}

// The workgroups of a launch go to the eight XCDs in turn: block b takes tile (b / 8) of the (b % 8)-th eighth, so that an XCD
// runs neighbouring tiles together and the lines that two runs share are completed in one L2.
inline unsigned round8(uint32_t n) { return (n + 7u) & ~7u; }
__device__ __forceinline__ uint32_t tile_of_block() { return (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3); }

// Place s of c in a mixed order (a permutation of 0 .. c - 1): steps that can be taken back on the first power of two of places, then
// on the last.
constexpr uint32_t kMixed = 256;
__device__ __forceinline__ uint32_t mixed_place(uint32_t s, uint32_t c)
{
    const int bits = 31 - __clz((int)c), half = bits / 2;
    const uint32_t mask = (1u << bits) - 1u, last = c - (1u << bits);
    auto mix = [&](uint32_t x) {
        x = __umul24(x, 0x4e5u) & mask;
        x ^= x >> half;
        x = __umul24(x, 0x2adu) & mask;
        return x ^ (x >> half);
    };
    if (s <= mask) s = mix(s);
    return s >= last ? last + mix(s - last) : s;
}

// The tile in registers (key k, bucket b, payload v; cnt entries, entry r * PT + tid in round r) to its buckets.  cur: LDS counters [B],
// all zero; stage: LDS, room for the tile's keys and buckets, then for its payloads; next / end: the buckets' places in memory.
// Entries of a bucket that is full go to the tile-sized stretch at `dump`, which nobody reads.
// MIX: a bucket that gets kMixed entries or more of the tile gets them in a mixed order.  Input that is sorted already would keep its
// neighbours together, and the kernels that count them later would have whole waves add to one address (bands of 64 entries, sorted,
// 8 M in CSR: cutting the buckets 61 us against 18 shuffled, the finishing kernels 79 + 237 against 35 + 119; the call 599 us, 402).
template <typename K, typename P, int PT, int R, int PER, bool MIX>
__device__ __forceinline__ void move_tile(const K (&k)[R], const uint32_t (&b)[R], const P (&v)[R], int cnt, int B, uint32_t *cur, uint32_t *wsum,
                                          void *stage, uint32_t *__restrict__ next, const uint32_t *__restrict__ end, uint32_t dump,
                                          K *__restrict__ kout, P *__restrict__ vout)
{
    constexpr int T = PT * R;
    K *sk = (K *)stage;
    uint16_t *sb = (uint16_t *)(sk + T);
    P *sv = (P *)stage;
    const int tid = threadIdx.x;
    uint32_t slot[R];
    // lanes that agree with the wave's first one take their numbers with one add: entries that come in the order of the keys or nearly
    // so would queue up at one counter
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r * PT + tid < cnt) {
            const uint32_t same = (uint32_t)__builtin_amdgcn_readfirstlane((int)b[r]);
            const uint64_t m = __ballot(b[r] == same);
            if (__popcll(m) < 16) slot[r] = atomicAdd(&cur[b[r]], 1u);
            else {
                uint32_t at = 0;
                if (b[r] == same) {
                    const uint32_t before = (uint32_t)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                    if (before == 0) at = atomicAdd(&cur[same], (uint32_t)__popcll(m));
                    slot[r] = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + before;
                } else slot[r] = atomicAdd(&cur[b[r]], 1u);
            }
        }
    }
    __syncthreads();
    const int per = (B + PT - 1) / PT;                             // <= PER consecutive buckets per thread
    uint32_t g[PER], tot = 0, all;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int x = tid * per + j;
        g[j] = 0;
        if (j < per && x < B) {
            const uint32_t c = cur[x];
            tot += c;
            if (c) {
                g[j] = atomicAdd(&next[x], c);
                if (g[j] + c > end[x] || g[j] + c < g[j]) g[j] = dump;
            }
        }
    }
    uint32_t start = block_exclusive_scan(tot, wsum, all);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int x = tid * per + j;
        if (j < per && x < B) {
            const uint32_t c = cur[x];
            cur[x] = MIX ? start | (c << 16) : start;                // both below 2^14
            g[j] -= start;
            start += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r * PT + tid < cnt) {
            const uint32_t at = cur[b[r]];
            if (MIX) slot[r] = (at & 0xffffu) + ((at >> 16) < kMixed ? slot[r] : mixed_place(slot[r], at >> 16));
            else slot[r] += at;
            sk[slot[r]] = k[r];
            sb[slot[r]] = (uint16_t)b[r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int x = tid * per + j;
        if (j < per && x < B) cur[x] = g[j];
    }
    __syncthreads();
    uint32_t q[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int s = r * PT + tid;
        if (s < cnt) {
            q[r] = cur[sb[s]] + (uint32_t)s;
            kout[q[r]] = sk[s];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (r * PT + tid < cnt) sv[slot[r]] = v[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int s = r * PT + tid;
        if (s < cnt) vout[q[r]] = sv[s];
    }
}

template <typename K, typename P>
constexpr size_t stage_bytes(int tile) { return (size_t)tile * (sizeof(K) + 2 > sizeof(P) ? sizeof(K) + 2 : sizeof(P)); }

// First partition.  Loads are marked as read once, so that the L2 keeps the lines that are being written (101 -> 91 us for the move
// alone, 16.9 M entries in 512 buckets).
template <typename K, typename P, int PT, int R, int PER>
__global__ __launch_bounds__(PT) void partition_kernel(source s, const P *__restrict__ vin, int64_t n, level1 t, int cell_shift, uint32_t dump,
                                                        K *__restrict__ kout, P *__restrict__ vout, int *__restrict__ flags)
{
    constexpr int T = PT * R;
    extern __shared__ __align__(16) unsigned char lds[];
    uint32_t *cur = (uint32_t *)lds;                                 // [B], padded to 16 bytes
    __shared__ uint32_t wsum[PT / 64];
    void *stage = lds + (((size_t)t.B * 4 + 15) & ~(size_t)15);
    uint64_t *lo = (uint64_t *)stage;                                // the buckets' table lies where the tile is staged later
    uint16_t *lut = (uint16_t *)(lo + t.B);
    const uint32_t tile = tile_of_block();
    const int64_t e0 = (int64_t)tile * T;
    if (e0 >= n) return;
    const int cnt = n - e0 < T ? (int)(n - e0) : T, tid = threadIdx.x;
    uint64_t key[R];
    P v[R];
    uint32_t b[R];
    bool any_bad = false;
    uint32_t bad = 0;
    if (s.keys) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = r * PT + tid;
            key[r] = __builtin_nontemporal_load(s.keys + e0 + (i < cnt ? i : cnt - 1));
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) key[r] = 0;
        for (int l = 0; l < s.rank; ++l) {
            const int64_t *__restrict__ c = s.coord[l] + e0;
            int64_t x[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int i = r * PT + tid;
                x[r] = __builtin_nontemporal_load(c + (i < cnt ? i : cnt - 1));
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (x[r] < 0 || x[r] >= s.size[l]) bad |= 1u << r;
                key[r] = key[r] * (uint64_t)s.size[l] + (uint64_t)x[r];
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * PT + tid;
        v[r] = __builtin_nontemporal_load(vin + e0 + (i < cnt ? i : cnt - 1));
    }
    for (int i = tid; i < t.B; i += PT) { cur[i] = 0; lo[i] = t.lo[i]; }
    for (int i = tid; i <= kCells; i += PT) lut[i] = t.lut[i];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if ((bad >> r) & 1u) { key[r] = 0; any_bad = true; }
        const uint32_t c = (uint32_t)(key[r] >> cell_shift);
        uint32_t a = lut[c], z = lut[c + 1];
        while (a < z) {
            const uint32_t mid = (a + z + 1) / 2;
            if (lo[mid] <= key[r]) a = mid;
            else z = mid - 1;
        }
        b[r] = a;
    }
    if (any_bad) atomicOr(&flags[0], 1);
    __syncthreads();
    K k[R];
#pragma unroll
    for (int r = 0; r < R; ++r) k[r] = (K)key[r];
    move_tile<K, P, PT, R, PER, true>(k, b, v, cnt, t.B, cur, wsum, stage, t.cur, t.end, dump, kout, vout);
}

struct level2 {
    uint64_t *lo;             // [parts + 1]
    uint32_t *start, *end, *cur;
    uint16_t *tile_bucket;    // [tiles] bucket a tile of the second partition belongs to
};

__device__ __forceinline__ uint32_t sub_samples(uint32_t parts)
{
    uint32_t s = 64;
    while (s < parts * (uint32_t)kShare && s < (uint32_t)kSubSample) s *= 2;
    return s;
}

// One block, after the first partition: the sizes of the buckets are known.  Where each begins in the sorted order, and, for a second
// partition, its parts, tiles and their room.
__global__ __launch_bounds__(1024) void bucket_sizes_kernel(level1 t, int two, uint32_t tile, uint32_t room2_end, int *__restrict__ flags)
{
    __shared__ uint32_t wsum[16];
    uint32_t out = 0, sub = 0, tiles = 0, room = 0;
    for (int b0 = 0; b0 < t.B; b0 += 1024) {
        const int b = b0 + (int)threadIdx.x;
        uint32_t cnt = 0, parts = 0, nt = 0, need = 0;
        if (b < t.B) {
            cnt = t.cur[b] - t.start[b];
            const uint32_t cap = t.end[b] - t.start[b];
            if (cnt > cap) flags[2] = 1;
            if (two) {
                const uint32_t held = cnt < cap ? cnt : cap;
                parts = held > (uint32_t)kTarget ? (held + kTarget - 1) / kTarget : 1u;
                nt = (held + tile - 1) / tile;
                if (parts == 1) need = (held + 15u) & ~15u;
                else {
                    const uint32_t S = sub_samples(parts);
                    need = parts * (uint32_t)room_for((double)S / (double)parts, (double)S, (double)held);
                }
            }
        }
        uint32_t all;
        const uint32_t o = out + block_exclusive_scan(cnt, wsum, all);
        out += all;
        if (b < t.B) t.out[b] = o;
        if (!two) continue;                                          // uniform
        const uint32_t s = sub + block_exclusive_scan(parts, wsum, all);
        sub += all;
        const uint32_t ti = tiles + block_exclusive_scan(nt, wsum, all);
        tiles += all;
        uint32_t r = room + block_exclusive_scan(need, wsum, all);
        room += all;
        if (b < t.B) {
            if (r > room2_end || need > room2_end - r) { flags[2] = 1; r = 0; }
            t.sub0[b] = s; t.tile0[b] = ti; t.room2[b] = r;
        }
    }
    if (threadIdx.x == 0) {
        t.out[t.B] = out;
        if (two) { t.sub0[t.B] = sub; t.tile0[t.B] = tiles; }
    }
}

// Block = bucket: splitters of its parts.  Its keys are counted by kPartCells equal intervals of its range; parts end where the count
// passes their share.  Where an interval holds too much for that, a sorted sample of the bucket gives the splitters instead.
// 4 bytes read per entry: 44 us for 16.9 M (1.5 TB/s).  A block per bucket is few blocks, in which loads, vector instructions (half of the busy
// cycles) and LDS atomics take turns.
template <typename K>
__global__ __launch_bounds__(1024) void parts_kernel(level1 t, level2 u, const K *__restrict__ keys, uint64_t total, const int *__restrict__ flags)
{
    __shared__ uint32_t key[kSubSample];                             // counts, then what comes before; or the sample
    __shared__ uint32_t wsum[16];
    __shared__ uint32_t heavy;
    const int b = blockIdx.x, tid = threadIdx.x;
    if (flags[2]) return;
    const uint32_t s0 = t.sub0[b], room = t.sub0[b + 1] - s0, cnt = t.cur[b] - t.start[b];
    const uint64_t lo = t.lo[b], range = t.lo[b + 1] - lo;
    const K *__restrict__ kp = keys + t.start[b];
    for (uint32_t i = t.tile0[b] + tid; i < t.tile0[b + 1]; i += 1024) u.tile_bucket[i] = (uint16_t)b;
    if (b == t.B - 1 && tid == 0) u.lo[s0 + room] = total;
    const uint32_t base = t.room2[b], exact = (cnt + (uint32_t)kExact - 1) / (uint32_t)kExact;
    if (exact <= 1) {
        if (tid == 0) t.used[b] = 1;
        for (uint32_t j = tid; j < room; j += 1024) {
            const uint32_t at = base + (j ? cnt : 0u);
            u.lo[s0 + j] = j ? t.lo[b + 1] : lo;
            u.start[s0 + j] = u.cur[s0 + j] = at;
            u.end[s0 + j] = base + cnt;
        }
        return;
    }
    const int bits = range > 1 ? 64 - __clzll((long long)(range - 1)) : 0, cshift = bits > 14 ? bits - 14 : 0;
    static_assert(kPartCells == 1 << 14 && kPartCells == 2 * kSubSample, "intervals of a bucket, two to a word");
    if (tid == 0) heavy = 0;
#pragma unroll
    for (int i = 0; i < kSubSample / 1024; ++i) key[i * 1024 + tid] = 0;
    __syncthreads();
    for (uint32_t i = tid; i < cnt; i += 16 * 1024) {
        K x[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) x[e] = kp[i + e * 1024 < cnt ? i + e * 1024 : cnt - 1];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            // 16-bit counts; more than 65535 keys in one interval would spoil its neighbour's: the parts overflow then
            const uint32_t cell = (uint32_t)((uint64_t)(K)(x[e] - (K)lo) >> cshift);
            if (i + e * 1024 < cnt) atomicAdd(&key[cell >> 1], 1u << ((cell & 1u) * 16u));
        }
    }
    __syncthreads();
    // eight words per thread, from the LDS in an order without bank conflicts
    uint32_t tot = 0, most = 0, all;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const uint32_t word = tid * 8 + ((e + tid) & 7);
        const uint32_t x = key[word], a = x & 0xffffu, z = x >> 16;
        tot += a + z;
        most = a > most ? a : most;
        most = z > most ? z : most;
    }
    if (most > (uint32_t)kHeavy) heavy = 1;
    uint32_t before = block_exclusive_scan(tot, wsum, all);
    if (!heavy && all == cnt) {
        // part j begins with the first interval that at least j * cnt / exact entries lie before.  A thread whose sixteen intervals
        // hold no such place has nothing to look for.
        const float share = (float)cnt / (float)exact;
        uint32_t j = (uint32_t)((float)before / share);              // first j with j * cnt > before * exact, from one below it
        j = j > 1 ? j - 1 : 1;
        while (j < exact && (uint64_t)j * cnt <= (uint64_t)before * exact) ++j;
        if (j < exact && (uint64_t)j * cnt <= (uint64_t)(before + tot) * exact) {
            for (uint32_t e = 0; e < 16; ++e) {
                const uint32_t after = before + ((key[tid * 8 + (e >> 1)] >> ((e & 1u) * 16u)) & 0xffffu);
                for (; j < exact && (uint64_t)j * cnt <= (uint64_t)after * exact; ++j) {
                    u.lo[s0 + j] = lo + ((uint64_t)(tid * 16 + e + 1) << cshift);
                    u.start[s0 + j] = u.cur[s0 + j] = base + after;
                    u.end[s0 + j - 1] = base + after;
                }
                before = after;
            }
        }
        if (tid == 0) {
            t.used[b] = exact;
            u.lo[s0] = lo;
            u.start[s0] = u.cur[s0] = base;
            u.end[s0 + exact - 1] = base + cnt;
        }
        for (uint32_t j = exact + tid; j < room; j += 1024) {
            u.lo[s0 + j] = t.lo[b + 1];
            u.start[s0 + j] = u.cur[s0 + j] = u.end[s0 + j] = base + cnt;
        }
        return;
    }
    __syncthreads();
    if (tid == 0) t.used[b] = room;
    const uint32_t S = sub_samples(room);
    const int shift = bits > 32 ? bits - 32 : 0;
    auto sampled = [&](uint32_t i) { return (uint32_t)((uint64_t)(K)(kp[sampled_position(i, S, cnt)] - (K)lo) >> shift); };
    if (S <= 1024) {
        uint32_t x[1] = {tid < (int)S ? sampled(tid) : 0u};
        block_sort<1>(x, S, key);
    } else if (S <= 2048) {
        uint32_t x[2];
        for (int e = 0; e < 2; ++e) x[e] = sampled(tid + e * 1024);
        block_sort<2>(x, S, key);
    } else {
        uint32_t x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = (uint32_t)e * 1024u < S ? sampled(tid + e * 1024) : 0u;
        block_sort<8>(x, S, key);
    }
    const uint32_t cap = room > 1 ? (uint32_t)room_for((double)S / (double)room, (double)S, (double)cnt) : (cnt + 15u) & ~15u;
    for (uint32_t j = tid; j < room; j += 1024) {
        const uint32_t at = base + j * cap;
        u.lo[s0 + j] = j ? lo + ((uint64_t)key[(j * S) / room] << shift) : lo;
        u.start[s0 + j] = u.cur[s0 + j] = at;
        u.end[s0 + j] = at + cap;
    }
}

constexpr int kDump = kWideT * kPR;          // entries of the largest tile
constexpr int kMaxParts = 1024;
// Second partition: a tile lies inside one bucket.
template <typename K, typename P, int R>
__global__ __launch_bounds__(kPT) void partition_again_kernel(const K *__restrict__ kin, const P *__restrict__ vin, level1 t, level2 u, uint32_t dump,
                                                              K *__restrict__ kout, P *__restrict__ vout, const int *__restrict__ flags)
{
    constexpr int T = kPT * R;
    __shared__ uint32_t cur[kMaxParts];
    __shared__ uint32_t wsum[kPT / 64];
    __shared__ __align__(16) unsigned char stage[stage_bytes<K, P>(kPT * R)];
    const uint32_t tile = tile_of_block();
    if (tile >= t.tile0[t.B] || flags[2]) return;
    const int bkt = u.tile_bucket[tile], tid = threadIdx.x;
    const uint32_t s0 = t.sub0[bkt], i0 = (tile - t.tile0[bkt]) * (uint32_t)T, held = t.cur[bkt] - t.start[bkt];
    const int parts = (int)t.used[bkt], cnt = held - i0 < (uint32_t)T ? (int)(held - i0) : T;
    const uint32_t e0 = t.start[bkt] + i0;
    const K lo = (K)t.lo[bkt];
    K *split = (K *)stage;
    K k[R];
    P v[R];
    uint32_t b[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * kPT + tid;
        k[r] = __builtin_nontemporal_load(kin + e0 + (i < cnt ? i : cnt - 1));
        v[r] = __builtin_nontemporal_load(vin + e0 + (i < cnt ? i : cnt - 1));
    }
    for (int i = tid; i < parts; i += kPT) { cur[i] = 0; split[i] = (K)((K)u.lo[s0 + i] - lo); }
    __syncthreads();
    int step = 1;
    while (2 * step < parts) step *= 2;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const K d = (K)(k[r] - lo);
        int a = 0;
        for (int w = step; w > 0; w >>= 1)
            if (a + w < parts && split[a + w] <= d) a += w;
        b[r] = (uint32_t)a;
    }
    __syncthreads();
    move_tile<K, P, kPT, R, (kMaxParts + kPT - 1) / kPT, false>(k, b, v, cnt, parts, cur, wsum, stage, u.cur + s0, u.end + s0, dump, kout, vout);
}

// ---- finish ---------------------------------------------------------------------------------
// A final bucket, as the finishing kernels take it.
struct final_bucket {
    uint64_t lo, next;        // its smallest key, the next bucket's
    uint32_t start, cnt;      // where its entries are, how many; kOverflow: more than fit
    uint32_t out;             // where they end up in the sorted order
    uint32_t scale;           // (distance from lo, shifted) * scale >> 32: its place in the bucket's range in 31 bits
    int shift;                // > 0: distances to the left, < 0: to the right, so that the range has 32 bits
};
constexpr uint32_t kOverflow = 0x80000000u;
// left: a bucket with a crowded interval, whose keys crowd inside it as well; the rows of one that has many
constexpr uint32_t kCrowded = 1u, kUneven = 2u, kUncounted = 4u;

struct final_args {
    const final_bucket *bucket;
    const uint32_t *count;               // DEVICE: number of final buckets (null: `most`)
    uint32_t most;
    int64_t n;
    uint32_t *left;                      // [most] what the finishing kernel left to finish_crowded_kernel
    int *flags;
    // what leaves: the keys (uint64), or what bucket_levels_kernel takes (dist), or crd / pos of an innermost compressed level under dense ones
    uint64_t *keys;
    uint32_t *dist;                      // every entry's distance from its bucket's lo
    uint32_t *heads;                     // [slot * most + bucket]: entries that begin a new prefix
    uint32_t *ends;                      // [2 * most]: first and last distance of a bucket
    const uint32_t *off;                 // [SP_MAX_RANK * most] levels: lo's coordinate at each compressed level, from the innermost on
    spmi_levels levels;
    void *crd, *pos;
    int32_t *rowblk;                     // row of every kSpmiStreamT-th entry (may be null)
    int64_t nblocks;
    spmi_divisor inner;
    int64_t rows;
    int pw, cw;
};

// Thread = final bucket: its description, from the partitions' tables.  One partition: start .. out by final bucket; two: out by
// bucket of the first one, whose parts [sub0[b], sub0[b + 1]) are block b's.
__global__ __launch_bounds__(256) void final_buckets_kernel(const uint64_t *__restrict__ lo, const uint32_t *__restrict__ start, const uint32_t *__restrict__ end,
                                                            const uint32_t *__restrict__ cur, const uint32_t *__restrict__ out,
                                                            const uint32_t *__restrict__ sub0, uint32_t count, final_bucket *__restrict__ bucket, uint32_t *__restrict__ off,
                                                            final_args f)
{
    __shared__ uint32_t wsum[4];
    if (blockIdx.x == 0 && threadIdx.x == 0 && f.pos) {              // the ends of the arrays
        if (f.pw == 32) ((int32_t *)f.pos)[f.rows] = (int32_t)f.n;
        else ((int64_t *)f.pos)[f.rows] = f.n;
        if (f.rowblk) { f.rowblk[0] = 0; f.rowblk[f.nblocks] = (int32_t)f.rows; }
    }
    if (f.flags[2]) return;
    const uint32_t first = sub0 ? sub0[blockIdx.x] : blockIdx.x * 256u;
    const uint32_t last = sub0 ? sub0[blockIdx.x + 1] : (first + 256u < count ? first + 256u : count);
    uint32_t at = sub0 ? out[blockIdx.x] : 0u;
    for (uint32_t b0 = first; b0 < last; b0 += 256) {
        const uint32_t b = b0 + threadIdx.x;
        final_bucket w;
        w.cnt = 0;
        if (b < last) {
            w.start = start[b];
            w.cnt = cur[b] - w.start;
        }
        uint32_t all, before = block_exclusive_scan(w.cnt, wsum, all);
        if (b < last) {
            w.out = sub0 ? at + before : out[b];
            w.lo = lo[b];
            w.next = lo[b + 1];
            const uint64_t range = w.next - w.lo;
            const int bits = range > 1 ? 64 - __clzll((long long)(range - 1)) : 0;
            w.shift = bits ? 32 - bits : 0;
            const uint64_t steps = bits ? (w.shift >= 0 ? range << w.shift : ((range - 1) >> -w.shift) + 1) : 1;   // in (2^31, 2^32]
            w.scale = bits ? (uint32_t)((1ull << 63) / steps) : 0u;
            if (w.cnt > end[b] - w.start || w.cnt > (uint32_t)kCap) { f.flags[3] = 1; w.cnt |= kOverflow; }
            uint64_t prefix = w.lo;
            for (int j = 0; j < f.levels.count; ++j) {
                const uint64_t up = spmi_div_by(prefix, f.levels.size[j]);
                off[(size_t)b * SP_MAX_RANK + j] = (uint32_t)(prefix - up * f.levels.size[j].d);
                prefix = up;
            }
            bucket[b] = w;
        }
        at += all;
    }
}

// (off + q) / size for 32-bit numbers: the half keeps every quotient further from a whole number than the arithmetic is off
__device__ __forceinline__ uint32_t quotient(uint32_t q, double off_and_half, double inv) { return (uint32_t)(((double)q + off_and_half) * inv); }

// The bucket's keys lie sorted in the LDS as distances from lo: what the format wants of them.
template <typename K, int T>
__device__ __forceinline__ void emit_sorted(const final_args &f, const final_bucket &w, const K *dist, uint32_t cnt)
{
    if (f.keys) {
        uint64_t *__restrict__ q = f.keys + w.out;
        for (uint32_t i = threadIdx.x; i < cnt; i += T) q[i] = w.lo + dist[i];
        return;
    }
    if (f.dist) {
        uint32_t *__restrict__ q = f.dist + w.out;
        for (uint32_t i = threadIdx.x; i < cnt; i += T) q[i] = (uint32_t)dist[i];
        return;
    }
    const uint64_t row0 = spmi_div_by(w.lo, f.inner), off = w.lo - row0 * f.inner.d;
    const double half = (double)off + 0.5;
    const bool narrow = sizeof(K) == 4 && f.inner.d <= 0xffffffffull;      // block-uniform: quotients and coordinates in 32 bits
    for (uint32_t i = threadIdx.x; i < cnt; i += T) {
        uint64_t row, col;
        if (narrow) {
            const uint32_t q = f.inner.shift >= 0 ? (uint32_t)((off + dist[i]) >> f.inner.shift) : quotient((uint32_t)dist[i], half, f.inner.inv);
            row = q;
            col = (uint32_t)((uint32_t)off + (uint32_t)dist[i] - q * (uint32_t)f.inner.d);
        } else {
            const uint64_t x = off + dist[i];
            row = spmi_div_by(x, f.inner);
            col = x - row * f.inner.d;
        }
        const uint32_t at = w.out + i;
        if (f.cw == 32) ((int32_t *)f.crd)[at] = (int32_t)col;
        else ((int64_t *)f.crd)[at] = (int64_t)col;
        if (f.rowblk && (at % (uint32_t)kSpmiStreamT) == 0 && at > 0) f.rowblk[at / (uint32_t)kSpmiStreamT] = (int32_t)(row0 + row);
    }
}

// Levels: how many entries of the bucket begin a new prefix at each compressed level above the innermost, but for its first entry
// (whose predecessor lies in another bucket: bucket_heads_kernel).  Block-wide, with barriers; cnt may be 0.  A wave takes entries
// that lie side by side, so that the predecessor's quotient is the neighbouring lane's.
constexpr int kSlots = SP_MAX_RANK - 1;
struct head_counts { uint32_t n[kSlots]; };

__device__ __forceinline__ uint32_t lane_before(uint32_t v, uint32_t first)
{
    // v of the lane below; lane 0 takes `first` (wave shift right by one lane)
    return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)v, 0x138, 0xf, 0xf, false);
}

template <typename K, int T>
__device__ __forceinline__ void emit_heads(const final_args &f, const K *dist, uint32_t cnt, uint32_t b, head_counts &h)
{
    if (!f.dist) return;
    const int slots = f.levels.count - 1, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < kSlots) h.n[tid] = 0;
    __syncthreads();
    const int rounds = (int)((cnt + T - 1) / T);
    const uint32_t i0 = (uint32_t)(wave * rounds) * 64u;
    if (i0 < cnt) {
        double half[kSlots];
        uint32_t edge[kSlots], heads[kSlots], e = i0 ? (uint32_t)dist[i0 - 1] : 0u;
#pragma unroll
        for (int j = 0; j < kSlots; ++j) {
            half[j] = 0;
            edge[j] = heads[j] = 0;
            if (j < slots) {
                half[j] = (double)(uint32_t)__builtin_amdgcn_readfirstlane((int)f.off[(size_t)b * SP_MAX_RANK + j]) + 0.5;
                e = edge[j] = quotient(e, half[j], f.levels.size[j].inv);
            }
        }
        for (int r = 0; r < rounds; ++r) {
            const uint32_t i = i0 + (uint32_t)(r * 64 + lane);
            uint32_t q = (uint32_t)dist[i < cnt ? i : cnt - 1];      // behind the last entry: the same again, no head
#pragma unroll
            for (int j = 0; j < kSlots; ++j) {
                if (j < slots) {
                    q = quotient(q, half[j], f.levels.size[j].inv);
                    heads[j] += (uint32_t)__popcll(__ballot(q != lane_before(q, edge[j]) && i > 0));
                    edge[j] = (uint32_t)__builtin_amdgcn_readlane((int)q, 63);
                }
            }
        }
#pragma unroll
        for (int j = 0; j < kSlots; ++j)
            if (j < slots && lane == 0) atomicAdd(&h.n[j], heads[j]);
    }
    __syncthreads();
    if (tid < slots) f.heads[(size_t)tid * f.most + b] = h.n[tid];
    if (tid == 0 && cnt) { f.ends[2 * b] = (uint32_t)dist[0]; f.ends[2 * b + 1] = (uint32_t)dist[cnt - 1]; }
}

// The rows (positions of the level above) that begin in [lo, next) are this bucket's: each looks up its first entry.  Those of a bucket
// with more than kManyRows are left to finish_crowded_kernel.
constexpr int kManyRows = 2048;
struct row_range { uint64_t first, end; };
__device__ __forceinline__ row_range rows_of(const final_args &f, const final_bucket &w)
{
    return {w.lo == 0 ? 0 : spmi_div_by(w.lo - 1, f.inner) + 1, w.next == 0 ? 0 : spmi_div_by(w.next - 1, f.inner) + 1};
}
__device__ __forceinline__ bool many_rows(const final_args &f, const final_bucket &w)
{
    const row_range rows = rows_of(f, w);
    return f.pos && rows.end - rows.first > (uint64_t)kManyRows;
}
__device__ __forceinline__ void put_pos(const final_args &f, uint64_t r, uint32_t at)
{
    if (f.pw == 32) ((int32_t *)f.pos)[r] = (int32_t)at;
    else ((int64_t *)f.pos)[r] = (int64_t)at;
}

template <typename K, int T>
__device__ __forceinline__ void emit_rows(const final_args &f, const final_bucket &w, const K *dist, uint32_t cnt)
{
    if (!f.pos) return;
    const row_range rows = rows_of(f, w);
    if (cnt && rows.end - rows.first > (uint64_t)kManyRows) return;  // block-uniform
    uint32_t top = 1;
    while (top <= cnt) top *= 2;
    const uint64_t last = cnt ? (uint64_t)dist[cnt - 1] : 0;
    for (uint64_t r = rows.first + threadIdx.x; r < rows.end; r += T) {
        const uint64_t first = r * f.inner.d - w.lo;                 // below next - lo: fits K
        uint32_t a = 0;
        if (cnt && first > last) a = cnt;                            // rows after the last entry
        else for (uint32_t s = top / 2; s > 0; s >>= 1)
            if (a + s <= cnt && (uint64_t)dist[a + s - 1] < first) a += s;
        put_pos(f, r, w.out + a);
    }
}

// Many rows (the last ones of an R-MAT graph, mostly empty: 65536 of them in a bucket) take too many reads of the LDS to be looked up:
// their entries are counted, from the keys as they came, kRowChunk rows at a time, and the counts summed.  R-MAT graph of 2^23
// vertices, 4 M f32 entries, CSR: finishing 362 + 330 us by looking up, 117 + 144 so; the same from 512 rows on, 3 % of the call
// longer from 8192.  (In the finishing kernel itself it costs registers: 4 % of that kernel where no bucket has many rows.)
// lds: kCap + kRowWords words.
constexpr int kRowChunk = 16 * kFT, kRowWords = 17 * kFT;            // one word more for every 16: no bank conflicts when a thread sums its 16
template <typename K>
__device__ __forceinline__ void count_rows(const final_args &f, const final_bucket &w, const K *__restrict__ kin, uint32_t *lds, uint32_t *wsum)
{
    const K *__restrict__ keys = kin + w.start;
    const uint32_t cnt = w.cnt;
    const row_range rows = rows_of(f, w);
    const uint32_t n = (uint32_t)(rows.end - rows.first);            // below 4 * entries (or this format is not written here)
    const int tid = threadIdx.x;
    uint32_t *rel = lds, *counts = lds + kCap;                       // an entry's row, counted from the one before the first
    __syncthreads();
    for (uint32_t i = tid; i < cnt; i += kFT) rel[i] = (uint32_t)(spmi_div_by(w.lo + (uint64_t)(K)(keys[i] - (K)w.lo), f.inner) + 1 - rows.first);
    uint32_t before = 0;
    for (uint32_t c = 0; c < n; c += kRowChunk) {
        for (int j = tid; j < kRowWords; j += kFT) counts[j] = 0;
        __syncthreads();
        for (uint32_t i = tid; i < cnt; i += kFT) {
            const uint32_t j = rel[i] - c;                           // below c: beyond the chunk as an unsigned number
            if (j < (uint32_t)kRowChunk) atomicAdd(&counts[j + (j >> 4)], 1u);
        }
        __syncthreads();
        uint32_t *mine = counts + tid * 17, sum = 0, all;
#pragma unroll
        for (int j = 0; j < 16; ++j) sum += mine[j];
        uint32_t up = before + block_exclusive_scan(sum, wsum, all);
#pragma unroll
        for (int j = 0; j < 16; ++j) mine[j] = up += mine[j];
        __syncthreads();
        for (int j = tid; j < kRowChunk && c + (uint32_t)j < n; j += kFT) put_pos(f, rows.first + c + (uint32_t)j, w.out + counts[j + (j >> 4)]);
        before += all;
        __syncthreads();
    }
}

// Distance from a bucket's smallest key -> place in its range, in 31 bits; never decreases with the distance.
template <typename K>
__device__ __forceinline__ uint32_t place_in_range(K d, const final_bucket &w)
{
    const uint32_t x = sizeof(K) == 4 ? (uint32_t)d << (w.shift & 31) : w.shift >= 0 ? (uint32_t)(d << w.shift) : (uint32_t)(d >> -w.shift);
    return __umulhi(x, w.scale);
}

template <typename K>
using lds_key = typename std::conditional<sizeof(K) == 8, unsigned long long, unsigned int>::type;

template <typename K, typename P, int ATTEMPT>
struct finish_lds {
    static constexpr int kWords = (kFE | 1) * kFT;
    static constexpr size_t kKeys = kCap * sizeof(K) + (kWords + 1) * 4 + kCells1 * 4, kValues = kCap * sizeof(P);
    __align__(16) unsigned char stage[kKeys > kValues ? kKeys : kValues];
    static_assert(sizeof(stage) >= (kCap + kRowWords) * 4, "count_rows");
    lds_key<K> least[ATTEMPT ? kCells1 : 1], most[ATTEMPT ? kCells1 : 1];     // second attempt: of a cell's keys
    uint32_t wsum[kFT / 64];
    uint32_t crowded;
    head_counts heads;
};

// Do the keys of an interval that holds len of them crowd inside it as well?  64 are counted by eighths from the least to the
// greatest: if one eighth has more than a third, cutting the interval again would leave a part with most of its keys.  The same answer in
// every wave.  (Not asked below kAsked keys, where the second attempt costs least.)
constexpr uint32_t kAsked = 64;
template <typename K>
__device__ __forceinline__ bool crowds_inside(const K *keys, uint32_t len)
{
    typedef lds_key<K> key;
    const key k = (key)keys[(threadIdx.x & 63u) * len >> 6];         // len <= kCap
    key least = k, most = k;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const key a = __shfl_xor(least, d, 64), c = __shfl_xor(most, d, 64);
        least = a < least ? a : least;
        most = c > most ? c : most;
    }
    const uint32_t p = (uint32_t)((float)(k - least) * (8.0f / ((float)(most - least) + 1.0f)));
    int largest = 0;
#pragma unroll
    for (uint32_t e = 0; e < 8; ++e) {
        const int c = __popcll(__ballot((p < 7 ? p : 7) == e));
        largest = c > largest ? c : largest;
    }
    return largest > 64 / 3 + 2;
}

// A bucket sorted by value.  Its range is cut into kCells1 equal intervals, each of those into twice as many as it holds
// entries (rows differ in length, so keys are not spread evenly over a bucket), in the second attempt, for bands and blocks, only from
// its smallest key to its largest; an entry takes a number in its interval with one returning LDS add, the counts are scanned,
// the keys are dropped into their intervals, and an entry's place is the interval's start plus the number of smaller keys
// there.  Counts are 16 bits, two to a word: intervals x and x + words share one, so that one addition per word scans both
// halves.  (Keys that occur twice may take one place and leave a place as it was: the build ends with an error then.)
// 0: done.  kCrowded, for the whole block and with nothing written: an interval is too crowded; with kUneven where the second attempt is
// not going to help.
// What bounds it: vector instructions, so a thread has up to sixteen entries and what all entries of a bucket share is worked out
// before (final_buckets_kernel).
template <typename K, typename P, int ATTEMPT>
__device__ __forceinline__ uint32_t finish_bucket(const K *__restrict__ kin, const P *__restrict__ vin, P *__restrict__ vout, const final_args &f, const final_bucket &w,
                                              finish_lds<K, P, ATTEMPT> &s, uint32_t b)
{
    constexpr int W = kFT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t cnt = w.cnt;
    K *dist = (K *)s.stage;
    uint32_t *cells = (uint32_t *)(dist + kCap), *bins = cells + kCells1;
    P *sval = (P *)s.stage;
    const int rounds = (int)((cnt + kFT - 1) / kFT);                 // <= kFE
    const int per = rounds | 1;                                      // words per thread when they are scanned: odd, no bank conflicts
    const uint32_t words = (uint32_t)per * kFT;                      // two intervals each
    K k[kFE];
    P v[kFE];
    uint32_t at[kFE], slot[kFE];
    const K *__restrict__ kp = kin + w.start;
    const P *__restrict__ vp = vin + w.start;
#pragma unroll
    for (int r = 0; r < kFE; ++r) {
        if (r < rounds) {
            const uint32_t i = (uint32_t)(r * kFT + tid) < cnt ? (uint32_t)(r * kFT + tid) : cnt - 1;
            k[r] = __builtin_nontemporal_load(kp + i);
        }
    }
#pragma unroll
    for (int r = 0; r < kFE; ++r) {
        if (r < rounds) {
            const uint32_t i = (uint32_t)(r * kFT + tid) < cnt ? (uint32_t)(r * kFT + tid) : cnt - 1;
            v[r] = __builtin_nontemporal_load(vp + i);
        }
    }
    if (tid == 0) s.crowded = 0;
    for (int j = 0; j < per; ++j) bins[j * kFT + tid] = 0;
#pragma unroll
    for (int j = 0; j < kCells1 / kFT; ++j) {
        cells[j * kFT + tid] = 0;
        if (ATTEMPT) { s.least[j * kFT + tid] = ~(lds_key<K>)0; s.most[j * kFT + tid] = 0; }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kFE; ++r) {
        if (r < rounds && (uint32_t)(r * kFT + tid) < cnt) {
            k[r] -= (K)w.lo;
            at[r] = place_in_range<K>(k[r], w);
            atomicAdd(&cells[at[r] >> 21], 1u);
            if (ATTEMPT) {
                atomicMin(&s.least[at[r] >> 21], (lds_key<K>)k[r]);
                atomicMax(&s.most[at[r] >> 21], (lds_key<K>)k[r]);
            }
        }
    }
    __syncthreads();
    static_assert(kCells1 == 1024 && kFT == 256, "four cells per thread, ten bits of the place");
    {
        const uint4 c = ((const uint4 *)cells)[tid];
        const uint32_t incl = wave_inclusive_scan(c.x + c.y + c.z + c.w, lane);
        if (lane == 63) s.wsum[wave] = incl;
        __syncthreads();
        uint32_t before = incl - c.x - c.y - c.z - c.w;
#pragma unroll
        for (int x = 0; x < W; ++x) before += x < wave ? s.wsum[x] : 0u;
        ((uint4 *)cells)[tid] = make_uint4(before | (c.x << 16), (before + c.x) | (c.y << 16), (before + c.x + c.y) | (c.z << 16),
                                           (before + c.x + c.y + c.z) | (c.w << 16));
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kFE; ++r) {
        if (r < rounds && (uint32_t)(r * kFT + tid) < cnt) {
            const uint32_t c = cells[at[r] >> 21];
            uint32_t x;                                              // interval: twice what comes before its cell, and where in the cell
            if (ATTEMPT == 0) x = ((at[r] >> 4) & 0x1ffffu) * (c >> 16) >> 16;
            else {
                const uint32_t twice = 2u * (c >> 16);
                const K least = (K)s.least[at[r] >> 21];
                const float span = (float)(K)((K)s.most[at[r] >> 21] - least);
                x = (uint32_t)((float)(K)(k[r] - least) * ((float)twice / (span + 1.0f)));
                x = x < twice ? x : twice - 1;
            }
            x += 2u * (c & 0xffffu);
            const bool upper = x >= words;
            const uint32_t word = upper ? x - words : x, half = upper ? 16u : 0u;
            at[r] = word | (half << 16);
            slot[r] = (atomicAdd(&bins[word], 1u << half) >> half) & 0xffffu;
        }
    }
    __syncthreads();
    // exclusive scan of the words, `per` consecutive ones per thread; the upper halves continue after the lower ones' total
    uint32_t tot = 0;
    for (int j = 0; j < per; ++j) tot += bins[tid * per + j];
    const uint32_t incl = wave_inclusive_scan(tot, lane);
    if (lane == 63) s.wsum[wave] = incl;
    __syncthreads();
    uint32_t start = incl - tot, all = 0;
#pragma unroll
    for (int x = 0; x < W; ++x) { start += x < wave ? s.wsum[x] : 0u; all += s.wsum[x]; }
    start += all << 16;
    for (int j = 0; j < per; ++j) {
        const uint32_t c = bins[tid * per + j];
        bins[tid * per + j] = start;
        start += c;
    }
    if (tid == kFT - 1) bins[words] = (all & 0xffffu) | (cnt << 16);
    __syncthreads();
    uint32_t longest = 0;
#pragma unroll
    for (int r = 0; r < kFE; ++r) {
        if (r < rounds && (uint32_t)(r * kFT + tid) < cnt) {
            const uint32_t word = at[r] & 0xffffu, half = at[r] >> 16;
            const uint32_t s0 = (bins[word] >> half) & 0xffffu, len = ((bins[word + 1] >> half) & 0xffffu) - s0;
            slot[r] += s0;
            dist[slot[r]] = k[r];
            at[r] = s0 | (len << 16);
            longest = at[r] > longest ? at[r] : longest;
        } else at[r] = 0;
    }
    if ((longest >> 16) > (uint32_t)(ATTEMPT ? kCrowd : kSpread)) s.crowded = longest;      // one of them
    __syncthreads();
    if (s.crowded) {
        const uint32_t len = s.crowded >> 16;
        return kCrowded | (ATTEMPT == 0 && len >= kAsked && crowds_inside<K>(dist + (s.crowded & 0xffffu), len) ? kUneven : 0u);
    }
    longest >>= 16;
    // all rounds side by side, one other key of every interval per step; smaller ones are counted in the upper half of slot
    bool dup = false;
    for (uint32_t j = 1; j < longest; ++j) {
#pragma unroll
        for (int r = 0; r < kFE; ++r) {
            if (r < rounds && j < (at[r] >> 16)) {
                const uint32_t x = (slot[r] & 0xffffu) + j, end = (at[r] & 0xffffu) + (at[r] >> 16);
                const K o = dist[x < end ? x : x - (at[r] >> 16)];
                slot[r] += o < k[r] ? 0x10000u : 0u;
                dup |= o == k[r];
            }
        }
    }
    if (dup) atomicOr(&f.flags[1], 1);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kFE; ++r) {
        if (r < rounds && (uint32_t)(r * kFT + tid) < cnt) {
            at[r] = (at[r] & 0xffffu) + (slot[r] >> 16);             // the entry's place
            dist[at[r]] = k[r];
        }
    }
    __syncthreads();
    emit_sorted<K, kFT>(f, w, dist, cnt);
    emit_rows<K, kFT>(f, w, dist, cnt);
    emit_heads<K, kFT>(f, dist, cnt, b, s.heads);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kFE; ++r)
        if (r < rounds && (uint32_t)(r * kFT + tid) < cnt) sval[at[r]] = v[r];
    __syncthreads();
    for (uint32_t i = tid; i < cnt; i += kFT) vout[w.out + i] = sval[i];
    return 0;
}

template <typename K, typename P>
__global__ __launch_bounds__(kFT, 4) void finish_kernel(const K *__restrict__ kin, const P *__restrict__ vin, P *__restrict__ vout, final_args f)
{
    __shared__ finish_lds<K, P, 0> s;
    const uint32_t b = blockIdx.x;
    if (f.flags[2]) {                                                // a bucket overflowed in the first partition: harmless output, the build will be done again
        for (int64_t i = (int64_t)b * kFT + threadIdx.x; i < f.n; i += (int64_t)f.most * kFT) {
            if (f.keys) f.keys[i] = 0;
        }
        return;
    }
    const bool any = b < (f.count ? *f.count : f.most);
    final_bucket w;
    w.cnt = 0;
    if (any) w = f.bucket[b];
    uint32_t left = 0;
    if ((w.cnt & kOverflow) || w.cnt == 0) {
        if ((w.cnt & kOverflow) && f.keys) for (uint32_t i = threadIdx.x; i < (w.cnt & ~kOverflow); i += kFT) f.keys[w.out + i] = 0;
        if (any) emit_rows<K, kFT>(f, w, (const K *)s.stage, 0);
        emit_heads<K, kFT>(f, (const K *)s.stage, 0, b, s.heads);
    } else left = finish_bucket<K, P, 0>(kin, vin, vout, f, w, s, b);
    if (any && threadIdx.x == 0) f.left[b] = left | ((int32_t)w.cnt > 0 && many_rows(f, w) ? kUncounted : 0u);
}

// The distances of up to kCap keys from lo, sorted in the LDS, and every one's number among them: a thread sorts up to 17 of them in
// registers (an odd number of them side by side, so that threads meet different banks), then runs are merged two by two, each thread
// finding by bisection where its part of the merged run begins.  In place of a bitonic sort through the LDS, whose 78 steps for 4096
// keys move every key each time.  Block-wide, with barriers.
template <typename K>
__device__ __forceinline__ void merge_sort(const K *__restrict__ keys, K lo, uint32_t cnt, K *dist, uint16_t *idx)
{
    constexpr int E = kFE | 1;
    const uint32_t tid = threadIdx.x;
    const uint32_t per = ((cnt + kFT - 1) / kFT) | 1u, x0 = tid * per;        // per <= E
    for (uint32_t i = tid; i < cnt; i += kFT) dist[i] = (K)(keys[i] - lo);
    __syncthreads();
    K k[E];
    uint32_t id[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const bool any = (uint32_t)e < per && x0 + e < cnt;
        k[e] = any ? dist[x0 + e] : (K)~(K)0;
        id[e] = any ? x0 + e : 0xffffu;                      // what fills up stays behind a largest key
    }
#pragma unroll
    for (int step = 0; step < E; ++step) {
#pragma unroll
        for (int e = step & 1; e + 1 < E; e += 2) {
            const K a = k[e], c = k[e + 1];
            const uint32_t ia = id[e], ic = id[e + 1];
            const bool swap = c < a || (c == a && ic < ia);
            k[e] = swap ? c : a; k[e + 1] = swap ? a : c;
            id[e] = swap ? ic : ia; id[e + 1] = swap ? ia : ic;
        }
    }
    for (uint32_t r = 0;; ++r) {
        const uint32_t w = per << r;                         // sorted runs of w
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e)
            if ((uint32_t)e < per && x0 + e < cnt) { dist[x0 + e] = k[e]; idx[x0 + e] = (uint16_t)id[e]; }
        __syncthreads();
        if (w >= cnt) return;
        if (x0 < cnt) {
            const uint32_t base = ((tid >> (r + 1)) << (r + 1)) * per, left = cnt - base;
            const uint32_t na = left < w ? left : w, nb = left - na < w ? left - na : w, at = x0 - base;     // at < na + nb
            const K *A = dist + base, *B = nb ? A + na : A;
            uint32_t a = at > nb ? at - nb : 0u, end = at < na ? at : na;
            while (a < end) {
                const uint32_t mid = (a + end) / 2;
                if (A[mid] <= B[at - 1 - mid]) a = mid + 1;
                else end = mid;
            }
            uint32_t b = at - a;
            K ka = A[a < na ? a : 0], kb = B[b < nb ? b : 0];
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if ((uint32_t)e < per && x0 + e < cnt) {
                    const bool first = a < na && (b >= nb || ka <= kb);
                    k[e] = first ? ka : kb;
                    id[e] = idx[base + (first ? a : na + b)];
                    if (first) { ++a; ka = A[a < na ? a : 0]; }
                    else { ++b; kb = B[b < nb ? b : 0]; }
                }
            }
        }
    }
}

// What the finishing kernel left.  Rows of buckets that have many are counted.  Entries that crowd in a few intervals: the second attempt,
// or, where that fails too or is not going to help, a merge sort in the LDS, the entry's number travelling with the key.  As many
// blocks as the chip holds: the registers are bounded so that the LDS decides how many (one block per CU without: bands of 64, 8 M f32
// entries, 123 us instead of 110).  7.0 M f32 entries in rows of 350 whose columns are spread evenly over their logarithm, DCSR: this
// kernel 278 us, 811 with bitonic sorts of what the second attempt leaves, 2331 with a second attempt that stands for 192 keys in an interval.
template <typename K, typename P>
__global__ __launch_bounds__(kFT, sizeof(K) + sizeof(P) == 8 ? 3 : 2) void finish_crowded_kernel(const K *__restrict__ kin, const P *__restrict__ vin, P *__restrict__ vout, final_args f)
{
    __shared__ union { finish_lds<K, P, 1> s; struct { K dist[kCap]; uint16_t idx[kCap]; head_counts heads; } sort; } lds;
    const int tid = threadIdx.x, lane = tid & 63;
    if (f.flags[2]) return;
    const uint32_t total = f.count ? *f.count : f.most;
    for (uint32_t first = blockIdx.x; first < total; first += 64u * gridDim.x) {       // 64 of the block's buckets looked at together
        const uint64_t mine = (uint64_t)first + (uint64_t)lane * gridDim.x;
        for (uint64_t todo = __ballot(mine < total && f.left[mine < total ? mine : 0] != 0); todo; todo &= todo - 1) {
            const uint32_t b = first + (uint32_t)__builtin_ctzll(todo) * gridDim.x;
            const final_bucket w = f.bucket[b];
            const uint32_t left = f.left[b];
            __syncthreads();
            if (left & kUncounted) count_rows<K>(f, w, kin, (uint32_t *)lds.s.stage, lds.s.wsum);
            if (!(left & kCrowded)) continue;
            if (!(left & kUneven) && !finish_bucket<K, P, 1>(kin, vin, vout, f, w, lds.s, b)) continue;
            __syncthreads();
            K *dist = lds.sort.dist;
            uint16_t *idx = lds.sort.idx;
            const uint32_t cnt = w.cnt;
            merge_sort<K>(kin + w.start, (K)w.lo, cnt, dist, idx);
            bool dup = false;
            for (uint32_t i = tid; i + 1 < cnt; i += kFT) dup |= dist[i] == dist[i + 1];
            if (dup) atomicOr(&f.flags[1], 1);
            emit_sorted<K, kFT>(f, w, dist, cnt);
            emit_rows<K, kFT>(f, w, dist, cnt);
            emit_heads<K, kFT>(f, dist, cnt, b, lds.sort.heads);
            for (uint32_t i = tid; i < cnt; i += kFT) vout[w.out + i] = vin[w.start + idx[i]];
        }
    }
}

// ---- levels ---------------------------------------------------------------------------------
// A bucket's first entry begins a new prefix at a level where it differs from the last entry of the bucket before it (empty ones
// skipped): counted, and kept as a bit per level.  Thread = bucket.
__global__ __launch_bounds__(256) void bucket_heads_kernel(final_args f, uint32_t *__restrict__ first_mask, uint64_t *__restrict__ before_key)
{
    const uint32_t b = blockIdx.x * 256u + threadIdx.x;
    if (f.flags[2] || f.flags[3] || b >= (f.count ? *f.count : f.most)) return;
    if (f.bucket[b].cnt == 0) return;
    int64_t p = (int64_t)b - 1;
    while (p >= 0 && f.bucket[p].cnt == 0) --p;
    uint64_t mine = f.bucket[b].lo + f.ends[2 * b], other = p < 0 ? 0 : f.bucket[p].lo + f.ends[2 * p + 1];
    before_key[b] = other;
    uint32_t mask = 0;
    for (int j = 0; j < f.levels.count; ++j) {
        mine = spmi_div_by(mine, f.levels.size[j]);
        other = spmi_div_by(other, f.levels.size[j]);
        if (p < 0 || mine != other) {
            mask |= 2u << j;                                         // bit j + 1: the level above the j-th
            if (j + 1 < f.levels.count) f.heads[(size_t)j * f.most + b] += 1u;
        }
    }
    first_mask[b] = mask;
}

__global__ void head_totals_kernel(const uint32_t *__restrict__ scanned, int64_t buckets, int slots, unsigned long long *__restrict__ totals)
{
    const int s = threadIdx.x;                                       // slot s: the (s + 1)-th level from the inside
    if (s < slots) totals[s] = (unsigned long long)(scanned[(int64_t)(s + 1) * buckets] - scanned[(int64_t)s * buckets]);
}

struct level_arrays {
    void *crd[SP_MAX_RANK], *pos[SP_MAX_RANK];                       // from the innermost level on
    const uint32_t *heads;                                           // scanned, slot after slot
    const uint32_t *first_mask;
    const uint64_t *before_key;
    int dense_above;                                                 // the outermost compressed level lies under dense ones
};

// Sorted entries -> crd and pos of all levels, for compressed levels that lie inside dense ones (or make up the format).  Block = a
// bucket; 32-bit distances and quotients relative to the bucket's smallest key, one multiplication per level.  From the
// innermost level outwards: the entry that begins a new prefix of the level above writes that position's pos entry.  pos
// under a dense level is left as counts (one integer add where a parent begins and one where the next does), to be scanned.
constexpr int kLT = 512;
template <typename PT, typename CT>
__global__ __launch_bounds__(kLT) void bucket_levels_kernel(final_args f, level_arrays a)
{
    constexpr int R = kCap / kLT, W = kLT / 64;
    static_assert(R * W <= 64, "one lane per wave and round");
    __shared__ uint32_t wcnt[2][R * W];
    typedef typename std::conditional<sizeof(PT) == 8, unsigned long long, unsigned int>::type UT;
    const uint32_t b = blockIdx.x;
    if (b >= (f.count ? *f.count : f.most)) return;
    const uint32_t cnt = f.bucket[b].cnt, out = f.bucket[b].out;
    if (cnt == 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, L = f.levels.count;
    const unsigned long long below = (1ull << lane) - 1ull;
    const uint32_t *__restrict__ dist = f.dist + out;
    uint32_t q[R], child[R], edge = 0;
    bool valid[R];
    uint32_t mark = 0;                                               // a bit per round: the entry begins a position of the current level
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t i = (uint32_t)(r * kLT + tid);
        valid[r] = i < cnt;
        q[r] = dist[valid[r] ? i : cnt - 1];
        child[r] = out + i;
        mark |= valid[r] ? 1u << r : 0u;
    }
    {   // lane r: the distance before the wave's first entry of round r
        const uint32_t i = (uint32_t)((lane & (R - 1)) * kLT + wave * 64);
        edge = i == 0 ? 0u : dist[i - 1 < cnt ? i - 1 : cnt - 1];
    }
    const bool first_here = tid == 0;                     // round 0 of this thread is the bucket's first entry
    const uint32_t first = first_here ? a.first_mask[b] : 0u;
    for (int j = 0; j < L; ++j) {                                    // uniform
        const uint32_t off = f.off[(size_t)b * SP_MAX_RANK + j], size = (uint32_t)f.levels.size[j].d;
        const double half = (double)off + 0.5, inv = f.levels.size[j].inv;
        const uint32_t eup = quotient(edge, half, inv);
        CT *__restrict__ crd = (CT *)a.crd[j];
        PT *__restrict__ pos = (PT *)a.pos[j];
        uint32_t up[R], began = 0, at[R], old[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            up[r] = quotient(q[r], half, inv);
            if ((mark >> r) & 1u) crd[child[r]] = (CT)(uint32_t)(off + q[r] - up[r] * size);
            old[r] = lane_before(up[r], (uint32_t)__builtin_amdgcn_readlane((int)eup, r));
            const bool begins = r == 0 && first_here ? ((first >> (j + 1)) & 1u) != 0 : up[r] != old[r];
            began |= valid[r] && begins ? 1u << r : 0u;
        }
        if (j + 1 < L) {                                             // positions of the compressed level above
            const uint32_t *before = a.heads + (size_t)j * f.most;
            const uint32_t base = before[b] - before[0];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const unsigned long long m = __ballot((began >> r) & 1u);
                at[r] = (uint32_t)__popcll(m & below);
                if (lane == 0) wcnt[j & 1][r * W + wave] = (uint32_t)__popcll(m);
            }
            __syncthreads();
            const uint32_t n = lane < R * W ? wcnt[j & 1][lane] : 0u, excl = wave_inclusive_scan(n, lane) - n;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const bool m = (began >> r) & 1u;
                at[r] += base + (uint32_t)__builtin_amdgcn_readlane((int)excl, r * W + wave) + (m ? 1u : 0u) - 1u;
                if (m) pos[at[r]] = (PT)child[r];
                if (valid[r] && out + (uint32_t)(r * kLT + tid) == (uint32_t)(f.n - 1)) pos[at[r] + 1] = (PT)(child[r] + 1);
                child[r] = at[r];
            }
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!valid[r]) continue;
                const bool m = (began >> r) & 1u, last = out + (uint32_t)(r * kLT + tid) == (uint32_t)(f.n - 1);
                if (!a.dense_above) {
                    if (last) { pos[0] = 0; pos[1] = (PT)(child[r] + 1); }
                } else if (m || last) {
                    // the dense position: what lo's prefix is, and the quotient on top of it
                    uint64_t top = f.bucket[b].lo, prev = a.before_key[b];
                    for (int k = 0; k < L; ++k) { top = spmi_div_by(top, f.levels.size[k]); prev = spmi_div_by(prev, f.levels.size[k]); }
                    const uint64_t P = top + up[r], Q = r == 0 && first_here ? prev : top + old[r];
                    if (m && child[r]) {
                        atomicAdd((UT *)&pos[P], (UT)0 - (UT)child[r]);
                        atomicAdd((UT *)&pos[Q], (UT)child[r]);
                    }
                    if (last) atomicAdd((UT *)&pos[P], (UT)(child[r] + 1));
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) q[r] = up[r];
        edge = eup;
        mark = began;
    }
}

inline size_t pad256(size_t b) { return (b + 255) & ~(size_t)255; }

struct tables {
    level1 t;
    level2 u;
    uint32_t *runs, *split, *frank, *left, *off, *heads, *ends, *first_mask;
    uint64_t *before_key;
    final_bucket *bucket;
    int *flags;
    uint64_t room1, room2;
    uint32_t parts_max, tiles_max;
    size_t bytes;
};

// The tables of a build, one after the other at `tab` (null: how much they take).
tables tables_of(const spmi_bucket_plan &plan, int64_t n, unsigned char *tab)
{
    tables x;
    const uint32_t Q = plan.Q, F = plan.F, S = plan.S;
    const size_t B = Q + F;
    // room of the first partition: the shares add up to n, the margins are largest when all buckets are alike
    x.room1 = (uint64_t)n + 64;
    if (S) x.room1 = (uint64_t)((double)n + (double)B * ((double)n / S * (6.0 * sqrt((double)S / (double)B + 4.0) + 10.0) + 32.0)) + 1024;
    x.room2 = plan.two ? (uint64_t)(2.2 * (double)n) + (uint64_t)B * 4096 : 0;
    x.parts_max = plan.two ? (uint32_t)(n / kTarget) + (uint32_t)B : (uint32_t)B;
    x.tiles_max = plan.two ? (uint32_t)(n / (kPT * kPR)) + (uint32_t)B : 1u;
    x.bytes = 0;
    auto place = [&](size_t b) { unsigned char *at = tab + x.bytes; x.bytes += pad256(b); return (void *)at; };
    x.flags = (int *)place(kSpmiFlagBytes);
    x.runs = (uint32_t *)place((size_t)(S ? S : 4) * 4); x.split = (uint32_t *)place((size_t)(Q + 1) * 4); x.frank = (uint32_t *)place((size_t)(F + 1) * 4);
    x.t.lo = (uint64_t *)place((B + 1) * 8); x.t.start = (uint32_t *)place(B * 4); x.t.end = (uint32_t *)place(B * 4); x.t.cur = (uint32_t *)place(B * 4);
    x.t.lut = (uint16_t *)place((size_t)(kCells + 1) * 2); x.t.out = (uint32_t *)place((B + 1) * 4); x.t.sub0 = (uint32_t *)place((B + 1) * 4);
    x.t.tile0 = (uint32_t *)place((B + 1) * 4); x.t.room2 = (uint32_t *)place(B * 4); x.t.used = (uint32_t *)place(B * 4); x.t.B = (int)B;
    const size_t parts = x.parts_max;
    x.u.lo = (uint64_t *)place((parts + 1) * 8); x.u.start = (uint32_t *)place(parts * 4); x.u.end = (uint32_t *)place(parts * 4); x.u.cur = (uint32_t *)place(parts * 4);
    x.u.tile_bucket = (uint16_t *)place((size_t)x.tiles_max * 2);
    x.left = (uint32_t *)place(parts * 4); x.bucket = (final_bucket *)place(parts * sizeof(final_bucket));
    x.off = (uint32_t *)place(parts * SP_MAX_RANK * 4);
    x.ends = (uint32_t *)place(parts * 8); x.first_mask = (uint32_t *)place(parts * 4); x.before_key = (uint64_t *)place(parts * 8);
    x.heads = (uint32_t *)place(((size_t)plan.slots * parts + 1) * 4);
    return x;
}

final_args final_args_of(const spmi_bucket_job &job, const tables &x)
{
    final_args f;
    memset(&f, 0, sizeof(f));
    f.bucket = x.bucket; f.count = job.plan.two ? x.t.sub0 + x.t.B : nullptr; f.most = x.parts_max; f.n = job.n;
    f.left = x.left; f.flags = x.flags; f.heads = x.heads; f.ends = x.ends; f.off = x.off; f.levels = job.levels;
    f.inner = spmi_make_divisor(1); f.nblocks = ceil_div(job.n, kSpmiStreamT);
    return f;
}

// Room for the entries in their buckets, behind the tables.
template <typename K, typename P>
struct moved {
    K *k1, *k2;
    P *v1, *v2;
    size_t bytes;
    moved(const tables &x, bool two, unsigned char *at)
    {
        const size_t n1 = x.room1 + kDump, n2 = two ? x.room2 + kDump : 0;
        bytes = 0;
        auto place = [&](size_t b) { unsigned char *p = at + bytes; bytes += pad256(b); return (void *)p; };
        v1 = (P *)place(n1 * sizeof(P)); k1 = (K *)place(n1 * sizeof(K));
        v2 = two ? (P *)place(n2 * sizeof(P)) : v1;
        k2 = two ? (K *)place(n2 * sizeof(K)) : k1;
    }
};

template <typename K, typename P>
sp_status move_entries(const spmi_bucket_job &job, const P *vals, hipStream_t st)
{
    const source &src = job.src;
    const spmi_bucket_plan &plan = job.plan;
    const int64_t n = job.n;
    const uint64_t total = job.total;
    const tables x = tables_of(plan, n, (unsigned char *)job.tab);
    const moved<K, P> m(x, plan.two, (unsigned char *)job.tab + x.bytes);
    K *k1 = m.k1, *k2 = m.k2;
    P *v1 = m.v1, *v2 = m.v2;
    const level1 &t = x.t;
    const level2 &u = x.u;
    const int B = t.B;
    const bool two = plan.two;
    const uint64_t room1 = x.room1, room2 = x.room2;
    const uint32_t tiles_max = x.tiles_max;
    int *flags = x.flags;
    int cell_shift = 0;
    while (((total - 1) >> cell_shift) >= (uint64_t)kCells) ++cell_shift;
    // first partition
    const bool small = n < (int64_t)kPT * kPR * 256;
    const int tile = small ? kPT * kSmallR : kWideT * kPR;
    const uint32_t tiles = (uint32_t)ceil_div(n, (int64_t)tile);
    const size_t stage = std::max(stage_bytes<K, P>(tile), (size_t)B * 8 + (kCells + 1) * 2);
    const size_t lds = (((size_t)B * 4 + 15) & ~(size_t)15) + stage + 16;
    const uint32_t dump1 = (uint32_t)room1;
#define SPMI_PART(T_, R_, PER_)                                                                                                    \
    do {                                                                                                                          \
        if (lds > 65536) SP_HIP(hipFuncSetAttribute((const void *)partition_kernel<K, P, T_, R_, PER_>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024 - 512)); \
        hipLaunchKernelGGL((partition_kernel<K, P, T_, R_, PER_>), dim3(round8(tiles)), dim3(T_), lds, st, src, vals, n, t, cell_shift, dump1, k1, v1, flags); \
    } while (0)
    if (!small) SPMI_PART(kWideT, kPR, kMaxBuckets / kWideT);
    else if (B > kPT) SPMI_PART(kPT, kSmallR, kMaxBuckets / kPT);
    else SPMI_PART(kPT, kSmallR, 1);
#undef SPMI_PART
    hipLaunchKernelGGL(bucket_sizes_kernel, dim3(1), dim3(1024), 0, st, t, two ? 1 : 0, (uint32_t)(kPT * kPR), (uint32_t)room2, flags);
    SP_HIP(hipGetLastError());
    if (two) {
        hipLaunchKernelGGL(parts_kernel<K>, dim3((unsigned)B), dim3(1024), 0, st, t, u, (const K *)k1, total, (const int *)flags);
        hipLaunchKernelGGL((partition_again_kernel<K, P, kPR>), dim3(round8(tiles_max)), dim3(kPT), 0, st, (const K *)k1, (const P *)v1, t, u, (uint32_t)room2, k2, v2,
                           (const int *)flags);
        SP_HIP(hipGetLastError());
    }
    return SP_OK;
}

template <typename K, typename P>
sp_status finish(const spmi_bucket_job &job, const spmi_bucket_out &o, sp_scratch &tmp, hipStream_t st)
{
    const spmi_bucket_plan &plan = job.plan;
    const tables x = tables_of(plan, job.n, (unsigned char *)job.tab);
    const moved<K, P> m(x, plan.two, (unsigned char *)job.tab + x.bytes);
    const K *k2 = m.k2;
    const P *v2 = m.v2;
    const level1 &t = x.t;
    const level2 &u = x.u;
    const int B = t.B;
    const bool two = plan.two;
    const uint32_t parts_max = x.parts_max;
    final_args f = final_args_of(job, x);
    f.keys = o.keys; f.dist = o.dist; f.crd = o.crd; f.pos = o.pos; f.rowblk = o.rowblk; f.rows = o.rows; f.pw = o.pw; f.cw = o.cw;
    f.inner = spmi_make_divisor(o.inner ? o.inner : 1);
    hipLaunchKernelGGL(final_buckets_kernel, dim3(two ? (unsigned)B : (unsigned)ceil_div(B, 256)), dim3(256), 0, st, (const uint64_t *)(two ? u.lo : t.lo),
                       (const uint32_t *)(two ? u.start : t.start), (const uint32_t *)(two ? u.end : t.end), (const uint32_t *)(two ? u.cur : t.cur),
                       (const uint32_t *)t.out, (const uint32_t *)(two ? t.sub0 : nullptr), (uint32_t)B, x.bucket, x.off, f);
    hipLaunchKernelGGL((finish_kernel<K, P>), dim3(parts_max), dim3(kFT), 0, st, (const K *)k2, (const P *)v2, (P *)o.values, f);
    hipLaunchKernelGGL((finish_crowded_kernel<K, P>), dim3(std::min(parts_max, 1024u)), dim3(kFT), 0, st, (const K *)k2, (const P *)v2, (P *)o.values, f);
    SP_HIP(hipGetLastError());
    if (!o.dist) return SP_OK;
    hipLaunchKernelGGL(bucket_heads_kernel, dim3((unsigned)ceil_div(parts_max, 256)), dim3(256), 0, st, f, x.first_mask, x.before_key);
    SP_HIP(hipGetLastError());
    if (plan.slots > 0) {
        const int64_t buckets = (int64_t)x.parts_max;
        SP_TRY(spmi_exclusive_scan(x.heads, plan.slots * buckets + 1, 32, tmp, st));          // the last element's input does not reach any output
        hipLaunchKernelGGL(head_totals_kernel, dim3(1), dim3(64), 0, st, (const uint32_t *)x.heads, buckets, plan.slots, (unsigned long long *)(x.flags + 16));
        SP_HIP(hipGetLastError());
    }
    return SP_OK;
}

}  // namespace

bool spmi_bucket_plan_for(int64_t n, uint64_t total, int key_bits, int64_t rows, spmi_bucket_plan *p)
{
    memset(p, 0, sizeof(*p));
    if (n < 1 || total < 1 || key_bits > 48) return false;            // sampled keys keep their upper 32 bits: 16 more may hide a crowd
    p->two = n > (int64_t)kTarget * kOnePartition;
    // blocks enough for the kernel that cuts the buckets (Zipf columns, 3.3 M entries, CSR to CSC: 475 us with buckets of 131072, 375 so)
    const int64_t first = std::min<int64_t>(std::max<int64_t>(n / 128, kFirstLeast), kFirst);
    uint64_t Q = p->two ? (uint64_t)std::max<int64_t>(std::min<int64_t>(ceil_div(n, first), 512), ceil_div(n, 2 * kFirst))
                        : n <= kCap ? 1u : (uint64_t)ceil_div(n, kTarget);
    p->wide = ((total - 1) >> 32) > (uint64_t)std::min<int64_t>(1024, n / kTarget);
    // equal steps of the key range that no bucket crosses: 2^32, so that its keys fit 32 bits, or less where the rows that begin in a
    // bucket, which its block looks up, could be many (a matrix whose last rows are empty)
    p->fbits = p->wide ? 63 : 32;
    const uint64_t stretches = rows > 65536 ? std::min<uint64_t>(std::min<uint64_t>((uint64_t)rows / 16384, 255), Q) : 0;
    if (stretches) {
        int bits = 0;
        while (((total - 1) >> bits) > stretches) ++bits;
        p->fbits = std::min(p->fbits, bits);
    }
    p->F = (uint32_t)((total - 1) >> p->fbits);
    // many equal steps cut the range finely already: fewer splitters besides them (76.9 M entries of rank 3, 745 steps: 2698 -> 2665 us;
    // 70 M of 42-bit keys, evenly 2101 -> 2062, in five steps 2183 -> 2117, 90 % in four 2127 -> 2106, R-MAT 2483 -> 2542)
    if (p->two && p->F >= 512) Q = std::max<uint64_t>(std::min<uint64_t>(Q, 256), (uint64_t)ceil_div(n, 2 * kFirst));
    if (Q + p->F > (uint64_t)kMaxBuckets) return false;
    p->Q = (uint32_t)Q;
    if (Q + p->F > 1) {
        int64_t S = ceil_div((int64_t)(p->two ? kShareFirst : kShare) * (int64_t)Q, kRun) * kRun;
        S = std::min<int64_t>(S, kMaxSample);
        while (S > n) S -= kRun;
        if (S < kRun) return false;
        p->S = (uint32_t)S;
    }
    return true;
}

sp_status spmi_bucket_begin(spmi_bucket_job *job, const void *vals, int payload_bytes, sp_scratch &tmp, hipStream_t st)
{
    const spmi_bucket_plan &plan = job->plan;
    job->payload_bytes = payload_bytes;
    size_t bytes = 0;
    {
        const tables s = tables_of(plan, job->n, nullptr);
        bytes = s.bytes + (payload_bytes == 4 ? (plan.wide ? moved<uint64_t, uint32_t>(s, plan.two, nullptr).bytes : moved<uint32_t, uint32_t>(s, plan.two, nullptr).bytes)
                                              : (plan.wide ? moved<uint64_t, uint64_t>(s, plan.two, nullptr).bytes : moved<uint32_t, uint64_t>(s, plan.two, nullptr).bytes));
    }
    job->tab = tmp.get(bytes);                                        // one block: an allocation costs the caller about 5 us
    if (!job->tab) return SP_ERR_ALLOC;
    const tables x = tables_of(plan, job->n, (unsigned char *)job->tab);
    if (x.room1 + kDump >= 0xfff00000ull || x.room2 + kDump >= 0xfff00000ull) return SP_ERR_TOO_LARGE;
    job->flags = x.flags;
    const uint32_t Q = plan.Q, F = plan.F, S = plan.S;
    const int sshift = job->key_bits > 32 ? job->key_bits - 32 : 0;
    int cell_shift = 0;
    while (((job->total - 1) >> cell_shift) >= (uint64_t)kCells) ++cell_shift;
    if (S) {
        hipLaunchKernelGGL(sample_runs_kernel, dim3(S / kRun), dim3(kRun), 0, st, job->src, job->n, S, sshift, x.runs);
        if ((size_t)S * 4 > 65536)
            SP_HIP(hipFuncSetAttribute((const void *)sample_ranks_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxSample * 4));
        hipLaunchKernelGGL(sample_ranks_kernel, dim3((S + F + kRankT - 1) / kRankT), dim3(kRankT), (size_t)S * 4, st, (const uint32_t *)x.runs, S, sshift, Q, F,
                           x.split, x.frank, plan.fbits);
        SP_HIP(hipGetLastError());
    }
    hipLaunchKernelGGL(buckets_kernel, dim3(1), dim3(1024), 0, st, (const uint32_t *)x.split, (const uint32_t *)x.frank, S, sshift, Q, F, plan.fbits, job->total,
                       cell_shift, job->n, x.t, x.flags);
    SP_HIP(hipGetLastError());
    if (payload_bytes == 4) return plan.wide ? move_entries<uint64_t, uint32_t>(*job, (const uint32_t *)vals, st) : move_entries<uint32_t, uint32_t>(*job, (const uint32_t *)vals, st);
    return plan.wide ? move_entries<uint64_t, uint64_t>(*job, (const uint64_t *)vals, st) : move_entries<uint32_t, uint64_t>(*job, (const uint64_t *)vals, st);
}

sp_status spmi_bucket_end(const spmi_bucket_job &job, const spmi_bucket_out &out, sp_scratch &tmp, hipStream_t st)
{
    if (job.payload_bytes == 4) return job.plan.wide ? finish<uint64_t, uint32_t>(job, out, tmp, st) : finish<uint32_t, uint32_t>(job, out, tmp, st);
    return job.plan.wide ? finish<uint64_t, uint64_t>(job, out, tmp, st) : finish<uint32_t, uint64_t>(job, out, tmp, st);
}

sp_status spmi_bucket_levels(const spmi_bucket_job &job, const uint32_t *dist, void *const *crd, void *const *pos, bool dense_above, int pw, int cw, hipStream_t st)
{
    const tables x = tables_of(job.plan, job.n, (unsigned char *)job.tab);
    final_args f = final_args_of(job, x);
    f.dist = const_cast<uint32_t *>(dist);
    level_arrays a;
    memset(&a, 0, sizeof(a));
    for (int j = 0; j < job.levels.count; ++j) { a.crd[j] = crd[j]; a.pos[j] = pos[j]; }
    a.heads = x.heads; a.first_mask = x.first_mask; a.before_key = x.before_key; a.dense_above = dense_above ? 1 : 0;
    const dim3 grid(x.parts_max);
    if (pw == 32 && cw == 32) hipLaunchKernelGGL((bucket_levels_kernel<int32_t, int32_t>), grid, dim3(kLT), 0, st, f, a);
    else if (pw == 32) hipLaunchKernelGGL((bucket_levels_kernel<int32_t, int64_t>), grid, dim3(kLT), 0, st, f, a);
    else if (cw == 32) hipLaunchKernelGGL((bucket_levels_kernel<int64_t, int32_t>), grid, dim3(kLT), 0, st, f, a);
    else hipLaunchKernelGGL((bucket_levels_kernel<int64_t, int64_t>), grid, dim3(kLT), 0, st, f, a);
    SP_HIP(hipGetLastError());
    return SP_OK;
}
