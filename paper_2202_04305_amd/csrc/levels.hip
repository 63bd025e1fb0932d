// The level sweep of the storage builder: sorted keys -> pos / crd of every level (arXiv 2202.04305, Section 4.1).
//
// The key prefix down to level l (the key divided by the product of the level sizes below) says which position of level l an
// entry belongs to: a dense level's position is parent * size + coordinate; a compressed level's is the number of distinct
// prefixes up to the entry, minus one.  So everything an entry has to write follows from its own key, the key before it and, per
// compressed level above the innermost, the number of distinct prefixes before its tile.  Two passes over the keys in tiles of
// 1024, whatever the rank: one counts the distinct prefixes of those levels per tile (their scan also gives the level sizes, all
// with one read-back), one writes the coordinates and pos entries of all levels at once.  Formats without such a level (CSR, CSC,
// ...) need the second pass only.
//   pos under a compressed level is written directly (every position has a child: its first child's position is known where it
//   begins); under a dense level, where positions may be empty, children are counted with one integer add where a parent begins
//   and one where the next begins (order-free), and the caller scans the counts.
// Bound: memory (rank 3, 76.9 M entries: the keys twice and 1.0 GB of coordinates and pos).  Measured there: 171 + 537 us, against
// 3.9 ms for a marks / scan / emit round per level with a parent position per entry between the levels.  The divisions are kept low by
// dividing each key once per level and taking the previous entry's prefix from the neighbouring lane.
#include "spmi_internal.h"

namespace {

constexpr int kThreads = 256;
constexpr int kRounds = 4;
constexpr int kTile = kThreads * kRounds;
constexpr int kWaves = kThreads / 64;

struct sweep_level {
    spmi_divisor stride;        // product of the level sizes below
    uint64_t size;
    void *crd, *pos;            // compressed levels
    const uint32_t *before;     // compressed levels above the innermost: distinct prefixes before each tile (less before[0], see base)
    int compressed;
};
struct sweep_args {
    sweep_level level[SP_MAX_RANK];
    int rank;
};

__device__ __forceinline__ uint64_t lane_before(uint64_t v, uint64_t first)
{
    // v of the lane below; lane 0 takes `first` (wave shift right by one lane)
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)first, (int)(uint32_t)v, 0x138, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(first >> 32), (int)(uint32_t)(v >> 32), 0x138, 0xf, 0xf, false);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t lane_value(uint64_t v, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// The keys of a thread: entry tile + r * kThreads + thread in round r.  `edge`, in lane r: the key before the wave's first entry of
// round r (the one of entry 0: itself; the marks treat entry 0 apart).
__device__ __forceinline__ void load_tile(const uint64_t *__restrict__ keys, int64_t n, int64_t tile, uint64_t (&k)[kRounds], uint64_t &edge)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const int64_t e = tile + r * kThreads + (int64_t)threadIdx.x;
        k[r] = keys[e < n ? e : n - 1];
    }
    int64_t b = tile + (lane & (kRounds - 1)) * kThreads + wave * 64 - 1;
    b = b < 0 ? 0 : b < n ? b : n - 1;
    edge = keys[b];
}

// counts[level slot * tiles + tile] = entries of the tile that begin a new prefix of a compressed level above the innermost
__global__ __launch_bounds__(kThreads) void sweep_count_kernel(const uint64_t *__restrict__ keys, int64_t n, sweep_args a, uint32_t *__restrict__ counts,
                                                               int64_t tiles)
{
    __shared__ uint32_t wsum[SP_MAX_RANK][kWaves];
    const int64_t tile = (int64_t)blockIdx.x * kTile;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t k[kRounds], edge;
    load_tile(keys, n, tile, k, edge);
    int slots = 0;
    for (int l = 0; l + 1 < a.rank; ++l) {                        // uniform
        if (!a.level[l].compressed) continue;
        const uint64_t pedge = spmi_div_by(edge, a.level[l].stride);
        uint32_t c = 0;
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int64_t e = tile + r * kThreads + (int64_t)threadIdx.x;
            const uint64_t pre = spmi_div_by(k[r], a.level[l].stride);
            c += (uint32_t)__popcll(__ballot(e < n && (e == 0 || pre != lane_before(pre, lane_value(pedge, r)))));
        }
        if (lane == 0) wsum[slots][wave] = c;
        ++slots;
    }
    __syncthreads();
    if ((int)threadIdx.x < slots) {
        uint32_t c = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) c += wsum[threadIdx.x][w];
        counts[(int64_t)threadIdx.x * tiles + blockIdx.x] = c;
    }
}

// totals[s] = the number of positions of level slot s, from the scanned counts (slots one after the other, one element more)
__global__ void sweep_totals_kernel(const uint32_t *__restrict__ scanned, int64_t tiles, int slots, unsigned long long *__restrict__ totals)
{
    const int s = threadIdx.x;
    if (s < slots) totals[s] = (unsigned long long)(scanned[(int64_t)(s + 1) * tiles] - scanned[(int64_t)s * tiles]);
}

template <typename PT, typename CT, typename W>
__global__ __launch_bounds__(kThreads) void sweep_emit_kernel(const uint64_t *__restrict__ keys, int64_t n, sweep_args a, const W *__restrict__ vals,
                                                              W *__restrict__ vout, int *__restrict__ dup_flags)
{
    __shared__ uint32_t wcnt[kRounds * kWaves];
    const int64_t tile = (int64_t)blockIdx.x * kTile;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long below = (1ull << lane) - 1ull;
    typedef typename std::conditional<sizeof(PT) == 8, unsigned long long, unsigned int>::type UT;
    uint64_t k[kRounds], edge;
    load_tile(keys, n, tile, k, edge);
    // position of the entry (P) and of the entry before it (Q) at the level above, their key prefixes (up, vp) and, a bit per round,
    // whether the two differ: the entry begins a position there
    uint64_t P[kRounds], Q[kRounds], up[kRounds], vp[kRounds];
    uint32_t began = 0;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        P[r] = Q[r] = up[r] = vp[r] = 0;
        if (tile + r * kThreads + (int64_t)threadIdx.x == 0) began |= 1u << r;
    }
    if (dup_flags) {
        bool dup = false;
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int64_t e = tile + r * kThreads + (int64_t)threadIdx.x;
            dup |= e > 0 && e < n && k[r] == lane_before(k[r], lane_value(edge, r));
        }
        if (dup) atomicOr(&dup_flags[1], 1);
    }
    bool dense_so_far = true;
    for (int l = 0; l < a.rank; ++l) {                            // uniform
        const sweep_level &lv = a.level[l];
        const bool inner = l == a.rank - 1;
        const uint64_t pedge = spmi_div_by(edge, lv.stride);
        uint64_t pre[kRounds], prv[kRounds];
        uint32_t mark = 0;
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int64_t e = tile + r * kThreads + (int64_t)threadIdx.x;
            pre[r] = spmi_div_by(k[r], lv.stride);
            prv[r] = lane_before(pre[r], lane_value(pedge, r));
            if (e < n && (e == 0 || pre[r] != prv[r])) mark |= 1u << r;
        }
        if (!lv.compressed) {
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                if (dense_so_far) { P[r] = pre[r]; Q[r] = prv[r]; }
                else {
                    P[r] = P[r] * lv.size + (pre[r] - up[r] * lv.size);
                    Q[r] = Q[r] * lv.size + (prv[r] - vp[r] * lv.size);
                }
            }
        } else {
            // where a mark's position lies: the marks before it in the tile's order (round, wave, lane)
            uint32_t at[kRounds];
            if (!inner) {
                __syncthreads();                                  // the table of the level before has been read
#pragma unroll
                for (int r = 0; r < kRounds; ++r) {
                    const unsigned long long m = __ballot((mark >> r) & 1u);
                    at[r] = (uint32_t)__popcll(m & below);
                    if (lane == 0) wcnt[r * kWaves + wave] = (uint32_t)__popcll(m);
                }
                __syncthreads();
                const uint32_t base = lv.before[blockIdx.x] - lv.before[0];
                uint32_t c = lane < kRounds * kWaves ? wcnt[lane] : 0;
                const uint32_t excl = wave_inclusive_scan(c, lane) - c;
#pragma unroll
                for (int r = 0; r < kRounds; ++r) at[r] += base + (uint32_t)__builtin_amdgcn_readlane((int)excl, r * kWaves + wave);
            }
            CT *__restrict__ crd = (CT *)lv.crd;
            PT *__restrict__ pos = (PT *)lv.pos;
            const bool parent_dense = l > 0 && !a.level[l - 1].compressed;
#pragma unroll
            for (int r = 0; r < kRounds; ++r) {
                const int64_t e = tile + r * kThreads + (int64_t)threadIdx.x;
                const bool m = (mark >> r) & 1u;
                const uint64_t child = inner ? (uint64_t)e : (uint64_t)at[r] + (m ? 1u : 0u) - 1u;
                if (e < n) {
                    if (m || inner) crd[child] = (CT)(pre[r] - up[r] * lv.size);
                    if ((began >> r) & 1u) {
                        if (parent_dense) {
                            if (child) {
                                atomicAdd((UT *)&pos[P[r]], (UT)0 - (UT)child);
                                atomicAdd((UT *)&pos[Q[r]], (UT)child);
                            }
                        } else pos[P[r]] = (PT)child;
                    }
                    if (e == n - 1) {
                        if (parent_dense) atomicAdd((UT *)&pos[P[r]], (UT)(child + 1));
                        else pos[P[r] + 1] = (PT)(child + 1);
                    }
                }
                P[r] = child;
                Q[r] = child - (m ? 1u : 0u);
            }
            dense_so_far = false;
        }
#pragma unroll
        for (int r = 0; r < kRounds; ++r) { up[r] = pre[r]; vp[r] = prv[r]; }
        began = mark;
    }
    if (vout) {                                                   // innermost level dense: the values go to their positions
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const int64_t e = tile + r * kThreads + (int64_t)threadIdx.x;
            if (e < n) vout[P[r]] = vals[e];
        }
    }
}

}  // namespace

static sweep_args make_args(const sp_tensor *t)
{
    sweep_args a;
    memset(&a, 0, sizeof(a));
    a.rank = t->enc.rank;
    for (int l = 0; l < a.rank; ++l) {
        uint64_t stride = 1;
        for (int k = l + 1; k < a.rank; ++k) stride *= (uint64_t)(t->size[k] > 0 ? t->size[k] : 1);
        a.level[l].stride = spmi_make_divisor(stride);
        a.level[l].size = (uint64_t)(t->size[l] > 0 ? t->size[l] : 1);
        a.level[l].compressed = t->enc.lt[l] == SP_COMPRESSED;
    }
    return a;
}

sp_status spmi_sweep_count(const sp_tensor *t, const uint64_t *keys, int64_t n, sp_scratch &tmp, hipStream_t st, unsigned long long *totals,
                           uint32_t **counts)
{
    *counts = nullptr;
    int slots = 0;
    for (int l = 0; l + 1 < t->enc.rank; ++l) slots += t->enc.lt[l] == SP_COMPRESSED;
    if (!slots || n <= 0) return SP_OK;
    const int64_t tiles = ceil_div(n, kTile);
    uint32_t *c = (uint32_t *)tmp.get((size_t)(slots * tiles + 1) * 4);
    if (!c) return SP_ERR_ALLOC;
    hipLaunchKernelGGL(sweep_count_kernel, dim3((unsigned)tiles), dim3(kThreads), 0, st, keys, n, make_args(t), c, tiles);
    SP_HIP(hipGetLastError());
    SP_TRY(spmi_exclusive_scan(c, slots * tiles + 1, 32, tmp, st));   // the last element's input does not reach any output
    hipLaunchKernelGGL(sweep_totals_kernel, dim3(1), dim3(64), 0, st, (const uint32_t *)c, tiles, slots, totals);
    SP_HIP(hipGetLastError());
    *counts = c;
    return SP_OK;
}

sp_status spmi_sweep_emit(const sp_tensor *t, const uint64_t *keys, int64_t n, const uint32_t *counts, const void *vals, void *vout, int *dup_flags,
                          hipStream_t st)
{
    if (n <= 0) return SP_OK;
    const int64_t tiles = ceil_div(n, kTile);
    sweep_args a = make_args(t);
    int slot = 0;
    for (int l = 0; l < a.rank; ++l) {
        if (!a.level[l].compressed) continue;
        a.level[l].crd = t->crd[l];
        a.level[l].pos = t->pos[l];
        if (l + 1 < a.rank) a.level[l].before = counts + (int64_t)(slot++) * tiles;
    }
#define SPMI_EMIT(PT, CT)                                                                                                          \
    do {                                                                                                                          \
        if (t->dtype == SP_F64)                                                                                                   \
            hipLaunchKernelGGL((sweep_emit_kernel<PT, CT, unsigned long long>), dim3((unsigned)tiles), dim3(kThreads), 0, st, keys, n, a,  \
                               (const unsigned long long *)vals, (unsigned long long *)vout, dup_flags);                          \
        else                                                                                                                      \
            hipLaunchKernelGGL((sweep_emit_kernel<PT, CT, uint32_t>), dim3((unsigned)tiles), dim3(kThreads), 0, st, keys, n, a,   \
                               (const uint32_t *)vals, (uint32_t *)vout, dup_flags);                                              \
    } while (0)
    if (t->enc.pw == 32 && t->enc.cw == 32) SPMI_EMIT(int32_t, int32_t);
    else if (t->enc.pw == 32) SPMI_EMIT(int32_t, int64_t);
    else if (t->enc.cw == 32) SPMI_EMIT(int64_t, int32_t);
    else SPMI_EMIT(int64_t, int64_t);
#undef SPMI_EMIT
    SP_HIP(hipGetLastError());
    return SP_OK;
}
