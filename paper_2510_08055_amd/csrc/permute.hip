// Token permutation: per-expert histogram, prefix sum and a STABLE rank of every
// assignment, so that the tokens routed to each expert (Sec. 3.1) form a contiguous,
// deterministically ordered batch: order = (expert, token, slot).
//
// Counting uses LDS integer atomics (order-free, hence deterministic).  The rank of an
// assignment inside its expert comes from an ordered scan, never from "claim a slot"
// atomics: tile prefix (from the per-tile histograms) + wave prefix + a running per-wave
// counter + the rank among equal experts inside one 64-wide chunk (ballot matching).
#include "common.h"

namespace moe {

// Expert ids are trusted to lie in [0, E); clamping keeps a corrupt id from indexing outside LDS.
__device__ __forceinline__ int clamp_expert(int e, int E) { return e < 0 ? 0 : (e >= E ? E - 1 : e); }

// What bounds these kernels is the chain inside a block (a round of ballots, LDS counters and scattered stores per
// 1024 assignments), not bytes: tiles of 2048 assignments give two rounds per block and more blocks.  Against tiles
// of 8192 (eight rounds; events around the launch): 5120 assignments 15.3 -> 9.1 us, 16896 18.3 -> 9.2 us, 66560
// 20.0 -> 9.6 us.
constexpr int kPermThreads = 1024;                       // 16 waves
constexpr int kPermWaves = kPermThreads / 64;
constexpr int kPermRounds = kPermTile / kPermThreads;    // 64-wide chunks per wave
static_assert(kPermRounds * kPermThreads == kPermTile, "tile must be a whole number of rounds");

// Pass 1 (only when there is more than one tile): tile_hist[tile][e].
__global__ __launch_bounds__(kPermThreads) void permute_hist_kernel(const int32_t* __restrict__ idx, int64_t A,
                                                                    int E, int32_t* __restrict__ tile_hist)
{
    __shared__ int32_t hist[kMaxExperts];
    for (int e = threadIdx.x; e < E; e += kPermThreads) hist[e] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kPermTile;
    for (int i = threadIdx.x; i < kPermTile; i += kPermThreads) {
        const int64_t f = base + i;
        if (f < A) atomicAdd(&hist[clamp_expert(idx[f], E)], 1);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += kPermThreads) tile_hist[(int64_t)blockIdx.x * E + e] = hist[e];
}

// Between the passes, for many tiles (see launch_permute): tile_hist[tile][e] becomes the sum over the tiles in front,
// tile_hist[n_tiles][e] the sum over all.  A block takes 64 experts, one per lane; each wave sums a run of tiles, the
// waves' sums meet in LDS, then the wave writes its run's running sums.
__global__ __launch_bounds__(kPermThreads) void permute_scan_kernel(int32_t* __restrict__ tile_hist, int n_tiles, int E)
{
    __shared__ int32_t wave_sum[kPermWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int e = (int)blockIdx.x * 64 + lane;
    const int run = (n_tiles + kPermWaves - 1) / kPermWaves;
    const int first = wave * run < n_tiles ? wave * run : n_tiles;
    const int last = first + run < n_tiles ? first + run : n_tiles;
    int sum = 0;
    if (e < E)
#pragma unroll 8
        for (int t = first; t < last; ++t) sum += tile_hist[(int64_t)t * E + e];
    wave_sum[wave][lane] = sum;
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wave; ++w) before += wave_sum[w][lane];
    if (e < E) {
        constexpr int AHEAD = 8;       // rows fetched in front of the chain of sums
        for (int t0 = first; t0 < last; t0 += AHEAD) {
            int h[AHEAD];
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) h[i] = t0 + i < last ? tile_hist[(int64_t)(t0 + i) * E + e] : 0;
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                if (t0 + i < last) tile_hist[(int64_t)(t0 + i) * E + e] = before;
                before += h[i];
            }
        }
        if (wave == kPermWaves - 1) tile_hist[(int64_t)n_tiles * E + e] = before;
    }
}

// Pass 2: every block derives the global offsets (all tiles' histograms are tiny) and the
// start of its own tile inside each expert, then ranks and scatters its assignments.
// COUNT: the block counts all assignments itself (a single tile, or few: see launch_permute) and pass 1 is skipped.
// SCANNED: the sums over the tiles are already in tile_hist.
//
// COUNT: an LDS atomic takes a turn per lane that shares its address, 0.7 ns each, and under skewed routing a wave's 64 assignments are of few
// experts.  So an expert has kCopies counters, one to eight neighbouring lanes (of neighbouring banks), and a counter's upper half is the
// count in front of the tile: one atomic per assignment, not two.  moe_permute of 12288 assignments, top-1, us, one counter for the
// count and one for what is in front / these: 16 experts, all of one of them 22.4 / 6.4, skewed (rank^-1.2) 10.7 / 5.8, even 7.1 / 5.6;
// 128 experts 22.9 / 6.9, 9.8 / 6.4, 6.7 / 6.3; 512 experts 24.2 / 8.3, 10.6 / 7.7, 8.0 / 7.8.
constexpr int kCopies = 8;
template <bool SCANNED, bool COUNT>
__global__ __launch_bounds__(kPermThreads) void permute_scatter_kernel(
    const int32_t* __restrict__ idx, int64_t A, int E, int n_tiles, const int32_t* __restrict__ tile_hist,
    int32_t* __restrict__ counts, int32_t* __restrict__ offsets, int32_t* __restrict__ perm,
    int32_t* __restrict__ inv, unsigned long long* __restrict__ active_total)
{
    __shared__ int32_t total[kMaxExperts];              // assignments per expert, whole batch
    __shared__ uint32_t copies[COUNT ? kMaxExperts * kCopies : 1];
    __shared__ int32_t start[kMaxExperts];              // first permuted row of this tile inside expert e
    __shared__ int32_t wave_cnt[kPermWaves][kMaxExperts];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile = blockIdx.x;
    const int64_t base = (int64_t)tile * kPermTile;

    // all of this thread's expert ids are fetched up front: one memory latency, under that of the histograms
    int my_e[kPermRounds], my_rank[kPermRounds];
#pragma unroll
    for (int r = 0; r < kPermRounds; ++r) {
        const int64_t f = base + (int64_t)wave * (kPermRounds * 64) + r * 64 + lane;
        my_e[r] = f < A ? idx[f] : -1;
    }
    if (COUNT) {
        for (int i = tid; i < E * kCopies; i += kPermThreads) copies[i] = 0;
    } else {
        for (int e = tid; e < E; e += kPermThreads) {
            total[e] = 0;
            start[e] = 0;
        }
    }
    for (int e = lane; e < E; e += 64) wave_cnt[wave][e] = 0;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPermRounds; ++r) {
        const int64_t f = base + (int64_t)wave * (kPermRounds * 64) + r * 64 + lane;
        my_e[r] = f < A ? clamp_expert(my_e[r], E) : -1;
    }
    if (SCANNED) {
        for (int e = tid; e < E; e += kPermThreads) {
            total[e] = tile_hist[(int64_t)n_tiles * E + e];
            start[e] = tile_hist[(int64_t)tile * E + e];
        }
    } else if (COUNT) {
        constexpr int AT_ONCE = 8;
        static_assert(kCountTiles * kPermTile < 1 << 16, "a half of a counter holds them all");
        uint32_t* const mine = copies + (lane >> 3);
        static_assert(kCopies == 8, "one to eight lanes of 64");
#pragma unroll 1
        for (int64_t f0 = tid; f0 < A; f0 += AT_ONCE * kPermThreads) {
            int e[AT_ONCE];
#pragma unroll
            for (int i = 0; i < AT_ONCE; ++i) e[i] = f0 + i * kPermThreads < A ? idx[f0 + i * kPermThreads] : -1;
#pragma unroll
            for (int i = 0; i < AT_ONCE; ++i) {
                const int64_t f = f0 + i * kPermThreads;
                if (f >= A) break;
                atomicAdd(mine + clamp_expert(e[i], E) * kCopies, f < base ? 0x10001u : 1u);
            }
        }
    } else {
        // the threads share out the (expert, eighth of the tiles) pairs: a few loads in flight per thread, not a
        // chain of n_tiles; integer sums do not depend on the order of the atomics
        for (int i = tid; i < 8 * E; i += kPermThreads) {
            const int eighth = i / E, e = i - eighth * E;
            int tot = 0, before = 0;
#pragma unroll 4
            for (int t = eighth; t < n_tiles; t += 8) {
                const int h = tile_hist[(int64_t)t * E + e];
                tot += h;
                before += t < tile ? h : 0;
            }
            if (tot) atomicAdd(&total[e], tot);
            if (before) atomicAdd(&start[e], before);
        }
    }
    __syncthreads();
    // exclusive scan over experts by wave 0, 64 at a time
    if (wave == 0) {
        int before = 0, act = 0;
#pragma unroll 1
        for (int e0 = 0; e0 < E; e0 += 64) {
            const int e = e0 + lane;
            int n = 0, in_front = 0;
            if (COUNT && e < E) {
                uint32_t both = 0;
#pragma unroll
                for (int i = 0; i < kCopies; ++i) both += copies[e * kCopies + i];
                n = (int)(both & 0xffffu);
                in_front = (int)(both >> 16);
            } else if (e < E) {
                n = total[e];
                in_front = start[e];
            }
            const int incl = wave_scan(n) + before;
            if (e < E) {
                start[e] = in_front + incl - n;
                if (tile == 0) {
                    counts[e] = n;
                    offsets[e] = incl - n;
                }
            }
            act += (int)__popcll(__ballot(n > 0));
            before = __builtin_amdgcn_readlane(incl, 63);
        }
        if (tile == 0 && lane == 0) {
            offsets[E] = before;
            if (active_total) atomicAdd(active_total, (unsigned long long)act);
        }
    }

    // Rank inside the wave's region of kPermRounds * 64 assignments, chunk by chunk in index order.
    int nbits = 0;
    while ((1 << nbits) < E) ++nbits;
    // (wave 0 meanwhile scans the counts: wave_cnt is the wave's own, and `start` is not read before the barrier behind this.)
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int r = 0; r < kPermRounds; ++r) {
        const bool valid = my_e[r] >= 0;
        const int e = valid ? my_e[r] : 0;
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < nbits; ++b) {
            const bool bit = (e >> b) & 1;
            const uint64_t bal = __ballot(valid && bit);
            peers &= bit ? bal : ~bal;
        }
        if (valid) {
            my_rank[r] = wave_cnt[wave][e] + __popcll(peers & lt_mask);
        } else {
            my_rank[r] = 0;
        }
        // wave_cnt[wave] is private to this wave and a wave's LDS operations execute in program order,
        // so the update below cannot overtake the reads above: no block barrier inside the rounds.
        __builtin_amdgcn_wave_barrier();
        if (valid && (63 - __clzll(peers)) == lane) wave_cnt[wave][e] += __popcll(peers);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // wave_cnt[w][e] becomes the first permuted row of wave w's assignments to expert e: this tile's
    // start inside the expert plus the counts of the waves in front (one pass per expert, instead of
    // every assignment adding up the waves in front of it)
    for (int e = tid; e < E; e += kPermThreads) {
        int c[kPermWaves];
#pragma unroll
        for (int wv = 0; wv < kPermWaves; ++wv) c[wv] = wave_cnt[wv][e];
        int run = start[e];
#pragma unroll
        for (int wv = 0; wv < kPermWaves; ++wv) {
            wave_cnt[wv][e] = run;
            run += c[wv];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPermRounds; ++r) {
        const int e = my_e[r];
        if (e < 0) continue;
        const int pos = wave_cnt[wave][e] + my_rank[r];
        const int64_t f = base + (int64_t)wave * (kPermRounds * 64) + r * 64 + lane;
        perm[pos] = (int32_t)f;
        inv[f] = pos;
    }
}

template <typename VT>
__global__ __launch_bounds__(256) void gather_rows_kernel(const VT* __restrict__ x, const int32_t* __restrict__ perm,
                                                          int K, int64_t A, int vec_per_row, VT* __restrict__ out)
{
    const int64_t r = blockIdx.x;
    if (r >= A) return;
    const int64_t src = perm[r] / K;
    const VT* s = x + src * vec_per_row;
    VT* d = out + r * vec_per_row;
    for (int i = threadIdx.x; i < vec_per_row; i += 256) d[i] = s[i];
}

hipError_t launch_permute(const int32_t* idx, int64_t A, int E, int32_t* counts, int32_t* offsets, int32_t* perm,
                          int32_t* inv, int32_t* tile_hist, bool hist_ready, unsigned long long* active_total,
                          hipStream_t s)
{
    const int n_tiles = (int)((A + kPermTile - 1) / kPermTile);
    // Few tiles are counted by every block of the scatter.  In a call of its own that is a launch less, us, with it / without, 12288 assignments,
    // even routing: 2 experts 5.5 / 6.3, 16 experts 5.6 / 6.4, 128 experts 6.3 / 7.5, 512 experts 7.8 / 10.1; all of one expert 5.9 / 6.9, 6.4 /
    // 7.3, 6.9 / 7.9, 8.3 / 10.4.  Behind a top-k it is its histogram that is saved, which costs less (a pass over rows of 64 values, top-1,
    // 128 experts, even routing / all of one expert): 4096 assignments 27.5 / 28.7 and 27.3 / 27.6, 8192 35.9 / 36.5 and 35.8 / 34.9,
    // 12288 38.2 / 38.2 and 38.4 / 36.5; 8 experts 22.1 / 23.3 and 22.0 / 22.7, 24.6 / 25.3 and 24.8 / 24.6, 27.9 / 28.7 and 28.3 / 27.9.
    if (!hist_ready && A <= (int64_t)kCountTiles * kPermTile) {
        permute_scatter_kernel<false, true><<<n_tiles, kPermThreads, 0, s>>>(idx, A, E, n_tiles, tile_hist, counts, offsets, perm, inv,
                                                                             active_total);
        return hipGetLastError();
    }
    if (!hist_ready) {
        permute_hist_kernel<<<n_tiles, kPermThreads, 0, s>>>(idx, A, E, tile_hist);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // Every block of the scatter reads all histograms, which grows with the square of their number: beyond 2^25 words read in
    // all, a pass over the tiles (one more launch) is cheaper.  Permutation alone, us, without / with it: 512 experts:
    // 786432 assignments 37.4 / 20.3, 2 M 140 / 38, 8 M 1628 / 127; 128 experts: 2 M 49.4 / 32.7, 8 M 435 / 109.  At the border
    // (524288 and 1 M) the direct sums take 23 and 21 us.
    if ((int64_t)n_tiles * n_tiles * E > ((int64_t)1 << 25)) {
        permute_scan_kernel<<<(E + 63) / 64, kPermThreads, 0, s>>>(tile_hist, n_tiles, E);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        permute_scatter_kernel<true, false><<<n_tiles, kPermThreads, 0, s>>>(idx, A, E, n_tiles, tile_hist, counts, offsets, perm,
                                                                      inv, active_total);
    } else {
        permute_scatter_kernel<false, false><<<n_tiles, kPermThreads, 0, s>>>(idx, A, E, n_tiles, tile_hist, counts, offsets, perm,
                                                                       inv, active_total);
    }
    return hipGetLastError();
}

// Zeroes n 32-bit words.  In place of hipMemsetAsync wherever a caller may be capturing the stream into a
// HIP graph (memset nodes have replayed wrongly on this platform).
__global__ __launch_bounds__(256) void fill_zero_kernel(uint32_t* __restrict__ p, int n)
{
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i < n) p[i] = 0u;
}

hipError_t launch_fill_zero(void* p, int n_words, hipStream_t s)
{
    if (n_words <= 0) return hipSuccess;
    fill_zero_kernel<<<(unsigned)((n_words + 255) / 256), 256, 0, s>>>(static_cast<uint32_t*>(p), n_words);
    return hipGetLastError();
}

hipError_t launch_gather_rows(int dtype, const void* x, const int32_t* perm, int K, int64_t A, int H, void* x_perm,
                              hipStream_t s)
{
    const int row_bytes = H * (dtype == MOE_BF16 ? 2 : 4);
    gather_rows_kernel<uint4><<<(unsigned)A, 256, 0, s>>>((const uint4*)x, perm, K, A, row_bytes / 16,
                                                          (uint4*)x_perm);
    return hipGetLastError();
}

}  // namespace moe
