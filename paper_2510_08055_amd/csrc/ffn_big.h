// What the persistent 256 x 256 grouped GEMMs share (bf16 weights in ffn.hip, 4-bit weights in ffn_w4.hip): the tile
// list a block works through and the activation rows of its tiles.
#pragma once
#include "ffn_tile.h"

namespace moe {

constexpr int kBigRows = 256, kBigBN = 256, kBigWaves = 8, kBigMinHeight = 4;

// Cost of a tile that does not depend on its height, in units of one of its 32-row blocks: about 8 us against 0.17 us per
// block and k-step, fitted to launches of different heights at nk = 12 and 32.  3 us of it lie between two k-loops
// (epilogue, change of tile); the rest are waits inside the k-loop that the MFMAs of the blocks do not cover.
__device__ __forceinline__ float big_tile_fixed(int nk) { return 48.0f / (float)nk + 0.35f; }

__device__ __forceinline__ int last_lane(int v) { return __builtin_amdgcn_readlane(v, 63); }
__device__ __forceinline__ float last_lane(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// The largest of the values of 8 neighbouring lanes, in all of them.
__device__ __forceinline__ float eight_max(float v)
{
    auto step = [&](auto ctrl) {
        v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value, 0xF, 0xF, true)));
    };
    step(std::integral_constant<int, 0xB1>{});       // lane ^ 1, lane ^ 2, mirrored within 8
    step(std::integral_constant<int, 0x4E>{});
    step(std::integral_constant<int, 0x141>{});
    return v;
}

struct BigTile {
    int expert, row0, row_end, n_tile;
};

// ceil(x / h) for 0 <= x < 2^28 and 4 <= h <= 8 (inverse: ceil(2^32 / h), exact in this range)
__device__ __forceinline__ uint32_t height_inverse(int h)
{
    return h == 8 ? 0x20000000u : h == 7 ? 0x24924925u : h == 6 ? 0x2aaaaaabu : h == 5 ? 0x33333334u : 0x40000000u;
}
__device__ __forceinline__ int div_up(int x, int h, uint32_t inverse) { return (int)__umulhi((uint32_t)(x + h - 1), inverse); }

// The block's share of the tile list: a range of it with a stride, and the expert the walk has reached.  Everything
// here is the same in all lanes.
//
// Every block works the list out for itself.  What that costs is instruction fetch (cold straight-line code runs at
// about 1 KB per us: a first version, unrolled over the 8 experts of a lane, was 11 KB and took 10 us of every
// launch), hence the loops that are kept loops and the walk over the experts in place of a search; then trips to memory one
// behind the other, hence two experts' offsets at a time and the first tile's expert by a scan.  128 experts 3.0 to 3.4 us, 32
// experts 2.3 (4.2 to 4.5 and 3.0 with a trip per 64 experts, a loop over the heights and a walk to the first tile).
struct BigQueue {
    const int32_t* offsets;
    int E, max_rows, n_tiles;
    int h;                     // tile height limit in row blocks
    uint32_t h_inv;
    int end;                   // end of the block's range
    bool mostly_alone;         // nearly every expert with rows has one m-tile: its weight tiles are read by one block
    int expert, before;        // the walk: an expert, tiles of the experts in front of it,
    int lo, hi, mt, per;       // its rows, its number of m-tiles and the row blocks of each

    __device__ __forceinline__ void load_expert()
    {
        // (one scalar load with its wait inside: through the compiler it might become a vector load, whose wait
        // would also be a wait for every asm-issued load in flight)
        unsigned long long pair;
        asm volatile("s_load_dwordx2 %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=&s"(pair) : "s"(offsets + expert) : "memory");
        lo = (int)(uint32_t)pair;
        hi = (int)(uint32_t)(pair >> 32);
        lo = lo < 0 ? 0 : (lo > max_rows ? max_rows : lo);
        hi = hi < lo ? lo : (hi > max_rows ? max_rows : hi);
        set_expert((hi - lo + 31) / 32);
    }
    __device__ __forceinline__ void set_expert(int rb)
    {
        mt = div_up(rb, h, h_inv);
        per = mt > 1 ? quotient(rb + mt - 1, mt) : rb;
    }
    // x / m for 0 <= x < 2^24 (the launch keeps lists of more tiles away), a few instructions instead of a division
    static __device__ __forceinline__ int quotient(int x, int m)
    {
        int q = (int)((float)x * __builtin_amdgcn_rcpf((float)m));
        if (q * m > x) q -= 1;
        if (x - q * m >= m) q += 1;
        return __builtin_amdgcn_readfirstlane(q);
    }

    // Tile j of the list; j never decreases from call to call and is below the number of tiles.
    __device__ __forceinline__ BigTile take(int j)
    {
        while (j >= before + mt * n_tiles && expert + 1 < E) {
            before += mt * n_tiles;
            expert += 1;
            load_expert();
        }
        const int m = mt > 0 ? mt : 1;
        const int rem = j - before;
        const int n = quotient(rem, m), t = rem - n * m;
        BigTile tile;
        tile.expert = expert;
        tile.n_tile = n;
        tile.row0 = lo + t * per * 32;
        tile.row_end = tile.row0 + per * 32;
        if (tile.row_end > hi) tile.row_end = hi;
        if (tile.row0 > tile.row_end) tile.row0 = tile.row_end;
        return tile;
    }

    // Every wave of the block calls it, with `scratch` a piece of LDS nothing else uses (kQueueWords).  Returns the block's first tile.
    static constexpr int kFrom = 64, kTo = kFrom + kMaxExperts, kRb = kTo + kMaxExperts, kQueueWords = kRb + kMaxExperts;
    __device__ __forceinline__ int init(const int32_t* offsets_, int E_, int n_tiles_, int max_rows_, float fixed, int* scratch)
    {
        offsets = offsets_;
        E = E_;
        max_rows = max_rows_;
        n_tiles = n_tiles_;
        const int lane = lane_id();
        const int k = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));       // wave
        int* const tiles_at = scratch;              // [8] tiles at height 8 - k
        float* const squares_at = reinterpret_cast<float*>(scratch + 8);     // [8] sum of their squared heights
        int* const border = scratch + 16;           // [2][8] first tile of piece k: equal numbers, equal costs
        float* const b_cost = reinterpret_cast<float*>(scratch + 32);        // [8] cost in front of border[0][k]
        int* const from = scratch + kFrom;          // [E] first row, end of the rows
        int* const to = scratch + kTo;
        int* const rb_of = scratch + kRb;           // [E] row blocks

        // wave k: number of tiles at height 8 - k
        int rb_sum = 0, t_sum = 0, used = 0;
        float sq_sum = 0.f;                         // sum of the tiles' squared heights
        {
            const int hh = kBigRows / 32 - k >= kBigMinHeight ? kBigRows / 32 - k : kBigMinHeight;
            const uint32_t inv = height_inverse(hh);
#pragma unroll 1
            for (int e0 = lane; e0 < E; e0 += 128) {       // (two experts at a time: one trip to memory up to 128 of them)
                int r0[2], r1[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int e = e0 + 64 * i < E ? e0 + 64 * i : E - 1;
                    r0[i] = offsets[e];
                    r1[i] = offsets[e + 1];
                }
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    if (e0 + 64 * i >= E) break;
                    const int lo_e = r0[i] < 0 ? 0 : (r0[i] > max_rows ? max_rows : r0[i]);
                    const int hi_e = r1[i] < lo_e ? lo_e : (r1[i] > max_rows ? max_rows : r1[i]);
                    const int rb = (hi_e - lo_e + 31) / 32;
                    if (k == 0) {
                        from[e0 + 64 * i] = lo_e;
                        to[e0 + 64 * i] = hi_e;
                        rb_of[e0 + 64 * i] = rb;
                    }
                    const int m = div_up(rb, hh, inv);
                    rb_sum += rb;
                    used += rb > 0;
                    t_sum += m;
                    sq_sum += rb > 0 ? (float)rb * (float)rb * __builtin_amdgcn_rcpf((float)m) : 0.f;
                }
            }
        }
        t_sum = last_lane(wave_scan(t_sum));
        sq_sum = last_lane(wave_scan(sq_sum));
        const float rb_all = (float)last_lane(wave_scan(rb_sum)) * (float)n_tiles;
        used = last_lane(wave_scan(used));
        if (lane == 0) {
            tiles_at[k] = t_sum;
            squares_at[k] = sq_sum;
        }
        __syncthreads();
        const float blocks = (float)gridDim.x;
        {
            // lane c: the launch at height 8 - c (whole rounds of the mean tile, and what the unluckiest block gets on top by chance)
            constexpr int LAST = kBigRows / 32 - kBigMinHeight;
            const int c = lane < LAST ? lane : LAST;
            const float tiles = fmaxf((float)tiles_at[c] * (float)n_tiles, 1.f), inv = __builtin_amdgcn_rcpf(tiles);
            const float rounds = ceilf(tiles * __builtin_amdgcn_rcpf(blocks) - 1e-3f), mean = rb_all * inv;
            const float var = fmaxf(squares_at[c] * (float)n_tiles * inv - mean * mean, 0.f);
            const float cost = rounds * (fixed + mean) + 1.5f * __builtin_amdgcn_sqrtf(rounds * var);
            static_assert(LAST < 8, "eight lanes hold every height");
            const unsigned long long best = __ballot(cost == -eight_max(-cost));
            h = kBigRows / 32 - (__ffsll((long long)best) - 1);       // (the highest of equal ones)
        }
        h_inv = height_inverse(h);
        const int m_tiles = __builtin_amdgcn_readfirstlane(tiles_at[kBigRows / 32 - h]);
        mostly_alone = m_tiles - used <= used / 16;
        const int total = m_tiles * n_tiles;
        const float ftotal = fixed * (float)total + rb_all;

        // Border k of the eight pieces: after k / 8 of the tiles, or where the running cost passes k / 8 of the total.
        // Pieces of equal cost suit tiles of different heights; pieces of equal number never need one more round
        // than the whole list does.  Wave k works both out for k (and the cost in front of the first), they meet in
        // LDS, and the kind whose slowest piece is estimated to end first is taken: whole rounds of its mean tile.
        {
            const float target = ftotal * (float)k * 0.125f;
            const int by_count = (int)((int64_t)total * k / 8);
            int sum = 0;
            float fsum = 0.f;
            bool found = false, found_n = false;
#pragma unroll 1
            for (int e0 = 0; e0 < E; e0 += 64) {
                const int rb = e0 + lane < E ? rb_of[e0 + lane] : 0;
                const int tiles = div_up(rb, h, h_inv) * n_tiles;
                const float c = fixed * (float)tiles + (float)rb * (float)n_tiles;
                const int cum = wave_scan(tiles) + sum;
                const float fcum = wave_scan(c) + fsum;
                const unsigned long long past_n = __ballot(cum > by_count), past = __ballot(fcum > target);
                // (one lane is picked: one whose number of tiles and cost are not zero)
                if (!found_n && past_n) {
                    found_n = true;
                    if (lane == __ffsll((long long)past_n) - 1) {
                        border[k] = by_count;
                        b_cost[k] = fcum - c * (float)(cum - by_count) * __builtin_amdgcn_rcpf((float)tiles);
                    }
                }
                if (!found && past) {
                    found = true;
                    if (lane == __ffsll((long long)past) - 1) {
                        const float behind = fminf((fcum - target) * __builtin_amdgcn_rcpf(c), 1.f);
                        border[8 + k] = k > 0 ? cum - (int)(behind * (float)tiles) : 0;
                    }
                }
                sum = last_lane(cum);
                fsum = last_lane(fcum);
            }
            if (lane == 0) {     // (only if rounding puts the last borders behind the last expert, or nothing has rows)
                if (!found_n) {
                    border[k] = total;
                    b_cost[k] = ftotal;
                }
                if (!found) border[8 + k] = total;
            }
        }
        __syncthreads();
        // lane y < 8 of every wave: piece y, both ways
        const int y = lane & 7;
        const float n0 = (float)(y < 7 ? border[y + 1] : total) - (float)border[y];
        const float n1 = (float)(y < 7 ? border[9 + y] : total) - (float)border[8 + y];
        const float per_block = 8.f * __builtin_amdgcn_rcpf(blocks);
        const float slow0 = n0 > 0.f ? ceilf(n0 * per_block - 1e-3f) * ((y < 7 ? b_cost[y + 1] : ftotal) - b_cost[y]) * __builtin_amdgcn_rcpf(n0) : 0.f;
        const float slow1 = n1 > 0.f ? ceilf(n1 * per_block - 1e-3f) * (ftotal * 0.125f) * __builtin_amdgcn_rcpf(n1) : 0.f;
        const int x = (int)(blockIdx.x % 8);
        const int at = (__builtin_amdgcn_readfirstlane(eight_max(slow1) < eight_max(slow0)) != 0 ? 8 : 0) + x;
        const int first = __builtin_amdgcn_readfirstlane(border[at]) + (int)(blockIdx.x / 8);
        end = x == 7 ? total : __builtin_amdgcn_readfirstlane(border[at + 1]);
        // the expert of the first tile, and the tiles in front of it (a block without a tile: the last expert)
        before = 0;
        expert = E - 1;
#pragma unroll 1
        for (int e0 = 0; e0 < E; e0 += 64) {
            const int rb = e0 + lane < E ? rb_of[e0 + lane] : 0;
            const int tiles = div_up(rb, h, h_inv) * n_tiles;
            const int cum = wave_scan(tiles) + before;
            const unsigned long long past = __ballot(cum > first);
            if (past != 0) {
                const int src = __ffsll((long long)past) - 1;
                expert = e0 + src;
                before = __builtin_amdgcn_readlane(cum - tiles, src);
                break;
            }
            before = last_lane(cum);
        }
        lo = __builtin_amdgcn_readfirstlane(from[expert]);
        hi = __builtin_amdgcn_readfirstlane(to[expert]);
        set_expert(__builtin_amdgcn_readfirstlane(rb_of[expert]));
        __syncthreads();       // `scratch` is free again
        return first;
    }
};

// The activation side of a tile: the wave's load p covers tile rows (wave + 8 p) * 8 .. + 7, lane = (row, 16-byte
// chunk); LDS chunk c of tile row r holds global chunk c ^ swz(r) (swz looks at the low four row bits only: the same
// for every p).
template <bool MAPPED> struct BigRows {
    static constexpr int LPW = kBigRows / 8 / kBigWaves;     // load instructions per wave and stage
    static constexpr int ROWB = 128;                         // bytes per row and stage of 64 k-values
    RowSrc X;
    int ldx;
    const int32_t* row_map;
    int map_div;
    uint32_t map_magic;
    int a_rows, wave, l_row;
    uint32_t l_chunk;
    int32_t row_id[MAPPED ? LPW : 1];  // looked-up rows of the next tile (asm-issued loads: see below)
    // the lane's 16 bytes of stage 0 of the tile whose stages are being loaded: addresses of gathered rows, or offsets
    // from the tile's first row (rows without a map lie in one buffer)
    const char* src[MAPPED ? LPW : 1];
    const char* base;
    uint32_t off[MAPPED ? 1 : LPW];
    int live;                          // of the wave's loads, how many hold rows of that tile

    __device__ __forceinline__ BigRows(const RowSrc& X_, int ldx_, const int32_t* row_map_, int map_div_, uint32_t map_magic_,
                                       int a_rows_, int wave_)
        : X(X_), ldx(ldx_), row_map(row_map_), map_div(map_div_), map_magic(map_magic_), a_rows(a_rows_), wave(wave_),
          l_row(lane_id() >> 3), base(nullptr), live(0)
    {
        l_chunk = (uint32_t)((lane_id() & 7) ^ swz(wave * 8 + l_row)) * 16;
    }

    // The look-ups are loads issued from inline asm: through the compiler they would be waited for with vmcnt(0),
    // i.e. together with all weight loads in flight.  They are picked up one step later, behind a wait that leaves only
    // younger loads in flight.
    __device__ __forceinline__ void look_up(const BigTile& t)
    {
        if constexpr (MAPPED) {
#pragma unroll
            for (int p = 0; p < LPW; ++p) {
                int r = t.row0 + (wave + kBigWaves * p) * 8 + l_row;
                if (r >= t.row_end) r = t.row_end - 1;
                asm volatile("global_load_dword %0, %1, off" : "=v"(row_id[p]) : "v"(row_map + r) : "memory");
            }
        }
    }
    __device__ __forceinline__ void use(const BigTile& t)
    {
        if constexpr (!MAPPED) base = uniform(static_cast<const char*>(X.p0) + (int64_t)t.row0 * ldx * 2);
#pragma unroll
        for (int p = 0; p < LPW; ++p) {
            if constexpr (MAPPED) {
                asm volatile("" : "+v"(row_id[p])::"memory");
                const uint32_t id = mapped_row(row_id[p], a_rows, map_div, map_magic);
                src[p] = reinterpret_cast<const char*>(row_ptr<bf16_t>(X, (int64_t)id, ldx)) + l_chunk;
            } else {
                int r = (wave + kBigWaves * p) * 8 + l_row;
                if (t.row0 + r >= t.row_end) r = t.row_end - 1 - t.row0;      // past the tile: a valid row, result unused
                off[p] = (uint32_t)r * (uint32_t)ldx * 2u + l_chunk;
            }
        }
        const int n = (t.row_end - t.row0 - wave * 8 + 63) / 64;
        live = n < 0 ? 0 : (n > LPW ? LPW : n);
    }
    // (a load whose 8 rows all lie past the tile's last row is left out: no wait count may include an activation load)
    __device__ __forceinline__ void issue_at(uint32_t byte, uint32_t lds_slot) const      // of the row
    {
#pragma unroll
        for (int p = 0; p < LPW; ++p)
            if (p < live) {
                const uint32_t at = lds_slot + (wave + kBigWaves * p) * 1024;
                if constexpr (MAPPED) load_lds_16(src[p] + byte, at);
                else load_lds_16_base(base + byte, off[p], at);
            }
    }
    __device__ __forceinline__ void issue(int stage, uint32_t lds_slot) const { issue_at((uint32_t)(stage * ROWB), lds_slot); }
};

// Host side: blocks of a launch (one per compute unit, the same number on every XCD), and whether the tile list is short
// enough to be counted (the device uses floats here and there).  Tiles are at least 4 row blocks high: sum_e
// ceil(m_e / 128) never exceeds A / 128 + min(A, E).
inline hipError_t big_grid(int* grid)
{
    int cus = 0;
    const hipError_t e = compute_units(&cus);
    *grid = cus / 8 * 8 > 0 ? cus / 8 * 8 : 8;
    return e;
}
inline bool big_list_fits(int64_t A, int E, int64_t n_tiles)
{
    return A < ((int64_t)1 << 28) && ((A + 127) / 128 + (A < E ? A : E)) * n_tiles < ((int64_t)1 << 24);
}

}  // namespace moe
