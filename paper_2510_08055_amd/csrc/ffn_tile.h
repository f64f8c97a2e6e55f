// Pieces shared by the grouped-GEMM kernels (bf16 weights in ffn.hip, 4-bit weights in ffn_w4.hip):
// the device-side tile search, the SwiGLU epilogue function and the helpers of the direct-to-LDS
// software pipeline.
#pragma once
#include "common.h"

namespace moe {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));

// ----------------------------------------------------------------------------------------------
// Work decomposition.  The launch grid is data-independent (an upper bound on the number of
// tiles); every block finds its own (expert, m-tile, n-tile) from the device-side offsets and
// blocks beyond the real tile count exit.  Experts without rows get no tile, so none of their
// weights is read.
//
// Hardware hands consecutive workgroup ids to the 8 XCDs round-robin.  Logical tile ids are
// therefore remapped so that each XCD walks one contiguous eighth of the logical order, and the
// logical order is expert-major, then n-tile, then m-tile: the m-tiles that share one weight
// tile run back to back on the same XCD (second and later reads hit that XCD's L2), and one
// expert's activation rows stay in the same L2 while its n-tiles stream by.
// ----------------------------------------------------------------------------------------------
struct TileCoord {
    int expert, row0, row_end, n_tile;   // rows [row0, row_end) of the permuted batch belong to this tile
    bool alone;                          // no other tile reads its weights (the expert has one m-tile)
    bool valid;
};

// An expert with m rows is cut into ceil(m / BM) m-tiles of (nearly) equal size, each a whole number of
// 32-row blocks: 1032 rows and BM = 256 give 224+224+224+192+168 rather than 4 x 256 + 8, so no block
// streams a whole weight tile for a handful of rows.
// (The host bounds the grid so that the tile count fits 31 bits.)
// Offsets are trusted to be a non-decreasing sequence in [0, max_rows]; they are clamped to that range and
// negative counts to zero all the same, so that offsets gone wrong (a caller's bug, an uninitialised buffer)
// give wrong results inside the output's rows, never a store outside them.
//
// Every block of a launch runs it before it can load anything, and code that runs once costs its instruction misses, about 1 us
// per KB: so it is short for up to 128 experts (two to a lane), what a tile needs is taken from its lane as scalars, and an expert
// with one m-tile needs no division.  Of a block's time at H = 2048, 128 experts, it takes 0.9 us; with eight experts to a lane, shuffles
// and divisions 1.5 to 2.0.  The two launches of 32 tokens: 111.5 + 58.8 -> 109.4 + 53.4 us; a pass of two layers 406 -> 392, of two 4-bit
// layers (2880 x 2880, 256 tokens) 726 -> 697, of one fp32 layer of 64 tokens 26.0 -> 24.1.
template <int BM, int EPL>
__device__ __forceinline__ TileCoord find_tile_in(const int32_t* __restrict__ offsets, int E, int n_tiles, int max_rows)
{
    const int lane = lane_id();
    int off[EPL + 1];
#pragma unroll
    for (int i = 0; i <= EPL; ++i) {
        const int e = lane * EPL + i;
        const int o = offsets[e <= E ? e : E];
        off[i] = o < 0 ? 0 : (o > max_rows ? max_rows : o);
    }
    int mt[EPL];
    int sum = 0;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        const int cnt = off[i + 1] > off[i] ? off[i + 1] - off[i] : 0;
        mt[i] = (cnt + BM - 1) / BM;
        sum += mt[i];
    }
    const int incl = wave_scan(sum);
    const int total = __builtin_amdgcn_readlane(incl, 63) * n_tiles;
    const int chunk = (total + 7) / 8;
    const int slot = blockIdx.x / 8;
    const int logical = (int)(blockIdx.x % 8) * chunk + slot;
    TileCoord tc;
    tc.valid = slot < chunk && logical < total;
    tc.expert = 0; tc.row0 = 0; tc.row_end = 0; tc.n_tile = 0; tc.alone = true;
    if (!tc.valid) return tc;
    // the lane whose experts contain the tile (tiles of an expert: mt_e * n_tiles, n-major), then the expert among that lane's
    const unsigned long long hit = __ballot(logical < incl * n_tiles);
    const int src = __ffsll((long long)hit) - 1;
    int rem = logical - __builtin_amdgcn_readlane(incl - sum, src) * n_tiles;
    int lo = __builtin_amdgcn_readlane(off[0], src), hi = lo, m = 0;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
        const int m_i = __builtin_amdgcn_readlane(mt[i], src), end = __builtin_amdgcn_readlane(off[i + 1], src);
        if (m == 0) {
            if (rem < m_i * n_tiles) {
                m = m_i;
                hi = end;
                tc.expert = src * EPL + i;
            } else {
                rem -= m_i * n_tiles;
                lo = end;
            }
        }
    }
    tc.n_tile = rem;
    tc.row0 = lo;
    tc.row_end = hi;
    tc.alone = m == 1;
    if (!tc.alone) {
        tc.n_tile = rem / m;
        const int t = rem - tc.n_tile * m;
        const int rb = (hi - lo + 31) / 32;                 // 32-row blocks of this expert
        const int per = (rb + m - 1) / m;                   // row blocks per tile
        tc.row0 = lo + t * per * 32;
        tc.row_end = tc.row0 + per * 32;
        if (tc.row_end > hi) tc.row_end = hi;
        if (tc.row0 > tc.row_end) tc.row0 = tc.row_end;     // cannot happen: per * (m - 1) < rb
    }
    // the same in every lane: handed out as scalars, so that what the kernels derive from them (base
    // addresses, row counts, the bookkeeping of the load pipeline) stays in scalar registers
    tc.expert = __builtin_amdgcn_readfirstlane(tc.expert);
    tc.row0 = __builtin_amdgcn_readfirstlane(tc.row0);
    tc.row_end = __builtin_amdgcn_readfirstlane(tc.row_end);
    tc.n_tile = __builtin_amdgcn_readfirstlane(tc.n_tile);
    return tc;
}
template <int BM>
__device__ __forceinline__ TileCoord find_tile(const int32_t* __restrict__ offsets, int E, int n_tiles, int max_rows)
{
    if (E <= 128) return find_tile_in<BM, 2>(offsets, E, n_tiles, max_rows);
    return find_tile_in<BM, kMaxExperts / 64>(offsets, E, n_tiles, max_rows);
}

// Entry `id` of a row map, below `rows`, as the row it stands for: id / div, with magic = map_magic_of(div).
__device__ __forceinline__ uint32_t mapped_row(int32_t id, int rows, int div, uint32_t magic)
{
    // (a row map holds indices below `rows`; the clamp keeps a bad entry from becoming a wild address)
    uint32_t r = id < 0 ? 0u : (uint32_t)id;
    r = r < (uint32_t)rows ? r : (uint32_t)rows - 1;
    if (div > 1) {       // ceil(2^32 / div) overshoots by at most one
        uint32_t q = __umulhi(r, magic);
        if (q * (uint32_t)div > r) q -= 1;
        r = q;
    }
    return r;
}
inline uint32_t map_magic_of(int map_div)
{
    return map_div > 1 ? (uint32_t)((((uint64_t)1 << 32) + map_div - 1) / map_div) : 0;
}

// Host side: tiles of `rows` rows a launch is expected to have when its A rows spread evenly over the experts (an
// expert's last tile is half full on average, and an expert with a row has a tile).
inline int64_t tiles_expected(int64_t A, int E, int rows, int64_t n_tiles)
{
    const int64_t used = A < E ? A : E, m_tiles = A / rows + used / 2;
    return (m_tiles > used ? m_tiles : used) * n_tiles;
}

// silu(g) * u with silu(g) = g / (1 + e^-g); hardware exp2 and reciprocal (1 ulp each), far inside the
// rounding of the bf16 (or the tolerance of the fp32) result.
__device__ __forceinline__ float silu_mul(float g, float u)
{
    return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;
}

// The value as it stands in a register: the compiler can no longer fuse the multiplication that produced it
// into a later subtraction (fp contraction would make `v - round(v)` depend on where it is compiled).
__device__ __forceinline__ float opaque(float v)
{
    asm volatile("" : "+v"(v));
    return v;
}

// Waits and barriers of the software pipeline are inline asm with a memory clobber: the compiler must
// not move LDS reads or the direct-to-LDS loads across them (the bare s_barrier intrinsic is not a
// memory barrier for the optimiser, and __syncthreads() would drain every load still in flight).
template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void block_barrier() { asm volatile("s_barrier" ::: "memory"); }

// One wave-level direct-to-LDS load: lane i's BYTES bytes from `src` land at LDS byte address lds_base + BYTES i
// (lds_base is wave-uniform and travels in M0).  Issued from inline asm on purpose.  The compiler's
// wait-count pass takes the builtin form for an access to both global memory and LDS, and while it
// believes one to be in flight (it never sees the explicit vmcnt waits above, so: always) it turns
// every LDS wait into lgkmcnt(0): an MFMA that needs the fragments read one k-slice ago then also waits
// for the reads just issued for the next slice.  With the asm form the waits carry the exact count.
// The kernels that use it must not leave anything else in M0 (nothing in them does: LDS instructions
// need no M0 on this target).
// STREAM: bytes that nobody asks for again, as a non-temporal load.  A weight tile that one block alone reads is such a stream,
// and most weight tiles of a batch with few rows per expert are: the loads then leave the L2 to the activations, and memory
// delivers more of them (6.8 TB/s against 6.1).  gate_up and down, us, plain / non-temporal: 128 experts, H = I = 2880, 256 tokens
// 697 / 624 and 366 / 338; H = 2048, I = 768, 32 tokens 128 / 114 and 67 / 60, 640 tokens 149 / 139 and 83 / 80.  Weights that several
// m-tiles share must stay: 520 rows per expert 388 / 437 and 225 / 248.  So must weights whose stage rows are not whole 128-byte
// lines (see whole_lines): a line that is gone between its two pieces is fetched twice.
template <int BYTES, bool STREAM = false> __device__ __forceinline__ void load_lds(const void* src, uint32_t lds_base)
{
    static_assert(BYTES == 16 || BYTES == 4 || BYTES == 2, "direct-to-LDS loads move 16, 4 or 2 bytes per lane");
    static_assert(!STREAM || BYTES == 16, "streams are read 16 bytes at a time");
    if (STREAM)
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(src), "s"(lds_base) : "memory");
    else if (BYTES == 16)
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_base) : "memory");
    else if (BYTES == 4)
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(src), "s"(lds_base) : "memory");
    else
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_ushort %0, off" ::"v"(src), "s"(lds_base) : "memory");
}
// Are 128-byte pieces of rows from `base` on, rows and pieces multiples of 128 bytes long, whole lines?  Weights may start at any
// multiple of 16 bytes.  Elsewhere the hint costs a third: gate_up + down, us, 16 bytes into a line, plain / non-temporal:
// 128 experts, H = I = 2880, 2 rows each 1080 / 1436; H = 2048, I = 768, 40 rows 264 / 334, 130 rows 326 / 412.
__device__ __forceinline__ bool whole_lines(const void* base) { return (reinterpret_cast<uintptr_t>(base) & 127u) == 0; }
template <bool STREAM = false> __device__ __forceinline__ void load_lds_16(const void* src, uint32_t lds_base)
{
    load_lds<16, STREAM>(src, lds_base);
}
// An address that is the same in every lane, as a scalar (the compiler does not see every uniform value as one).
__device__ __forceinline__ const char* uniform(const char* p)
{
    const uint64_t b = reinterpret_cast<uint64_t>(p);
    return reinterpret_cast<const char*>((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b) |
                                         (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32)) << 32);
}
// The same load with a wave-uniform base address and a 32-bit byte offset per lane.
template <bool STREAM = false> __device__ __forceinline__ void load_lds_16_base(const void* base, uint32_t offset, uint32_t lds_base)
{
    if (STREAM)
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(offset), "s"(base), "s"(lds_base) : "memory");
    else
        asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(offset), "s"(base), "s"(lds_base) : "memory");
}
// LDS byte address of a pointer into the block's dynamic shared memory
__device__ __forceinline__ uint32_t lds_address(const void* p)
{
    return (uint32_t)(uintptr_t)(lds_ptr_t*)p;
}

// Source-side swizzle of a tile row: which LDS 16-byte chunk slot holds global chunk c of row r is
// c ^ swz(r).  Chosen so that the 16-byte operand reads of 8 (and of 16) consecutive rows fall into
// distinct bank groups whether the LDS serves 128 or 256 bytes per clock.
// (rows of 128 bytes: eight chunks)
__device__ __forceinline__ int swz(int r) { return (r & 7) ^ ((r >> 3) & 1); }

// Epilogue of a wave's TMV row blocks (wm, wm + WM, ... of the tile whose rows are [row0, row_end)) by TNO * 32 output columns
// from `col0` on.  A lane holds, for output row fr of a row block, groups of 4 consecutive columns (accumulator element v of
// tile (i, j): column (v/4)*8 + fq*4 + v%4); storing them directly would scatter 8-byte pieces over 32 rows per
// instruction.  The wave instead turns one row block at a time through `epi`, 32 * TNO * 64 bytes of LDS (float output: 4 KB) that only it uses
// (no block barrier: a wave's own LDS operations execute in program order), and writes it out as whole 16-byte chunks,
// consecutive lanes along a row (64- or 128-byte runs per row).
template <bool GATED, bool OUT_F32, bool SPLIT, int TMV, int TNO, int WM, typename ACC>
__device__ __forceinline__ void store_tile(ACC& acc, int row0, int row_end, int wm, int col0, char* epi, void* Out_, int ldo,
                                           int N)
{
    if (TMV == 0) return;
    // (the lane number as an unknown value: a persistent kernel's compiler would otherwise work the addresses below out once,
    // in front of the block's loop over its tiles, and hold them in registers the k-loop needs)
    int lane = lane_id();
    asm volatile("" : "+v"(lane));
    const int fr = lane & 31, fq = lane >> 5;
    constexpr int RB = TNO * 64;              // bytes of one row of the wave's output tile
    constexpr int CPRW = TNO * 4;             // 16-byte chunks per such row
    constexpr int RPI = 64 / CPRW;            // rows one wave-level 16-byte access covers
    static_assert(TNO <= 2, "columns of a wave");
    if constexpr (OUT_F32) {
        // float output: one 32 x 32 tile (4 KB: 32 rows of 8 16-byte chunks) at a time; a lane's 4 consecutive columns are
        // one chunk, chunk c of row r sits in chunk slot c ^ (r & 7), and the tile goes out as 128-byte runs per row
        float* Out = static_cast<float*>(Out_);
#pragma unroll
        for (int i = 0; i < TMV; ++i) {
            const int64_t row_base = (int64_t)row0 + (wm + WM * i) * 32;
#pragma unroll
            for (int j = 0; j < TNO; ++j) {
#pragma unroll
                for (int a = 0; a < 4; ++a)
                    *reinterpret_cast<float4*>(epi + fr * 128 + (((a * 2 + fq) ^ (fr & 7)) << 4)) =
                        make_float4(acc[i][j][a * 4], acc[i][j][a * 4 + 1], acc[i][j][a * 4 + 2], acc[i][j][a * 4 + 3]);
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const int r = h * 8 + (lane >> 3), c = lane & 7;
                    const float4 v = *reinterpret_cast<const float4*>(epi + r * 128 + ((c ^ (r & 7)) << 4));
                    const int64_t row = row_base + r;
                    const int col = col0 + j * 32 + c * 4;
                    if (row < row_end && col < N)    // N is a multiple of 8: the 4 columns are in or out together
                        *reinterpret_cast<float4*>(Out + row * ldo + col) = v;
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
    } else {
        bf16_t* Out = static_cast<bf16_t*>(Out_);
        auto eswz = [](int r) { return (r >> (RB == 64 ? 2 : 1)) & (CPRW - 1); };
        constexpr int PARTS = (SPLIT && GATED) ? 2 : 1;      // the values, then what their bf16 rounding left over
#pragma unroll
        for (int i = 0; i < TMV; ++i) {
            if (GATED) {
#pragma unroll
                for (int j = 0; j < TNO; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        acc[i][j][v] = silu_mul(acc[i][j][v], acc[i][j + TNO][v]);
                        if (SPLIT) acc[i][j][v] = opaque(acc[i][j][v]);
                    }
            }
#pragma unroll
            for (int part = 0; part < PARTS; ++part) {
#pragma unroll
                for (int j = 0; j < TNO; ++j) {
#pragma unroll
                    for (int a = 0; a < 4; ++a) {
                        float val[4];
#pragma unroll
                        for (int b = 0; b < 4; ++b) val[b] = acc[i][j][a * 4 + b];
                        const uint32_t p01 = pack_bf16x2(val[0], val[1]), p23 = pack_bf16x2(val[2], val[3]);
                        if (PARTS == 2 && part == 0) {      // keep the remainders for the second part
                            acc[i][j][a * 4 + 0] = val[0] - __uint_as_float(p01 << 16);
                            acc[i][j][a * 4 + 1] = val[1] - __uint_as_float(p01 & 0xffff0000u);
                            acc[i][j][a * 4 + 2] = val[2] - __uint_as_float(p23 << 16);
                            acc[i][j][a * 4 + 3] = val[3] - __uint_as_float(p23 & 0xffff0000u);
                        }
                        const int chunk = (j * 4 + a) ^ eswz(fr);
                        *reinterpret_cast<uint2*>(epi + fr * RB + chunk * 16 + fq * 8) = make_uint2(p01, p23);
                    }
                }
                __builtin_amdgcn_wave_barrier();
                const int64_t row_base = (int64_t)row0 + (wm + WM * i) * 32;
#pragma unroll
                for (int h = 0; h < 32 / RPI; ++h) {
                    const int r = h * RPI + lane / CPRW, c = lane % CPRW;
                    const uint4 v = *reinterpret_cast<const uint4*>(epi + r * RB + ((c ^ eswz(r)) * 16));
                    const int64_t row = row_base + r;
                    const int col = col0 + c * 8;
                    if (row < row_end && col < N)    // N is a multiple of 8: a chunk is in or out as a whole
                        *reinterpret_cast<uint4*>(Out + row * ldo + part * N + col) = v;
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
}

}  // namespace moe
