// Grouped expert FFN with 4-bit expert weights (MXFP4) and bf16 activations.
//
// The paper's broader validation (Table 7) runs a model whose expert weights are fp4; what changes for
// the MoE layer is the bytes per expert, hence where the ridge of Sec. 2.5 lies: a decode-heavy batch
// streams 17/32 of a byte per weight instead of 2.  The format is the published OCP Microscaling MXFP4:
// FP4 E2M1 elements, two per byte (even element in the low nibble), one E8M0 scale byte (2^(s-127)) per
// 32 consecutive elements along k.  A dequantised weight is exactly representable in bf16, so the GEMM
// is the bf16 MFMA GEMM of ffn.hip on weights widened on the fly (v_cvt_scalef32_pk_bf16_fp4).
//
// Three kernel shapes.  The first, for many rows per expert in few tiles or with short rows (K < 512): 64-row x
// 256-weight-row tiles, 4 waves side by side along the weight rows (each widens and multiplies its own
// 64 weight rows against the tile's one or two 32-row blocks), 64 k-values per stage; activation rows
// come through a 2-stage LDS ring as in ffn.hip.  The packed weight rows and their scale bytes are
// fetched for TWO stages at a time (64 bytes of codes and 4 scale bytes per row) into a ring of 3 such
// double stages: the layer is bound by the number of memory requests, not their bytes, when every row
// contributes 32 + 2 bytes per stage (measured: 2.7x slower).  72 KB of LDS: two blocks share a compute
// unit.  The second, the weight-streaming shape for decode-heavy batches, and the third, the compute-bound one, are
// described further down.  In all, within a 64-wide stage lane (row, q) feeds k-block q (32 values) to four successive MFMAs, 8
// values each, and the activation fragments follow the same k assignment; stages and MFMAs run in the
// same ascending order, so the shapes produce bit-identical results and a chunked and a layered pass
// may pick different ones.
#include "ffn_big.h"

namespace moe {

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

namespace {

constexpr int kW4Rows = 64, kW4BN = 256, kW4Waves = 4, kW4K = 64;
constexpr size_t kW4BigLds = (size_t)(2 * 256 * 128 + 4 * 256 * 64 + 3 * 256 * 16);     // see the kernel
constexpr int kW4NSA = 2, kW4NSB = 3;     // activation stages; weight DOUBLE stages (two stages each)

// Loads that may still be in flight while the wave goes on: the pipeline keeps count of the load
// instructions it has issued and of the last one each stage needs, so the wait is exact in the start-up
// and drain steps as well.  s_waitcnt takes an immediate: the count is rounded down to the next value in the tree.
__device__ __forceinline__ void wait_vmcnt_at_most(int n)
{
    if (n >= 10) {
        if (n >= 16) {
            if (n >= 20) wait_vmcnt<20>();
            else if (n >= 18) wait_vmcnt<18>();
            else wait_vmcnt<16>();
        } else {
            if (n >= 14) wait_vmcnt<14>();
            else if (n >= 12) wait_vmcnt<12>();
            else wait_vmcnt<10>();
        }
    } else {
        if (n >= 4) {
            if (n >= 8) wait_vmcnt<8>();
            else if (n >= 6) wait_vmcnt<6>();
            else wait_vmcnt<4>();
        } else {
            if (n >= 3) wait_vmcnt<3>();
            else if (n >= 2) wait_vmcnt<2>();
            else if (n >= 1) wait_vmcnt<1>();
            else wait_vmcnt<0>();
        }
    }
}

// 8 FP4 values (one dword) times the block's scale -> 8 bf16, in k order.
__device__ __forceinline__ bf16x8_t widen_fp4x8(uint32_t v, float scale)
{
    const bf16x2_t p0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(v, scale, 0);
    const bf16x2_t p1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(v, scale, 1);
    const bf16x2_t p2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(v, scale, 2);
    const bf16x2_t p3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(v, scale, 3);
    return bf16x8_t{p0[0], p0[1], p1[0], p1[1], p2[0], p2[1], p3[0], p3[1]};
}

// E8M0 scale byte -> float 2^(s - 127); s = 0 is 2^-127, a subnormal float.
// (any other byte gives at least 0x00800000.)
__device__ __forceinline__ float e8m0_to_float(uint32_t s)
{
    const uint32_t bits = s << 23;
    return __uint_as_float(bits > 0x00400000u ? bits : 0x00400000u);
}

// The same for byte SH / 8 of a word, in three instructions: the byte is moved into the exponent field
// in place, and 2^-127 = 0x00400000 exceeds the result only when the byte is 0.  (Written as a compare
// and select the compiler extracts the byte twice, with three constants moved into registers per use.)
template <int SH> __device__ __forceinline__ float e8m0_byte_to_float(uint32_t word)
{
    uint32_t bits = (SH <= 23 ? word << (23 - SH) : word >> (SH - 23)) & 0x7f800000u, out;
    asm("v_max_u32 %0, %1, %2" : "=v"(out) : "s"(0x00400000u), "v"(bits));
    return __uint_as_float(out);
}

//   Out[r, n] = sum_k X[src(r), k] * W[e, n, k]                                        (GATED = false)
//   Out[r, n] = silu(sum_k X.. * W[e, n, k]) * (sum_k X.. * W[e, N + n, k])            (GATED = true)
// W: packed codes [E][rows][K/2] bytes, S: scales [E][rows][K/32] bytes; rows = N (or 2N when GATED).
// Requires K % 64 == 0.
// OUT_F32: the output is stored as float (down GEMM of a context that keeps y_perm in fp32).
template <bool GATED, bool OUT_F32>
__global__ __launch_bounds__(kW4Waves * 64, 2) void grouped_gemm_w4_kernel(
    RowSrc X, int ldx, const int32_t* __restrict__ row_map, int map_div, uint32_t map_magic,
    const int32_t* __restrict__ offsets, int E,
    const uint8_t* __restrict__ W, const uint8_t* __restrict__ S, int64_t rows_per_expert, int N, int K,
    void* __restrict__ Out_, int ldo, int a_rows)
{
    static_assert(!(GATED && OUT_F32), "the intermediate of the gated GEMM is always bf16");
    constexpr int BM = kW4Rows, BN = kW4BN, NW = kW4Waves, NSA = kW4NSA, NSB = kW4NSB, PBK = kW4K;
    constexpr int WN = NW;                      // the waves sit side by side along the weight rows
    constexpr int TM = BM / 32;                 // every wave multiplies all row blocks of the tile
    constexpr int NO = GATED ? BN / 2 : BN;     // output columns per block
    constexpr int WNO = NO / WN;                // output columns per wave
    constexpr int TNO = WNO / 32;
    constexpr int TN = GATED ? 2 * TNO : TNO;
    constexpr int A_ROWB = PBK * 2, A_SLOT = BM * A_ROWB;        // 128-byte activation rows, 8 KB per stage
    constexpr int B_ROWB = PBK, B_SLOT = BN * B_ROWB;            // 64 bytes of codes per weight row and DOUBLE stage
    constexpr int S_SLOT = BN * 4;                               // 4 scale bytes per weight row and double stage
    constexpr int SW_STAGES = 8, SW_SLOT = BN * 16;              // or, for rows of 16+ scale bytes: 16 per 8 stages
    constexpr int A_LPW = BM / 8 / NW;                           // activation loads per wave and stage (8 rows each)
    constexpr int B_LPW = BN / 16 / NW;                          // code loads per wave and double stage (16 rows each)
    constexpr int B_BASE = NSA * A_SLOT, S_BASE = B_BASE + NSB * B_SLOT;   // the scale area: max(NSB * S_SLOT, 2 * SW_SLOT)
    static_assert(A_LPW == 2 && B_LPW == 4 && TNO >= 1 && TM == 2, "tile configuration");
    static_assert((NSA - 1) * A_LPW + (NSB - 1) * (B_LPW + 1) + 2 <= 20, "wait_vmcnt_at_most covers up to 20 loads in flight");

    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const uint32_t ldsb = lds_address(smem);    // LDS byte address of the block's dynamic shared memory

    const int n_tiles = (N + NO - 1) / NO;
    const TileCoord tc = find_tile<BM>(offsets, E, n_tiles, a_rows);
    if (!tc.valid) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);    // wave-uniform: the load bookkeeping stays in scalar registers
    const int wn = wave;
    const int n0 = tc.n_tile * NO;
    const int nk = K / PBK;
    const int64_t row_bytes = K / 2, row_scales = K / 32;
    const uint8_t* We = W + (int64_t)tc.expert * rows_per_expert * row_bytes;
    const uint8_t* Se = S + (int64_t)tc.expert * rows_per_expert * row_scales;

    // ---- source addresses ----
    // activations: load p of this wave covers tile rows (wave + NW p) * 8 .. + 7, lane = (row, 16-byte chunk)
    const int a_lrow = lane >> 3, a_chunk = lane & 7;
    int32_t a_row_id[A_LPW];
#pragma unroll
    for (int p = 0; p < A_LPW; ++p) {
        int r = tc.row0 + (wave + NW * p) * 8 + a_lrow;
        if (r >= tc.row_end) r = tc.row_end - 1;
        a_row_id[p] = row_map ? (int32_t)mapped_row(row_map[r], a_rows, map_div, map_magic) : r;
    }
    // weights: the wave's load covers tile rows wave * 32 .. + 31, lane = (row, 16-byte MX block of the stage)
    auto weight_row = [&](int rb) {       // tile row -> row of the expert's weight matrix
        int n;
        if (GATED) n = (rb < NO) ? (n0 + rb) : (n0 + rb - NO);
        else n = n0 + rb;
        if (n >= N) n = N - 1;
        if (GATED && rb >= NO) n += N;
        return n;
    };
    // Code load p of this wave covers tile rows (wave + NW p) * 16 .. + 15, lane = (row, 16-byte MX block of
    // the double stage); LDS block slot c of tile row r holds block c ^ bswz(r), so that the 16-byte operand
    // reads of consecutive rows (64 bytes apart) spread over the banks.
    auto bswz = [](int r) { return (r >> 2) & 3; };
    const uint8_t* b_src[B_LPW];
    bool b_first_half[B_LPW];     // this lane's block lies in the first stage of the double stage
#pragma unroll
    for (int p = 0; p < B_LPW; ++p) {
        const int rb = (wave + NW * p) * 16 + (lane >> 2);
        const int blk = (lane & 3) ^ bswz(rb);
        b_src[p] = We + (int64_t)weight_row(rb) * row_bytes + blk * 16;
        b_first_half[p] = blk < 2;
    }
    // Scales: wave w covers tile rows 64 w .. 64 w + 63, one row per lane, the 4 scale bytes of a
    // double stage as one (2-byte-aligned) dword.  When K is an odd number of stages the last double stage
    // has only 2 scale bytes left in the row: the dword is then taken 2 bytes earlier (or, for K = 64, the
    // load is 2 bytes wide), so that nothing past the row is read.
    // Rows with at least 16 scale bytes (K >= 512) fetch them 16 at a time instead, one load per row and 8
    // stages, into a ring of two such chunks; a chunk that would run past the row starts 16 bytes before
    // the row's end.  (Every row costs a memory request however few bytes it asks for, and the scales
    // were half of the requests.)
    const bool wide_scales = row_scales >= 16;
    const int n_chunks = (nk + SW_STAGES - 1) / SW_STAGES;
    auto chunk_start = [&](int c) {      // first scale byte of chunk c within the row
        const int b = c * 16;
        return b + 16 <= (int)row_scales ? b : (int)row_scales - 16;
    };
    const uint8_t* s_src = Se + (int64_t)weight_row(wave * 64 + lane) * row_scales;
    const int n_double = (nk + 1) / 2;
    const bool odd_tail = (nk & 1) != 0;

    int issued = 0;                    // load instructions this wave has issued
    int last_b[NSB], last_a[NSA];      // `issued` right after the last load of the (double) stage in each ring slot
    auto issue_b = [&](int d) {        // double stage d = stages 2d and 2d + 1
        const uint32_t bs = ldsb + B_BASE + (d % NSB) * B_SLOT;
        const bool tail = odd_tail && d == n_double - 1;
#pragma unroll
        for (int p = 0; p < B_LPW; ++p)
            if (!tail || b_first_half[p]) load_lds<16>(b_src[p] + (int64_t)d * B_ROWB, bs + (wave + NW * p) * 1024);
        issued += B_LPW;     // (every wave has lanes on both sides of the tail mask, so both loads are always issued)
        if (!wide_scales) {
            const uint32_t dst = ldsb + S_BASE + (d % NSB) * S_SLOT + wave * 256;
            if (!tail) load_lds<4>(s_src + d * 4, dst);
            else if (row_scales >= 4) load_lds<4>(s_src + row_scales - 4, dst);
            else load_lds<2>(s_src, dst);
            issued += 1;
        }
#pragma unroll
        for (int i = 0; i < NSB; ++i)
            if (i == d % NSB) last_b[i] = issued;
    };
    int last_s[2] = {0, 0};
    auto issue_s = [&](int c) {        // wide scale chunk c = stages 8c .. 8c + 7
        load_lds<16>(s_src + chunk_start(c), ldsb + S_BASE + (c & 1) * SW_SLOT + wave * 1024);
        issued += 1;
        if (c & 1) last_s[1] = issued;
        else last_s[0] = issued;
    };
#pragma unroll
    for (int i = 0; i < NSB; ++i) last_b[i] = 0;
#pragma unroll
    for (int i = 0; i < NSA; ++i) last_a[i] = 0;
    // the weight stages of the prologue go in flight while the row-map lookups return
    if (wide_scales) issue_s(0);
#pragma unroll
    for (int d = 0; d < NSB - 1; ++d)
        if (d < n_double) issue_b(d);
    const bf16_t* a_src[A_LPW];
#pragma unroll
    for (int p = 0; p < A_LPW; ++p) {
        const int tr = (wave + NW * p) * 8 + a_lrow;
        a_src[p] = row_ptr<bf16_t>(X, (int64_t)a_row_id[p], ldx) + ((a_chunk ^ swz(tr)) << 3);
    }
    // A load whose 8 tile rows all lie past the tile's last row is left out (a decode batch puts a
    // handful of rows into a 64-row tile; with 4-bit weights the activation tile would otherwise be most
    // of the requests); within a load, lanes past the last row are masked.  The choice is uniform over
    // the wave and counted, so the wait counts stay exact.  LDS rows never loaded feed only accumulator
    // rows that are never stored.
    const int tile_rows = (tc.row_end - tc.row0) < BM ? (tc.row_end - tc.row0) : BM;
    auto issue_a = [&](int kt) {
#pragma unroll
        for (int p = 0; p < A_LPW; ++p) {
            if ((wave + NW * p) * 8 >= tile_rows) continue;
            if ((wave + NW * p) * 8 + a_lrow < tile_rows)
                load_lds<16>(a_src[p] + kt * PBK, ldsb + (kt % NSA) * A_SLOT + (wave + NW * p) * 1024);
            issued += 1;
        }
#pragma unroll
        for (int i = 0; i < NSA; ++i)
            if (i == kt % NSA) last_a[i] = issued;
    };
#pragma unroll
    for (int st = 0; st < NSA - 1; ++st)
        if (st < nk) issue_a(st);

    // ---- LDS offsets of the operand rows this lane feeds to the MFMAs ----
    const int fr = lane & 31, fq = lane >> 5;
    const int fsw = swz(fr);
    const int a_off = fr * A_ROWB;                 // row block i: + i * 32 * A_ROWB
    int b_off[TN], s_row[TN], b_sw[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        int r;
        if (GATED) r = (j < TNO) ? (wn * WNO + j * 32 + fr) : (NO + wn * WNO + (j - TNO) * 32 + fr);
        else r = wn * WNO + j * 32 + fr;
        b_off[j] = r * B_ROWB;          // + the block's slot, which depends on the stage's half
        b_sw[j] = bswz(r);
        s_row[j] = r;
    }
    const bool two_blocks = tile_rows > 32;        // the tile's second 32-row block holds rows

    float16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    for (int g = 0; g < nk; ++g) {
        const int d = g >> 1, half = g & 1;
        // stage g has landed when at most the loads issued after its last one are still in flight
        int need = 0;
#pragma unroll
        for (int i = 0; i < NSA; ++i)
            if (i == g % NSA) need = last_a[i];
#pragma unroll
        for (int i = 0; i < NSB; ++i)
            if (i == d % NSB && last_b[i] > need) need = last_b[i];
        const int sc_chunk = g / SW_STAGES;
        if (wide_scales && last_s[sc_chunk & 1] > need) need = last_s[sc_chunk & 1];
        wait_vmcnt_at_most(issued - need);
        block_barrier();       // every wave's part of stage g is in LDS; every wave is done reading stage g-1
        if (g + NSA - 1 < nk) issue_a(g + NSA - 1);                            // into the slot stage g-1 used
        if (half == 0 && d + NSB - 1 < n_double) issue_b(d + NSB - 1);         // into the slot double stage d-1 used
        if (wide_scales && g % SW_STAGES == 0 && sc_chunk + 1 < n_chunks) issue_s(sc_chunk + 1);   // slot of chunk c-1
        {
            const char* a_base = smem + (g % NSA) * A_SLOT + a_off;
            const char* bs_base = smem + B_BASE + (d % NSB) * B_SLOT;
            // where this stage's two scale bytes of a row sit: in the 16-byte chunk, or in the double stage's
            // dword (a clamped tail dword holds them in its upper half)
            const char* ss_base = wide_scales ? smem + S_BASE + (sc_chunk & 1) * SW_SLOT + (2 * g - chunk_start(sc_chunk))
                                              : smem + S_BASE + (d % NSB) * S_SLOT +
                                                    ((odd_tail && d == n_double - 1 && row_scales >= 4) ? 2 : half * 2);
            const int s_mul = wide_scales ? 4 : 1;     // rows are 16 bytes apart in a chunk, 4 in a dword slot
            bf16x8_t af[TM][4];
            u32x4_t bq[TN];
            float sc[TN];
#pragma unroll
            for (int j4 = 0; j4 < 4; ++j4) {
                af[0][j4] = *reinterpret_cast<const bf16x8_t*>(a_base + (((fq * 4 + j4) ^ fsw) << 4));
                if (two_blocks)
                    af[1][j4] = *reinterpret_cast<const bf16x8_t*>(a_base + 32 * A_ROWB + (((fq * 4 + j4) ^ fsw) << 4));
            }
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                bq[j] = *reinterpret_cast<const u32x4_t*>(bs_base + b_off[j] + (((half * 2 + fq) ^ b_sw[j]) << 4));
                sc[j] = e8m0_to_float(*reinterpret_cast<const uint8_t*>(ss_base + s_row[j] * 4 * s_mul + fq));
            }
#pragma unroll
            for (int j4 = 0; j4 < 4; ++j4)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    // weight rows as the MFMA's row operand: a lane ends up with 4 consecutive output columns
                    const bf16x8_t wv = widen_fp4x8(bq[j][j4], sc[j]);
                    acc[0][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, af[0][j4], acc[0][j], 0, 0, 0);
                    if (two_blocks) acc[1][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, af[1][j4], acc[1][j], 0, 0, 0);
                }
            wait_lds_reads();   // this wave's reads of stage g have returned before it reaches the next barrier
        }
    }

    // accumulator element v of tile (i, j): output row 32 i + fr, column (v/4)*8 + fq*4 + v%4
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        if (i == 1 && !two_blocks) break;
        const int64_t row = (int64_t)tc.row0 + i * 32 + fr;
#pragma unroll
        for (int j = 0; j < TNO; ++j) {
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const int col = n0 + wn * WNO + j * 32 + a * 8 + fq * 4;
                float val[4];
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    if (GATED) val[b] = silu_mul(acc[i][j][a * 4 + b], acc[i][j + TNO][a * 4 + b]);
                    else val[b] = acc[i][j][a * 4 + b];
                }
                if (row < tc.row_end && col < N) {  // N is a multiple of 8: the 4 columns are in or out together
                    if (OUT_F32)
                        *reinterpret_cast<float4*>(static_cast<float*>(Out_) + row * ldo + col) =
                            make_float4(val[0], val[1], val[2], val[3]);
                    else
                        *reinterpret_cast<uint2*>(static_cast<bf16_t*>(Out_) + row * ldo + col) =
                            make_uint2(pack_bf16x2(val[0], val[1]), pack_bf16x2(val[2], val[3]));
                }
            }
        }
    }
}

// ----------------------------------------------------------------------------------------------
// The weight-streaming shape for decode-heavy batches (on average at most 48 rows per expert) and launches of few tiles.
//
// With 4-bit weights a 64-value stage is 32 bytes of a weight row: fetched stage by stage (or two
// stages at a time) every 128-byte line of the weights is requested several times, a few stages
// apart, and a row whose start is not line-aligned (1440-byte rows: every row but one in four)
// straddles lines on top of that.  Measured on 128 experts x 5760 x 2880: 1.5x the weight bytes
// cross the fabric and the kernel stays at 0.37 of the HBM peak.  Here every weight row is fetched
// in whole, ALIGNED 128-byte lines: line L of a row holds the row's bytes [128 L - phase, 128 L -
// phase + 128), phase = (row address) mod 128, a multiple of 32, so a stage's 32 bytes never cross a
// line and stage s of a row of class c = phase / 32 lies in line (c + s) / 4 at 32-byte slot
// (c + s) % 4.  A row keeps two lines in LDS; when it moves on to line L - 1 (top of stage
// 4 (L - 1) - c) the line slot it has just left takes line L, four stages ahead of its first use.
// Rows of different classes turn over at different stages, so in the common case (row bytes an odd
// multiple of 32) a quarter of the rows fetches a line at every stage and the traffic is even.
//
// 32 x 256 tiles, 8 waves, each with its own 32 weight rows: a wave fetches the lines of its own
// rows, so only the activation tile is shared between waves.  The per-stage work of a wave is small
// (4 MFMAs behind 16 conversions) and the stage is a chain of dependent waits, so the kernel lives on
// the number of waves per SIMD (4) and on the length of that chain: every instruction on it costs.
// The load schedule is therefore fixed, with nothing to keep count of.  Stages are taken in pairs, with one block barrier per pair
// (gate_up + down, us, one per stage / per pair: 128 experts, H = 2048, I = 768, 2 rows each 85 / 73, 16 rows 89 / 82; 32 experts,
// 4096 x 2048, 8 rows 95 / 82; 128 experts, 2880 x 2880, 2 rows 293 / 286, 8 rows 338 / 332, 16 rows 361 / 353; only 32 experts of 2880 x 2880 with
// 4 and 8 rows are faster with one per stage, 92 / 94 and 94 / 97, and from 16 rows on they are level).  The top of pair g, g + 1
// issues the activations of stages g + 2 and g + 3 into the slots of the pair before; every stage g issues
// line ((c + g) / 4) + 1 of the rows whose class c has (c + g) % 4 = 0; the start-up issues what stages -3, -2, -1
// would have.  Past a row's end the rule fetches the row's last line once more (into the line slot the row has left for
// good), past the last stage the activation load repeats the last stage into a free slot: harmless and served by the
// caches.  At the top of a pair only the lines of the two stages before may be in flight: loads return in order, the pair's
// activations were issued in front of those, its own lines a pair earlier.  So the wait count is a constant (row bytes an odd multiple
// of 32: one line load per stage) or one of two (else).  The scale bytes
// never touch LDS: a lane needs one byte per stage for its weight row and holds them in registers
// (128 bytes of the row at a time).  For the gated GEMM waves 0-3 hold the gate rows and waves 4-7
// the matching up rows; the up accumulators cross through LDS once, after the last stage.  80 KB of
// LDS, two blocks per compute unit.
// ----------------------------------------------------------------------------------------------
constexpr int kS4Rows = 32, kS4NSA = 4, kS4Waves = 8;

// 16 bytes into registers without a compiler-inserted wait: the value may be used only after an explicit
// wait that covers the load, followed by settle().
__device__ __forceinline__ u32x4_t load_u32x4_async(const uint8_t* p)
{
    u32x4_t v;
    asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(v) : "v"(p) : "memory");
    return v;
}
__device__ __forceinline__ void settle(u32x4_t& v) { asm volatile("" : "+v"(v)::"memory"); }

// ODD: the row bytes are an odd multiple of 32 (the four line loads of a wave have the four classes).
// (second launch bound: waves per SIMD; two blocks of 8 waves per compute unit = 4)
template <bool GATED, bool ODD, bool OUT_F32>
__global__ __launch_bounds__(kS4Waves * 64, 4) void grouped_gemm_w4_stream_kernel(
    RowSrc X, int ldx, const int32_t* __restrict__ row_map, int map_div, uint32_t map_magic,
    const int32_t* __restrict__ offsets, int E,
    const uint8_t* __restrict__ W, const uint8_t* __restrict__ S, int64_t rows_per_expert, int N, int K,
    void* __restrict__ Out_, int ldo, int a_rows)
{
    static_assert(!(GATED && OUT_F32), "the intermediate of the gated GEMM is always bf16");
    constexpr int BM = kS4Rows, BN = kW4BN, NW = kS4Waves, NSA = kS4NSA, PBK = kW4K;
    constexpr int NO = GATED ? BN / 2 : BN;     // output columns per block
    constexpr int A_ROWB = PBK * 2, A_SLOT = BM * A_ROWB;        // 128-byte activation rows, 4 KB per stage
    constexpr int B_SLOT = BN * 128;                             // one 128-byte line of every weight row
    constexpr int B_BASE = NSA * A_SLOT;
    constexpr int B_LPW = BN / 8 / NW;                           // line loads per wave to cover its rows once (8 rows each)
    static_assert(BM == 32 && BN == 32 * NW && B_LPW == 4 && NSA == 4, "tile configuration");

    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const uint32_t ldsb = lds_address(smem);    // LDS byte address of the block's dynamic shared memory

    const int n_tiles = (N + NO - 1) / NO;
    const TileCoord tc = find_tile<BM>(offsets, E, n_tiles, a_rows);
    if (!tc.valid) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);    // wave-uniform: what depends on it stays in scalar registers
    const int n0 = tc.n_tile * NO;
    const int nk = K / PBK;
    const int64_t row_bytes = K / 2, row_scales = K / 32;
    const uint8_t* We = W + (int64_t)tc.expert * rows_per_expert * row_bytes;
    const uint8_t* Se = S + (int64_t)tc.expert * rows_per_expert * row_scales;
    const uint8_t* W_last = W + (int64_t)E * rows_per_expert * row_bytes - 16;     // last 16 bytes of the codes
    const uint8_t* S_end = S + (int64_t)E * rows_per_expert * row_scales;

    // activations: waves 0..3 fetch tile rows wave * 8 .. + 7, lane = (row, 16-byte chunk)
    const int a_lrow = lane >> 3, a_chunk = lane & 7;
    const int tile_rows = tc.row_end - tc.row0;     // 1 .. 32
    const bool a_loader = wave * 8 < tile_rows;     // (false for waves 4..7); a load whose rows all lie past the tile's last row is left out
    int32_t a_row_id, a_own;
    {
        int r = tc.row0 + wave * 8 + a_lrow;
        if (r >= tc.row_end) r = tc.row_end - 1;
        a_own = r;
        // fetched without a compiler-tracked wait: the weight loads below go out while it is in flight, and
        // the explicit wait in front of its first use leaves exactly those outstanding.  The load is issued
        // in every case (without a row map it reads a valid dummy word, offsets[0], and the result is
        // ignored): a conditional load would be an asm output merged with an earlier value, i.e. a register
        // copy that the compiler may place behind the load.
        const int32_t* src = row_map ? row_map + r : offsets;
        asm volatile("global_load_dword %0, %1, off" : "=v"(a_row_id) : "v"(src) : "memory");
    }

    // Tile row t -> row of the expert's weight matrix.  A row past the matrix (ragged last n-tile) is
    // replaced by the last real row with the same index mod 4, which has the same line phase; what it
    // produces is never stored.
    auto weight_row = [&](int t) {
        const bool up = GATED && t >= NO;
        int n = n0 + (up ? t - NO : t);
        if (n >= N) n -= ((n - N) / 4 + 1) * 4;
        return up ? n + N : n;
    };
    // Line loads: load k of this wave covers its 8 rows 32 wave + 4 i + q_k, i = lane / 8: rows 4 apart start
    // a multiple of 128 bytes apart, so they share a class.  When the row bytes are an odd multiple of 32
    // the four residues q have four different classes and q_k is the residue of class k (load k has class
    // k, known at compile time); otherwise q_k = k.  The instruction's 8 lines are LDS rows 8 (4 wave +
    // k) .. + 7; LDS chunk x of a row holds the line's chunk x ^ sw(row), sw chosen so that 16 lanes
    // reading the chunks of their stage (which differ between classes) fall into 16 different bank
    // groups.
    const int rb32 = (int)(row_bytes >> 5) & 3;
    const int c0 = __builtin_amdgcn_readfirstlane(
        (int)((uintptr_t)(We + (int64_t)weight_row(32 * wave) * row_bytes) >> 5) & 3);     // class of residue 0
    auto line_sw = [&](int t) {
        const int i = (t >> 2) & 7, q = t & 3;
        const int xq = ODD ? 0 : (rb32 == 2 ? (q >> 1) : q);
        return ((i >> 1) & 1) | (xq << 1);
    };
    const uint8_t* b_src[B_LPW];       // this lane's 16 bytes of line 0
    int cls[B_LPW], lmax[B_LPW];       // the load's class (wave-uniform; = k when ODD) and its rows' last line
    bool clamp_any = false;            // some address this wave will ask for lies outside W (wave-uniform)
#pragma unroll
    for (int k = 0; k < B_LPW; ++k) {
        const int q = ODD ? ((k - c0) * rb32) & 3 : k;     // rb32 is its own inverse mod 4
        const int t = 32 * wave + 4 * (lane >> 3) + q;
        const uint8_t* row = We + (int64_t)weight_row(t) * row_bytes;
        const int phase = (int)((uintptr_t)row & 127);
        b_src[k] = row - phase + (((lane & 7) ^ line_sw(t)) << 4);
        cls[k] = ODD ? k : __builtin_amdgcn_readfirstlane(phase >> 5);
        lmax[k] = (cls[k] + nk - 1) >> 2;
        // the first line may begin in front of W, the last one may end behind it
        clamp_any = clamp_any || __ballot(b_src[k] < W || b_src[k] + (int64_t)lmax[k] * 128 > W_last) != 0;
    }
    // ODD: the four loads of a lane differ by the same amount in every lane ((q_k - q_0) rows and the
    // difference of the two line phases: the stand-in rows of a ragged tile keep their distance as well),
    // so one address and three scalar offsets do, which frees six registers.
    const uint8_t* b_lane = b_src[0];
    int k_off[B_LPW];
#pragma unroll
    for (int k = 0; k < B_LPW; ++k) k_off[k] = ODD ? __builtin_amdgcn_readfirstlane((int)(b_src[k] - b_src[0])) : 0;
    auto line_addr = [&](int k, int L) {
        return ODD ? b_lane + (k_off[k] + L * 128) : b_src[k] + (int64_t)L * 128;
    };
    // this lane's operand row: tile row 32 wave + fr, k-half fq of every stage
    const int fr = lane & 31, fq = lane >> 5;
    const int t_own = 32 * wave + fr;
    const int wr_own = weight_row(t_own);
    const int k_own = ODD ? (c0 + rb32 * (fr & 3)) & 3 : (fr & 3);     // the load that fetches this row
    const int b_off = ((wave * 4 + k_own) * 8 + (fr >> 2)) * 128;
    const int b_sw = line_sw(t_own);
    const int b_cls = ODD ? k_own : (int)((uintptr_t)(We + (int64_t)wr_own * row_bytes) >> 5) & 3;
    const uint8_t* s_src = Se + (int64_t)wr_own * row_scales;     // both k-halves of a row fetch the same scale bytes
    // A row's scale bytes are fetched 128 at a time (64 stages; the whole row when K <= 4096) as up to 8
    // 16-byte pieces: neighbouring rows then touch the lines they share at the same moment, whereas
    // piecemeal fetches of 16 bytes every 8 stages brought each line in several times.  A lane keeps the 8
    // bytes of a piece that belong to its k-half (byte u of them is the scale of stage 8 piece + u).
    const int s_row_pieces = (int)((row_scales + 15) / 16);     // 16-byte pieces that hold bytes of the row
    int s_over = 0;                    // bytes by which the row's LAST piece would pass the end of S: it is fetched that much earlier
    {
        const int over = (int)(s_src + (int64_t)s_row_pieces * 16 - S_end);
        s_over = over > 0 ? over : 0;
    }
    uint32_t s_lo[8], s_hi[8], s_cur_lo = 0, s_cur_hi = 0;
    auto fetch_piece = [&](int piece) {
        return load_u32x4_async(s_src + piece * 16 - (piece == s_row_pieces - 1 ? s_over : 0));
    };
    auto keep_piece = [&](u32x4_t v, int piece, uint32_t& lo_out, uint32_t& hi_out) {
        settle(v);
        if (piece == s_row_pieces - 1 && s_over > 0) {      // the row's last piece started s_over bytes early
            uint64_t lo = (uint64_t)v[0] | ((uint64_t)v[1] << 32);
            uint64_t hi = (uint64_t)v[2] | ((uint64_t)v[3] << 32);
            const int sh = s_over * 8;
            if (sh >= 64) {
                lo = hi >> (sh - 64);
                hi = 0;
            } else {
                lo = (lo >> sh) | (hi << (64 - sh));
                hi >>= sh;
            }
            v = u32x4_t{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
        }
        const uint32_t sel = fq ? 0x07050301u : 0x06040200u;      // bytes fq, fq + 2, fq + 4, fq + 6 of a dword pair
        lo_out = __builtin_amdgcn_perm(v[1], v[0], sel);
        hi_out = __builtin_amdgcn_perm(v[3], v[2], sel);
    };

    // ---- the fixed load schedule ----
    const bf16_t* a_src = nullptr;
    // activations of stage kt
    auto issue_rows = [&](int kt, int a_slot) {
        if (a_loader) {
            kt = kt < nk ? kt : nk - 1;
            if (wave * 8 + a_lrow < tile_rows)
                load_lds<16>(a_src + kt * PBK, ldsb + a_slot * A_SLOT + wave * 1024);
        }
    };
    // the lines that come due in (pseudo-)stage g, g >= -3
    auto issue_lines = [&](int g) {
#pragma unroll
        for (int k = 0; k < B_LPW; ++k) {
            if (ODD ? ((k + g) & 3) != 0 : ((cls[k] + g) & 3) != 0) continue;
            const int L = ((cls[k] + g) >> 2) + 1;
            // past the row's last line the load repeats that line (it has just been fetched: no memory
            // traffic), still into the slot the rule names, which the row has left for good
            const int Lsrc = L < lmax[k] ? L : lmax[k];
            const uint8_t* a = line_addr(k, Lsrc);
            if (clamp_any) {      // only the wave that holds the last rows of W: a branch, not a select on every load
                asm volatile("");
                a = a > W_last ? W_last : a;
            }
            const uint32_t to = ldsb + B_BASE + (L & 1) * B_SLOT + (wave * B_LPW + k) * 1024;
            // (a stream if no other block reads the row; gate_up + down, us, plain / so: 128 experts, H = I = 2880, 2 rows each 314 / 293,
            // 4 rows 339 / 311, 16 rows 372 / 361; 32 experts, 8 rows 105 / 96; wherever in a line the codes start.  The shapes that
            // fetch half lines lose 5 to 12 % by it and stay plain; so does line 0 of the start-up.)
            if (tc.alone) load_lds<16, true>(a, to);
            else load_lds<16>(a, to);
        }
    };
    // Loads in flight at the top of a pair of stages g, g + 1 that the pair does not need: the lines of stages g - 2 and g - 1
    // (the activations of the pair were issued in front of those).
    int lines_at[4];                   // line loads of a stage = r (mod 4)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        lines_at[r] = 0;
#pragma unroll
        for (int k = 0; k < B_LPW; ++k) lines_at[r] += ((cls[k] + r) & 3) == 0;
    }
    auto wait_for_pair = [&](int r) {     // r = g mod 4, a compile-time constant where it is called
        if (ODD) wait_vmcnt<2>();
        else wait_vmcnt_at_most(lines_at[(r + 2) & 3] + lines_at[(r + 3) & 3]);
    };

    // ---- start-up: scale bytes, line 0 of every row, then what stages -3, -2, -1 would issue ----
    // the first 8 pieces, until the row-map lookup below has returned (a row with fewer pieces fetches its
    // last one again: with conditional loads the compiler treats the eight values as one 32-register tuple
    // and copies it around)
    u32x4_t s_raw[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) s_raw[i] = fetch_piece(i < s_row_pieces ? i : s_row_pieces - 1);
#pragma unroll
    for (int k = 0; k < B_LPW; ++k) {
        const uint8_t* a = line_addr(k, 0);
        if (clamp_any) {
            a = a < W ? W : a;
            a = a > W_last ? W_last : a;
        }
        load_lds<16>(a, ldsb + B_BASE + (wave * B_LPW + k) * 1024);
    }
    {
        // the row-map load and the scale pieces came before the 4 line loads: wait for them, cut the pieces
        // down to this lane's bytes
        wait_vmcnt<B_LPW>();
        asm volatile("" : "+v"(a_row_id)::"memory");
        const uint32_t mapped = mapped_row(a_row_id, a_rows, map_div, map_magic);
        a_row_id = row_map ? (int32_t)mapped : a_own;
#pragma unroll
        for (int i = 0; i < 8; ++i) keep_piece(s_raw[i], i < s_row_pieces ? i : s_row_pieces - 1, s_lo[i], s_hi[i]);
        const int tr = wave * 8 + a_lrow;
        a_src = row_ptr<bf16_t>(X, (int64_t)a_row_id, ldx) + ((a_chunk ^ swz(tr)) << 3);
    }
    issue_lines(-3);
    issue_rows(0, 0);
    issue_rows(1, 1);
    issue_lines(-2);
    issue_lines(-1);

    // activation fragment j4 of this lane's token row: LDS offset inside a stage's slot (the slot's own
    // offset is a constant of the unrolled step and goes into the instruction)
    // (LDS addresses as integers in the LDS address space: the compiler then folds the slot into the
    // instruction's offset field instead of adding the array's base at every read)
    typedef __attribute__((address_space(3))) const bf16x8_t lds_bf16x8_t;
    typedef __attribute__((address_space(3))) const u32x4_t lds_u32x4_t;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr_t*)smem;
    uint32_t a_rd[4];
#pragma unroll
    for (int j4 = 0; j4 < 4; ++j4) a_rd[j4] = lds0 + fr * A_ROWB + (((fq * 4 + j4) ^ swz(fr)) << 4);
    const uint32_t b_rd = lds0 + B_BASE + b_off;
    const uint32_t b_rd_odd = b_rd + ((fq ^ (b_sw & 1)) << 4);
    // token columns past the tile's rows are never stored: their lanes skip the activation reads (with a
    // handful of rows per expert most of the LDS read traffic would be for nothing; reading them anyway
    // measured 3 % slower)
    const bool a_reader = fr < ((tile_rows + 7) & ~7);

    float16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    bf16x8_t af[4];
#pragma unroll
    for (int j4 = 0; j4 < 4; ++j4)
#pragma unroll
        for (int v = 0; v < 8; ++v) af[j4][v] = (__bf16)0.f;

    for (int g0 = 0; g0 < nk; g0 += 8) {
        const int chunk = g0 >> 3;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int g = g0 + u;
            if (g >= nk) break;
            if ((u & 1) == 0) {
                wait_for_pair(u & 3);
                block_barrier();   // every wave's part of stages g and g + 1 is in LDS; every wave is done reading the pair before
            }
            if (u == 0) {          // the scale bytes of stages g0 .. g0 + 7: piece g0 / 8 of the row
                if (chunk > 0 && (chunk & 7) == 0) {
                    // K > 4096: the next 128 scale bytes, two pieces at a time, each pair awaited on the spot
                    // (once per 64 stages; everything issued earlier lands as well, which the fixed wait
                    // counts of the next stages allow for)
#pragma unroll
                    for (int i = 0; i < 8; i += 2) {
                        const int last = s_row_pieces - 1;
                        const int p0 = chunk + i < last ? chunk + i : last;
                        const int p1 = chunk + i + 1 < last ? chunk + i + 1 : last;
                        u32x4_t t0 = fetch_piece(p0), t1 = fetch_piece(p1);
                        wait_vmcnt<0>();
                        keep_piece(t0, p0, s_lo[i], s_hi[i]);
                        keep_piece(t1, p1, s_lo[i + 1], s_hi[i + 1]);
                    }
                }
                switch (chunk & 7) {
                    case 0: s_cur_lo = s_lo[0]; s_cur_hi = s_hi[0]; break;
                    case 1: s_cur_lo = s_lo[1]; s_cur_hi = s_hi[1]; break;
                    case 2: s_cur_lo = s_lo[2]; s_cur_hi = s_hi[2]; break;
                    case 3: s_cur_lo = s_lo[3]; s_cur_hi = s_hi[3]; break;
                    case 4: s_cur_lo = s_lo[4]; s_cur_hi = s_hi[4]; break;
                    case 5: s_cur_lo = s_lo[5]; s_cur_hi = s_hi[5]; break;
                    case 6: s_cur_lo = s_lo[6]; s_cur_hi = s_hi[6]; break;
                    default: s_cur_lo = s_lo[7]; s_cur_hi = s_hi[7]; break;
                }
            }
            // the operand reads go out first (the weight piece before the activation fragments: the conversions
            // start from it), the loads of this stage are issued while they return
            // stage g of this lane's row: 32-byte piece (b_cls + g) % 4 of the line in slot ((b_cls + g) / 4) % 2
            uint32_t b_addr;
            if (ODD) {      // (the swizzle only touches the 16-byte half: folded into b_rd_odd; one multiply puts
                            // the piece at bits 5-6 and the slot at bit 15)
                static_assert(B_SLOT == 1 << 15, "the slot bit");
                b_addr = b_rd_odd + ((((uint32_t)(b_cls + u) & 7u) * 0x2020u) & 0x8060u);
            } else {
                const int tt = b_cls + g;
                const int y = ((tt & 3) << 1) | fq;
                b_addr = b_rd + ((tt >> 2) & 1) * B_SLOT + ((y ^ b_sw) << 4);
            }
            const u32x4_t bq = *(lds_u32x4_t*)(uintptr_t)b_addr;
            if (a_reader) {
#pragma unroll
                for (int j4 = 0; j4 < 4; ++j4)
                    af[j4] = *(lds_bf16x8_t*)(uintptr_t)(a_rd[j4] + (u & 3) * A_SLOT);
            }
            if ((u & 1) == 0) {
                issue_rows(g + 2, (u + 2) & 3);
                issue_rows(g + 3, (u + 3) & 3);
            }
            issue_lines(g);
            const uint32_t s_word = (u & 4) ? s_cur_hi : s_cur_lo;
            const float sc = (u & 3) == 0   ? e8m0_byte_to_float<0>(s_word)
                             : (u & 3) == 1 ? e8m0_byte_to_float<8>(s_word)
                             : (u & 3) == 2 ? e8m0_byte_to_float<16>(s_word)
                                            : e8m0_byte_to_float<24>(s_word);
#pragma unroll
            for (int j4 = 0; j4 < 4; ++j4) {
                // weight rows as the MFMA's row operand: a lane ends up with 4 consecutive output columns
                bf16x8_t wv = widen_fp4x8(bq[j4], sc);
                // This wave's reads of stage g must have returned before the next stage's line takes their slot, or the next
                // barrier hands it to the activations.  The wait
                // hangs on the last widened operand: placed after the loop it would have no data dependence
                // on the conversions and the scheduler would hoist it above them, so that they waited for
                // the activation fragments as well as for the weight piece they need.
                if (j4 == 3) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(wv)::"memory");
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wv, af[j4], acc, 0, 0, 0);
            }
        }
    }
    // The line and activation loads of the last stages are still in flight; nothing reads them, but the
    // accumulator exchange below writes LDS, and a block must not end with loads into LDS outstanding.
    wait_vmcnt<0>();

    // accumulator element v: output row fr, column (v/4)*8 + fq*4 + v%4 of the wave's 32 columns
    if (GATED) {
        // The up waves hand their accumulators to the gate waves through their own weight rows in LDS (no
        // other wave reads those, and every line fetched into them has been used): 4 KB per wave, quad a of
        // lane l at a * 1024 + l * 16.
        char* xch = smem + B_BASE + wave * 4 * 1024;
        if (wave >= 4) {
#pragma unroll
            for (int a = 0; a < 4; ++a)
                *reinterpret_cast<float4*>(xch + a * 1024 + lane * 16) =
                    make_float4(acc[a * 4], acc[a * 4 + 1], acc[a * 4 + 2], acc[a * 4 + 3]);
            wait_lds_reads();
        }
        block_barrier();
        if (wave >= 4) return;
    }
    const int64_t row = (int64_t)tc.row0 + fr;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int col = n0 + (wave & (GATED ? 3 : 7)) * 32 + a * 8 + fq * 4;
        float val[4];
        if (GATED) {
            const float4 up = *reinterpret_cast<const float4*>(smem + B_BASE + (wave + 4) * 4 * 1024 + a * 1024 + lane * 16);
            val[0] = silu_mul(acc[a * 4 + 0], up.x);
            val[1] = silu_mul(acc[a * 4 + 1], up.y);
            val[2] = silu_mul(acc[a * 4 + 2], up.z);
            val[3] = silu_mul(acc[a * 4 + 3], up.w);
        } else {
#pragma unroll
            for (int b = 0; b < 4; ++b) val[b] = acc[a * 4 + b];
        }
        if (row < tc.row_end && col < N) {  // N is a multiple of 8: the 4 columns are in or out together
            if (OUT_F32)
                *reinterpret_cast<float4*>(static_cast<float*>(Out_) + row * ldo + col) =
                    make_float4(val[0], val[1], val[2], val[3]);
            else
                *reinterpret_cast<uint2*>(static_cast<bf16_t*>(Out_) + row * ldo + col) =
                    make_uint2(pack_bf16x2(val[0], val[1]), pack_bf16x2(val[2], val[3]));
        }
    }
}

// ----------------------------------------------------------------------------------------------
// Compute-bound shape: the persistent 256 x 256 kernel of ffn.hip (its tile list, activation path and epilogue) on
// weights that stay packed in LDS and are widened by the wave that multiplies them.
//
// A stage of weights is 8 KB instead of 32, so a wave reads 2 x 16 bytes of codes per stage where it read 8 x 16 bytes
// of bf16, and two conversions per MFMA take the matrix pipe's shadow.  Codes are fetched for two stages at a time (64
// bytes per row; a request per row and stage would be the limit) into a ring of four double stages, one 8 KB piece
// (128 rows) per step, five pieces ahead of the step that loads it: the next tile's first pieces go out in the last
// five steps of a tile.  When a row is an odd number of stages its last double stage is half empty (the lanes behind
// the row's end repeat what is in front of it) and an extra piece is issued between two tiles, so that every tile
// starts with the same lead.  Scale bytes come 16 per row and 8 stages into a ring of three 4 KB slots.
// Within a stage lane (row, q) feeds MX block q (32 k-values) to four successive MFMAs, as in the other two shapes.
// 140 KB of LDS: 2 x 32 activations, 4 x 16 codes, 3 x 4 scales.  Needs K >= 512 (16 scale bytes per row).
// 32 experts, H = I = 2880, top-4, against the 64-row shape, us: 2112 tokens (264 rows per expert) gate_up 375 -> 300,
// down 215 -> 156; 900 tokens 170 -> 136, 116 -> 88.  What bounds it: the matrix pipe at the clock the power limit
// leaves, as in ffn.hip (bf16 weights take 312 and 166 us); the conversions hide under it.
// ----------------------------------------------------------------------------------------------
template <bool GATED, bool OUT_F32, bool MAPPED>
__global__ __launch_bounds__(kBigWaves * 64, 2) void grouped_gemm_w4_big_kernel(
    RowSrc X, int ldx, const int32_t* __restrict__ row_map, int map_div, uint32_t map_magic,
    const int32_t* __restrict__ offsets, int E, const uint8_t* __restrict__ W, const uint8_t* __restrict__ S,
    int64_t rows_per_expert, int N, int K, void* __restrict__ Out_, int ldo, int a_rows)
{
    static_assert(!(GATED && OUT_F32), "the intermediate of the gated GEMM is always bf16");
    constexpr int BM = kBigRows, BN = kBigBN, NW = kBigWaves, WM = 2, WN = NW / WM, PBK = 64;
    constexpr int NO = GATED ? BN / 2 : BN;     // output columns per block
    constexpr int TM = BM / 32 / WM;            // row blocks per wave: rb = wm + WM * i
    constexpr int WNO = NO / WN;                // output columns per wave
    constexpr int TNO = WNO / 32;
    constexpr int TN = GATED ? 2 * TNO : TNO;
    constexpr int ROWB = PBK * 2;               // bytes per activation row and stage
    constexpr int KS = PBK / 16;                // MFMA k-slices per stage
    constexpr uint32_t A_SLOT = BM * ROWB;                       // activation stage
    constexpr uint32_t B_BASE = 2 * A_SLOT, B_SLOT = BN * 64;    // double stage of codes, four of them
    constexpr uint32_t B_PIECE = B_SLOT / 2;
    constexpr uint32_t S_BASE = B_BASE + 4 * B_SLOT, S_SLOT = BN * 16;   // scale bytes of 8 stages, three of them
    constexpr int LEAD = 5;                     // pieces in front of the one a step would need if it waited
    static_assert(TN == 2 && TM == 4 && KS == 4 && NW * TNO * 2048 <= (int)A_SLOT, "tile configuration");
    static_assert(S_BASE + 3 * S_SLOT == kW4BigLds, "LDS layout");

    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const uint32_t lds0 = lds_address(smem);

    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wm = wave / WN, wn = wave % WN;
    const int nk = K / PBK, nd = (nk + 1) / 2;
    const bool odd = (nk & 1) != 0;
    const uint32_t row_bytes = (uint32_t)K / 2, row_scales = (uint32_t)K / 32;

    BigQueue queue;
    int at = queue.init(offsets, E, (N + NO - 1) / NO, a_rows, big_tile_fixed(nk), reinterpret_cast<int*>(smem));
    if (at >= queue.end) return;
    const int stride = (int)gridDim.x / 8;

    BigRows<MAPPED> rows(X, ldx, row_map, map_div, map_magic, a_rows, wave);

    // ---- codes: piece p of a double stage holds tile rows 128 p + 16 wave .. + 15, lane = (row, 16-byte block); LDS
    // block slot c of row r holds block c ^ ((r >> 2) & 3) ----
    const int b_row = wave * 16 + (lane >> 2);
    const uint32_t b_blk = (uint32_t)((lane & 3) ^ ((b_row >> 2) & 3));
    const int b_tail = odd && b_blk >= 2 ? -32 : 0;      // in a half-empty double stage: the block two in front
    const char *b0 = nullptr, *b1 = nullptr;             // next double stage of the rows of piece 0 and of piece 1
    uint32_t b_off0 = 0, b_off1 = 0, b_slot = 0;         // b_slot: where the double stage being loaded goes
    int np = 0;                                          // next piece (2 per double stage) of the tile being loaded
    auto use_weights = [&](const BigTile& t) {
        const int n0 = t.n_tile * NO, last = N - 1 - n0;
        const uint8_t* We = W + (int64_t)t.expert * rows_per_expert * row_bytes;
        b0 = uniform(reinterpret_cast<const char*>(We + (int64_t)n0 * row_bytes));
        b1 = GATED ? uniform(reinterpret_cast<const char*>(We + ((int64_t)N + n0) * row_bytes)) : b0;
        const int r0 = b_row < last ? b_row : last;      // past the matrix: a valid row, result unused
        const int r1 = GATED ? r0 : (BN / 2 + b_row < last ? BN / 2 + b_row : last);
        b_off0 = (uint32_t)r0 * row_bytes + b_blk * 16;
        b_off1 = (uint32_t)r1 * row_bytes + b_blk * 16;
        np = 0;
    };
    auto issue_piece = [&]() {
        const bool second = (np & 1) != 0;
        const uint32_t off = (second ? b_off1 : b_off0) + (uint32_t)((np >> 1) == nd - 1 ? b_tail : 0);
        load_lds_16_base(second ? b1 : b0, off, lds0 + B_BASE + b_slot + (second ? B_PIECE : 0) + wave * 1024);
        np += 1;
        if (second) {
            b0 += 64;
            b1 += 64;
            b_slot = (b_slot + B_SLOT) & (3 * B_SLOT);
        }
    };
    static_assert((B_SLOT & (B_SLOT - 1)) == 0, "the ring of four wraps with a mask");

    // ---- scales: lanes 0 .. 31 of a wave fetch 16 bytes of rows 32 wave + lane ----
    const char* s_base = nullptr;
    uint32_t s_off = 0, s_load = 0;                      // s_load: ring slot of the next chunk to load
    auto use_scales = [&](const BigTile& t) {
        const int n0 = t.n_tile * NO, last = N - 1 - n0;
        s_base = uniform(reinterpret_cast<const char*>(S + (int64_t)t.expert * rows_per_expert * row_scales));
        int r = wave * 32 + (lane & 31);
        const bool up = GATED && r >= NO;
        if (up) r -= NO;
        r = r < last ? r : last;
        s_off = (uint32_t)(n0 + r + (up ? N : 0)) * row_scales;
    };
    auto chunk_start = [&](int c) {      // first scale byte of chunk c within the row: a chunk never runs past the row
        const uint32_t b = (uint32_t)c * 16;
        return b + 16 <= row_scales ? b : row_scales - 16;
    };
    auto issue_scales = [&](int c) {
        if (lane < 32) load_lds_16_base(s_base + chunk_start(c), s_off, lds0 + S_BASE + s_load + wave * 512);
        s_load = s_load == 2 * S_SLOT ? 0u : s_load + S_SLOT;
    };
    // ---- LDS addresses of the operands this lane feeds to the MFMAs ----
    typedef __attribute__((address_space(3))) const bf16x8_t lds_bf16x8_t;
    typedef __attribute__((address_space(3))) const u32x4_t lds_u32x4_t;
    typedef __attribute__((address_space(3))) const uint8_t lds_u8_t;
    const int fr = lane & 31, fq = lane >> 5;
    uint32_t k_lane[KS];                 // activation chunk of slice kk: k-values 32 fq + 8 kk .. + 7 of the stage
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) k_lane[kk] = lds0 + fr * ROWB + (((fq * 4 + kk) ^ swz(fr)) << 4);
    const uint32_t w_lane = lds0 + B_BASE + fr * 64 + ((fq ^ ((fr >> 2) & 3)) << 4);    // the even stage's block; odd: ^ 32
    const uint32_t s_lane = lds0 + S_BASE + fr * 16 + fq;
    const uint32_t a_wave = wm * 32 * ROWB;
    const uint32_t row_of[2] = {(uint32_t)(wn * WNO), (uint32_t)(GATED ? NO + wn * WNO : wn * WNO + 32)};   // first tile row of a fragment

    // ---- first tile ----
    BigTile cur = queue.take(at), nxt = cur;
    uint32_t a_slot = 0, w_slot = 0, s_slot = 0;         // slots of the stage being multiplied
    rows.look_up(cur);
    use_weights(cur);
    use_scales(cur);
    issue_piece();
    issue_piece();
    issue_scales(0);
    wait_vmcnt<3>();                       // the look-ups came first
    rows.use(cur);
    rows.issue(0, lds0);
#pragma unroll 1
    for (int i = 2; i < LEAD; ++i) issue_piece();
    wait_vmcnt<LEAD - 2>();                // (of what the first two stages need: nothing is asked for ahead of it, see ffn.hip)
    block_barrier();

    auto run = [&](auto tmv_const) {
        constexpr int TMV = decltype(tmv_const)::value;
        constexpr int TMA = TMV > 0 ? TMV : 1;
        float16_t acc[TMA][TN];
#pragma unroll
        for (int i = 0; i < TMA; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
        bf16x8_t af[2][TMA], bfr[2][TN];
        u32x4_t codes[TN];
        uint32_t scale[TN];
        auto read_rows = [&](uint32_t as, int kk, int set) {
            if (TMV == 0) return;
            const uint32_t av = k_lane[kk] + (as + a_wave);
#pragma unroll
            for (int i = 0; i < TMV; ++i) af[set][i] = *(lds_bf16x8_t*)(uintptr_t)(av + i * (WM * 32 * ROWB));
        };
        auto read_weights = [&](int stage) {     // a whole stage of this wave's weight rows
            if (TMV == 0) return;
            const uint32_t wv = (w_lane ^ ((stage & 1) * 32u)) + w_slot;
            const uint32_t sv = s_lane + (s_slot + 2u * (uint32_t)stage - chunk_start(stage >> 3));
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                codes[j] = *(lds_u32x4_t*)(uintptr_t)(wv + row_of[j] * 64);
                scale[j] = *(lds_u8_t*)(uintptr_t)(sv + row_of[j] * 16);
            }
        };
        auto widen = [&](int kk, int set) {
            if (TMV == 0) return;
#pragma unroll
            for (int j = 0; j < TN; ++j) bfr[set][j] = widen_fp4x8(codes[j][kk], e8m0_to_float(scale[j]));
        };
        auto mfma_set = [&](int set) {
#pragma unroll
            for (int i = 0; i < TMV; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[set][j], af[set][i], acc[i][j], 0, 0, 0);
        };
        // (as in ffn.hip: the LDS reads of a region one by one between its MFMAs)
        auto interleave = [](int n_ds, int n_mfma) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if (i < n_ds && i < n_mfma) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
                }
            }
        };
        // Step s but its last slice.  `loads`: load instructions this step issues (all of them younger than the next
        // stage's activation loads, so that many may stay in flight).
        auto step_head = [&](auto loads) {
#pragma unroll
            for (int kk = 0; kk < KS - 1; ++kk) {
                read_rows(a_slot, kk + 1, (kk + 1) & 1);
                mfma_set(kk & 1);
                widen(kk + 1, (kk + 1) & 1);
                interleave(TMV, TMV * TN);
            }
            if constexpr (std::is_same<decltype(loads), int>::value) {
                if (loads == 1) wait_vmcnt<1>();
                else wait_vmcnt<2>();
            } else {
                wait_vmcnt<decltype(loads)::value>();
            }
            wait_lds_reads();          // all of this wave's reads of the stage have returned before its slots are refilled
            block_barrier();
        };
        // Behind the barrier: the last slice, under the reads of stage `next` (< 0: the tile ends here).
        auto step_tail = [&](int stage, int next) {
            a_slot ^= A_SLOT;
            if ((stage & 1) != 0 || next < 0) w_slot = (w_slot + B_SLOT) & (3 * B_SLOT);
            if ((stage & 7) == 7 || next < 0) s_slot = s_slot == 2 * S_SLOT ? 0u : s_slot + S_SLOT;
            if (next >= 0) {
                read_weights(next);
                read_rows(a_slot, 0, 0);
            }
            mfma_set((KS - 1) & 1);
            interleave(next >= 0 && TMV > 0 ? TMV + 2 * TN : 0, TMV * TN);
            if (next >= 0) widen(0, 0);
        };

        read_weights(0);
        read_rows(a_slot, 0, 0);
        widen(0, 0);
        for (int s = 0; s < nk - 3; ++s) {
            if (np == 2 * nd) use_weights(nxt);
            const bool more_scales = (s & 7) == 4 && s + 4 < nk;        // chunk s / 8 + 1 exists
            if (more_scales) issue_scales((s >> 3) + 1);
            issue_piece();
            step_head(more_scales ? 2 : 1);
            rows.issue(s + 2, lds0 + a_slot);
            step_tail(s, s + 1);
        }
        // step nk - 3: look-ups and scales of the next tile (its first codes are on their way: the last piece of this tile went
        // out two steps ago or earlier)
        rows.look_up(nxt);
        use_scales(nxt);
        issue_scales(0);
        issue_piece();
        step_head(std::integral_constant<int, 2>{});
        rows.issue(nk - 1, lds0 + a_slot);
        step_tail(nk - 3, nk - 2);
        // step nk - 2
        rows.use(nxt);
        issue_piece();
        step_head(std::integral_constant<int, 1>{});
        rows.issue(0, lds0 + a_slot);
        step_tail(nk - 2, nk - 1);
        // step nk - 1
        issue_piece();
        step_head(std::integral_constant<int, 1>{});
        const uint32_t epi_slot = a_slot;        // every wave has read the last stage: its activation slot is free
        step_tail(nk - 1, -1);
        store_tile<GATED, OUT_F32, false, TMV, TNO, WM>(acc, cur.row0, cur.row_end, wm, cur.n_tile * NO + wn * WNO,
                                                        smem + epi_slot + wave * (TNO * 2048), Out_, ldo, N);
    };

    for (;;) {
        // (the last tile is followed by itself: its first stages are loaded once more and never used)
        rows.issue(1, lds0 + (a_slot ^ A_SLOT));
        at += stride;
        const bool more = at < queue.end;
        if (more) nxt = queue.take(at);
        const int rb_valid = (cur.row_end - cur.row0 + 31) / 32;
        const int tm_valid = (rb_valid - wm + WM - 1) / WM;      // row blocks wm, wm + WM, ... below rb_valid belong to this wave
        if (tm_valid >= 4) run(std::integral_constant<int, 4>{});
        else if (tm_valid >= 3) run(std::integral_constant<int, 3>{});
        else if (tm_valid >= 2) run(std::integral_constant<int, 2>{});
        else if (tm_valid >= 1) run(std::integral_constant<int, 1>{});
        else run(std::integral_constant<int, 0>{});
        if (!more) break;
        cur = nxt;
        if (odd) issue_piece();
        wait_lds_reads();
        block_barrier();       // every wave has read its piece of the epilogue's slot: the next activation loads may overwrite it
    }
    wait_vmcnt<0>();           // a block must not end with loads into LDS outstanding
}

// Which kernel shape a launch uses.  K: length of a weight row.
enum W4Shape { W4_TILE64, W4_STREAM, W4_BIG };
hipError_t w4_shape(int pinned, bool gated, int64_t A, int E, int N, int K, W4Shape* v)
{
    const int cols = gated ? kW4BN / 2 : kW4BN;      // per tile, in all three shapes
    static_assert(kW4BN == kBigBN, "one number of columns");
    const int64_t n_tiles = (N + cols - 1) / cols;
    // (the big tiles read 16 scale bytes of a row at a time and run eight stages ahead; their tile list has a limit)
    const bool big_runs = K >= 512 && big_list_fits(A, E, n_tiles);
    *v = W4_TILE64;
    if (pinned == MOE_FFN_W4_TILE64 || (pinned == MOE_FFN_W4_BIG && !big_runs)) return hipSuccess;
    *v = W4_BIG;
    if (pinned == MOE_FFN_W4_BIG) return hipSuccess;
    // The streaming shape up to 48 rows per expert on average.  Its 32-row tiles re-read (from L2) and re-widen the weights
    // once per 32 rows.  Layer, us, streaming against big tiles (32 experts, H = I = 2880): 32 rows per expert 170 / 185,
    // 41 rows 183 / 186, 50 rows 192 / 189, 64 rows 211 / 210, 77 rows 249 / 220.
    *v = W4_STREAM;
    if (pinned == MOE_FFN_W4_STREAM || A <= (int64_t)48 * E) return hipSuccess;
    int cus = 0;
    const hipError_t e = compute_units(&cus);
    if (e != hipSuccess) return e;
    // Few tiles: a launch that leaves compute units without a block is bound by the chain of one tile, which is shortest
    // with 32 rows and longest with the big tiles' start and end.  Up to one streaming tile per unit (gate_up, us,
    // streaming / 64-row / big): 8 experts, H = I = 1024, 96 rows, 224 tiles expected 18.5 / 19.8 / 23.6, 130 rows, 292 tiles
    // 23.0 / 20.6 / 24.3; H = 2048, I = 768, 130 rows, 219 tiles 26.8 / 31.7 / 35.3.  Rows of up to four stages are level or
    // better with 64 rows (down, 95 rows, 224 tiles: K = 256 13.0 / 12.9; K = 448 13.2 / 15.5).
    if (K >= 320 && tiles_expected(A, E, kS4Rows, n_tiles) <= cus) return hipSuccess;
    // 64-row tiles up to one per unit, unless the experts' rows fit one tile of either shape, and up to two (which share a
    // unit) for rows of up to eleven stages: K = 1024, 8 experts, 200 rows, 232 tiles 21.4 / 24.0 (64-row / big), 400 rows, 432
    // tiles 25.9 / 25.2, 32 experts, 48 rows, 164 tiles 20.6 / 19.1; K = 2048, 130 rows, 324 tiles 41.5 / 36.3; K = 512, 8 experts,
    // 1000 rows, 516 tiles 18.4 / 20.7, 64 experts, 96 rows, 512 tiles 18.0 / 20.8, 130 rows, 648 tiles 26.1 / 21.7; K = 704,
    // 32 experts, 130 rows, 486 tiles 21.4 / 22.7.
    *v = W4_TILE64;
    const int64_t limit = K < 768 ? 2 * cus : A > (int64_t)64 * E ? cus : 0;
    if (!big_runs || tiles_expected(A, E, kW4Rows, n_tiles) <= limit) return hipSuccess;
    *v = W4_BIG;
    return hipSuccess;
}

template <bool GATED, bool OUT_F32, bool MAPPED>
hipError_t launch_w4_big(RowSrc X, int ldx, const int32_t* row_map, int map_div, const int32_t* offsets, int E, int64_t A,
                         const uint8_t* W, const uint8_t* S, int64_t rows_per_expert, int N, int K, void* Out, int ldo,
                         hipStream_t s)
{
    auto kern = grouped_gemm_w4_big_kernel<GATED, OUT_F32, MAPPED>;
    static bool attr_set[kMaxDevices] = {};
    hipError_t e = ensure_lds_limit(kern, kW4BigLds, attr_set);
    if (e != hipSuccess) return e;
    int grid = 0;
    e = big_grid(&grid);
    if (e != hipSuccess) return e;
    kern<<<(unsigned)grid, kBigWaves * 64, kW4BigLds, s>>>(X, ldx, row_map, map_div, map_magic_of(map_div), offsets, E, W, S,
                                                           rows_per_expert, N, K, Out, ldo, (int)A);
    return hipGetLastError();
}

template <bool GATED, bool OUT_F32>
hipError_t launch_w4(int variant, RowSrc X, int ldx, const int32_t* row_map, int map_div, const int32_t* offsets, int E,
                     int64_t A, const uint8_t* W, const uint8_t* S, int64_t rows_per_expert, int N, int K, void* Out,
                     int ldo, hipStream_t s)
{
    constexpr int NO = GATED ? kW4BN / 2 : kW4BN;
    if (!GATED && row_map != nullptr) return hipErrorInvalidValue;      // (only the gate_up GEMM is ever called with a row map)
    // the streaming kernel takes a row's address mod 128 for a multiple of 32 (the callers check it)
    if ((reinterpret_cast<uintptr_t>(W) & 31u) != 0) return hipErrorInvalidValue;
    W4Shape shape;
    hipError_t e = w4_shape(variant, GATED, A, E, N, K, &shape);
    if (e != hipSuccess) return e;
    if (shape == W4_BIG) {
        if (row_map)
            return launch_w4_big<GATED, OUT_F32, GATED>(X, ldx, row_map, map_div, offsets, E, A, W, S, rows_per_expert, N, K, Out, ldo, s);
        return launch_w4_big<GATED, OUT_F32, false>(X, ldx, row_map, map_div, offsets, E, A, W, S, rows_per_expert, N, K, Out, ldo, s);
    }
    const bool stream = shape == W4_STREAM;
    const int tile_rows = stream ? kS4Rows : kW4Rows;
    const size_t lds_bytes = stream ? (size_t)kS4NSA * kS4Rows * kW4K * 2 + (size_t)2 * kW4BN * 128
                                    : (size_t)kW4NSA * kW4Rows * kW4K * 2 + (size_t)kW4NSB * kW4BN * kW4K +
                                          2 * kW4BN * 16;   // scale area: max(3 dword slots, 2 chunk slots)
    const bool odd = ((K / 2) >> 5) & 1;     // row bytes an odd multiple of 32
    auto kern = stream ? (odd ? grouped_gemm_w4_stream_kernel<GATED, true, OUT_F32>
                              : grouped_gemm_w4_stream_kernel<GATED, false, OUT_F32>)
                       : grouped_gemm_w4_kernel<GATED, OUT_F32>;
    static bool attr_set[3][kMaxDevices] = {};
    const int which = stream ? (odd ? 2 : 1) : 0;
    e = ensure_lds_limit(kern, lds_bytes, attr_set[which]);
    if (e != hipSuccess) return e;
    const int64_t n_tiles = (N + NO - 1) / NO;
    const int64_t m_tiles_max = (A + tile_rows - 1) / tile_rows + (A < E ? A : E);
    const int64_t grid = ((m_tiles_max * n_tiles + 7) / 8) * 8;
    if (grid >= ((int64_t)1 << 31)) return hipErrorInvalidValue;   // the device-side tile search counts in 32 bits
    kern<<<(unsigned)grid, (stream ? kS4Waves : kW4Waves) * 64, lds_bytes, s>>>(X, ldx, row_map, map_div, map_magic_of(map_div), offsets, E, W, S,
                                                                                  rows_per_expert, N, K, Out, ldo, (int)A);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_ffn_gate_up_w4(int variant, RowSrc x, const int32_t* row_map, int map_div, const int32_t* offsets,
                                 int64_t A, int E, int H, int I, const uint8_t* w_gate_up, const uint8_t* s_gate_up,
                                 void* act, hipStream_t s)
{
    return launch_w4<true, false>(variant, x, H, row_map, map_div, offsets, E, A, w_gate_up, s_gate_up, (int64_t)2 * I, I,
                                  H, act, I, s);
}

hipError_t launch_ffn_down_w4(int variant, bool out_f32, const void* act, const int32_t* offsets, int64_t A, int E, int H,
                              int I, const uint8_t* w_down, const uint8_t* s_down, void* y_perm, hipStream_t s)
{
    if (out_f32)
        return launch_w4<false, true>(variant, single_src(act), I, nullptr, 1, offsets, E, A, w_down, s_down, (int64_t)H, H,
                                      I, y_perm, H, s);
    return launch_w4<false, false>(variant, single_src(act), I, nullptr, 1, offsets, E, A, w_down, s_down, (int64_t)H, H, I,
                                   y_perm, H, s);
}

const char* ffn_w4_variant_name(int variant, int64_t A, int E, int H, int I)
{
    W4Shape v;
    if (w4_shape(variant, true, A, E, I, H, &v) != hipSuccess) return "";
    switch (v) {
        case W4_STREAM: return "grouped_gemm_w4_stream_kernel<gated>";
        case W4_BIG: return "grouped_gemm_w4_big_kernel<gated>";
        default: return "grouped_gemm_w4_kernel<gated>";
    }
}

}  // namespace moe
