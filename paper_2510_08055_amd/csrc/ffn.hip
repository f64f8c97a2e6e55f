// Grouped expert FFN: per expert, gate_up GEMM with the SwiGLU epilogue fused, then the
// down GEMM (Sec. 2.1: FC layers with a SwiGLU non-linearity; Sec. 2.5: each expert's FC
// runs over the tokens routed to it and is memory-bound below the ridge point, compute-
// bound above it).  bf16 x bf16 -> fp32 on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16).
//
// Both operands are K-contiguous (activations [rows,K], weights [N,K]), which is exactly
// the MFMA operand layout: each lane feeds 8 consecutive k-values of one row.
#include "ffn_big.h"

namespace moe {

constexpr int kBK = 64;        // k-extent of one LDS stage
constexpr int kLdsStride = 72; // bf16 elements per LDS row: 64 + 8 pad -> 144 B, conflict-free 16 B reads

// ----------------------------------------------------------------------------------------------
// LDS-tiled MFMA grouped GEMM.  256 threads = 4 waves arranged 2 (rows) x 2 (columns).
//   Out[r, n] = sum_k X[src(r), k] * W[e, n, k]                       (GATED = false)
//   Out[r, n] = silu(sum_k X.. * W[e, n, k]) * (sum_k X.. * W[e, N + n, k])   (GATED = true)
// GATED stages BN/2 gate rows and the matching BN/2 up rows so that each wave owns both halves
// of its output columns and the SwiGLU product is taken in registers.
// Global -> register -> LDS double buffering: the loads of stage s+1 are in flight while the
// MFMAs of stage s run.
// ----------------------------------------------------------------------------------------------
// SPLIT (the intermediate held as a pair of bf16 values, value = hi + lo): the gated GEMM writes hi to
// column n and lo = bf16(value - hi) to column N + n of its output; the plain GEMM reads such rows
// (K = 2 * ldw k-values) against weight rows of ldw values used twice: 64 values of the hi half, the same 64 of the lo half, the
// next 64 of the hi half, ..., so that a weight stage serves two steps.  (Where ldw is no multiple of 64, which only this kernel
// runs: the hi half, then the lo half.)
template <int BM, int BN, bool GATED, typename OT, bool SPLIT>
__global__ __launch_bounds__(256) void grouped_gemm_bf16_kernel(
    RowSrc X, int ldx, const int32_t* __restrict__ row_map, int map_div,
    const int32_t* __restrict__ offsets, int E, const bf16_t* __restrict__ W, int64_t w_expert_stride, int N, int K,
    OT* __restrict__ Out, int ldo, int a_rows)
{
    const int ldw = (SPLIT && !GATED) ? K / 2 : K;      // k-values per weight row
    constexpr int NO = GATED ? BN / 2 : BN;          // output columns per block
    constexpr int TM = BM / 2 / 32;                  // 32-row MFMA tiles per wave
    constexpr int TNO = NO / 2 / 32;                 // 32-column output tiles per wave
    constexpr int TN = GATED ? 2 * TNO : TNO;        // MFMA column tiles per wave (gate tiles then up tiles)
    constexpr int A_LOADS = BM / 32, B_LOADS = BN / 32;
    constexpr int A_ELEMS = BM * kLdsStride, B_ELEMS = BN * kLdsStride;
    static_assert(TM >= 1 && TNO >= 1, "tile too small for a 2x2 wave grid of 32x32 MFMAs");

    extern __shared__ __attribute__((aligned(16))) bf16_t lds[];
    auto ldsA = [&](int buf) { return lds + buf * (A_ELEMS + B_ELEMS); };
    auto ldsB = [&](int buf) { return lds + buf * (A_ELEMS + B_ELEMS) + A_ELEMS; };

    const int n_tiles = (N + NO - 1) / NO;
    const TileCoord tc = find_tile<BM>(offsets, E, n_tiles, a_rows);
    if (!tc.valid) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // wave-uniform: what depends on it stays in scalar registers
    const int wm = wave >> 1, wn = wave & 1;
    const int n0 = tc.n_tile * NO;
    const bf16_t* We = W + (int64_t)tc.expert * w_expert_stride;

    // global source rows of this thread's 16-byte loads (fixed over the k-loop)
    const int ld_chunk = tid & 7, ld_row = tid >> 3;
    const bf16_t* a_src[A_LOADS];
    const bf16_t* b_src[B_LOADS];
#pragma unroll
    for (int p = 0; p < A_LOADS; ++p) {
        int r = tc.row0 + ld_row + 32 * p;
        if (r >= tc.row_end) r = tc.row_end - 1;            // ragged tail: re-read a valid row, result unused
        // (a row map holds indices below a_rows; the clamp keeps a bad entry from becoming a wild address)
        int id = row_map ? row_map[r] : r;
        id = id < 0 ? 0 : (id < a_rows ? id : a_rows - 1);
        const int64_t src = row_map ? (int64_t)(id / map_div) : (int64_t)r;
        a_src[p] = row_ptr<bf16_t>(X, src, ldx) + ld_chunk * 8;
    }
#pragma unroll
    for (int p = 0; p < B_LOADS; ++p) {
        const int rb = ld_row + 32 * p;
        int n;
        if (GATED) n = (rb < NO) ? (n0 + rb) : (n0 + rb - NO);
        else n = n0 + rb;
        if (n >= N) n = N - 1;
        if (GATED && rb >= NO) n += N;
        b_src[p] = We + (int64_t)n * ldw + ld_chunk * 8;
    }

    float16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    uint4 a_reg[A_LOADS], b_reg[B_LOADS];
    auto load_stage = [&](int k0) {
        const bool in = (k0 + ld_chunk * 8) < K;
        const bool in_pairs = SPLIT && !GATED && ldw % kBK == 0;
        const int ka = in_pairs ? k0 / (2 * kBK) * kBK + (k0 / kBK & 1) * ldw : k0;
#pragma unroll
        for (int p = 0; p < A_LOADS; ++p)
            a_reg[p] = in ? *reinterpret_cast<const uint4*>(a_src[p] + ka) : make_uint4(0, 0, 0, 0);
        // second half of a split k-range: the same weight values again (ldw is a multiple of 8: a 16-byte
        // chunk lies in one half)
        const int kw = in_pairs ? k0 / (2 * kBK) * kBK : (k0 + ld_chunk * 8 >= ldw) ? k0 - ldw : k0;
#pragma unroll
        for (int p = 0; p < B_LOADS; ++p)
            b_reg[p] = in ? *reinterpret_cast<const uint4*>(b_src[p] + kw) : make_uint4(0, 0, 0, 0);
    };
    auto store_stage = [&](int buf) {
#pragma unroll
        for (int p = 0; p < A_LOADS; ++p)
            *reinterpret_cast<uint4*>(ldsA(buf) + (ld_row + 32 * p) * kLdsStride + ld_chunk * 8) = a_reg[p];
#pragma unroll
        for (int p = 0; p < B_LOADS; ++p)
            *reinterpret_cast<uint4*>(ldsB(buf) + (ld_row + 32 * p) * kLdsStride + ld_chunk * 8) = b_reg[p];
    };

    // LDS rows this lane feeds to the MFMAs
    const int fr = lane & 31, fq = lane >> 5;
    int a_row[TM], b_row[TN];
#pragma unroll
    for (int i = 0; i < TM; ++i) a_row[i] = wm * (BM / 2) + i * 32 + fr;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        if (GATED) b_row[j] = (j < TNO) ? (wn * (NO / 2) + j * 32 + fr) : (NO + wn * (NO / 2) + (j - TNO) * 32 + fr);
        else b_row[j] = wn * (NO / 2) + j * 32 + fr;
    }

    const int nk = (K + kBK - 1) / kBK;
    load_stage(0);
    store_stage(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const int buf = kt & 1;
        if (kt + 1 < nk) load_stage((kt + 1) * kBK);
#pragma unroll
        for (int kk = 0; kk < kBK / 16; ++kk) {
            bf16x8_t af[TM], bfr[TN];
#pragma unroll
            for (int i = 0; i < TM; ++i)
                af[i] = *reinterpret_cast<const bf16x8_t*>(ldsA(buf) + a_row[i] * kLdsStride + kk * 16 + fq * 8);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                bfr[j] = *reinterpret_cast<const bf16x8_t*>(ldsB(buf) + b_row[j] * kLdsStride + kk * 16 + fq * 8);
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
        }
        if (kt + 1 < nk) store_stage(buf ^ 1);
        __syncthreads();
    }

    // Epilogue.  Accumulator element v of a 32x32 tile: row (v/4)*8 + (lane/32)*4 + v%4, column lane%32.
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int j = 0; j < TNO; ++j) {
            const int col = n0 + wn * (NO / 2) + j * 32 + fr;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = tc.row0 + wm * (BM / 2) + i * 32 + (v >> 2) * 8 + fq * 4 + (v & 3);
                float val;
                if (GATED) val = silu_mul(acc[i][j][v], acc[i][j + TNO][v]);
                else val = acc[i][j][v];
                if (SPLIT && GATED) val = opaque(val);
                if (row < tc.row_end && col < N) {
                    const OT hi = elem<OT>::from_f32(val);
                    Out[(int64_t)row * ldo + col] = hi;
                    if (SPLIT && GATED) Out[(int64_t)row * ldo + N + col] = elem<OT>::from_f32(val - elem<OT>::to_f32(hi));
                }
            }
        }
    }
}


// Epilogue of a fragment with 16 gate rows and the 16 matching up rows: accumulator elements v and v + 8 of a lane belong to
// output column col + (v / 4) * 8 + v % 4, v < 8, of `row`.  8-byte stores: such a launch has few rows.
template <bool SPLIT>
__device__ __forceinline__ void store_pairs(const float16_t& acc, int row, int row_end, int col, void* Out_, int ldo, int N)
{
    bf16_t* const out = static_cast<bf16_t*>(Out_) + (int64_t)row * ldo + col;
    if (row >= row_end) return;
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        float val[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            val[b] = silu_mul(acc[a * 4 + b], acc[8 + a * 4 + b]);
            if (SPLIT) val[b] = opaque(val[b]);
        }
        if (col + a * 8 >= N) continue;          // N is a multiple of 8: the 4 columns are in or out together
        const uint32_t p01 = pack_bf16x2(val[0], val[1]), p23 = pack_bf16x2(val[2], val[3]);
        *reinterpret_cast<uint2*>(out + a * 8) = make_uint2(p01, p23);
        if (SPLIT)
            *reinterpret_cast<uint2*>(out + N + a * 8) =
                make_uint2(pack_bf16x2(val[0] - __uint_as_float(p01 << 16), val[1] - __uint_as_float(p01 & 0xffff0000u)),
                           pack_bf16x2(val[2] - __uint_as_float(p23 << 16), val[3] - __uint_as_float(p23 & 0xffff0000u)));
    }
}

// ----------------------------------------------------------------------------------------------
// Weight-streaming shape (few rows per expert): global -> LDS copies issued as direct-to-LDS loads
// (global_load_lds_dwordx4: no staging registers, no LDS store instructions) into two rings of NS LDS slots, one for
// the activation rows and one for the weight rows, each stage 64 k-values deep; one barrier per stage.
// 64 x 128 tiles, 4 waves, 3 stages of 24 KB: two blocks share a compute unit.  Launches of few tiles take 32 x 64 tiles (two waves, 5 stages), short rows 256 x 256 (8
// waves, 2 stages): see pick_variant.
// NW waves arranged WM x WN.
// One wave-level load moves 64 lanes x 16 B = 8 whole tile rows into 1 KB of LDS.  LDS rows
// are unpadded (the hardware writes lanes contiguously), so bank conflicts on the 16-byte operand
// reads are avoided by an XOR swizzle applied on the SOURCE side: LDS chunk c of tile row r holds
// global 16-byte chunk c ^ swz(r).
// Row blocks (32 rows) of the m-tile that hold no real row are skipped by every wave.
// The k-order of the MFMAs is the same as in the other variants (bit-identical results).
// Requires K % PBK == 0.
// ----------------------------------------------------------------------------------------------
// OUT_F32: the output is stored as float (the down GEMM of a context that keeps y_perm in fp32).
// SPLIT: the intermediate is a pair of bf16 values, as in the kernel above.
// MAPPED: the rows come through a row map (the fused gather of the gate_up GEMM); without one the look-ups and
// their wait, a round trip to L2 at the start of every tile, are left out altogether.
template <int RBM, int BN, int WM, int NS, int MINW, int NW, bool GATED, bool OUT_F32, bool SPLIT, bool MAPPED>
__global__ __launch_bounds__(NW * 64, MINW) void grouped_gemm_bf16_pipe_kernel(
    RowSrc X, int ldx, const int32_t* __restrict__ row_map, int map_div, uint32_t map_magic,
    const int32_t* __restrict__ offsets, int E, const bf16_t* __restrict__ W, int64_t w_expert_stride, int N, int K,
    void* __restrict__ Out_, int ldo, int a_rows)
{
    static_assert(!(GATED && OUT_F32), "the intermediate of the gated GEMM is always held in the activation dtype");
    constexpr int PBK = 64;                      // k-values per stage
    constexpr int BM = RBM * 32, WN = NW / WM;   // NW waves arranged WM (rows) x WN (columns)
    constexpr int NO = GATED ? BN / 2 : BN;     // output columns per block
    constexpr int TM = RBM / WM;                // row blocks per wave: rb = wm + WM * i
    constexpr int WNO = NO / WN;                // output columns per wave
    constexpr int TNO = WNO < 32 ? 1 : WNO / 32;
    constexpr int TN = GATED && WNO >= 32 ? 2 * TNO : TNO;
    constexpr int ROWB = PBK * 2;                       // bytes per LDS tile row
    constexpr int CPR = PBK / 8;                        // 16-byte chunks per row
    constexpr int RPL = 64 / CPR;                       // tile rows moved by one wave-level load (1 KB)
    constexpr int KS = PBK / 16;                        // MFMA k-slices per stage
    constexpr int A_LPW = BM / RPL / NW, B_LPW = BN / RPL / NW;   // load groups per wave and stage
    constexpr int A_SLOT = BM * ROWB, B_SLOT = BN * ROWB;   // bytes of one stage of either operand
    constexpr int B_BASE = NS * A_SLOT;                 // the weight ring follows the activation ring
    static_assert(RBM % WM == 0 && TM <= 4 && TNO >= 1, "bad tile configuration");
    static_assert(NS >= 2, "a stage is loaded while another is multiplied");
    static_assert(BM % (RPL * NW) == 0 && BN % (RPL * NW) == 0, "tile rows must split evenly over the waves");
    constexpr int AHEAD = NS - 1;                       // stages loaded ahead of the one being multiplied
    // Tiles of 32 rows: where 8 rows or fewer are real, the loads of the others are left out (in a launch of few tiles a wave's
    // own instructions set its pace).
    constexpr bool MAY_BE_SLIM = RBM == 1;
    // A wave with 16 output columns of a gated GEMM has their gate rows and their up rows in one fragment.
    constexpr bool PAIRED = GATED && WNO == 16;

    extern __shared__ __attribute__((aligned(1024))) char smem[];

    const int n_tiles = (N + NO - 1) / NO;
    const TileCoord tc = find_tile<BM>(offsets, E, n_tiles, a_rows);
    if (!tc.valid) return;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // wave-uniform: what depends on it stays in scalar registers
    const int wm = wave / WN, wn = wave % WN;
    const int n0 = tc.n_tile * NO;
    const bf16_t* We = W + (int64_t)tc.expert * w_expert_stride;
    const int rows_here = (tc.row_end - tc.row0) < BM ? (tc.row_end - tc.row0) : BM;
    const int rb_valid = (rows_here + 31) / 32;   // row blocks of this tile with at least one real row

    // ---- source addresses of this lane's loads: group g = wave + NW*p covers tile rows RPL*g .. RPL*g + RPL-1 ----
    // Order matters for the start-up latency: the row-map lookups are issued first, then (without waiting
    // for them) the weight addresses are formed and the weight stages of the prologue are put in flight,
    // and only then are the looked-up rows turned into activation addresses.
    const int l_row = lane / CPR, l_chunk = lane % CPR;
    const int nk_ = K / PBK;
    // with a split intermediate the plain GEMM multiplies every weight stage by hi and by lo values (and loads it for each)
    constexpr bool TWICE = SPLIT && !GATED;
    const int ldw = TWICE ? K / 2 : K;
    // The lookups are loads issued from inline asm, picked up after an explicit wait further down: a
    // lookup through the compiler would be waited for with vmcnt(0) (it does not know of the asm-issued
    // weight loads that follow), i.e. together with the first weight stages out of HBM.  Until that wait
    // the destination registers hold nothing; they are not touched in between.
    int32_t a_own[A_LPW], a_row_id[A_LPW];
#pragma unroll
    for (int p = 0; p < A_LPW; ++p) {
        int r = tc.row0 + (wave + NW * p) * RPL + l_row;
        if (r >= tc.row_end) r = tc.row_end - 1;
        a_own[p] = r;
        a_row_id[p] = 0;
        if (MAPPED) asm volatile("global_load_dword %0, %1, off" : "=v"(a_row_id[p]) : "v"(row_map + r) : "memory");
    }
    const bf16_t* b_src[B_LPW];
#pragma unroll
    for (int p = 0; p < B_LPW; ++p) {
        const int rb = (wave + NW * p) * RPL + l_row;
        int n;
        if (GATED) n = (rb < NO) ? (n0 + rb) : (n0 + rb - NO);
        else n = n0 + rb;
        if (n >= N) n = N - 1;
        if (GATED && rb >= NO) n += N;
        b_src[p] = We + (int64_t)n * ldw + ((l_chunk ^ swz(rb)) << 3);
    }
    const uint32_t lds0 = lds_address(smem);
    // (stream: the weights of this tile are read by this block alone; see load_lds.  The wide shape is for many rows per expert.)
    constexpr bool MAY_STREAM = BM <= 64;
    const bool streamed = MAY_STREAM && tc.alone && whole_lines(W);
    auto issue_b = [&](int kt, int p, auto stream) {
        const int kw = TWICE ? kt >> 1 : kt;
        load_lds_16<decltype(stream)::value>(b_src[p] + kw * PBK, lds0 + B_BASE + (kt % NS) * B_SLOT + (wave + NW * p) * 1024);
    };
    auto issue_first = [&](auto stream) {
#pragma unroll 1
        for (int st = 0; st < AHEAD && st < nk_; ++st)
#pragma unroll
            for (int p = 0; p < B_LPW; ++p) issue_b(st, p, stream);
    };
    if (streamed) issue_first(std::integral_constant<bool, MAY_STREAM>{});
    else issue_first(std::false_type{});
    if (MAPPED) {
        // the lookups came before the weight loads of the prologue: wait for them alone
        if (nk_ >= AHEAD) wait_vmcnt<AHEAD * B_LPW>();
        else wait_vmcnt<0>();
#pragma unroll
        for (int p = 0; p < A_LPW; ++p) {
            asm volatile("" : "+v"(a_row_id[p])::"memory");
            a_row_id[p] = (int32_t)mapped_row(a_row_id[p], a_rows, map_div, map_magic);
        }
    } else {
#pragma unroll
        for (int p = 0; p < A_LPW; ++p) a_row_id[p] = a_own[p];
    }
    const bf16_t* a_src[A_LPW];
#pragma unroll
    for (int p = 0; p < A_LPW; ++p) {
        const int tr = (wave + NW * p) * RPL + l_row;      // row inside the tile
        a_src[p] = row_ptr<bf16_t>(X, (int64_t)a_row_id[p], ldx) + ((l_chunk ^ swz(tr)) << 3);
    }
    // Loads of one stage, cut into KS parts that are issued in the shadow of the MFMAs of the KS
    // k-slices of the stage being multiplied: load q of the step (activation loads first) goes with slice q % KS.
    auto issue_a = [&](int kt, int p) {
        const int ka = TWICE ? (kt >> 1) * PBK + (kt & 1) * ldw : kt * PBK;
        load_lds_16(a_src[p] + ka, lds0 + (kt % NS) * A_SLOT + (wave + NW * p) * 1024);
    };
    auto issue_part = [&](int kt, int part, auto stream, auto a_loads) {
        constexpr int NA = decltype(a_loads)::value;
#pragma unroll
        for (int q = 0; q < NA + B_LPW; ++q) {
            if (q % KS != part) continue;
            if (q < NA) issue_a(kt, q);
            else issue_b(kt, q - NA, stream);
        }
    };
    // ---- LDS byte offsets of the operand rows this lane feeds to the MFMAs ----
    const int fr = lane & 31, fq = lane >> 5;
    const int fsw = swz(fr);     // the swizzle only looks at the low 4 row bits; row blocks are 32 rows
    int a_row[TM], b_row[TN], k_off[KS];
#pragma unroll
    for (int i = 0; i < TM; ++i) a_row[i] = ((wm + WM * i) * 32 + fr) * ROWB;
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        int r;
        if (PAIRED) r = wn * 16 + (fr & 15) + (fr >> 4) * NO;
        else if (GATED) r = (j < TNO) ? (wn * WNO + j * 32 + fr) : (NO + wn * WNO + (j - TNO) * 32 + fr);
        else r = wn * WNO + j * 32 + fr;
        b_row[j] = B_BASE + r * ROWB;
    }
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) k_off[kk] = ((kk * 2 + fq) ^ fsw) << 4;

    // Software pipeline.  Global side: stages g+1 .. g+NS-1 are in flight while stage g is multiplied.  LDS side: the
    // operand fragments of k-slice kk+1 are read while the MFMAs of slice kk run; the last slice of a stage runs after
    // the barrier that hands over the next stage, under the reads of that stage's first slice.
    // The body is instantiated for the number TMV of row blocks this wave really has (0..TM), so the
    // hot loop is straight-line code; a wave with no row block still loads and synchronises.
    // NA: activation loads of a stage.
    auto run = [&](auto tmv_const, auto stream, auto a_loads) {
        constexpr int TMV = decltype(tmv_const)::value, NA = decltype(a_loads)::value;
        constexpr int LPS = NA + B_LPW;             // load instructions per wave and stage
        // In a step the loads of stage g+AHEAD are issued; loads return in issue order, so when stage g+1 is needed the
        // loads that may still be in flight are the ones issued after it.
        constexpr int WAIT_MAIN = (AHEAD - 1) * LPS;
        constexpr int WAIT_FIRST = (AHEAD - 1) * NA;   // prologue: all weight stages, then the activation stages
        // The prologue's loads are not in stage order: while stage g + 1 is one of the prologue's, the loads issued after it
        // are its later activation stages and the steps' own; the fewest, at g = 0, serve all of these steps.  (With up
        // to two stages ahead this is no fewer than WAIT_MAIN.)
        constexpr int WAIT_EARLY = AHEAD > 2 ? (AHEAD - 2) * NA + LPS : WAIT_MAIN;
        static_assert(WAIT_MAIN + LPS < 64 && AHEAD * LPS + NA < 64, "vmcnt is a 6-bit counter");
        constexpr int TMA = TMV > 0 ? TMV : 1;
        float16_t acc[TMA][TN];
#pragma unroll
        for (int i = 0; i < TMA; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
        bf16x8_t af[2][TMA], bfr[2][TN];
        auto read_frags = [&](int g, int kk, int set) {
            if (TMV == 0) return;
            const char* base_a = smem + (g % NS) * A_SLOT;
            const char* base_b = smem + (g % NS) * B_SLOT;
#pragma unroll
            for (int i = 0; i < TMV; ++i)
                af[set][i] = *reinterpret_cast<const bf16x8_t*>(base_a + a_row[i] + k_off[kk]);
#pragma unroll
            for (int j = 0; j < TN; ++j)
                bfr[set][j] = *reinterpret_cast<const bf16x8_t*>(base_b + b_row[j] + k_off[kk]);
        };
        auto mfma_set = [&](int set) {
#pragma unroll
            for (int i = 0; i < TMV; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    // weight rows as the MFMA's row operand, activation rows as its column operand: a lane then
                    // holds 4 consecutive OUTPUT COLUMNS of one output row, which the epilogue stores as 8 bytes
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[set][j], af[set][i], acc[i][j], 0, 0, 0);
        };

        // prologue: the weight stages are already in flight; the activation stages follow, and the first
        // wait lets through only the activation loads issued after stage 0's (so all weight stages of the prologue have landed then)
#pragma unroll 1
        for (int st = 0; st < AHEAD && st < nk_; ++st)
#pragma unroll
            for (int p = 0; p < NA; ++p) issue_a(st, p);
        if (nk_ >= AHEAD) wait_vmcnt<WAIT_FIRST>();
        else wait_vmcnt<0>();
        block_barrier();
        read_frags(0, 0, 0);
        // One k-step.  MORE: stage g+AHEAD exists and is loaded (in parts, between the MFMAs) into the slot stage g-1
        // used, free since the last barrier.  NEXT: stage g+1 exists; it is waited for and handed over by the
        // barrier before the last slice of this stage is multiplied.
        // Ask the scheduler to issue the LDS reads and the global loads of a region one by one between
        // its MFMAs (they then execute in the shadow of the matrix pipe) instead of in a clump.
        auto interleave = [](int n_ds, int n_vmem, int n_mfma) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if (i < n_ds && i < n_mfma) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
                }
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if (i < n_vmem && n_ds + i < n_mfma) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // one global load
                }
            }
        };
        auto parts_in = [](int part) { return (LPS - part + KS - 1) / KS; };
        auto step = [&](int g, auto more_c, auto next_c) {
            constexpr bool MORE = decltype(more_c)::value, NEXT = decltype(next_c)::value;
#pragma unroll
            for (int kk = 0; kk < KS - 1; ++kk) {
                read_frags(g, kk + 1, (kk + 1) & 1);
                if (MORE) issue_part(g + AHEAD, kk, stream, a_loads);
                mfma_set(kk & 1);
                interleave(TMV > 0 ? TMV + TN : 0, MORE ? parts_in(kk) : 0, TMV * TN);
            }
            if (MORE) issue_part(g + AHEAD, KS - 1, stream, a_loads);
            if (NEXT) {
                if (MORE && AHEAD > 2 && g < AHEAD - 1) wait_vmcnt<WAIT_EARLY>();
                else if (MORE) wait_vmcnt<WAIT_MAIN>();
                else wait_vmcnt<0>();        // the pipeline drains: wait for everything
                // all of this wave's reads of stage g have returned before its slots may be refilled
                wait_lds_reads();
                block_barrier();
                read_frags(g + 1, 0, 0);
            }
            mfma_set((KS - 1) & 1);
            interleave(NEXT && TMV > 0 ? TMV + TN : 0, 0, TMV * TN);
        };
        using T = std::true_type;
        using F = std::false_type;
        const int n_main = nk_ > AHEAD ? nk_ - AHEAD : 0;   // steps that still start loads
        int g = 0;
        for (; g < n_main; ++g) step(g, T{}, T{});
        for (; g < nk_ - 1; ++g) step(g, F{}, T{});
        step(g, F{}, F{});

        if constexpr (PAIRED) {
            store_pairs<SPLIT>(acc[0][0], tc.row0 + fr, tc.row_end, n0 + wn * 16 + fq * 4, Out_, ldo, N);
            return;
        }
        // The epilogue's LDS is an activation slot no stage occupies any more: stage nk-1, the last one, sits in slot
        // (nk-1) % NS, and the readers of the other slots passed their barrier long ago.
        constexpr int REG = OUT_F32 ? 4096 : TNO * 2048;           // bytes per wave
        constexpr int WPS = A_SLOT / REG;         // waves per free activation slot
        static_assert(WPS >= 1 && (NS - 1) * WPS >= NW, "the epilogue staging does not fit the free slots");
        store_tile<GATED, OUT_F32, SPLIT, TMV, TNO, WM>(acc, tc.row0, tc.row_end, wm, n0 + wn * WNO,
                                                        smem + ((nk_ + wave / WPS) % NS) * A_SLOT + (wave % WPS) * REG, Out_, ldo, N);
    };

    // row blocks wm, wm + WM, ... below rb_valid belong to this wave
    const int tm_valid = (rb_valid - wm + WM - 1) / WM;
    auto run_rows = [&](auto stream) {
        using std::integral_constant;
        const integral_constant<int, A_LPW> all;
        if constexpr (MAY_BE_SLIM)
            if (rows_here <= 8) {
                if (wave == 0) return run(integral_constant<int, 1>{}, stream, integral_constant<int, 1>{});
                return run(integral_constant<int, 1>{}, stream, integral_constant<int, 0>{});
            }
        if (TM >= 4 && tm_valid >= 4) run(integral_constant<int, (TM >= 4 ? 4 : 0)>{}, stream, all);
        else if (TM >= 3 && tm_valid >= 3) run(integral_constant<int, (TM >= 3 ? 3 : 0)>{}, stream, all);
        else if (TM >= 2 && tm_valid >= 2) run(integral_constant<int, (TM >= 2 ? 2 : 0)>{}, stream, all);
        else if (tm_valid >= 1) run(integral_constant<int, 1>{}, stream, all);
        else run(integral_constant<int, 0>{}, stream, all);
    };
    if (streamed) run_rows(std::integral_constant<bool, MAY_STREAM>{});
    else run_rows(std::false_type{});
}

// ----------------------------------------------------------------------------------------------
// Compute-bound shape: 256 x 256 tiles, 8 waves (2 per SIMD, 128 rows x 64 weight rows each), one persistent block
// per compute unit.
//
// Per k-step of 64 values a block multiplies one stage of activation rows (ring of 2 LDS slots) by one stage of
// weight rows (ring of 3: the weights are what comes from HBM); the two rings are all 160 KB of LDS.  Steps of one
// tile and of the next one follow each other without a gap:
//   - in step s the weight loads of stage s + 2 are issued between the MFMAs, and behind the barrier that ends
//     step s the activation loads of stage s + 2 go into the slot stage s has just left; past the tile's last stage
//     these are the first stages of the block's NEXT tile;
//   - the epilogue works in the weight slot of the tile's last stage, which nobody needs until the next tile's first
//     step;
//   - the row ids of the next tile are looked up while the current tile is multiplied.
// A block that started anew for every tile spent 7 us of each tile outside the k-loop (timestamps written by the kernel:
// tile search 1.8, first loads 2.6, epilogue 2.2, 1-3 until the next block ran) against k-loops of 17 us (K = 768) and 53
// us (K = 2048); now it is 3 us.  Before and after, us (same box, in turn): 66560 rows, 128 experts, H = 2048, I = 768: gate_up 405 -> 384, down
// 245 -> 225; 8448 rows, 32 experts, H = I = 2880: 336 -> 317, 197 -> 170; 8256 rows, 8 skewed experts, H = 4096,
// I = 14336: 1718 -> 1630, 1007 -> 911.  What bounds it, by the counters of whole launches: at 66560 rows the
// matrix pipes are busy 62 % of the gate_up and 47 % of the down GEMM (70 and 72 % of the skewed layer's), at the clock that
// the power limit leaves, with waves waiting 30 and 35 % of their cycles; at 132 rows per expert (16896 rows) they are busy
// 28 and 24 %, and 919 and 516 MB cross the fabric at 4.5 and 5.0 TB/s.
//
// Which tiles: experts are cut into m-tiles of at most `h` 32-row blocks, tiles are ordered by expert, n-tile, m-tile
// (the m-tiles that share a weight tile run side by side on one XCD and share its L2), the list is cut into eight
// pieces, one per XCD, and the blocks of an XCD walk its piece with a common stride.  A tile
// costs a fixed part (big_tile_fixed) plus its row blocks.  `h` is the height,
// 4 to 8, for which the rounds of tiles over the chip cost least; equal tiles are worth a few more of them, because
// the blocks' shares are not evened out at run time.
// ----------------------------------------------------------------------------------------------
template <bool GATED, bool OUT_F32, bool SPLIT, bool MAPPED>
__global__ __launch_bounds__(kBigWaves * 64, 2) void grouped_gemm_bf16_big_kernel(
    RowSrc X, int ldx, const int32_t* __restrict__ row_map, int map_div, uint32_t map_magic,
    const int32_t* __restrict__ offsets, int E, const bf16_t* __restrict__ W, int64_t w_expert_stride, int N, int K,
    void* __restrict__ Out_, int ldo, int a_rows)
{
    static_assert(!(GATED && OUT_F32), "the intermediate of the gated GEMM is always held in the activation dtype");
    constexpr int BM = kBigRows, BN = kBigBN, NW = kBigWaves, WM = 2, WN = NW / WM, PBK = 64;
    constexpr int NO = GATED ? BN / 2 : BN;     // output columns per block
    constexpr int TM = BM / 32 / WM;            // row blocks per wave: rb = wm + WM * i
    constexpr int WNO = NO / WN;                // output columns per wave
    constexpr int TNO = WNO / 32;
    constexpr int TN = GATED ? 2 * TNO : TNO;
    constexpr int ROWB = PBK * 2;               // bytes per LDS tile row
    constexpr int KS = PBK / 16;                // MFMA k-slices per stage
    constexpr int LPW = BM / 8 / NW;            // load instructions per wave, stage and operand (8 rows of 128 bytes each)
    constexpr uint32_t SLOT = BM * ROWB;        // bytes of one stage of either operand
    constexpr uint32_t B_BASE = 2 * SLOT;       // the weight ring (3 slots) follows the activation ring (2 slots)
    static_assert(BM == BN && LPW == 4 && TM == 4 && KS == 4 && NW * TNO * 2048 <= (int)SLOT, "tile configuration");

    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const uint32_t lds0 = lds_address(smem);

    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wm = wave / WN, wn = wave % WN;
    const int nk = K / PBK;
    // with a split intermediate the plain GEMM multiplies every weight stage by hi and by lo values, one step after the other
    constexpr bool TWICE = SPLIT && !GATED;
    const int ldw = TWICE ? K / 2 : K;
    auto a_byte = [&](int stage) { return (uint32_t)(TWICE ? (stage >> 1) * ROWB + (stage & 1) * ldw * 2 : stage * ROWB); };

    BigQueue queue;
    int at = queue.init(offsets, E, (N + NO - 1) / NO, a_rows, big_tile_fixed(nk), reinterpret_cast<int*>(smem));
    if (at >= queue.end) return;
    const int stride = (int)gridDim.x / 8;

    // Load p of this wave covers weight rows (wave + 8 p) * 8 .. + 7 of the tile, as on the activation side (BigRows).
    const int l_row = lane >> 3;
    const uint32_t l_chunk = (uint32_t)((lane & 7) ^ swz(wave * 8 + l_row)) * 16;

    BigRows<MAPPED> rows(X, ldx, row_map, map_div, map_magic, a_rows, wave);

    // ---- weight rows: a uniform base per half of the tile, small lane offsets ----
    const char *b_gate = nullptr, *b_up = nullptr;      // next weight stage to load: rows n0 .. and, gated, N + n0 ..
    uint32_t b_off[LPW];
    auto use_weights = [&](const BigTile& t) {
        const int n0 = t.n_tile * NO;
        const bf16_t* We = W + (int64_t)t.expert * w_expert_stride;
        b_gate = uniform(reinterpret_cast<const char*>(We + (int64_t)n0 * ldw));
        b_up = uniform(reinterpret_cast<const char*>(We + ((int64_t)N + n0) * ldw));
#pragma unroll
        for (int p = 0; p < LPW; ++p) {
            int r = (wave + NW * p) * 8 + l_row;
            if (GATED && r >= NO) r -= NO;
            if (n0 + r >= N) r = N - 1 - n0;            // past the matrix: a valid row, result unused
            b_off[p] = (uint32_t)r * (uint32_t)ldw * 2u + l_chunk;
        }
    };
    // The block's walk over its tiles.  STREAM: of weights that no other block reads (see load_lds): whether they are is a
    // matter of the whole launch, because the policy is part of the load instruction.
    auto walk = [&](auto stream) {
        constexpr bool STREAM = decltype(stream)::value;
        auto issue_b = [&](int p, uint32_t slot) {
            load_lds_16_base<STREAM>(GATED && p >= LPW / 2 ? b_up : b_gate, b_off[p], lds0 + B_BASE + slot + (wave + NW * p) * 1024);
        };
        auto advance_b = [&]() {      // after the loads of a weight stage
            b_gate += ROWB;
            if (GATED) b_up += ROWB;
        };
        auto next_b_slot = [](uint32_t s) { return s == 2 * SLOT ? 0u : s + SLOT; };

        // ---- LDS addresses of the operand rows this lane feeds to the MFMAs ----
        // k-slice kk of tile row r sits at r * 128 + ((2 kk + fq) ^ swz(r)) * 16; the row blocks of a wave are constants
        // apart and go into the read instructions.  (Addresses are integers in the LDS address space: the compiler then
        // folds those constants instead of adding the array's base at every read.)
        typedef __attribute__((address_space(3))) const bf16x8_t lds_bf16x8_t;
        const int fr = lane & 31, fq = lane >> 5;
        uint32_t k_lane[KS];
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) k_lane[kk] = lds0 + fr * ROWB + (((kk * 2 + fq) ^ swz(fr)) << 4);
        const uint32_t a_wave = wm * 32 * ROWB, b_wave = B_BASE + wn * WNO * ROWB;

        // ---- first tile: its first weight stage, first activation stage and second weight stage, in this order: all units start at
        // once and wait for what they have asked memory for, so nothing is asked for ahead of what is multiplied first ----
        BigTile cur = queue.take(at), nxt = cur;
        uint32_t a_slot = 0, b_slot = 0;       // slots of the stage being multiplied
        rows.look_up(cur);
        use_weights(cur);
#pragma unroll
        for (int p = 0; p < LPW; ++p) issue_b(p, 0);
        advance_b();
        wait_vmcnt<LPW>();                     // the look-ups came before the weight loads
        rows.use(cur);
        rows.issue_at(a_byte(0), lds0);
#pragma unroll
        for (int p = 0; p < LPW; ++p) issue_b(p, SLOT);
        advance_b();
        wait_vmcnt<LPW>();
        block_barrier();
        rows.issue_at(a_byte(1), lds0 + SLOT);

        // One tile.  On entry stage 0 of both operands is in LDS for every wave, weight stage 1 is in flight and the
        // activation loads of stage 1 have been issued.  The body is instantiated for the number TMV of row blocks this
        // wave really has (0..TM), so the hot loop is straight-line code; a wave with no row block still loads and
        // synchronises.
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
            auto read_frags = [&](uint32_t as, uint32_t bs, int kk, int set) {
                if (TMV == 0) return;
                const uint32_t av = k_lane[kk] + (as + a_wave), bv = k_lane[kk] + (bs + b_wave);
#pragma unroll
                for (int i = 0; i < TMV; ++i) af[set][i] = *(lds_bf16x8_t*)(uintptr_t)(av + i * (WM * 32 * ROWB));
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    bfr[set][j] = *(lds_bf16x8_t*)(uintptr_t)(bv + (j < TNO ? j * 32 : NO + (j - TNO) * 32) * ROWB);
            };
            auto mfma_set = [&](int set) {
#pragma unroll
                for (int i = 0; i < TMV; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        // weight rows as the MFMA's row operand, activation rows as its column operand: a lane then
                        // holds 4 consecutive OUTPUT COLUMNS of one output row
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[set][j], af[set][i], acc[i][j], 0, 0, 0);
            };
            // Ask the scheduler to issue the LDS reads and the global loads of a region one by one between its MFMAs
            // (they then execute in the shadow of the matrix pipe) instead of in a clump.
            auto interleave = [](int n_ds, int n_vmem, int n_mfma) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    if (i < n_ds && i < n_mfma) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
                    }
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    if (i < n_vmem && n_ds + i < n_mfma) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // one MFMA
                        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // one global load
                    }
                }
            };
            // The k-slices of step s but the last, with the weight loads of the stage two steps on; then the wait for
            // the next stage and the barrier that hands it over.  On return the last slice's operands are in registers.
            uint32_t b_ahead = next_b_slot(next_b_slot(b_slot));     // slot of the weight stage two steps on
            auto step_head = [&]() {
#pragma unroll
                for (int kk = 0; kk < KS - 1; ++kk) {
                    read_frags(a_slot, b_slot, kk + 1, (kk + 1) & 1);
                    issue_b(kk, b_ahead);
                    mfma_set(kk & 1);
                    interleave(TMV > 0 ? TMV + TN : 0, 1, TMV * TN);
                }
                issue_b(KS - 1, b_ahead);
                advance_b();
                // Loads return in issue order.  Everything of the next stage was issued before this step's four weight
                // loads (its activation loads behind the barrier that began this step), so those four may stay.
                wait_vmcnt<LPW>();
                wait_lds_reads();          // all of this wave's reads of the stage have returned before its slots are refilled
                block_barrier();
            };
            auto step_tail = [&](bool read_next) {
                const uint32_t a_next = a_slot ^ SLOT, b_next = next_b_slot(b_slot);
                if (read_next) read_frags(a_next, b_next, 0, 0);
                mfma_set((KS - 1) & 1);
                interleave(read_next && TMV > 0 ? TMV + TN : 0, 0, TMV * TN);
                a_slot = a_next;
                b_ahead = b_slot;
                b_slot = b_next;
            };

            read_frags(a_slot, b_slot, 0, 0);
            if constexpr (TWICE) {
                // Two steps to a weight stage: step s loads half s & 1 (two of the four loads) of the weight stage two on, which is
                // needed three or four steps later; the last four steps load the next tile's first two.  A step fetches half as much
                // of the weights as when they were walked once for all hi and then for all lo values (whose second walk came from
                // memory again).  8 experts, H = 4096, I = 14336, layer, us, before / now: 16 tokens 583 / 509, 160 tokens 632 / 586, 400
                // tokens 846 / 735, 1000 tokens 1066 / 1021, 4128 tokens of skewed routing 3477 / 3396; relative error of the GEMMs against 64 bits
                // 2.57e-6 / 2.53e-6 (I = 4096), 2.81e-6 / 2.69e-6 (14336).
                auto step = [&](int s, auto last_c) {
                    constexpr bool LAST = decltype(last_c)::value;
                    const bool second = (s & 1) != 0;
                    const uint32_t a_next = a_slot ^ SLOT, b_next = second ? next_b_slot(b_slot) : b_slot;
#pragma unroll
                    for (int kk = 0; kk < KS - 1; ++kk) {
                        read_frags(a_slot, b_slot, kk + 1, (kk + 1) & 1);
                        if (kk < 2)
                            load_lds_16_base<STREAM>(b_gate, second ? b_off[kk + 2] : b_off[kk],
                                                     lds0 + B_BASE + b_ahead + (wave + NW * (second ? kk + 2 : kk)) * 1024);
                        mfma_set(kk & 1);
                        interleave(TMV > 0 ? TMV + TN : 0, kk < 2 ? 1 : 0, TMV * TN);
                    }
                    if (second) advance_b();
                    wait_vmcnt<2>();           // (the step's own; everything of the next step was issued before them)
                    wait_lds_reads();
                    block_barrier();
                    rows.issue_at(a_byte(s + 2 < nk ? s + 2 : s + 2 - nk), lds0 + a_slot);
                    if (!LAST) read_frags(a_next, b_next, 0, 0);
                    mfma_set((KS - 1) & 1);
                    interleave(!LAST && TMV > 0 ? TMV + TN : 0, 0, TMV * TN);
                    a_slot = a_next;
                    if (second) b_ahead = b_slot;
                    b_slot = b_next;
                };
                for (int s = 0; s < nk - 1; ++s) {
                    if (s == nk - 4) use_weights(nxt);
                    if (s == nk - 2) rows.use(nxt);
                    step(s, std::false_type{});
                }
                const uint32_t epi_slot = B_BASE + b_slot;
                step(nk - 1, std::true_type{});
                store_tile<GATED, OUT_F32, SPLIT, TMV, TNO, WM>(acc, cur.row0, cur.row_end, wm, cur.n_tile * NO + wn * WNO,
                                                                smem + epi_slot + wave * (TNO * 2048), Out_, ldo, N);
                return;
            }
            for (int s = 0; s < nk - 3; ++s) {
                step_head();
                rows.issue(s + 2, lds0 + a_slot);
                step_tail(true);
            }
            // step nk - 3: the next tile's rows are looked up.  (Not earlier: the registers the look-ups land on must not
            // be copied before they have landed, and the shorter they live the less reason the compiler has to; the
            // build checks the listing.)
            rows.look_up(nxt);
            step_head();
            rows.issue(nk - 1, lds0 + a_slot);
            step_tail(true);
            // step nk - 2: from here on the loads are those of the next tile
            use_weights(nxt);
            rows.use(nxt);
            step_head();
            rows.issue(0, lds0 + a_slot);
            step_tail(true);
            // step nk - 1
            step_head();
            // every wave has read the last stage: its activation slot takes stage 1 of the next tile, its weight slot
            // (free until the next tile's first step) is where the epilogue works
            rows.issue(1, lds0 + a_slot);
            const uint32_t epi_slot = B_BASE + b_slot;
            step_tail(false);

            store_tile<GATED, OUT_F32, SPLIT, TMV, TNO, WM>(acc, cur.row0, cur.row_end, wm, cur.n_tile * NO + wn * WNO,
                                                            smem + epi_slot + wave * (TNO * 2048), Out_, ldo, N);
        };

        for (;;) {
            // (the last tile is followed by itself: its first stages are loaded once more and never used)
            at += stride;
            const bool more = at < queue.end;
            if (more) nxt = queue.take(at);
            const int rb_valid = (cur.row_end - cur.row0 + 31) / 32;
            // row blocks wm, wm + WM, ... below rb_valid belong to this wave
            const int tm_valid = (rb_valid - wm + WM - 1) / WM;
            if (tm_valid >= 4) run(std::integral_constant<int, 4>{});
            else if (tm_valid >= 3) run(std::integral_constant<int, 3>{});
            else if (tm_valid >= 2) run(std::integral_constant<int, 2>{});
            else if (tm_valid >= 1) run(std::integral_constant<int, 1>{});
            else run(std::integral_constant<int, 0>{});
            if (!more) break;
            cur = nxt;
            wait_lds_reads();
            block_barrier();       // every wave has read its piece of the epilogue's slot: the next weight loads may overwrite it
        }
        wait_vmcnt<0>();           // a block must not end with loads into LDS outstanding
    };
    if (queue.mostly_alone && whole_lines(W)) walk(std::true_type{});
    else walk(std::false_type{});
}

// ----------------------------------------------------------------------------------------------
// fp32 path: v_mfma_f32_16x16x4_f32 (fp32 products, fp32 accumulation) on operands that go straight from
// global memory into registers.
//
// What bounds it: these layers are small (a few dozen rows per expert, k-extents of a few hundred), so a launch
// is a handful of memory latencies long, whatever the arithmetic; the tile is therefore small (32 rows x 16
// output columns), which gives hundreds of blocks at 128 rows, and the four waves of a block split the k-range
// (wave w takes the 16-wide chunks w, w + 4, ...), which cuts the chain of loads and MFMAs to a quarter.  Their
// partial tiles are added in wave order through LDS: the summation order of an output depends on K alone, never
// on the batch.  Lane (r, q) = (lane % 16, lane / 16) fetches 16 bytes, k-values [16 c + 4 q, + 4) of row r, for
// four successive MFMAs; the operands of the next chunk are in flight while a chunk is multiplied.
// 64 tokens, H = 256, E = 8, top-2, I = 512, against one thread per output element (uncoalesced weight reads):
// gate_up 82.9 -> 9.5 us, down 74.8 -> 9.6 us (events around the launch); 128 tokens, H = 512, E = 16, top-4, I = 768:
// 1495 -> 31 us and 829 -> 19 us.
// ----------------------------------------------------------------------------------------------
typedef float f32x4_t __attribute__((ext_vector_type(4)));
constexpr int kF32Rows = 32, kF32Cols = 16, kF32Chunk = 16;

template <bool GATED>
__global__ __launch_bounds__(256) void grouped_gemm_f32_kernel(RowSrc X, int ldx,
                                                               const int32_t* __restrict__ row_map, int map_div,
                                                               const int32_t* __restrict__ offsets, int E,
                                                               const float* __restrict__ W, int64_t w_expert_stride,
                                                               int N, int K, float* __restrict__ Out, int ldo, int a_rows)
{
    constexpr int RB = kF32Rows / 16, CB = GATED ? 2 : 1;        // 16-row blocks; weight-row blocks (gate, up)
    __shared__ f32x4_t part[3][RB][CB][64];                      // partial tiles of waves 1..3
    const TileCoord tc = find_tile<kF32Rows>(offsets, E, (N + kF32Cols - 1) / kF32Cols, a_rows);
    if (!tc.valid) return;
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r = lane & 15, q = lane >> 4;
    const int n0 = tc.n_tile * kF32Cols;

    const float *xp[RB], *wp[CB];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        int row = tc.row0 + i * 16 + r;
        if (row >= tc.row_end) row = tc.row_end - 1;             // ragged tail: re-read a valid row, result unused
        int id = row_map ? row_map[row] : row;
        id = id < 0 ? 0 : (id < a_rows ? id : a_rows - 1);       // a bad map entry must not become a wild address
        xp[i] = row_ptr<float>(X, row_map ? (int64_t)(id / map_div) : (int64_t)row, ldx) + q * 4;
    }
#pragma unroll
    for (int j = 0; j < CB; ++j) {
        int n = n0 + r;
        if (n >= N) n = N - 1;
        wp[j] = W + (int64_t)tc.expert * w_expert_stride + ((int64_t)j * N + n) * K + q * 4;
    }

    f32x4_t acc[RB][CB];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
        for (int j = 0; j < CB; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    struct Operands {
        f32x4_t x[RB], w[CB];
    };
    auto fetch = [&](int c) {        // K is a multiple of 8: a lane's 16 bytes lie inside the row or behind its end
        Operands o;
        const bool in = c * kF32Chunk + q * 4 < K;
#pragma unroll
        for (int i = 0; i < RB; ++i)
            o.x[i] = in ? *reinterpret_cast<const f32x4_t*>(xp[i] + c * kF32Chunk) : f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < CB; ++j)
            o.w[j] = in ? *reinterpret_cast<const f32x4_t*>(wp[j] + c * kF32Chunk) : f32x4_t{0.f, 0.f, 0.f, 0.f};
        return o;
    };
    const int n_chunks = (K + kF32Chunk - 1) / kF32Chunk;
    if (wave < n_chunks) {
        Operands cur = fetch(wave);
        for (int c = wave; c < n_chunks; c += 4) {
            const int ahead = c + 4 < n_chunks ? c + 4 : c;      // (the last chunk is fetched twice rather than tested for)
            const Operands nxt = fetch(ahead);
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int i = 0; i < RB; ++i)
#pragma unroll
                    for (int j = 0; j < CB; ++j)
                        // weight rows as the row operand: a lane ends up with 4 consecutive output columns of one row
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(cur.w[j][v], cur.x[i][v], acc[i][j], 0, 0, 0);
            cur = nxt;
        }
    }
    if (wave > 0) {
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
            for (int j = 0; j < CB; ++j) part[wave - 1][i][j][lane] = acc[i][j];
    }
    __syncthreads();
    if (wave != 0) return;
    // accumulator element v of block (i, j): row i * 16 + r, column 4 q + v
    const int col = n0 + q * 4;
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        f32x4_t sum[CB];
#pragma unroll
        for (int j = 0; j < CB; ++j)
            sum[j] = ((acc[i][j] + part[0][i][j][lane]) + part[1][i][j][lane]) + part[2][i][j][lane];
        f32x4_t o = sum[0];
        if (GATED) {
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = sum[0][v] / (1.0f + expf(-sum[0][v])) * sum[CB - 1][v];
        }
        const int row = tc.row0 + i * 16 + r;
        if (row < tc.row_end && col < N)      // N is a multiple of 8: the 4 columns are in or out together
            *reinterpret_cast<f32x4_t*>(Out + (int64_t)row * ldo + col) = o;
    }
}

template <bool GATED>
static hipError_t launch_f32(RowSrc X, int ldx, const int32_t* row_map, int map_div, const int32_t* offsets, int E,
                             int64_t A, const float* W, int64_t w_expert_stride, int N, int K, float* Out, int ldo,
                             hipStream_t s)
{
    const int64_t n_tiles = (N + kF32Cols - 1) / kF32Cols;
    const int64_t m_tiles_max = (A + kF32Rows - 1) / kF32Rows + (A < E ? A : E);
    const int64_t grid = ((m_tiles_max * n_tiles + 7) / 8) * 8;
    if (grid >= ((int64_t)1 << 31)) return hipErrorInvalidValue;   // the device-side tile search counts in 32 bits
    grouped_gemm_f32_kernel<GATED><<<(unsigned)grid, 256, 0, s>>>(X, ldx, row_map, map_div, offsets, E, W, w_expert_stride,
                                                                  N, K, Out, ldo, (int)A);
    return hipGetLastError();
}

// ----------------------------------------------------------------------------------------------
// Host side: variant choice and launches.  The host never sees the per-expert counts (they live on
// the device), so the variant is chosen from the mean rows per expert A/E and from the number of tiles these
// make; every variant is correct for any distribution of rows.
// ----------------------------------------------------------------------------------------------
enum Variant { V_TILE128 = 0, V_PIPE_SMALL, V_PIPE_FEW, V_PIPE_BIG, V_PIPE_WIDE };

// The shape of a launch: the one `pinned` names if it can run, else the library's rule.  K: length of a weight row.
static hipError_t pick_variant(int pinned, bool gated, int64_t A, int E, int N, int K, Variant* v)
{
    *v = V_TILE128;
    if (K % 64 != 0 || pinned == MOE_FFN_TILE128) return hipSuccess;      // the pipelined kernels have no k-tail path
    *v = V_PIPE_SMALL;
    if (pinned == MOE_FFN_PIPE_SMALL) return hipSuccess;
    *v = V_PIPE_FEW;
    if (pinned == MOE_FFN_PIPE_FEW) return hipSuccess;
    *v = V_PIPE_WIDE;
    if (pinned == MOE_FFN_PIPE_WIDE) return hipSuccess;
    // (the persistent kernel's pipeline is at least four stages long, and its tile list has a limit)
    const int big_cols = gated ? kBigBN / 2 : kBigBN;
    const bool big_runs = K >= 256 && big_list_fits(A, E, (N + big_cols - 1) / big_cols);
    *v = V_PIPE_BIG;
    if (pinned == MOE_FFN_PIPE_BIG && big_runs) return hipSuccess;
    int cus = 0;
    const hipError_t e = compute_units(&cus);
    if (e != hipSuccess) return e;
    // Two blocks of either streaming shape share a compute unit: up to two tiles per unit a launch is one round of
    // blocks, whatever the number of rows per expert; the first tile beyond that costs a second round.
    const int cols = gated ? 64 : 128;
    const bool small_is_one_round = tiles_expected(A, E, 64, (N + cols - 1) / cols) <= 2 * cus;
    const bool few_is_one_round = tiles_expected(A, E, 32, (N + cols / 2 - 1) / (cols / 2)) < 2 * cus;
    // Big tiles from 56 rows per expert on average, unless the 64 x 128 tiles are one round.  With many tiles (layer, us,
    // streaming against big): 128 experts, H = 2048, I = 768: 47 rows 277 / 280, 56 rows 299 / 299, 64 rows 320 / 304; 32
    // experts, H = I = 2880: 32 rows 318 / 316, 50 rows 339 / 336, 64 rows 385 / 344.  Around one round of 512 (gate_up, us):
    // 8 experts, H = I = 1024, 200 rows, 464 tiles expected 16.2 / 20.5, 400 rows, 864 tiles 26.4 / 23.3; 8 experts, H = I =
    // 2048, 80 rows, 448 tiles 26.4 / 29.5, 130 rows, 648 tiles 37.4 / 32.2; 2 experts, H = I = 512, 1000 rows, 256 tiles 11.0 /
    // 15.7.
    if (A > (int64_t)56 * E && big_runs && !small_is_one_round) return hipSuccess;
    // Rows too short for the persistent kernel (K < 256): 256 x 256 tiles, a block each, from 64 rows per expert on average.
    // Such a GEMM is bound by its outputs and the activation rows it reads per column tile.  gate_up, us, 64 x 128 against
    // 256 x 256 tiles: 64 experts, K = 192, N = 2048: 58 rows 32.1 / 34.3, 64 rows 34.3 / 34.9, 80 rows 41.2 / 37.5, 300 rows
    // 96 / 71, 1000 rows 311 / 206; K = 64, N = 1024, 1000 rows 120 / 63; 8 experts, K = 128, N = 1024, one round of 64 x 128
    // tiles at 150 rows 8.3 / 10.3, more than one at 300 rows 11.5 / 10.6.
    *v = V_PIPE_WIDE;
    if (K < 256 && A > (int64_t)64 * E && !small_is_one_round) return hipSuccess;
    // Narrow tiles (32 x 64, two waves, five stages of 12 KB) while they are one round.  What bounds such a launch is how
    // much it has in flight: 96 tiles of 64 x 128 for one token at 8 of 128 experts (H = 2048, I = 768) with two stages of
    // weights each, 16 KB, ask for 2.6 TB/s; 192 narrow ones ask for four stages of 8 KB.  Then it is a wave's own instructions: with one
    // wave to a tile the k-loop took 9.8 us whether four, five or six stages were on their way, with two waves it takes 7.9 (6.3
    // TB/s; gate_up and down of one token, clocks in the kernel, 13.2 -> 11.0 and 7.2 -> 6.3 us; a pass of four layers 139 -> 129).
    // 64 x 128 against narrow tiles, us (kernel trace, weights from memory).  Tiles of one row are level at one round: gate_up of that
    // shape, 8 experts (192 narrow tiles) 18.6 / 12.6, 16 (384) 20.4 / 19.0, 21 (504) 25.0 / 23.6, 24 (576) 32.1 / 31.3, 28 (672) 35.1 /
    // 36.4; down, 8 (256) 8.6 / 7.1, 16 (512) 10.8 / 11.0, 18 (576) 13.6 / 14.8; H = I = 2880, gate_up, 4 (360) 25.8 / 25.4, 5 (450) 27.5 /
    // 28.3, down, 4 (180) 23.2 / 13.9, 8 (360) 25.3 / 24.9.  Full tiles, whose activations two column tiles read where one did, lose a
    // little ahead of it and much behind it: gate_up, 8 experts, H = I = 1024, 24 rows (256) 11.3 / 8.8, 40 rows (512, 448 expected) 11.5 /
    // 12.2, 80 rows (768) 12.1 / 16.9; H = I = 512, 100 rows (512, 464 expected) 6.6 / 7.7, 130 rows (640) 6.8 / 11.2.
    *v = few_is_one_round ? V_PIPE_FEW : V_PIPE_SMALL;
    return hipSuccess;
}

template <int BM, int BN, bool GATED, typename OT, bool SPLIT>
static hipError_t launch_tile(RowSrc X, int ldx, const int32_t* row_map, int map_div, const int32_t* offsets,
                              int E, int64_t A, const bf16_t* W, int64_t w_expert_stride, int N, int K, void* Out,
                              int ldo, hipStream_t s)
{
    constexpr int NO = GATED ? BN / 2 : BN;
    const size_t lds_bytes = 2 * (size_t)(BM + BN) * kLdsStride * sizeof(bf16_t);
    auto kern = grouped_gemm_bf16_kernel<BM, BN, GATED, OT, SPLIT>;
    static bool attr_set[kMaxDevices] = {};
    hipError_t e = ensure_lds_limit(kern, lds_bytes, attr_set);
    if (e != hipSuccess) return e;
    const int64_t n_tiles = (N + NO - 1) / NO;
    const int64_t m_tiles_max = (A + BM - 1) / BM + (A < E ? A : E);   // sum_e ceil(m_e / BM) never exceeds this
    const int64_t grid = ((m_tiles_max * n_tiles + 7) / 8) * 8;
    if (grid >= ((int64_t)1 << 31)) return hipErrorInvalidValue;   // the device-side tile search counts in 32 bits
    kern<<<(unsigned)grid, 256, lds_bytes, s>>>(X, ldx, row_map, map_div, offsets, E, W, w_expert_stride, N, K,
                                                static_cast<OT*>(Out), ldo, (int)A);
    return hipGetLastError();
}

template <int BM, int BN, int WM, int NS, int MINW, int NW, bool GATED, bool OUT_F32, bool SPLIT, bool MAPPED>
static hipError_t launch_pipe(RowSrc X, int ldx, const int32_t* row_map, int map_div, const int32_t* offsets,
                                    int E, int64_t A, const bf16_t* W, int64_t w_expert_stride, int N, int K, void* Out,
                                    int ldo, hipStream_t s)
{
    constexpr int PBK = 64;
    constexpr int NO = GATED ? BN / 2 : BN;
    const size_t lds_bytes = (size_t)NS * (BM + BN) * PBK * 2;
    auto kern = grouped_gemm_bf16_pipe_kernel<BM / 32, BN, WM, NS, MINW, NW, GATED, OUT_F32, SPLIT, MAPPED>;
    static bool attr_set[kMaxDevices] = {};
    hipError_t e = ensure_lds_limit(kern, lds_bytes, attr_set);
    if (e != hipSuccess) return e;
    const int64_t n_tiles = (N + NO - 1) / NO;
    const int64_t m_tiles_max = (A + BM - 1) / BM + (A < E ? A : E);
    const int64_t grid = ((m_tiles_max * n_tiles + 7) / 8) * 8;
    if (grid >= ((int64_t)1 << 31)) return hipErrorInvalidValue;   // the device-side tile search counts in 32 bits
    kern<<<(unsigned)grid, NW * 64, lds_bytes, s>>>(X, ldx, row_map, map_div, map_magic_of(map_div), offsets, E, W, w_expert_stride, N, K, Out,
                                                ldo, (int)A);
    return hipGetLastError();
}

template <bool GATED, bool OUT_F32, bool SPLIT, bool MAPPED>
static hipError_t launch_big(RowSrc X, int ldx, const int32_t* row_map, int map_div, const int32_t* offsets, int E,
                             int64_t A, const bf16_t* W, int64_t w_expert_stride, int N, int K, void* Out, int ldo,
                             hipStream_t s)
{
    const size_t lds_bytes = (size_t)5 * kBigRows * 128;
    auto kern = grouped_gemm_bf16_big_kernel<GATED, OUT_F32, SPLIT, MAPPED>;
    static bool attr_set[kMaxDevices] = {};
    hipError_t e = ensure_lds_limit(kern, lds_bytes, attr_set);
    if (e != hipSuccess) return e;
    int grid = 0;
    e = big_grid(&grid);
    if (e != hipSuccess) return e;
    kern<<<(unsigned)grid, kBigWaves * 64, lds_bytes, s>>>(X, ldx, row_map, map_div, map_magic_of(map_div), offsets, E, W, w_expert_stride,
                                                           N, K, Out, ldo, (int)A);
    return hipGetLastError();
}

// K: k-extent of the GEMM (twice the weight rows' length when the plain GEMM reads a split intermediate)
template <bool GATED, bool OUT_F32, bool SPLIT>
static hipError_t launch_bf16(int variant, RowSrc X, int ldx, const int32_t* row_map, int map_div,
                              const int32_t* offsets, int E, int64_t A, const bf16_t* W, int64_t w_expert_stride,
                              int N, int K, void* Out, int ldo, hipStream_t s)
{
    // weight streaming: 64 x 128 tiles, 4 waves, 72 KB of LDS: two blocks share a compute unit, so one
    // block's prologue and epilogue are covered by the other's loads, and the many small tiles balance
    // well over the chip.  launches of few tiles: 32 x 64, 2 waves, five stages.  compute bound: up to 256 x 256 tiles,
    // one persistent block per compute unit; for rows of fewer than four stages the same tiles, a block each, two stages.
    // (only the gate_up GEMM is ever called with a row map)
    const bool mapped = GATED && row_map != nullptr;
    if (!GATED && row_map != nullptr) return hipErrorInvalidValue;
    Variant v;
    const hipError_t e = pick_variant(variant, GATED, A, E, N, (SPLIT && !GATED) ? K / 2 : K, &v);
    if (e != hipSuccess) return e;
    switch (v) {
        case V_PIPE_SMALL:
            if (mapped)
                return launch_pipe<64, 128, 2, 3, 2, 4, GATED, OUT_F32, SPLIT, GATED>(X, ldx, row_map, map_div, offsets, E, A, W, w_expert_stride, N, K, Out, ldo, s);
            return launch_pipe<64, 128, 2, 3, 2, 4, GATED, OUT_F32, SPLIT, false>(X, ldx, row_map, map_div, offsets, E, A, W, w_expert_stride, N, K, Out, ldo, s);
        case V_PIPE_FEW:
            if (mapped)
                return launch_pipe<32, 64, 1, 5, 1, 2, GATED, OUT_F32, SPLIT, GATED>(X, ldx, row_map, map_div, offsets, E, A, W, w_expert_stride, N, K, Out, ldo, s);
            return launch_pipe<32, 64, 1, 5, 1, 2, GATED, OUT_F32, SPLIT, false>(X, ldx, row_map, map_div, offsets, E, A, W, w_expert_stride, N, K, Out, ldo, s);
        case V_PIPE_WIDE:
            if (mapped)
                return launch_pipe<256, 256, 2, 2, 2, 8, GATED, OUT_F32, SPLIT, GATED>(X, ldx, row_map, map_div, offsets, E, A, W, w_expert_stride, N, K, Out, ldo, s);
            return launch_pipe<256, 256, 2, 2, 2, 8, GATED, OUT_F32, SPLIT, false>(X, ldx, row_map, map_div, offsets, E, A, W, w_expert_stride, N, K, Out, ldo, s);
        case V_PIPE_BIG:
            if (mapped)
                return launch_big<GATED, OUT_F32, SPLIT, GATED>(X, ldx, row_map, map_div, offsets, E, A, W, w_expert_stride, N, K, Out, ldo, s);
            return launch_big<GATED, OUT_F32, SPLIT, false>(X, ldx, row_map, map_div, offsets, E, A, W, w_expert_stride, N, K, Out, ldo, s);
        default:
            if (OUT_F32)
                return launch_tile<128, 128, GATED, float, SPLIT>(X, ldx, row_map, map_div, offsets, E, A, W,
                                                                  w_expert_stride, N, K, Out, ldo, s);
            return launch_tile<128, 128, GATED, bf16_t, SPLIT>(X, ldx, row_map, map_div, offsets, E, A, W,
                                                               w_expert_stride, N, K, Out, ldo, s);
    }
}

hipError_t launch_ffn_gate_up(int dtype, int variant, bool split, RowSrc x, const int32_t* row_map, int map_div,
                              const int32_t* offsets, int64_t A, int E, int H, int I, const void* w_gate_up, void* act,
                              hipStream_t s)
{
    if (dtype == MOE_BF16) {
        if (split)      // act [A, 2I]: the values' bf16 roundings in columns [0, I), the remainders in [I, 2I)
            return launch_bf16<true, false, true>(variant, x, H, row_map, map_div, offsets, E, A, (const bf16_t*)w_gate_up,
                                                  (int64_t)2 * I * H, I, H, act, 2 * I, s);
        return launch_bf16<true, false, false>(variant, x, H, row_map, map_div, offsets, E, A, (const bf16_t*)w_gate_up,
                                               (int64_t)2 * I * H, I, H, act, I, s);
    }
    return launch_f32<true>(x, H, row_map, map_div, offsets, E, A, (const float*)w_gate_up, (int64_t)2 * I * H, I, H,
                            (float*)act, I, s);
}

hipError_t launch_ffn_down(int dtype, int variant, bool out_f32, bool split, const void* act, const int32_t* offsets,
                           int64_t A, int E, int H, int I, const void* w_down, void* y_perm, hipStream_t s)
{
    if (dtype == MOE_BF16) {
        if (split)      // (a split intermediate comes with fp32 expert outputs)
            return launch_bf16<false, true, true>(variant, single_src(act), 2 * I, nullptr, 1, offsets, E, A,
                                                  (const bf16_t*)w_down, (int64_t)H * I, H, 2 * I, y_perm, H, s);
        if (out_f32)
            return launch_bf16<false, true, false>(variant, single_src(act), I, nullptr, 1, offsets, E, A,
                                                   (const bf16_t*)w_down, (int64_t)H * I, H, I, y_perm, H, s);
        return launch_bf16<false, false, false>(variant, single_src(act), I, nullptr, 1, offsets, E, A,
                                                (const bf16_t*)w_down, (int64_t)H * I, H, I, y_perm, H, s);
    }
    return launch_f32<false>(single_src(act), I, nullptr, 1, offsets, E, A, (const float*)w_down, (int64_t)H * I, H, I,
                             (float*)y_perm, H, s);
}

const char* ffn_variant_name(int dtype, int variant, int64_t A, int E, int H, int I)
{
    if (dtype != MOE_BF16) return "grouped_gemm_f32_kernel<gated>";
    Variant v;
    if (pick_variant(variant, true, A, E, I, H, &v) != hipSuccess) return "";
    switch (v) {
        case V_PIPE_SMALL: return "grouped_gemm_bf16_pipe_kernel<2,128,2,3,2,4,gated>";
        case V_PIPE_FEW: return "grouped_gemm_bf16_pipe_kernel<1,64,1,5,1,2,gated>";
        case V_PIPE_WIDE: return "grouped_gemm_bf16_pipe_kernel<8,256,2,2,2,8,gated>";
        case V_PIPE_BIG: return "grouped_gemm_bf16_big_kernel<gated>";
        default: return "grouped_gemm_bf16_kernel<128,128,gated>";
    }
}

}  // namespace moe
