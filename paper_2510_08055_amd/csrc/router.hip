// Router: fp64 logits on the f64 matrix cores, then a wavefront-level top-k with
// lowest-index tie-break and the softmax mixing weights (MoE router, Sec. 2.4).
//
// Logits are accumulated in fp64 so that the K selected experts and their order
// agree with an fp64 definition: products of two bf16 (or two fp32) values are
// exact in fp64 and the summation error (~1e-16 relative) is far below any
// realistic gap between neighbouring logits.  The reduction order of a token's
// logits depends only on H, never on the batch, so routing is batch-invariant:
// the chunked and the layered schedule route every token identically.
#include <type_traits>

#include "common.h"

namespace moe {

typedef double double4_t __attribute__((ext_vector_type(4)));

// 8 consecutive elements widened to double.  load_async() issues the global load as inline asm, so that
// the compiler neither moves it nor waits for it: the caller waits with wait_loads<N>() (N = loads that may
// still be in flight), which also names the registers as in/out operands, so no use of them can be
// scheduled above the wait.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
template <typename T> struct vec8;
template <> struct vec8<bf16_t> {
    static constexpr int kLoads = 1;
    u32x4_t raw;
    __device__ __forceinline__ void load(const bf16_t* p) { raw = *reinterpret_cast<const u32x4_t*>(p); }
    __device__ __forceinline__ void load_async(const bf16_t* p)
    {
        asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(raw) : "v"(p) : "memory");
    }
    __device__ __forceinline__ void zero() { raw = u32x4_t{0, 0, 0, 0}; }
    __device__ __forceinline__ double get(int j) const
    {
        const uint32_t w = (j < 2) ? raw.x : (j < 4) ? raw.y : (j < 6) ? raw.z : raw.w;
        return (double)__uint_as_float((j & 1) ? (w & 0xffff0000u) : (w << 16));
    }
};
template <> struct vec8<float> {
    static constexpr int kLoads = 2;
    f32x4_t a, b;
    __device__ __forceinline__ void load(const float* p)
    {
        a = *reinterpret_cast<const f32x4_t*>(p);
        b = *reinterpret_cast<const f32x4_t*>(p + 4);
    }
    __device__ __forceinline__ void load_async(const float* p)
    {
        asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(a) : "v"(p) : "memory");
        asm volatile("global_load_dwordx4 %0, %1, off offset:16" : "=v"(b) : "v"(p) : "memory");
    }
    __device__ __forceinline__ void zero() { a = b = f32x4_t{0.f, 0.f, 0.f, 0.f}; }
    __device__ __forceinline__ double get(int j) const
    {
        const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        return (double)v[j];
    }
};
template <int N> __device__ __forceinline__ void wait_loads(vec8<bf16_t>& x, vec8<bf16_t>& w)
{
    asm volatile("s_waitcnt vmcnt(%2)" : "+v"(x.raw), "+v"(w.raw) : "n"(N) : "memory");
}
template <int N> __device__ __forceinline__ void wait_loads(vec8<float>& x, vec8<float>& w)
{
    asm volatile("s_waitcnt vmcnt(%4)" : "+v"(x.a), "+v"(x.b), "+v"(w.a), "+v"(w.b) : "n"(N) : "memory");
}

// Drain of a ring of four operand buffers: waits for every load in flight and names ALL ring registers, so
// that none of them can be handed to another value while a look-ahead load may still land on it.
__device__ __forceinline__ void wait_ring(vec8<bf16_t> (&x)[4], vec8<bf16_t> (&w)[4])
{
    asm volatile("s_waitcnt vmcnt(0)"
                 : "+v"(x[0].raw), "+v"(x[1].raw), "+v"(x[2].raw), "+v"(x[3].raw), "+v"(w[0].raw), "+v"(w[1].raw),
                   "+v"(w[2].raw), "+v"(w[3].raw)
                 :
                 : "memory");
}
__device__ __forceinline__ void wait_ring(vec8<float> (&x)[4], vec8<float> (&w)[4])
{
    asm volatile("s_waitcnt vmcnt(0)"
                 : "+v"(x[0].a), "+v"(x[0].b), "+v"(x[1].a), "+v"(x[1].b), "+v"(x[2].a), "+v"(x[2].b), "+v"(x[3].a),
                   "+v"(x[3].b), "+v"(w[0].a), "+v"(w[0].b), "+v"(w[1].a), "+v"(w[1].b), "+v"(w[2].a), "+v"(w[2].b),
                   "+v"(w[3].a), "+v"(w[3].b)
                 :
                 : "memory");
}

// One block: a 16-token x 16-expert tile of logits with v_mfma_f64_16x16x4.  The hidden dimension is cut
// into 32-wide chunks, chunk c belongs to partial sum c % 16, and the 16 partial sums are added in a fixed
// tree (p, p + 4, p + 8, p + 12 in order for p = 0..3, then those four in order), so the summation order of a
// logit is fixed by H alone, whichever of the two block shapes computes it:
//   NW = 4:  wave w holds partial sums w, w + 4, w + 8, w + 12 (four independent MFMA chains).  The shape of the
//            stand-alone logits kernel (16 waves per block were no faster there at 272 to 640 tokens: 11.5 against
//            11.9 us and 16.4 against 18.4 us).
//   NW = 16: one partial sum per wave.  The shape of the one-launch routing of a decode batch, whose few blocks are
//            a serial chain of load latencies and 64-clock MFMAs: 1 us shorter than with 4 waves at H = 2048, 2 us
//            at H = 2880.
// Lane l supplies row (l % 16) of both operands; its quarter q = l / 16 owns the 8 consecutive
// k-values [c*32 + q*8, c*32 + q*8 + 8) of chunk c and feeds them to 8 successive MFMAs (any fixed
// pairing of k-slots is a valid summation order).  The raw operands of the next chunks are fetched
// while the MFMAs of the current one run; many short waves per SIMD hide the rest of the latency.
// (32 x 32 tiles per block, each widened operand feeding two MFMAs, measured slower: a quarter as
// many blocks leaves a 20 % tail on 256 compute units, and the matrix pipe, not the loads, is the limit.)
constexpr int kRouterBufs = 4;      // (wait_ring names exactly four buffers)

// Stores and loads that meet at the level every block of the launch sees (past the caches of one XCD), for data
// that one block hands to another inside a launch; the order between them comes from the ticket counters.
template <typename V> __device__ __forceinline__ void store_shared(V* p, V v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename V> __device__ __forceinline__ V load_shared(const V* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The tile of logits at (t0, e0), written by wave 0 of the block; every thread of the block calls it.
// SHARED: another block of the same launch reads the logits.
template <typename T, int NW, bool SHARED>
__device__ __forceinline__ void logits_tile(const RowSrc& x, int64_t n_tok, int H, const T* __restrict__ wr,
                                            const float* __restrict__ bias, int E, double* __restrict__ logits, int64_t t0,
                                            int e0)
{
    constexpr int NACC = 16 / NW;                // partial sums per wave
    static_assert(NW == 4 || NW == 16, "16 partial sums over 4 or 16 waves");
    __shared__ double part[NW - 1][4][64];       // [wave-1][element v][lane]: a wave's partial sums, already added up
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r = lane & 15, q = lane >> 4;
    const int64_t tr = (t0 + r < n_tok) ? (t0 + r) : (n_tok - 1);  // clamp: loads stay in bounds
    const int er = (e0 + r < E) ? (e0 + r) : (E - 1);
    const T* xp = row_ptr<T>(x, tr, H) + q * 8;
    const T* wp = wr + (int64_t)er * H + q * 8;

    double4_t acc[NACC];
#pragma unroll
    for (int a = 0; a < NACC; ++a) acc[a] = double4_t{0.0, 0.0, 0.0, 0.0};
    // Ring of kRouterBufs operand buffers: the raw operands of this wave's next kRouterBufs - 1 chunks are
    // in flight while the MFMAs of the current chunk run.  Loads and waits of the ring are explicit (the
    // compiler would otherwise sink the loads next to their uses and wait for all of them); the look-ahead
    // index is clamped to the wave's last whole chunk rather than tested, so the loop body is branch-free.
    vec8<T> xa[kRouterBufs], wa[kRouterBufs];
    auto multiply = [&](int buf, double4_t& a) {
#pragma unroll
        for (int j = 0; j < 8; ++j)
            a = __builtin_amdgcn_mfma_f64_16x16x4f64(xa[buf].get(j), wa[buf].get(j), a, 0, 0, 0);
    };
    auto multiply_into = [&](int buf, int i) {   // the i-th chunk of this wave, i not known at compile time
#pragma unroll
        for (int a = 0; a < NACC; ++a)
            if (a == i % NACC) multiply(buf, acc[a]);
    };
    const int n_whole = H / 32;                                            // whole 32-wide chunks of a row
    const int mine = n_whole > wave ? (n_whole - wave + NW - 1) / NW : 0;   // of which this wave takes chunks wave, wave + NW, ...
    auto fetch = [&](int buf, int i) {                                      // this wave's i-th chunk
        const int k0 = (wave + NW * i) * 32;
        xa[buf].load_async(xp + k0);
        wa[buf].load_async(wp + k0);
    };
    constexpr int kPerChunk = 2 * vec8<T>::kLoads;                          // load instructions per chunk
    int i = 0;
    if (mine >= kRouterBufs) {
#pragma unroll
        for (int b = 0; b < kRouterBufs - 1; ++b) fetch(b, b);
        for (; i + kRouterBufs <= mine; i += kRouterBufs) {
#pragma unroll
            for (int b = 0; b < kRouterBufs; ++b) {
                const int ahead = i + b + kRouterBufs - 1;
                fetch((b + kRouterBufs - 1) % kRouterBufs, ahead < mine ? ahead : mine - 1);
                wait_loads<(kRouterBufs - 1) * kPerChunk>(xa[b], wa[b]);
                multiply(b, acc[b % NACC]);      // (i is a multiple of kRouterBufs, which NACC divides)
            }
        }
        // the look-ahead loads of the last round are still in flight; they target ring registers
        wait_ring(xa, wa);
    }
    for (; i < mine; ++i) {        // the last few whole chunks, one at a time
        fetch(0, i);
        wait_loads<0>(xa[0], wa[0]);
        multiply_into(0, i);
    }
    if (H % 32 != 0 && wave == n_whole % NW) {      // the row's partial chunk: lanes past the end feed zeros
        const int k0 = n_whole * 32;
        if (k0 + q * 8 < H) {
            xa[0].load(xp + k0);
            wa[0].load(wp + k0);
        } else {
            xa[0].zero();
            wa[0].zero();
        }
        multiply_into(0, n_whole / NW);
    }
    double4_t mysum = acc[0];
#pragma unroll
    for (int a = 1; a < NACC; ++a) mysum += acc[a];
    if (wave > 0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) part[wave - 1][v][lane] = mysum[v];
    }
    __syncthreads();
    if (wave != 0) return;
    // D layout of the f64 16x16x4 MFMA: lane l, element v holds row 4*v + l/16 (token), column l % 16 (expert).
    const int e = e0 + r;
    if (e < E) {
        const double b = bias ? (double)bias[e] : 0.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t t = t0 + v * 4 + q;
            double z = 0.0;
#pragma unroll
            for (int p = 0; p < 4; ++p) {        // partial sums p, p + 4, p + 8, p + 12
                double s = p == 0 ? mysum[v] : part[p - 1][v][lane];
#pragma unroll
                for (int w = p + 4; w < NW; w += 4) s += part[w - 1][v][lane];
                z = p == 0 ? s : z + s;
            }
            if (t < n_tok) {
                if (SHARED) store_shared(logits + t * E + e, z + b);
                else logits[t * E + e] = z + b;
            }
        }
    }
}

template <typename T>
__global__ __launch_bounds__(256) void router_logits_kernel(RowSrc x, int64_t n_tok, int H,
                                                            const T* __restrict__ wr,
                                                            const float* __restrict__ bias, int E,
                                                            double* __restrict__ logits,
                                                            int32_t* __restrict__ zero_buf, int zero_n)
{
    // side job of block (0,0): clear the per-tile expert histogram that the top-k kernel, next on the
    // stream, counts into (saves a separate fill launch)
    if (blockIdx.x == 0 && blockIdx.y == 0)
        for (int i = threadIdx.x; i < zero_n; i += 256) zero_buf[i] = 0;
    logits_tile<T, 4, false>(x, n_tok, H, wr, bias, E, logits, (int64_t)blockIdx.x * 16, (int)blockIdx.y * 16);
}

// (value, index) "greater" under the routing order: larger logit first, equal logits by lower index.
__device__ __forceinline__ bool before(double va, int ia, double vb, int ib)
{
    return va > vb || (va == vb && ia < ib);
}

// One wave per token (TPW tokens one after the other).  Lane l holds logits of experts l, l+64, ...;
// K rounds of a wave-wide arg-max, each removing the winner.  Lane j keeps the j-th winner and
// computes its weight.  The block also counts its assignments per (permutation tile, expert) in LDS
// and adds the non-zero bins to the global per-tile histogram: integer counts do not depend on the
// order of the atomics, and few experts (a skewed top-2 of 8) no longer serialise on one address.
constexpr int kTopkWaves = 8;
template <int NPL>
__global__ __launch_bounds__(kTopkWaves * 64) void topk_kernel(const double* __restrict__ logits, int64_t n_tok, int E,
                                                               int K, int renorm, int tpw, int32_t* __restrict__ idx,
                                                               float* __restrict__ w, int32_t* __restrict__ tile_hist)
{
    // a block's assignments (at most 8 waves x tpw tokens x K <= kPermTile) touch at most two tiles
    __shared__ int32_t hist[2][kMaxExperts];
    const int lane = lane_id();
    const int wave = threadIdx.x >> 6;
    const int64_t tb0 = (int64_t)blockIdx.x * (kTopkWaves * tpw);
    const int64_t tile0 = tb0 * K / kPermTile;
    if (tile_hist) {
        for (int i = threadIdx.x; i < 2 * E; i += kTopkWaves * 64) hist[i / E][i % E] = 0;
        __syncthreads();
    }
    const double NEG = -__builtin_huge_val();
    for (int it = 0; it < tpw; ++it) {
        const int64_t t = tb0 + (int64_t)wave * tpw + it;
        if (t >= n_tok) break;
        double v[NPL];
#pragma unroll
        for (int i = 0; i < NPL; ++i) {
            const int e = lane + 64 * i;
            v[i] = (e < E) ? logits[t * E + e] : NEG;
        }
        double my_z = NEG;
        int my_e = 0;
        double z_max = 0.0;
        for (int j = 0; j < K; ++j) {
            double bv = v[0];
            int bi = 0;
#pragma unroll
            for (int i = 1; i < NPL; ++i)
                if (v[i] > bv) { bv = v[i]; bi = i; }
            int be = lane + 64 * bi;
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) {
                const double ov = __shfl_xor(bv, off, 64);
                const int oe = __shfl_xor(be, off, 64);
                if (before(ov, oe, bv, be)) { bv = ov; be = oe; }
            }
            if (j == 0) z_max = bv;
            if (lane == j) { my_z = bv; my_e = be; }
            if ((be & 63) == lane) {
                const int slot = be >> 6;
#pragma unroll
                for (int i = 0; i < NPL; ++i)
                    if (i == slot) v[i] = NEG;
            }
        }
        // softmax numerator of the selected expert; denominator over all E unless renormalising
        double p = (lane < K) ? exp(my_z - z_max) : 0.0;
        double denom;
        if (renorm) {
            denom = p;
        } else {
            denom = 0.0;
#pragma unroll
            for (int i = 0; i < NPL; ++i) {
                const int e = lane + 64 * i;
                if (e < E) denom += exp(logits[t * E + e] - z_max);
            }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) denom += __shfl_xor(denom, off, 64);
        if (lane < K) {
            idx[t * K + lane] = my_e;
            w[t * K + lane] = (float)(p / denom);
            if (tile_hist) atomicAdd(&hist[(t * K + lane) / kPermTile - tile0][my_e], 1);
        }
    }
    if (tile_hist) {
        __syncthreads();
        for (int i = threadIdx.x; i < 2 * E; i += kTopkWaves * 64) {
            const int c = hist[i / E][i % E];
            if (c) atomicAdd(&tile_hist[(tile0 + i / E) * E + i % E], c);
        }
    }
}

// ----------------------------------------------------------------------------------------------
// Top-k for K <= 16: one token per 16-lane row, four tokens per wave.  Lane c of a row holds the
// logits of experts c, c+16, c+32, ...; a round takes the lane's best, then an all-reduce over the
// row in four DPP steps (lane ^ 1, lane ^ 2, mirror within 8, mirror within 16: register-to-register
// moves, no LDS), under the same total order (logit desc, index asc), so every lane of the row ends
// with the same winner.  Lane j of the row keeps winner j.
// ----------------------------------------------------------------------------------------------
template <int CTRL> __device__ __forceinline__ int dpp_mov(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true);
}
template <int CTRL> __device__ __forceinline__ double dpp_mov(double v)
{
    return __hiloint2double(dpp_mov<CTRL>(__double2hiint(v)), dpp_mov<CTRL>(__double2loint(v)));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;

template <int CTRL> __device__ __forceinline__ void row_best_step(double& bv, int& be)
{
    const double ov = dpp_mov<CTRL>(bv);
    const int oe = dpp_mov<CTRL>(be);
    if (before(ov, oe, bv, be)) { bv = ov; be = oe; }
}
template <int CTRL> __device__ __forceinline__ double row_sum_step(double v) { return v + dpp_mov<CTRL>(v); }

// Top-k of token t by the 16 lanes of a row (c = lane % 16): lane c < K ends with the c-th winner and its
// weight.  All lanes of the row hold the same t.
template <int NPL>   // logits per lane: experts c + 16 i, i < NPL
__device__ __forceinline__ void topk_of_row(const double* z, int E, int K, int renorm, int c, bool shared, int& my_e,
                                            float& my_w)
{
    const double NEG = -__builtin_huge_val();
    double v[NPL];
#pragma unroll
    for (int i = 0; i < NPL; ++i) {
        const int e = c + 16 * i;
        v[i] = (e < E) ? (shared ? load_shared(z + e) : z[e]) : NEG;
    }
    double esum = 0.0;      // only without renormalisation: this lane's share of sum_e exp(z_e - z_max)
    double my_z = NEG, z_max = 0.0;
    my_e = 0;
    for (int j = 0; j < K; ++j) {
        double bv = v[0];
        int be = c;
#pragma unroll
        for (int i = 1; i < NPL; ++i)
            if (v[i] > bv) { bv = v[i]; be = c + 16 * i; }     // equal values: the lower index stays
        row_best_step<kDppXor1>(bv, be);
        row_best_step<kDppXor2>(bv, be);
        row_best_step<kDppHalfMirror>(bv, be);
        row_best_step<kDppMirror>(bv, be);
        if (j == 0) {
            z_max = bv;
            if (!renorm) {
#pragma unroll
                for (int i = 0; i < NPL; ++i)
                    if (c + 16 * i < E) esum += exp(v[i] - z_max);
            }
        }
        if (c == j) { my_z = bv; my_e = be; }
        if ((be & 15) == c) {
            const int slot = be >> 4;
#pragma unroll
            for (int i = 0; i < NPL; ++i)
                if (i == slot) v[i] = NEG;
        }
    }
    const double p = (c < K) ? exp(my_z - z_max) : 0.0;
    double denom = renorm ? p : esum;
    denom = row_sum_step<kDppXor1>(denom);
    denom = row_sum_step<kDppXor2>(denom);
    denom = row_sum_step<kDppHalfMirror>(denom);
    denom = row_sum_step<kDppMirror>(denom);
    my_w = (float)(p / denom);
}

template <int NPL>
__global__ __launch_bounds__(kTopkWaves * 64) void topk_rows_kernel(const double* __restrict__ logits, int64_t n_tok,
                                                                    int E, int K, int renorm, int32_t* __restrict__ idx,
                                                                    float* __restrict__ w,
                                                                    int32_t* __restrict__ tile_hist)
{
    // a block's assignments (32 tokens x K <= 512) touch at most two permutation tiles
    __shared__ int32_t hist[2][kMaxExperts];
    const int lane = lane_id();
    const int wave = threadIdx.x >> 6;
    const int c = lane & 15;
    const int64_t tb0 = (int64_t)blockIdx.x * (kTopkWaves * 4);
    const int64_t tile0 = tb0 * K / kPermTile;
    if (tile_hist) {
        for (int i = threadIdx.x; i < 2 * E; i += kTopkWaves * 64) hist[i / E][i % E] = 0;
        __syncthreads();
    }
    const int64_t t = tb0 + wave * 4 + (lane >> 4);
    const bool live = t < n_tok;
    const int64_t tl = live ? t : n_tok - 1;      // rows past the end work on a copy of the last token, store nothing
    int my_e;
    float my_w;
    topk_of_row<NPL>(logits + tl * E, E, K, renorm, c, false, my_e, my_w);
    if (live && c < K) {
        idx[t * K + c] = my_e;
        w[t * K + c] = my_w;
        if (tile_hist) atomicAdd(&hist[(t * K + c) / kPermTile - tile0][my_e], 1);
    }
    if (tile_hist) {
        __syncthreads();
        for (int i = threadIdx.x; i < 2 * E; i += kTopkWaves * 64) {
            const int cnt = hist[i / E][i % E];
            if (cnt) atomicAdd(&tile_hist[(tile0 + i / E) * E + i % E], cnt);
        }
    }
}

// ----------------------------------------------------------------------------------------------
// Router, top-k and permutation of a decode batch (at most kSmallTokens tokens, K <= 16) in one launch.
//
// On such a batch the three kernels are a chain of launches with almost nothing in each: one token through
// E = 128 took 8.1 + 5.0 + 8.9 us, of which the arithmetic is a microsecond.  Here every block computes its
// tile of logits and takes a ticket of its 16 tokens; the block that draws the last one finds their logits
// written and does their top-k; of those blocks, the one that draws the last ticket of the batch does the
// permutation (no block ever waits for another).  A token's experts are distinct as long as K of its logits are finite;
// the stable rank of an assignment inside its expert is then the number of earlier tokens that chose the expert: one
// bit per token and expert in LDS, counted with popcounts.  A bit that is set twice (a removed expert and one with a
// logit of -infinity compare equal, NaN compares with nothing) sends the batch to a count of the earlier assignments
// one by one.  What crosses between blocks goes past the XCD's caches by itself
// (store_shared / load_shared): a fence would write back and drop the whole L2, 2 us with a few blocks and 15 us
// with a hundred.  Every last drawer puts its counter back to zero.
// Measured (H = 2048, E = 128, top-8; events around the launches, three launches -> one): 1 token 28.9 -> 15.4 us,
// 32 tokens 29.3 -> 17.8 us, 128 tokens 30.2 -> 19.0 us; 256 tokens at H = 2880, top-4 31.0 -> 20.8 us.  A last
// block that does the top-k of all tokens was slower from 32 tokens on (26 us; 46 us at 128).
// ----------------------------------------------------------------------------------------------
constexpr int kSmallWaves = 16;
constexpr int kSmallWords = kSmallTokens / 64;

// Draws a ticket for the block once everything it has stored is visible; true for the last of n drawers.
// Every thread of the block calls it (`flag`: a word of LDS).
__device__ __forceinline__ bool last_to_arrive(uint32_t* ticket, uint32_t n, int32_t* flag)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // this wave's stores have reached the shared level
    __syncthreads();
    if (threadIdx.x == 0) {
        const bool last = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
        if (last) store_shared(ticket, 0u);
        *flag = last;
    }
    __syncthreads();
    return *flag != 0;
}

template <typename T, int NPL>
__global__ __launch_bounds__(kSmallWaves * 64) void route_small_kernel(
    RowSrc x, int n_tok, int H, const T* __restrict__ wr, const float* __restrict__ bias, int E, int K, int renorm,
    double* logits, int32_t* idx, float* __restrict__ w, int32_t* __restrict__ offsets, int32_t* __restrict__ perm,
    int32_t* __restrict__ inv, unsigned long long* __restrict__ active_total, uint32_t* tickets)
{
    __shared__ unsigned long long chosen[kSmallExperts][kSmallWords];      // bit t of an expert: token t chose it
    __shared__ int32_t count[kSmallExperts], start[kSmallExperts];
    __shared__ int32_t own[16 * 16];                                       // the experts of this block's 16 tokens
    __shared__ uint8_t expert_of[kSmallTokens * 16];                       // only when a token chose an expert twice
    __shared__ int32_t flag, twice;
    static_assert(kSmallExperts <= 256, "an expert is one byte of expert_of");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t0 = (int)blockIdx.x * 16;
    logits_tile<T, kSmallWaves, true>(x, n_tok, H, wr, bias, E, logits, t0, (int)blockIdx.y * 16);
    for (int i = tid; i < E * kSmallWords; i += kSmallWaves * 64) (&chosen[0][0])[i] = 0ull;
    if (tid < E) count[tid] = 0;
    if (tid == 0) twice = 0;
    if (!last_to_arrive(tickets + 1 + blockIdx.x, gridDim.y, &flag)) return;

    // top-k of this block's 16 tokens: 16 lanes per token, four waves
    const bool single = gridDim.x == 1;       // a batch of one token tile: nothing to hand to another block
    if (wave < 4) {
        const int c = lane & 15, row = wave * 4 + (lane >> 4);
        const int t = t0 + row;
        int e;
        float wt;
        topk_of_row<NPL>(logits + (int64_t)(t < n_tok ? t : n_tok - 1) * E, E, K, renorm, c, true, e, wt);
        if (t < n_tok && c < K) {
            w[t * K + c] = wt;
            if (single) own[row * K + c] = e;
            else store_shared(idx + t * K + c, (int32_t)e);
        }
    }
    if (single) __syncthreads();
    else if (!last_to_arrive(tickets, gridDim.x, &flag)) return;

    const int A = n_tok * K;
    constexpr int PER = kSmallTokens * 16 / (kSmallWaves * 64);            // assignments per thread, at most
    int my_e[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int f = p * kSmallWaves * 64 + tid;
        my_e[p] = -1;
        if (f < A) my_e[p] = single ? own[f] : load_shared(idx + f);
    }
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int f = p * kSmallWaves * 64 + tid;
        if (my_e[p] >= 0) {
            const int t = f / K;
            const unsigned long long bit = 1ull << (t & 63);
            if (atomicOr(&chosen[my_e[p]][t >> 6], bit) & bit) twice = 1;
            atomicAdd(&count[my_e[p]], 1);
        }
    }
    __syncthreads();
    // exclusive scan of the expert counts by wave 0: lane l owns experts [4 l, 4 l + 4)
    if (wave == 0) {
        constexpr int EPL = kSmallExperts / 64;
        int cnt[EPL], sum = 0, act = 0;
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            const int e = lane * EPL + i;
            cnt[i] = e < E ? count[e] : 0;
            sum += cnt[i];
            act += cnt[i] > 0;
        }
        int incl = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(incl, off, 64);
            if (lane >= off) incl += o;
        }
        int run = incl - sum;
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            const int e = lane * EPL + i;
            if (e < E) {
                start[e] = run;
                offsets[e] = run;
            }
            run += cnt[i];
        }
        if (lane == 63) offsets[E] = incl;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) act += __shfl_xor(act, off, 64);
        if (lane == 0) atomicAdd(active_total, (unsigned long long)act);
    }
    __syncthreads();
    const bool recount = twice != 0;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int f = p * kSmallWaves * 64 + tid;
        const int e = my_e[p];
        if (e < 0) continue;
        const int t = f / K;
        int pos = start[e];
        for (int j = 0; j <= (t >> 6); ++j) {
            const unsigned long long m = chosen[e][j];
            pos += __popcll(j < (t >> 6) ? m : m & ((1ull << (t & 63)) - 1));
        }
        if (recount) continue;                // (asked this late: the answer is here when the position is)
        perm[pos] = f;
        inv[f] = pos;
    }
    if (__builtin_expect(recount, 0)) {
#pragma unroll
        for (int p = 0; p < PER; ++p)
            if (my_e[p] >= 0) expert_of[p * kSmallWaves * 64 + tid] = (uint8_t)my_e[p];
        __syncthreads();
#pragma unroll 1
        for (int f = tid; f < A; f += kSmallWaves * 64) {
            const int e = expert_of[f];
            int pos = start[e];
            for (int g = 0; g < f; ++g) pos += expert_of[g] == e;
            perm[pos] = f;
            inv[f] = pos;
        }
    }
}

hipError_t launch_route_small(int dtype, RowSrc x, int64_t T, int H, const void* w_router, const float* bias, int E, int K,
                              int renorm, double* logits, int32_t* idx, float* w, int32_t* offsets, int32_t* perm, int32_t* inv,
                              unsigned long long* active_total, uint32_t* tickets, hipStream_t s)
{
    if (!route_is_small(T, E, K)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((T + 15) / 16), (unsigned)((E + 15) / 16));
    const int npl = (E + 15) / 16;
    auto go = [&](auto npl_const) {
        constexpr int NPL = decltype(npl_const)::value;
        if (dtype == MOE_BF16)
            route_small_kernel<bf16_t, NPL><<<grid, kSmallWaves * 64, 0, s>>>(
                x, (int)T, H, (const bf16_t*)w_router, bias, E, K, renorm, logits, idx, w, offsets, perm, inv, active_total, tickets);
        else
            route_small_kernel<float, NPL><<<grid, kSmallWaves * 64, 0, s>>>(
                x, (int)T, H, (const float*)w_router, bias, E, K, renorm, logits, idx, w, offsets, perm, inv, active_total, tickets);
        return hipGetLastError();
    };
    if (npl <= 1) return go(std::integral_constant<int, 1>{});
    if (npl <= 2) return go(std::integral_constant<int, 2>{});
    if (npl <= 8) return go(std::integral_constant<int, 8>{});
    return go(std::integral_constant<int, 16>{});
}

hipError_t launch_router_logits(int dtype, RowSrc x, int64_t T, int H, const void* w_router, const float* bias,
                                int E, double* logits, int32_t* zero_buf, int zero_n, hipStream_t s)
{
    dim3 grid((unsigned)((T + 15) / 16), (unsigned)((E + 15) / 16));
    if (dtype == MOE_BF16)
        router_logits_kernel<bf16_t><<<grid, 256, 0, s>>>(x, T, H, (const bf16_t*)w_router, bias, E, logits, zero_buf,
                                                          zero_n);
    else
        router_logits_kernel<float><<<grid, 256, 0, s>>>(x, T, H, (const float*)w_router, bias, E, logits, zero_buf,
                                                         zero_n);
    return hipGetLastError();
}

hipError_t launch_topk(const double* logits, int64_t T, int E, int K, int renorm, int32_t* idx, float* w,
                       int32_t* tile_hist, hipStream_t s)
{
    if (K <= 16) {
        const unsigned grid = (unsigned)((T + kTopkWaves * 4 - 1) / (kTopkWaves * 4));
        const int npl = (E + 15) / 16;
#define MOE_TOPK_ROWS(N) topk_rows_kernel<N><<<grid, kTopkWaves * 64, 0, s>>>(logits, T, E, K, renorm, idx, w, tile_hist)
        if (npl <= 1) MOE_TOPK_ROWS(1);
        else if (npl <= 2) MOE_TOPK_ROWS(2);
        else if (npl <= 4) MOE_TOPK_ROWS(4);
        else if (npl <= 8) MOE_TOPK_ROWS(8);
        else if (npl <= 16) MOE_TOPK_ROWS(16);
        else MOE_TOPK_ROWS(32);
#undef MOE_TOPK_ROWS
        return hipGetLastError();
    }
    // more than 16 winners per token: one token per wave, lane j keeps winner j
    const int tpw = T <= 2048 ? 1 : 4;
    const unsigned grid = (unsigned)((T + kTopkWaves * tpw - 1) / (kTopkWaves * tpw));
    const int npl = (E + 63) / 64;
    if (npl <= 1) topk_kernel<1><<<grid, kTopkWaves * 64, 0, s>>>(logits, T, E, K, renorm, tpw, idx, w, tile_hist);
    else if (npl <= 2) topk_kernel<2><<<grid, kTopkWaves * 64, 0, s>>>(logits, T, E, K, renorm, tpw, idx, w, tile_hist);
    else if (npl <= 4) topk_kernel<4><<<grid, kTopkWaves * 64, 0, s>>>(logits, T, E, K, renorm, tpw, idx, w, tile_hist);
    else topk_kernel<8><<<grid, kTopkWaves * 64, 0, s>>>(logits, T, E, K, renorm, tpw, idx, w, tile_hist);
    return hipGetLastError();
}

}  // namespace moe
