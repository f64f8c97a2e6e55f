// Router: fp64 logits on the f64 matrix cores, then a wavefront-level top-k with
// lowest-index tie-break and the softmax mixing weights (MoE router, Sec. 2.4).
//
// Logits are accumulated in fp64 so that the K selected experts and their order
// agree with an fp64 definition: products of two bf16 (or two fp32) values are
// exact in fp64 and the summation error (~1e-16 relative) is far below any
// realistic gap between neighbouring logits.  The reduction order of a token's
// logits depends only on H, never on the batch, so routing is batch-invariant:
// the chunked and the layered schedule route every token identically.  Large bf16
// batches take exact integer sums instead (route_exact_kernel): tokens whose experts
// or weights the difference to the fp64 chain (its rounding) could change are found
// by a bound on it and take the chain after all, so the results are the chain's.
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
    __device__ __forceinline__ void load_lds(const char* p) { raw = *reinterpret_cast<const u32x4_t*>(p); }      // a load's 1 KB apart
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
    __device__ __forceinline__ void load_lds(const char* p)
    {
        a = *reinterpret_cast<const f32x4_t*>(p);
        b = *reinterpret_cast<const f32x4_t*>(p + 1024);
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
//   NW = 4:  wave w holds partial sums w, w + 4, w + 8, w + 12: four independent MFMA chains.  (16 waves per block were no faster at 272 to
//            640 tokens: 11.5 against 11.9 us and 16.4 against 18.4 us.)
//   NW = 16: one partial sum per wave.  The shape of a decode batch's one-launch routing where a block has a whole tile of logits
//            (see route_small_tile_kernel; where it has a fourth of one, route_small_kernel, with the same order of summation).
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
    return __builtin_amdgcn_readfirstlane(*flag) != 0;
}

// The tile of logits of rows row(0 .. 15) and experts e0 .. e0 + 15, stored by wave 0; every thread of the block calls it.
// Rows from n_rows on are read and not used.  store(i, j, z) takes the logit z of row i < n_rows and expert e0 + j < E.
template <typename T, int NW, typename Row, typename Store>
__device__ __forceinline__ void logits_tile(Row row, int n_rows, int H, const T* __restrict__ wr,
                                            const float* __restrict__ bias, int E, int e0, Store store)
{
    constexpr int NACC = 16 / NW;                // partial sums per wave
    static_assert(NW == 4 || NW == 16, "16 partial sums over 4 or 16 waves");
    __shared__ double part[NW - 1][4][64];       // [wave-1][element v][lane]: a wave's partial sums, already added up
    const int lane = lane_id();
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int r = lane & 15, q = lane >> 4;
    const int er = (e0 + r < E) ? (e0 + r) : (E - 1);              // clamp: loads stay in bounds
    const T* xp = row(r) + q * 8;
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
            double z = 0.0;
#pragma unroll
            for (int p = 0; p < 4; ++p) {        // partial sums p, p + 4, p + 8, p + 12
                double s = p == 0 ? mysum[v] : part[p - 1][v][lane];
#pragma unroll
                for (int w = p + 4; w < NW; w += 4) s += part[w - 1][v][lane];
                z = p == 0 ? s : z + s;
            }
            if (v * 4 + q < n_rows) store(v * 4 + q, r, z + b);
        }
    }
}

// The 16 rows from t0 on, the last row again past the end.
template <typename T> __device__ __forceinline__ auto rows_from(const RowSrc& x, int64_t t0, int64_t n_tok, int H)
{
    return [=](int i) { return row_ptr<T>(x, t0 + i < n_tok ? t0 + i : n_tok - 1, H); };
}
__device__ __forceinline__ int rows_left(int64_t t0, int64_t n_tok, int most) { return n_tok - t0 < most ? (int)(n_tok - t0) : most; }

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
    const int64_t t0 = (int64_t)blockIdx.x * 16;
    const int e0 = (int)blockIdx.y * 16;
    logits_tile<T, 4>(rows_from<T>(x, t0, n_tok, H), rows_left(t0, n_tok, 16), H, wr, bias, E, e0,
                      [&](int i, int j, double z) { logits[(t0 + i) * E + e0 + j] = z; });
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
// logits of experts c, c+16, c+32, ...; a round takes the row's largest logit and then the lowest index that has it, either an
// all-reduce over the row in four DPP steps (lane ^ 1, lane ^ 2, mirror within 8, mirror within 16: register-to-register
// moves, no LDS), which is the same total order (logit desc, index asc); every lane of the row ends
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

template <int CTRL> __device__ __forceinline__ double row_sum_step(double v) { return v + dpp_mov<CTRL>(v); }
template <int CTRL> __device__ __forceinline__ double row_max_step(double v) { return __builtin_fmax(v, dpp_mov<CTRL>(v)); }
template <int CTRL> __device__ __forceinline__ int row_min_step(int v)
{
    const int o = dpp_mov<CTRL>(v);
    return o < v ? o : v;
}
__device__ __forceinline__ double row_max(double v)
{
    return row_max_step<kDppMirror>(row_max_step<kDppHalfMirror>(row_max_step<kDppXor2>(row_max_step<kDppXor1>(v))));
}
__device__ __forceinline__ int row_min(int v)
{
    return row_min_step<kDppMirror>(row_min_step<kDppHalfMirror>(row_min_step<kDppXor2>(row_min_step<kDppXor1>(v))));
}

// How far the logits of R tokens may be from those of the fp64 chain (see route_exact_kernel), and what comes of it.
struct NoMargin {
    static constexpr bool kCheck = false;
};
template <int R, typename Head> struct Margin {
    static constexpr bool kCheck = true;
    Head row[R];
    const Head* experts;
    double product[R];      // |x| max |w|
    double chain_error;     // a logit without its bias is at most chain_error * product from the chain's
    bool sure[R];           // out, the same in all lanes of the row: indices and weights are the same with the chain's logits

    // May the chain round a logit of token r and expert e: 0 nowhere, 1 where its partial sums meet, 2 anywhere?
    __device__ __forceinline__ int rounds(int r, int e) const
    {
        const Head w = experts[e];
        const float exact = ldexpf(1.f, 53 + row[r].last + w.last);
        return row[r].norm * w.norm < exact ? 0 : (row[r].part * w.part < exact ? 1 : 2);
    }
};

// Top-k of R tokens by the 16 lanes of a row (c = lane % 16): lane c < K ends with the c-th winner of each and its weight.
// logit(r, e): that of token r and expert e < E.  (A round is a chain of dependent instructions; two tokens fill its gaps.)
// With a margin K must be less than E.
// Whatever the logits are, it ends after its rounds, with indices below E, and waits for no other wave: route_small_kernel has one wave walk
// through it over LDS that loads still write.  So no barrier and no loop whose end hangs on a logit may come in.
template <int NPL, int R, typename M, typename Logit>   // logits per lane: experts c + 16 i, i < NPL
__device__ __forceinline__ void topk_of_rows(Logit logit, int E, int K, int renorm, int c, int (&my_e)[R], float (&my_w)[R],
                                             M& margin)
{
    const double NEG = -__builtin_huge_val();
    double v[R][NPL];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int i = 0; i < NPL; ++i) {
            const int e = c + 16 * i;
            v[r][i] = (e < E) ? logit(r, e) : NEG;
        }
    double esum[R];         // only without renormalisation: this lane's share of sum_e exp(z_e - z_max)
    double my_z[R], z_max[R], before_z[R];
    bool close[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        esum[r] = z_max[r] = before_z[r] = 0.0;
        my_z[r] = NEG;
        my_e[r] = 0;
        close[r] = false;
    }
    const int rounds = M::kCheck ? K + 1 : K;        // (the last of K + 1: what the K-th winner is ahead of)
    for (int j = 0; j < rounds; ++j) {
        // The largest logit, then the lowest of the experts that have it: a maximum is one instruction where a comparison
        // of (value, index) pairs is eight, and it does not wait for a condition.
        double bv[R];
        int be[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            double m[NPL];
#pragma unroll
            for (int i = 0; i < NPL; ++i) m[i] = v[r][i];
#pragma unroll
            for (int d = 1; d < NPL; d *= 2)
#pragma unroll
                for (int i = 0; i + d < NPL; i += 2 * d) m[i] = __builtin_fmax(m[i], m[i + d]);
            bv[r] = row_max(m[0]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            int e = kMaxExperts;
#pragma unroll
            for (int i = NPL - 1; i >= 0; --i) e = v[r][i] == bv[r] ? c + 16 * i : e;
            e = row_min(e);
            be[r] = e < E ? e : 0;       // (only if all that is left is NaN)
        }
        if (j == 0) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                z_max[r] = bv[r];
                if (!renorm) {
#pragma unroll
                    for (int i = 0; i < NPL; ++i)
                        if (c + 16 * i < E) esum[r] += exp(v[r][i] - bv[r]);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (M::kCheck) {
                // Each winner ahead of the next by more than both can move.  (A NaN is ahead of nothing.)
                const double room = 2.0 * margin.chain_error * margin.product[r] + 0x1p-48 * __builtin_fmax(__builtin_fabs(before_z[r]), __builtin_fabs(bv[r]));
                if (j > 0 && !(before_z[r] - bv[r] > room)) close[r] = true;
                before_z[r] = bv[r];
                if (j == K) continue;
            }
            if (c == j) { my_z[r] = bv[r]; my_e[r] = be[r]; }
#pragma unroll
            for (int i = 0; i < NPL; ++i) v[r][i] = be[r] == c + 16 * i ? NEG : v[r][i];
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const double p = (c < K) ? exp(my_z[r] - z_max[r]) : 0.0;
        double denom = renorm ? p : esum[r];
        denom = row_sum_step<kDppXor1>(denom);
        denom = row_sum_step<kDppXor2>(denom);
        denom = row_sum_step<kDppHalfMirror>(denom);
        denom = row_sum_step<kDppMirror>(denom);
        const double q = p / denom;
        my_w[r] = (float)q;
        if constexpr (M::kCheck) {
            // Without a rounding in the K logits q is the same number.  (Without renormalisation it has all E in it.)
            auto of_row = [](bool p) { return (uint32_t)(__ballot(p) >> (lane_id() & 48)) & 0xffffu; };
            const int how = renorm ? (c < K ? margin.rounds(r, my_e[r]) : 0) : 2;
            const uint32_t some = of_row(how > 0), any = of_row(how > 1);
            const double d = (any != 0 ? margin.chain_error : 8.0 * 1.03 * 0x1p-53) * margin.product[r];
            // Logits that move by d move ln q by at most 2 d.  The bias moves them by 2^-49 |z|, and the roundings of the differences,
            // exp, the sum and the quotient, on either side, come to less than 2^-52 (2 |z| + 2 |z_max| + 16).  Is the fp32 weight the
            // same at both ends?
            const double rel = 2.0 * d + 0x1p-47 * (1.0 + __builtin_fabs(my_z[r]) + __builtin_fabs(z_max[r]));
            const uint32_t moves = of_row(c < K && !((float)(q - q * rel) == (float)(q + q * rel)));
            // (a product of 0: a row of zeros or a router of zeros, whose logits are the bias in any order)
            margin.sure[r] = margin.product[r] == 0.0 || (!close[r] && (some == 0 || moves == 0));
        }
    }
}
template <int NPL, typename Logit>
__device__ __forceinline__ void topk_of_row(Logit logit, int E, int K, int renorm, int c, int& my_e, float& my_w)
{
    int e[1];
    float w[1];
    NoMargin none;
    topk_of_rows<NPL, 1>([&](int, int e) { return logit(e); }, E, K, renorm, c, e, w, none);
    my_e = e[0];
    my_w = w[0];
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
    topk_of_row<NPL>([&](int e) { return logits[tl * E + e]; }, E, K, renorm, c, my_e, my_w);
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
// Router and top-k of larger batches of bf16 rows (at most kExactMaxExperts experts, K <= 16): the logits are exact integer
// sums on the i8 matrix cores.
//
// The fp64 pass above is bound by the fp64 matrix pipe (two widenings beside every MFMA).  Here a row of x, and a row
// of w_router, becomes 32-bit fixed point under the row's own power of two, v = trunc(x 2^(156 - eb)) (eb: largest
// biased exponent of the row, so |v| < 2^30), and v is written in four balanced base-256 digits: the bytes of
// (v + 0x80808080) ^ 0x80808080.  A logit is then sum_ij 2^(8 (i + j)) sum_k d_i d_j, and every sum over k is a chain of
// v_mfma_i32_32x32x32_i8 that cannot overflow (7 sums for i + j = 0 .. 6, each at most 4 H 2^14 < 2^31).  Nothing is rounded
// until the 7 sums meet: one rounding to fp64, closer to the true sum than the fp64 chain's H of them, and the same
// whatever the tile, the order of the chain or the rest of the batch.
// The lowest digit of most values is zero (it is used by values 2^14 and more below their row's largest, one in 10^4 of
// normally distributed ones): a chunk of 32 k-values whose lowest digits are all zero on either side leaves
// those products out, which makes 10 of 16.
// A value with bits below the window (2^22 and more below the row's largest: one in 2 10^6 of normally distributed ones)
// leaves a remainder that the digits do not hold.  Such values of a row are listed, up to kStray of them, and their remainders
// times the other operand are added to the logit in fp64.
//
// The fp64 pass takes the sums in another order with a rounding at every step, so its logits are not the same bits, and a
// token must not change its experts or its weights with the size of its batch.  So a token's top-k is taken from these
// logits only where it is shown to be what the fp64 logits give.  A product is a multiple of 2^l, l the last places of the two
// rows' smallest values added up, so a sum below 2^(53 + l) is not rounded in any order, and |x|_2 |w|_2 bounds the sums (of all
// products, or of those of one partial sum of the chain).  The two logits before the bias are then at most this far apart:
//     0                   where no sum can be rounded: 96 % of the pairs of normally distributed rows at H = 2048,
//     8 |x| |w| 2^-53     where only those can that add up the 16 partial sums (6 additions on the way to a logit, and 1 rounding here),
//     off = (products of a partial sum + 40) |x| max |w| 2^-52    else (a unit in the last place for each addition),
// and the bias rounds either by 2^-53 of itself.  Where two of the first K + 1 logits are closer than that by the last line, or a
// weight so near the middle between two fp32 values that it could round the other way, the token is listed.  So are rows of
// x that are not held (more than kStray strays, infinities, NaN, a largest value outside 2^-40 .. 2^40), and all of the batch
// with a row of w_router that is not.  Listed tokens take the fp64 pass (route_listed_kernel), 16 at a time whichever block
// they come from: of normally distributed tokens one in 30000 at H = 2048, 128 experts (in 800 by the last line alone).
//
// A block takes 32 tokens and all experts, WE groups of 32; its waves are WE x WK: WK shares of the k-range, in each of
// them one wave per group; the WE waves of a share turn 32 tokens x 64 k-values at a time into digits (whole 128-byte
// lines, each value once) and hand them to each other through LDS, a step ahead of the MFMAs that use them.  w_router's
// digits come from a launch of their own (for several layers at once), laid out as the operands' registers.  The logits
// stay in LDS, where the top-k reads them.
// Measured, H = 2048, E = 128, top-8: moe_router_topk with the fp64 pass -> this one 55 -> 36 us at 4100 tokens, 97 -> 52 at 8200,
// of which the digits (of up to 8 layers) 5, this kernel 47 (8320 tokens; 44 without the rows' forms and the test of the winners),
// the empty list 4.5 (with a token on it 14).  What bounds it: the MFMAs alone take 10.5 us of the 24 of the k-loop; the rest is the
// 36 KB per step that a compute unit's address unit and L2 deliver (eight loads issued in a row, in place of one by one between
// the MFMAs, cost 6 us, the branches around four groups of MFMAs in place of one 5 us; the conversions are hidden).
// Every row listed (more than kStray values below the window in each of them): 141 us in all at 8320 tokens against 97.
// ----------------------------------------------------------------------------------------------
typedef int i32x4_t __attribute__((ext_vector_type(4)));
typedef int i32x16_t __attribute__((ext_vector_type(16)));
typedef uint16_t u16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

constexpr int kDigitK = 64;           // k-values per step: rows are padded to it with zeros
constexpr int kWindow = 22;           // exponents below the row's largest that the fixed point holds exactly
constexpr int kStray = 4;             // values of a row that may lie below it
constexpr int kHeld = 40;             // rows whose largest value is in 2^-40 .. 2^40: their squares stay in the fp32 range
constexpr uint32_t kBalance = 0x80808080u, kNoStray = 0xffffffffu;

// How a row is held: the biased exponent eb of its scale (-1: not at all); its 2-norm and the largest one of the values that belong
// to one partial sum of the fp64 chain (or a little more); all its values are multiples of 2^last (with strays: some small number).
struct RowHead {
    int eb;
    float norm, part;
    int last;
};
struct RowForm : RowHead {
    uint32_t stray[kStray];           // the k-values whose remainders the digits miss, in ascending order, kNoStray past the last
};
// 2^(156 - eb); any scale will do for a row that is not held
__device__ __forceinline__ float digit_scale(int eb) { return __uint_as_float((uint32_t)(283 - (eb < 0 ? 127 : eb)) << 23); }
// value = what the digits hold + remainder
__device__ __forceinline__ double digit_part(bf16_t v, int eb) { return (double)truncf(bf16_to_f32(v) * digit_scale(eb)) / digit_scale(eb); }
__device__ __forceinline__ double remainder_part(bf16_t v, int eb) { return (double)bf16_to_f32(v) - digit_part(v, eb); }

// The largest and the smallest non-zero magnitude of a row, as bf16 bits, gathered 8 values at a time (zero counts as
// 0xffff on the small side).
struct RowRange {
    u16x2_t top, low;
    __device__ __forceinline__ void clear()
    {
        top = u16x2_t{0, 0};
        low = u16x2_t{0xffff, 0xffff};
    }
    // returns sum + the squares of the values
    __device__ __forceinline__ float add(const u32x4_t& raw, float sum)
    {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u16x2_t m = __builtin_bit_cast(u16x2_t, raw[i] & 0x7fff7fffu);
            top = __builtin_elementwise_max(top, m);
            low = __builtin_elementwise_min(low, m - u16x2_t{1, 1});       // zero wraps to 0xffff
            const bf16x2_t v = __builtin_bit_cast(bf16x2_t, raw[i]);
            sum = __builtin_amdgcn_fdot2_f32_bf16(v, v, sum, false);
        }
        return sum;
    }
    // Over W neighbouring lanes that hold the row, of these sums of squares; strays: some value lies below the window.
    template <int W> __device__ __forceinline__ RowForm form(float squares, float part_squares, bool& strays) const
    {
        int hi = top[0] > top[1] ? top[0] : top[1], lo = low[0] < low[1] ? low[0] : low[1];
#pragma unroll
        for (int o = 1; o < W; o <<= 1) {
            const int h2 = __shfl_xor(hi, o, 64), l2 = __shfl_xor(lo, o, 64);
            hi = h2 > hi ? h2 : hi;
            lo = l2 < lo ? l2 : lo;
        }
        const int eb = hi == 0 ? 127 : hi >> 7;      // (a row of zeros: any)
        const int e_low = (lo + 1) >> 7;             // of the smallest value (or 512)
        strays = e_low < eb - kWindow;
        const bool held = eb >= 127 - kHeld && eb < 127 + kHeld;
        // (the sum of H <= 16384 squares in fp32 is right to a part in 2^9)
        RowForm f;
        f.eb = held ? eb : -1;
        f.norm = held ? 1.01f * sqrtf(squares) : 0.f;
        f.part = held ? 1.01f * sqrtf(part_squares) : 0.f;
        f.last = strays ? -512 : (hi == 0 ? 0 : e_low - 134);
#pragma unroll
        for (int i = 0; i < kStray; ++i) f.stray[i] = kNoStray;
        return f;
    }
};

// Lists the strays of a row of scale eb, or marks the row as not held.  Called by one whole wave; lane `owner`, which wrote the form,
// writes to it.  (Rare: short rather than fast.)
__device__ __forceinline__ void list_strays(const bf16_t* row, int H, int eb, int owner, RowForm* form)
{
    const int lane = lane_id();
    int n = 0;
#pragma unroll 1
    for (int k0 = 0; k0 < H && n <= kStray; k0 += 512) {
        const int k = k0 + lane * 8;
        u32x4_t raw = {0, 0, 0, 0};
        if (k < H) raw = *reinterpret_cast<const u32x4_t*>(row + k);
        uint32_t mine = 0;                // bit j: value k + j is a stray
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const uint32_t m = (raw[j / 2] >> (16 * (j & 1))) & 0x7fffu;
            if (m != 0 && (int)(m >> 7) < eb - kWindow) mine |= 1u << j;
        }
        unsigned long long hit = __ballot(mine != 0);
#pragma unroll 1
        while (hit) {
            const int from = __ffsll((long long)hit) - 1;
            uint32_t bits = (uint32_t)__builtin_amdgcn_readlane((int)mine, from);
#pragma unroll 1
            for (; bits; bits &= bits - 1, ++n)
                if (n < kStray && lane == owner) form->stray[n] = (uint32_t)(k0 + from * 8 + __ffs((int)bits) - 1);
            hit &= hit - 1;
        }
    }
    if (n > kStray && lane == owner) form->eb = -1;
}

// The digits of 8 consecutive values: digit p of values 0 .. 3 in d[p][0], of values 4 .. 7 in d[p][1].
__device__ __forceinline__ void digits_of_8(const u32x4_t& raw, float scale, uint32_t (&d)[4][2])
{
    uint32_t u[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        u[2 * i] = (uint32_t)(int)(__uint_as_float(raw[i] << 16) * scale) + kBalance;
        u[2 * i + 1] = (uint32_t)(int)(__uint_as_float(raw[i] & 0xffff0000u) * scale) + kBalance;
    }
#pragma unroll
    for (int g = 0; g < 2; ++g) {       // 4 x 4 bytes, transposed
        const uint32_t a = u[4 * g], b = u[4 * g + 1], c = u[4 * g + 2], e = u[4 * g + 3];
        const uint32_t ab01 = __builtin_amdgcn_perm(b, a, 0x05010400u), ce01 = __builtin_amdgcn_perm(e, c, 0x05010400u);
        const uint32_t ab23 = __builtin_amdgcn_perm(b, a, 0x07030602u), ce23 = __builtin_amdgcn_perm(e, c, 0x07030602u);
        d[0][g] = __builtin_amdgcn_perm(ce01, ab01, 0x05040100u) ^ kBalance;
        d[1][g] = __builtin_amdgcn_perm(ce01, ab01, 0x07060302u) ^ kBalance;
        d[2][g] = __builtin_amdgcn_perm(ce23, ab23, 0x05040100u) ^ kBalance;
        d[3][g] = __builtin_amdgcn_perm(ce23, ab23, 0x07060302u) ^ kBalance;
    }
}

// Digits of w_router, in the order in which the waves below load them: [64 k-values][group of 32 experts][32 k-values][digit]
// [lane][16 bytes], lane (r, q) = expert r, k-values 16 q .. + 15.  A block per expert (the last group is padded with rows
// of zeros) and layer.
constexpr int kPrepThreads = 128;
__global__ __launch_bounds__(kPrepThreads) void router_digits_kernel(RouterWeights w, int H, int E, uint8_t* digits,
                                                                      int64_t layer_bytes, RowForm* forms, int32_t* zero_buf,
                                                                      int64_t zero_n)
{
    __shared__ int s_hi[kPrepThreads / 64], s_lo[kPrepThreads / 64];
    __shared__ float s_sq[kPrepThreads / 64][16];
    __shared__ RowForm s_form;
    // side job: clear the counters of the layers' routing
    for (int64_t i = ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kPrepThreads + threadIdx.x; i < zero_n;
         i += (int64_t)gridDim.x * gridDim.y * kPrepThreads)
        zero_buf[i] = 0;
    const int e = (int)blockIdx.x, layer = (int)blockIdx.y, groups = (int)gridDim.x / 32;
    const bf16_t* row = static_cast<const bf16_t*>(w.p[layer]) + (int64_t)(e < E ? e : 0) * H;
    const int pieces = e < E ? H / 8 : 0;
    const u32x4_t zero = {0, 0, 0, 0};
    RowRange range;
    range.clear();
    float sq = 0.f;                      // all of one partial sum: piece p is of chunk p / 4, which is of partial sum p / 4 % 16
    static_assert(kPrepThreads == 128, "two waves' ranges meet here; a thread's pieces are 32 chunks apart");
    for (int p = threadIdx.x; p < pieces; p += kPrepThreads) sq = range.add(*reinterpret_cast<const u32x4_t*>(row + p * 8), sq);
    int hi = range.top[0] > range.top[1] ? range.top[0] : range.top[1];
    int lo = range.low[0] < range.low[1] ? range.low[0] : range.low[1];
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int h2 = __shfl_xor(hi, o, 64), l2 = __shfl_xor(lo, o, 64);
        hi = h2 > hi ? h2 : hi;
        lo = l2 < lo ? l2 : lo;
    }
    sq += __shfl_xor(sq, 1, 64);
    sq += __shfl_xor(sq, 2, 64);
    if ((threadIdx.x & 3) == 0) s_sq[threadIdx.x >> 6][(threadIdx.x & 63) >> 2] = sq;
    if ((threadIdx.x & 63) == 0) {
        s_hi[threadIdx.x >> 6] = hi;
        s_lo[threadIdx.x >> 6] = lo;
    }
    __syncthreads();
    range.top = u16x2_t{(uint16_t)s_hi[0], (uint16_t)s_hi[1]};
    range.low = u16x2_t{(uint16_t)s_lo[0], (uint16_t)s_lo[1]};
    float squares = 0.f, part_squares = 0.f;
#pragma unroll
    for (int p = 0; p < 16; ++p) {
        const float of_p = s_sq[0][p] + s_sq[1][p];
        squares += of_p;
        part_squares = of_p > part_squares ? of_p : part_squares;
    }
    bool strays;
    const RowForm form = range.form<1>(squares, part_squares, strays);
    const int eb = form.eb;
    if (threadIdx.x < 64) {
        if (threadIdx.x == 0) s_form = form;
        if (strays && eb >= 0) list_strays(row, H, eb, 0, &s_form);
        if (threadIdx.x == 0) forms[layer * (int)gridDim.x + e] = s_form;
    }
    const float scale = digit_scale(eb);
    const int steps = (H + kDigitK - 1) / kDigitK;
    for (int i = threadIdx.x; i < steps * 4; i += kPrepThreads) {        // 16 k-values: step i / 4, half (i / 2) % 2, q = i % 2
        uint32_t a[4][2], b[4][2];
        digits_of_8(2 * i < pieces ? *reinterpret_cast<const u32x4_t*>(row + i * 16) : zero, scale, a);
        digits_of_8(2 * i + 1 < pieces ? *reinterpret_cast<const u32x4_t*>(row + i * 16 + 8) : zero, scale, b);
        uint8_t* out = digits + layer * layer_bytes + (((int64_t)(i >> 2) * groups + e / 32) * 2 + ((i >> 1) & 1)) * 4096 +
                       ((i & 1) * 32 + (e & 31)) * 16;
#pragma unroll
        for (int p = 0; p < 4; ++p) *reinterpret_cast<u32x4_t*>(out + p * 1024) = u32x4_t{a[p][0], a[p][1], b[p][0], b[p][1]};
    }
}

// sum_s 2^(8 s) S[s], rounded once: either half is exact (|S[s]| <= 4 H 2^14 and, its digits being at most 64, |S[6]| <= H 2^12,
// H <= 16384: the halves stay below 2^52)
__device__ __forceinline__ double join_sums(const int (&s)[7])
{
    double hi = (double)s[6], lo = (double)s[2];
    hi = __builtin_fma(hi, 256.0, (double)s[5]);
    hi = __builtin_fma(hi, 256.0, (double)s[4]);
    hi = __builtin_fma(hi, 256.0, (double)s[3]);
    lo = __builtin_fma(lo, 256.0, (double)s[1]);
    lo = __builtin_fma(lo, 256.0, (double)s[0]);
    return __builtin_fma(hi, 16777216.0, lo);
}

// LDS traffic of the block is visible to all its waves; loads from global memory stay in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int WE, int WK>
__global__ __launch_bounds__(WE * WK * 64, 2) void route_exact_kernel(
    RowSrc x, int64_t n_tok, int H, const bf16_t* __restrict__ wr, const float* __restrict__ bias, int E, int K, int renorm,
    const uint8_t* __restrict__ digits, const RowForm* __restrict__ forms, double chain_error, int32_t* __restrict__ idx,
    float* __restrict__ w, int32_t* __restrict__ tile_hist, int32_t* n_listed, int32_t* __restrict__ listed)
{
    constexpr int NW = WE * WK, NT = NW * 64;    // waves, threads
    constexpr int XL = 4 / WE;                   // 16-byte loads per lane and step: 32 rows x 128 bytes over WE waves
    constexpr int SHARE = 2 * 8192;              // digits of one share of the k-range: [buffer][digit][32 rows][64 bytes]
    constexpr int SUMS = (WK / 2) * WE * 28672;  // then: the sums of half the waves
    constexpr int ZLD = WE * 32 + 1, LOGITS = 32 * ZLD * 8;      // then: the logits
    constexpr int LDS = SUMS > WK * SHARE ? SUMS : WK * SHARE;
    __shared__ __attribute__((aligned(16))) uint8_t lds[LDS > LOGITS ? LDS : LOGITS];
    __shared__ RowForm form[32];                 // of the token rows
    __shared__ RowHead head[WE * 32];            // of the experts
    __shared__ int32_t hist[2][WE * 32];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int we = wave % WE, wk = wave / WE;
    const int64_t t0 = (int64_t)blockIdx.x * 32;
    const int groups = (E + 31) / 32;
    auto token_row = [&](int r) {
        const int64_t t = t0 + r < n_tok ? t0 + r : n_tok - 1;
        return row_ptr<bf16_t>(x, t, H);
    };
    const int pieces = H / 8;                                // 16-byte pieces of a row

    // ---- w_router: two steps of digits in registers, the next one's on their way ----
    const int steps = (H + kDigitK - 1) / kDigitK;
    const int mine = (steps + WK - 1) / WK;                  // steps of every share (its last ones may be empty: zeros)
    const uint8_t* w_src = digits + (int64_t)(we < groups ? we : groups - 1) * 8192 + lane * 16;
    i32x4_t wd[2][2][4];
    auto load_w = [&](int i, int buf) {
        const int c = i * WK + wk;
        const uint8_t* p = w_src + (int64_t)(c < steps ? c : steps - 1) * groups * 8192;
#pragma unroll
        for (int d = 0; d < 8; ++d) wd[buf][d / 4][d % 4] = *reinterpret_cast<const i32x4_t*>(p + d * 1024);
    };

    // ---- the form of the token rows: NT / 32 neighbouring lanes per row (the experts' forms come in meanwhile) ----
    const RowHead form_a = forms[lane < E ? lane : E - 1], form_b = forms[lane + 64 < E ? lane + 64 : E - 1];
    if (wave == 0) {
        head[lane] = form_a;
        if (WE > 2) head[lane + 64] = form_b;
    }
    for (int i = tid; i < 2 * WE * 32; i += NT) (&hist[0][0])[i] = 0;
    {
        constexpr int W = NT / 32, AHEAD = 8;
        constexpr int PARTS = 64 / W;            // partial sums a lane's pieces fall into: every PARTS-th piece into the same
        static_assert(AHEAD % PARTS == 0, "the pieces of a round begin with the same partial sum");
        const bf16_t* row = token_row(tid / W);
        RowRange range;
        range.clear();
        float sq[PARTS];
#pragma unroll
        for (int i = 0; i < PARTS; ++i) sq[i] = 0.f;
#pragma unroll 1
        for (int p0 = tid % W; p0 < pieces; p0 += AHEAD * W) {
            u32x4_t v[AHEAD];
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                const int p = p0 + i * W < pieces ? p0 + i * W : pieces - 1;      // (a piece may count twice)
                v[i] = *reinterpret_cast<const u32x4_t*>(row + p * 8);
            }
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) sq[i % PARTS] = range.add(v[i], sq[i % PARTS]);
        }
        float squares = 0.f, part_squares = 0.f;
#pragma unroll
        for (int i = 0; i < PARTS; ++i) {        // four neighbouring lanes have a chunk
            sq[i] += __shfl_xor(sq[i], 1, 64);
            sq[i] += __shfl_xor(sq[i], 2, 64);
            squares += sq[i];
            part_squares = sq[i] > part_squares ? sq[i] : part_squares;
        }
#pragma unroll
        for (int o = 4; o < W; o <<= 1) {
            squares += __shfl_xor(squares, o, 64);
            const float other = __shfl_xor(part_squares, o, 64);
            part_squares = other > part_squares ? other : part_squares;
        }
        bool strays;
        const RowForm f = range.form<W>(squares, part_squares, strays);
        if (tid % W == 0) form[tid / W] = f;
        // (a row's lanes are neighbours: each wave lists the strays of its own rows)
        unsigned long long left = __ballot(strays && f.eb >= 0 && tid % W == 0);
#pragma unroll 1
        for (; left != 0; left &= left - 1) {
            const int from = __ffsll((long long)left) - 1, r = (tid - lane + from) / W;
            list_strays(token_row(r), H, __builtin_amdgcn_readlane(f.eb, from), from, &form[r]);
        }
    }
    __syncthreads();

    // ---- nothing to do here for a block that holds no row, or with an expert that is not held ----
    const int rows = rows_left(t0, n_tok, 32);
    if (__ballot(form_a.eb < 0 || form_b.eb < 0) != 0 || __ballot(lane < rows && form[lane & 31].eb >= 0) == 0) {
        if (wave == 0) {
            int32_t at = 0;
            if (lane == 0) at = atomicAdd(n_listed, rows);
            at = __builtin_amdgcn_readfirstlane(at);
            if (lane < rows) listed[at + lane] = (int32_t)(t0 + lane);
        }
        return;
    }
    float w_norm = form_a.norm > form_b.norm ? form_a.norm : form_b.norm;      // the largest of all experts'
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float other = __shfl_xor(w_norm, o, 64);
        w_norm = other > w_norm ? other : w_norm;
    }

    // ---- x: load p of this wave covers rows (we + WE p) * 8 .. + 7 of the tile, lane = (row, 16-byte piece of the step) ----
    const int piece = lane & 7;
    const bf16_t* x_src[XL];
    float x_scale[XL];
    uint32_t x_dst[XL];
    // 16-byte slot c of a row's 64 digit bytes sits at slot c ^ f(row): 8, and 16, consecutive rows then fall into
    // different banks
    auto slot = [](int r, int c) { return (uint32_t)(r * 64 + ((c ^ (((r >> 1) & 1) * 2) ^ ((r >> 2) & 3)) << 4)); };
#pragma unroll
    for (int p = 0; p < XL; ++p) {
        const int r = (we + WE * p) * 8 + (lane >> 3);
        x_src[p] = token_row(r);
        x_scale[p] = digit_scale(form[r].eb);
        x_dst[p] = slot(r, piece >> 1) + (piece & 1) * 8;
    }
    u32x4_t xr[2][XL];                   // (issued in front of the step's weights, so that waiting for one is not waiting for the other)
    auto load_x = [&](int i, int buf) {
        const int at = (i * WK + wk) * 8 + piece;
        // (past the row: a valid piece, turned into zeros below; a load under a condition would make the compiler wait for
        // every load in flight)
        const int from = at < pieces ? at : pieces - 1;
#pragma unroll
        for (int p = 0; p < XL; ++p) xr[buf][p] = *reinterpret_cast<const u32x4_t*>(x_src[p] + from * 8);
    };
    auto store_digits = [&](int i, int buf) {                // of this share's step i
        const bool in = (i * WK + wk) * 8 + piece < pieces;
        uint8_t* dig = lds + wk * SHARE + (i & 1) * 8192;
#pragma unroll
        for (int p = 0; p < XL; ++p) {
            uint32_t d[4][2];
            digits_of_8(xr[buf][p], in ? x_scale[p] : 0.f, d);
#pragma unroll
            for (int q = 0; q < 4; ++q) *reinterpret_cast<uint2*>(dig + q * 2048 + x_dst[p]) = make_uint2(d[q][0], d[q][1]);
        }
    };
    const int fr = lane & 31, fq = lane >> 5;

    i32x16_t acc[7];
#pragma unroll
    for (int s = 0; s < 7; ++s)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[s][v] = 0;
    auto step = [&](int i, auto buf_const) {
        constexpr int BUF = decltype(buf_const)::value;
        lds_barrier();                   // the digits of step i are there, and those of step i - 1 have been read
        load_x(i + 2, BUF);
        load_w(i + 1, BUF ^ 1);
        const uint8_t* dig = lds + wk * SHARE + (i & 1) * 8192;
        i32x4_t xd[2][4];
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int d = 0; d < 4; ++d) xd[half][d] = *reinterpret_cast<const i32x4_t*>(dig + d * 2048 + slot(fr, half * 2 + fq));
        // expert rows as the MFMA's row operand: a lane ends up with 4 consecutive experts of one token
        auto multiply = [&](int half, int a, int b) {
            acc[a + b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wd[BUF][half][a], xd[half][b], acc[a + b], 0, 0, 0);
        };
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            // (neighbours in this order belong to different sums)
            multiply(half, 3, 3); multiply(half, 1, 1); multiply(half, 3, 2); multiply(half, 1, 2); multiply(half, 1, 3);
            multiply(half, 2, 3); multiply(half, 2, 1); multiply(half, 2, 2); multiply(half, 3, 1);
        }
        auto any_of = [](const i32x4_t& d) { return __ballot((d[0] | d[1] | d[2] | d[3]) != 0) != 0; };
        // bits 0, 1: lowest digits of the weights' halves that are not zero; 2, 3: of x's
        const int low = (any_of(wd[BUF][0][0]) ? 1 : 0) | (any_of(wd[BUF][1][0]) ? 2 : 0) | (any_of(xd[0][0]) ? 4 : 0) |
                        (any_of(xd[1][0]) ? 8 : 0);
        store_digits(i + 1, BUF ^ 1);    // (past the last step: zeros nobody reads)
        // The loads one by one between the MFMAs: a wave issues in order, and eight loads in a row keep its MFMAs waiting
        // for the address unit, which takes 16 clocks of each of the four waves' loads.
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);           // LDS reads of the first half
#pragma unroll
        for (int n = 0; n < 9; ++n) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);       // one MFMA
            if (n < 8 + XL) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // one global load
            if (n < 4) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
        if (__builtin_expect(low != 0, 0)) {
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const bool w_low = (low >> half & 1) != 0, x_low = (low >> half & 4) != 0;
                if (w_low) { multiply(half, 0, 1); multiply(half, 0, 2); multiply(half, 0, 3); }
                if (x_low) { multiply(half, 1, 0); multiply(half, 2, 0); multiply(half, 3, 0); }
                if (w_low && x_low) multiply(half, 0, 0);
            }
        }
    };
    load_x(0, 0);
    load_x(1, 1);
    load_w(0, 0);                        // (in the loop's order: the compiler's waits in the loop allow for what comes before it)
    store_digits(0, 0);
#pragma unroll 1
    for (int i = 0; i < mine; i += 2) {
        step(i, std::integral_constant<int, 0>{});
        step(i + 1, std::integral_constant<int, 1>{});
    }

    // ---- the shares' sums meet, the upper half of them handing theirs to the lower half ----
#pragma unroll
    for (int half = WK / 2; half >= 1; half /= 2) {
        __syncthreads();
        if (wk >= half && wk < 2 * half) {
            i32x4_t* to = reinterpret_cast<i32x4_t*>(lds) + ((wk - half) * WE + we) * 1792 + lane;
#pragma unroll
            for (int s = 0; s < 7; ++s)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    to[(s * 4 + v) * 64] = i32x4_t{acc[s][4 * v], acc[s][4 * v + 1], acc[s][4 * v + 2], acc[s][4 * v + 3]};
        }
        __syncthreads();
        if (wk < half) {
            const i32x4_t* from = reinterpret_cast<const i32x4_t*>(lds) + (wk * WE + we) * 1792 + lane;
#pragma unroll
            for (int s = 0; s < 7; ++s)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const i32x4_t o = from[(s * 4 + v) * 64];
#pragma unroll
                    for (int u = 0; u < 4; ++u) acc[s][4 * v + u] += o[u];
                }
        }
    }
    __syncthreads();
    double* const z = reinterpret_cast<double*>(lds);        // [32][ZLD]
    const int own = we * 32 + fr < E ? we * 32 + fr : E - 1;             // lane l knows expert l % 32 of its wave's group
    const RowForm own_form = forms[own];
    const bool real = lane < 32 && we * 32 + fr < E;
    if (wk == 0) {
        // accumulator element v: expert (v / 4) * 8 + fq * 4 + v % 4 of the group, token fr
        const int xe = form[fr].eb;
        const float own_bias = bias ? bias[own] : 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int e = (v >> 2) * 8 + fq * 4 + (v & 3);
            const int s[7] = {acc[0][v], acc[1][v], acc[2][v], acc[3][v], acc[4][v], acc[5][v], acc[6][v]};
            // (exponents of 29 and more: the power of two is a normal number; of rows that are not held, anything)
            const double unit = __hiloint2double((1023 + xe + __shfl(own_form.eb, e, 64) - 312) << 20, 0);
            z[fr * ZLD + we * 32 + e] = join_sums(s) * unit + (double)__shfl(own_bias, e, 64);
        }
    }
    __syncthreads();
    // ---- remainders: of x first, then of w_router, in ascending k (bit = token row, or expert of this wave's group) ----
    const uint32_t t_stray = (uint32_t)__ballot(lane < rows && form[fr].eb >= 0 && form[fr].stray[0] != kNoStray);
    if (t_stray != 0) {                  // (the same in every wave)
#pragma unroll 1
        for (uint32_t left = t_stray; left != 0; left &= left - 1) {
            const int r = __ffs((int)left) - 1;
            if (r % NW != wave) continue;
#pragma unroll 1
            for (int i = 0; i < kStray; ++i) {
                const uint32_t k = form[r].stray[i];
                if (k == kNoStray) break;
                const double rest = remainder_part(token_row(r)[k], form[r].eb);
                for (int e = lane; e < E; e += 64) z[r * ZLD + e] += rest * (double)bf16_to_f32(wr[(int64_t)e * H + k]);
            }
        }
        __syncthreads();
    }
    if (wk == 0) {
#pragma unroll 1
        for (uint32_t left = (uint32_t)__ballot(real && own_form.stray[0] != kNoStray); left != 0; left &= left - 1) {
            const int e = __ffs((int)left) - 1, eb = __builtin_amdgcn_readlane(own_form.eb, e);
            const bf16_t* w_row = wr + (int64_t)(we * 32 + e) * H;
#pragma unroll
            for (int i = 0; i < kStray; ++i) {
                const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)own_form.stray[i], e);
                if (k != kNoStray && lane < 32 && form[fr].eb >= 0)
                    z[fr * ZLD + we * 32 + e] += digit_part(token_row(fr)[k], form[fr].eb) * remainder_part(w_row[k], eb);
            }
        }
    }
    __syncthreads();

    // ---- top-k: 16 lanes per token ----
    const int64_t tile0 = t0 * K / kPermTile;        // 32 tokens x K <= 512 assignments touch at most two permutation tiles
    const int c = lane & 15;
    constexpr int AT_ONCE = 512 / NT;                // rows tid / 16, tid / 16 + NT / 16, ...
    const double* zs[AT_ONCE];
    int my_e[AT_ONCE];
    float my_w[AT_ONCE];
    Margin<AT_ONCE, RowHead> margin;
    bool held[AT_ONCE];
#pragma unroll
    for (int u = 0; u < AT_ONCE; ++u) {
        const int r = tid / 16 + u * (NT / 16);
        zs[u] = z + r * ZLD;
        margin.row[u] = form[r];
        margin.product[u] = (double)w_norm * (double)form[r].norm;
        held[u] = form[r].eb >= 0;
    }
    margin.experts = head;
    margin.chain_error = chain_error;
    topk_of_rows<WE * 2, AT_ONCE>([&](int u, int e) { return zs[u][e]; }, E, K, renorm, c, my_e, my_w, margin);
#pragma unroll
    for (int u = 0; u < AT_ONCE; ++u) {
        const int64_t t = t0 + tid / 16 + u * (NT / 16);
        const bool sure = held[u] && margin.sure[u];
        const unsigned long long open = __ballot(t < n_tok && c == 0 && !sure);
        if (open != 0) {                 // (rare) on the list
            int32_t at = 0;
            if (lane == 0) at = atomicAdd(n_listed, (int32_t)__popcll(open));
            at = __builtin_amdgcn_readfirstlane(at) + (int32_t)__popcll(open & ((1ull << lane) - 1));
            if (t < n_tok && c == 0 && !sure) listed[at] = (int32_t)t;
        }
        if (t < n_tok && c < K && sure) {
            idx[t * K + c] = my_e[u];
            w[t * K + c] = my_w[u];
            if (tile_hist) atomicAdd(&hist[(t * K + c) / kPermTile - tile0][my_e[u]], 1);
        }
    }
    if (tile_hist) {
        __syncthreads();
        for (int i = tid; i < 2 * E; i += NT) {
            const int cnt = hist[i / E][i % E];
            if (cnt) atomicAdd(&tile_hist[(tile0 + i / E) * E + i % E], cnt);
        }
    }
}

// The tokens that route_exact_kernel listed, 16 to a tile: block (g, e) takes the logits of tiles g, g + gridDim.x, ... and
// 16 experts from the fp64 pass (the same bits as in any other launch); the last block of a tile does its top-k.
// tickets: one per 16 tokens of the batch, zero at the start.
template <int NPL>
__global__ __launch_bounds__(256, 3) void route_listed_kernel(RowSrc x, int H, const bf16_t* __restrict__ wr,
                                                           const float* __restrict__ bias, int E, int K, int renorm,
                                                           const int32_t* __restrict__ n_listed,
                                                           const int32_t* __restrict__ listed, double* logits, uint32_t* tickets,
                                                           int32_t* __restrict__ idx, float* __restrict__ w,
                                                           int32_t* __restrict__ tile_hist)
{
    __shared__ int32_t flag;
    const int n = *n_listed, e0 = (int)blockIdx.y * 16;
    for (int64_t at = (int64_t)blockIdx.x * 16; at < n; at += (int64_t)gridDim.x * 16) {
        const int rows = rows_left(at, n, 16);
        logits_tile<bf16_t, 4>([&](int i) { return row_ptr<bf16_t>(x, listed[at + (i < rows ? i : rows - 1)], H); }, rows, H, wr,
                               bias, E, e0, [&](int i, int j, double z) { store_shared(logits + (at + i) * E + e0 + j, z); });
        if (last_to_arrive(tickets + at / 16, gridDim.y, &flag)) {
            const int c = (int)threadIdx.x & 15, row = (int)threadIdx.x >> 4;
            int e;
            float wt;
            const double* z = logits + (at + (row < rows ? row : rows - 1)) * E;
            topk_of_row<NPL>([&](int e) { return load_shared(z + e); }, E, K, renorm, c, e, wt);
            if (row < rows && c < K) {
                const int64_t f = (int64_t)listed[at + row] * K + c;
                idx[f] = e;
                w[f] = wt;
                if (tile_hist) atomicAdd(&tile_hist[f / kPermTile * E + e], 1);
            }
        }
        __syncthreads();                 // the tile's LDS is used again
    }
}

// ----------------------------------------------------------------------------------------------
// Router, top-k and permutation of a decode batch (at most kSmallTokens tokens, K <= 16) in one launch.
//
// On such a batch the three kernels are a chain of launches with almost nothing in each.  Here the blocks of a 16-token tile
// compute its logits and take a ticket; the one that draws the last finds them written and does the top-k of the tile; of
// those blocks, the one that draws the last ticket of the batch does the permutation (no block ever waits for another).
//
// What bounds it are three chains, one behind the other: the fp64 matrix pipes, instruction fetches, and the trips to the level
// that all blocks see.  (1) A tile of 16 x 16 logits is H / 4 MFMAs of 64 clocks, whatever the number of tokens, so it is cut into
// the kClasses sums of four partial sums each that the tree of a logit ends in (see logits_tile), a block each: its four
// summing waves hold one partial sum each, one to a SIMD.  A class has its own value in memory, [class][token][expert]; who does
// the top-k adds the four in order, the same bits.  (2) Code that runs once comes in at the speed of its misses, about a
// microsecond per KB, so loops are kept loops (the operands of a wave's chunks wait in LDS, not in as many registers), and
// the first of the other waves walks through the top-k once, on whatever the buffers hold, while the sums are formed: its
// instructions are there when they are needed.  (3) What crosses between blocks goes past the XCD's caches by
// itself (store_shared, load_shared): a fence would write back and drop the whole L2, 2 us with a few blocks and 15 us with a
// hundred.  Every last drawer puts its counter back to zero.
//
// Measured with clocks in the kernel, us from its start until the sums are stored, the last ticket is drawn, the winners are known, the
// end; 128 experts, H = 2048, top-8: one token 3.3, 4.0, 6.5, 8.0, 32 tokens 3.7, 4.8, 8.5, 11.2.  With one block to a tile, no walk,
// unrolled loops and rounds that compare (value, index) pairs: one token 6.5, 7.5, 11, 12.7, 32 tokens 7.9, 8.9, 12.4, 15.6; a pass of
// four layers over one token 162 us then, 147 now.
//
// Where a tile is not cut, route_small_tile_kernel has a block of 16 waves for it, one partial sum to a wave, and its code is not walked:
// that is the shorter way where the rows are short (the MFMAs are soon done, the walk is not), where there are many experts (the
// last block of a tile reads kClasses times as many sums) and where the blocks would not all find a compute unit.  This kernel / that one,
// us (kernel trace, caches as a pass leaves them), top-8, bf16: 64 experts, 16 tokens, H = 512 9.2 / 8.4, 1024 10.1 / 10.2, 2048 10.8 / 13.3;
// 128 experts, 16 tokens, 512 10.1 / 8.7, 1024 10.8 / 10.6, 2048 11.0 / 12.8, 128 tokens, 1024 13.6 / 12.0, 2048 14.3 / 14.7, 4096 16.7 / 19.5;
// 256 experts, 16 tokens, 1024 14.1 / 11.9, 2048 14.0 / 14.7, 64 tokens, 2048 17.5 / 16.4, 4096 19.8 / 20.8; with four classes to a block,
// 256 tokens, 2048 27.1 / 18.8, 4096 36.6 / 24.1; 128 experts, 200 tokens, two classes, 2880 19.1 / 18.0.  fp32: 128 experts, 16 tokens, 256
// 11.1 / 8.9, 1024 10.7 / 11.5, 2048 11.9 / 18.8, 200 tokens, two classes, 2048 18.9 / 20.9.
//
// A token's experts are distinct as long as K of its logits are finite; the stable rank of an assignment inside its expert is then the
// number of earlier tokens that chose the expert: one bit per token and expert in LDS, counted with popcounts.  A bit that is set twice
// (a removed expert and one with a logit of -infinity compare equal, NaN compares with nothing) sends the batch to a count of
// the earlier assignments one by one.
// ----------------------------------------------------------------------------------------------
constexpr int kClasses = 4;
static_assert(kSmallSumBytes == kClasses * (int)sizeof(double), "a logit's sums");
constexpr int kSmallWaves = 8, kSumWaves = 4, kTileWaves = 16;
constexpr int kSmallWords = kSmallTokens / 64;

// The choices of a batch, and its permutation by one block.
struct SmallLists {
    unsigned long long chosen[kSmallExperts][kSmallWords];      // bit t of an expert: token t chose it
    int32_t count[kSmallExperts], start[kSmallExperts];
    uint8_t expert_of[kSmallTokens * 16];
    int32_t twice;
    static_assert(kSmallExperts <= 256, "an expert is one byte of expert_of");

    // by n threads, of which this is thread i
    __device__ __forceinline__ void clear(int E, int i, int n)
    {
        for (int j = i; j < E * kSmallWords; j += n) (&chosen[0][0])[j] = 0ull;
        for (int j = i; j < E; j += n) count[j] = 0;
        if (i == 0) twice = 0;
    }

    // single: expert_of holds the choices already (idx otherwise)
    template <int NT>
    __device__ __forceinline__ void permute(const int32_t* idx, bool single, int n_tok, int E, int K, uint32_t k_inverse,
                                            int32_t* __restrict__ offsets, int32_t* __restrict__ perm, int32_t* __restrict__ inv,
                                            unsigned long long* __restrict__ active_total)
    {
        const int tid = threadIdx.x, lane = tid & 63, A = n_tok * K;
        auto token_of = [&](int f) { return (int)((uint32_t)f * k_inverse >> 16); };      // f / K: k_inverse = ceil(2^16 / K)
        if (!single) {
            constexpr int PER = kSmallTokens * 16 / NT;            // assignments per thread, at most
            int32_t my_e[PER];
#pragma unroll
            for (int p = 0; p < PER; ++p) my_e[p] = p * NT + tid < A ? load_shared(idx + p * NT + tid) : 0;
#pragma unroll
            for (int p = 0; p < PER; ++p) expert_of[p * NT + tid] = (uint8_t)my_e[p];
            // (a thread reads its own)
        }
#pragma unroll 1
        for (int f = tid; f < A; f += NT) {
            const int t = token_of(f), e = expert_of[f];
            const unsigned long long bit = 1ull << (t & 63);
            if (atomicOr(&chosen[e][t >> 6], bit) & bit) twice = 1;
            atomicAdd(&count[e], 1);
        }
        __syncthreads();
        // exclusive scan of the expert counts by wave 0: lane l owns experts [4 l, 4 l + 4)
        if (tid < 64) {
            constexpr int EPL = kSmallExperts / 64;
            int cnt[EPL], sum = 0, act = 0;
#pragma unroll
            for (int i = 0; i < EPL; ++i) {
                const int e = lane * EPL + i;
                cnt[i] = e < E ? count[e] : 0;
                sum += cnt[i];
                act += (int)__popcll(__ballot(cnt[i] > 0));
            }
            int run = wave_scan(sum) - sum;
#pragma unroll
            for (int i = 0; i < EPL; ++i) {
                const int e = lane * EPL + i;
                if (e <= E) offsets[e] = run;       // (lanes behind the experts hold the total: the first of them has entry E)
                if (e < E) start[e] = run;
                run += cnt[i];
            }
            if (lane == 63 && E == kSmallExperts) offsets[E] = run;
            if (lane == 0) atomicAdd(active_total, (unsigned long long)act);
        }
        __syncthreads();
        if (__builtin_expect(twice == 0, 1)) {
#pragma unroll 1
            for (int f = tid; f < A; f += NT) {
                const int t = token_of(f), e = expert_of[f];
                int pos = start[e] + (int)__popcll(chosen[e][t >> 6] & ((1ull << (t & 63)) - 1));
#pragma unroll 1
                for (int j = 0; j < t >> 6; ++j) pos += (int)__popcll(chosen[e][j]);
                perm[pos] = f;
                inv[f] = pos;
            }
        } else {
#pragma unroll 1
            for (int f = tid; f < A; f += NT) {
                const int e = expert_of[f];
                int pos = start[e];
                for (int g = 0; g < f; ++g) pos += expert_of[g] == e;
                perm[pos] = f;
                inv[f] = pos;
            }
        }
    }
};

// One partial sum (p of 16) of a 16 x 16 tile of logits by a wave: chunks p, p + 16, ... of the rows, a group of them at a
// time.  x_row and w_row: the lane's rows (lane % 16); stage: the wave's LDS, 1 KB per load and chunk of a group.
template <typename T, int GROUP>
__device__ __forceinline__ double4_t partial_sum(const T* x_row, const T* w_row, int H, int p, char* stage)
{
    constexpr int LOADS = (int)sizeof(T) / 2;        // 16-byte loads for the lane's 8 values of a chunk
    constexpr int PER = 16 / (int)sizeof(T);         // values in one
    const int lane = lane_id(), q = lane >> 4;
    const int n_whole = H / 32, mine = n_whole > p ? (n_whole - p + 15) / 16 : 0;
    const char* const own = stage + lane * 16;
    double4_t acc = {0.0, 0.0, 0.0, 0.0};
    auto multiply = [&](auto value) {        // value(operand, j): the j-th of the lane's 8 values
#pragma unroll
        for (int j = 0; j < 8; ++j) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(value(0, j), value(1, j), acc, 0, 0, 0);
    };
#pragma unroll 1
    for (int i0 = 0; i0 < mine; i0 += GROUP) {
        const int n = mine - i0 < GROUP ? mine - i0 : GROUP;
#pragma unroll 1
        for (int i = 0; i < n; ++i) {
            const int k = (p + 16 * (i0 + i)) * 32 + q * 8;
#pragma unroll
            for (int l = 0; l < LOADS; ++l) {
                char* const to = stage + (i * 2 * LOADS + l) * 1024;
                __builtin_amdgcn_global_load_lds((glb_ptr_t*)(x_row + k + l * PER), (lds_ptr_t*)to, 16, 0, 0);
                __builtin_amdgcn_global_load_lds((glb_ptr_t*)(w_row + k + l * PER), (lds_ptr_t*)(to + LOADS * 1024), 16, 0, 0);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll 1
        for (int i = 0; i < n; ++i) {
            vec8<T> o[2];
#pragma unroll
            for (int x = 0; x < 2; ++x) o[x].load_lds(own + (i * 2 + x) * LOADS * 1024);
            multiply([&](int x, int j) { return o[x].get(j); });
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // (the stage is filled again)
    }
    if (H % 32 != 0 && p == n_whole % 16) {      // the row's partial chunk: lanes past the end feed zeros
        const int k = n_whole * 32 + q * 8;
        vec8<T> o[2];
        o[0].zero();
        o[1].zero();
        if (k < H) {
            o[0].load(x_row + k);
            o[1].load(w_row + k);
        }
        multiply([&](int x, int j) { return o[x].get(j); });
    }
    return acc;
}

template <typename T, int NPL>
__global__ __launch_bounds__(kSmallWaves * 64) void route_small_kernel(
    RowSrc x, int n_tok, int H, const T* __restrict__ wr, const float* __restrict__ bias, int E, uint32_t e_inverse, int K,
    uint32_t k_inverse, int renorm, double* sums, int32_t* idx, float* __restrict__ w, int32_t* __restrict__ offsets, int32_t* __restrict__ perm,
    int32_t* __restrict__ inv, unsigned long long* __restrict__ active_total, uint32_t* tickets)
{
    constexpr int NT = kSmallWaves * 64;
    constexpr int GROUP = 12 / (int)sizeof(T), STAGE = GROUP * (int)sizeof(T) * 1024;      // chunks at a time; their bytes
    constexpr int ZLD = NPL * 16 + 1;                // logits per token
    constexpr int LDS = kSumWaves * STAGE > 16 * ZLD * 8 ? kSumWaves * STAGE : 16 * ZLD * 8;
    __shared__ __attribute__((aligned(1024))) char lds[LDS];               // the summing waves' stages, then the tile's logits
    double* const z = reinterpret_cast<double*>(lds);
    __shared__ SmallLists lists;
    __shared__ int32_t flag;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t0 = (int)blockIdx.x * 16, e0 = (int)blockIdx.y * 16;
    const int r = lane & 15, q = lane >> 4;
    const bool single = gridDim.x == 1;       // a batch of one token tile: nothing to hand to another block
    char* const stage = lds + (wave < kSumWaves ? wave * STAGE : 0);

    // Turn 0, of the first wave that has no sums to form: its way through the top-k.  Turn 1: the work.
    int turn = wave == kSumWaves ? 0 : 1;
#pragma unroll 1
    for (;; turn = 1) {
        asm volatile("" : "+v"(turn));       // (or the compiler would write the top-k down twice)
        turn = __builtin_amdgcn_readfirstlane(turn);
        if (turn != 0) {
            if (wave >= kSumWaves) lists.clear(E, tid - kSumWaves * 64, NT - kSumWaves * 64);
#pragma unroll 1
            for (int cls = (int)blockIdx.z; cls < kClasses; cls += (int)gridDim.z) {
                double4_t acc;
                if (wave < kSumWaves) {
                    const T* const w_row = wr + (int64_t)(e0 + r < E ? e0 + r : E - 1) * H;      // clamp: loads stay in bounds
                    acc = partial_sum<T, GROUP>(row_ptr<T>(x, t0 + r < n_tok ? t0 + r : n_tok - 1, H), w_row, H, cls + 4 * wave, stage);
                    if (wave > 0) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) reinterpret_cast<double*>(stage)[v * 64 + lane] = acc[v];
                    }
                }
                __syncthreads();
                if (wave == 0 && e0 + r < E) {
                    // D layout of the f64 16x16x4 MFMA: lane l, element v holds row 4*v + l/16 (token), column l % 16 (expert).
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        double s = acc[v];
#pragma unroll
                        for (int o = 1; o < kSumWaves; ++o) s += reinterpret_cast<const double*>(lds + o * STAGE)[v * 64 + lane];
                        const int t = t0 + v * 4 + q;
                        if (t < n_tok) store_shared(sums + ((int64_t)cls * n_tok + t) * E + e0 + r, s);
                    }
                }
                if (cls + (int)gridDim.z < kClasses) __syncthreads();       // the stages are filled again
            }
            if (!last_to_arrive(tickets + 1 + blockIdx.x, gridDim.y * gridDim.z, &flag)) return;
            // The tile's logits: all threads load, whole lines of the four classes.  (Read by the lanes that need them, a 16-lane row
            // per token, the same bytes took 2.8 us in place of 0.6 to 1.8.)
            const int rows = n_tok - t0 < 16 ? n_tok - t0 : 16;
#pragma unroll 4
            for (int i = tid; i < rows * E; i += NT) {
                const int row = (int)((uint32_t)i * e_inverse >> 20), e = i - row * E;
                const double* const from = sums + (int64_t)t0 * E + i;
                double s[kClasses];
#pragma unroll
                for (int c = 0; c < kClasses; ++c) s[c] = load_shared(from + (int64_t)c * n_tok * E);
                z[row * ZLD + e] = (((s[0] + s[1]) + s[2]) + s[3]) + (bias ? (double)bias[e] : 0.0);
            }
            __syncthreads();
        }
        // top-k of this block's 16 tokens: 16 lanes per token, four waves
        const int row = (wave & 3) * 4 + q, t = t0 + row;
        if (turn == 0 || (wave < 4 && t0 + wave * 4 < n_tok)) {
            int e;
            float wt;
            const double* const own = z + (t < n_tok ? row : 0) * ZLD;
            topk_of_row<NPL>([&](int x) { return own[x]; }, E, turn == 0 ? 1 : K, renorm, r, e, wt);
            if (turn != 0 && t < n_tok && r < K) {
                w[t * K + r] = wt;
                if (single) lists.expert_of[t * K + r] = (uint8_t)e;
                else store_shared(idx + t * K + r, (int32_t)e);
            }
            asm volatile("" ::"v"(e), "v"(wt));
        }
        if (turn != 0) break;
    }
    if (single) __syncthreads();
    else if (!last_to_arrive(tickets, gridDim.x, &flag)) return;

    lists.permute<NT>(idx, single, n_tok, E, K, k_inverse, offsets, perm, inv, active_total);
}

// The same where a block has a tile's logits whole, with a partial sum to a wave.
template <typename T, int NPL>
__global__ __launch_bounds__(kTileWaves * 64) void route_small_tile_kernel(
    RowSrc x, int n_tok, int H, const T* __restrict__ wr, const float* __restrict__ bias, int E, int K, uint32_t k_inverse, int renorm,
    double* logits, int32_t* idx, float* __restrict__ w, int32_t* __restrict__ offsets, int32_t* __restrict__ perm,
    int32_t* __restrict__ inv, unsigned long long* __restrict__ active_total, uint32_t* tickets)
{
    constexpr int NT = kTileWaves * 64;
    __shared__ SmallLists lists;
    __shared__ int32_t flag;
    const int tid = threadIdx.x;
    const int t0 = (int)blockIdx.x * 16, e0 = (int)blockIdx.y * 16;
    const bool single = gridDim.x == 1;
    logits_tile<T, kTileWaves>(rows_from<T>(x, t0, n_tok, H), rows_left(t0, n_tok, 16), H, wr, bias, E, e0,
                               [&](int i, int j, double z) { store_shared(logits + (int64_t)(t0 + i) * E + e0 + j, z); });
    lists.clear(E, tid, NT);
    if (!last_to_arrive(tickets + 1 + blockIdx.x, gridDim.y, &flag)) return;

    const int r = tid & 15, row = tid >> 4, t = t0 + row;
    if (row < 16 && t0 + (row & ~3) < n_tok) {      // (whole waves)
        int e;
        float wt;
        const double* const own = logits + (int64_t)(t < n_tok ? t : n_tok - 1) * E;
        topk_of_row<NPL>([&](int x) { return load_shared(own + x); }, E, K, renorm, r, e, wt);
        if (t < n_tok && r < K) {
            w[t * K + r] = wt;
            if (single) lists.expert_of[t * K + r] = (uint8_t)e;
            else store_shared(idx + t * K + r, (int32_t)e);
        }
    }
    if (single) __syncthreads();
    else if (!last_to_arrive(tickets, gridDim.x, &flag)) return;
    lists.permute<NT>(idx, single, n_tok, E, K, k_inverse, offsets, perm, inv, active_total);
}

hipError_t launch_route_small(int dtype, RowSrc x, int64_t T, int H, const void* w_router, const float* bias, int E, int K,
                              int renorm, double* sums, int32_t* idx, float* w, int32_t* offsets, int32_t* perm, int32_t* inv,
                              unsigned long long* active_total, uint32_t* tickets, hipStream_t s)
{
    if (!route_is_small(T, E, K)) return hipErrorInvalidValue;
    int cus = 0;
    const hipError_t err = compute_units(&cus);
    if (err != hipSuccess) return err;
    const int npl = (E + 15) / 16, tiles = (int)((T + 15) / 16) * npl;
    // A tile's sums in kClasses blocks, each on a compute unit of its own, where that shortens the chain of MFMAs by more than its costs
    // (figures at route_small_kernel; the line is drawn through the lengths at which the two were level, from 1 to 256 tokens and 8 to
    // 256 experts).  fp32 rows, twice the bytes, gain twice as much, and with two classes to a block too.
    const int length = dtype == MOE_BF16 ? H : 2 * H, rows = T < 16 ? (int)T : 16;
    int blocks = 0;      // of a tile's sums; none: a block has the tile
    if (length >= 512 + E * (rows + 4) / 4 + 11 * tiles)
        blocks = tiles * kClasses <= cus ? kClasses : dtype == MOE_F32 && tiles * 2 <= cus ? 2 : 0;
    const uint32_t k_inverse = (65536u + K - 1) / K, e_inverse = ((1u << 20) + E - 1) / E;
    static_assert(kSmallTokens * 16 * 15 < 65536, "f / K for f < 256 K, K <= 16");
    static_assert(16 * kSmallExperts * (kSmallExperts - 1) < 1 << 20, "i / E for i < 16 E, E <= 256");
    auto launch = [&](auto elem_t, auto npl_const) {
        typedef decltype(elem_t) X;
        constexpr int NPL = decltype(npl_const)::value;
        const X* const wr = static_cast<const X*>(w_router);
        if (blocks > 0)
            route_small_kernel<X, NPL><<<dim3((unsigned)((T + 15) / 16), (unsigned)npl, (unsigned)blocks), kSmallWaves * 64, 0, s>>>(
                x, (int)T, H, wr, bias, E, e_inverse, K, k_inverse, renorm, sums, idx, w, offsets, perm, inv, active_total, tickets);
        else
            route_small_tile_kernel<X, NPL><<<dim3((unsigned)((T + 15) / 16), (unsigned)npl), kTileWaves * 64, 0, s>>>(
                x, (int)T, H, wr, bias, E, K, k_inverse, renorm, sums, idx, w, offsets, perm, inv, active_total, tickets);
        return hipGetLastError();
    };
    auto go = [&](auto npl_const) { return dtype == MOE_BF16 ? launch(bf16_t(), npl_const) : launch(float(), npl_const); };
    if (npl <= 1) return go(std::integral_constant<int, 1>{});
    if (npl <= 2) return go(std::integral_constant<int, 2>{});
    if (npl <= 8) return go(std::integral_constant<int, 8>{});
    return go(std::integral_constant<int, 16>{});
}

int64_t router_digit_bytes(int H, int E) { return (int64_t)((H + kDigitK - 1) / kDigitK) * ((E + 31) / 32) * 8192; }

hipError_t launch_router_digits(const RouterWeights& w, int layers, int H, int E, uint8_t* digits, void* forms, int32_t* zero_buf,
                                int64_t zero_n, hipStream_t s)
{
    const int rows = (E + 31) / 32 * 32;
    static_assert(sizeof(RowForm) == 32, "router_form_bytes");
    router_digits_kernel<<<dim3((unsigned)rows, (unsigned)layers), kPrepThreads, 0, s>>>(
        w, H, E, digits, router_digit_bytes(H, E), static_cast<RowForm*>(forms), zero_buf, zero_n);
    return hipGetLastError();
}

hipError_t launch_route_exact(RowSrc x, int64_t T, int H, const void* w_router, const float* bias, int E, int K, int renorm,
                              const uint8_t* digits, const void* forms, const RouteList& list, double* logits, int32_t* idx,
                              float* w, int32_t* tile_hist, hipStream_t s)
{
    const int64_t tiles = (T + 31) / 32;
    int cus = 0;
    hipError_t e = compute_units(&cus);
    if (e != hipSuccess) return e;
    // (see route_exact_kernel; a partial sum of the fp64 chain has every 16th 32-wide chunk of the row)
    const double chain_error = 0x1p-52 * 1.02 * (((H + 31) / 32 + 15) / 16 * 32 + 40);
    auto go = [&](auto we, auto wk) {
        constexpr int WE = decltype(we)::value, WK = decltype(wk)::value;
        route_exact_kernel<WE, WK><<<(unsigned)tiles, WE * WK * 64, 0, s>>>(
            x, T, H, static_cast<const bf16_t*>(w_router), bias, E, K, renorm, digits, static_cast<const RowForm*>(forms),
            chain_error, idx, w, tile_hist, list.count, list.tokens);
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
        // Usually none or one tile of 16 tokens (14 us); when it is all of the batch, 8320 tokens of 128 experts, 120 us against
        // 149 with a block's place on the chip each.
        const int64_t most = (T + 15) / 16;
        const unsigned n_e = (unsigned)((E + 15) / 16), per = 8 * (unsigned)cus / n_e + 1;
        const unsigned n_t = most < per ? (unsigned)most : per;
        route_listed_kernel<WE * 2><<<dim3(n_t, n_e), 256, 0, s>>>(x, H, static_cast<const bf16_t*>(w_router), bias, E, K, renorm,
                                                                   list.count, list.tokens, logits, list.tickets, idx, w, tile_hist);
        return hipGetLastError();
    };
    using std::integral_constant;
    if (E <= 64) return go(integral_constant<int, 2>{}, integral_constant<int, 2>{});      // (6700 tokens and more)
    // With a block per compute unit at most, twice the waves (registers leave room for two per SIMD either way), us before the
    // check of the winners: 2112 tokens, H = 2048, 128 experts 26.4 against 29.7, 6000 tokens 35 / 37; 8320 tokens, 260 blocks, 53 / 44.
    return tiles <= cus ? go(integral_constant<int, 4>{}, integral_constant<int, 2>{}) : go(integral_constant<int, 4>{}, integral_constant<int, 1>{});
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
