// Shared device/host helpers for the gfx950 MoE kernels (not used by the CPU oracle).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>

#include "moe_lp.h"

namespace moe {

typedef uint16_t bf16_t;  // raw bfloat16 bit pattern

constexpr int kWave = 64;
constexpr int kMaxExperts = 512;
constexpr int kMaxTopK = 64;

__device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// Round to nearest, ties to even, with the hardware conversion of gfx950 (v_cvt_pk_bf16_f32).
typedef __bf16 hw_bf16x2_t __attribute__((ext_vector_type(2)));
typedef float hw_float2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    const hw_float2_t v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, hw_bf16x2_t));
}

__device__ __forceinline__ bf16_t f32_to_bf16(float f) { return (bf16_t)(pack_bf16x2(f, 0.0f) & 0xffffu); }

template <typename T> struct elem;
template <> struct elem<float> {
    static __device__ __forceinline__ float to_f32(float v) { return v; }
    static __device__ __forceinline__ float from_f32(float v) { return v; }
};
template <> struct elem<bf16_t> {
    static __device__ __forceinline__ float to_f32(bf16_t v) { return bf16_to_f32(v); }
    static __device__ __forceinline__ bf16_t from_f32(float v) { return f32_to_bf16(v); }
};

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }

typedef __attribute__((address_space(3))) void lds_ptr_t;
typedef __attribute__((address_space(1))) const void glb_ptr_t;

// Inclusive scan over the wave's lanes in six register-to-register steps (row shifts, then the last lane of a row to
// the next row, then lane 31 to the upper half).
template <typename V> __device__ __forceinline__ V wave_scan(V v)
{
    auto step = [&](auto ctrl, auto row_mask) {
        const int o = __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), decltype(ctrl)::value,
                                                  decltype(row_mask)::value, 0xF, true);
        v += __builtin_bit_cast(V, o);
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>{}, integral_constant<int, 0xF>{});      // from 1, 2, 4 and 8 lanes below, within 16
    step(integral_constant<int, 0x112>{}, integral_constant<int, 0xF>{});
    step(integral_constant<int, 0x114>{}, integral_constant<int, 0xF>{});
    step(integral_constant<int, 0x118>{}, integral_constant<int, 0xF>{});
    step(integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});      // rows 1 and 3: last lane of the row below
    step(integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});      // upper half: lane 31
    return v;
}

// A batch of rows that lives in two buffers: rows [0, n0) in p0, the rest in p1 (row t - n0).  The
// layer-group driver reads the first layer's input straight from x_decode / x_prefill this way instead
// of copying the two pieces together first.
struct RowSrc {
    const void* p0;
    int64_t n0;
    const void* p1;
};
inline RowSrc single_src(const void* p) { return RowSrc{p, (int64_t)1 << 62, p}; }
template <typename T> __device__ __forceinline__ const T* row_ptr(const RowSrc& s, int64_t t, int64_t ld)
{
    return t < s.n0 ? static_cast<const T*>(s.p0) + t * ld : static_cast<const T*>(s.p1) + (t - s.n0) * ld;
}

// ---- launchers implemented in the .hip files; all return hipError_t from hipGetLastError() ----

// router.hip
hipError_t launch_router_logits(int dtype, RowSrc x, int64_t T, int H, const void* w_router, const float* bias,
                                int E, double* logits, int32_t* zero_buf, int zero_n, hipStream_t s);
// Batches whose routing (logits, top-k, permutation) is one launch: a single block can hold the permutation, and
// 16 lanes a token's logits (at E > 256 they no longer fit the registers of a 16-wave block).
constexpr int kSmallTokens = 256, kSmallExperts = 256;
inline bool route_is_small(int64_t T, int E, int K) { return T <= kSmallTokens && E <= kSmallExperts && K <= 16; }

// Router and top-k of larger bf16 batches by exact integer sums (see router.hip), with the results of the fp64 pass: a launch
// that makes the digits of the layers' w_router (router_digit_bytes and router_form_bytes for each) and clears zero_n words,
// then two launches per layer; tile_hist as for launch_topk; logits: [T, E] of scratch.
constexpr int kDigitLayers = 8;      // layers per digits launch
struct RouterWeights {
    const void* p[kDigitLayers];
};
int64_t router_digit_bytes(int H, int E);
inline int64_t router_form_bytes(int E) { return (int64_t)((E + 31) / 32 * 32) * 32; }
hipError_t launch_router_digits(const RouterWeights& w, int layers, int H, int E, uint8_t* digits, void* forms, int32_t* zero_buf,
                                int64_t zero_n, hipStream_t s);
// The tokens that the exact sums leave to the fp64 pass: count and tickets (one per 16 tokens of the batch) are zero before the launch.
struct RouteList {
    int32_t* count;
    uint32_t* tickets;
    int32_t* tokens;      // [T]
};
inline int64_t route_list_words(int64_t T) { return 1 + (T + 15) / 16; }      // count and tickets
hipError_t launch_route_exact(RowSrc x, int64_t T, int H, const void* w_router, const float* bias, int E, int K, int renorm,
                              const uint8_t* digits, const void* forms, const RouteList& list, double* logits, int32_t* idx,
                              float* w, int32_t* tile_hist, hipStream_t s);
// (its sums are at most 4 H 2^14; a block holds all experts' logits of its tokens.)  A block of 32 tokens takes as long as the chip
// with a block on every unit, and about in proportion to H, while the fp64 pass grows with the 16 x 16 tiles of logits: so the
// line is a number of logits, at short rows a higher one (the launches' own 20 us).  moe_router_topk, us, fp64 pass / this
// one with the digits of one layer:
//   E = 128:  H = 512: 3000 tokens 19 / 21, 4100 23 / 22;  1024: 2500 23 / 25, 3500 28 / 27;  2048: 2500 36 / 37, 4100 55 / 36,
//             8200 97 / 52;  2880: 3000 53 / 56, 3500 59 / 52;  4096: 2500 61 / 65, 4100 98 / 71;  8192: 3000 128 / 123;
//             16384: 300 56 / 198, 2500 207 / 249, 3500 281 / 262
//   E = 96:   2048: 3000 35 / 36, 4100 45 / 35;  8192: 4100 146 / 142;  16384: 4100 281 / 303
//   E = 64:   512: 8200 24 / 24;  2048: 5000 35 / 38, 6500 45 / 37;  4096: 6500 78 / 74;  16384: 577 55 / 156
//   E = 48 (a fourth of the MFMAs for nothing): 2048: 8200 46 / 46, 16384 72 / 56;  4096: 8200 78 / 86, 12000 99 / 93
//   E = 32 and less (one group of experts to a block): 2048: 16384 50 / 53;  4096: 16384 89 / 106, 32768 170 / 170
constexpr int kExactMaxH = 16384, kExactMinExperts = 49, kExactMaxExperts = 128;
inline bool route_is_exact(int dtype, int64_t T, int H, int E, int K)
{
    const int64_t logits = T * ((E + 15) / 16 * 16);
    return dtype == MOE_BF16 && H <= kExactMaxH && E >= kExactMinExperts && E <= kExactMaxExperts && K <= 16 &&
           (logits - 425984) * H >= (int64_t)1 << 26;
}
static_assert(kSmallTokens * kSmallExperts < 425984, "a batch of the one-launch routing is below the line");
// tile_hist (or NULL): [ceil(T*K / kPermTile), E] counters, already zero, that receive the expert histogram
hipError_t launch_topk(const double* logits, int64_t T, int E, int K, int renorm, int32_t* idx, float* w,
                       int32_t* tile_hist, hipStream_t s);

// tickets: kSmallTickets counters, zero before the first launch; every launch leaves them at zero
// sums: scratch of kSmallSumBytes per logit
constexpr int kSmallTickets = 1 + kSmallTokens / 16, kSmallSumBytes = 32;
hipError_t launch_route_small(int dtype, RowSrc x, int64_t T, int H, const void* w_router, const float* bias, int E, int K,
                              int renorm, double* sums, int32_t* idx, float* w, int32_t* offsets, int32_t* perm, int32_t* inv,
                              unsigned long long* active_total, uint32_t* tickets, hipStream_t s);

// permute.hip
constexpr int kPermTile = 2048;  // assignments per block of the permutation kernels
// Batches whose expert counts every block of the scatter takes from the assignments themselves (see launch_permute): in a call of its own,
// and behind a top-k, which could count them too.
constexpr int kCountTiles = 6, kCountTilesBehindTopk = 4;
inline bool topk_counts(int64_t A) { return A > (int64_t)kCountTilesBehindTopk * kPermTile; }
// hist_ready: tile_hist already holds the per-tile histograms (the top-k kernel counted them)
hipError_t launch_permute(const int32_t* idx, int64_t A, int E, int32_t* counts, int32_t* offsets,
                          int32_t* perm, int32_t* inv, int32_t* tile_hist, bool hist_ready,
                          unsigned long long* active_total, hipStream_t s);
hipError_t launch_fill_zero(void* p, int n_words, hipStream_t s);   // a fill kernel, not a memset node
hipError_t launch_gather_rows(int dtype, const void* x, const int32_t* perm, int K, int64_t A, int H,
                              void* x_perm, hipStream_t s);

// combine.hip
// y_perm_f32: y_perm holds float whatever dtype is
hipError_t launch_combine(int dtype, bool y_perm_f32, const void* y_perm, const int32_t* inv, const float* w,
                          bool has_residual, RowSrc residual, int64_t T, int K, int H, void* y0, int64_t rows0,
                          void* y1, hipStream_t s);

// ffn.hip
// x: [*, H]; row_map (or NULL): permuted row r reads x row row_map[r] / map_div; offsets [E+1].
// variant: a moe_ffn_variant_id (MOE_FFN_AUTO: chosen from the mean rows per expert); out_f32: y_perm is float;
// split: act is [A, 2I], every value a pair of bf16 (hi in column i, lo in column I + i); needs out_f32
hipError_t launch_ffn_gate_up(int dtype, int variant, bool split, RowSrc x, const int32_t* row_map, int map_div,
                              const int32_t* offsets, int64_t A, int E, int H, int I, const void* w_gate_up,
                              void* act, hipStream_t s);
hipError_t launch_ffn_down(int dtype, int variant, bool out_f32, bool split, const void* act, const int32_t* offsets,
                           int64_t A, int E, int H, int I, const void* w_down, void* y_perm, hipStream_t s);
const char* ffn_variant_name(int dtype, int variant, int64_t A, int E, int H, int I);

// Sets a kernel's dynamic-LDS limit once per device (the attribute belongs to the device's copy of the code
// object).  `done` is the caller's per-kernel array of kMaxDevices flags.
constexpr int kMaxDevices = 16;
template <typename K> inline hipError_t ensure_lds_limit(K kern, size_t lds_bytes, bool* done)
{
    int d = 0;
    hipError_t e = hipGetDevice(&d);
    if (e != hipSuccess) return e;
    if (d < 0 || d >= kMaxDevices) return hipErrorInvalidDevice;
    if (done[d]) return hipSuccess;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds_bytes);
    if (e == hipSuccess) done[d] = true;
    return e;
}

// Compute units of the current device, looked up once per device.
inline hipError_t compute_units(int* out)
{
    static std::atomic<int> known[kMaxDevices];
    int d = 0;
    hipError_t e = hipGetDevice(&d);
    if (e != hipSuccess) return e;
    if (d < 0 || d >= kMaxDevices) return hipErrorInvalidDevice;
    int n = known[d].load(std::memory_order_relaxed);
    if (n == 0) {
        e = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, d);
        if (e != hipSuccess) return e;
        known[d].store(n, std::memory_order_relaxed);
    }
    *out = n;
    return hipSuccess;
}

// ffn_w4.hip: the same two GEMMs with MXFP4 expert weights (codes + scale bytes), bf16 activations
hipError_t launch_ffn_gate_up_w4(int variant, RowSrc x, const int32_t* row_map, int map_div, const int32_t* offsets,
                                 int64_t A, int E, int H, int I, const uint8_t* w_gate_up, const uint8_t* s_gate_up,
                                 void* act, hipStream_t s);
hipError_t launch_ffn_down_w4(int variant, bool out_f32, const void* act, const int32_t* offsets, int64_t A, int E, int H,
                              int I, const uint8_t* w_down, const uint8_t* s_down, void* y_perm, hipStream_t s);
const char* ffn_w4_variant_name(int variant, int64_t A, int E, int H, int I);

}  // namespace moe
