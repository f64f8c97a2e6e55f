// Weighted un-permute and combine: a token's output is the mix of its K selected
// experts' outputs under the router's weights (Sec. 2.4), plus the residual stream.
// Pure bandwidth: one block per token, 16-byte loads of the K source rows, fp32
// accumulation in slot order, one rounding.
#include <type_traits>

#include "common.h"

namespace moe {

typedef uint32_t chunk16_t __attribute__((ext_vector_type(4)));
template <typename T> struct pack16;   // 16 bytes of elements
template <> struct pack16<bf16_t> {
    static constexpr int N = 8;
    uint4 raw;
    __device__ __forceinline__ void unpack(float* f) const
    {
        const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(w[i] << 16);
            f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
    __device__ __forceinline__ void pack(const float* f)
    {
        raw.x = pack_bf16x2(f[0], f[1]);
        raw.y = pack_bf16x2(f[2], f[3]);
        raw.z = pack_bf16x2(f[4], f[5]);
        raw.w = pack_bf16x2(f[6], f[7]);
    }
};
template <> struct pack16<float> {
    static constexpr int N = 4;
    float4 raw;
    __device__ __forceinline__ void unpack(float* f) const { f[0] = raw.x; f[1] = raw.y; f[2] = raw.z; f[3] = raw.w; }
    __device__ __forceinline__ void pack(const float* f) { raw = make_float4(f[0], f[1], f[2], f[3]); }
};

// y rows [0, rows0) go to y0, rows [rows0, T) to y1 (row t - rows0): lets the layer-group driver
// write decode rows and prefill rows to their separate output buffers without a copy.
// YT: element type of y_perm (T, or float when the context keeps the expert outputs in fp32).
// STREAM: y_perm as non-temporal loads (each of its rows is read once; see launch_combine).
// KB, TAIL: a token's K rows are asked for KB at once, and TAIL = K % KB of them at the end.  With few tokens the kernel is a chain of
// latencies, and a loop over the rows waited for them two by two: now the token's indices and weights are scalar loads (no trip through
// LDS), KB rows and the residual are in flight together.  A pass of four layers over one token (top-8) 129 -> 123 us, an fp32 layer of
// 64 tokens (top-2) 24.1 -> 23.4; level with many tokens, which are bound by bandwidth (6 TB/s at 8320).  A group that divides K would leave 11,
// 13, 17 ... rows to be waited for one by one; us, two by two / by the largest divisor / as now, H = 2048, bf16: one token, top-9 3.3 / 2.8 / 2.6,
// top-13 3.7 / 4.1 / 2.7, top-29 5.6 / 6.8 / 3.6; 256 tokens 4.9 / 4.5 / 3.7, 5.8 / 6.8 / 4.0, 11.2 / 15.4 / 6.3; 2112 tokens, top-11 21.0 /
// 22.3 / 18.8, top-13 24.6 / 26.0 / 22.0; fp32 rows under bf16 output, 256 tokens, top-8 4.0 / 3.7 / 3.0, top-13 6.4 / 6.5 / 4.0.
template <typename T, typename YT, bool STREAM, int KB, int TAIL>
__global__ __launch_bounds__(256) void combine_kernel(const YT* __restrict__ y_perm, const int32_t* __restrict__ inv,
                                                      const float* __restrict__ w, bool has_residual,
                                                      RowSrc residual, int K, int H, T* y0, int64_t rows0, T* y1)
{
    typedef pack16<T> P;
    typedef pack16<YT> PY;
    static_assert(!STREAM || sizeof(T) == sizeof(YT), "a line that is read in two pieces would be fetched twice");
    constexpr int NY = P::N / PY::N;      // 16-byte pieces of y_perm per 16 bytes of output (1, or 2 for fp32 under bf16)
    const int64_t t = blockIdx.x;
    const int32_t* const t_inv = inv + t * K;
    const float* const t_w = w + t * K;
    const int32_t last = (int32_t)gridDim.x * K - 1;
    T* out = (t < rows0) ? (y0 + t * (int64_t)H) : (y1 + (t - rows0) * (int64_t)H);
    for (int c = threadIdx.x * P::N; c < H; c += 256 * P::N) {
        float acc[P::N], v[P::N];
#pragma unroll
        for (int i = 0; i < P::N; ++i) acc[i] = 0.f;
        P res;
        if (has_residual) res.raw = *reinterpret_cast<const decltype(res.raw)*>(row_ptr<T>(residual, t, H) + c);
        auto add_rows = [&](int j0, auto n_const) {
            constexpr int N = decltype(n_const)::value;
            PY p[N][NY];
#pragma unroll
            for (int j = 0; j < N; ++j) {
                // (entries are trusted to lie in [0, T K); the clamp keeps a bad one from becoming a wild address)
                const int32_t row = max(min(t_inv[j0 + j], last), 0);
                const YT* src = y_perm + (uint64_t)(uint32_t)row * (uint32_t)H + c;
#pragma unroll
                for (int h = 0; h < NY; ++h) {
                    if (STREAM)
                        p[j][h].raw = __builtin_bit_cast(decltype(p[j][h].raw), __builtin_nontemporal_load(reinterpret_cast<const chunk16_t*>(src)));
                    else
                        p[j][h].raw = *reinterpret_cast<const decltype(p[j][h].raw)*>(src + h * PY::N);
                }
            }
#pragma unroll
            for (int j = 0; j < N; ++j) {
#pragma unroll
                for (int h = 0; h < NY; ++h) p[j][h].unpack(v + h * PY::N);
                const float wj = t_w[j0 + j];
#pragma unroll
                for (int i = 0; i < P::N; ++i) acc[i] = fmaf(wj, v[i], acc[i]);
            }
        };
#pragma unroll 1
        for (int j0 = 0; j0 < K - TAIL; j0 += KB) add_rows(j0, std::integral_constant<int, KB>());
        if constexpr (TAIL > 0) add_rows(K - TAIL, std::integral_constant<int, TAIL>());
        if (has_residual) {
            res.unpack(v);
#pragma unroll
            for (int i = 0; i < P::N; ++i) acc[i] += v[i];
        }
        P o;
        o.pack(acc);
        *reinterpret_cast<decltype(o.raw)*>(out + c) = o.raw;
    }
}

// Are the expert outputs read as a stream?  Where their rows are whole 128-byte lines: the kernel is level up to 100 MB of them and
// faster beyond (behind the down GEMM, top-8, H = 2048, us, plain / stream: 69 MB (2112 tokens) 18.2 / 18.7, 197 MB 46.8 / 44.3,
// 273 MB (8320) 67.1 / 59.3), and what it leaves in the caches is worth 5 us of the next layer (2112 tokens, 340 / 335).  Where
// neighbouring blocks share lines, only if there are more of them than the last-level cache (256 MB) holds: it still has most of
// what the down GEMM has just written, and a line that is gone between its two readers is fetched twice.  H = 8200: 84 MB
// 23.5 / 26.9, 157 MB 35.8 / 38.8, 315 MB 84.7 / 72.5; H = 1160: 154 MB 33.2 / 34.4, 297 MB 71 / 60.  fp32 rows under bf16 output stay
// plain: a lane reads its 32 bytes of those in two pieces (33.8 / 48).
constexpr int64_t kStreamFrom = (int64_t)160 << 20;
inline bool combine_streams(const void* y_perm, int64_t row_bytes, int64_t rows)
{
    return ((reinterpret_cast<uintptr_t>(y_perm) | (uintptr_t)row_bytes) & 127u) == 0 || row_bytes * rows > kStreamFrom;
}

hipError_t launch_combine(int dtype, bool y_perm_f32, const void* y_perm, const int32_t* inv, const float* w,
                          bool has_residual, RowSrc residual, int64_t T, int K, int H, void* y0, int64_t rows0, void* y1,
                          hipStream_t s)
{
    auto go = [&](auto elem_t, auto y_elem_t, auto stream) {
        typedef decltype(elem_t) X;
        typedef decltype(y_elem_t) Y;
        auto with = [&](auto kb, auto tail) {
            combine_kernel<X, Y, decltype(stream)::value, decltype(kb)::value, decltype(tail)::value><<<(unsigned)T, 256, 0, s>>>(
                static_cast<const Y*>(y_perm), inv, w, has_residual, residual, K, H, static_cast<X*>(y0), rows0, static_cast<X*>(y1));
            return hipGetLastError();
        };
        auto even = [&](auto kb) { return with(kb, std::integral_constant<int, 0>()); };
        auto eights = [&](auto tail) { return with(std::integral_constant<int, 8>(), tail); };
        // Up to 8 rows at once, up to 16 in two equal groups where there are such, of more 8 and then the rest.
        switch (K <= 8 ? K : K <= 16 && K % 2 == 0 ? K / 2 : 0) {
            case 8: return even(std::integral_constant<int, 8>());
            case 7: return even(std::integral_constant<int, 7>());
            case 6: return even(std::integral_constant<int, 6>());
            case 5: return even(std::integral_constant<int, 5>());
            case 4: return even(std::integral_constant<int, 4>());
            case 3: return even(std::integral_constant<int, 3>());
            case 2: return even(std::integral_constant<int, 2>());
            case 1: return even(std::integral_constant<int, 1>());
        }
        switch (K % 8) {
            case 7: return eights(std::integral_constant<int, 7>());
            case 6: return eights(std::integral_constant<int, 6>());
            case 5: return eights(std::integral_constant<int, 5>());
            case 4: return eights(std::integral_constant<int, 4>());
            case 3: return eights(std::integral_constant<int, 3>());
            case 2: return eights(std::integral_constant<int, 2>());
            case 1: return eights(std::integral_constant<int, 1>());
            default: return eights(std::integral_constant<int, 0>());
        }
    };
    const std::true_type stream;
    const std::false_type plain;
    if (dtype == MOE_BF16 && y_perm_f32) return go(bf16_t(), float(), plain);
    if (dtype == MOE_BF16)
        return combine_streams(y_perm, (int64_t)H * 2, T * K) ? go(bf16_t(), bf16_t(), stream) : go(bf16_t(), bf16_t(), plain);
    return combine_streams(y_perm, (int64_t)H * 4, T * K) ? go(float(), float(), stream) : go(float(), float(), plain);
}

}  // namespace moe
