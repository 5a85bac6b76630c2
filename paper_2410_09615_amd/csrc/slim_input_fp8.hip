// 8-bit input quantization as the paper evaluates it (App. "Input Quantization"): AbsMax
// quantization of an input tensor to FP8 with one scale per tensor; the quantized values,
// back on the fp16 grid, are what the layer then sees.  E4M3 (largest value 448) unless the
// tensor's maximum exceeds that, then E5M2 (largest value 57344).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "slim_internal.h"

namespace slim {

constexpr int kInMaxBlocks = 256;

// partial maxima of |X|, one per workgroup (X as 16-byte pieces of 8 halves; `tail` halves after them)
__global__ __launch_bounds__(1024) void input_absmax_kernel(const half_t *__restrict__ X, size_t count, float *part)
{
    __shared__ float red[16];
    const size_t n8 = count / 8;
    float a = 0.f;
    // four independent loads per lane and round: the grid is small (one partial per workgroup)
    const half8_t *X8 = reinterpret_cast<const half8_t *>(X);
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    auto take = [&](const half8_t &v) {
#pragma unroll
        for (int e = 0; e < 8; ++e) a = fmaxf(a, fabsf((float)v[e]));
    };
    for (; i + 3 * stride < n8; i += 4 * stride) {
        const half8_t v0 = X8[i], v1 = X8[i + stride], v2 = X8[i + 2 * stride], v3 = X8[i + 3 * stride];
        take(v0);
        take(v1);
        take(v2);
        take(v3);
    }
    for (; i < n8; i += stride) take(X8[i]);
    if (blockIdx.x == 0)
        for (size_t t = n8 * 8 + threadIdx.x; t < count; t += blockDim.x) a = fmaxf(a, fabsf((float)X[t]));
    a = wave_max(a);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = a;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) a = fmaxf(a, red[w]);
        part[blockIdx.x] = a;
    }
}

// Codes of X (and, where Xq is wanted, the values they stand for).  Streaming: what has to stay small is the work per element.
// The format's own conversion instruction rounds (to nearest even, subnormals included), and the IEEE quotient x / s takes three
// instructions by Markstein's division: with y = 1 / s correctly rounded, q = x y is within one unit in the last place, and
// q + (x - q s) y, the remainder exact, is the quotient correctly rounded.  (|x| is 0 or at least 2^-24 and s is from 2^-33 to
// 2^8: nothing over- or underflows; the quotients of all pairs of fp16 significands are the divisions'.  Only an infinite X
// has another s, and its quotients are divisions.)  With divisions and the rounding written out, about 50 instructions per
// element, the two kernels of a call took 17 us on 2048 x 4096; they take 11, this one 6.6 (3.8 TB/s).
template <bool E5>
__device__ __forceinline__ void input_fp8_pass(const half_t *__restrict__ X, size_t count, float M, half_t *Xq, uint8_t *Xb, float *info)
{
    constexpr float fmax = E5 ? 57344.0f : 448.0f;
    const float s = M == 0.f ? 1.0f : M / fmax;
    const float y = 1.0f / s;
    const bool infinite = s == __builtin_inff();
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        info[0] = s;
        info[1] = E5 ? 1.0f : 0.0f;
    }
    // |x| / s, at most the format's largest value (a NaN becomes that)
    auto scaled = [&](half_t x) {
        const float a = fabsf((float)x);
        float v;
        if (infinite) {
            v = a / s;
        } else {
            const float q = a * y;
            v = __builtin_fmaf(__builtin_fmaf(-q, s, a), y, q);
        }
        return fminf(v, fmax);
    };
    auto four_codes = [&](float v0, float v1, float v2, float v3) {
        if constexpr (E5)
            return (uint32_t)__builtin_amdgcn_cvt_pk_bf8_f32(v2, v3, __builtin_amdgcn_cvt_pk_bf8_f32(v0, v1, 0, false), true);
        else
            return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(v2, v3, __builtin_amdgcn_cvt_pk_fp8_f32(v0, v1, 0, false), true);
    };
    // the value of code e of the dword, times s, with the sign of x.  The sign is carried over as a bit: the product's conversion to
    // half may be contracted into a fused multiply-add with a +0 addend, which would turn a result of -0 into +0.
    auto value = [&](uint32_t codes, auto ec, half_t x) {
        constexpr int e = decltype(ec)::value;
        const float r = E5 ? __builtin_amdgcn_cvt_f32_bf8((int)codes, e) : __builtin_amdgcn_cvt_f32_fp8((int)codes, e);
        // product rounded to binary32, then to binary16 (two roundings, as defined): the empty asm hides the
        // product from the compiler, which would otherwise fuse the two into one mixed-precision
        // multiply-add that rounds once
        float prod = r * s;
        asm volatile("" : "+v"(prod));
        const half_t h = (half_t)prod;
        return __builtin_bit_cast(half_t, (uint16_t)(__builtin_bit_cast(uint16_t, h) | (__builtin_bit_cast(uint16_t, x) & 0x8000u)));
    };
    auto piece = [&](size_t i, half8_t v) {
        const uint4_t u = __builtin_bit_cast(uint4_t, v);
        uint2_t c;
#pragma unroll
        for (int d = 0; d < 2; ++d) {
            const uint32_t codes = four_codes(scaled(v[4 * d]), scaled(v[4 * d + 1]), scaled(v[4 * d + 2]), scaled(v[4 * d + 3]));
            c[d] = codes;
        }
        if (Xq) {
            half8_t o;
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                o[4 * d] = value(c[d], std::integral_constant<int, 0>{}, v[4 * d]);
                o[4 * d + 1] = value(c[d], std::integral_constant<int, 1>{}, v[4 * d + 1]);
                o[4 * d + 2] = value(c[d], std::integral_constant<int, 2>{}, v[4 * d + 2]);
                o[4 * d + 3] = value(c[d], std::integral_constant<int, 3>{}, v[4 * d + 3]);
            }
            reinterpret_cast<half8_t *>(Xq)[i] = o;
        }
        if (Xb) {
            // bit 7 of a code is the sign of its half: the high bytes of four halves
#pragma unroll
            for (int d = 0; d < 2; ++d) c[d] |= __builtin_amdgcn_perm(u[2 * d + 1], u[2 * d], 0x07050301u) & 0x80808080u;
            reinterpret_cast<uint2_t *>(Xb)[i] = c;
        }
    };
    const size_t n8 = count / 8, stride = (size_t)gridDim.x * blockDim.x;
    const half8_t *const X8 = reinterpret_cast<const half8_t *>(X);
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i + stride < n8; i += 2 * stride) {           // two loads in flight per lane
        const half8_t v0 = X8[i], v1 = X8[i + stride];
        piece(i, v0);
        piece(i + stride, v1);
    }
    if (i < n8) piece(i, X8[i]);
    if (blockIdx.x == 0)
        for (size_t t = n8 * 8 + threadIdx.x; t < count; t += blockDim.x) {
            const half_t x = X[t];
            const uint32_t c = four_codes(scaled(x), 0.f, 0.f, 0.f);
            if (Xq) Xq[t] = value(c, std::integral_constant<int, 0>{}, x);
            if (Xb) Xb[t] = (uint8_t)(c | ((__builtin_bit_cast(uint16_t, x) >> 8) & 0x80u));
        }
}

__global__ __launch_bounds__(256) void input_fp8_kernel(const half_t *__restrict__ X, size_t count, const float *part, int nparts,
                                                        half_t *Xq, uint8_t *Xb, float *info)
{
    __shared__ float red[4];
    float a = (int)threadIdx.x < nparts ? part[threadIdx.x] : 0.f;
    a = wave_max(a);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = a;
    __syncthreads();
    const float M = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    if (M > 448.0f)
        input_fp8_pass<true>(X, count, M, Xq, Xb, info);
    else
        input_fp8_pass<false>(X, count, M, Xq, Xb, info);
}

}  // namespace slim

using namespace slim;

extern "C" int slim_input_quant_fp8_codes(const slim_half *X, size_t count, slim_half *Xq, uint8_t *Xb, float *info,
                                          void *workspace, size_t workspace_bytes, void *stream)
{
    if (!X || (!Xq && !Xb) || !info || !workspace) return SLIM_ERR_NULL;
    if (count < 1) return SLIM_ERR_SHAPE;
    if (!aligned16(X) || (Xq && !aligned16(Xq)) || !aligned16(workspace) || (Xb && !aligned16(Xb))) return SLIM_ERR_ALIGN;
    if (workspace_bytes < kInMaxBlocks * sizeof(float)) return SLIM_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const size_t g = (count / 8 + 255) / 256;
    const size_t ga = (count / 8 + 1023) / 1024;
    const unsigned grid_a = (unsigned)(ga < 1 ? 1 : (ga < kInMaxBlocks ? ga : kInMaxBlocks));
    const unsigned grid_q = (unsigned)(g < 1 ? 1 : (g < 2048 ? g : 2048));
    float *part = static_cast<float *>(workspace);
    hipLaunchKernelGGL(input_absmax_kernel, dim3(grid_a), dim3(1024), 0, st, reinterpret_cast<const half_t *>(X), count, part);
    hipLaunchKernelGGL(input_fp8_kernel, dim3(grid_q), dim3(256), 0, st, reinterpret_cast<const half_t *>(X), count,
                       (const float *)part, (int)grid_a, reinterpret_cast<half_t *>(Xq), Xb, info);
    return hip_status(hipGetLastError());
}

extern "C" int slim_input_quant_fp8(const slim_half *X, size_t count, slim_half *Xq, float *info, void *workspace,
                                    size_t workspace_bytes, void *stream)
{
    if (!Xq) return SLIM_ERR_NULL;
    return slim_input_quant_fp8_codes(X, count, Xq, nullptr, info, workspace, workspace_bytes, stream);
}
