// slim_quant_search: the per-tensor scale of SLiM-Quant (Sec. 3.1, Eq. 4-7,
// Alg. 1): alpha* minimises E_quant(alpha) + E_clip(alpha), the squared error of
// the symmetric 4-bit quantizer with full scale alpha, integrated over the
// histogram of |W| (every element of a bin taken at the bin's centre).
//
//   histogram  B = max(512, min(n k / 1000, 20000)) uniform bins over [0, M],
//              M = max|W|; bin = min(B - 1, floor(|w| * (B / M))), quotient and
//              product in binary32 (so the counts are reproducible integers)
//   coarse     E at alpha = M i / 10, i = 1..10 (the last one is AbsMax)
//   fine       E at 21 samples of a tenth of that spacing around the best
//              coarse one (those inside (0, M])
//   alpha*     the first minimum over all of them; scale = alpha* / 7 (binary32)
//
// Three passes over memory in all: max, histogram (both read W once, HBM-bound),
// and the candidates, which only touch the histogram.  Everything stays on the
// device; the error sums are fp64.
//
// The candidates are one launch: the fine samples around every coarse one are evaluated beside the coarse ones
// (220 workgroups, at most one per compute unit, of which 31 count), and the workgroup that ends last picks.  What bounds it is
// launches and latency, not work: with coarse, fine and pick as three launches (23 us on 20000 bins) the call on 11008 x 4096
// took 128.7 us, with one 119.3 (the adds of the histograms, from another bin in every workgroup, included).
#include "slim_internal.h"

namespace slim {

constexpr int kCoarse = 10;
constexpr int kFine = 21;
constexpr int kMaxBins = 20000;
constexpr int kRowBins = 512;           // the fewest, which rows below 513000 inputs have
constexpr int kCandidates = kCoarse * (1 + kFine);   // coarse ones, then the fine ones around each of them
constexpr int kMaxBlocks = 1024;        // workgroups of the maximum pass (one partial maximum each)

// workspace (32-bit words): [0] bits of M, [1] and every 14th after it to [113]: counts of candidates that have ended,
// [128 .. 128 + B) counts, then kMaxBlocks per-workgroup maxima, over which (from the next 8-byte boundary) the
// candidates' errors are written
struct QuantWs {
    unsigned *mbits, *done;
    unsigned *counts;
    float *bmax;
    double *err;
};
__host__ __device__ inline QuantWs quant_ws(void *ws, int B)
{
    QuantWs q;
    q.mbits = static_cast<unsigned *>(ws);
    q.done = q.mbits + 1;
    q.counts = q.mbits + 128;
    q.bmax = reinterpret_cast<float *>(q.counts + B);
    q.err = reinterpret_cast<double *>(q.counts + (B + 1) / 2 * 2);
    return q;
}
static_assert(2 * kCandidates + 1 <= kMaxBlocks, "the errors fit where the maxima were");

__host__ __device__ inline int quant_bins(long numel)
{
    const long b = numel / 1000 < kMaxBins ? numel / 1000 : kMaxBins;
    return (int)(b > kRowBins ? b : kRowBins);
}

// partial maxima of |W|, one per workgroup (no atomics: thousands of them on one
// address would serialize at memory)
__global__ __launch_bounds__(256) void quant_absmax_kernel(const float *__restrict__ W, size_t numel4, float *bmax,
                                                           unsigned *ws, int words)
{
    __shared__ float part[4];
    // the words the later kernels add into start at zero (this kernel runs before them)
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < words; i += gridDim.x * blockDim.x) ws[i] = 0u;
    float a = 0.f;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < numel4; i += (size_t)gridDim.x * blockDim.x) {
        const float4 v = reinterpret_cast<const float4 *>(W)[i];
        a = fmaxf(a, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
    }
    a = wave_max(a);
    if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = a;
    __syncthreads();
    if (threadIdx.x == 0) bmax[blockIdx.x] = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
}

// per-workgroup histogram in LDS, then one global add per non-empty bin
__global__ __launch_bounds__(1024) void quant_hist_kernel(const float *__restrict__ W, size_t numel4, int B,
                                                          const float *bmax, int nblocks, unsigned *mbits, unsigned *counts)
{
    extern __shared__ unsigned hist[];
    __shared__ float part[16];
    for (int i = threadIdx.x; i < B; i += blockDim.x) hist[i] = 0u;
    // M from the partial maxima (every workgroup for itself; workgroup 0 publishes it)
    float a = (int)threadIdx.x < nblocks ? bmax[threadIdx.x] : 0.f;
    a = wave_max(a);
    if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = a;
    __syncthreads();
    float M = part[0];
    for (int w = 1; w < (int)blockDim.x / kWave; ++w) M = fmaxf(M, part[w]);
    if (blockIdx.x == 0 && threadIdx.x == 0) *mbits = __float_as_uint(M);
    if (M > 0.f) {
        const float inv = (float)B / M;
        auto put = [&](float w) {
            const int b = (int)floorf(fabsf(w) * inv);
            atomicAdd(&hist[b < B - 1 ? b : B - 1], 1u);
        };
        const float4 *W4 = reinterpret_cast<const float4 *>(W);
        const size_t stride = (size_t)gridDim.x * blockDim.x;
        size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
        for (; i + 3 * stride < numel4; i += 4 * stride) {   // four loads in flight per lane
            float4 v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = W4[i + q * stride];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                put(v[q].x);
                put(v[q].y);
                put(v[q].z);
                put(v[q].w);
            }
        }
        for (; i < numel4; i += stride) {
            const float4 v = W4[i];
            put(v.x);
            put(v.y);
            put(v.z);
            put(v.w);
        }
    }
    __syncthreads();
    // every workgroup starts at another bin: adds to one address serialize at memory
    const int first = (int)((size_t)blockIdx.x * B / gridDim.x) & ~(kWave - 1);
    for (int j = threadIdx.x; j < B; j += blockDim.x) {
        const int i = first + j < B ? first + j : first + j - B;
        if (hist[i]) atomicAdd(&counts[i], hist[i]);
    }
}

// E(alpha) over the histogram: one workgroup, fp64
__device__ __forceinline__ double quant_error_block(const unsigned *counts, int B, double M, double alpha, double *red)
{
    const double step = alpha / 7.0, width = M / B, inv_step = 1.0 / step;
    double e = 0.0;
    constexpr int N = 10;                        // counts in flight: they come from memory, where the adds put them
    for (int b0 = threadIdx.x; b0 < B; b0 += N * blockDim.x) {
        unsigned cnt[N];
#pragma unroll
        for (int i = 0; i < N; ++i) cnt[i] = b0 + i * (int)blockDim.x < B ? counts[b0 + i * blockDim.x] : 0u;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double x = ((double)(b0 + i * (int)blockDim.x) + 0.5) * width;
            double d = alpha - x;
            if (x <= alpha) {
                // rint(x / step) without the division wherever that cannot change it (see quant_rows_kernel)
                const double q = x * inv_step;
                double r = rint(q);
                if (fabs(q - r) > 0.5 - 1e-9) r = rint(x / step);
                d = r * step - x;
            }
            e += (double)cnt[i] * (d * d);
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) e += __shfl_xor(e, off, kWave);
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = e;
    __syncthreads();
    double t = 0.0;
    for (int w = 0; w < (int)blockDim.x / kWave; ++w) t += red[w];
    return t;
}

__device__ __forceinline__ double coarse_alpha(double M, int i) { return M / 10.0 * (i + 1); }
__device__ __forceinline__ double fine_alpha(double M, int i, int f) { return M / 10.0 * (i + 1) + M / 10.0 * ((f - 10) / 10.0); }

// Workgroup c evaluates candidate c: c < kCoarse coarse, else fine sample (c - kCoarse) % kFine around coarse candidate
// (c - kCoarse) / kFine.  The last one to end picks: alpha* = first minimum over the coarse ones and the fine ones
// around the best of them; scale_out[o] = alpha* / 7 for every row.
__global__ __launch_bounds__(1024) void quant_eval_kernel(const unsigned *mbits, const unsigned *counts, int B, double *err,
                                                          unsigned *done, float *scale_out, int n, float *alpha_out)
{
    __shared__ double red[16];
    __shared__ unsigned last;
    const int c = blockIdx.x;
    const double M = (double)__uint_as_float(*mbits);
    const double alpha = c < kCoarse ? coarse_alpha(M, c) : fine_alpha(M, (c - kCoarse) / kFine, (c - kCoarse) % kFine);
    double e = __builtin_inf();
    if (M != 0.0 && (c < kCoarse || (alpha > 0.0 && alpha <= M))) e = quant_error_block(counts, B, M, alpha, red);
    if (threadIdx.x == 0) {
        // handed over by the counts: one of eight, then the one of those (adds to one address serialize at memory).  The
        // release and the acquires cost the call 1 us (11008 x 4096: 119.6 -> 120.5).
        __hip_atomic_store(err + c, e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned g = blockIdx.x % 8, of = (gridDim.x - g + 7) / 8;
        last = 0u;
        if (__hip_atomic_fetch_add(done + 14 * (g + 1), 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT) == of - 1) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            if (__hip_atomic_fetch_add(done, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT) == 7u) {
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                last = 1u;
            }
        }
    }
    __syncthreads();
    if (!last) return;
    __shared__ double all[kCandidates];
    if (threadIdx.x < kCandidates) all[threadIdx.x] = __hip_atomic_load(err + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    float a = 0.f, s = 1.f;
    if (M > 0.0) {
        int best = 0, pick = -1;
        double low = all[0];
#pragma unroll
        for (int i = 1; i < kCoarse; ++i)
            if (all[i] < low) {
                low = all[i];
                best = i;
            }
        const double *const fine = all + kCoarse + best * kFine;
#pragma unroll
        for (int f = 0; f < kFine; ++f)
            if (fine[f] < low) {
                low = fine[f];
                pick = f;
            }
        a = (float)(pick < 0 ? coarse_alpha(M, best) : fine_alpha(M, best, pick));
        s = a / 7.0f;
    }
    for (int o = threadIdx.x; o < n; o += blockDim.x) scale_out[o] = s;
    if (alpha_out && threadIdx.x == 0) *alpha_out = a;
}

// ---- the same search with one scale per output row: one workgroup per row, everything in LDS ----
// (the histogram of a row has quant_bins(k) bins: 512 for every k below 513000)
// What bounds it is the binary64 arithmetic of 31 candidates times 512 bins per row.  TABLE: B = 512, and the centre and the count
// of a bin are made once per row, as binary64 in LDS, instead of by every candidate, and four bins go without a branch (4096 x 4096: 54.5 -> 49.2 us, 512 x 512 13.0 -> 8.8).
template <bool TABLE>
__global__ __launch_bounds__(256) void quant_rows_kernel(const float *__restrict__ W, int n, int k, int B_any, float *scale_out,
                                                         float *alpha_out)
{
    extern __shared__ unsigned hist[];
    struct Bin {
        double x, count;
    };
    __shared__ Bin bins[TABLE ? kRowBins + 4 * 24 : 1];
    const int B = TABLE ? kRowBins : B_any;
    __shared__ double err[kCoarse + kFine];
    __shared__ double psum[(kCoarse + kFine) * 24];
    __shared__ float part[4];
    const int k4 = k / 4;
    for (int row = blockIdx.x; row < n; row += gridDim.x) {
        const float4 *w4 = reinterpret_cast<const float4 *>(W + (size_t)row * k);
        float a = 0.f;
        for (int i = threadIdx.x; i < k4; i += blockDim.x) {
            const float4 v = w4[i];
            a = fmaxf(a, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
        }
        a = wave_max(a);
        __syncthreads();                      // the previous row is done with hist, part and err
        if ((threadIdx.x & (kWave - 1)) == 0) part[threadIdx.x / kWave] = a;
        for (int i = threadIdx.x; i < B; i += blockDim.x) hist[i] = 0u;
        __syncthreads();
        const float Mf = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
        float alpha_f = 0.f, s = 1.f;
        if (Mf > 0.f) {
            const float inv = (float)B / Mf;
            auto put = [&](float w) {
                const int b = (int)floorf(fabsf(w) * inv);
                atomicAdd(&hist[b < B - 1 ? b : B - 1], 1u);
            };
            for (int i = threadIdx.x; i < k4; i += blockDim.x) {
                const float4 v = w4[i];
                put(v.x);
                put(v.y);
                put(v.z);
                put(v.w);
            }
            __syncthreads();
            const double M = (double)Mf, eta = M / 10.0;
            if constexpr (TABLE) {
                for (int b = threadIdx.x; b < B + 4 * 24; b += blockDim.x)
                    bins[b] = b < B ? Bin{((double)b + 0.5) * (M / B), (double)hist[b]} : Bin{0.0, 0.0};
                __syncthreads();
            }
            // all candidates of a stage at once: G lanes share a candidate, each takes every G-th bin
            auto eval = [&](int c, double alpha, bool ok, int j, int G) {
                double e = 0.0;
                if (ok) {
                    // rint(x / step) without the binary64 division wherever that cannot change the result:
                    // x * (1 / step) is within a few ulp of the quotient (at most 700), so the two round to the
                    // same integer unless the product lies within 1e-9 of a half; there the quotient decides.
                    // Empty bins add an exact zero.
                    const double step = alpha / 7.0, width = M / B, inv_step = 1.0 / step;
                    if constexpr (TABLE) {
                        // four bins at a time, without branches but for quotients near a half (past the last bin there are empty ones)
                        for (int b = j; b < B; b += 4 * G) {
                            Bin bin[4];
                            double r[4];
                            bool near_half = false;
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                bin[i] = bins[b + i * G];
                                const double q = bin[i].x * inv_step;
                                r[i] = rint(q);
                                near_half = near_half || fabs(q - r[i]) > 0.5 - 1e-9;
                            }
                            if (near_half)
#pragma unroll
                                for (int i = 0; i < 4; ++i) r[i] = rint(bin[i].x / step);
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const double d = bin[i].x <= alpha ? r[i] * step - bin[i].x : alpha - bin[i].x;
                                e += bin[i].count * (d * d);
                            }
                        }
                    } else {
                        for (int b = j; b < B; b += G) {
                            const unsigned cnt = hist[b];
                            if (cnt == 0u) continue;
                            const double x = ((double)b + 0.5) * width;
                            double d = alpha - x;
                            if (x <= alpha) {
                                const double q = x * inv_step;
                                double r = rint(q);
                                if (fabs(q - r) > 0.5 - 1e-9) r = rint(x / step);
                                d = r * step - x;
                            }
                            e += (double)cnt * (d * d);
                        }
                    }
                }
                // the G partial sums of a candidate are added up in lane order by its first lane
                if (c < kCoarse + kFine) psum[c * 24 + j] = e;
                __syncthreads();
                if (j == 0 && c < kCoarse + kFine) {
                    double t = 0.0;
                    for (int i = 0; i < G; ++i) t += psum[c * 24 + i];
                    err[c] = ok ? t : __builtin_inf();
                }
            };
            {
                const int c = threadIdx.x / 24;                     // 24 lanes per coarse candidate: 240 of 256 busy
                eval(c, eta * (c + 1), c < kCoarse, threadIdx.x - 24 * c, 24);
            }
            __syncthreads();
            int best = 0;
            double low = err[0];
#pragma unroll
            for (int i = 1; i < kCoarse; ++i) {
                const double v = err[i];
                best = v < low ? i : best;
                low = v < low ? v : low;
            }
            const double lo = eta * (best + 1);
            {
                const int f = threadIdx.x / 12;                     // 12 lanes per fine candidate: 252 of 256 busy
                const double alpha = lo + eta * ((f - 10) / 10.0);
                eval(kCoarse + f, alpha, f < kFine && alpha > 0.0 && alpha <= M, threadIdx.x - 12 * f, 12);
            }
            __syncthreads();
            int pick = best;
#pragma unroll
            for (int c = kCoarse; c < kCoarse + kFine; ++c) {
                const double v = err[c];
                pick = v < low ? c : pick;
                low = v < low ? v : low;
            }
            const double al = pick < kCoarse ? eta * (pick + 1) : lo + eta * ((pick - kCoarse - 10) / 10.0);
            alpha_f = (float)al;
            s = alpha_f / 7.0f;
        }
        if (threadIdx.x == 0) {
            scale_out[row] = s;
            if (alpha_out) alpha_out[row] = alpha_f;
        }
    }
}

}  // namespace slim

using namespace slim;

extern "C" int slim_quant_workspace_bytes(slim_shape shape, size_t *bytes)
{
    if (!bytes) return SLIM_ERR_NULL;
    if (shape.n < 1 || shape.k < 8 || shape.k % 8) return SLIM_ERR_SHAPE;
    *bytes = (size_t)(128 + quant_bins((long)shape.n * shape.k) + kMaxBlocks) * 4;
    return SLIM_OK;
}

extern "C" int slim_quant_search(const float *W, slim_shape shape, float *scale_out, float *alpha_out, void *workspace,
                                 size_t workspace_bytes, void *stream)
{
    if (!W || !scale_out || !workspace) return SLIM_ERR_NULL;
    if (shape.n < 1 || shape.k < 8 || shape.k % 8) return SLIM_ERR_SHAPE;
    if (!aligned16(W) || !aligned16(workspace)) return SLIM_ERR_ALIGN;
    const size_t numel = (size_t)shape.n * shape.k;
    const int B = quant_bins((long)numel);
    if (workspace_bytes < (size_t)(128 + B + kMaxBlocks) * 4) return SLIM_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const QuantWs q = quant_ws(workspace, B);
    const size_t numel4 = numel / 4;
    size_t g = (numel4 + 255) / 256;
    const unsigned grid_a = (unsigned)(g < (size_t)kMaxBlocks ? g : (size_t)kMaxBlocks);
    g = (numel4 + 1023) / 1024;
    // every workgroup ends with one global add per non-empty bin of its own histogram: few workgroups
    // (one per compute unit; half of that below 2^25 elements, where those adds outweigh the reading)
    const size_t hcap = numel < ((size_t)1 << 25) ? 128 : 256;
    const unsigned grid_h = (unsigned)(g < hcap ? g : hcap);
    hipLaunchKernelGGL(quant_absmax_kernel, dim3(grid_a), dim3(256), 0, st, W, numel4, q.bmax, q.mbits, 128 + B);
    hipLaunchKernelGGL(quant_hist_kernel, dim3(grid_h), dim3(1024), (size_t)B * 4, st, W, numel4, B, q.bmax, (int)grid_a, q.mbits,
                       q.counts);
    hipLaunchKernelGGL(quant_eval_kernel, dim3(kCandidates), dim3(1024), 0, st, q.mbits, q.counts, B, q.err, q.done, scale_out, shape.n,
                       alpha_out);
    return hip_status(hipGetLastError());
}

extern "C" int slim_quant_search_rows(const float *W, slim_shape shape, float *scale_out, float *alpha_out, void *stream)
{
    if (!W || !scale_out) return SLIM_ERR_NULL;
    if (shape.n < 1 || shape.k < 8 || shape.k % 8) return SLIM_ERR_SHAPE;
    if (!aligned16(W)) return SLIM_ERR_ALIGN;
    const int B = quant_bins((long)shape.k);
    const unsigned grid = (unsigned)(shape.n < 4096 ? shape.n : 4096);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (B == kRowBins)
        hipLaunchKernelGGL((quant_rows_kernel<true>), dim3(grid), dim3(256), (size_t)B * 4, st, W, shape.n, shape.k, B, scale_out, alpha_out);
    else
        hipLaunchKernelGGL((quant_rows_kernel<false>), dim3(grid), dim3(256), (size_t)B * 4, st, W, shape.n, shape.k, B, scale_out, alpha_out);
    return hip_status(hipGetLastError());
}
