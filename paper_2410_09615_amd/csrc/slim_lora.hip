// Low-rank adapter computation: Naive-LoRA and SLiM-LoRA (paper Sec. 3.2, Eq. 8-11, Alg. 2).
//
//   E = W - W^C,  x = x~ + min|x~|,  S = E diag(x)            ([n][k], input channels are columns)
//   S ~= L R~ with L [n][r] orthonormal columns spanning the r leading left singular vectors,
//   R~ = L^T S;   R = R~ diag(1 / x)                          (W ~= W^C + L R)
//
// The truncated SVD is reached by subspace iteration: Q <- orth(S orth(S^T Q)), started from a
// seeded random block of r columns.  The product Q Q^T S converges to the best rank-r
// approximation of S (Eckart-Young); how far it is from it after `iters` rounds shows in the
// captured energy ||Q^T S||_F^2 the call reports.  Orthonormalisation is Cholesky QR in fp32
// (slim_lora_orth.hip), most of them a scaling of the columns where that loses nothing; the
// products of the iteration, and that for R~, run on the fp16 matrix cores with both operands as two fp16 numbers
// (slim_lora_split.hip: as near to the exact product as fp32); the Gram matrix of the report is an fp32 product.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "slim_internal.h"

namespace slim {

typedef float float16v_t __attribute__((ext_vector_type(16)));

// ---- C = op(A) B, fp32, row-major, optional split over K with atomic adds ----
struct SgemmArgs {
    const float *A, *B;
    float *C;
    int M, N, K;          // C is [M][N]; K is the summed dimension
    int lda, ldb;         // A is [M][K], or [K][M] when TA; B is [K][N]; C is contiguous
    int kchunk;           // K values per grid.z slice (a multiple of 16); C (zeroed before) is added to atomically when there are several
};

constexpr int kGM = 128, kGN = 128, kGK = 16, kGLd = kGM + 8;      // LDS: a k-value is one row of 128 values, padded to 136 floats

// Workgroup of 4 wavefronts, tile 128 x 128, each wavefront 64 x 64 = 2 x 2 matrix
// instruction blocks.  Both operand tiles sit in LDS as [k][row or column], as B and a transposed A come from memory, so that
// they are stored by 128 bits; lane (r = lane % 32, h = lane / 32) of a block reads the k-values 8 s + 4 h .. + 3 of
// its row, 32 neighbouring words per half of the lanes, four rows apart in different banks (hence the padding), and feeds
// them to four instructions; A and B use the same assignment of k-values to (lane half, instruction), so the sum is complete.
// (As [row][k] with one 128-bit read for the four they were stored word by word, eight lanes to a bank: 416 x 4096 over
// 4096 218 us, now 156, which the products of slim_lora_split.hip do in 50.)
template <bool TA>
__global__ __launch_bounds__(256) void sgemm_kernel(SgemmArgs a)
{
    static_assert(kGM == kGN, "one row length");
    __shared__ __attribute__((aligned(16))) float As[kGK * kGLd];
    __shared__ __attribute__((aligned(16))) float Bs[kGK * kGLd];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int m0 = blockIdx.y * kGM, n0 = blockIdx.x * kGN;
    const int kb = blockIdx.z * a.kchunk, ke = min(a.K, kb + a.kchunk);
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;
    const int r = lane & 31, h = lane >> 5;

    float16v_t acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    float4_t ra[2], rb[2];
    // loads of the k-slab starting at k0 into registers (zeros outside the matrices)
    auto load_slab = [&](int k0) {
        if constexpr (!TA) {
            // A [M][K]: thread -> row tid / 4 (+ 64), k-values 4 (tid % 4) .. + 3
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int row = m0 + (tid >> 2) + 64 * i, kk = k0 + (tid & 3) * 4;
                ra[i] = (row < a.M && kk < ke) ? *reinterpret_cast<const float4_t *>(a.A + (size_t)row * a.lda + kk)
                                               : float4_t{0.f, 0.f, 0.f, 0.f};
            }
        } else {
            // A [K][M]: thread -> k-value tid / 32 (+ 8), rows 4 (tid % 32) .. + 3
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int kk = k0 + (tid >> 5) + 8 * i, row = m0 + (tid & 31) * 4;
                ra[i] = (kk < ke && row < a.M) ? *reinterpret_cast<const float4_t *>(a.A + (size_t)kk * a.lda + row)
                                               : float4_t{0.f, 0.f, 0.f, 0.f};
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int kk = k0 + (tid >> 5) + 8 * i, col = n0 + (tid & 31) * 4;
            rb[i] = (kk < ke && col < a.N) ? *reinterpret_cast<const float4_t *>(a.B + (size_t)kk * a.ldb + col)
                                           : float4_t{0.f, 0.f, 0.f, 0.f};
        }
    };
    auto store_slab = [&]() {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if constexpr (!TA) {
#pragma unroll
                for (int e = 0; e < 4; ++e) As[((tid & 3) * 4 + e) * kGLd + (tid >> 2) + 64 * i] = ra[i][e];
            } else {
                *reinterpret_cast<float4_t *>(As + ((tid >> 5) + 8 * i) * kGLd + (tid & 31) * 4) = ra[i];
            }
            *reinterpret_cast<float4_t *>(Bs + ((tid >> 5) + 8 * i) * kGLd + (tid & 31) * 4) = rb[i];
        }
    };

    // M and N are multiples of 4 wherever a 128-bit load straddles the edge (row counts
    // that are not appear only as K or as the row index of an untransposed A)
    load_slab(kb);
    for (int k0 = kb; k0 < ke; k0 += kGK) {
        __syncthreads();                      // the previous slab has been read
        store_slab();
        __syncthreads();
        if (k0 + kGK < ke) load_slab(k0 + kGK);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            float4_t av[2], bv[2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    av[i][e] = As[(8 * s + 4 * h + e) * kGLd + wm + 32 * i + r];
                    bv[i][e] = Bs[(8 * s + 4 * h + e) * kGLd + wn + 32 * i + r];
                }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[i][e], bv[j][e], acc[i][j], 0, 0, 0);
        }
    }
    // register 4 b + e of a block: row 8 b + 4 h + e, column r
    const bool add = gridDim.z > 1;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int col = n0 + wn + 32 * j + r;
            if (col >= a.N) continue;
#pragma unroll
            for (int b = 0; b < 4; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = m0 + wm + 32 * i + 8 * b + 4 * h + e;
                    if (row >= a.M) continue;
                    float *c = a.C + (size_t)row * a.N + col;
                    if (add)
                        atomicAdd(c, acc[i][j][4 * b + e]);
                    else
                        *c = acc[i][j][4 * b + e];
                }
        }
}

__global__ void fill_kernel(float *p, size_t count, float v)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

static int launch_fill(float *p, size_t count, float v, hipStream_t st)
{
    const unsigned grid = (unsigned)std::min<size_t>((count + 255) / 256, 2048);
    hipLaunchKernelGGL(fill_kernel, dim3(grid ? grid : 1), dim3(256), 0, st, p, count, v);
    return hip_status(hipGetLastError());
}

// C = op(A) B.  Few tiles and a long K: K is split over grid.z and C (zeroed first) is added to.
static int sgemm(bool ta, const float *A, int lda, const float *B, int ldb, float *C, int M, int N, int K, hipStream_t st)
{
    if (M <= 0 || N <= 0 || K <= 0) return SLIM_OK;
    SgemmArgs a{A, B, C, M, N, K, lda, ldb, 0};
    const int tm = (M + kGM - 1) / kGM, tn = (N + kGN - 1) / kGN;
    int splits = 1;
    if (tm * tn < 512) splits = (512 + tm * tn - 1) / (tm * tn);
    const int kslabs = (K + kGK - 1) / kGK;
    if (splits > kslabs / 16) splits = kslabs / 16 > 0 ? kslabs / 16 : 1;   // at least 256 k-values per slice (416 x 416 over 4096: with 64 37 us, now 32)
    a.kchunk = (kslabs + splits - 1) / splits * kGK;
    splits = (K + a.kchunk - 1) / a.kchunk;
    if (splits > 1) {
        const int rc = launch_fill(C, (size_t)M * N, 0.f, st);
        if (rc != SLIM_OK) return rc;
    }
    const dim3 grid(tn, tm, splits);
    if (ta)
        hipLaunchKernelGGL((sgemm_kernel<true>), grid, dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((sgemm_kernel<false>), grid, dim3(256), 0, st, a);
    return hip_status(hipGetLastError());
}

// The sums of the report, in kSumSlots words a line apart each: adds to one word serialise (10 ns each, 1024 workgroups), and
// so do the maxima, of which only those that change the word are sent.
constexpr int kSumSlots = 32, kSumStride = 16;
// One atomic add per workgroup of 256 threads.
__device__ __forceinline__ void block_add(float part, float *slots)
{
    __shared__ float red4[4];
    part = wave_sum(part);
    if ((threadIdx.x & 63) == 0) red4[threadIdx.x >> 6] = part;
    __syncthreads();
    if (threadIdx.x == 0) atomicAdd(slots + (blockIdx.x + blockIdx.y * gridDim.x) % kSumSlots * kSumStride, red4[0] + red4[1] + red4[2] + red4[3]);
}
// The largest of a workgroup's non-negative values into a word that holds the bits of one (they order as integers).
__device__ __forceinline__ void block_max(float mx, float *dst)
{
    __shared__ float mx4[4];
    mx = wave_max(mx);
    if ((threadIdx.x & 63) == 0) mx4[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x != 0) return;
    unsigned *const word = reinterpret_cast<unsigned *>(dst);
    const unsigned bits = __float_as_uint(fmaxf(fmaxf(mx4[0], mx4[1]), fmaxf(mx4[2], mx4[3])));
    if (bits > __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(word, bits);
}

// ---- x = x~ + min|x~| (Alg. 2), or ones ----
__global__ __launch_bounds__(1024) void lora_shift_kernel(const float *xt, int k, float *x)
{
    __shared__ float red[16];
    float mn = INFINITY;
    if (xt)
        for (int i = threadIdx.x; i < k; i += blockDim.x) mn = fminf(mn, fabsf(xt[i]));
    mn = -wave_max(-mn);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mn;
    __syncthreads();
    mn = red[0];
    for (int w = 1; w < (int)blockDim.x / 64; ++w) mn = fminf(mn, red[w]);
    for (int i = threadIdx.x; i < k; i += blockDim.x) x[i] = xt ? xt[i] + mn : 1.0f;
}

// ---- S = (W - W^C) diag(x); the packed bytes are read in their tiled layout ----
// A workgroup has the 32 groups of four inputs of a column tile and every eighth of its rows in turn, so that a thread keeps the maxima of its four
// channels in registers.  s2: slots of ||S||_F^2, mx_word: bits of the largest magnitude, channel_max: kChannelSlots rows of bits of the channels' largest.
// HBM-bound (W and S, 8 bytes per weight): 4096 x 4096 26 us (27 with a thread per group of any column and no channels' maxima).
constexpr int kErrorRows = 8;
__global__ __launch_bounds__(32 * kErrorRows) void lora_error_kernel(const float *__restrict__ W, const uint8_t *__restrict__ qvals,
                                                                     const uint8_t *__restrict__ meta, const float *__restrict__ scale,
                                                                     const float *__restrict__ x, int n, int k, int rows, float *__restrict__ S,
                                                                     float *s2, float *mx_word, unsigned *channel_max)
{
    __shared__ float4_t red[kErrorRows][32];
    const uint32_t groups = (uint32_t)k / 4, kt = pk_ktiles(k), g = 32 * blockIdx.x + threadIdx.x % 32;
    const int first = (int)blockIdx.y * rows + (int)threadIdx.x / 32, end = min(n, (int)blockIdx.y * rows + rows);
    const float4_t xv = reinterpret_cast<const float4_t *>(x)[g];
    float part = 0.f;
    float4_t mx = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int o = first; o < end; o += kErrorRows) {
        const uint32_t q = qvals[pk_qoff((uint32_t)o, g, kt)];
        const uint32_t mb = meta[pk_moff((uint32_t)o, g >> 1, kt)];
        const uint32_t m4 = (g & 1) ? (mb >> 4) : (mb & 15u);
        const float s = scale[o];
        const float4_t w = reinterpret_cast<const float4_t *>(W)[(size_t)o * groups + g];
        const uint32_t i0 = m4 & 3u, i1 = (m4 >> 2) & 3u;
        const float w0 = (float)nibble_to_int(q & 15u) * s, w1 = (float)nibble_to_int(q >> 4) * s;
        float4_t e;
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            const float wc = i == i1 ? w1 : (i == i0 ? w0 : 0.f);
            e[i] = (w[i] - wc) * xv[i];
            part += e[i] * e[i];
            mx[i] = fmaxf(mx[i], fabsf(e[i]));
        }
        reinterpret_cast<float4_t *>(S)[(size_t)o * groups + g] = e;
    }
    block_add(part, s2);
    red[threadIdx.x / 32][threadIdx.x % 32] = mx;
    block_max(fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3])), mx_word);
    __syncthreads();
    if (threadIdx.x >= 128) return;
    const float *const column = reinterpret_cast<const float *>(red) + threadIdx.x;
    float c = 0.f;
#pragma unroll
    for (int i = 0; i < kErrorRows; ++i) c = fmaxf(c, column[128 * i]);
    atomicMax(channel_max + (size_t)(blockIdx.y % kChannelSlots) * k + 128 * blockIdx.x + threadIdx.x, __float_as_uint(c));
}

// ---- start block: uniform in (-1, 1) from a hash of (seed, element), columns >= r zero ----
__device__ __forceinline__ uint32_t mix32(uint32_t v)
{
    v ^= v >> 16;
    v *= 0x7feb352du;
    v ^= v >> 15;
    v *= 0x846ca68bu;
    v ^= v >> 16;
    return v;
}

// Element t = row * l + column; written to Z, or as the two fp16 numbers of the split products, columns as rows: blockIdx.y is
// the column, so that the stores are contiguous (4096 x 416: 20 -> 5 us).
__global__ __launch_bounds__(256) void lora_init_kernel(float *Z, half_t *hi, half_t *lo, int rows, int l, int r, uint32_t seed)
{
    const int c = blockIdx.y;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < rows; i += gridDim.x * blockDim.x) {
        const size_t t = (size_t)i * l + c;
        const uint32_t hsh = mix32(mix32((uint32_t)t ^ seed) + (uint32_t)(t >> 32) + 0x9e3779b9u * seed);
        const float z = c < r ? ((float)(hsh >> 8) + 0.5f) * (2.0f / 16777216.0f) - 1.0f : 0.f;
        if (Z) {
            Z[t] = z;
            continue;
        }
        const float v = z * kBlockSplit;
        const half_t x = (half_t)v;
        hi[(size_t)c * rows + i] = x;
        lo[(size_t)c * rows + i] = (half_t)((v - (float)x) * kLowSplit);
    }
}

constexpr int kSplitMax = 1 << 22;       // n and k below this: a tile's rows of the split matrices have 32-bit offsets
constexpr int kMaxBlock = 1024;          // columns of the iteration block (rank_pad)

size_t orth_floats(int l);                                                                           // slim_lora_orth.hip
size_t orth_hand_words();
int launch_orth(const float *in, float *out, half_t *hi, half_t *lo, int rows, int l, float *ws, unsigned *hand, unsigned seq, int h, int last,
                hipStream_t st);
unsigned *orth_column_max(float *ws, int l, int which);
int split_gemm_splits(int rows, int cols, int K);                                                    // slim_lora_split.hip
int launch_lora_split(const float *S, int n, int k, const unsigned *max_bits, const unsigned *channel_max, half_t *Sh, half_t *Sl, half_t *Th, half_t *Tl,
                      float *channel_factor, hipStream_t st);
int launch_lora_split_gemm(const half_t *Ah, const half_t *Al, const unsigned *max_bits, const float *row_factor, const half_t *Bh, const half_t *Bl, int rows,
                           int cols, int K, float *P, float *Y, unsigned *colmax, hipStream_t st);

// ---- results: L fp16 [n][r] = Q[:, :r];  R fp16 [r][k] = R~[:r] / x;  r2: slots of ||R~[:r]||_F^2 ----
__global__ void lora_out_l_kernel(const float *Q, int n, int l, int r, half_t *L)
{
    const size_t total = (size_t)n * r;
    for (size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (size_t)gridDim.x * blockDim.x) {
        const size_t i = t / r, c = t % r;
        L[t] = (half_t)Q[i * l + c];
    }
}

// Rt: [k][l], R~ transposed.  A workgroup turns 64 channels x 64 columns.
__global__ __launch_bounds__(256) void lora_out_r_kernel(const float *__restrict__ Rt, const float *__restrict__ x, int k, int l, int r,
                                                         half_t *__restrict__ R, float *r2)
{
    __shared__ float t[64][65];
    const int j0 = blockIdx.x * 64, c0 = blockIdx.y * 64;        // (k is a multiple of 64, l of 32)
    float part = 0.f;
    for (int q = threadIdx.x; q < 64 * 16; q += 256) {
        const int j = q >> 4, c = (q & 15) * 4;
        float4_t v = {0.f, 0.f, 0.f, 0.f};
        if (c0 + c < l) v = *reinterpret_cast<const float4_t *>(Rt + (size_t)(j0 + j) * l + c0 + c);
        const float xj = x[j0 + j];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (c0 + c + e < r) part += v[e] * v[e];
            t[j][c + e] = v[e] / xj;
        }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < 64 * 16; q += 256) {
        const int c = q >> 4, j = (q & 15) * 4;
        if (c0 + c < r)
            *reinterpret_cast<half4_t *>(R + (size_t)(c0 + c) * k + j0 + j) =
                half4_t{(half_t)t[j][c], (half_t)t[j + 1][c], (half_t)t[j + 2][c], (half_t)t[j + 3][c]};
    }
    block_add(part, r2);
}

// sq[2] = max |G - I| over the leading r x r block (orthonormality of the final Q), infinite where an entry is a NaN, which the
// maxima on the way to the report would drop
__global__ __launch_bounds__(256) void lora_ortho_kernel(const float *G, int l, int r, float *sq)
{
    float mx = 0.f;
    for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < r * r; t += gridDim.x * blockDim.x) {
        const int i = t / r, c = t % r;
        const float d = fabsf(G[(size_t)i * l + c] - (i == c ? 1.0f : 0.f));
        mx = fmaxf(mx, d == d ? d : __builtin_inff());
    }
    block_max(mx, sq + 2);
}

// the four numbers of the report, out of the workspace (a kernel, so that the call is kernels only)
__global__ __launch_bounds__(64) void lora_report_kernel(const float *sq, const float *sums, float *diag)
{
    const int t = threadIdx.x;
    if (t < 2) {
        float s = 0.f;
        for (int i = 0; i < kSumSlots; ++i) s += sums[(t * kSumSlots + i) * kSumStride];
        diag[t] = s;
    }
    if (t == 2) diag[2] = sq[2];
    if (t == 3) diag[3] = 0.f;
}

// Words that a call clears: maxima, slots of the two sums, the words that the orth()s' workgroups hand over by, the channels' maxima.
static size_t lora_cleared(int k) { return 64 + 2 * kSumSlots * kSumStride + orth_hand_words() + (size_t)kChannelSlots * k; }

struct LoraPlan {
    int l;                      // columns of the iteration block: rank padded as the layer's adapters are
    bool split;                 // products on the fp16 matrix cores (lora_split_gemm_kernel)
    size_t x, S, half[4], Q, Y, Z, P, blk[4], G, O, Rt, factor, sq, total;      // byte offsets (O: the orthonormalisation's own)
};

static size_t up256(size_t v) { return (v + 255) / 256 * 256; }

static LoraPlan plan_lora(int n, int k, int rank)
{
    LoraPlan p{};
    p.l = slim_rank_pad(rank);
    const size_t l = p.l, big = n > k ? n : k;
    size_t off = 0;
    auto take = [&](size_t floats) {
        const size_t at = off;
        off += up256(floats * sizeof(float));
        return at;
    };
    p.x = take(k);
    p.S = take((size_t)n * k);
    p.Q = take(big * l);
    p.Y = take(big * l);
    const int n32 = (n + 31) / 32 * 32;
    p.split = n32 < kSplitMax && k < kSplitMax;
    if (p.split) {
        // S and S^T as two fp16 matrices each, the blocks [l][n32] and [l][k] likewise, partial sums of the products
        for (int i = 0; i < 4; ++i) p.half[i] = take(((size_t)n32 * k + 1) / 2);
        for (int i = 0; i < 4; ++i) p.blk[i] = take((l * (i < 2 ? n32 : k) + 1) / 2);
        const size_t pn = (size_t)split_gemm_splits(n, p.l, k) * n * l, pk = (size_t)split_gemm_splits(k, p.l, n32) * k * l;
        p.P = take(pn > pk ? pn : pk);
    } else {
        p.Z = take((size_t)k * l);
    }
    p.G = take(l * l);
    p.O = take(orth_floats(p.l));
    p.Rt = take(l * k);
    p.factor = take(k);
    p.sq = take(lora_cleared(k));
    p.total = off;
    return p;
}

}  // namespace slim

using namespace slim;

extern "C" int slim_adapters_workspace_bytes(slim_shape shape, size_t *bytes)
{
    if (!bytes) return SLIM_ERR_NULL;
    if (shape.n < 1 || shape.k < 128 || shape.k % 128 || shape.rank < 1 || shape.rank > shape.n || shape.rank > shape.k ||
        slim_rank_pad(shape.rank) > kMaxBlock)
        return SLIM_ERR_SHAPE;
    *bytes = plan_lora(shape.n, shape.k, shape.rank).total;
    return SLIM_OK;
}

extern "C" int slim_compute_adapters(const float *W, const uint8_t *qvals, const uint8_t *meta, const float *scale,
                                     slim_shape shape, const float *x_tilde, int32_t iters, uint32_t seed, slim_half *L,
                                     slim_half *R, float *diag, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!W || !qvals || !meta || !scale || !L || !R) return SLIM_ERR_NULL;
    const int n = shape.n, k = shape.k, r = shape.rank;
    if (n < 1 || k < 128 || k % 128 || r < 1 || r > n || r > k || slim_rank_pad(r) > kMaxBlock || iters < 0 || iters > 1000)
        return SLIM_ERR_SHAPE;
    if (!aligned16(W) || !aligned16(qvals) || !aligned16(meta) || !aligned16(scale) || !aligned16(L) || !aligned16(R) ||
        (x_tilde && !aligned16(x_tilde)) || !aligned16(workspace))
        return SLIM_ERR_ALIGN;
    const LoraPlan p = plan_lora(n, k, r);
    if (!workspace || workspace_bytes < p.total) return SLIM_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    char *ws = static_cast<char *>(workspace);
    float *x = reinterpret_cast<float *>(ws + p.x), *S = reinterpret_cast<float *>(ws + p.S);
    float *Q = reinterpret_cast<float *>(ws + p.Q), *Y = reinterpret_cast<float *>(ws + p.Y);
    float *P = p.split ? reinterpret_cast<float *>(ws + p.P) : nullptr, *G = reinterpret_cast<float *>(ws + p.G);
    float *O = reinterpret_cast<float *>(ws + p.O), *Rt = reinterpret_cast<float *>(ws + p.Rt);
    float *sq = reinterpret_cast<float *>(ws + p.sq), *factor = reinterpret_cast<float *>(ws + p.factor);
    const int l = p.l;
    const int q = iters == 0 ? 16 : iters;
    int rc;
#define SLIM_TRY(call)            \
    do {                          \
        rc = (call);              \
        if (rc != SLIM_OK) return rc; \
    } while (0)
    auto launched = [&]() { return hip_status(hipGetLastError()); };
    auto grid_for = [](size_t count) { return dim3((unsigned)std::min<size_t>((count + 255) / 256, 4096)); };

    // (in the order of lora_cleared())
    float *const s2 = sq + 64, *const r2 = s2 + kSumSlots * kSumStride;
    unsigned *const hand = reinterpret_cast<unsigned *>(r2 + kSumSlots * kSumStride);
    unsigned *const channel_max = hand + orth_hand_words();
    unsigned orths = 0;
    auto orth = [&](const float *in, float *out, half_t *hi, half_t *lo, int rows, int h, int last) {
        return launch_orth(in, out, hi, lo, rows, p.l, O, hand, ++orths, h, last, st);
    };
    SLIM_TRY(launch_fill(sq, lora_cleared(k), 0.f, st));
    hipLaunchKernelGGL(lora_shift_kernel, dim3(1), dim3(1024), 0, st, x_tilde, k, x);
    SLIM_TRY(launched());
    // about 1024 workgroups
    const int column_tiles = k / 128, passes = (n + kErrorRows - 1) / kErrorRows, chunks = std::min(passes, (1023 + column_tiles) / column_tiles);
    const int rows = (passes + chunks - 1) / chunks * kErrorRows;
    hipLaunchKernelGGL(lora_error_kernel, dim3((unsigned)column_tiles, (unsigned)((n + rows - 1) / rows)), dim3(32 * kErrorRows), 0, st, W, qvals, meta, scale,
                       (const float *)x, n, k, rows, S, s2, sq + 4, channel_max);
    SLIM_TRY(launched());

    float *Z = p.split ? nullptr : reinterpret_cast<float *>(ws + p.Z);
    half_t *Sh[4] = {}, *blk[4] = {};        // S, S^T: hi and lo; Q, Z: hi and lo
    const unsigned *mx = reinterpret_cast<const unsigned *>(sq + 4);
    const int n32 = (n + 31) / 32 * 32;
    if (p.split) {
        for (int i = 0; i < 4; ++i) {
            Sh[i] = reinterpret_cast<half_t *>(ws + p.half[i]);
            blk[i] = reinterpret_cast<half_t *>(ws + p.blk[i]);
        }
        SLIM_TRY(launch_lora_split(S, n, k, mx, channel_max, Sh[0], Sh[1], Sh[2], Sh[3], factor, st));
    }
    hipLaunchKernelGGL(lora_init_kernel, dim3((unsigned)std::min((k + 255) / 256, 1024), (unsigned)l), dim3(256), 0, st, Z, blk[2], blk[3], k, l, r, seed);
    SLIM_TRY(launched());
    const int last = 2 * q;                  // products with S^T and S, in turn, after the first
    // (column maxima: for a block that may only be scaled)
    auto colmax = [&](int h) { return h > 0 && h < last ? orth_column_max(O, l, h & 1) : nullptr; };
    auto times_z = [&](int h) {              // Y = S Z     [n][l]
        return p.split ? launch_lora_split_gemm(Sh[0], Sh[1], mx, nullptr, blk[2], blk[3], n, l, k, P, Y, colmax(h), st)
                       : sgemm(false, S, k, Z, l, Y, n, l, k, st);
    };
    auto times = [&](const float *q, float *to, unsigned *cm) {          // S^T q     [k][l]
        return p.split ? launch_lora_split_gemm(Sh[2], Sh[3], nullptr, factor, blk[0], blk[1], k, l, n32, P, to, cm, st) : sgemm(true, S, k, q, l, to, k, l, n, st);
    };
    auto times_q = [&](int h) { return times(Q, Y, colmax(h)); };        // Y = S^T Q

    SLIM_TRY(times_z(0));
    for (int h = 0; h < last; h += 2) {
        SLIM_TRY(orth(Y, p.split ? nullptr : Q, blk[0], blk[1], n, p.split ? h : -1, last));
        SLIM_TRY(times_q(h + 1));
        SLIM_TRY(orth(Y, Z, blk[2], blk[3], k, p.split ? h + 1 : -1, last));
        SLIM_TRY(times_z(h + 2));
    }
    SLIM_TRY(orth(Y, Q, nullptr, nullptr, n, -1, last));
    SLIM_TRY(orth(Q, Y, blk[0], blk[1], n, -1, last));      // second pass: orthonormal to rounding
    SLIM_TRY(times(Y, Rt, nullptr));         // R~ = Q^T S, transposed
    SLIM_TRY(sgemm(true, Y, l, Y, l, G, l, l, n, st));           // Gram of the final block, for the report
    hipLaunchKernelGGL(lora_ortho_kernel, dim3(std::min(grid_for((size_t)r * r).x, 256u)), dim3(256), 0, st, (const float *)G, l, r, sq);
    SLIM_TRY(launched());
    hipLaunchKernelGGL(lora_out_l_kernel, grid_for((size_t)n * r), dim3(256), 0, st, (const float *)Y, n, l, r,
                       reinterpret_cast<half_t *>(L));
    SLIM_TRY(launched());
    hipLaunchKernelGGL(lora_out_r_kernel, dim3((unsigned)(k / 64), (unsigned)((r + 63) / 64)), dim3(256), 0, st, (const float *)Rt, (const float *)x, k, l, r,
                       reinterpret_cast<half_t *>(R), r2);
    SLIM_TRY(launched());
    if (diag) {
        hipLaunchKernelGGL(lora_report_kernel, dim3(1), dim3(64), 0, st, (const float *)sq, (const float *)s2, diag);
        SLIM_TRY(launched());
    }
#undef SLIM_TRY
    return SLIM_OK;
}
