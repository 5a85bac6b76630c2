// Products of the error saliency S (fp32) with a block of columns (fp32) on the fp16 matrix cores: both operands are
// split into two fp16 numbers, v = (hi + lo) 2^-e, and
//   S Z = Sh Zh + Sl Zh + Sh Zl     (what is left out, Sl Zl, is 2^-22 of a product)
// is added up in fp32 by V_MFMA_F32_32X32X16_F16.  hi + lo is v up to 2^-23 of v while lo is a normal number; e is one for all
// of S (and one for all of a block), so elements of S below 2^-17 of the largest, and of a block below 2^-8, are off by 2^-39 of the
// largest and by 2^-31 instead.  fp16 products are exact in fp32, and a sum of sixteen of them is rounded less often than
// with the fp32 instruction, which adds up two at a time, so the result is nearer to the exact one.  Measured against
// 64 bits (2-norm of the product, largest of a column and of a row, each relative; in brackets the fp32 instruction),
// 4096 x 4096 times 416 leading singular vectors:
//   S Z    saliency of calibration inputs          2.2e-7 (5.5e-7)   2.7e-7 (7.3e-7)   4.1e-7 (1.1e-6)
//          spanning 1e6, even in the logarithm     2.3e-7 (4.2e-7)   2.6e-7 (5.2e-7)   2.9e-7 (5.5e-7)
//          5 % of the channels 1e4 above the rest  1.4e-7 (1.4e-7)   2.4e-5 (4.1e-7)   1.8e-7 (1.7e-7)
//   S^T Q  saliency of calibration inputs          1.2e-7 (3.0e-7)   2.5e-7 (6.8e-7)   2.5e-7 (4.9e-7)
//          spanning 1e6, even in the logarithm     1.1e-7 (2.9e-7)   2.1e-7 (5.1e-7)   7.0e-6 (7.2e-7)
// The columns that lose in the third line are those of directions 1e4 below the leading ones: the error is of the direction of
// the leading ones, which the orthonormalisation takes out.  Adapters of saliencies that span up to 1e8 capture what they did
// with fp32 products, to the digits reported.
// Three fp16 instructions do the work of eight fp32 ones that take twice the time each.  4096 x 4096 times 416 columns: 200 us with the fp32 instruction (70 TFLOP/s),
// 58 us like this (52 and 6 to add the shares of K).
//   S is split once per call, into the operand order of the instruction, for S Z and for S^T Q;
//   the blocks are split where they are written (lora_apply_kernel, lora_init_kernel), columns as rows.
#include "slim_mma.h"

namespace slim {

// Largest magnitude of S -> the power of two that moves it to [2^13, 2^14); 1 for a zero matrix.
__device__ __forceinline__ float split_scale(unsigned max_bits)
{
    const int e = (int)(max_bits >> 23) - 127;                  // (S is finite; a subnormal maximum counts as 2^-127)
    return max_bits == 0u ? 1.0f : exp2f((float)min(13 - e, 126));
}

// S [n][k] -> hi and lo in the adapter layout (tiles of 32 rows x 16 columns), for S (rows n) and S^T (rows k,
// n padded to 32 columns).  A workgroup moves 64 x 64.
__global__ __launch_bounds__(256) void lora_split_kernel(const float *__restrict__ S, int n, int k, const unsigned *max_bits,
                                                         half_t *__restrict__ Sh, half_t *__restrict__ Sl, half_t *__restrict__ Th,
                                                         half_t *__restrict__ Tl)
{
    __shared__ float t[64][65];
    const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64, tid = threadIdx.x;
    const float sc = split_scale(*max_bits);
    for (int q = tid; q < 64 * 16; q += 256) {
        const int r = q >> 4, c = (q & 15) * 4;
        float4_t v = {0.f, 0.f, 0.f, 0.f};
        if (i0 + r < n) v = *reinterpret_cast<const float4_t *>(S + (size_t)(i0 + r) * k + j0 + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) t[r][c + e] = v[e] * sc;
    }
    __syncthreads();
    const int n32 = (n + 31) / 32 * 32;
    // (a 64-bit tl_piece(): columns 8 c8 .. of `row`, kcols columns)
    auto piece = [](int row, int c8, int kcols) {
        return ((size_t)(row >> 5) * (size_t)(kcols >> 4) + (size_t)(c8 >> 1)) * 1024u + (size_t)(((c8 & 1) << 5) + (row & 31)) * 16u;
    };
    auto put = [](half_t *hi, half_t *lo, size_t off, const float (&v)[8]) {
        half8_t h, l;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            h[e] = (half_t)v[e];
            l[e] = (half_t)(v[e] - (float)h[e]);
        }
        *reinterpret_cast<half8_t *>(reinterpret_cast<char *>(hi) + off) = h;
        *reinterpret_cast<half8_t *>(reinterpret_cast<char *>(lo) + off) = l;
    };
    // 64 lanes of one round write one tile of 32 x 16: contiguous
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int p = tid + 256 * q, tile = p >> 6, half = (p >> 5) & 1, r = p & 31;
        const int a = (tile & 1) * 32 + r, b = (tile >> 1) * 16 + half * 8;           // row a, columns b .. b + 7 of the block
        float v[8];
        if (i0 + a < n32) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = t[a][b + e];
            put(Sh, Sl, piece(i0 + a, (j0 + b) / 8, k), v);
        }
        if (i0 + b < n32) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = t[b + e][a];
            put(Th, Tl, piece(j0 + a, (i0 + b) / 8, n32), v);
        }
    }
}

struct SplitGemmArgs {
    const half_t *Ah, *Al;      // [rows][K] in the adapter layout
    const half_t *Bh, *Bl;      // [cols][K]
    const unsigned *max_bits;   // largest magnitude of what Ah + Al was split from
    float *P;                   // [splits][rows][cols]
    int rows, cols, K, ks;      // K a multiple of 32, ks (inputs per split) of 128
    int tiles_o;                // row tiles of 256
};

// Workgroup: 4 wavefronts, tile 256 rows x 128 columns, each wavefront 64 x 128 on fixed accumulators; the k-loop is
// dense_phase(), three times over the workgroup's share of K.
__global__ __launch_bounds__(256, 1) void lora_split_gemm_kernel(SplitGemmArgs a)
{
    constexpr int AT = 2;
    extern __shared__ __attribute__((aligned(16))) half_t lds[];   // two stage buffers
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, li = lane & 31, lb = lane >> 5;
    // the workgroups of a die (index mod 8) take neighbouring positions of the blocked order
    const int gx = (int)gridDim.x;
    const int q = gx % kDies == 0 ? ((int)blockIdx.x % kDies) * (gx / kDies) + (int)blockIdx.x / kDies : (int)blockIdx.x;
    const int w = blocked_tile(q, a.tiles_o, gx / a.tiles_o);
    const int o0 = (w % a.tiles_o) * 256 + wave * 64;
    const int t0 = (w / a.tiles_o) * 128;
    const int k0 = blockIdx.y * a.ks;
    const int klen = max(0, min(a.ks, a.K - k0));

    acc_reserve<AT>();
    static_for<16 * AT * NT>([&](auto r) { acc_write<r>(0.0f); });
    const uint32_t K = (uint32_t)a.K;
    const half_t *const lr = lds + li * SG_LD + 8 * lb;
    const int srow = tid >> 4, scol = (tid & 15) * 8;
    half_t *const lw = lds + srow * SG_LD + scol;
    uint4_t xs[XR];
    auto stage_store = [&](int u, const uint4_t (&reg)[XR], int only = -1) {
#pragma unroll
        for (int p = 0; p < XR; ++p)
            if (only < 0 || only == p) *reinterpret_cast<uint4_t *>(lw + u * SG_STAGE + p * 16 * SG_LD) = reg[p];
    };
    // descriptors of this tile's rows alone, so that the offsets stay in 32 bits whatever the matrices hold
    const int ob = (w % a.tiles_o) * 256;
    const uint32_t bytes_a = (uint32_t)min(8, ((a.rows + 31) / 32 - ob / 32)) * (K / 16) * 1024u;
    const uint32_t bytes_b = (uint32_t)min(128, a.cols - t0) * K * 2u;
    const size_t at_a = (size_t)ob * K, at_b = (size_t)t0 * K;
    const rsrc_t dah = make_rsrc(a.Ah + at_a, bytes_a), dal = make_rsrc(a.Al + at_a, bytes_a);
    const rsrc_t dbh = make_rsrc(a.Bh + at_b, bytes_b), dbl = make_rsrc(a.Bl + at_b, bytes_b);
    const uint32_t av = tl_piece((uint32_t)(wave * 64 + li), (uint32_t)k0 / 8 + lb, K);
    const uint32_t bv = ((uint32_t)srow * K + (uint32_t)k0 + (uint32_t)scol) * 2u;
    // smallest products first
    dense_phase<AT>(dal, av, (K / 16) * 1024u, 1024u, dbh, bv, 32u * K, klen, lr, xs, stage_store);
    dense_phase<AT>(dah, av, (K / 16) * 1024u, 1024u, dbl, bv, 32u * K, klen, lr, xs, stage_store);
    dense_phase<AT>(dah, av, (K / 16) * 1024u, 1024u, dbh, bv, 32u * K, klen, lr, xs, stage_store);
    acc_settle();
    const float sc = 1.0f / (split_scale(*a.max_bits) * kBlockSplit);
    // lane holds column t0 + 32 it + li, rows o .. o + 3 per (i, blk)
    float *const out = a.P + (size_t)blockIdx.y * a.rows * a.cols;
    static_for<NT>([&](auto itc) {
        constexpr int it = itc;
        const int t = t0 + 32 * it + li;
        if (t >= a.cols) return;
        static_for<AT>([&](auto ic) {
            constexpr int i = ic;
            static_for<16>([&](auto ec) {
                constexpr int e = ec;
                const int o = o0 + 32 * i + 8 * (e / 4) + 4 * lb + e % 4;
                const float v = acc_read<16 * (i * NT + it) + e>();
                if (o < a.rows) out[(size_t)o * a.cols + t] = v * sc;
            });
        });
    });
}

// Y[i] = sum_z P[z][i]
__global__ __launch_bounds__(256) void lora_split_reduce_kernel(const float4_t *__restrict__ P, int splits, size_t count4, float4_t *__restrict__ Y)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < count4; i += (size_t)gridDim.x * blockDim.x) {
        float4_t s = P[i];
        for (int z = 1; z < splits; ++z) s += P[(size_t)z * count4 + i];
        Y[i] = s;
    }
}

// The same, a workgroup per 16 rows of cols4 float4s, with the bits of the columns' largest magnitudes, in kColSlots rows of
// 4 cols4 words (zero before), a workgroup's in row blockIdx mod kColSlots.  In one row the adds to a word were 256 in
// turn, and 22 of 28 us (4096 x 416); now 8.
__global__ __launch_bounds__(512) void lora_split_reduce_max_kernel(const float4_t *__restrict__ P, int splits, int rows, int cols4,
                                                                    float4_t *__restrict__ Y, unsigned *__restrict__ colmax)
{
    __shared__ uint4_t part[512];
    const int rpp = 512 / cols4, row = threadIdx.x / cols4, col = threadIdx.x % cols4;
    const size_t count4 = (size_t)rows * cols4;
    const int end = min((int)blockIdx.x * 16 + 16, rows);
    float4_t mx = {0.f, 0.f, 0.f, 0.f};
    if (row < rpp)
        for (int r = blockIdx.x * 16 + row; r < end; r += rpp) {
            const size_t i = (size_t)r * cols4 + col;
            float4_t s = P[i];
            for (int z = 1; z < splits; ++z) s += P[(size_t)z * count4 + i];
            Y[i] = s;
#pragma unroll
            for (int e = 0; e < 4; ++e) mx[e] = fmaxf(mx[e], fabsf(s[e]));
        }
    part[threadIdx.x] = __builtin_bit_cast(uint4_t, mx);
    __syncthreads();
    if (row == 0) {
        for (int q = 1; q < rpp; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) mx[e] = fmaxf(mx[e], __uint_as_float(part[q * cols4 + col][e]));
        unsigned *const to = colmax + (size_t)(blockIdx.x % kColSlots) * 4 * cols4 + 4 * col;
#pragma unroll
        for (int e = 0; e < 4; ++e) atomicMax(&to[e], __float_as_uint(mx[e]));     // non-negative floats order as integers
    }
}

// Split-K factor: enough workgroups for the chip, shares of at least 128 of K.
int split_gemm_splits(int rows, int cols, int K)
{
    const long tiles = (long)((rows + 255) / 256) * ((cols + 127) / 128);
    int s = 1;
    while (tiles * s < 192 && s < 16 && K / (2 * s) >= 128) s *= 2;
    return s;
}

int launch_lora_split(const float *S, int n, int k, const unsigned *max_bits, half_t *Sh, half_t *Sl, half_t *Th, half_t *Tl, hipStream_t st)
{
    hipLaunchKernelGGL(lora_split_kernel, dim3((unsigned)(k / 64), (unsigned)((n + 63) / 64)), dim3(256), 0, st, S, n, k, max_bits, Sh, Sl, Th, Tl);
    return hip_status(hipGetLastError());
}

// Y [rows][cols] = A B^T (A scaled by split_scale(*max_bits), B by kBlockSplit); P: split_gemm_splits() x rows x cols floats.
// colmax (or null): kColSlots rows of zeros, which become bits of the columns' largest magnitudes (cols <= 1024).
int launch_lora_split_gemm(const half_t *Ah, const half_t *Al, const unsigned *max_bits, const half_t *Bh, const half_t *Bl, int rows, int cols,
                           int K, float *P, float *Y, unsigned *colmax, hipStream_t st)
{
    SplitGemmArgs a{Ah, Al, Bh, Bl, max_bits, nullptr, rows, cols, K, 0, (rows + 255) / 256};
    const int splits = split_gemm_splits(rows, cols, K);
    a.P = splits > 1 || colmax ? P : Y;
    a.ks = ((K + 127) / 128 + splits - 1) / splits * 128;
    const size_t lds = (size_t)2 * SG_STAGE * sizeof(half_t);
    hipLaunchKernelGGL(lora_split_gemm_kernel, dim3((unsigned)(a.tiles_o * ((cols + 127) / 128)), (unsigned)splits), dim3(256), lds, st, a);
    if (colmax) {
        hipLaunchKernelGGL(lora_split_reduce_max_kernel, dim3((unsigned)((rows + 15) / 16)), dim3(512), 0, st, reinterpret_cast<const float4_t *>(P),
                           splits, rows, cols / 4, reinterpret_cast<float4_t *>(Y), colmax);
    } else if (splits > 1) {
        const size_t count4 = (size_t)rows * cols / 4;          // cols is a multiple of 32
        const unsigned grid = (unsigned)((count4 + 255) / 256 < 2048 ? (count4 + 255) / 256 : 2048);
        hipLaunchKernelGGL(lora_split_reduce_kernel, dim3(grid), dim3(256), 0, st, reinterpret_cast<const float4_t *>(P), splits, count4,
                           reinterpret_cast<float4_t *>(Y));
    }
    return hip_status(hipGetLastError());
}

}  // namespace slim
