// Products of the error saliency S (fp32) with a block of columns (fp32) on the fp16 matrix cores: both operands are
// split into two fp16 numbers, v = (hi + 2^-11 lo) 2^-e, and
//   S Z = Sh Zh + 2^-11 (Sl Zh + Sh Zl)     (what is left out, 2^-22 Sl Zl, is 2^-22 of a product)
// is added up in fp32 by V_MFMA_F32_32X32X16_F16, the second sum by itself.  hi + 2^-11 lo is v up to 2^-22 of v while hi is a normal number; e is one for all
// of S, one for a channel of S^T and one for all of a block, so elements of S (of a channel of S^T) below 2^-27 of the largest, and of a block below 2^-20, are off by 2^-49 of the
// largest and by 2^-42 instead.  fp16 products are exact in fp32, and a sum of sixteen of them is rounded less often than
// with the fp32 instruction, which adds up two at a time.  Measured against 64 bits (2-norm of the product, largest of a column and of a row, each
// relative; in brackets a product in fp32 by the host's library, in blocks), 4096 x 4096 times 409 leading singular vectors:
//   S Z    saliency of calibration inputs          2.0e-7 (2.5e-7)   2.6e-7 (3.1e-7)   3.4e-7 (4.3e-7)
//          saliency spanning 1e6                   2.3e-7 (2.0e-7)   2.7e-7 (2.6e-7)   2.9e-7 (2.5e-7)
//          5 % of the channels 1e4 above the rest  1.5e-7 (1.2e-7)   1.9e-7 (1.8e-7)   1.8e-7 (1.5e-7)
//          rows of W spanning 1e6                  1.1e-7 (1.2e-7)   2.0e-7 (2.2e-7)   2.7e-7 (3.1e-7)
//          rows of W spanning 1e9                  1.1e-7 (1.2e-7)   2.5e-7 (2.9e-7)   4.7e-6 (3.1e-7)
//   S^T Q  saliency of calibration inputs          1.1e-7 (1.3e-7)   2.6e-7 (3.0e-7)   1.8e-7 (2.1e-7)
//          saliency spanning 1e6                   1.1e-7 (1.2e-7)   1.9e-7 (2.2e-7)   2.7e-7 (3.1e-7)
//          spanning 1e9, weights of channels 1 / that   1.4e-7 (1.6e-7)   1.6e-7 (1.8e-7)   1.8e-7 (2.1e-7)
//          rows of W spanning 1e6                  2.3e-7 (2.1e-7)   2.7e-7 (2.5e-7)   2.8e-7 (2.5e-7)
// (With lo unscaled a row of S Z was off by 9e-6 and 8e-3 where the rows of W span 1e6 and 1e9, a column by 1.2e-5 where 5 % of the channels are 1e4 above
// the rest; with a channel of S^T scaled by its saliency instead of its own maximum S^T Q was off by 4.7e-4 in the last line but one.)
// The shares of K are added up in 64 bits and rounded once.
// Three fp16 instructions do the work of eight fp32 ones that take twice the time each.  4096 x 4096 times 416 columns: 200 us with the fp32 instruction (70 TFLOP/s),
// 53 us like this (44, and 9 to add the shares of K and find the columns' largest magnitudes).
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

// S [n][k] -> hi and lo in the adapter layout (tiles of 32 rows x 16 columns), for S (rows n) and S^T (rows k, each scaled by its own largest
// magnitude; n padded to 32 columns).  max_bits: the largest magnitude of S; channel_max: kChannelSlots rows of the channels';
// channel_factor: the reciprocals of their scales.  A workgroup moves 64 x 64.
__global__ __launch_bounds__(256) void lora_split_kernel(const float *__restrict__ S, int n, int k, const unsigned *max_bits,
                                                         const unsigned *__restrict__ channel_max, half_t *__restrict__ Sh, half_t *__restrict__ Sl,
                                                         half_t *__restrict__ Th, half_t *__restrict__ Tl, float *__restrict__ channel_factor)
{
    __shared__ float t[64][65], channel_scale[64];
    const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64, tid = threadIdx.x;
    const float sc = split_scale(*max_bits);
    if (tid < 64) {
        unsigned mx = 0u;
#pragma unroll
        for (int q = 0; q < kChannelSlots; ++q) mx = max(mx, channel_max[(size_t)q * k + j0 + tid]);
        channel_scale[tid] = split_scale(mx);
        if (i0 == 0) channel_factor[j0 + tid] = 1.0f / split_scale(mx);
    }
    for (int q = tid; q < 64 * 16; q += 256) {
        const int r = q >> 4, c = (q & 15) * 4;
        float4_t v = {0.f, 0.f, 0.f, 0.f};
        if (i0 + r < n) v = *reinterpret_cast<const float4_t *>(S + (size_t)(i0 + r) * k + j0 + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) t[r][c + e] = v[e];
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
            l[e] = (half_t)((v[e] - (float)h[e]) * kLowSplit);
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
            for (int e = 0; e < 8; ++e) v[e] = t[a][b + e] * sc;
            put(Sh, Sl, piece(i0 + a, (j0 + b) / 8, k), v);
        }
        if (i0 + b < n32) {
            const float sca = channel_scale[a];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = t[b + e][a] * sca;
            put(Th, Tl, piece(j0 + a, (i0 + b) / 8, n32), v);
        }
    }
}

struct SplitGemmArgs {
    const half_t *Ah, *Al;      // [rows][K] in the adapter layout
    const half_t *Bh, *Bl;      // [cols][K]
    const unsigned *max_bits;   // largest magnitude of what Ah + Al was split from, or null: rows with scales of their own
    float *P;                   // [splits][rows][cols]
    int rows, cols, K, ks;      // K a multiple of 32, ks (inputs per split) of 128
    int tiles_o;                // row tiles of 256
};

// acc(i, it) += Ah_i Bh_it^T and small(i, it) += Al_i Bh_it^T + Ah_i Bl_it^T over K inputs (a multiple of 32), 16 per step of
// V_MFMA_F32_32X32X16_F16, accumulators as in dense_phase() (slim_mma.h).  Both parts of both operands are at hand, so
// each is fetched once for the three products.  Accumulator tiles 0 .. are acc, kSmall .. are small: what is of the
// order of 2^-11 is added up by itself.
//   A: from memory into registers, seven steps (of 24 matrix instructions) ahead in eight rotating sets;
//   B: 128 columns x 128 inputs per stage and part in LDS, written by the loads themselves while the stage before it is
//      multiplied.  A column's stage is a row of 256 bytes without padding, its pieces of 16 bytes permuted by the
//      column number, so that the sixteen lanes that read together hit all banks once.
constexpr int kSplitAT = 2, kSmall = kSplitAT * NT;
constexpr uint32_t kSplitStage = 128 * SG_BK * 2;       // bytes of a stage of one part of B
struct SplitOperands {
    rsrc_t a[2], b[2];                // hi, lo
    uint32_t av, a_tile, a_step;      // A: this lane's offset for row tile 0, step 0; bytes between row tiles, between steps
    uint32_t bv, b_pass;              // B: this lane's offset for stage 0; bytes between the passes of 16 columns
    uint32_t b_lds;                   // LDS address of this wavefront's part of pass 0 of buffer 0, hi
};
__device__ __forceinline__ void split_phase(const SplitOperands &o, int K, const char *lds_c, int li, int lb)
{
    constexpr int AT = kSplitAT;
    const int nst = K / 16;
    const int stages = (K + SG_BK - 1) / SG_BK;
    // (everything in the lane's offset, which is range-checked)
    auto fetch_b = [&](int s, int u, int q) {        // load q of a stage: pass q / 2 of part q % 2, to buffer u
        load_to_lds(o.b[q & 1], o.bv + (uint32_t)s * (SG_BK * 2) + (uint32_t)(q >> 1) * o.b_pass, 0u,
                    o.b_lds + (uint32_t)(2 * u + (q & 1)) * kSplitStage + (uint32_t)(q >> 1) * 4096u);
    };
    uint4_t la[8][AT][2];
    // steps past the last read zeros (2^31 more than a lane's offset is past the end of every descriptor here), so that every
    // stage is whole: with exits from the middle of a stage the compiler copies the sets, and waits for all of them
    auto fetch_a = [&](int g, int i, int h) { return load16(o.a[h], o.av, g < nst ? (uint32_t)i * o.a_tile + (uint32_t)g * o.a_step : 0x80000000u); };
    const char *const lr = lds_c + li * 256;
    half8_t b[2][2];
    auto read_b = [&](int u, int it, int j) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            b[it & 1][h] = *reinterpret_cast<const half8_t *>(lr + (2 * u + h) * kSplitStage + it * 32 * 256 + (((2 * j + lb) ^ (li & 15)) << 4));
    };
#pragma unroll
    for (int q = 0; q < 2 * XR; ++q) fetch_b(0, 0, q);
#pragma unroll
    for (int g = 0; g < 7; ++g)
#pragma unroll
        for (int i = 0; i < AT; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) la[g][i][h] = fetch_a(g, i, h);
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(7 * AT * 2) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" : : : "memory");
    for (int s = 0; s < stages; ++s) {
        const int u = s & 1;
        const int sn = min(s + 1, stages - 1);
        read_b(u, 0, 0);
        static_for<8>([&](auto jc) {
            constexpr int j = jc;
            const int g = 8 * s + j;
            static_for<NT>([&](auto itc) {
                constexpr int it = itc;
                static_assert(NT == 2 * AT && 2 * XR == 4 * NT, "one load of A and, in half of the steps, one of B per block");
                la[(j + 7) & 7][it / 2][it % 2] = fetch_a(g + 7, it / 2, it % 2);
                if constexpr (j < 4) fetch_b(sn, u ^ 1, 4 * j + it);
                if constexpr (it + 1 < NT)
                    read_b(u, it + 1, j);
                else if constexpr (j + 1 < 8)
                    read_b(u, 0, j + 1);
                __builtin_amdgcn_sched_barrier(0);
                static_for<AT>([&](auto ic) {
                    constexpr int i = ic;
                    mfma_fixed<kSmall + i * NT + it>(__builtin_bit_cast(half8_t, la[j & 7][i][1]), b[it & 1][0]);
                });
                static_for<AT>([&](auto ic) {
                    constexpr int i = ic;
                    mfma_fixed<i * NT + it>(__builtin_bit_cast(half8_t, la[j & 7][i][0]), b[it & 1][0]);
                });
                static_for<AT>([&](auto ic) {
                    constexpr int i = ic;
                    mfma_fixed<kSmall + i * NT + it>(__builtin_bit_cast(half8_t, la[j & 7][i][0]), b[it & 1][1]);
                });
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        // the next stage's loads to LDS, the last of them ahead of the loads of A of four steps, have landed; this one has been read
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(4 * AT * 2) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" : : : "memory");
    }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");   // what the last stage fetched for none after it
}

// Workgroup: 4 wavefronts, tile 256 rows x 128 columns, each wavefront 64 x 128 on fixed accumulators.  One wavefront per
// SIMD, which its 24 matrix instructions per step of 16 inputs keep busy while the loads of the next are on their way:
// 4096 x 4096 times 416 columns 44 to 46 us, of them 37 in the loop (matrix pipes busy 77 % of the time, at 1.75 GHz) and 5
// to write four shares of K; the three products one after the other, with every operand fetched for each, took 51.
__global__ __launch_bounds__(256, 1) void lora_split_gemm_kernel(SplitGemmArgs a)
{
    constexpr int AT = kSplitAT;
    extern __shared__ __attribute__((aligned(16))) char lds_c[];   // two stage buffers of hi and lo
    const int tid = threadIdx.x, lane = tid & (kWave - 1), li = lane & 31, lb = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    // the column tiles of a row tile on one die (index mod 8), whose L2 then reads the rows, most of what there is to read, once
    const int gx = (int)gridDim.x, tiles_t = gx / a.tiles_o;
    const int w = gx % kDies == 0 ? ((int)blockIdx.x % kDies) * (gx / kDies) + (int)blockIdx.x / kDies : (int)blockIdx.x;
    const int ob = w / tiles_t * 256, o0 = ob + wave * 64;
    const int t0 = w % tiles_t * 128;
    const int k0 = blockIdx.y * a.ks;
    const int klen = max(0, min(a.ks, a.K - k0));

    acc_reserve<2 * AT>();
    static_for<2 * 16 * AT * NT>([&](auto r) { acc_write<r>(0.0f); });
    const uint32_t K = (uint32_t)a.K;
    // descriptors of this tile's rows alone, so that the offsets stay in 32 bits whatever the matrices hold
    const uint32_t bytes_a = (uint32_t)min(8, ((a.rows + 31) / 32 - ob / 32)) * (K / 16) * 1024u;
    const uint32_t bytes_b = (uint32_t)min(128, a.cols - t0) * K * 2u;
    const size_t at_a = (size_t)ob * K, at_b = (size_t)t0 * K;
    SplitOperands op;
    op.a[0] = make_rsrc(a.Ah + at_a, bytes_a);
    op.a[1] = make_rsrc(a.Al + at_a, bytes_a);
    op.b[0] = make_rsrc(a.Bh + at_b, bytes_b);
    op.b[1] = make_rsrc(a.Bl + at_b, bytes_b);
    op.av = tl_piece((uint32_t)(wave * 64 + li), (uint32_t)k0 / 8 + lb, K);
    op.a_tile = (K / 16) * 1024u;
    op.a_step = 1024u;
    // a load instruction moves four columns: lane -> (column, slot of 16 bytes), source piece = slot ^ column
    const uint32_t bc = (uint32_t)(4 * wave + (lane >> 4));
    op.bv = (bc * K + (uint32_t)k0) * 2u + (((uint32_t)(lane & 15) ^ bc) << 4);
    op.b_pass = 32u * K;
    op.b_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds_c + (uint32_t)wave * 1024u;
    split_phase(op, klen, lds_c, li, lb);
    acc_settle();
    const float sc = 1.0f / ((a.max_bits ? split_scale(*a.max_bits) : 1.0f) * kBlockSplit);
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
                const float v = acc_read<16 * (i * NT + it) + e>() + acc_read<16 * (kSmall + i * NT + it) + e>() * (1.0f / kLowSplit);
                if (o < a.rows)        // (written through: 27 MB left in the L2s to the end of the kernel cost 2 us)
                    __hip_atomic_store(&out[(size_t)o * a.cols + t], v * sc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            });
        });
    });
}

// sum_z P[z][i], rounded once
__device__ __forceinline__ float4_t sum_shares(const float4_t *__restrict__ P, int splits, size_t count4, size_t i)
{
    const float4_t p = P[i];
    double s[4] = {p[0], p[1], p[2], p[3]};
    for (int z = 1; z < splits; ++z) {
        const float4_t q = P[(size_t)z * count4 + i];
#pragma unroll
        for (int e = 0; e < 4; ++e) s[e] += (double)q[e];
    }
    return float4_t{(float)s[0], (float)s[1], (float)s[2], (float)s[3]};
}

// Y[i] = sum_z P[z][i]
__global__ __launch_bounds__(256) void lora_split_reduce_kernel(const float4_t *__restrict__ P, int splits, size_t count4, float4_t *__restrict__ Y)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < count4; i += (size_t)gridDim.x * blockDim.x) {
        Y[i] = sum_shares(P, splits, count4, i);
    }
}

// The same, a workgroup per 16 rows of cols4 float4s; row_factor (or null): of each row; colmax (or null): the
// bits of the columns' largest magnitudes, in kColSlots rows of
// 4 cols4 words (zero before), a workgroup's in row blockIdx mod kColSlots.  In one row the adds to a word were 256 in
// turn, and 22 of 28 us (4096 x 416); now 8.
__global__ __launch_bounds__(512) void lora_split_reduce_max_kernel(const float4_t *__restrict__ P, const float *__restrict__ row_factor, int splits, int rows, int cols4,
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
            const float4_t s = sum_shares(P, splits, count4, i) * (row_factor ? row_factor[r] : 1.0f);
            Y[i] = s;
#pragma unroll
            for (int e = 0; e < 4; ++e) mx[e] = fmaxf(mx[e], fabsf(s[e]));
        }
    if (!colmax) return;
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

int launch_lora_split(const float *S, int n, int k, const unsigned *max_bits, const unsigned *channel_max, half_t *Sh, half_t *Sl, half_t *Th, half_t *Tl,
                      float *channel_factor, hipStream_t st)
{
    hipLaunchKernelGGL(lora_split_kernel, dim3((unsigned)(k / 64), (unsigned)((n + 63) / 64)), dim3(256), 0, st, S, n, k, max_bits,
                       channel_max, Sh, Sl, Th, Tl, channel_factor);
    return hip_status(hipGetLastError());
}

// Y [rows][cols] = A B^T (A scaled by split_scale(*max_bits), or with max_bits null a row by the reciprocal of its row_factor; B by kBlockSplit; cols <= 1024).
// P: split_gemm_splits() x rows x cols floats.
// colmax (or null): kColSlots rows of zeros, which become bits of the columns' largest magnitudes (cols <= 1024).
int launch_lora_split_gemm(const half_t *Ah, const half_t *Al, const unsigned *max_bits, const float *row_factor, const half_t *Bh, const half_t *Bl, int rows,
                           int cols, int K, float *P, float *Y, unsigned *colmax, hipStream_t st)
{
    SplitGemmArgs a{Ah, Al, Bh, Bl, max_bits, nullptr, rows, cols, K, 0, (rows + 255) / 256};
    const int splits = split_gemm_splits(rows, cols, K);
    a.P = splits > 1 || colmax || row_factor ? P : Y;
    a.ks = ((K + 127) / 128 + splits - 1) / splits * 128;
    const size_t lds = (size_t)4 * kSplitStage;
    hipLaunchKernelGGL(lora_split_gemm_kernel, dim3((unsigned)(a.tiles_o * ((cols + 127) / 128)), (unsigned)splits), dim3(256), lds, st, a);
    if (colmax || row_factor) {
        hipLaunchKernelGGL(lora_split_reduce_max_kernel, dim3((unsigned)((rows + 15) / 16)), dim3(512), 0, st, reinterpret_cast<const float4_t *>(P),
                           row_factor, splits, rows, cols / 4, reinterpret_cast<float4_t *>(Y), colmax);
    } else if (splits > 1) {
        const size_t count4 = (size_t)rows * cols / 4;          // cols is a multiple of 32
        const unsigned grid = (unsigned)((count4 + 255) / 256 < 2048 ? (count4 + 255) / 256 : 2048);
        hipLaunchKernelGGL(lora_split_reduce_kernel, dim3(grid), dim3(256), 0, st, reinterpret_cast<const float4_t *>(P), splits, count4,
                           reinterpret_cast<float4_t *>(Y));
    }
    return hip_status(hipGetLastError());
}

}  // namespace slim
