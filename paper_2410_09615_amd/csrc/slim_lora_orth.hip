// out = orth(in) for a block in [rows][l] of fp32 columns, l <= 1024: Cholesky QR, the orthonormalisation of the
// subspace iteration in slim_lora.hip.
//
//   G = in^T in = Lc Lc^T,  out = in Lc^-T     (columns in order: in = out Lc^T with a positive diagonal)
//
// The call is a chain (products, 64-column steps of the factorisation, products), so what bounds it is the
// number of launches (4 us each) and the latency of the 64 x 64 diagonal blocks, not arithmetic:
//   lora_gram_kernel    lower tiles of G, the rows divided among the workgroups, partial tiles to memory;
//   lora_chol_kernel    the factorisation, a workgroup per tile, which hand finished tiles to one another through
//                       memory; one of them factors and inverts the diagonal tiles, in blocks of 16 that live in the
//                       registers of a wavefront;
//   lora_apply_kernel   a workgroup carries 16 rows of `in` through all block columns, which stay in LDS:
//                       out_J = (in_J - sum_{K<J} out_K L_JK^T) X_JJ^T, one launch for the whole block.
// 4096 x 416: 3 launches (gram 22 us, factorisation 94, apply 25) where a factorisation with one launch per 64 columns took
// 148 us and seven launches of 4 us where the block is only scaled, and with separate panel, trailing and column products
// and a 64-step one-workgroup diagonal 700.
//
// A pivot below 1e-9 of the largest diagonal entry of G marks a column that lies in the span of the ones before it
// (or a padding column of zeros): it gets pivot 1 and no column is subtracted for it, in the blocks that follow either,
// so the block carries what is left of it, a (numerically) zero column if `in` is of order one.  (What is left of such
// a column in G is rounding, 1e-7 of the largest entry: subtracted as a panel it takes the pivots of that size after it along.)  (Where 1e-9 of that entry is more than 1, the pivot is
// that: what is left stays within the range of the split into fp16 numbers.)
//
// Not every block of the subspace iteration need be orthonormal: columns scaled to magnitudes up to 1 span the same, and
// what the Gram matrix, the factorisation and the rounding of the products have to carry is the condition of the block, which
// grows by that of S per product.  So several products follow on one another; how many is decided where the pivots are known, in
// memory, and the kernels of a block that is only scaled return at once, but for the last (the host does not know).
// The rule (orth_run()): one product after the first block, then two while the pivots of a block span at most kSpread (a
// condition of 100), then twice as many as before, up to kMaxRun, while their span allows that many: rounding in the
// direction of the largest singular value grows by its ratio to the smallest with each product, and 2e-7 (of a column) times that
// ratio to the power of the run has to stay below 0.2, which is 1e3 for the span, the ratio's square, at four products and 30 at
// eight; beginning with four asks for 100.  A span above kSpread is followed by a quarter as many.
// That is so where the columns have separated.  Before, they hold a part of the direction of the largest by themselves, and what
// they lose beside it is not only in that direction: with four products in a row from the third on, L was up to 110 times further
// from the span of the exact iterate (one singular value 10 times the others, 6 rounds: 9e-4 of a column, where L in fp16 is
// rounded at 5e-4).  So four begin with the seventh product, and the last run has no more than four (orth_due()), after which
// L is as near as with two products at most in a row, up to a factor of 1.5 (tests/test_orth_rule.py).
// 16 rounds of a layer of 4096 x 4096 with 409 columns (singular values over a factor of 3): 11 blocks of 34 are orthonormalised,
// where every other one was 19 (127 us more for each than for one that is only scaled).
#include <utility>

#include "slim_internal.h"

namespace slim {

typedef float float16v_t __attribute__((ext_vector_type(16)));

constexpr int kOb = 64;                        // block of columns
constexpr int kTileFloats = kOb * kOb;
constexpr int kGramTiles = 640;                // partial tiles of G the workspace has room for
constexpr float kSpread = 1e4f;                // largest / smallest pivot up to which more than one product may follow
constexpr int kMaxRun = 8;                     // products between two blocks that are orthonormalised, at most
constexpr int kLastRun = 4;                    // before the last of them, at most
constexpr int kSeparated = 7;                  // products before more than two in a row
constexpr int kMaxBlocks = 1024 / kOb, kMaxTri = kMaxBlocks * (kMaxBlocks + 1) / 2;      // blocks of columns, tiles of a lower triangle

// Words of an orth() that its kernels and the next orth() read: the product after which the next block has to be
// orthonormalised, and how many it is away.
struct OrthWords {
    int due, run;
};
// A conditional orth(): `h` products with S or S^T after the first block; the block is only scaled where h < in->due.
// The words of the call before it are `in` (null: orthonormal whatever they say), its own are `out`; `last`: the products
// after which a call that is not conditional follows.
struct OrthStep {
    const OrthWords *in;
    OrthWords *out;
    int h, last;
    __device__ bool skip() const { return in && h < in->due; }
};

// Tiles of 64 x 64 are stored in the operand order of V_MFMA_F32_16X16X4_F32, four of its steps at a time: the
// element (n, k) at [n / 16][k / 16][(k % 16) / 4][n % 16][k % 4], so a wavefront's load of 16 rows x 16 columns
// is one contiguous KiB, and the same tile serves as the A operand (rows m) and the B operand (columns n).
__device__ __forceinline__ int op_at(int n, int k) { return ((n >> 4) * 4 + (k >> 4)) * 256 + ((k >> 2) & 3) * 64 + (n & 15) * 4 + (k & 3); }
// tile (i, j), j <= i, of a lower triangle
__device__ __host__ __forceinline__ int tri(int i, int j) { return i * (i + 1) / 2 + j; }

// c += A B^T over 16 columns: a, b the operands of the lane (row or column lane % 16, columns 4 (lane / 16) .. + 3)
__device__ __forceinline__ void mma16(float4_t a, float4_t b, float4_t &c)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], c, 0, 0, 0);
}

// Partial tile of G = Y^T Y: tile t = tri(i, j) over the rows z * zrows .. ; wavefront w takes a quarter of them.  Two
// rows of Y are the operands of V_MFMA_F32_32X32X2_F32 as they lie in memory: no LDS on the way.
__global__ __launch_bounds__(256) void lora_gram_kernel(const float *__restrict__ Y, int rows, int l, int zrows, int tiles,
                                                        float *__restrict__ P, OrthStep step)
{
    if (step.skip()) return;
    __shared__ __attribute__((aligned(16))) float red[kTileFloats];
    const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int i = 0;
    while (tri(i + 1, 0) <= (int)blockIdx.x) ++i;
    const int j = (int)blockIdx.x - tri(i, 0);
    const int per = zrows / 4;                  // even
    const int k0 = (int)blockIdx.y * zrows + wave * per;
    const int cnt = max(0, min(per, rows - k0));
    // (a base of its own keeps the offsets in 32 bits for any number of rows; reads past the range are zeros)
    const rsrc_t rs = make_rsrc(Y + (size_t)min(k0, rows) * l, (uint32_t)cnt * (uint32_t)l * 4u);
    uint32_t ca[2], cb[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int na = kOb * i + 32 * b + r, nb = kOb * j + 32 * b + r;
        ca[b] = na < l ? (uint32_t)(h * l + na) * 4u : 0xFFFFFF00u;
        cb[b] = nb < l ? (uint32_t)(h * l + nb) * 4u : 0xFFFFFF00u;
    }
    float16v_t acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.f;
    auto ld = [&](uint32_t c, uint32_t row) {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, c < 0xFFFFFF00u ? (int)(c + row * (uint32_t)l * 4u) : (int)c, 0, 0));
    };
    constexpr int U = 8;                        // pairs of rows per trip, the next trip's loads in flight
    float av[U][2], bv[U][2];
    auto load = [&](int k) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                av[u][b] = ld(ca[b], (uint32_t)(k + 2 * u));
                bv[u][b] = ld(cb[b], (uint32_t)(k + 2 * u));
            }
    };
    load(0);
    for (int k = 0; k < cnt; k += 2 * U) {
        float ac[U][2], bc[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                ac[u][b] = av[u][b];
                bc[u][b] = bv[u][b];
            }
        load(k + 2 * U);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(ac[u][a], bc[u][b], acc[a][b], 0, 0, 0);
    }
    // register 4 q + e of a block: row 8 q + 4 h + e, column r
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            float *p = red + op_at(32 * a + 8 * q + 4 * h + e, 32 * b + r);
                            *p = w == 0 ? acc[a][b][4 * q + e] : *p + acc[a][b][4 * q + e];
                        }
        }
        __syncthreads();
    }
    float4_t *const out = reinterpret_cast<float4_t *>(P + ((size_t)blockIdx.y * tiles + blockIdx.x) * kTileFloats);
#pragma unroll
    for (int q = 0; q < 4; ++q) out[threadIdx.x + 256 * q] = reinterpret_cast<const float4_t *>(red)[threadIdx.x + 256 * q];
}

template <int N>
__device__ __forceinline__ float row_lane(float v)       // lane N of the sixteen, to all of them
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + N, 0xF, 0xF, true));
}
template <int... Is, class F>
__device__ __forceinline__ void for_each_impl(std::integer_sequence<int, Is...>, F &&f)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void for_each(F &&f)
{
    for_each_impl(std::make_integer_sequence<int, N>{}, f);
}

// The value that lane i % 16 of the G-th sixteen lanes holds, to lane i of all four.
template <int G>
__device__ __forceinline__ float from_group(float v)
{
    const unsigned b = __builtin_bit_cast(unsigned, v);
    const auto p = __builtin_amdgcn_permlane16_swap(b, b, false, false);        // groups 0, 0, 2, 2 and 1, 1, 3, 3
    const unsigned h = p[G & 1];
    const auto q = __builtin_amdgcn_permlane32_swap(h, h, false, false);
    return __builtin_bit_cast(float, (unsigned)q[G >> 1]);
}

// 16 x 16: lane i of group g (sixteen lanes) holds row i, columns 4 g .. 4 g + 3, of the symmetric block a = Lc Lc^T; on
// return those of Lc^-1.  The steps run on a = M diag(d) M^T, M with a unit diagonal, whose chain has a reciprocal and no square
// root, and the rows of M^-1 are scaled by 1 / sqrt(d) at the end.  Step c adds m_i = -a_ic / d_c times row c to the rows i
// below it: to the columns of a after c, to those of M^-1 before it, and column c becomes that of M^-1, so that one register
// holds a column of the one and then of the other.  Broadcasts are between lanes, without LDS or barriers.  (With a row
// of both in each of sixteen lanes the 64 x 64 block took 13 us instead of 9: twice the instructions per step.)
// pmax, pmin: the largest and the smallest pivot of this lane's rows so far, but for those of `dead`.  Returns whether this row's
// pivot is above the floor.
__device__ __forceinline__ bool factor16(float4_t &w, int i, int g, float floor_, float dead, float &pmax, float &pmin)
{
    float d_i = 1.0f;                            // this row's pivot
    for_each<16>([&](auto cc) {
        constexpr int c = cc;
        const float col = from_group<c / 4>(w[c % 4]);
        const float d = row_lane<c>(col);
        d_i = i == c ? d : d_i;
        float q = __builtin_amdgcn_rcpf(d);
        q = q * (2.0f - d * q);                  // to rounding
        const float m = d > floor_ && i > c ? -col * q : 0.f;    // (d below: a column in the span of the ones before it: nothing to subtract)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float s = __builtin_fmaf(row_lane<c>(w[e]), m, w[e]);
            w[e] = e == c % 4 && g == c / 4 ? (i == c ? 1.0f : m) : s;
        }
    });
    const bool alive = d_i > floor_;
    pmax = alive ? fmaxf(pmax, d_i) : pmax;
    pmin = alive ? fminf(pmin, d_i) : pmin;
    const float p = alive ? d_i : dead;
    float q = __builtin_amdgcn_rsqf(p);
    q = q * (1.5f - 0.5f * p * q * q);           // 1 / sqrt(d) to rounding
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] *= q;
    return alive;
}

// How many products may follow before the next block that is orthonormalised, after the one `h` products into the iteration that
// took `done` of them (0, or a power of two up to kMaxRun) to pivots from pmin to pmax.
__host__ __device__ int orth_run(int done, int h, float pmax, float pmin)
{
    if (!(pmax <= kSpread * pmin)) return done >= 4 ? done / 4 : 1;
    if (done < 2) return done + 1;
    if (h < kSeparated) return 2;
    const float spread = pmax / pmin;
    int run = 2 * done < kMaxRun ? 2 * done : kMaxRun;
    if (run == 8 && !(spread <= 30.0f)) run = 4;
    if (run == 4 && !(spread <= (done == 2 ? 100.0f : 1e3f))) run = 2;
    return run;
}
// The product after which the next block is orthonormalised, where `run` may follow the one after h of them: the last run begins at
// last - kLastRun or later.
__host__ __device__ int orth_due(int h, int run, int last)
{
    const int end = h + run < last ? h + run : last;
    return h < last - kLastRun && end > last - kLastRun ? last - kLastRun : end;
}

// What the workgroups of a factorisation hand to one another: a tile of the factor (at tri(I, J)), a diagonal tile and the
// one to its left before the last column is subtracted, the inverse of a diagonal tile.  A word each, in a line of its own,
// holds the number of the orth() whose tile it is (kHandFailed: that of one whose wait ran out).
enum { kHandL = 0, kHandT = kMaxTri, kHandA = kHandT + kMaxBlocks, kHandD = kHandA + kMaxBlocks, kHandFailed = kHandD + kMaxBlocks, kHandWords };
constexpr int kHandStride = 16;
constexpr int kHandPolls = 1 << 24;            // half a microsecond or more each; a wait is over after some tens of them, or when other
                                               // work on the chip has let the rest of the launch start

// Everything the workgroup has stored -> visible to who sees the word.
__device__ __forceinline__ void hand_over(unsigned *hand, int what, unsigned seq)
{
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    __syncthreads();
    if (threadIdx.x == 192) {                    // (not of the wavefront that factors)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __hip_atomic_store(hand + what * kHandStride, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}
// One lane waits; false: the word has not come.
__device__ __forceinline__ bool hand_taken(unsigned *hand, int what, unsigned seq, int limit)
{
    for (int polls = 0; __hip_atomic_load(hand + what * kHandStride, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != seq; ++polls) {
        if (polls >= limit) return false;
        __builtin_amdgcn_s_sleep(1);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return true;
}

// G = Lc Lc^T in one launch.  What it waits for is the chain of diagonal tiles, so workgroup 0 factors and inverts all of
// them, one after the other (D[J] whole, Dp[J] with the rows of pivots below the floor as zeros), and nothing on that chain
// goes through memory but what the others have ready: the tiles (J, J) and (J, J - 1) with the columns before J - 1
// subtracted.  The panel between those and the column J - 1 it makes itself, from the inverse it has in LDS.  Every other
// workgroup has a tile (I, J), I >= J, column after column: it adds up the tile's partial tiles, subtracts L_IK L_JK^T for the
// columns before its own as they come, and hands the tile to workgroup 0 or waits for D[J] and hands on L_IJ = A_IJ Dp_J^T.
// A workgroup waits for workgroup 0 and for tiles of columns before its own, of a lower index, and workgroup 0 for tiles whose
// workgroups wait for it in no more than it has handed on: with workgroups started in the order of their index there is always
// one that runs.  A wait is bounded all the same; should a tile not come, lora_apply_kernel makes the block NaN.
// 4096 x 416: 94 us, 4.5 where the block is only scaled; one launch per 64 columns took 148 and 30.  (With a diagonal tile's
// inverse handed through memory to the workgroup of the next one: 4 us more.)
__global__ __launch_bounds__(256) void lora_chol_kernel(int nb, int l, const float *__restrict__ P, int splits, int tiles, float *G,
                                                        float *Lf, float *D, float *Dp, unsigned *hand, unsigned seq, int polls, OrthStep step)
{
    if (step.skip()) return;
    __shared__ __attribute__((aligned(16))) float T[kTileFloats], LI[kTileFloats], LJ[kTileFloats];
    __shared__ float mx_s[4];
    __shared__ int missing;
    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 15, mq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int j = 0, left = (int)blockIdx.x;           // the tile's column
    while (left >= nb - j) left -= nb - j++;
    const int I = j + left;
    if (tid == 0) missing = 0;
    // (words in turn: wavefront w waits for the w-th; the barrier makes it the workgroup's)
    auto wait_for = [&](int first, int second) {
        if (lane == 0 && wave < 2 && !missing && !hand_taken(hand, wave == 0 ? first : second, seq, polls)) {
            missing = 1;                         // (and the waits after this one are none)
            __hip_atomic_store(hand + kHandFailed * kHandStride, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
    };
    float4_t *const T4 = reinterpret_cast<float4_t *>(T);
    {
        const float4_t *p = reinterpret_cast<const float4_t *>(P + (size_t)tri(I, j) * kTileFloats);
        float4_t s[4] = {};
#pragma unroll 4
        for (int z = 0; z < splits; ++z)
#pragma unroll
            for (int q = 0; q < 4; ++q) s[q] += p[(size_t)z * tiles * (kTileFloats / 4) + tid + 256 * q];
#pragma unroll
        for (int q = 0; q < 4; ++q) T4[tid + 256 * q] = s[q];
    }
    __syncthreads();
    // 16 rows of the tile per wavefront
    auto subtract = [&](const float4_t (&a)[4], const float4_t *b) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            float4_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 4; ++t) mma16(a[t], b[(cb * 4 + t) * 64 + lane], c);
#pragma unroll
            for (int e = 0; e < 4; ++e) T[op_at(16 * wave + 4 * mq + e, 16 * cb + ln)] -= c[e];
        }
    };
    // to = a d^T
    auto panel = [&](const float4_t (&a)[4], const float4_t *d, float *to) {
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
            float4_t c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 4; ++t) mma16(a[t], d[(cb * 4 + t) * 64 + lane], c);
#pragma unroll
            for (int e = 0; e < 4; ++e) to[op_at(16 * wave + 4 * mq + e, 16 * cb + ln)] = c[e];
        }
    };
    auto rows_of = [&](const float *tile, float4_t (&a)[4]) {
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t] = reinterpret_cast<const float4_t *>(tile)[(wave * 4 + t) * 64 + lane];
    };
    auto store_tile = [&](float *to, const float *tile) {
#pragma unroll
        for (int q = 0; q < 4; ++q) reinterpret_cast<float4_t *>(to)[tid + 256 * q] = reinterpret_cast<const float4_t *>(tile)[tid + 256 * q];
    };
    float4_t a[4];
    if (blockIdx.x > 0) {
        for (int K = 0; K < (I == j ? j - 1 : j); ++K) {
            wait_for(kHandL + tri(I, K), kHandL + tri(j, K));
            rows_of(Lf + (size_t)tri(I, K) * kTileFloats, a);
            subtract(a, reinterpret_cast<const float4_t *>(Lf + (size_t)tri(j, K) * kTileFloats));
        }
        __syncthreads();
        if (I <= j + 1) {
            store_tile(G + (size_t)tri(I, j) * kTileFloats, T);
            hand_over(hand, (I == j ? kHandT : kHandA) + I, seq);
            if (I == j) return;
        }
        wait_for(kHandD + j, kHandD + j);
        rows_of(T, a);
        panel(a, reinterpret_cast<const float4_t *>(Dp + (size_t)j * kTileFloats), LI);
        __syncthreads();
        store_tile(Lf + (size_t)tri(I, j) * kTileFloats, LI);
        hand_over(hand, kHandL + tri(I, j), seq);
        return;
    }

    // ---- the diagonal tiles ----
    float mx = 0.f;                              // the largest diagonal entry of G
    for (int c = tid; c < l; c += 256) {
        float s = 0.f;
#pragma unroll 8
        for (int z = 0; z < splits; ++z) s += P[((size_t)z * tiles + tri(c / kOb, c / kOb)) * kTileFloats + op_at(c % kOb, c % kOb)];
        mx = fmaxf(mx, s);
    }
    mx = wave_max(mx);
    if (lane == 0) mx_s[wave] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(mx_s[0], mx_s[1]), fmaxf(mx_s[2], mx_s[3]));
    // Far from 1 the block is factored as 4^h G (exact): the reciprocals of factor16() know no subnormal numbers
    int h = 0;
    if (mx > 0.f && !(mx > 0x1p-60f && mx < 0x1p60f)) h = min(max(-(__builtin_amdgcn_frexp_expf(mx) / 2), -63), 63);
    const float dead = ldexpf(fmaxf(1.0f, mx * 1e-9f), 2 * h), floor_ = ldexpf(mx, 2 * h) * 1e-9f;
    float pmax = 0.f, pmin = __builtin_inff();   // (of the rows of a lane of wavefront 0)
    float *const X = LI;                         // the inverse, and
    float *const XT = LJ;                        // the inverse transposed: block (c, r) holds block (r, c) of X
    auto block = [](float *base, int bi, int bj) { return base + (bi * 4 + bj) * 256; };
    auto operand = [&](const float *blk) { return reinterpret_cast<const float4_t *>(blk)[lane]; };
    __shared__ __attribute__((aligned(16))) float M[3][256];
    __shared__ int alive[kOb];                   // pivot above the floor
    for (j = 0; j < nb; ++j) {
        if (j > 0) {
            wait_for(kHandT + j, kHandA + j);
            rows_of(G + (size_t)tri(j, j - 1) * kTileFloats, a);
            store_tile(T, G + (size_t)tri(j, j) * kTileFloats);
            panel(a, reinterpret_cast<const float4_t *>(X), XT);
            __syncthreads();
            rows_of(XT, a);
            subtract(a, reinterpret_cast<const float4_t *>(XT));
            __syncthreads();
        }
        if (h != 0)                                  // (a thread's own pieces)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) T[4 * (tid + 256 * q) + e] = ldexpf(T[4 * (tid + 256 * q) + e], 2 * h);
        for (int idx = tid; idx < kTileFloats; idx += 256) X[idx] = 0.f;
        __syncthreads();
        for (int b = 0; b < 4; ++b) {
            if (wave == 0) {
                float4_t w = operand(block(T, b, b));
                const bool ok = factor16(w, ln, mq, floor_, dead, pmax, pmin);
                if (lane < 16) alive[16 * b + ln] = ok;
                reinterpret_cast<float4_t *>(block(X, b, b))[lane] = w;
#pragma unroll
                for (int e = 0; e < 4; ++e) block(XT, b, b)[(ln >> 2) * 64 + (4 * mq + e) * 4 + (ln & 3)] = w[e];
            }
            __syncthreads();
            // panel: block rows b + 1 .. 3, one per wavefront
            if (wave > b) {
                float4_t c = {0.f, 0.f, 0.f, 0.f};
                mma16(operand(block(T, wave, b)), operand(block(X, b, b)), c);
#pragma unroll
                for (int e = 0; e < 4; ++e) block(T, wave, b)[(ln >> 2) * 64 + (4 * mq + e) * 4 + (ln & 3)] = alive[16 * b + ln] ? c[e] : 0.f;
            }
            __syncthreads();
            if (wave > b) {
                const float4_t a = operand(block(T, wave, b));
                for (int k = b + 1; k <= wave; ++k) {
                    float4_t c = {0.f, 0.f, 0.f, 0.f};
                    mma16(a, operand(block(T, k, b)), c);
#pragma unroll
                    for (int e = 0; e < 4; ++e) block(T, wave, k)[(ln >> 2) * 64 + (4 * mq + e) * 4 + (ln & 3)] -= c[e];
                }
            }
            __syncthreads();
        }
        // the inverse below its diagonal blocks: X_ij = -X_ii sum_{j <= k < i} L_ik X_kj, block row after block row
        for (int i = 1; i < 4; ++i) {
            if (wave < i) {
                float4_t c = {0.f, 0.f, 0.f, 0.f};
                for (int k = wave; k < i; ++k) mma16(operand(block(T, i, k)), operand(block(XT, wave, k)), c);
                reinterpret_cast<float4_t *>(M[wave])[mq * 16 + ln] = c;          // transposed: operand order of its columns
                asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
                float4_t y = {0.f, 0.f, 0.f, 0.f};
                mma16(operand(block(X, i, i)), operand(M[wave]), y);
                reinterpret_cast<float4_t *>(block(XT, wave, i))[mq * 16 + ln] = -y;
#pragma unroll
                for (int e = 0; e < 4; ++e) block(X, i, wave)[(ln >> 2) * 64 + (4 * mq + e) * 4 + (ln & 3)] = -y[e];
            }
            __syncthreads();
        }
        // both forms to memory; the second stays in X
        float4_t *const out = reinterpret_cast<float4_t *>(D + (size_t)j * kTileFloats);
        float4_t *const outp = reinterpret_cast<float4_t *>(Dp + (size_t)j * kTileFloats);
#pragma unroll
        for (int q = 0; q < 4; ++q) {            // (piece tid + 256 q is of row 16 q + tid % 16)
            float4_t v = reinterpret_cast<const float4_t *>(X)[tid + 256 * q];
            if (h != 0)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = ldexpf(v[e], h);
            out[tid + 256 * q] = v;
            if (!alive[16 * q + (tid & 15)]) v = float4_t{0.f, 0.f, 0.f, 0.f};
            outp[tid + 256 * q] = v;
            reinterpret_cast<float4_t *>(X)[tid + 256 * q] = v;
        }
        if (j + 1 < nb) hand_over(hand, kHandD + j, seq);
    }
    if (wave != 0) return;
    pmax = wave_max(pmax);
    pmin = -wave_max(-pmin);
    if (tid == 0) {
        const int run = orth_run(step.in ? step.in->run : 0, step.h, pmax, pmin);
        step.out->run = run;
        step.out->due = orth_due(step.h, run, step.last);
    }
}

// The power of two that brings a column whose largest magnitude has the bits `max_bits` below 1.
__device__ __forceinline__ float column_scale(unsigned max_bits)
{
    const int e = (int)(max_bits >> 23);         // |v| < 2^(e - 126)
    return max_bits == 0u ? 1.0f : __uint_as_float((unsigned)max(253 - e, 1) << 23);
}

// Where the step skips the orthonormalisation: 16 rows of out = `in` with scaled columns (colmax: kColSlots rows of bits of their
// largest magnitudes).  clear: those of the next block, set to zero.
// 16 rows of out = in Lc^-T, block column after block column; wavefront w computes the columns 16 w .. 16 w + 15 of each.
__global__ __launch_bounds__(256) void lora_apply_kernel(const float *__restrict__ in, float *__restrict__ out, int rows, int l, int nb,
                                                         const float *__restrict__ Lf, const float *__restrict__ D, half_t *__restrict__ hi,
                                                         half_t *__restrict__ lo, int ldk, OrthStep step,
                                                         const unsigned *colmax, unsigned *clear, const unsigned *hand, unsigned seq)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int ldo = nb * kOb + 4;
    float *const O = lds;                        // [16][ldo]: the rows of out so far
    float *const V = lds + 16 * ldo;             // [16][68]
    const int lane = threadIdx.x & 63, ln = lane & 15, mq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // neighbouring rows on one die (index mod 8): the lines of hi and lo, 64 rows each, leave its L2 whole (a block that is
    // only scaled, 4096 x 416: 14 -> 7 us with this and without the way through LDS)
    const int gx = (int)gridDim.x, bx = (int)blockIdx.x;
    const int r0 = (gx % 8 == 0 ? bx % 8 * (gx / 8) + bx / 8 : bx) * 16;
    // the sixteen rows of column c as two fp16 numbers, columns as rows
    auto emit = [&](int c, const float (&v16)[16]) {
        half8_t h[2], g[2];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float s = v16[r] * kBlockSplit, v = fabsf(s) > 65000.0f ? copysignf(65000.0f, s) : s;
            const half_t x = (half_t)v;
            h[r / 8][r % 8] = x;
            g[r / 8][r % 8] = (half_t)(v - (float)x);
        }
        const size_t at = (size_t)c * ldk + r0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            *reinterpret_cast<half8_t *>(hi + at + 8 * q) = h[q];
            *reinterpret_cast<half8_t *>(lo + at + 8 * q) = g[q];
        }
    };
    if (clear)
        for (int q = blockIdx.x; q < kColSlots; q += gridDim.x)
            for (int c = threadIdx.x; c < l; c += 256) clear[q * l + c] = 0u;
    if (step.skip()) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            step.out->due = step.in->due;
            step.out->run = step.in->run;
        }
        for (int c = threadIdx.x; c < l; c += 256) {
            float v16[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) v16[r] = r0 + r < rows ? in[(size_t)(r0 + r) * l + c] : 0.f;
            unsigned mx = 0u;
#pragma unroll
            for (int q = 0; q < kColSlots; ++q) mx = max(mx, colmax[q * l + c]);
            const float sc = column_scale(mx);
#pragma unroll
            for (int r = 0; r < 16; ++r) v16[r] *= sc;
            emit(c, v16);
        }
        return;
    }
    const float poison = hand[kHandFailed * kHandStride] == seq ? __builtin_nanf("") : 0.f;      // the factor is not whole: must not pass for one
    // block column J: its part of `in`, the inverse of its diagonal block, the first tile of the factor (the loads of
    // the next column go out before this one's last products)
    float v[4];
    float4_t d[4], b[4];
    auto load_column = [&](int J) {
        const int col = kOb * J + 16 * wave + ln;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = r0 + 4 * mq + e;
            v[e] = row < rows && col < l ? in[(size_t)row * l + col] + poison : 0.f;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            d[t] = reinterpret_cast<const float4_t *>(D + (size_t)J * kTileFloats)[(wave * 4 + t) * 64 + lane];
            b[t] = reinterpret_cast<const float4_t *>(Lf + (size_t)tri(J, 0) * kTileFloats)[(wave * 4 + t) * 64 + lane];
        }
    };
    load_column(0);
    for (int J = 0; J < nb; ++J) {
        const int col = kOb * J + 16 * wave + ln;
        float4_t c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0;
        const float4_t *const Lj = reinterpret_cast<const float4_t *>(Lf + (size_t)tri(J, 0) * kTileFloats);
        for (int K = 0; K < J; ++K) {
            float4_t bc[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) bc[t] = b[t];
            const int Kn = K + 1 < J ? K + 1 : K;
#pragma unroll
            for (int t = 0; t < 4; ++t) b[t] = Lj[(size_t)Kn * (kTileFloats / 4) + (wave * 4 + t) * 64 + lane];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const float4_t a = *reinterpret_cast<const float4_t *>(O + ln * ldo + kOb * K + 16 * t + 4 * mq);
                mma16(a, bc[t], t & 1 ? c1 : c0);
            }
        }
        float4_t dc[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) dc[t] = d[t];
#pragma unroll
        for (int e = 0; e < 4; ++e) V[(4 * mq + e) * 68 + 16 * wave + ln] = v[e] - (c0[e] + c1[e]);
        load_column(J + 1 < nb ? J + 1 : J);
        __syncthreads();
        float4_t y0 = {0.f, 0.f, 0.f, 0.f}, y1 = y0;
#pragma unroll
        for (int t = 0; t < 4; ++t) mma16(*reinterpret_cast<const float4_t *>(V + ln * 68 + 16 * t + 4 * mq), dc[t], t & 1 ? y1 : y0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = r0 + 4 * mq + e;
            const float y = y0[e] + y1[e];
            O[(4 * mq + e) * ldo + kOb * J + 16 * wave + ln] = y;
            if (out && row < rows && col < l) out[(size_t)row * l + col] = y;
        }
        __syncthreads();
    }
    if (hi)
        for (int c = threadIdx.x; c < l; c += 256) {         // (rows past the last are zeros)
            float v16[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) v16[r] = O[r * ldo + c];
            emit(c, v16);
        }
}

// Workspace of the orth()s of a call, in floats: partial tiles, tiles of G and of the factor, inverses of the diagonal
// blocks (twice), three sets of OrthWords, two times kColSlots rows of column maxima.
constexpr int kOrthWords = 64;
size_t orth_floats(int l)
{
    const size_t nb = (size_t)(l + kOb - 1) / kOb, t = nb * (nb + 1) / 2;
    return (kGramTiles + 2 * t + 2 * nb) * kTileFloats + kOrthWords + 2 * (size_t)kColSlots * l;
}
unsigned *orth_column_max(float *ws, int l, int which)
{
    return reinterpret_cast<unsigned *>(ws + orth_floats(l) - (size_t)(2 - which) * kColSlots * l);
}

// out (or null): fp32 [rows][l]; hi, lo (or null): the block for lora_split_gemm_kernel, [l][rows rounded up to 32].
// h < 0: always orthonormal.  Else the block after h products, of `last`, in a call's sequence of them (hi, lo only, out = null):
// orthonormal for h = 0, conditional from then on, where orth_column_max(h % 2) holds the column maxima of `in`; that of
// the next block is cleared.
// hand: orth_hand_words() words, zero at the start of a call's sequence, of which this is number seq (from 1).
size_t orth_hand_words() { return (size_t)kHandWords * kHandStride; }
int launch_orth(const float *in, float *out, half_t *hi, half_t *lo, int rows, int l, float *ws, unsigned *hand, unsigned seq, int h, int last,
                hipStream_t st)
{
    const int nb = (l + kOb - 1) / kOb, tiles = tri(nb, 0);
    float *const P = ws, *const G = P + (size_t)kGramTiles * kTileFloats, *const Lf = G + (size_t)tiles * kTileFloats;
    float *const D = Lf + (size_t)tiles * kTileFloats, *const Dp = D + (size_t)nb * kTileFloats;
    OrthWords *const words = reinterpret_cast<OrthWords *>(Dp + (size_t)nb * kTileFloats);
    static_assert(3 * sizeof(OrthWords) <= kOrthWords * sizeof(float), "words of the orth()s");
    const OrthStep step{h > 0 ? words + (h & 1) : nullptr, h < 0 ? words + 2 : words + ((h + 1) & 1), h, last};
    const unsigned *const colmax = h > 0 ? orth_column_max(ws, l, h & 1) : nullptr;
    unsigned *const clear = h >= 0 ? orth_column_max(ws, l, (h + 1) & 1) : nullptr;
    // about two workgroups per compute unit, at least 64 rows each
    int splits = kGramTiles / tiles;
    if (splits > (rows + 63) / 64) splits = (rows + 63) / 64;
    const int zrows = ((rows + splits - 1) / splits + 31) / 32 * 32;
    splits = (rows + zrows - 1) / zrows;
    hipLaunchKernelGGL(lora_gram_kernel, dim3((unsigned)tiles, (unsigned)splits), dim3(256), 0, st, in, rows, l, zrows, tiles, P, step);
    const bool wait_test = adapters_wait_test();     // (slim_decode_override: only the workgroup that waits for the others)
    hipLaunchKernelGGL(lora_chol_kernel, dim3((unsigned)(wait_test ? 1 : tiles)), dim3(256), 0, st, nb, l, (const float *)P, splits, tiles, G, Lf, D, Dp,
                       hand, seq, wait_test ? 256 : kHandPolls, step);
    const size_t lds = (size_t)(16 * (nb * kOb + 4) + 16 * 68) * sizeof(float);
    hipLaunchKernelGGL(lora_apply_kernel, dim3((unsigned)((rows + 31) / 32 * 2)), dim3(256), lds, st, in, out, rows, l, nb, (const float *)Lf,
                       (const float *)D, hi, lo, (rows + 31) / 32 * 32, step, colmax, clear, (const unsigned *)hand, seq);
    return hip_status(hipGetLastError());
}

}  // namespace slim
