// slim_linear_gemm on few tokens: Y = scale * (X Wc^T) + T L^T where the 512 x 128 tiles of
// slim_gemm_sparse.hip leave most of the chip idle.
//
// What bounds such a call is not a rate but launches (a dependent one costs 4 us) and the latency of
// a workgroup's chain of loads, on the few compute units that have a tile.  So the tiles are
// smaller, the inputs of a tile are divided among the eight wavefronts of its workgroup, X and the
// weights go from memory to LDS without registers, a round of stages at a time and several rounds
// ahead, and T = X R^T is made by other workgroups of the same launch meanwhile:
//
//   T role  (the first workgroups; they wait for nothing) tiles of 16 ranks x 16 or 32 tokens, the inputs divided
//           among the wavefronts and added up in LDS: no partial sums in memory.  T leaves as 16-byte
//           pieces that carry the number of the call (slim_decode.h), written through to memory.
//   Y role  a tile of 32 RT RG rows x 32 NT tokens.  Wavefront (rg, kw) of the RG x KW = 8 owns RT row
//           tiles and every KW-th stage of 128 inputs, then every KW-th unit of ranks, for which it
//           re-reads its pieces of T until they carry this call's number; the KW partial tiles meet in LDS.
//           Four more wavefronts (helpers) only bring X: loads return in order, so a wavefront that waited for its
//           X (from the L2) would wait for all weights (from memory) it has asked for before.
//
// The two roles share a launch only if all its workgroups are resident at once (one workgroup per
// compute unit); otherwise they are two launches.  That T is made does not depend on it: other work on the chip (calls
// on other streams, whose workgroups take whole compute units and wait likewise) can keep a T role from being dispatched
// while the Y role already waits, in a circle if there are three such calls.  So the wait is short, and a workgroup whose wait
// runs out makes T of its tokens itself and starts again: the same pieces, bit for bit, whoever stores them.
// Should a piece still be missing then (it cannot be), the outputs are NaN and the workspace's error word is set.
//
// X in LDS: a token's stage is one row without padding (the loads write LDS in lane order), so the
// pieces of 16 bytes of a row are stored permuted by the token number: the sixteen lanes that read
// together then hit all banks once.
#include "slim_decode.h"
#include "slim_mma.h"

namespace slim {

int gemm_t_splits(int32_t m, int32_t rank_pad, int32_t k);   // slim_api.hip

typedef int int4_t __attribute__((ext_vector_type(4)));
typedef int int8v_t __attribute__((ext_vector_type(8)));

struct MidArgs {
    const uint8_t *qvals;
    const uint8_t *meta;
    const float *scale;
    const half_t *X;      // [m][k] fp16, or (XF != 0) the same tensor as 8-bit codes
    const float *x_scale; // XF != 0: the tensor's scale (device memory)
    const half_t *R, *L;  // fp16 adapters in the adapter layout, or null with the 4-bit form:
    const uint8_t *Rq, *Lq;
    const half_t *Rs, *Ls;
    uint4_t *T;           // pieces of T (mid_t_piece()), or null with
    half_t *T_rows;       //   fp16 [m][rank_pad] (the T role alone)
    unsigned *err;        // set to 1 when a wait gave up
    CallEpoch epoch;
    half_t *Y;            // [m][n]
    int n, k, rank, rank_pad, m;
    int tiles_o;          // row tiles of the Y role
    int n_t;              // workgroups in the T role, the first of the grid (a multiple of 8)
    int t_tiles;          // tiles of T
    int spin_limit;       // polls after which a wait gives up
    int stages;           // stages of 128 inputs of the weight term (0: the adapter term alone)
    int accumulate;       // add to what Y holds
};

constexpr int kMidWaves = 8, kMidHelpers = 4, kMidThreads = (kMidWaves + kMidHelpers) * kWave;
constexpr uint32_t kPastEnd = 0xFFFFFFF0u;      // byte offset past the end of every buffer here

// Eight 8-bit codes (two dwords) -> eight fp16 values, exactly (E4M3: XF 1, E5M2: XF 2).
template <int XF>
__device__ __forceinline__ half8_t codes8_to_half8(uint32_t lo, uint32_t hi)
{
    typedef float f2_t __attribute__((ext_vector_type(2)));
    uint4_t out;
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        const int src = (int)(d ? hi : lo);
        const f2_t p0 = XF == 1 ? __builtin_amdgcn_cvt_pk_f32_fp8(src, false) : __builtin_amdgcn_cvt_pk_f32_bf8(src, false);
        const f2_t p1 = XF == 1 ? __builtin_amdgcn_cvt_pk_f32_fp8(src, true) : __builtin_amdgcn_cvt_pk_f32_bf8(src, true);
        out[2 * d] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(p0[0], p0[1]));
        out[2 * d + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(p1[0], p1[1]));
    }
    return __builtin_bit_cast(half8_t, out);
}

// The adapter term runs in units of 32 ranks, two steps of V_MFMA_F32_32X32X16_F16 each.  Step s of unit u
// multiplies on lane half h the ranks
//   fp16 L   32 u + 16 s + 8 h + [0, 8): a wavefront's load of L is one contiguous KiB per step
//   4-bit L  64 (u / 2) + 32 h + 16 (u % 2) + 8 s + [0, 8): 8 bytes of codes are both steps of a row
// (of 4-bit L the last unit can lie past the padded rank in part: zeros on both sides).
template <bool AQ>
__host__ __device__ __forceinline__ int mid_units(int rank_pad) { return AQ ? 2 * ((rank_pad + 63) / 64) : rank_pad / 32; }
template <bool AQ>
__device__ __forceinline__ uint32_t mid_rank(uint32_t u, uint32_t s, uint32_t h)
{
    return AQ ? 64u * (u >> 1) + 32u * h + 16u * (u & 1u) + 8u * s : 32u * u + 16u * s + 8u * h;
}
// T as pieces {call number, four fp16 ranks, checksum}, ordered [32 tokens][unit][step][four ranks of the eight][h]
// [token]: the B operand of a step is two contiguous KiB.  The piece of token t and ranks r .. r + 3 (r % 4 == 0):
template <bool AQ>
__device__ __forceinline__ uint32_t mid_t_piece(uint32_t t, uint32_t r, int rank_pad)
{
    const uint32_t u = AQ ? 2u * (r >> 6) + ((r >> 4) & 1u) : r >> 5;
    const uint32_t st = AQ ? (r >> 3) & 1u : (r >> 4) & 1u, h = AQ ? (r >> 5) & 1u : (r >> 3) & 1u;
    return ((t >> 5) * (uint32_t)mid_units<AQ>(rank_pad) + u) * 4096u + (2u * st + ((r >> 2) & 1u)) * 1024u + (32u * h + (t & 31u)) * 16u;
}
template <bool AQ>
__host__ __device__ __forceinline__ uint32_t mid_t_bytes(int m, int rank_pad) { return (uint32_t)((m + 31) / 32 * mid_units<AQ>(rank_pad)) * 4096u; }

// Tile j of a role whose workgroups are dealt to the dies in turn (index mod 8): the tiles of one row tile
// run on one die, whose L2 then reads the row tile once.  A role has die_tiles() workgroups; false: no tile.
__device__ __forceinline__ bool tile_on_die(int b, int tiles_o, int &ot, int &tt)
{
    const int per = (tiles_o + kDies - 1) / kDies, j = b / kDies;
    ot = b % kDies + kDies * (j % per);
    tt = j / per;
    return ot < tiles_o;
}
static int die_tiles(int tiles_o, int tiles_t) { return (tiles_o + kDies - 1) / kDies * kDies * tiles_t; }

// T tile of 16 ranks x 16 TT tokens.  A unit is 256 / TT inputs: steps of V_MFMA_F32_16X16X32_F16, R from memory
// into registers in operand order (runs of 256 bytes), X through LDS: in operand order neighbouring lanes are
// different tokens, and such a load costs the address unit four times one that reads along the rows.
// Wavefront w takes the units w, w + 12, ..., with 8 KiB of LDS of its own.
// Which columns step t multiplies on lane quarter ly is free as long as R and X agree:
//   fp16 R, fp16 X   32 t + 8 ly + [0, 8)
//   fp16 R, 8-bit X  64 (t / 2) + 16 ly + 8 (t % 2) + [0, 8): two steps share one 16-byte load of codes
//   4-bit R          (64 / TT) ly + 8 t + [0, 8): the columns of a lane are consecutive (16 bytes of codes for four steps, one scale)
constexpr int kTUnitLds = 8192;
template <int XF, bool AQ, int TT, bool HIDE>
__device__ __forceinline__ void t_tile(const MidArgs &a, int rt, int tt, char *lds_c, unsigned epoch)
{
    constexpr int TW = kMidWaves + kMidHelpers, UN = 256 / TT, STEPS = UN / 32;
    constexpr int ROWB = XF ? UN : 2 * UN, PIECES = ROWB / 16, TPI = 64 / PIECES, NX = 16 * TT / TPI;
    // (HIDE: a thread number the compiler knows nothing of, so that nothing worked out of it stays in registers from one tile to the next)
    unsigned tid = threadIdx.x;
    if constexpr (HIDE) asm volatile("" : "+v"(tid));
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lx = lane & 15, ly = lane >> 4;
    const int units = (a.k + UN - 1) / UN;
    const uint32_t k = (uint32_t)a.k, xb = XF ? 1u : 2u;
    const rsrc_t x_rs = make_rsrc(a.X, (uint32_t)a.m * k * xb);
    const rsrc_t r_rs = AQ ? make_rsrc(a.Rq, (uint32_t)q4_code_bytes(a.rank, a.k)) : make_rsrc(a.R, (uint32_t)tl_bytes(a.rank_pad, a.k));
    const rsrc_t s_rs = make_rsrc(AQ ? a.Rs : nullptr, AQ ? (uint32_t)q4_scale_bytes(a.rank, a.k) : 0u);
    char *const xl = lds_c + wave * kTUnitLds;
    const uint32_t xl0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds_c + (uint32_t)(wave * kTUnitLds);

    auto column = [&](int u, int t) -> uint32_t {
        if (AQ) return (uint32_t)(UN * u) + (uint32_t)(UN / 4) * ly + 8u * t;
        if (XF) return (uint32_t)(UN * u) + 64u * (t >> 1) + 16u * ly + 8u * (t & 1);
        return (uint32_t)(UN * u) + 32u * t + 8u * ly;
    };
    // the pieces of 16 bytes of a token's row of LDS are permuted by the token number (two rows of 128 bytes go round the banks together)
    auto swz = [](int tok) { return (uint32_t)(ROWB >= 256 ? tok & 15 : (tok >> 1) & 7); };
    float4_t acc0[TT], acc1[TT];
#pragma unroll
    for (int it = 0; it < TT; ++it) acc0[it] = acc1[it] = float4_t{0.f, 0.f, 0.f, 0.f};
    __syncthreads();                            // the tile before this one is done with LDS
    for (int u = wave; u < units; u += TW) {
        // a token's inputs are one row of LDS
#pragma unroll
        for (int j = 0; j < NX; ++j) {
            const int tj = TPI * j + lane / PIECES;
            const uint32_t col = ((uint32_t)(lane % PIECES) ^ swz(tj)) * (16u / xb);
            const bool ok = 16 * TT * tt + tj < a.m && (uint32_t)(UN * u) + col < k;
            load_to_lds(x_rs, ok ? ((uint32_t)(16 * TT * tt + tj) * k + (uint32_t)(UN * u) + col) * xb : kPastEnd, 0u, xl0 + (uint32_t)j * 1024u);
        }
        uint4_t rv[AQ ? 2 / TT : STEPS];
        half_t sc = (half_t)1.0f;
        if constexpr (AQ) {
            const bool ok = column(u, 0) < k;
            const uint32_t base = ok ? q4_piece(16u * rt + lx, (uint32_t)(UN / 64) * u + ly / TT, q4_ctiles(a.k)) + (TT == 2 ? 16u * (ly & 1) : 0u) : kPastEnd;
#pragma unroll
            for (int t = 0; t < 2 / TT; ++t) rv[t] = load16(r_rs, ok ? base + 16u * t : kPastEnd, 0);
            sc = load_half(s_rs, ok ? ((16u * rt + lx) * q4_groups(a.k) + (uint32_t)(UN / 128) * u + ly / (2 * TT)) * 2u : kPastEnd, 0);
        } else {
#pragma unroll
            for (int t = 0; t < STEPS; ++t) {
                const uint32_t c = column(u, t);
                rv[t] = load16(r_rs, c < k ? tl_piece(16u * rt + lx, c >> 3, k) : kPastEnd, 0);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
#pragma unroll
        for (int t = 0; t < STEPS; ++t) {
            const uint32_t c = column(0, t) * xb;               // byte of the row
            half8_t av;
            if constexpr (AQ)
                av = codes_to_half8(rv[t >> 2][t & 3]) * sc;
            else
                av = __builtin_bit_cast(half8_t, rv[t]);
#pragma unroll
            for (int it = 0; it < TT; ++it) {
                const uint4_t xv = *reinterpret_cast<const uint4_t *>(xl + (16 * it + lx) * ROWB + (((c >> 4) ^ swz(lx)) << 4));
                half8_t bv;
                if constexpr (XF == 0)
                    bv = __builtin_bit_cast(half8_t, xv);
                else
                    bv = codes8_to_half8<XF>(xv[2 * (t & 1)], xv[2 * (t & 1) + 1]);
                if (t & 1)
                    acc1[it] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bv, acc1[it], 0, 0, 0);
                else
                    acc0[it] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bv, acc0[it], 0, 0, 0);
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");     // the row of LDS has been read
    }
    float4_t *const red = reinterpret_cast<float4_t *>(lds_c);
    // wavefront it < TT adds up 16 tokens.  Lane: token lx, ranks 16 rt + 4 ly .. + 3
    __syncthreads();
#pragma unroll
    for (int it = 0; it < TT; ++it)
        if (wave != it) red[(it * TW + wave) * kWave + lane] = acc0[it] + acc1[it];
    __syncthreads();
    if (wave >= TT) return;
#pragma unroll
    for (int it = 0; it < TT; ++it) {
        if (TT > 1 && wave != it) continue;
        float4_t acc = acc0[it] + acc1[it];
#pragma unroll
        for (int w = 0; w < TW; ++w)
            if (w != it) acc += red[(it * TW + w) * kWave + lane];
        if (XF) acc *= *a.x_scale;
        const int tok = 16 * (TT * tt + it) + lx;
        const half4_t h = {(half_t)acc[0], (half_t)acc[1], (half_t)acc[2], (half_t)acc[3]};
        if (a.T_rows) {
            if (tok < a.m) *reinterpret_cast<half4_t *>(a.T_rows + (size_t)tok * a.rank_pad + 16 * rt + 4 * ly) = h;
        } else if (TT == 1 || tok < (a.m + 15) / 16 * 16) {
            store_piece(make_rsrc(a.T, mid_t_bytes<AQ>(a.m, a.rank_pad)), mid_t_piece<AQ>((uint32_t)tok, 16u * rt + 4u * ly, a.rank_pad),
                        epoch, __builtin_bit_cast(uint2_t, h));
        }
    }
}

// ---- T = X R^T as a launch of its own: larger tiles, for batches that fill the chip with them ----
// Tile of 32 RT ranks x 32 TT tokens per workgroup; the twelve wavefronts divide the inputs in units of 128 / TT, each the
// whole tile on its units with V_MFMA_F32_32X32X16_F16 (R from memory into registers, X through 8 KiB of LDS
// of its own, no barrier on the way), and add up in LDS.  What bounds it is the 64 bytes a compute unit
// draws per clock from its L2: (32 RT + 32 TT) x 2 bytes of them per input, which is why the tile grows
// with the batch.
//   Whole calls, against a product split over workgroups (256 x 128): 8192 x 8192 at 1000 tokens 125.0 -> 117.4 us, 11008 x 4096 at 333 tokens 55.2 -> 45.2.
// Columns of a unit that step j multiplies on lane half h:
//   fp16 R, fp16 X   16 j + 8 h + [0, 8)
//   fp16 R, 8-bit X  32 (j / 2) + 16 h + 8 (j % 2) + [0, 8): two steps share one piece of codes
//   4-bit R          64 (j / 4) + 32 h + 8 (j % 4) + [0, 8): four steps share one 16-byte load of codes, one scale
struct TArgs {
    const half_t *X;
    const float *x_scale;
    const half_t *R;
    const uint8_t *Rq;
    const half_t *Rs;
    int k, rank, rank_pad, m;
    int tiles_t, tiles_r;    // token tiles, rank tiles
    half_t *T;               // fp16 [m][rank_pad], or
    uint4_t *pieces;         // pieces of T (mid_t_piece()) with this call's number
    bool q4_order;           //   in the order for 4-bit L
    CallEpoch epoch;
};

template <int RT, int TT, int XF, bool AQ>
__global__ __launch_bounds__(kMidThreads, 3) void t_product_kernel(TArgs a)
{
    constexpr int TW = kMidWaves + kMidHelpers;
    constexpr int U = 128 / TT, STEPS = U / 16;          // inputs and steps of a unit
    constexpr int ROWB = XF ? U : 2 * U;                 // bytes of a token's unit
    constexpr int P = ROWB / 16, RPB = 16 / P;           // pieces of 16 bytes per row, rows per 256 bytes
    constexpr int TPI = 64 / P, NX = 32 * TT / TPI;      // tokens per load instruction, instructions per unit
    extern __shared__ __attribute__((aligned(16))) char lds_c[];
    const int lane = threadIdx.x & (kWave - 1), li = lane & 31, lb = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    // the tiles of one token tile run on one die, whose L2 then reads X once (R, the smaller operand, is read by every die)
    int rt, tt;
    if (!tile_on_die((int)blockIdx.x, a.tiles_t, tt, rt)) return;
    const int t0 = tt * 32 * TT, r0 = rt * 32 * RT;
    const uint32_t k = (uint32_t)a.k, xb = XF ? 1u : 2u;
    const rsrc_t x_rs = make_rsrc(a.X, (uint32_t)a.m * k * xb);
    const rsrc_t r_rs = AQ ? make_rsrc(a.Rq, (uint32_t)q4_code_bytes(a.rank, a.k)) : make_rsrc(a.R, (uint32_t)tl_bytes(a.rank_pad, a.k));
    const rsrc_t s_rs = make_rsrc(AQ ? a.Rs : nullptr, AQ ? (uint32_t)q4_scale_bytes(a.rank, a.k) : 0u);
    const uint32_t x_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds_c + (uint32_t)(wave * kTUnitLds);
    const char *const xl = lds_c + wave * kTUnitLds + li * ROWB;
    const int units = (a.k + U - 1) / U;                 // (k is a multiple of 128)
    // loads of X: lane -> (token, slot piece), source piece = slot piece ^ swizzle(token)
    const int stok = lane / P;
    const uint32_t xoff = (uint32_t)(t0 + stok) * k * xb;
    auto swz = [](int tok) { return (uint32_t)((tok / RPB) & (P - 1)); };
    auto col = [&](int j) -> uint32_t {
        if (AQ) return 64u * (j >> 2) + 32u * lb + 8u * (j & 3);
        if (XF) return 32u * (j >> 1) + 16u * lb + 8u * (j & 1);
        return 16u * j + 8u * lb;
    };
    float16_t acc[RT][TT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int it = 0; it < TT; ++it)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][it][e] = 0.f;
    for (int u = wave; u < units; u += TW) {
#pragma unroll
        for (int q = 0; q < NX; ++q) {
            const int tok = TPI * q + stok;
            load_to_lds(x_rs, xoff + (uint32_t)(TPI * q) * k * xb + (((uint32_t)(lane % P) ^ swz(tok)) << 4), (uint32_t)(u * U) * xb, x_lds + (uint32_t)q * 1024u);
        }
        uint4_t rv[RT][AQ ? STEPS / 4 : STEPS];
        half_t sc[RT];
#pragma unroll
        for (int i = 0; i < RT; ++i) {
            const uint32_t row = (uint32_t)(r0 + 32 * i + li);
            if constexpr (AQ) {
#pragma unroll
                for (int q = 0; q < STEPS / 4; ++q)
                    rv[i][q] = load16(r_rs, q4_piece(row, (uint32_t)(u * U) / 64u + q, q4_ctiles(a.k)) + 16u * lb, 0);
                sc[i] = load_half(s_rs, (row * q4_groups(a.k) + (uint32_t)(u * U) / 128u) * 2u, 0);
            } else {
#pragma unroll
                for (int j = 0; j < STEPS; ++j) rv[i][j] = load16(r_rs, tl_piece(row, ((uint32_t)(u * U) + col(j)) >> 3, k), 0);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
#pragma unroll
        for (int j = 0; j < STEPS; ++j) {
            half8_t av[RT], bv[TT];
            const uint32_t piece = XF ? col(j) >> 4 : col(j) >> 3;
#pragma unroll
            for (int it = 0; it < TT; ++it) {
                const uint4_t v = *reinterpret_cast<const uint4_t *>(xl + it * 32 * ROWB + ((piece ^ swz(li)) << 4));
                if constexpr (XF == 0)
                    bv[it] = __builtin_bit_cast(half8_t, v);
                else
                    bv[it] = codes8_to_half8<XF>(v[2 * (j & 1)], v[2 * (j & 1) + 1]);
            }
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                if constexpr (AQ)
                    av[i] = codes_to_half8(rv[i][j >> 2][j & 3]) * sc[i];
                else
                    av[i] = __builtin_bit_cast(half8_t, rv[i][j]);
            }
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int it = 0; it < TT; ++it) acc[i][it] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[i], bv[it], acc[i][it], 0, 0, 0);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");     // the unit's LDS has been read
    }
    // add up: the upper six wavefronts to the lower six, then all of those by (tile, block of 8 rows)
    constexpr int TILES = RT * TT, HALF = TW / 2;
    float4_t *const red = reinterpret_cast<float4_t *>(lds_c);
    auto put = [&](int w) {
#pragma unroll
        for (int x = 0; x < TILES; ++x)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const float16_t &v = acc[x / TT][x % TT];
                red[((w * TILES + x) * 4 + b) * kWave + lane] = float4_t{v[4 * b], v[4 * b + 1], v[4 * b + 2], v[4 * b + 3]};
            }
    };
    __syncthreads();
    if (wave >= HALF) put(wave - HALF);
    __syncthreads();
    if (wave < HALF) {
#pragma unroll
        for (int x = 0; x < TILES; ++x)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const float4_t v = red[((wave * TILES + x) * 4 + b) * kWave + lane];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[x / TT][x % TT][4 * b + e] += v[e];
            }
        put(wave);                               // (its own place, which only it has read)
    }
    __syncthreads();
    const float xs = XF ? *a.x_scale : 1.0f;
    const unsigned epoch = a.pieces ? call_epoch(a.epoch) : 0u;
    for (int q = wave; q < 4 * TILES; q += TW) {
        const int x = q >> 2, b = q & 3;
        float4_t v = red[(x * 4 + b) * kWave + lane];
#pragma unroll
        for (int w = 1; w < HALF; ++w) v += red[((w * TILES + x) * 4 + b) * kWave + lane];
        if (XF) v *= xs;
        const half4_t h = {(half_t)v[0], (half_t)v[1], (half_t)v[2], (half_t)v[3]};
        // lane holds token t, ranks r .. r + 3
        const int t = t0 + 32 * (x % TT) + li, r = r0 + 32 * (x / TT) + 8 * b + 4 * lb;
        if (r >= a.rank_pad) continue;
        if (a.pieces) {
            const rsrc_t p_rs = make_rsrc(a.pieces, a.q4_order ? mid_t_bytes<true>(a.m, a.rank_pad) : mid_t_bytes<false>(a.m, a.rank_pad));
            const uint32_t off = a.q4_order ? mid_t_piece<true>((uint32_t)t, (uint32_t)r, a.rank_pad) : mid_t_piece<false>((uint32_t)t, (uint32_t)r, a.rank_pad);
            store_piece(p_rs, t < (a.m + 31) / 32 * 32 ? off : kPastEnd, epoch, __builtin_bit_cast(uint2_t, h));
        } else if (t < a.m) {
            *reinterpret_cast<half4_t *>(a.T + (size_t)t * a.rank_pad + r) = h;
        }
    }
}

template <int RT, int TT>
static void launch_t_tiles(TArgs a, int xf, hipStream_t st)
{
    a.tiles_t = (a.m + 32 * TT - 1) / (32 * TT);
    a.tiles_r = (a.rank_pad + 32 * RT - 1) / (32 * RT);
    const dim3 grid((unsigned)die_tiles(a.tiles_t, a.tiles_r)), blk(kMidThreads);
    constexpr size_t lds = (size_t)(kMidWaves + kMidHelpers) * kTUnitLds;        // the partial tiles, 24 RT TT KiB, fit
    static_assert((kMidWaves + kMidHelpers) / 2 * RT * TT * 4096 <= (kMidWaves + kMidHelpers) * kTUnitLds, "partial tiles");
    if (a.Rq) {
        if (xf == 0)
            hipLaunchKernelGGL((t_product_kernel<RT, TT, 0, true>), grid, blk, lds, st, a);
        else if (xf == 1)
            hipLaunchKernelGGL((t_product_kernel<RT, TT, 1, true>), grid, blk, lds, st, a);
        else
            hipLaunchKernelGGL((t_product_kernel<RT, TT, 2, true>), grid, blk, lds, st, a);
    } else {
        if (xf == 0)
            hipLaunchKernelGGL((t_product_kernel<RT, TT, 0, false>), grid, blk, lds, st, a);
        else if (xf == 1)
            hipLaunchKernelGGL((t_product_kernel<RT, TT, 1, false>), grid, blk, lds, st, a);
        else
            hipLaunchKernelGGL((t_product_kernel<RT, TT, 2, false>), grid, blk, lds, st, a);
    }
}

// ---- the same in tiles of 128 ranks x 128 tokens, the inputs split over workgroups where there are few ----
// What bounds the tiles above on many tokens is what they draw from the L2 (64 x 64: 21 TB/s over the chip); these draw half of that.
//   X and R come by direct-to-LDS loads, a stage of 64 inputs at a time, three stages ahead in a ring of four.  The eight wavefronts are four groups, each
// on one of the four steps of a stage, and a wavefront has 128 ranks x 64 tokens (4 x 2 tiles of V_MFMA_F32_32X32X16_F16): six operands read from LDS
// for eight products.  They read one stage ahead, and the loads stand between the products: issued together before them they kept
// the matrix core waiting for a place in the load queue.  The groups add up in LDS at the end.
//   A stage takes 0.34 us on a part of the chip, 0.47 on all of it (LDS 0.29, products 0.21).  Neither the reads one stage ahead (64.8 -> 61.3 us at
// 4096 x 832 x 8192) nor fewer reads (60.3) changed much; conversion of 4-bit codes adds 0.2 us.
//   A die works on one range of the inputs (or several dies on the same), so that all dies together read X and R little more than once.  The partial sums
// cost their way through memory and a launch that adds them up: 8 us at two ranges of 2048 x 416, 13 at four of 1000 x 832.
//   tokens x ranks x inputs, us: this / split product with 256 x 128 tiles, before / 64 x 64 tiles:
//   4096 x 832 x 8192 60 / 72 / 103, 2048 x 1120 x 5120 35 / 50 / 52, with 8-bit X (k 4096) 29 / 42 / 40, 4-bit R (4096 x 832 x 8192) 79 / 86 / 116;
//   over 500 drawn products (128 to 4096 tokens, ranks 32 to 1400, 512 to 28672 inputs) the kind now taken is 8 % faster on average than the one launch with
//   fp16 R, up to 2.5 times, and 2 % in 4 bits.
// Columns of a stage that step j (of four) multiplies on lane half h
//   fp16 R, fp16 X   16 j + 8 h + [0, 8)
//   fp16 R, 8-bit X  32 (j / 2) + 16 h + 8 (j % 2) + [0, 8)
//   4-bit R          32 h + 8 j + [0, 8)
constexpr int kBigStage = 64, kBigRing = 4, kBigWaves = 8;
constexpr int kBigRange = 32768;     // inputs whose 4-bit scales fit in LDS beside the ring
struct TBigArgs {
    TArgs t;
    int splits, ks;          // ranges of the inputs (1, 2, 4 or 8), inputs in each (a multiple of 128)
    int per;                 // tiles of a die
    float *P;                // splits > 1: fp32 [splits][m][rank_pad]
};
template <int XF, bool AQ>
__global__ __launch_bounds__(kBigWaves * kWave, 2) void t_big_kernel(TBigArgs b)
{
    const TArgs &a = b.t;
    constexpr int XROW = XF ? 64 : 128, PIECES = XROW / 16, TPI = 64 / PIECES;        // bytes of a token's stage, pieces of it, tokens per load
    constexpr int XBYTES = 128 * XROW, RBYTES = AQ ? 4096 : 16384, SLOT = XBYTES + RBYTES;
    constexpr int NX = XBYTES / 1024, NR = RBYTES / 1024, NL = (NX + NR) / kBigWaves;  // loads of a stage; per wavefront
    constexpr int LEFT = (NX + NR) % kBigWaves;                                       // (4-bit R and 16-bit X: the first wavefronts have one more)
    extern __shared__ __attribute__((aligned(16))) char lds_c[];
    const int lane = threadIdx.x & (kWave - 1), li = lane & 31, lb = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int group = wave >> 1, th = wave & 1;             // this wavefront's step of a stage, its half of the tokens
    const int die = (int)blockIdx.x % kDies, share = kDies / b.splits, z = die / share;
    const int tile = (die % share) * b.per + (int)blockIdx.x / kDies;
    if (tile >= a.tiles_t * a.tiles_r) return;
    const int r0 = tile % a.tiles_r * 128, t0 = tile / a.tiles_r * 128;
    const uint32_t k = (uint32_t)a.k, xb = XF ? 1u : 2u;
    int k0 = z * b.ks;
    const int k_end = min(a.k, k0 + b.ks);
    int stages = 0;                                         // of the part of the range that starts at k0
    const rsrc_t x_rs = make_rsrc(a.X, (uint32_t)a.m * k * xb);
    const rsrc_t r_rs = AQ ? make_rsrc(a.Rq, (uint32_t)q4_code_bytes(a.rank, a.k)) : make_rsrc(a.R, (uint32_t)tl_bytes(a.rank_pad, a.k));
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds_c;
    auto swz = [](int tok) { return (uint32_t)(XF ? (tok >> 2) & 3 : (tok >> 1) & 7); };
    const uint32_t ct = q4_ctiles(a.k);
    // load i of this wavefront's NL of stage s, to its place in the ring (the last stage again past the end; nobody uses it)
    auto load = [&](int s, auto ic) {
        constexpr int i = ic;
        const uint32_t to = lds0 + (uint32_t)(s % kBigRing) * SLOT + (uint32_t)wave * 1024u, c0 = (uint32_t)(k0 + min(s, stages - 1) * kBigStage);
        if constexpr (i < NX / kBigWaves) {
            const int tok = TPI * (kBigWaves * i + wave) + lane / PIECES;
            load_to_lds(x_rs, (uint32_t)(t0 + tok) * k * xb + (((uint32_t)(lane % PIECES) ^ swz(tok)) << 4), c0 * xb, to + (uint32_t)i * 8192u);
        } else if constexpr (AQ) {
            if (wave < LEFT) {
                const uint32_t row = (uint32_t)(r0 + 32 * wave + li);
                load_to_lds(r_rs, q4_piece(row, 0, ct) + 16u * lb, (c0 >> 8) * 2048u + ((c0 >> 6) & 3u) * 32u, to + XBYTES);
            }
        } else {
            constexpr int j = i - NX / kBigWaves;
            const uint32_t p = (uint32_t)(kBigWaves * j + wave);     // row tile p / 4, columns 16 (p % 4) .. of the stage
            load_to_lds(r_rs, ((uint32_t)(r0 / 32) + p / 4) * (k >> 4) * 1024u + (uint32_t)lane * 16u, ((c0 >> 4) + p % 4) * 1024u,
                        to + XBYTES + (uint32_t)j * 8192u);
        }
    };
    auto load_stage = [&](int s) { static_for<NL + (LEFT > 0)>([&](auto ic) { load(s, ic); }); };
    half_t *const scales = reinterpret_cast<half_t *>(lds_c + kBigRing * SLOT);       // 4-bit R: [group of 128][row]
    float16_t acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int it = 0; it < 2; ++it)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][it][e] = 0.f;
    // what a wavefront multiplies of a stage: one step of its two tiles of X and four of R
    using XPart = std::conditional_t<XF != 0, uint2_t, uint4_t>;
    using RPart = std::conditional_t<AQ, uint32_t, uint4_t>;
    struct Part {
        XPart x[2];
        RPart r[4];
    };
    // every wavefront's loads of stage s are here when at most the two after it are in flight; past the barrier all may read it, and the place of the
    // one before, whose reads have ended, is free
    auto arrive = [&]() {
        if (LEFT > 0 && wave < LEFT)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"((kBigRing - 2) * (NL + 1)) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"((kBigRing - 2) * NL) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" : : : "memory");
    };
    auto read = [&](Part &f, int s) {
        const char *const xs = lds_c + (s % kBigRing) * SLOT, *const rs = xs + XBYTES;
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const int tok = 64 * th + 32 * it + li;
            const uint32_t piece = XF ? (AQ ? 2u * lb + group / 2 : 2u * (group / 2) + lb) : (AQ ? 4u * lb + group : 2u * group + lb);
            f.x[it] = *reinterpret_cast<const XPart *>(xs + tok * XROW + ((piece ^ swz(tok)) << 4) + (XF ? 8 * (group % 2) : 0));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            f.r[i] = *reinterpret_cast<const RPart *>(AQ ? rs + i * 1024 + lane * 16 + 4 * group
                                                         : rs + i * 4096 + (XF ? (2 * (group / 2) + lb) * 1024 + (32 * (group % 2) + li) * 16
                                                                               : group * 1024 + lane * 16));
    };
    half_t sc[4] = {};
    // the loads of stage `next` between the products, so that a full load queue does not keep the matrix core waiting
    auto multiply = [&](const Part &f, int next) {
        half8_t bv[2];
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            if constexpr (XF == 0)
                bv[it] = __builtin_bit_cast(half8_t, f.x[it]);
            else
                bv[it] = codes8_to_half8<XF>(f.x[it][0], f.x[it][1]);
        }
        // (4-bit R: the conversion of the next row tile's codes, 17 vector instructions, beside this one's products)
        auto row_tile = [&](int i) {
            if constexpr (AQ)
                return codes_to_half8(f.r[i]) * sc[i];
            else
                return __builtin_bit_cast(half8_t, f.r[i]);
        };
        half8_t av = row_tile(0);
        if constexpr (AQ) __builtin_amdgcn_sched_barrier(0);
        static_for<4>([&](auto ic) {
            constexpr int i = ic;
            half8_t next_av = av;
            if constexpr (i < 3) next_av = row_tile(i + 1);
#pragma unroll
            for (int it = 0; it < 2; ++it) acc[i][it] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, bv[it], acc[i][it], 0, 0, 0);
            if constexpr (AQ && i < 3) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x2, 8, 0);
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x2, 9, 0);
            }
            av = next_av;
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (i < NL + (LEFT > 0)) load(next, ic);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    for (; k0 < k_end; k0 += kBigRange) {
        // (more than one part only with 4-bit R: without it a range has one)
        const int klen = AQ ? min(kBigRange, k_end - k0) : k_end - k0;
        stages = klen / kBigStage;
        if constexpr (AQ) {
            const rsrc_t s_rs = make_rsrc(a.Rs, (uint32_t)q4_scale_bytes(a.rank, a.k));
            for (int i = threadIdx.x; i < klen; i += kBigWaves * kWave)
                scales[i] = load_half(s_rs, ((uint32_t)(r0 + i % 128) * q4_groups(a.k) + (uint32_t)(k0 / 128 + i / 128)) * 2u, 0);
        }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : : : "memory");
#pragma unroll
        for (int s = 0; s < kBigRing - 1; ++s) load_stage(s);
        arrive();
        Part f0, f1;
        read(f0, 0);
        load_stage(kBigRing - 1);
        for (int s = 0; s < stages; s += 2) {
            if constexpr (AQ)
#pragma unroll
                for (int i = 0; i < 4; ++i) sc[i] = scales[s / 2 * 128 + 32 * i + li];
            arrive();
            read(f1, s + 1);
            multiply(f0, s + kBigRing);
            arrive();
            read(f0, s + 2);
            multiply(f1, s + 1 + kBigRing);
        }
        // the loads past the end have landed and every wavefront has read what it reads
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : : : "memory");
        __syncthreads();
        if constexpr (!AQ) break;
    }
    // the groups add up: group g stores row tile g, 32 tokens at a time, with what the three others have left in LDS
    float4_t *const red = reinterpret_cast<float4_t *>(lds_c) + th * 12 * 256 + lane;       // [th][row tile][of three][4][lane]
    const float xscale = XF ? *a.x_scale : 1.0f;
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        if (it) __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i != group)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    red[(3 * i + ((group - i) & 3) - 1) * 256 + q * kWave] = float4_t{acc[i][it][4 * q], acc[i][it][4 * q + 1], acc[i][it][4 * q + 2], acc[i][it][4 * q + 3]};
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i == group)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float4_t v = {acc[i][it][4 * q], acc[i][it][4 * q + 1], acc[i][it][4 * q + 2], acc[i][it][4 * q + 3]};
#pragma unroll
                    for (int o = 0; o < 3; ++o) v += red[(3 * i + o) * 256 + q * kWave];
                    if (XF) v *= xscale;
                    // lane holds token t, ranks r .. r + 3
                    const int t = t0 + 64 * th + 32 * it + li, r = r0 + 32 * i + 8 * q + 4 * lb;
                    if (t >= a.m || r >= a.rank_pad) continue;
                    if (b.splits > 1)
                        *reinterpret_cast<float4_t *>(b.P + ((size_t)z * a.m + t) * a.rank_pad + r) = v;
                    else
                        *reinterpret_cast<half4_t *>(a.T + (size_t)t * a.rank_pad + r) = half4_t{(half_t)v[0], (half_t)v[1], (half_t)v[2], (half_t)v[3]};
                }
    }
}

// T[i] = fp16(sum_z P[z][i]), four at a time
template <int S>
__global__ __launch_bounds__(256) void t_sum_kernel(const float4_t *__restrict__ P, size_t count, half4_t *__restrict__ T)
{
    const size_t i = blockIdx.x * (size_t)256 + threadIdx.x;
    if (i >= count) return;
    float4_t v[S];
#pragma unroll
    for (int z = 0; z < S; ++z) v[z] = P[(size_t)z * count + i];
#pragma unroll
    for (int z = 1; z < S; ++z) v[0] += v[z];
    T[i] = half4_t{(half_t)v[0][0], (half_t)v[0][1], (half_t)v[0][2], (half_t)v[0][3]};
}

static void launch_t_big(const TArgs &t, int xf, int splits, float *P, hipStream_t st)
{
    TBigArgs b{};
    b.t = t;
    b.t.tiles_t = (t.m + 127) / 128;
    b.t.tiles_r = (t.rank_pad + 127) / 128;
    b.splits = splits;
    b.ks = (t.k / 128 + splits - 1) / splits * 128;
    b.P = P;
    const int share = kDies / splits, tiles = b.t.tiles_t * b.t.tiles_r;
    b.per = (tiles + share - 1) / share;
    const dim3 grid((unsigned)(kDies * b.per)), blk(kBigWaves * kWave);
    // the ring and the scales of a range, and not less than what the groups leave at the end
    auto bytes = [&](int x, int r) {
        const int range = b.ks < kBigRange ? b.ks : kBigRange;
        const size_t v = (size_t)kBigRing * (128 * (x ? 64 : 128) + (r ? 4096 : 16384)) + (r ? 2 * (size_t)range : 0);
        return v > 98304 ? v : (size_t)98304;
    };
    if (t.Rq) {
        if (xf == 0)
            hipLaunchKernelGGL((t_big_kernel<0, true>), grid, blk, bytes(0, 1), st, b);
        else if (xf == 1)
            hipLaunchKernelGGL((t_big_kernel<1, true>), grid, blk, bytes(1, 1), st, b);
        else
            hipLaunchKernelGGL((t_big_kernel<2, true>), grid, blk, bytes(2, 1), st, b);
    } else {
        if (xf == 0)
            hipLaunchKernelGGL((t_big_kernel<0, false>), grid, blk, bytes(0, 0), st, b);
        else if (xf == 1)
            hipLaunchKernelGGL((t_big_kernel<1, false>), grid, blk, bytes(1, 0), st, b);
        else
            hipLaunchKernelGGL((t_big_kernel<2, false>), grid, blk, bytes(2, 0), st, b);
    }
    if (splits > 1) {
        const size_t count = (size_t)t.m * t.rank_pad / 4;
        const dim3 sums((unsigned)((count + 255) / 256));
        const float4_t *p = reinterpret_cast<const float4_t *>(P);
        half4_t *out = reinterpret_cast<half4_t *>(t.T);
        if (splits == 2)
            hipLaunchKernelGGL(t_sum_kernel<2>, sums, dim3(256), 0, st, p, count, out);
        else if (splits == 4)
            hipLaunchKernelGGL(t_sum_kernel<4>, sums, dim3(256), 0, st, p, count, out);
        else
            hipLaunchKernelGGL(t_sum_kernel<8>, sums, dim3(256), 0, st, p, count, out);
    }
}

// As launch_t_product(), in tiles of 128 x 128 with the inputs in `splits` (1, 2, 4, 8) ranges; P: fp32 [splits][m][rank_pad] where that is
// more than one.  The caller keeps X and R below 4 GiB each.
int launch_t_split(const half_t *X, int xf, const float *x_scale, int m, int k, const half_t *R, const uint8_t *Rq, const half_t *Rs, int rank,
                   int rank_pad, half_t *T, float *P, int splits, hipStream_t st)
{
    TArgs a{};
    a.X = X;
    a.x_scale = x_scale;
    a.R = R;
    a.Rq = R ? nullptr : Rq;
    a.Rs = Rs;
    a.k = k;
    a.rank = rank;
    a.rank_pad = rank_pad;
    a.m = m;
    a.T = T;
    launch_t_big(a, xf, splits, P, st);
    return hip_status(hipGetLastError());
}

// ---- which kernel makes T ----
// 0, 1, 2: t_product_kernel with tiles of 32 x 32, 32 x 64, 64 x 64 (ranks x tokens); 3: the 16 x 16 tiles of the T role; 4:
// t_big_kernel, the inputs in t_splits() ranges.  The one whose estimated time is the shortest.  A kind
// that deals its tiles to the dies takes as many rounds as its fullest die has tiles for its compute units (with 10 tiles of
// tokens two dies have two, and 18 rank tiles make that 36 workgroups on 32 units: twice the time), and
//   time = a + rounds (b + k / 1000 (c + d w)),   w = the share of that die's units with a tile in the first round,
// or, where several dies read all of R, what that takes at 7 TB/s for all eight, three of them no faster (28672 inputs, rank 832,
// 48 MB: kind 0 44 us at 64 tokens, 54 at 100, 55 at 200 and 256, where the first estimate says 38).  For kind 4, k is that of a range, the dies of one
// range share the tiles, and several ranges add e + f per million partial sums.  The constants (us) are
// fitted to 6048 measured products (ranks 32 to 1408, 17 to 4096 tokens, 512 to 28672 inputs, X in fp16 and 8 bits, R in
// fp16 and 4 bits; kind 4: 500, at every number of ranges): off by 5 to 15 %, 4 % for kind 4, which makes the kind taken 1 % slower than the best one on
// average.  Those of kind 4 with fp16 R are a tenth above the fit: where both are about as fast the one launch is taken, which needs no memory
// for partial sums (4096 x 416 x 4096 29.7 / 24.8, 8192 inputs, rank 832, 512 tokens 21.2 / 18.6).  Up to 128 tokens, one tile of them, kind 4 is not taken: the one launch is the faster
// there as long as a workgroup of it has one tile (rank 416 at 128 tokens, 8192 inputs 7.9 / 13.5, 28672 inputs 21.7 / 25.0), and where it has more (28672 inputs, rank 832, 100
// tokens 39 / 25) the calls are those of layers with too many rows for the small batches' tiles.
//   8192 inputs, fp16 (us; kinds 0 to 3): rank 64 at 800 tokens 10.6 / 14.8 / 20.5 / 20.3, rank 512 at 1000 tokens
//   27.0 / 20.6 / 25.8 / -, rank 832 at 600 tokens 37.1 / 37.2 / 27.6 / -, at 1000 tokens 49.2 / 37.5 / 27.8 / - (kind 4 there 25 to 26).
struct TCost {
    double a, b, c, d, e, f;
};
constexpr TCost kTCost[2][5] = {{{2.1, 1.1, 0.8, 0.5}, {2.0, 1.4, 1.2, 0.7}, {2.7, 1.6, 1.8, 1.0}, {1.9, 1.5, 0.3, 0.2}, {4.7, 1.7, 4.9, 1.5, 2.0, 2.2}},      // R in fp16
                                {{1.9, 1.6, 0.9, 0.2}, {1.8, 1.8, 1.4, 0.3}, {2.3, 2.4, 2.1, 0.7}, {1.6, 2.1, 0.5, 0.2}, {5.5, 0.2, 8.3, 0.75, 1.8, 2.0}}};   // in 4 bits

static double t_big_cost(int splits, int rank_pad, int m, int k, bool q4)
{
    const TCost &c = kTCost[q4][4];
    const int cus = device_info().cus, share = kDies / splits;
    const long tiles = (long)((rank_pad + 127) / 128) * ((m + 127) / 128), per_die = (tiles + share - 1) / share;
    const long units = cus / kDies > 0 ? cus / kDies : 1;
    const double w = per_die < units ? (double)per_die / units : 1.0;
    const double t = c.a + (double)((per_die + units - 1) / units) * (c.b + (k / 128 + splits - 1) / splits * 0.128 * (c.c + c.d * w));
    return splits > 1 ? t + c.e + c.f * splits * m * rank_pad * 1e-6 : t;
}

// The ranges of the inputs, up to those that the workspace has room for.
int t_splits(int rank_pad, int m, int k, bool q4)
{
    int best = 1;
    for (int s = 2; s <= gemm_t_splits(m, rank_pad, k); s *= 2)
        if (t_big_cost(s, rank_pad, m, k, q4) < t_big_cost(best, rank_pad, m, k, q4)) best = s;
    return best;
}

static double t_cost(int kind, int rank_pad, int m, int k, bool q4)
{
    if (kind == 4) return t_big_cost(t_splits(rank_pad, m, k, q4), rank_pad, m, k, q4);
    const TCost &c = kTCost[q4][kind];
    const int cus = device_info().cus;
    // tiles along the side that is dealt to the dies, and along the other
    constexpr int kSide[4][2] = {{32, 32}, {64, 32}, {64, 64}, {16, 16}};
    const int dealt = kind == 3 ? rank_pad : m, other = kind == 3 ? m : rank_pad;
    const long sides = (dealt + kSide[kind][0] - 1) / kSide[kind][0];
    const long per_die = (sides + kDies - 1) / kDies * ((other + kSide[kind][1] - 1) / kSide[kind][1]);
    const long units = cus / kDies > 0 ? cus / kDies : 1;
    const double w = per_die < units ? (double)per_die / units : 1.0;
    const double t = c.a + (double)((per_die + units - 1) / units) * (c.b + k * 1e-3 * (c.c + c.d * w));
    if (kind == 3) return t;
    const double r_us = c.a + (double)rank_pad * k * (q4 ? 0.53 : 2.0) * (sides > 2 ? kDies : sides) / 7e6;
    return r_us > t ? r_us : t;
}

// `split`: kind 4 may be taken (it leaves T as rows, not as pieces)
int t_kind(int rank_pad, int m, int k, bool q4, bool split)
{
    int best = 0;
    for (int kind = 1; kind < (split && m > 128 ? 5 : 4); ++kind)
        if (t_cost(kind, rank_pad, m, k, q4) < t_cost(best, rank_pad, m, k, q4)) best = kind;
    return best;
}

static void launch_t_role(const TArgs &a, int xf, hipStream_t st);
static int launch_t_product_args(const TArgs &a, int xf, hipStream_t st)
{
    switch (t_kind(a.rank_pad, a.m, a.k, a.Rq != nullptr, false)) {
        case 3: launch_t_role(a, xf, st); break;
        case 0: launch_t_tiles<1, 1>(a, xf, st); break;
        case 1: launch_t_tiles<1, 2>(a, xf, st); break;
        default: launch_t_tiles<2, 2>(a, xf, st); break;
    }
    return hip_status(hipGetLastError());
}

// T fp16 [m][rank_pad] = X R^T.  xf: 0 = X fp16; 1, 2 = X as E4M3 / E5M2 codes with the tensor's scale at x_scale.
// R: fp16 in the adapter layout, or null with Rq / Rs: the 4-bit codes and scales of R [rank][k].  The caller keeps the
// operands below 4 GiB each.
int launch_t_product(const half_t *X, int xf, const float *x_scale, int m, int k, const half_t *R, const uint8_t *Rq, const half_t *Rs, int rank,
                     int rank_pad, half_t *T, hipStream_t st)
{
    TArgs a{};
    a.X = X;
    a.x_scale = x_scale;
    a.R = R;
    a.Rq = R ? nullptr : Rq;
    a.Rs = Rs;
    a.k = k;
    a.rank = rank;
    a.rank_pad = rank_pad;
    a.m = m;
    a.T = T;
    return launch_t_product_args(a, xf, st);
}

// Geometry of mid_kernel: the LDS of a round of X (shared) and of a round of weights (private to the wavefronts),
// and how many rounds of each are there at a time.
template <int NT_, int RT, int RG, int KW, int XF>
struct MidLds {
    static constexpr int ROWB = XF ? 128 : 256;                 // bytes of a token's stage
    static constexpr int STAGE = NT_ * 32 * ROWB;               // bytes of a stage of X
    static constexpr int XSLOT = KW * STAGE;
    static constexpr int WBYTES = RT * 2048;                    // a wavefront's weights of a stage, or its rows of L of a unit of ranks
    static constexpr int WSLOT = kMidWaves * WBYTES;
    static constexpr int LDS = 160 * 1024;
    static constexpr int XRING = 3 * XSLOT + 4 * WSLOT <= LDS ? 3 : 2;
    static constexpr int WFIT = (LDS - XRING * XSLOT) / WSLOT;
    static constexpr int WRING = WFIT > 8 ? 8 : WFIT;
    // a round of the adapter term: UPR units of 32 ranks per wavefront of a row tile, as pieces (4 KiB per unit and 32 tokens)
    // (XRING == 2: the helpers wait for every load anyway, and rounds may have different numbers of them)
    static constexpr int UFIT = XSLOT / (KW * NT_ * 4096);
    static constexpr int UPR = XRING == 2 && UFIT > WRING - 1 ? WRING - 1 : UFIT;
    static constexpr int PARTS = (KW - 1) * RG * RT * NT_ * 4096;
    static constexpr int TROLE = (kMidWaves + kMidHelpers) * kTUnitLds;
    static constexpr int EITHER = PARTS > TROLE ? PARTS : TROLE;
    static constexpr int ROUNDS = XRING * XSLOT + WRING * WSLOT;
    static constexpr int BYTES = ROUNDS > EITHER ? ROUNDS : EITHER;
    static_assert(RG * KW == kMidWaves, "eight working wavefronts");
    static_assert(WRING >= 2 && BYTES <= LDS, "LDS of a compute unit");
};

// The Y role.  SECOND: T of the tile's tokens has been made by this workgroup.  True: a wait for the T role ran out, and
// nothing has been stored.
template <int NT_, int RT, int RG, int KW, int XF, bool AQ, bool SECOND>
__device__ __forceinline__ bool y_role(const MidArgs &a, int tid, int ot, int tt, char *lds_c, unsigned epoch)
{
    using G = MidLds<NT_, RT, RG, KW, XF>;
    constexpr int ROWB = G::ROWB, STAGE = G::STAGE, XRING = G::XRING, WRING = G::WRING;
    constexpr int TPI = 1024 / ROWB;                     // tokens per load instruction
    constexpr int PIECES = ROWB / 16;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int li = lane & 31, lb = lane >> 5;
    const int rg = wave % RG, kw = wave / RG;
    const int o0 = (ot * RG + rg) * RT * 32;             // this wavefront's rows
    const int t0 = tt * NT_ * 32;
    const uint32_t k = (uint32_t)a.k, rp = (uint32_t)a.rank_pad;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds_c;

    constexpr int UPR = G::UPR;
    const int units = mid_units<AQ>(a.rank_pad);         // of 32 ranks
    // whether the wavefronts' waits ran out, behind the partial tiles
    int *const ran_out = reinterpret_cast<int *>(lds_c + G::PARTS);
    static_assert(kMidWaves == 8 && G::PARTS + kMidWaves * 4 <= G::BYTES, "LDS behind the partial tiles");
    const bool may_help = !SECOND && a.n_t > 0 && a.rank_pad > 0;
    auto any_ran_out = [&] {
        const uint4_t lo = *reinterpret_cast<const uint4_t *>(ran_out), hi = *reinterpret_cast<const uint4_t *>(ran_out + 4);
        const uint4_t any = lo | hi;
        return __builtin_amdgcn_readfirstlane((int)(any[0] | any[1] | any[2] | any[3])) != 0;
    };
    const int rounds = (a.stages + KW - 1) / KW, t_rounds = (units + KW * UPR - 1) / (KW * UPR);
    const rsrc_t dt = make_rsrc(a.T, mid_t_bytes<AQ>(a.m, a.rank_pad));
    const uint32_t kt = k / 128;
    const uint32_t xb = XF ? 1u : 2u;
    if (wave >= kMidWaves) {
        // ---- helpers: X -> LDS ----
        // A round has KW * 32 NT / TPI load instructions, NX to a helper; instruction q moves the tokens
        // TPI (q mod IPS) .. of stage q / IPS; lane -> (token, slot piece), source piece = slot piece ^ swizzle(token).
        // Tokens past the last read as zeros; stages past the last, whose data nobody uses, repeat the last.
        constexpr int IPS = NT_ * 32 / TPI, NX = KW * IPS / kMidHelpers;
        static_assert(KW * IPS % kMidHelpers == 0 && IPS % kMidHelpers == 0, "every helper issues the same loads for every stage");
        const int hw = wave - kMidWaves;
        const rsrc_t dx = make_rsrc(a.X, (uint32_t)a.m * k * xb);
        uint32_t xv[IPS / kMidHelpers];
#pragma unroll
        for (int j = 0; j < IPS / kMidHelpers; ++j) {
            const int tok = TPI * (hw + kMidHelpers * j) + lane / PIECES;
            const uint32_t piece = (uint32_t)((lane % PIECES) ^ (XF ? (tok >> 1) & 7 : tok & 15));
            xv[j] = (uint32_t)(t0 + tok) * k * xb + piece * 16u;
        }
        // Rounds of the adapter term follow: the units of 32 ranks (u KW + kw) of this round, each 4 KiB of pieces per
        // 32 tokens.  In the launch that makes T they are read from memory, not through the L2, and may come too early:
        // the reader of a piece checks it.  Units past the last and tokens past the last tile read as zeros.
        auto load_round = [&](int round, int slot) {
            const uint32_t base = lds0 + (uint32_t)(slot * G::XSLOT + hw * 1024);
            if (round < rounds || t_rounds == 0) {
#pragma unroll
                for (int q = 0; q < KW; ++q) {
                    const int s = min(round * KW + q, a.stages - 1);
#pragma unroll
                    for (int j = 0; j < IPS / kMidHelpers; ++j)
                        load_to_lds(dx, xv[j], (uint32_t)s * ROWB, base + (uint32_t)(q * STAGE + kMidHelpers * j * 1024));
                }
            } else {
                // instruction (q, it, i): quarter hw of unit u, tokens 32 it .. 32 it + 31
#pragma unroll
                for (int q = 0; q < KW; ++q)
#pragma unroll
                    for (int i = 0; i < UPR; ++i) {
                        const int u = ((round - rounds) * UPR + i) * KW + q;
#pragma unroll
                        for (int it = 0; it < NT_; ++it) {
                            const uint32_t off = u < units ? (uint32_t)((t0 / 32 + it) * units + u) * 4096u + (uint32_t)(hw * 1024 + lane * 16) : kPastEnd;
                            const uint32_t to = base + (uint32_t)((q * UPR + i) * NT_ + it) * 4096u;
                            if (a.n_t > 0)
                                load_to_lds<true>(dt, off, 0u, to);
                            else
                                load_to_lds(dt, off, 0u, to);
                        }
                    }
            }
        };
        const int total = rounds + t_rounds;
#pragma unroll
        for (int r = 0; r < XRING - 1; ++r) load_round(r, r);
        int slot = XRING - 1;
        for (int r = 0; r < total; ++r) {
            // round r is here when at most the loads of the XRING - 2 rounds after it are in flight; past the barrier
            // every wavefront may read it, and the slot of round r - 1 is free
            asm volatile("s_waitcnt vmcnt(%0)" : : "n"((XRING - 2) * NX) : "memory");
            __builtin_amdgcn_s_barrier();
            load_round(r + XRING - 1, slot);
            slot = slot + 1 == XRING ? 0 : slot + 1;
        }
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        __syncthreads();                 // the loads past the end have landed: LDS is free
        __syncthreads();
        return may_help && any_ran_out();
    }

    float16_t acc[RT][NT_];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int it = 0; it < NT_; ++it)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][it][e] = 0.f;

    const rsrc_t dl = AQ ? make_rsrc(a.Lq, (uint32_t)q4_code_bytes(a.n, a.rank)) : make_rsrc(a.L, (uint32_t)tl_bytes(a.n, a.rank_pad));
    const rsrc_t dls = make_rsrc(AQ ? a.Ls : nullptr, AQ ? (uint32_t)q4_scale_bytes(a.n, a.rank) : 0u);
    // 4-bit L, for a round of the adapter term: codes of both steps, scale
    uint4_t lreg[UPR][RT];
    auto load_l = [&](int t_round) {
#pragma unroll
        for (int q = 0; q < UPR; ++q) {
            const int u = (t_round * UPR + q) * KW + kw;
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                {
                    const uint32_t row = (uint32_t)(o0 + 32 * i + li), u64 = (uint32_t)u / 2u;
                    const uint2_t c = load8(dl, u < units ? q4_piece(row, u64, q4_ctiles(a.rank)) + 16u * lb + 8u * (u & 1) : kPastEnd, 0);
                    const half_t sc = load_half(dls, u < units ? (row * q4_groups(a.rank) + u64 / 2u) * 2u : kPastEnd, 0);
                    lreg[q][i] = uint4_t{c[0], c[1], (uint32_t)__builtin_bit_cast(unsigned short, sc), 0u};
                }
            }
        }
    };
    float4_t rscale[RT][4];                      // of the rows 32 i + 8 blk + 4 lb + [0, 4)
    if (a.stages > 0) {
        const rsrc_t rs = make_rsrc(a.scale, (uint32_t)a.n * 4u);
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int blk = 0; blk < 4; ++blk)
                rscale[i][blk] = __builtin_bit_cast(float4_t, load16(rs, (uint32_t)(o0 + 32 * i + 8 * blk + 4 * lb) * 4u, 0));
    }
    if (AQ && t_rounds > 0) load_l(0);
    int slot = 0;                                // of the round that is due

    // This wavefront's weights, round after round, then (fp16) its rows of L, unit after unit -> its own part of LDS,
    // WRING - 1 slots ahead.  Row tiles past the last and units past the last read as zeros; every slot has the same
    // number of loads, so the count of loads in flight says which slots have arrived.
    constexpr int NW = 2 * RT;
    const rsrc_t dq = make_rsrc(a.qvals, (uint32_t)pk_qbytes(a.n, a.k));
    const rsrc_t dm = make_rsrc(a.meta, (uint32_t)pk_mbytes(a.n, a.k));
    const uint32_t w_lds = lds0 + (uint32_t)(XRING * G::XSLOT + wave * G::WBYTES);
    const int rt0 = o0 / 32;
    auto load_w = [&](int r, int at) {
        const uint32_t base = w_lds + (uint32_t)(at * G::WSLOT);
        if (r < rounds) {
            const int s = min(r * KW + kw, a.stages - 1);         // (nobody uses a stage past the last)
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                load_to_lds(dq, (uint32_t)(rt0 + i) * kt * 1024u + (uint32_t)lane * 16u, (uint32_t)s * 1024u, base + (uint32_t)i * 2048u);
                if (lane < 32) load_to_lds(dm, (uint32_t)(rt0 + i) * kt * 512u + (uint32_t)lane * 16u, (uint32_t)s * 512u, base + (uint32_t)i * 2048u + 1024u);
            }
        } else {
            const int u = (r - rounds) * KW + kw;
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    load_to_lds(dl, !AQ && u < units ? ((uint32_t)(rt0 + i) * (rp / 16) + 2u * u + j) * 1024u + (uint32_t)lane * 16u : kPastEnd, 0u,
                                base + (uint32_t)(i * 2048 + j * 1024));
        }
    };
#pragma unroll
    for (int r = 0; r < WRING - 1; ++r) load_w(r, r);
    int wslot = 0;                               // of the weights that are due
    if (a.stages > 0) {
        // B fragments: token li of tile it
        const int sw_read = XF ? (li >> 1) & 7 : li & 15;
        const uint32_t rbase = (uint32_t)(kw * STAGE + li * ROWB);
        const uint32_t rx = (uint32_t)(lb ^ sw_read) * 16u;
        for (int r = 0; r < rounds; ++r) {
            // this round's weights are here when at most the WRING - 2 rounds after it are in flight; X is, past the barrier
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"((WRING - 2) * NW) : "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" : : : "memory");
            load_w(r + WRING - 1, wslot == 0 ? WRING - 1 : wslot - 1);
            __builtin_amdgcn_sched_barrier(0);
            if (r * KW + kw < a.stages) {
                const char *const bp = lds_c + slot * G::XSLOT + rbase;
                const char *const wp = lds_c + XRING * G::XSLOT + wslot * G::WSLOT + wave * G::WBYTES;
                uint4_t q[RT];
                uint2_t mm[RT];
#pragma unroll
                for (int i = 0; i < RT; ++i) {
                    q[i] = *reinterpret_cast<const uint4_t *>(wp + i * 2048 + lane * 16);
                    mm[i] = *reinterpret_cast<const uint2_t *>(wp + i * 2048 + 1024 + lane * 8);
                }
                // the fragments of the next slice are read while the matrix instructions of this one run
                if constexpr (XF == 0) {
                    half16_t b[2][NT_];
                    auto read_b = [&](int t) {
#pragma unroll
                        for (int it = 0; it < NT_; ++it) {
                            const half8_t b1 = *reinterpret_cast<const half8_t *>(bp + (rx ^ (32u * t)) + it * 32 * ROWB);
                            const half8_t b2 = *reinterpret_cast<const half8_t *>(bp + (rx ^ (32u * t) ^ 128u) + it * 32 * ROWB);
                            b[t & 1][it] = __builtin_shufflevector(b1, b2, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
                        }
                    };
                    read_b(0);
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        if (t + 1 < 4) read_b(t + 1);
                        __builtin_amdgcn_sched_barrier(0);
                        half8_t av[RT];
#pragma unroll
                        for (int i = 0; i < RT; ++i) av[i] = codes_to_half8(q[i][t]);
#pragma unroll
                        for (int it = 0; it < NT_; ++it)
#pragma unroll
                            for (int i = 0; i < RT; ++i) {
                                if (t & 1)
                                    acc[i][it] = __builtin_amdgcn_smfmac_f32_32x32x32_f16(av[i], b[t & 1][it], acc[i][it], (int)mm[i][t >> 1], 0, 1);
                                else
                                    acc[i][it] = __builtin_amdgcn_smfmac_f32_32x32x32_f16(av[i], b[t & 1][it], acc[i][it], (int)mm[i][t >> 1], 0, 0);
                            }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else {
                    int8v_t b[2][NT_];
                    auto read_b = [&](int u) {
#pragma unroll
                        for (int it = 0; it < NT_; ++it) {
                            const uint4_t b1 = *reinterpret_cast<const uint4_t *>(bp + (rx ^ (32u * u)) + it * 32 * ROWB);
                            const uint4_t b2 = *reinterpret_cast<const uint4_t *>(bp + (rx ^ (32u * u) ^ 64u) + it * 32 * ROWB);
                            b[u][it] = int8v_t{(int)b1[0], (int)b1[1], (int)b1[2], (int)b1[3], (int)b2[0], (int)b2[1], (int)b2[2], (int)b2[3]};
                        }
                    };
                    read_b(0);
                    read_b(1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        int4_t av[RT];
#pragma unroll
                        for (int i = 0; i < RT; ++i) {
                            const uint4_t h0 = __builtin_bit_cast(uint4_t, codes_to_half8(q[i][2 * u]));
                            const uint4_t h1 = __builtin_bit_cast(uint4_t, codes_to_half8(q[i][2 * u + 1]));
                            av[i] = int4_t{(int)__builtin_amdgcn_perm(h0[1], h0[0], 0x07050301u), (int)__builtin_amdgcn_perm(h0[3], h0[2], 0x07050301u),
                                           (int)__builtin_amdgcn_perm(h1[1], h1[0], 0x07050301u), (int)__builtin_amdgcn_perm(h1[3], h1[2], 0x07050301u)};
                        }
#pragma unroll
                        for (int it = 0; it < NT_; ++it)
#pragma unroll
                            for (int i = 0; i < RT; ++i) {
                                if (XF == 1)
                                    acc[i][it] = __builtin_amdgcn_smfmac_f32_32x32x64_bf8_fp8(av[i], b[u][it], acc[i][it], (int)mm[i][u], 0, 0);
                                else
                                    acc[i][it] = __builtin_amdgcn_smfmac_f32_32x32x64_bf8_bf8(av[i], b[u][it], acc[i][it], (int)mm[i][u], 0, 0);
                            }
                    }
                }
            }
            slot = slot + 1 == XRING ? 0 : slot + 1;
            wslot = wslot + 1 == WRING ? 0 : wslot + 1;
        }
    }
    if (a.stages > 0) {
        float xs = 1.0f;
        if constexpr (XF != 0) xs = *a.x_scale;
        // element 4 blk + e of a tile is row 8 blk + 4 lb + e
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int blk = 0; blk < 4; ++blk)
#pragma unroll
                for (int it = 0; it < NT_; ++it)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i][it][4 * blk + e] *= rscale[i][blk][e] * xs;
    }
    bool gave_up = false;
    if (t_rounds > 0) {
        const int made = (a.m + 15) / 16 * 16;       // tokens of T that exist; the lanes of the others take anything
        int spins = 0;
        for (int tr = 0; tr < t_rounds; ++tr) {
            // the UPR slots of this round
            static_assert(WRING >= UPR + 1, "the ring holds a round of L");
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"((WRING - 1 - UPR) * NW) : "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" : : : "memory");
            const char *const pieces = lds_c + slot * G::XSLOT + kw * UPR * NT_ * 4096 + lane * 16;
            half8_t av[UPR][2][RT], bv[UPR][2][NT_];
#pragma unroll
            for (int q = 0; q < UPR; ++q) {
                const int u = (tr * UPR + q) * KW + kw;
                uint4_t pc[2][NT_][2];
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int it = 0; it < NT_; ++it)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            pc[s][it][j] = *reinterpret_cast<const uint4_t *>(pieces + (q * NT_ + it) * 4096 + (2 * s + j) * 1024);
                auto exists = [&](int s, int it) { return u < units && mid_rank<AQ>(u, s, lb) < rp && t0 + 32 * it + li < made; };
                // a piece that is not this call's (it came through the L2 too early) is read again from memory
                for (;;) {
                    bool there = true;
#pragma unroll
                    for (int s = 0; s < 2; ++s)
#pragma unroll
                        for (int it = 0; it < NT_; ++it)
#pragma unroll
                            for (int j = 0; j < 2; ++j) there = there && (!exists(s, it) || piece_valid(pc[s][it][j], epoch));
                    if (__all(there)) break;
                    if (++spins >= a.spin_limit) {
                        gave_up = true;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(4);
#pragma unroll
                    for (int s = 0; s < 2; ++s)
#pragma unroll
                        for (int it = 0; it < NT_; ++it)
#pragma unroll
                            for (int j = 0; j < 2; ++j)
                                pc[s][it][j] = load_piece(dt, exists(s, it) ? mid_t_piece<AQ>((uint32_t)(t0 + 32 * it + li), mid_rank<AQ>(u, s, lb) + 4u * j, a.rank_pad) : kPastEnd);
                }
#pragma unroll
                for (int s = 0; s < 2; ++s) {
#pragma unroll
                    for (int it = 0; it < NT_; ++it) {
                        uint4_t v = {pc[s][it][0][1], pc[s][it][0][2], pc[s][it][1][1], pc[s][it][1][2]};
                        if (AQ && mid_rank<AQ>(u, s, lb) >= rp) v = uint4_t{0u, 0u, 0u, 0u};
                        if (gave_up) v = uint4_t{0x7E007E00u, 0x7E007E00u, 0x7E007E00u, 0x7E007E00u};    // NaN: must not pass for a result
                        bv[q][s][it] = __builtin_bit_cast(half8_t, v);
                    }
#pragma unroll
                    for (int i = 0; i < RT; ++i) {
                        if constexpr (AQ)
                            av[q][s][i] = codes_to_half8(lreg[q][i][s]) * __builtin_bit_cast(half_t, (unsigned short)lreg[q][i][2]);
                        else
                            av[q][s][i] = *reinterpret_cast<const half8_t *>(lds_c + XRING * G::XSLOT + wslot * G::WSLOT + wave * G::WBYTES +
                                                                             i * 2048 + s * 1024 + lane * 16);
                    }
                }
                wslot = wslot + 1 == WRING ? 0 : wslot + 1;
            }
            if (AQ) load_l(tr + 1);
            asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");       // L has been read
#pragma unroll
            for (int q = 0; q < UPR; ++q) {
                const int ahead = wslot + q + WRING - 1 - UPR;
                load_w(rounds + tr * UPR + q + WRING - 1, ahead >= WRING ? ahead - WRING : ahead);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < UPR; ++q)
                if ((tr * UPR + q) * KW + kw < units) {
#pragma unroll
                    for (int s = 0; s < 2; ++s)
#pragma unroll
                        for (int i = 0; i < RT; ++i)
#pragma unroll
                            for (int it = 0; it < NT_; ++it)
                                acc[i][it] = __builtin_amdgcn_mfma_f32_32x32x16_f16(av[q][s][i], bv[q][s][it], acc[i][it], 0, 0, 0);
                }
            slot = slot + 1 == XRING ? 0 : slot + 1;
        }
        if (gave_up && !may_help && lane == 0) __hip_atomic_store(a.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }

    // the KW partial tiles meet in LDS
    float4_t *const red = reinterpret_cast<float4_t *>(lds_c);
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");     // the loads past the end have landed
    __syncthreads();                         // and X has been read
    if (may_help && lane == 0) ran_out[wave] = gave_up;
    if (kw > 0) {
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int it = 0; it < NT_; ++it)
#pragma unroll
                for (int blk = 0; blk < 4; ++blk)
                    red[((((kw - 1) * RG + rg) * RT + i) * NT_ + it) * 256 + blk * 64 + lane] =
                        float4_t{acc[i][it][4 * blk], acc[i][it][4 * blk + 1], acc[i][it][4 * blk + 2], acc[i][it][4 * blk + 3]};
    }
    __syncthreads();
    if (may_help && any_ran_out()) return true;
    if (kw > 0) return false;
    // store: lane holds token t0 + 32 it + li, rows 8 blk + 4 lb .. + 3 of tile i
    const bool vec_ok = (a.n & 3) == 0;
#pragma unroll
    for (int it = 0; it < NT_; ++it) {
        const int t = t0 + 32 * it + li;
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int blk = 0; blk < 4; ++blk) {
                float4_t v = {acc[i][it][4 * blk], acc[i][it][4 * blk + 1], acc[i][it][4 * blk + 2], acc[i][it][4 * blk + 3]};
#pragma unroll
                for (int w = 0; w < KW - 1; ++w) v += red[(((w * RG + rg) * RT + i) * NT_ + it) * 256 + blk * 64 + lane];
                const int o = o0 + 32 * i + 8 * blk + 4 * lb;
                if (t >= a.m || o >= a.n) continue;
                half_t *y = a.Y + (size_t)t * a.n + o;
                if (vec_ok) {
                    if (a.accumulate) {
                        const half4_t old = *reinterpret_cast<const half4_t *>(y);
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += (float)old[e];
                    }
                    *reinterpret_cast<half4_t *>(y) = half4_t{(half_t)v[0], (half_t)v[1], (half_t)v[2], (half_t)v[3]};
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (o + e < a.n) y[e] = (half_t)(a.accumulate ? v[e] + (float)y[e] : v[e]);
                }
            }
    }
    return false;
}

// Tiles j, j + step, ... of T, and all of those along `count` token tiles from `first` on.
template <int XF, bool AQ, int TT, bool HIDE>
__device__ __forceinline__ void t_tiles(const MidArgs &a, int j, int step, char *lds_c, unsigned epoch)
{
    for (; j < a.t_tiles; j += step) {
        int rt, tr;
        if (tile_on_die(j, a.rank_pad / 16, rt, tr)) t_tile<XF, AQ, TT, HIDE>(a, rt, tr, lds_c, epoch);
    }
}
template <int XF, bool AQ, int TT, bool HIDE>
__device__ __forceinline__ void t_of_tokens(const MidArgs &a, int first, int count, char *lds_c, unsigned epoch)
{
    for (int j = 0; j < a.rank_pad / 16 * count; ++j) {
        const int tr = first + j % count;
        if (16 * TT * tr < a.m) t_tile<XF, AQ, TT, HIDE>(a, j / count, tr, lds_c, epoch);
    }
}

// TT: a tile of T is of 16 TT tokens.
template <int NT_, int RT, int RG, int KW, int XF, bool AQ, int TT>
__global__ __launch_bounds__(kMidThreads, 3) void mid_kernel(MidArgs a)
{
    extern __shared__ __attribute__((aligned(16))) char lds_c[];
    // with tiles of T of 16 tokens: beside tiles of 32 and 64 rows 1 to 2 % faster, with 8-bit X and 4-bit adapters up to 8 %, but 5 % slower beside 64 rows with fp16 X and
    // 4-bit adapters, and beside larger tiles 1 to 5 % slower
    constexpr bool HIDE = TT == 2 || RG == 1 || (RT == 1 && RG == 2 && (XF != 0 || !AQ));
    const unsigned epoch = a.rank_pad > 0 && a.T ? call_epoch(a.epoch) : 0u;
    if ((int)blockIdx.x < a.n_t) {
        t_tiles<XF, AQ, TT, HIDE>(a, blockIdx.x, a.n_t, lds_c, epoch);
        return;
    }
    int ot, tt;
    if (!tile_on_die((int)blockIdx.x - a.n_t, a.tiles_o, ot, tt)) return;
    if (!y_role<NT_, RT, RG, KW, XF, AQ, false>(a, threadIdx.x, ot, tt, lds_c, epoch)) return;
    t_of_tokens<XF, AQ, TT, HIDE>(a, 2 / TT * NT_ * tt, 2 / TT * NT_, lds_c, epoch);
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");     // the pieces are in memory
    __syncthreads();
    // (a thread number the compiler knows nothing of: what it works out of it above would stay in registers until here)
    unsigned tid = threadIdx.x;
    asm volatile("" : "+v"(tid), "+s"(ot), "+s"(tt));
    y_role<NT_, RT, RG, KW, XF, AQ, true>(a, (int)tid, ot, tt, lds_c, epoch);
}

// The T role of mid_kernel in a launch of its own.
template <int XF, bool AQ>
static void launch_t_role_of(const TArgs &t, hipStream_t st)
{
    MidArgs a{};
    a.X = t.X;
    a.x_scale = t.x_scale;
    a.R = t.R;
    a.Rq = t.Rq;
    a.Rs = t.Rs;
    a.T = t.pieces;
    a.T_rows = t.T;
    a.epoch = t.epoch;
    a.k = t.k;
    a.rank = t.rank;
    a.rank_pad = t.rank_pad;
    a.m = t.m;
    a.n_t = a.t_tiles = die_tiles(t.rank_pad / 16, (t.m + 15) / 16);
    constexpr size_t lds = MidLds<1, 1, 1, 8, XF>::TROLE;
    hipLaunchKernelGGL((mid_kernel<1, 1, 1, 8, XF, AQ, 1>), dim3((unsigned)a.n_t), dim3(kMidThreads), lds, st, a);
}
static void launch_t_role(const TArgs &t, int xf, hipStream_t st)
{
    if (t.Rq) {
        if (xf == 0)
            launch_t_role_of<0, true>(t, st);
        else if (xf == 1)
            launch_t_role_of<1, true>(t, st);
        else
            launch_t_role_of<2, true>(t, st);
    } else {
        if (xf == 0)
            launch_t_role_of<0, false>(t, st);
        else if (xf == 1)
            launch_t_role_of<1, false>(t, st);
        else
            launch_t_role_of<2, false>(t, st);
    }
}

// Tests of the wait (slim_decode_override): nobody makes T, which ends in NaN, or the Y role has to make it.
enum class WaitTest { none, fail, help };

// How many tiles of T (of `tokens` tokens) each workgroup of the T role has to make beside n_y workgroups of the Y role, one per compute
// unit; n_t: those workgroups.  None are free: more than any rule takes.
static int t_trips(int rank_pad, int m, int tokens, int n_y, int cus, int *n_t = nullptr)
{
    const int spare = (cus - n_y) / kDies * kDies, tiles = die_tiles(rank_pad / 16, (m + tokens - 1) / tokens);
    const int n = tiles < spare ? tiles : spare;
    if (n_t) *n_t = n > 0 ? n : 0;
    return n > 0 ? (tiles + n - 1) / n : 1 << 20;
}

template <int NT_, int RT, int RG, int KW, int XF, bool AQ, int TT>
static int launch_mid_tiles(MidArgs a, int t_tokens, WaitTest wait_test, hipStream_t st)
{
    constexpr size_t lds = MidLds<NT_, RT, RG, KW, XF>::BYTES;
    a.tiles_o = (a.n + 32 * RT * RG - 1) / (32 * RT * RG);
    const int n_y = die_tiles(a.tiles_o, (a.m + 32 * NT_ - 1) / (32 * NT_));
    int n_t = 0;
    if (t_tokens > 0) t_trips(a.rank_pad, a.m, t_tokens, n_y, device_info().cus, &n_t);
    a.t_tiles = die_tiles(a.rank_pad / 16, (a.m + 16 * TT - 1) / (16 * TT));
    if (wait_test == WaitTest::fail) {
        n_t = 0;                             // nobody makes T
    } else if (wait_test == WaitTest::help && n_t > 0) {
        a.t_tiles = 0;                       // the T role makes nothing
    } else if (a.t_tiles > 0 && n_t == 0) {
        TArgs t{};
        t.X = a.X;
        t.x_scale = a.x_scale;
        t.R = AQ ? nullptr : a.R;
        t.Rq = AQ ? a.Rq : nullptr;
        t.Rs = a.Rs;
        t.k = a.k;
        t.rank = a.rank;
        t.rank_pad = a.rank_pad;
        t.m = a.m;
        t.pieces = a.T;
        t.q4_order = AQ;
        t.epoch = a.epoch;
        const int rc = launch_t_product_args(t, XF, st);
        if (rc != SLIM_OK) return rc;
    }
    a.n_t = n_t;
    hipLaunchKernelGGL((mid_kernel<NT_, RT, RG, KW, XF, AQ, TT>), dim3((unsigned)(n_t + n_y)), dim3(kMidThreads), lds, st, a);
    return hip_status(hipGetLastError());
}

// A kernel for each of the two tiles of T: one with both had twice the scalar registers to spill (<1, 1, 2, 4, 0, true> 43 instead of 23).
template <int NT_, int RT, int RG, int KW, int XF, bool AQ>
static int launch_mid(const MidArgs &a, int t_tokens, WaitTest wait_test, hipStream_t st)
{
    return t_tokens == 32 ? launch_mid_tiles<NT_, RT, RG, KW, XF, AQ, 2>(a, t_tokens, wait_test, st)
                          : launch_mid_tiles<NT_, RT, RG, KW, XF, AQ, 1>(a, t_tokens, wait_test, st);
}

// The geometries, by growing tile: rows x tokens.
constexpr int kMidTiles[4][2] = {{32, 32}, {64, 32}, {128, 32}, {128, 64}};

// Which geometry, by the sizes alone (index into kMidTiles), or -1: the tiles of slim_gemm_sparse.hip (or, for the
// adapter term alone, the dense product); and the tokens of a tile of T in the same launch, or 0: T gets a launch of its own.
struct MidPlan {
    int geometry, t_tokens;
};
// The smallest tile that gives every compute unit at most one workgroup and leaves room to make T in the same launch: a second workgroup
// on a unit doubles the time of a call that is a chain of latencies, a smaller tile shortens the chain.  4096 x 4096, r = 409: 64 tokens
// 14.6 / 10.4 / 13.7 / 20.5 us (256 / 128 / 64 / 32 workgroups, in the order of kMidTiles; the 512 x 128 tiles 29), 128 tokens 23.2 / 16.8 /
// 14.5 / 20.4 (31), 512 tokens 76 / 46 / 37 / 31 (36).  Where no tile fits, the large ones win: 11008 x 4096 at 256
// tokens 36.6 against 49.7.
// T is best made in one tile per workgroup.  Where tiles of 16 tokens are more than that, those of 32 tokens come next (which read R
// half as often, and each take longer), then two tiles, then three, and then a launch of T's own (us: 7452 x 2432 at 31 tokens, two tiles 10.1, one
// of 32 tokens 8.6, one of 16 beside the next tile of Y 8.2; 2244 x 3968 at 343 tokens T by itself 25.8, one of 32 tokens 17.6).
//   few: where few workgroups have a second tile of 16 tokens, at most a quarter, and the ranks are many, most of the ranks' work on Y is done while
// those are made: 288 ranks and more beside tiles of 64 rows and more (16 against 32 tokens: 12572 x 3072, rank 499, at 20 tokens 10.3 against 11.8, 2610 x 3200, 261, at
// 74 10.2 / 11.2, 4399 x 4352, 435, at 56 11.7 / 12.5; the adapter term alone 9600 x 9728, 960, at 27 19.5 / 21.4; up to 256 ranks the other way round: 2304 x 8064,
// 230, at 100 15.5 / 14.1, 2560 x 2432, 243, at 106 9.6 / 8.6; and so with a second tile on 0.29 of them: 3031 x 6656, 303, at 96 15.4 / 13.9).
//   4-bit adapters on long sums, beside tiles of 128 x 32: a tile of 32 tokens converts the codes half as often, but waits for memory twice as often as one
// of 16, and two of those are as fast or faster from 2048 inputs on (2048 x 9856, 8-bit X, at 205 tokens 22.6 / 25.6, 4951 x 7296 at 90 22.3 / 24.8, with fp16 X 1 to 3 %; up to 1024 inputs 32 tokens are 3 to 10 % faster).
//   A larger tile of Y that leaves room for one tile of T per workgroup instead of two: worth it from the smallest to the next; from 64 rows to 128
// but for 8-bit X with fp16 R (4096 x 7168 at 86 tokens 18.8 against 20.5, 2304 x 3328 at 153 11.4 / 13.0; with 8-bit X 3840 x 5120 at 86 15.1 / 11.6); from 128 x 32 to 128 x 64 on short sums only (9600 x 896 at 69 tokens 8.3 / 9.5, 3596 x 1152 at 209 9.1 / 10.1; 13184 x 6400, 8-bit X, at 33 27.9 / 19.6,
// 7101 x 6016 at 86 29.0 / 22.5).
// Against two tiles of 16 tokens at most or else the next tile of Y, over drawn layers of 512 to 28672 rows and 512 to 11008 inputs at 17 to 512 tokens: a
// fifth of the calls differ, of 300 of those one is slower by more than 2 % (2.2 %) and the mean is 12 % faster, up to 1.5 times.
// The adapter term alone has nothing to hide a chain of T behind: 4096 x 4096 at 128 tokens 15.7 / 12.5 / 15.2 / 20.1
// against 14.1 of the dense product (12.7 to 12.8 with T in the same launch, in tiles of 32 tokens), 28672 x 4096 at 48 tokens 20.2 at best against 13.6.
// Above 512 tokens the workspace has no room for the pieces of T.
MidPlan mid_plan(int n, int k, int rank_pad, int m, int cus, bool weight_term, bool q4, bool fp8)
{
    constexpr MidPlan none{-1, 0};
    if (m > 512) return none;
    auto workgroups = [&](int g) { return die_tiles((n + kMidTiles[g][0] - 1) / kMidTiles[g][0], (m + kMidTiles[g][1] - 1) / kMidTiles[g][1]); };
    MidPlan first = none, more = none;           // the first tile that fits, the first with room for more than one tile of T
    for (int g = 0; g < 4; ++g) {
        const int n_y = workgroups(g);
        if (n_y > cus) continue;
        if (rank_pad == 0) return {g, 0};
        int n16 = 0;
        const int t16 = t_trips(rank_pad, m, 16, n_y, cus, &n16), t32 = t_trips(rank_pad, m, 32, n_y, cus);
        const bool few = t16 == 2 && g > 0 && rank_pad > 256 && die_tiles(rank_pad / 16, (m + 15) / 16) - n16 <= n16 / 4;
        if (!weight_term) {
            if (g == 3 || n >= 16384) {
                if (t16 <= 1) return {g, 16};
                continue;
            }
            if (t16 <= 1 || t16 > 2) return {g, t16 <= 1 ? 16 : 0};
            if (g == 0 && t_trips(rank_pad, m, 16, workgroups(1), cus) <= 1) return {1, 16};
            return {g, t32 <= 1 && !few ? 32 : 16};
        }
        if (first.geometry < 0) first = {g, 0};
        if (t16 <= 1 || t32 <= 1) {
            const bool next = more.geometry == 0 || (more.t_tokens == 32 && (more.geometry == 1 ? q4 || !fp8 : k < 1280));
            if (more.geometry >= 0 && !(next && g == more.geometry + 1)) return more;
            const bool long_codes = t16 == 2 && g == 2 && q4 && k > 2048;
            return {g, t16 <= 1 || few || long_codes ? 16 : 32};
        }
        if (more.geometry < 0 && (t16 <= 3 || t32 <= 2)) more = {g, t16 <= 2 || t32 > 2 ? 16 : 32};
    }
    return more.geometry >= 0 ? more : first;
}

template <int XF, bool AQ>
static int launch_mid_call(const MidArgs &a, MidPlan plan, WaitTest wait_test, hipStream_t st)
{
    switch (plan.geometry) {
        case 0: return launch_mid<1, 1, 1, 8, XF, AQ>(a, plan.t_tokens, wait_test, st);
        case 1: return launch_mid<1, 1, 2, 4, XF, AQ>(a, plan.t_tokens, wait_test, st);
        case 2: return launch_mid<1, 2, 2, 4, XF, AQ>(a, plan.t_tokens, wait_test, st);
        default: return launch_mid<2, 1, 4, 2, XF, AQ>(a, plan.t_tokens, wait_test, st);
    }
}

// The whole call (T and Y) if the sizes are this path's: *taken says so.  weight_term false: the adapter term alone
// (slim_lowrank).  T: t_room bytes of the workspace, ctrl: its control words.
int launch_gemm_mid(const slim_layer *layer, const half_t *X, int xf, const float *x_scale, int m, half_t *Y, void *T, size_t t_room,
                    unsigned *ctrl, bool weight_term, int accumulate, hipStream_t st, bool *taken)
{
    *taken = false;
    const slim_shape s = layer->shape;
    const bool q4 = layer->adapter_bits == 4 && s.rank > 0;
    const MidPlan plan = mid_plan(s.n, s.k, layer->rank_pad, m, device_info().cus, weight_term, q4, xf != 0);
    if (plan.geometry < 0) return SLIM_OK;
    // 32-bit offsets, tiles past the end included; room for the pieces of T
    constexpr uint64_t kLimit = 0x80000000ull;
    const uint64_t t_bytes = q4 ? mid_t_bytes<true>(m, layer->rank_pad) : mid_t_bytes<false>(m, layer->rank_pad);
    if ((uint64_t)(m + 64) * s.k * 2 >= kLimit || (uint64_t)pk_qbytes(s.n + 128, s.k) >= kLimit ||
        (uint64_t)tl_bytes(s.n + 128, layer->rank_pad) >= kLimit || (uint64_t)tl_bytes(layer->rank_pad, s.k) >= kLimit || t_bytes > t_room)
        return SLIM_OK;
    *taken = true;
    MidArgs a{};
    a.qvals = layer->qvals;
    a.meta = layer->meta;
    a.scale = layer->scale;
    a.X = X;
    a.x_scale = x_scale;
    a.R = reinterpret_cast<const half_t *>(layer->R);
    a.L = reinterpret_cast<const half_t *>(layer->L);
    a.Rq = layer->Rq;
    a.Lq = layer->Lq;
    a.Rs = reinterpret_cast<const half_t *>(layer->Rs);
    a.Ls = reinterpret_cast<const half_t *>(layer->Ls);
    a.T = static_cast<uint4_t *>(T);
    a.err = ctrl + 2;                        // read by slim_workspace_check
    const WaitTest wait_test = decode_path_override() != 3 || layer->rank_pad == 0 ? WaitTest::none : decode_lds_limit() == 0 ? WaitTest::fail : WaitTest::help;
    if (layer->rank_pad > 0) a.epoch = next_call_epoch(ctrl + 3, st);
    // (a poll takes half a microsecond or more; T is there after a few where the T role runs)
    a.spin_limit = wait_test != WaitTest::none ? 256 : 2048;
    a.Y = Y;
    a.n = s.n;
    a.k = s.k;
    a.rank = s.rank;
    a.rank_pad = layer->rank_pad;
    a.m = m;
    a.stages = weight_term ? s.k / 128 : 0;
    a.accumulate = accumulate;
    if (q4) {
        if (xf == 0) return launch_mid_call<0, true>(a, plan, wait_test, st);
        return xf == 1 ? launch_mid_call<1, true>(a, plan, wait_test, st) : launch_mid_call<2, true>(a, plan, wait_test, st);
    }
    if (xf == 0) return launch_mid_call<0, false>(a, plan, wait_test, st);
    return xf == 1 ? launch_mid_call<1, false>(a, plan, wait_test, st) : launch_mid_call<2, false>(a, plan, wait_test, st);
}

}  // namespace slim
