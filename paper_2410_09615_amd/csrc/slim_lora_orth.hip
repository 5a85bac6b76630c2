// out = orth(in) for a block in [rows][l] of fp32 columns, l <= 1024: Cholesky QR, the orthonormalisation of the
// subspace iteration in slim_lora.hip.
//
//   G = in^T in = Lc Lc^T,  out = in Lc^-T     (columns in order: in = out Lc^T with a positive diagonal)
//
// The call is a chain (products, 16-column steps of the factorisation, products), so what bounds it is the
// number of launches (4 us each) and the latency of the diagonal blocks, not arithmetic:
//   lora_factor_kernel  lower tiles of G, the rows divided among workgroups; then the factorisation: a workgroup that factors and
//                       inverts the diagonal tiles, in blocks of 16 that live in the registers of a wavefront, and workgroups for the
//                       other tiles, in strips of 16 rows, which hand what they make to one another through memory;
//   lora_apply_kernel   a workgroup carries 16 rows of `in` through all block columns, which stay in LDS:
//                       out_J = (in_J - sum_{K<J} out_K L_JK^T) X_JJ^T, one launch for the whole block.
// 4096 x 416: 90 us (G 15, the diagonal tiles 7.3 each, apply 20).  With G in a launch of its own and a workgroup per tile that hands it on
// with release and acquire 141 (22, 12.1, 25), with one launch per 64 columns 200, and with separate panel, trailing and column
// products and a 64-step one-workgroup diagonal 700.
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
// where every other one was 19 (80 us more for each than for one that is only scaled).
#include <utility>

#include "slim_internal.h"

namespace slim {

typedef float float16v_t __attribute__((ext_vector_type(16)));

constexpr int kOb = 64;                        // block of columns
constexpr int kTileFloats = kOb * kOb;
constexpr float kSpread = 1e4f;                // largest / smallest pivot up to which more than one product may follow
constexpr int kMaxRun = 8;                     // products between two blocks that are orthonormalised, at most
constexpr int kLastRun = 4;                    // before the last of them, at most
constexpr int kSeparated = 7;                  // products before more than two in a row
constexpr int kDies = 8;
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

// What lane i % 16 of the G-th sixteen lanes holds, to lane i of all four: four registers side by side, in asm because a swap has to
// come two wait states after what it moves, which the other registers' instructions are (an s_nop is 9 cycles, an instruction 5).
template <int G>
__device__ __forceinline__ void from_group(const float4_t &w, float (&out)[4])
{
    float t[4];
    asm volatile("v_mov_b32 %0, %8\n\tv_mov_b32 %4, %8\n\tv_mov_b32 %1, %9\n\tv_mov_b32 %5, %9\n\t"
                 "v_mov_b32 %2, %10\n\tv_mov_b32 %6, %10\n\tv_mov_b32 %3, %11\n\tv_mov_b32 %7, %11\n\t"
                 "v_permlane16_swap_b32 %0, %4\n\tv_permlane16_swap_b32 %1, %5\n\ts_nop 0\n\t"
                 "v_permlane16_swap_b32 %2, %6\n\tv_permlane16_swap_b32 %3, %7"          // groups 0, 0, 2, 2 and 1, 1, 3, 3
                 : "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3]), "=&v"(out[0]), "=&v"(out[1]), "=&v"(out[2]), "=&v"(out[3])
                 : "v"(w[0]), "v"(w[1]), "v"(w[2]), "v"(w[3]));
#define SLIM_MOVES(to, from) "v_mov_b32 %" #to ", %" #from "\n\t"
    if constexpr (G & 1)
        asm volatile("s_nop 1\n\t" SLIM_MOVES(0, 4) SLIM_MOVES(1, 5) SLIM_MOVES(2, 6) SLIM_MOVES(3, 7)
                     "v_permlane32_swap_b32 %0, %4\n\tv_permlane32_swap_b32 %1, %5\n\ts_nop 0\n\tv_permlane32_swap_b32 %2, %6\n\tv_permlane32_swap_b32 %3, %7\n\ts_nop 1"
                     : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(out[0]), "+v"(out[1]), "+v"(out[2]), "+v"(out[3]));
    else
        asm volatile("s_nop 1\n\t" SLIM_MOVES(4, 0) SLIM_MOVES(5, 1) SLIM_MOVES(6, 2) SLIM_MOVES(7, 3)
                     "v_permlane32_swap_b32 %0, %4\n\tv_permlane32_swap_b32 %1, %5\n\ts_nop 0\n\tv_permlane32_swap_b32 %2, %6\n\tv_permlane32_swap_b32 %3, %7\n\ts_nop 1"
                     : "+v"(t[0]), "+v"(t[1]), "+v"(t[2]), "+v"(t[3]), "+v"(out[0]), "+v"(out[1]), "+v"(out[2]), "+v"(out[3]));
#undef SLIM_MOVES
    if constexpr (G < 2)                         // (lower halves in both of t, upper in both of out)
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = t[e];
}

// Step C of factor16(): w[f] += m times w[f] of lane C of the sixteen, m = col above / d, for the registers of w and for those of c4
// that are still ahead (FIRST on); then the pivot of the next step, d = c4[FIRST] of its lane or the floor, and its reciprocal q, behind
// which the last of w hide.  The broadcast rides on the multiply-add.  Outside the compiler's hazard bookkeeping: two wait states between a
// write and a read by another lane, one behind a reciprocal.  The four instructions of m come first in the same asm, so that a register the
// compiler writes or copies right before it is not read by another lane too early (an s_nop would be 9 cycles, an instruction is 5).
template <int C, int FIRST>
__device__ __forceinline__ void factor_step(float4_t &w, float (&c4)[4], float col, float above, float floor_, float &d, float &q)
{
    float m, t;
#define SLIM_M "v_mul_f32 %10, %12, %13\n\tv_fma_f32 %11, -%8, %9, 2.0\n\tv_mul_f32 %11, %9, %11\n\tv_mul_f32 %10, %11, %10\n\t"      // (q to rounding)
#define SLIM_ROW(x) "v_fmac_f32_dpp " x ", " x ", %10 row_newbcast:%15 row_mask:0xf bank_mask:0xf\n\t"
#define SLIM_NEXT(x) "v_max_f32_dpp %8, " x ", %14 row_newbcast:%16 row_mask:0xf bank_mask:0xf\n\tv_rcp_f32 %9, %8\n\t"
#define SLIM_REGS "+v"(w[0]), "+v"(w[1]), "+v"(w[2]), "+v"(w[3]), "+v"(c4[0]), "+v"(c4[1]), "+v"(c4[2]), "+v"(c4[3]), "+v"(d), "+v"(q), \
                  "=&v"(m), "=&v"(t) : "v"(col), "v"(above), "v"(floor_), "n"(C), "n"((C + 1) % 16)
    if constexpr (FIRST == 1)
        asm volatile(SLIM_M SLIM_ROW("%5") SLIM_ROW("%6") SLIM_ROW("%7") SLIM_NEXT("%5") SLIM_ROW("%1") SLIM_ROW("%2") SLIM_ROW("%3") SLIM_ROW("%0") : SLIM_REGS);
    else if constexpr (FIRST == 2)
        asm volatile(SLIM_M SLIM_ROW("%6") SLIM_ROW("%7") SLIM_ROW("%2") SLIM_NEXT("%6") SLIM_ROW("%3") SLIM_ROW("%0") SLIM_ROW("%1") : SLIM_REGS);
    else if constexpr (FIRST == 3)
        asm volatile(SLIM_M SLIM_ROW("%7") SLIM_ROW("%3") SLIM_ROW("%0") SLIM_NEXT("%7") SLIM_ROW("%1") SLIM_ROW("%2") : SLIM_REGS);
    else
        asm volatile(SLIM_M SLIM_ROW("%0") SLIM_ROW("%1") SLIM_ROW("%2") SLIM_ROW("%3") : SLIM_REGS);
#undef SLIM_M
#undef SLIM_ROW
#undef SLIM_NEXT
#undef SLIM_REGS
}

// 16 x 16: lane i of group g (sixteen lanes) holds row i, columns 4 g .. 4 g + 3, of the symmetric block a = Lc Lc^T; on
// return those of Lc^-1.  The steps run on a = M diag(d) M^T, M with a unit diagonal, whose chain has a reciprocal and no square
// root, and the rows of M^-1 are scaled by 1 / sqrt(d) at the end.  Step c adds m_i = -a_ic / d_c times row c to the rows i
// below it: to the columns of a after c, to those of M^-1 before it, and column c becomes that of M^-1, so that one register
// holds a column of the one and then of the other.  Every group works on a copy of the four columns in turn, so that what the
// steps wait for is the pivot's broadcast, its reciprocal and one multiply-add, in registers; no LDS, no barriers.
// A lone wavefront issues an instruction in 5 cycles whether or not it waits for the one before, so instructions are what counts, and
// those that select by a comparison count threefold (the mask has to be waited for): rows and pivots that take no part are
// multiplied by zero instead.  0.9 us a block; with each column fetched from its group by itself, moves for the broadcasts and selections
// 1.15.
// pmax, pmin: the largest and the smallest pivot of this lane's rows so far, but for those of `dead`.  Returns whether this row's
// pivot is above the floor (2^-120 or more).
__device__ __forceinline__ bool factor16(float4_t &w, int i, int g, float floor_, float dead, float &pmax, float &pmin)
{
    float d_i = 1.0f;                            // this row's pivot
    for_each<4>([&](auto pc) {
        constexpr int p = pc;
        float c4[4];
        from_group<p>(w, c4);
        float d = fmaxf(row_lane<4 * p>(c4[0]), floor_), q = __builtin_amdgcn_rcpf(d);
        for_each<4>([&](auto ec) {
            constexpr int e = ec, c = 4 * p + e;
            const float below = i > c ? -1.0f : 0.f;
            // (d at the floor: a column in the span of the ones before it, nothing to subtract)
            const float above = __builtin_amdgcn_fmed3f((d - floor_) * 0x1p127f, 0.f, 1.f);
            const float col = c4[e] * below;
            w[e] = g == p ? (i == c ? 1.0f : 0.f) : w[e];
            factor_step<c, e + 1>(w, c4, col, above, floor_, d, q);
        });
        const float mine = (i & 2) ? ((i & 1) ? c4[3] : c4[2]) : ((i & 1) ? c4[1] : c4[0]);
        d_i = i / 4 == p ? mine : d_i;           // (a pivot stays where it was used)
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

// ---- G = Y^T Y = Lc Lc^T in one launch ----
// Three kinds of workgroups, in the order of their index:
//   gram units   a tile of 64 x 64 of G over a range of rows each; they wait for nothing;
//   the chain    one workgroup, which factors and inverts the diagonal tiles one after the other;
//   strips       16 rows of a tile below the diagonal (or of a diagonal tile, for the chain) each.
// What bounds the launch is the chain: 64 columns at a time, each of which needs what the one before it left.  So the chain's
// workgroup does nothing but what the next 16 columns wait for, and everything else is done beside it: by its other wavefronts
// while one factors 16 columns, and by the strips.
// What one workgroup makes for others goes through memory: stored past the L2 (device scope), waited for, and then named by words
// that hold the number of the orth(), which the readers poll.  They read it past their L2 as well, so there are no fences (write-back and
// invalidation of an L2 are over a microsecond each).
// A gram unit waits for nothing, a strip for strips of a lower index and for diagonal tiles, and a diagonal tile of column j for strips that come
// before all strips that wait for it: with workgroups started in the order of their index, room for the chain and one strip is enough.
// A workgroup that made several strips, one after the other, would wait with its second for strips of a higher index, whose workgroups may not have
// room to start.  A wait is bounded all the same; should something not come, lora_apply_kernel makes the block NaN.
constexpr int kGramUnits = 640;                // partial tiles, at most
constexpr int kGramRun = 256;                  // rows added up by themselves
struct FactorArgs {
    const float *Y;
    int rows, l, nb, tiles;
    int splits, zrows;                         // ranges of rows, rows in each
    float *ws;                                 // orth_floats() (offsets: FactorPlaces)
    unsigned *hand;
    unsigned seq;
    int polls;
    OrthStep step;
};
// Byte offsets in the workspace of an orth(): partial tiles, their diagonals, tiles (of the lower triangle) on their way to the chain, tiles
// of the factor, inverses of the diagonal tiles.
struct FactorPlaces {
    uint32_t P, diag, G, Lf, D, end;
    __host__ __device__ explicit FactorPlaces(int nb)
    {
        const uint32_t t = (uint32_t)tri(nb, 0), b = kTileFloats * 4;
        P = 0;
        diag = kGramUnits * b;
        G = diag + kGramUnits * kOb * 4;
        Lf = G + t * b;
        D = Lf + t * b;
        end = D + (uint32_t)nb * b;
    }
};
// The words: one per gram unit; then four per strip (one of each wavefront), those of the strips of a tile together: of a tile of the factor
// (at tri(I, J)), of a diagonal tile and of the one to its left before the last columns are subtracted, and four of the inverse of a
// diagonal tile; last the number of an orth() in which a wait ran out.
enum { kHandGram = 0, kHandL = kGramUnits, kHandT = kHandL + 16 * kMaxTri, kHandA = kHandT + 16 * kMaxBlocks, kHandD = kHandA + 16 * kMaxBlocks,
       kHandFailed = kHandD + 16 * kMaxBlocks, kHandWords = kHandFailed + 16 };
constexpr int kHandPolls = 1 << 24;            // half a microsecond or more each; a wait is over after some tens of them, or when other
                                               // work on the chip has let the rest of the launch start
constexpr int kDevice = 16;                    // cache policy of a buffer access: device scope (written through / read from memory)

__device__ __forceinline__ float4_t load_dev(rsrc_t r, uint32_t off)
{
    return __builtin_bit_cast(float4_t, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, kDevice));
}
__device__ __forceinline__ void store_dev(rsrc_t r, uint32_t off, float4_t v)
{
    typedef unsigned int store4_t __attribute__((__vector_size__(16)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(store4_t, v), r, (int)off, 0, kDevice);
}
// What this wavefront has stored is in memory -> its word, or words.
template <int N = 1>
__device__ __forceinline__ void hand_over(const FactorArgs &a, int word, int lane)
{
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    if (lane < N) __hip_atomic_store(a.hand + word + lane, a.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// A wavefront's waits: each lane for four words from `word` on (a multiple of 4; or for none, with a negative number).  `lost`: a
// wait has run out, and those after it are none.
__device__ __forceinline__ bool words_there(const FactorArgs &a, rsrc_t hand, int word)
{
    const uint4_t v = __builtin_bit_cast(uint4_t, __builtin_amdgcn_raw_buffer_load_b128(hand, word < 0 ? 0 : 4 * word, 0, kDevice));
    return __all(word < 0 || (v[0] == a.seq && v[1] == a.seq && v[2] == a.seq && v[3] == a.seq));
}
__device__ __forceinline__ void wait_words(const FactorArgs &a, rsrc_t hand, int word, bool &lost)
{
    for (int polls = 0; !lost; ++polls) {
        if (words_there(a, hand, word)) break;
        if (polls >= a.polls) {
            lost = true;
            __hip_atomic_store(a.hand + kHandFailed, a.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (polls > 32) __builtin_amdgcn_s_sleep(1);
        asm volatile("" : : : "memory");
    }
    asm volatile("" : : : "memory");
}
// The same for `count` gram units, lanes and turns; unit(i): which.
template <class F>
__device__ __forceinline__ void wait_gram(const FactorArgs &a, rsrc_t hand, int count, int lane, bool &lost, F &&unit)
{
    for (int i = lane; i - lane < count; i += kWave)
        for (int polls = 0; !lost; ++polls) {
            const unsigned v = __builtin_amdgcn_raw_buffer_load_b32(hand, i < count ? 4 * (kHandGram + unit(i)) : 0, 0, kDevice);
            if (__all(i >= count || v == a.seq)) break;
            if (polls >= a.polls) {
                lost = true;
                __hip_atomic_store(a.hand + kHandFailed, a.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            __builtin_amdgcn_s_sleep(1);
            asm volatile("" : : : "memory");
        }
    asm volatile("" : : : "memory");
}

// Partial tile of G: tile t = tri(i, j) over the rows z * zrows .. ; wavefront w takes a quarter of them.  Two
// rows of Y are the operands of V_MFMA_F32_32X32X2_F32 as they lie in memory, two neighbouring columns a lane: no LDS on the way.  What bounds
// it is how much is in flight (64 KB per compute unit at 2 us): a register is loaded again as soon as it has been used.  The wavefronts
// then add up a quarter of the tile each; columns of the tile are rows of the instruction's result, so that a lane holds four next to one
// another, as the operand order has them.
__device__ __forceinline__ void gram_unit(const FactorArgs &a, int tile, int z, rsrc_t ws, float4_t *red)
{
    const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = a.l;
    int i = 0;
    while (tri(i + 1, 0) <= tile) ++i;
    const int j = tile - tri(i, 0);
    const int per = a.zrows / 4;                // even
    const int k0 = z * a.zrows + wave * per;
    const int cnt = max(0, min(per, a.rows - k0));
    // (a base of its own keeps the offsets in 32 bits for any number of rows; reads past the range are zeros)
    const rsrc_t rs = make_rsrc(a.Y + (size_t)min(k0, a.rows) * l, (uint32_t)cnt * (uint32_t)l * 4u);
    const int na = kOb * i + 2 * r, nb = kOb * j + 2 * r;         // (l is even)
    const uint32_t ca = (uint32_t)(h * l + na) * 4u, cb = (uint32_t)(h * l + nb) * 4u;
    float16v_t acc[4];                           // rows 2 x + n / 2, columns 2 y + n % 2 of the tile (x: column, y: row of the instruction's result)
#pragma unroll
    for (int n = 0; n < 4; ++n)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[n][e] = 0.f;
    auto ld = [&](bool ok, uint32_t c, uint32_t row) { return load8(rs, ok ? c + row * (uint32_t)l * 4u : 0xFFFFFF00u, 0u); };
    // What kGramRun rows add up to goes to LDS (there are no registers left), to what came before: a sum is rounded once for every pair of rows,
    // at the size it has by then.
    float4_t *const before = red + wave * 16 * kWave + lane;
    bool any = false;
    auto add_before = [&] {
#pragma unroll
        for (int n = 0; n < 4; ++n)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4_t v = before[(4 * n + q) * kWave];
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[n][4 * q + e] += v[e];
            }
    };
    constexpr int U = 16;                       // pairs of rows in flight
    static_assert(kGramRun % (2 * U) == 0, "whole trips");
    uint2_t av[U], bv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        av[u] = ld(na < l, ca, (uint32_t)(2 * u));
        bv[u] = ld(nb < l, cb, (uint32_t)(2 * u));
    }
    for (int k = 0; k < cnt;) {
        for (const int end = min(cnt, k + kGramRun); k < end; k += 2 * U)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float av2[2], bv2[2];
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    const uint32_t x = av[u][b], y = bv[u][b];
                    av2[b] = __builtin_bit_cast(float, x);
                    bv2[b] = __builtin_bit_cast(float, y);
                }
#pragma unroll
                for (int n = 0; n < 4; ++n) acc[n] = __builtin_amdgcn_mfma_f32_32x32x2f32(bv2[n % 2], av2[n / 2], acc[n], 0, 0, 0);
                av[u] = ld(na < l, ca, (uint32_t)(k + 2 * (U + u)));
                bv[u] = ld(nb < l, cb, (uint32_t)(k + 2 * (U + u)));
                __builtin_amdgcn_sched_barrier(0);
            }
        if (k >= cnt) break;
        if (any) add_before();
        any = true;
#pragma unroll
        for (int n = 0; n < 4; ++n)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                before[(4 * n + q) * kWave] = float4_t{acc[n][4 * q], acc[n][4 * q + 1], acc[n][4 * q + 2], acc[n][4 * q + 3]};
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[n][4 * q + e] = 0.f;
            }
    }
    if (any) add_before();
    if (per > kGramRun) __syncthreads();         // (LDS is used again)
    // register 4 q + e of acc[n], row 8 q + 4 h + e of the result.  Wavefront w adds up those with q = w: the others leave their part of
    // them (q, slot of three) in LDS
    auto slot = [](int q, int w) { return (3 * q + (w < q ? w : w - 1)) * 4 * kWave; };
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (q != wave)
#pragma unroll
            for (int n = 0; n < 4; ++n)
                red[slot(q, wave) + n * kWave + lane] = float4_t{acc[n][4 * q], acc[n][4 * q + 1], acc[n][4 * q + 2], acc[n][4 * q + 3]};
    __syncthreads();
    float4_t sum[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (q == wave)
#pragma unroll
            for (int n = 0; n < 4; ++n) sum[n] = float4_t{acc[n][4 * q], acc[n][4 * q + 1], acc[n][4 * q + 2], acc[n][4 * q + 3]};
#pragma unroll
    for (int w = 0; w < 4; ++w)
        if (w != wave)
#pragma unroll
            for (int n = 0; n < 4; ++n) sum[n] += red[slot(wave, w) + n * kWave + lane];
    // lane: rows 2 r + p, columns 16 wave + 8 h + 4 f .. + 3
    const FactorPlaces at(a.nb);
    const uint32_t to = at.P + (uint32_t)(z * a.tiles + tile) * (kTileFloats * 4);
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            const float4_t v = {sum[2 * p][2 * f], sum[2 * p + 1][2 * f], sum[2 * p][2 * f + 1], sum[2 * p + 1][2 * f + 1]};
            const int row = 2 * r + p, col = 16 * wave + 8 * h + 4 * f;
            store_dev(ws, to + 4u * (uint32_t)op_at(row, col), v);
            if (i == j && row / 4 == col / 4) {  // (this lane's entry of the diagonal)
                const float d = (row & 2) ? ((row & 1) ? v[3] : v[2]) : ((row & 1) ? v[1] : v[0]);
                __hip_atomic_store(a.ws + at.diag / 4 + (size_t)z * a.nb * kOb + kOb * i + row, d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(a.hand + kHandGram + tile * a.splits + z, a.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// a b^T of 16 x 16 blocks in operand order, added to c in the same order
__device__ __forceinline__ void mul16(float4_t a, float4_t b, float4_t &c) { mma16(b, a, c); }

// Blocks (q, w) .. (q, w + N - 1) of a tile, lane by lane: the sums of its partial tiles.
template <int N>
__device__ __forceinline__ void gram_blocks(const FactorArgs &a, rsrc_t ws, int tile, int q, int w, int lane, float4_t (&s)[N])
{
    constexpr int U = N > 1 ? 4 : 8;            // shares in flight
    const uint32_t from = FactorPlaces(a.nb).P + (uint32_t)tile * (kTileFloats * 4) + (uint32_t)((q * 4 + w) * 64 + lane) * 16u;
    const uint32_t step = (uint32_t)a.tiles * (kTileFloats * 4);
#pragma unroll
    for (int n = 0; n < N; ++n) s[n] = float4_t{0.f, 0.f, 0.f, 0.f};
    for (int z = 0; z < a.splits; z += U) {
        float4_t v[U][N];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int n = 0; n < N; ++n) v[u][n] = load_dev(ws, z + u < a.splits ? from + (uint32_t)(z + u) * step + 1024u * n : 0xFFFFFFF0u);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int n = 0; n < N; ++n) s[n] += v[u][n];
    }
}

// The strips in the order (column j, row tile I, sixteen rows q), but for those of the first diagonal tile, which is the chain's alone.
__host__ __device__ void strip_at(int strip, int nb, int *I, int *j, int *q)
{
    int c = 0, left = strip / 4 + 1;
    while (left >= nb - c) left -= nb - c++;
    *I = c + left;
    *j = c;
    *q = strip % 4;
}

// Wavefront w makes the 16 columns 16 w .. of 16 rows of the tile (I, j).
// It adds up the partial tiles, subtracts L_IK L_jK^T for the columns K before its own as they come, and hands the strip to the chain or waits
// for the inverse of the diagonal tile and hands on L_Ij = A_Ij X_j^T.
__device__ __forceinline__ void strip_role(const FactorArgs &a, int strip, rsrc_t ws, rsrc_t hand, float4_t *sh)
{
    const int lane = threadIdx.x & 63, mq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const FactorPlaces at(a.nb);
    auto block = [&](uint32_t region, int tile, int q, int t) { return region + (uint32_t)tile * (kTileFloats * 4) + (uint32_t)((q * 4 + t) * 64 + lane) * 16u; };
    bool lost = false;
    int I, j, q;
    strip_at(strip, a.nb, &I, &j, &q);
    wait_gram(a, hand, a.splits, lane, lost, [&](int i) { return tri(I, j) * a.splits + i; });
    float4_t sum[1];
    gram_blocks(a, ws, tri(I, j), q, wave, lane, sum);
    float4_t c = sum[0];
    for (int K = 0; K < (I == j ? j - 1 : j); ++K) {
        wait_words(a, hand, lane == 0 ? kHandL + 16 * tri(I, K) + 4 * q : lane == 1 ? kHandL + 16 * tri(j, K) + 4 * wave : -1, lost);
        float4_t x[4], y[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            x[t] = load_dev(ws, block(at.Lf, tri(I, K), q, t));
            y[t] = load_dev(ws, block(at.Lf, tri(j, K), wave, t));
        }
        // (one column at a time: what is left of c grows smaller, and its rounding with it, where the sum of all columns would grow)
        float4_t s0 = {0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
        for (int t = 0; t < 4; ++t) mul16(x[t], y[t], t & 1 ? s1 : s0);
        c -= s0 + s1;
    }
    if (I <= j + 1) {
        store_dev(ws, block(at.G, tri(I, j), q, wave), c);
        hand_over(a, (I == j ? kHandT : kHandA) + 16 * I + 4 * q + wave, lane);
        if (I == j) return;
    }
    sh[wave * 64 + lane] = c;
    __syncthreads();
    wait_words(a, hand, lane == 0 ? kHandD + 16 * j : -1, lost);
    float4_t x[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) x[t] = t <= wave ? load_dev(ws, block(at.D, j, wave, t)) : float4_t{0.f, 0.f, 0.f, 0.f};
    const float4_t alive = load_dev(ws, at.D + (uint32_t)j * (kTileFloats * 4) + 1024u + (uint32_t)(16 * wave + 4 * mq) * 4u);
    float4_t y0 = {0.f, 0.f, 0.f, 0.f}, y1 = y0;
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (t <= wave) mul16(sh[t * 64 + lane], x[t], t & 1 ? y1 : y0);
    float4_t y = y0 + y1;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = alive[e] != 0.f ? y[e] : 0.f;
    store_dev(ws, block(at.Lf, tri(I, j), q, wave), y);
    hand_over(a, kHandL + 16 * tri(I, j) + 4 * q + wave, lane);
}

// LDS of the chain, in 16 x 16 blocks in operand order.
struct ChainLds {
    float4_t T[10][64];                          // the diagonal tile, block (i, k) at tri(i, k), as far as it is worked on
    float4_t L[6][64];                           // its factor, below the diagonal: (i, k) at tri(i - 1, k)
    float4_t X0[2][64];                          // its inverse: block (0, 0), of this tile and of the one before it,
    float4_t X[9][64];                           //   and the others, (i, k) at tri(i, k) - 1
    float4_t XT[6][64];                          // the blocks (i, k) of the inverse, i < 3, transposed
    float4_t P[16][64];                          // the panel between the tile before and this one
    float4_t next[3][64];                        // for wavefront 0, of the next tile: block (0, 0), and (0, 0) and (0, 1) of the tile to its left;
    int have;                                    //   whether they are there
    float alive[2][kOb];                         // whether a pivot is above the floor: of this tile, of the one before it
    float mx[4];
};

// The diagonal tiles.  Wavefront 0 factors blocks of 16; wavefront w > 0 owns row w of the blocks of a tile and brings it up to date
// meanwhile, one step behind.  What wavefront 0 needs next it works out itself, the others in registers of their own again: barriers
// are only between the steps.  A tile is 7.3 us: 0.9 to factor each of its four blocks and 0.2 to 0.4 around that, 1.4 for the panel between the tile
// before and this one, 0.6 to end the inverse, and, about as long on the whole, what passes between the inverse of a tile and what
// the tile after next needs of the strips (two hand-overs of 2.5 us): both would have to be shorter.
__device__ __forceinline__ void chain_role(const FactorArgs &a, rsrc_t ws, rsrc_t hand, ChainLds &s)
{
    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 15, mq = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const FactorPlaces at(a.nb);
    auto block = [&](uint32_t region, int tile, int q, int t) { return region + (uint32_t)tile * (kTileFloats * 4) + (uint32_t)((q * 4 + t) * 64 + lane) * 16u; };
    const float4_t zero = {0.f, 0.f, 0.f, 0.f};
    bool lost = false;
    // row `wave` of the first tile
    float4_t to[3], td;                          // blocks (wave, k), k < wave, and (wave, wave)
    wait_gram(a, hand, a.nb * a.splits, lane, lost, [&](int i) { return tri(i / a.splits, i / a.splits) * a.splits + i % a.splits; });
    float mx = 0.f;                              // the largest diagonal entry of G
    for (int c = 4 * tid; c < a.nb * kOb; c += 4 * 256) {
        float4_t d = zero;
#pragma unroll 8
        for (int z = 0; z < a.splits; ++z) d += load_dev(ws, at.diag + (uint32_t)(z * a.nb * kOb + c) * 4u);
#pragma unroll
        for (int e = 0; e < 4; ++e) mx = fmaxf(mx, d[e]);
    }
    {
        float4_t row[4];
        gram_blocks(a, ws, 0, wave, 0, lane, row);
#pragma unroll
        for (int k = 0; k < 3; ++k) to[k] = row[k];
        td = wave == 0 ? row[0] : wave == 1 ? row[1] : wave == 2 ? row[2] : row[3];
    }
    mx = wave_max(mx);
    if (lane == 0) s.mx[wave] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(s.mx[0], s.mx[1]), fmaxf(s.mx[2], s.mx[3]));
    // Far from 1 the block is factored as 4^h G (exact): the reciprocals of factor16() know no subnormal numbers
    int h = 0;
    if (mx > 0.f && !(mx > 0x1p-60f && mx < 0x1p60f)) h = min(max(-(__builtin_amdgcn_frexp_expf(mx) / 2), -63), 63);
    const float dead = ldexpf(fmaxf(1.0f, mx * 1e-9f), 2 * h), floor_ = fmaxf(ldexpf(mx, 2 * h) * 1e-9f, 0x1p-120f);
    float pmax = 0.f, pmin = __builtin_inff();   // (of the rows of a lane of wavefront 0)
    auto scaled = [&](float4_t v, int by) {
        if (h != 0)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = ldexpf(v[e], by);
        return v;
    };
    // columns of dead pivots as zeros (lane: columns 4 mq .. of block k)
    auto living = [&](float4_t v, int which, int k) {
        const float4_t f = reinterpret_cast<const float4_t *>(s.alive[which])[4 * k + mq];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = f[e] != 0.f ? v[e] : 0.f;
        return v;
    };
    // what tile j needs: row `wave` of it, rows 0 (the blocks up to `wave`) and `wave` of the tile to its left; wavefront 1 looks out for
    // wavefront 0 too
    float4_t a0[4], aw[4], t00 = zero;
    bool there = false;
    auto words_of = [&](int j) {
        const int t = kHandT + 16 * j, l = kHandA + 16 * j;
        return lane == 0 ? t + 4 * wave : lane == 1 ? l : lane == 2 ? l + 4 * wave : lane == 3 && wave == 1 ? t : -1;
    };
    auto load_tile = [&](int j) {
#pragma unroll
        for (int t = 0; t < 4; ++t) a0[t] = wave < 3 && (t < 2 || wave > 0) ? load_dev(ws, block(at.G, tri(j, j - 1), 0, t)) : zero;
#pragma unroll
        for (int t = 0; t < 4; ++t) aw[t] = wave > 0 ? load_dev(ws, block(at.G, tri(j, j - 1), wave, t)) : zero;
#pragma unroll
        for (int k = 0; k < 3; ++k) to[k] = k < wave ? load_dev(ws, block(at.G, tri(j, j), wave, k)) : zero;
        td = load_dev(ws, block(at.G, tri(j, j), wave, wave));
        if (wave == 1) t00 = load_dev(ws, block(at.G, tri(j, j), 0, 0));
    };
    for (int j = 0; j < a.nb; ++j) {
        const int cur = j & 1, prev = cur ^ 1;
        auto X = [&](int which, int i, int k) { return i == 0 ? s.X0[which][lane] : s.X[tri(i, k) - 1][lane]; };
        float4_t pw[4] = {zero, zero, zero, zero};       // row `wave` of the panel
        float4_t p0, p1;
        auto panel_diagonal = [&] {
            p0 = p1 = zero;
#pragma unroll
            for (int t = 0; t < 4; ++t) mul16(pw[t], pw[t], t & 1 ? p1 : p0);
            td -= p0 + p1;
        };
        if (j > 0) {
            if (wave == 0 && s.have) {
                td = s.next[0][lane];
                a0[0] = s.next[1][lane];
                a0[1] = s.next[2][lane];
            } else if (!there) {
                wait_words(a, hand, words_of(j), lost);
                load_tile(j);
            }
            // block (0, wave) of the panel
            // (wavefront 3 is busy handing over)
            auto panel_block = [&](int c) {
                p0 = p1 = zero;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (t <= c) mul16(scaled(a0[t], 2 * h), X(prev, c, t), t & 1 ? p1 : p0);
                s.P[c][lane] = living(p0 + p1, prev, c);
            };
            if (wave == 0) {
                panel_block(0);
                panel_block(1);
            } else if (wave < 3) {
                panel_block(wave == 1 ? 3 : 2);
            }
            __syncthreads();
            td = scaled(td, 2 * h);
            if (wave > 0) {
#pragma unroll
                for (int t = 0; t < 4; ++t) aw[t] = scaled(aw[t], 2 * h);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    p0 = p1 = zero;
#pragma unroll
                    for (int t = 0; t <= c; ++t) mul16(aw[t], X(prev, c, t), t & 1 ? p1 : p0);
                    pw[c] = living(p0 + p1, prev, c);
                    s.P[4 * wave + c][lane] = pw[c];
                }
                p0 = p1 = zero;
#pragma unroll
                for (int t = 0; t < 4; ++t) mul16(pw[t], s.P[t][lane], t & 1 ? p1 : p0);
                to[0] = scaled(to[0], 2 * h) - (p0 + p1);
                if (wave == 1) panel_diagonal();         // (the others' have time until the next step)
            } else {
                p0 = p1 = zero;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const float4_t p = s.P[t][lane];
                    mul16(p, p, t & 1 ? p1 : p0);
                }
                td -= p0 + p1;
            }
        } else {
            to[0] = scaled(to[0], 2 * h);
            td = scaled(td, 2 * h);
        }
        // (the columns between are brought up to date when their turn comes)
        to[1] = scaled(to[1], 2 * h);
        to[2] = scaled(to[2], 2 * h);
        if (wave > 0) {
            s.T[tri(wave, 0)][lane] = to[0];
            if (wave == 1) s.T[tri(1, 1)][lane] = td;
        }
        // wavefront 0: block (b, b)
        auto factor = [&](int b, float4_t w) {
            const bool ok = factor16(w, ln, mq, floor_, dead, pmax, pmin);
            if (lane < 16) s.alive[cur][16 * b + ln] = ok ? 1.f : 0.f;
            if (b == 0)
                s.X0[cur][lane] = w;
            else
                s.X[tri(b, b) - 1][lane] = w;
            if (b < 3) {
                float *const xt = reinterpret_cast<float *>(s.XT[tri(b, b)]);
#pragma unroll
                for (int e = 0; e < 4; ++e) xt[(ln >> 2) * 64 + (4 * mq + e) * 4 + (ln & 3)] = w[e];
            }
        };
        // block (i, k) of the inverse, -X_ii sum_{k <= m < i} L_im X_mk
        auto inverse = [&](int i, int k) {
            float4_t m0 = zero, m1 = zero, y = zero;
            for (int m = k; m < i; ++m) mul16(s.XT[tri(m, k)][lane], s.L[tri(i - 1, m)][lane], (m - k) & 1 ? m1 : m0);
            m0 += m1;                            // transposed
            const float4_t x = X(cur, i, i);
            mul16(x, m0, y);
            s.X[tri(i, k) - 1][lane] = -y;
            if (i < 3) {
                y = zero;
                mul16(m0, x, y);
                s.XT[tri(i, k)][lane] = -y;
            }
        };
        if (wave == 0) factor(0, td);
        __syncthreads();
        there = false;
        for_each<3>([&](auto bc) {
            constexpr int b = bc + 1;
            if constexpr (b == 3)
                if (wave > 0 && j + 1 < a.nb) {
                    // what the next tile needs, if it is ready: (the registers of this one are free)
                    there = words_there(a, hand, words_of(j + 1)) || words_there(a, hand, words_of(j + 1));
                    if (there) load_tile(j + 1);
                }
            if (wave == 0 || wave >= b) {
                const float4_t x = X(cur, b - 1, b - 1);
                float4_t lb = zero;
                if (wave != b) {
                    mul16(s.T[tri(b, b - 1)][lane], x, lb);
                    lb = living(lb, cur, b - 1);
                }
                if (wave == 0) {
                    float4_t c = zero;
                    mul16(lb, lb, c);
                    factor(b, s.T[tri(b, b)][lane] - c);
                } else {
                    float4_t lw = zero, c = zero;
                    mul16(s.T[tri(wave, b - 1)][lane], x, lw);
                    lw = living(lw, cur, b - 1);
                    s.L[tri(wave - 1, b - 1)][lane] = lw;
                    if (wave > b) {
                        if (b == 1) panel_diagonal();
                        mul16(lw, lw, c);
                        td -= c;
                        s.T[tri(wave, wave)][lane] = td;
                        if constexpr (b < 3) {
                            // column b of this row
                            float4_t c0 = zero, c1 = zero;
                            if (j > 0) {
#pragma unroll
                                for (int t = 0; t < 4; ++t) mul16(pw[t], s.P[4 * b + t][lane], t & 1 ? c1 : c0);
                                to[b] -= c0 + c1;
                                c0 = c1 = zero;
                            }
                            for (int k = 0; k < b - 1; ++k) mul16(s.L[tri(wave - 1, k)][lane], s.L[tri(b - 1, k)][lane], c0);
                            mul16(lw, lb, c1);
                            s.T[tri(wave, b)][lane] = to[b] - (c0 + c1);
                        }
                    }
                }
            } else if (b == 2) {
                inverse(1, 0);                   // (wavefront 1)
            } else if (b == 3) {
                inverse(2, wave == 1 ? 1 : 0);   // (wavefronts 1 and 2)
            }
            __syncthreads();
        });
        const uint32_t out = at.D + (uint32_t)j * (kTileFloats * 4);
        auto publish = [&](int i) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k <= i) store_dev(ws, out + (uint32_t)((i * 4 + k) * 64 + lane) * 16u, scaled(X(cur, i, k), h));
        };
        if (wave < 3) {
            inverse(3, wave);
        } else {
            publish(0);
            publish(1);
            publish(2);
        }
        if (wave == 1) {
            if (there) {
                s.next[0][lane] = t00;
                s.next[1][lane] = a0[0];
                s.next[2][lane] = a0[1];
            }
            if (lane == 0) s.have = there;
        }
        __syncthreads();
        // the rest of the inverse to memory, and the living pivots
        if (wave == 3) {
            publish(3);
            if (lane < 16) store_dev(ws, out + 1024u + (uint32_t)lane * 16u, reinterpret_cast<const float4_t *>(s.alive[cur])[lane]);
            hand_over<4>(a, kHandD + 16 * j, lane);
        }
    }
    if (wave != 0) return;
    pmax = wave_max(pmax);
    pmin = -wave_max(-pmin);
    if (tid == 0) {
        const int run = orth_run(a.step.in ? a.step.in->run : 0, a.step.h, pmax, pmin);
        a.step.out->run = run;
        a.step.out->due = orth_due(a.step.h, run, a.step.last);
    }
}

__global__ __launch_bounds__(256, 2) void lora_factor_kernel(FactorArgs a)
{
    if (a.step.skip()) return;
    __shared__ float4_t lds[4 * 16 * kWave];                 // (of a gram unit: the registers of its wavefronts)
    static_assert(sizeof(ChainLds) <= sizeof(lds), "LDS of the chain");
    ChainLds &s = *reinterpret_cast<ChainLds *>(lds);
    const rsrc_t ws = make_rsrc(a.ws, FactorPlaces(a.nb).end), hand = make_rsrc(a.hand, kHandWords * 4u);
    const int units = a.tiles * a.splits, b = (int)blockIdx.x;
    if (b < units)
        gram_unit(a, b / a.splits, b % a.splits, ws, lds);       // (a range of rows on one die, where their number is a multiple of 8)
    else if (b == units)
        chain_role(a, ws, hand, s);
    else
        strip_role(a, b - units - 1, ws, hand, s.P[0]);
}

// The power of two that brings a column whose largest magnitude has the bits `max_bits` below 1.
__device__ __forceinline__ float column_scale(unsigned max_bits)
{
    const int e = (int)(max_bits >> 23);         // |v| < 2^(e - 126)
    return max_bits == 0u ? 1.0f : __uint_as_float((unsigned)max(253 - e, 1) << 23);
}

// 16 rows of out = in Lc^-T, block column after block column; wavefront w computes the columns 16 w .. 16 w + 15 of each.
// Where the step skips the orthonormalisation: 16 rows of out = `in` with scaled columns (colmax: kColSlots rows of bits of their
// largest magnitudes).  clear: those of the next block, set to zero.
// The orthonormalisation is a chain of latencies (matrix cores 6.5 us of the 20).  The two fp16 numbers go out from the registers that hold a block column, and the wavefronts meet
// before they need one another's columns, not after each block column: 1.2 us less than with the whole rows converted from LDS at the end.
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
    // N rows of column c from `row` on as two fp16 numbers, columns as rows
    auto emit = [&](int c, int row, const auto &v16) {
        constexpr int N = sizeof(v16) / sizeof(v16[0]), Q = N < 8 ? N : 8;
        typedef half_t piece_t __attribute__((ext_vector_type(Q)));
        const size_t at = (size_t)c * ldk + row;
#pragma unroll
        for (int q = 0; q < N / Q; ++q) {
            piece_t h, g;
#pragma unroll
            for (int r = 0; r < Q; ++r) {
                const float s = v16[Q * q + r] * kBlockSplit, v = fabsf(s) > 65000.0f ? copysignf(65000.0f, s) : s;
                const half_t x = (half_t)v;
                h[r] = x;
                g[r] = (half_t)((v - (float)x) * kLowSplit);
            }
            *reinterpret_cast<piece_t *>(hi + at + Q * q) = h;
            *reinterpret_cast<piece_t *>(lo + at + Q * q) = g;
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
            emit(c, r0, v16);
        }
        return;
    }
    const float poison = hand[kHandFailed] == seq ? __builtin_nanf("") : 0.f;      // the factor is not whole: must not pass for one
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
            d[t] = t <= wave ? reinterpret_cast<const float4_t *>(D + (size_t)J * kTileFloats)[(wave * 4 + t) * 64 + lane] : float4_t{0.f, 0.f, 0.f, 0.f};
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
            if (K == J - 1) __syncthreads();     // (the other wavefronts' columns of the block column before this one)
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
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = r0 + 4 * mq + e;
            y[e] = y0[e] + y1[e];
            O[(4 * mq + e) * ldo + kOb * J + 16 * wave + ln] = y[e];
            if (out && row < rows && col < l) out[(size_t)row * l + col] = y[e];
        }
        if (hi && col < l) emit(col, r0 + 4 * mq, y);         // (rows past the last are zeros)
    }
}

// Into how many ranges of rows the units of a tile of G go, and how many rows each has.  A workgroup per compute unit, at least 64 rows each, and no
// more than kGramRange as long as there is room: the matrix cores' work decides then, which 136 units (1024 columns) would leave to half of the chip, and
// the bytes of a quarter of a range (a wavefront's part) have to have 32-bit offsets.
// us and relative error of a block, in brackets with a workgroup per compute unit at any number of rows and no kGramRun: 28672 x 832 556, 6.7e-7 (596, 1.9e-6),
// 28672 x 1024 806, 7.4e-7 (954, 3.9e-6), 4096 x 1024 265, 1.0e-6 (266, 2.2e-6).
constexpr int kGramRange = 4096;
int gram_ranges(int rows, int l, int *rows_each)
{
    const int nb = (l + kOb - 1) / kOb, tiles = tri(nb, 0);
    int n = 256 / tiles;
    if (n > (rows + 63) / 64) n = (rows + 63) / 64;
    if (((long)rows + n - 1) / n > kGramRange) n = (int)min((long)kGramUnits / tiles, ((long)rows + kGramRange - 1) / kGramRange);
    if (n > kDies) n = n / kDies * kDies;
    *rows_each = (int)((((long)rows + n - 1) / n + 31) / 32 * 32);
    return (int)(((long)rows + *rows_each - 1) / *rows_each);
}

// Workspace of the orth()s of a call, in floats: what the workgroups of a factorisation hand on, three sets of OrthWords, two times
// kColSlots rows of column maxima.
constexpr int kOrthWords = 64;
size_t orth_floats(int l) { return FactorPlaces((l + kOb - 1) / kOb).end / 4 + kOrthWords + 2 * (size_t)kColSlots * l; }
unsigned *orth_column_max(float *ws, int l, int which)
{
    return reinterpret_cast<unsigned *>(ws + orth_floats(l) - (size_t)(2 - which) * kColSlots * l);
}

// out (or null): fp32 [rows][l]; hi, lo (or null): the block for lora_split_gemm_kernel, [l][rows rounded up to 32].
// h < 0: always orthonormal.  Else the block after h products, of `last`, in a call's sequence of them (hi, lo only, out = null):
// orthonormal for h = 0, conditional from then on, where orth_column_max(h % 2) holds the column maxima of `in`; that of
// the next block is cleared.
// hand: orth_hand_words() words, zero at the start of a call's sequence, of which this is number seq (from 1).
size_t orth_hand_words() { return kHandWords; }
int launch_orth(const float *in, float *out, half_t *hi, half_t *lo, int rows, int l, float *ws, unsigned *hand, unsigned seq, int h, int last,
                hipStream_t st)
{
    const int nb = (l + kOb - 1) / kOb, tiles = tri(nb, 0);
    const FactorPlaces at(nb);
    OrthWords *const words = reinterpret_cast<OrthWords *>(ws + at.end / 4);
    static_assert(3 * sizeof(OrthWords) <= kOrthWords * sizeof(float), "words of the orth()s");
    const OrthStep step{h > 0 ? words + (h & 1) : nullptr, h < 0 ? words + 2 : words + ((h + 1) & 1), h, last};
    const unsigned *const colmax = h > 0 ? orth_column_max(ws, l, h & 1) : nullptr;
    unsigned *const clear = h >= 0 ? orth_column_max(ws, l, (h + 1) & 1) : nullptr;
    FactorArgs f{};
    f.Y = in;
    f.rows = rows;
    f.l = l;
    f.nb = nb;
    f.tiles = tiles;
    f.ws = ws;
    f.hand = hand;
    f.seq = seq;
    f.step = step;
    f.splits = gram_ranges(rows, l, &f.zrows);
    const bool wait_test = adapters_wait_test();     // (slim_decode_override: only the workgroup that waits for the others)
    f.polls = wait_test ? 256 : kHandPolls;
    hipLaunchKernelGGL(lora_factor_kernel, dim3((unsigned)(tiles * f.splits + 1 + (wait_test ? 0 : 4 * (tiles - 1)))), dim3(256), 0, st, f);
    const size_t lds = (size_t)(16 * (nb * kOb + 4) + 16 * 68) * sizeof(float);
    hipLaunchKernelGGL(lora_apply_kernel, dim3((unsigned)((rows + 31) / 32 * 2)), dim3(256), lds, st, in, out, rows, l, nb,
                       (const float *)(ws + at.Lf / 4), (const float *)(ws + at.D / 4), hi, lo, (rows + 31) / 32 * 32, step, colmax, clear,
                       (const unsigned *)hand, seq);
    return hip_status(hipGetLastError());
}

}  // namespace slim
