// slim_pack / slim_unpack / slim_pack_adapters: the encoding side of the layer.
//
// slim_pack is a streaming kernel bound by HBM: it reads 4 bytes per weight
// and writes 3 bits per weight.  One workgroup owns one output row: it keeps
// the row in registers while the row maximum is reduced (so W is read from
// memory once), then each lane encodes the groups of 4 it holds.
#include "slim_internal.h"

namespace slim {

constexpr int kPackSlotsMax = 12;   // float4 groups a lane keeps at most: rows up to 4 * 1024 * 12 inputs stay in registers

// The codes of a row divide by its scale s.  rint(w / s) is taken from w (1 / s) wherever that decides: the product is within
// 2e-6 of the IEEE quotient for codes up to 8 in magnitude, so the two round to the same integer unless the product
// lies within 4e-6 of a half; there, and where the reciprocal is not a normal number with room on both sides, it is divided.
struct RowScale {
    float s, inv;
};
__device__ __forceinline__ RowScale row_scale(float s)
{
    return RowScale{s, s > 0x1p-100f && s < 0x1p100f ? 1.0f / s : __builtin_nanf("")};
}

// Encode one group: returns the qvals byte, *m4 the metadata nibble i0 | (i1 << 2).  The kept positions i0 < i1 are the first two in the
// order (|w| sal descending, position ascending); sal: the saliency of the four inputs (all ones: the magnitude mask), the
// products are single binary32 multiplications.  Six comparisons, whose combinations are scalar operations on the masks of a
// wavefront, and selects.  The kernels here are as much bound by vector instructions as by memory: a chain of selections
// with branches and two IEEE divisions were 150 per group, these are about 60 (11008 x 4096 with scales and saliency given
// 38 -> 30 us, and that only with both of it: pack_scaled_kernel with the chain took as long as the rows did).
__device__ __forceinline__ uint32_t encode_group(float4 v, const RowScale &rs, uint32_t *m4, float4 sal = make_float4(1.f, 1.f, 1.f, 1.f))
{
    // (a NaN loses against everything, but for one in position 0, which nothing beats)
    const float a0 = fabsf(v.x) * sal.x, a1 = fmaxf(fabsf(v.y) * sal.y, -1.0f), a2 = fmaxf(fabsf(v.z) * sal.z, -1.0f),
                a3 = fmaxf(fabsf(v.w) * sal.w, -1.0f);
    // the later one comes before the earlier one, a bit per lane
    auto mask = [](bool b) { return __builtin_amdgcn_ballot_w64(b); };
    const uint64_t b01 = mask(a1 > a0), b02 = mask(a2 > a0), b03 = mask(a3 > a0), b12 = mask(a2 > a1), b13 = mask(a3 > a1), b23 = mask(a3 > a2);
    // kept: at most one of the other three comes before it
    auto one_at_most = [](uint64_t x, uint64_t y, uint64_t z) { return __builtin_amdgcn_inverse_ballot_w64(~((x & y) | (z & (x | y)))); };
    const bool k0 = one_at_most(b01, b02, b03), k1 = one_at_most(~b01, b12, b13), k2 = one_at_most(~b02, ~b12, b23),
               k3 = one_at_most(~b03, ~b13, ~b23);
    const float w0 = k0 ? v.x : (k1 ? v.y : v.z), w1 = k3 ? v.w : (k2 ? v.z : v.y);
    *m4 = (k0 ? 0u : (k1 ? 1u : 2u)) | (k3 ? 12u : (k2 ? 8u : 4u));
    const float q0 = w0 * rs.inv, q1 = w1 * rs.inv;
    float r0 = rintf(q0), r1 = rintf(q1);
    if (!(fmaxf(fabsf(q0 - r0), fabsf(q1 - r1)) <= 0.499996f)) {
        r0 = rintf(w0 / rs.s);                // IEEE division, round half to even
        r1 = rintf(w1 / rs.s);
    }
    r0 = fminf(fmaxf(r0, -8.0f), 7.0f);
    r1 = fminf(fmaxf(r1, -8.0f), 7.0f);
    return ((uint32_t)(int)r0 & 0xFu) | (((uint32_t)(int)r1 & 0xFu) << 4);
}

// THREADS lanes per row; SLOTS = float4 groups of the row each lane keeps in
// registers (the row has at most 4 THREADS SLOTS inputs); 0 = rows of any
// length, read twice.  Few slots per lane keep the register count low enough
// for eight wavefronts per SIMD, which is what hides the load latency here.
// The kernel is as much bound by its vector ALU work as by memory, so the stores stay plain byte stores: lane
// t writes group t + i THREADS of slot i, whose place in the packed layout is a
// per-lane base plus a constant per slot.
// EX: the variant behind slim_pack_ex: saliency [k] weighs the magnitudes in the
// 2:4 choice.
template <int THREADS, int SLOTS, bool EX = false>
__global__ __launch_bounds__(THREADS) void pack_kernel(const float *__restrict__ W, int n, int k,
                                                            uint8_t *__restrict__ qvals,
                                                            uint8_t *__restrict__ meta,
                                                            float *__restrict__ scale,
                                                            const float *__restrict__ saliency = nullptr)
{
    __shared__ float wave_part[THREADS / kWave];
    const int ngroups = k / 4;
    const int tid = threadIdx.x;
    const uint32_t kt = pk_ktiles(k);
    const int gpad = (int)kt * 32;             // groups per row of the packed layout
    const int npad = (n + 31) / 32 * 32;
    // Workgroups go to the 8 dies round-robin and each die has its own L2.  The 32
    // rows of a row tile write into the same cache lines, so they are kept on one
    // die: die x takes a contiguous range of row tiles, its workgroups walk that
    // range row by row.  (The grid is a multiple of 8.)
    const int die = blockIdx.x & 7, local = blockIdx.x >> 3, per_die = gridDim.x >> 3;
    const int rows_per_die = ((npad / 32 + 7) / 8) * 32;
    const int o_end = min(npad, (die + 1) * rows_per_die);
    for (int o = die * rows_per_die + local; o < o_end; o += per_die) {
        // the row in the packed layout, and this lane's byte of a slot in it (group tid, position byte tid / 2): one address
        // in scalar registers and one offset, where an address per slot took the registers of the second workgroup of a unit
        uint8_t *const qrow = qvals + pk_qoff(o, 0, kt), *const mrow = meta + pk_moff(o, 0, kt);
        const uint32_t ql = (uint32_t)pk_qoff(0, tid, kt), ml = (uint32_t)pk_moff(0, tid >> 1, kt);
        constexpr size_t q_slot = (size_t)(THREADS / 32) * 1024, m_slot = (size_t)(THREADS / 32) * 512;
        if (o >= n) {
            // padding row of the last row tile: zero bytes
            for (int g = tid, i = 0; g < gpad; g += THREADS, ++i) {
                (qrow + i * q_slot)[ql] = 0;
                if ((g & 1) == 0) (mrow + i * m_slot)[ml] = 0;
            }
            continue;
        }
        const float4 *row = reinterpret_cast<const float4 *>(W + (size_t)o * k);
        constexpr bool CACHED = SLOTS > 0;
        // Not kept: four groups at a time, because a wait for a load is also one for the stores before it, and a group's work is
        // short (one at a time, 2048 x 60000 177 and 183 us, without and with saliency, this 153 and 161; 33 x 131072 119 and 125,
        // this 85 and 91; with loads that leave the L2 first 193 and 218, what the second pass reads there)
        constexpr int AHEAD = 4;
        auto weights = [&](int g) { return row[min(g, ngroups - 1)]; };
        float4 cache[CACHED ? SLOTS : 1];
        float a = 0.0f;
        if (CACHED) {
#pragma unroll
            for (int i = 0; i < SLOTS; ++i) {
                int g = tid + i * THREADS;
                float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                if (g < ngroups) v = row[g];
                cache[i] = v;
                a = fmaxf(a, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
            }
        } else {
            for (int g0 = 0; g0 < ngroups; g0 += 4 * THREADS) {
                float4 v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = weights(g0 + u * THREADS + tid);
#pragma unroll
                for (int u = 0; u < 4; ++u) a = fmaxf(a, fmaxf(fmaxf(fabsf(v[u].x), fabsf(v[u].y)), fmaxf(fabsf(v[u].z), fabsf(v[u].w))));
            }
        }
        a = wave_max(a);
        __syncthreads();                       // wave_part is reused across rows
        if ((tid & (kWave - 1)) == 0) wave_part[tid / kWave] = a;
        __syncthreads();
        a = wave_part[0];
#pragma unroll
        for (int w = 1; w < THREADS / kWave; ++w) a = fmaxf(a, wave_part[w]);
        const float s = (a == 0.0f) ? 1.0f : a / 7.0f;
        const RowScale rs = row_scale(s);
        if (tid == 0) scale[o] = s;

        // Lanes g and g^1 hold the two groups of one position byte (the stride is
        // even, so both are active together).  Groups past the end of the row
        // (padding of the last tile) are zero bytes.
        auto emit = [&](int i, int g, float4 v, auto sal_of) {
            uint32_t q = 0, m4 = 0;
            if (g < ngroups) {
                if (EX)
                    q = encode_group(v, rs, &m4, sal_of(g));
                else
                    q = encode_group(v, rs, &m4);
            }
            const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m4, 0xB1, 0xF, 0xF, true);     // of lane ^ 1
            if (g < gpad) {
                (qrow + i * q_slot)[ql] = (uint8_t)q;
                if ((g & 1) == 0) (mrow + i * m_slot)[ml] = (uint8_t)(m4 | (other << 4));
            }
        };
        if (CACHED) {
#pragma unroll
            for (int i = 0; i < SLOTS; ++i) emit(i, tid + i * THREADS, cache[i], [&](int g) { return reinterpret_cast<const float4 *>(saliency)[g]; });
        } else {
            // (from the end of the row, whose last part is what the first pass left in the L2)
            for (int i = ((gpad + THREADS - 1) / THREADS - 1) / AHEAD * AHEAD; i >= 0; i -= AHEAD) {
                const int g0 = i * THREADS;
                float4 v[AHEAD], sal[AHEAD];
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
                    v[u] = weights(g0 + u * THREADS + tid);
                    if (EX) sal[u] = reinterpret_cast<const float4 *>(saliency)[min(g0 + u * THREADS + tid, ngroups - 1)];
                }
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) emit(i + u, g0 + u * THREADS + tid, v[u], [&](int) { return sal[u]; });
            }
        }
    }
}

// The same with the scales given (slim_pack_ex): nothing is to be known of a row, so a workgroup takes half a tile of the packed
// layout, 16 rows x 128 inputs, two groups per lane, at a time, with the loads of its next one under way.  Sixteen lanes read
// 256 contiguous bytes of a row, and a workgroup's codes are two runs of 256 bytes: by rows they were 16 bytes of a line that
// the workgroups of other rows filled up.  16384 workgroups: 11008 x 4096 29.9 us, 16115 x 7296 94.7 (2048: 31.2 and 103.7; whole
// tiles 29.2 and 95.1, on 4096 x 4096 13.5 instead of 12.9; quarters 33 and 107).  saliency: [k], or null.
constexpr int kPackScaledGrid = 16384;
__global__ __launch_bounds__(256) void pack_scaled_kernel(const float *__restrict__ W, int n, int k, const float *__restrict__ saliency,
                                                          const float *scale_in, uint8_t *__restrict__ qvals, uint8_t *__restrict__ meta,
                                                          float *scale)
{
    const uint32_t kt = pk_ktiles(k), ngroups = (uint32_t)k / 4, parts = (uint32_t)((n + 31) / 32) * kt * 2;
    const uint32_t r = threadIdx.x >> 4, c = threadIdx.x & 15;
    struct Part {
        float4 w[2], sal[2];
        float s;
        uint32_t row, col;                   // of the lane's first group
    };
    // (lanes of the padding load the last row and group)
    auto load = [&](uint32_t u) {
        Part t;
        const uint32_t tile = u / 2, rt = tile / kt;
        t.row = rt * 32 + (u & 1) * 16 + r;
        t.col = (tile - rt * kt) * 32 + c;
        if (saliency)
#pragma unroll
            for (int h = 0; h < 2; ++h) t.sal[h] = reinterpret_cast<const float4 *>(saliency)[min(t.col + 16 * h, ngroups - 1)];
        const uint32_t o = min(t.row, (uint32_t)n - 1);
        const float4 *const row = reinterpret_cast<const float4 *>(W) + (size_t)o * ngroups;
        t.s = scale_in[o];
#pragma unroll
        for (int h = 0; h < 2; ++h) t.w[h] = row[min(t.col + 16 * h, ngroups - 1)];
        return t;
    };
    uint32_t u = blockIdx.x;
    Part next = load(u);
    for (; u < parts; u += gridDim.x) {
        const Part t = next;
        next = load(min(u + gridDim.x, parts - 1));
        uint8_t *const qt = qvals + (size_t)(u / 2) * 1024 + (u & 1) * 256, *const mt = meta + (size_t)(u / 2) * 512 + (u & 1) * 128;
        const RowScale rs = row_scale(t.s);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint32_t m4 = 0, q = encode_group(t.w[h], rs, &m4, saliency ? t.sal[h] : make_float4(1.f, 1.f, 1.f, 1.f));
            if (t.row >= (uint32_t)n || t.col + 16 * h >= ngroups) q = m4 = 0;           // padding is zero bytes
            const uint32_t other = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m4, 0xB1, 0xF, 0xF, true);     // of lane ^ 1
            qt[threadIdx.x + h * 512] = (uint8_t)q;
            if ((c & 1) == 0) mt[threadIdx.x / 2 + h * 256] = (uint8_t)(m4 | (other << 4));
        }
        if (t.col == 0 && t.row < (uint32_t)n) scale[t.row] = t.s;
    }
}

// One lane decodes one group: 4 codes and 4 mask bytes, one dword store each.
__global__ __launch_bounds__(256) void unpack_kernel(const uint8_t *__restrict__ qvals,
                                                     const uint8_t *__restrict__ meta, int n, int k,
                                                     int8_t *__restrict__ codes, uint8_t *__restrict__ mask)
{
    const uint32_t ngroups = (uint32_t)k / 4, kt = pk_ktiles(k);
    const size_t total_groups = (size_t)n * ngroups;
    for (size_t g = blockIdx.x * (size_t)blockDim.x + threadIdx.x; g < total_groups;
         g += (size_t)gridDim.x * blockDim.x) {
        const uint32_t o = (uint32_t)(g / ngroups), gi = (uint32_t)(g - (size_t)o * ngroups);
        uint32_t q = qvals[pk_qoff(o, gi, kt)];
        uint32_t m4 = (meta[pk_moff(o, gi >> 1, kt)] >> (4 * (gi & 1))) & 0xFu;
        uint32_t i0 = m4 & 3u, i1 = m4 >> 2;
        uint32_t c0 = (uint32_t)nibble_to_int(q & 0xFu) & 0xFFu;
        uint32_t c1 = (uint32_t)nibble_to_int(q >> 4) & 0xFFu;
        // a malformed nibble with i1 == i0 keeps the later write, as a
        // sequential decoder would
        uint32_t cw = (i0 == i1) ? (c1 << (8 * i1)) : ((c0 << (8 * i0)) | (c1 << (8 * i1)));
        uint32_t mw = (1u << (8 * i0)) | (1u << (8 * i1));
        reinterpret_cast<uint32_t *>(codes)[g] = cw;
        reinterpret_cast<uint32_t *>(mask)[g] = mw;
    }
}

// dst (tiled layout of a [rows][kcols] matrix, see slim_internal.h) <- src
// [src_rows][src_cols] row-major, zero outside the source.  One lane per piece
// of 8 halves, pieces in destination order: the stores are contiguous.
__global__ __launch_bounds__(256) void tile_copy_kernel(const uint16_t *__restrict__ src, int src_rows,
                                                        int src_cols, uint16_t *__restrict__ dst, uint32_t rows,
                                                        uint32_t kcols)
{
    const size_t pieces = (size_t)rows * (kcols / 8);
    for (size_t p = blockIdx.x * (size_t)blockDim.x + threadIdx.x; p < pieces;
         p += (size_t)gridDim.x * blockDim.x) {
        const uint32_t tile = (uint32_t)(p >> 6), q = (uint32_t)p & 63u;
        const uint32_t rt = tile / (kcols >> 4), kt = tile - rt * (kcols >> 4);
        const int row = (int)(rt * 32 + (q & 31u));
        const int c0 = (int)(kt * 16 + (q >> 5) * 8);
        uint16_t v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            v[e] = (row < src_rows && c0 + e < src_cols) ? src[(size_t)row * src_cols + c0 + e] : (uint16_t)0;
        uint4_t out;
#pragma unroll
        for (int e = 0; e < 4; ++e) out[e] = (uint32_t)v[2 * e] | ((uint32_t)v[2 * e + 1] << 16);
        reinterpret_cast<uint4_t *>(dst)[p] = out;
    }
}

// Workgroups for slim_pack: one per row up to `cap`, a multiple of 8.
static int pack_grid(int npad, int cap)
{
    int g = npad < cap ? npad : cap;
    return (g + 7) / 8 * 8;
}

static int grid_for(size_t items, int threads, int cap = 256 * 16)
{
    size_t b = (items + threads - 1) / threads;
    if (b > (size_t)cap) b = cap;
    if (b < 1) b = 1;
    return (int)b;
}

}  // namespace slim

using namespace slim;

template <bool EX>
static int launch_pack(const float *W, slim_shape shape, uint8_t *qvals, uint8_t *meta, float *scale,
                       const float *saliency, hipStream_t st)
{
    const int npad = (shape.n + 31) / 32 * 32;      // the padding rows of the last tile get a workgroup too
    // lanes per row: enough that a lane keeps at most 4 groups, 8 from 512 lanes on
    const int groups = shape.k / 4;
    // (two rounds of resident workgroups at most; a workgroup walks the rows it owns)
#define SLIM_PACK_LAUNCH(T, S)                                                                                    \
    hipLaunchKernelGGL((pack_kernel<T, S, EX>), dim3(pack_grid(npad, 256 * (4096 / T))), dim3(T), 0, st, W, shape.n, \
                       shape.k, qvals, meta, scale, saliency)
    if (groups <= 256 * 2)
        SLIM_PACK_LAUNCH(256, 2);
    else if (groups <= 256 * 4)
        SLIM_PACK_LAUNCH(256, 4);
    else if (groups <= 512 * 4)
        SLIM_PACK_LAUNCH(512, 4);
    else if (groups <= 512 * 8)              // (1024 lanes with four groups each: 4096 x 11008 48 and 45 us, with and without saliency, these 42 and 34)
        SLIM_PACK_LAUNCH(512, 8);
    else if (groups <= 1024 * 8)
        SLIM_PACK_LAUNCH(1024, 8);
    else if (groups <= 1024 * kPackSlotsMax)     // (read twice instead, with saliency: 1024 x 32776 42 -> 45 us, up to 49152 the same)
        SLIM_PACK_LAUNCH(1024, kPackSlotsMax);
    else
        SLIM_PACK_LAUNCH(1024, 0);
#undef SLIM_PACK_LAUNCH
    return hip_status(hipGetLastError());
}

extern "C" int slim_pack(const float *W, slim_shape shape, uint8_t *qvals, uint8_t *meta, float *scale,
                         void *stream)
{
    if (!W || !qvals || !meta || !scale) return SLIM_ERR_NULL;
    if (shape.n < 1 || shape.k < 8 || shape.k % 8) return SLIM_ERR_SHAPE;
    if (!aligned16(W) || !aligned16(qvals) || !aligned16(meta) || !aligned16(scale)) return SLIM_ERR_ALIGN;
    return launch_pack<false>(W, shape, qvals, meta, scale, nullptr, static_cast<hipStream_t>(stream));
}

extern "C" int slim_pack_ex(const float *W, slim_shape shape, const float *saliency, const float *scale_in,
                            uint8_t *qvals, uint8_t *meta, float *scale, void *stream)
{
    if (!W || !qvals || !meta || !scale) return SLIM_ERR_NULL;
    if (shape.n < 1 || shape.k < 8 || shape.k % 8) return SLIM_ERR_SHAPE;
    if (!aligned16(W) || !aligned16(qvals) || !aligned16(meta) || !aligned16(scale) || !aligned16(saliency) ||
        !aligned16(scale_in))
        return SLIM_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (!scale_in && !saliency) return launch_pack<false>(W, shape, qvals, meta, scale, nullptr, st);
    if (!scale_in) return launch_pack<true>(W, shape, qvals, meta, scale, saliency, st);
    const size_t tiles = (size_t)((shape.n + 31) / 32) * pk_ktiles(shape.k);
    hipLaunchKernelGGL(pack_scaled_kernel, dim3((unsigned)(2 * tiles < kPackScaledGrid ? 2 * tiles : kPackScaledGrid)), dim3(256), 0, st, W, shape.n, shape.k, saliency, scale_in, qvals, meta, scale);
    return hip_status(hipGetLastError());
}

extern "C" int slim_unpack(const uint8_t *qvals, const uint8_t *meta, slim_shape shape, int8_t *codes,
                           uint8_t *mask, void *stream)
{
    if (!qvals || !meta || !codes || !mask) return SLIM_ERR_NULL;
    if (shape.n < 1 || shape.k < 8 || shape.k % 8) return SLIM_ERR_SHAPE;
    if (!aligned16(qvals) || !aligned16(meta) || !aligned16(codes) || !aligned16(mask)) return SLIM_ERR_ALIGN;
    size_t groups = (size_t)shape.n * (shape.k / 4);
    hipLaunchKernelGGL(unpack_kernel, dim3(grid_for(groups, 256)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), qvals, meta, shape.n, shape.k, codes, mask);
    return hip_status(hipGetLastError());
}

extern "C" int slim_pack_adapters(const slim_half *L, const slim_half *R, slim_shape shape, slim_half *L_pad,
                                  slim_half *R_pad, void *stream)
{
    if (!L || !R || !L_pad || !R_pad) return SLIM_ERR_NULL;
    if (shape.n < 1 || shape.k < 8 || shape.k % 8 || shape.rank < 1) return SLIM_ERR_SHAPE;
    if (!aligned16(L_pad) || !aligned16(R_pad)) return SLIM_ERR_ALIGN;
    int rp = slim_rank_pad(shape.rank);
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(tile_copy_kernel, dim3(grid_for(tl_bytes(shape.n, rp) / 16, 256)), dim3(256), 0, st, L, shape.n,
                       shape.rank, L_pad, tl_rows(shape.n), tl_cols(rp));
    hipLaunchKernelGGL(tile_copy_kernel, dim3(grid_for(tl_bytes(rp, shape.k) / 16, 256)), dim3(256), 0, st, R,
                       shape.rank, shape.k, R_pad, tl_rows(rp), tl_cols(shape.k));
    return hip_status(hipGetLastError());
}
