// Compositing with BF16 features on MFMA (gfx950), FP32 accumulation.
//
// The feature part of the forward pass is a dense contraction per tile:
//   F[256 px x D] += W[256 px x K] . Feat[K x D]     (w = alpha T, Section 3.1)
// computed with v_mfma_f32_16x16x32_bf16.  W is split into two BF16 terms,
// W = hi + lo (hi = bf16(w), lo = bf16(w - hi)), so the product keeps about 16
// bits of w; the features are BF16 already.  Everything else (alpha, the
// transmittance walk, colour) stays on the VALU in FP32.
//
// SURF: the surfel primitive (Section 3.1): four-float4 records, alpha at the
// ray-plane intersection; the rest is the same.
//
// Work mapping: one workgroup per (tile, group of ROWS pixel rows, channel
// slice of DS); wave w is pixel row w of its group; lane l handles pixel
// x = l % 16 and Gaussians 8 (l / 16) .. 8 (l / 16) + 7 of each 32-Gaussian
// chunk.  The lane's eight weights are exactly its MFMA A-operand (rows =
// pixels, k = Gaussians).  The four lanes of a pixel combine their
// transmittance with an exclusive product scan, which reproduces the sequential
// walk (skip rule, stop rule) up to rounding.  Features lie in LDS as they come,
// a position's channels in a row, and reach the B operand by transposed reads
// (writing them transposed took 16 two-byte stores a thread and chunk).
//
// Bound: VALU of the walk (62 % of the issue slots at 256 channels, matrix cores
// 18 %), then the store of F.  256 channels, 500k Gaussians, 1920x1080, BF16 form:
// 1.13 -> 0.79 ms, of which 0.34 is F at the HBM rate: a branch-free walk (1.13 ->
// 1.02), four-row workgroups at three a CU with barriers of their own instead of
// one of eight rows (0.86), and one multiply a feature row's address (0.79);
// surfels 1.30 -> 0.88 ms; 128 channels, 1M Gaussians, 16 views 5.75 -> 4.75 ms.
#include <type_traits>

#include "kernels.hpp"

namespace fh {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int FK = 32;        // Gaussians per chunk

// LDS row of list position k of a chunk: positions 8 q + m (m < 4) in rows 4 q + m,
// the others 16 rows on, so that the four lane groups of one transposed read take
// sixteen consecutive rows (an odd multiple of 32 bytes apart: no bank conflicts).
__device__ __forceinline__ int feat_row(int k) { return (k & 3) | ((k >> 1) & 12) | ((k & 4) << 2); }

// Four rows (positions) by sixteen 16-bit columns (channels) per group of
// sixteen lanes: lane i of a group gives the address of columns 4 (i % 4) of row
// i / 4 and receives column i of the four rows.
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
__device__ __forceinline__ bf16x8 read_tr(const unsigned char* at, int rows16) {
    const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)at));
    const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(at + rows16)));
    return __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
}

// Two values rounded to BF16 (to nearest even), packed; and back.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ float lo_f32(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float hi_f32(uint32_t p) { return __uint_as_float(p & 0xFFFF0000u); }

// Software pipeline over the tile's chunks of FK list positions.  While chunk
// c is composited, threads 0..FK-1 hold in registers the list entries (depth
// ranks) of chunk c+3 and the records and Gaussians of chunk c+2 (one load each,
// from the rank-ordered records), and every thread holds its share of chunk
// c+1's features.  All of them are requested at the top of the chunk and only
// stored to LDS at its end, so no global latency sits between two chunks.
// Records and Gaussians are triple-buffered in LDS, features double-buffered.
constexpr uint32_t BUF_DWORD3 = 0x00020000u;   // raw buffer, 32-bit data format

__device__ __forceinline__ uint32_t list_load(__amdgpu_buffer_rsrc_t rs, uint32_t pos) {
    return __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(pos * 4u), 0, 0);
}

// FS: FP32 features (the FP32 form).  Weights and features are each split
// into three BF16 terms (x = h + m + l, h = bf16(x), m = bf16(x - h),
// l = bf16(x - h - m)) and F takes the six products hh, hm, mh, hl, lh, mm:
// what is left out is below 2^-24 of w f, so F keeps FP32 accuracy on MFMA.
template <int DS, int ROWS, bool FS, bool SURF>
// (shapes up to 128 channels keep four waves per SIMD, 4-row ones of 256 three:
// several workgroups per CU, each with its own barriers)
__global__ __launch_bounds__(64 * ROWS, (ROWS <= 8 && DS <= 128 && !FS) ? 4 : (ROWS == 4 ? 3 : 1)) void k_render_fwd_bf16(
    RenderArgs a, ViewTable vt) {
    constexpr int NB = DS / 16;
    static_assert(NB % 2 == 0, "channel blocks are processed in pairs");
    constexpr int NT = 64 * ROWS;                        // threads
    constexpr int NIT = (FK * (DS / 8) + NT - 1) / NT;   // feature items per thread
    constexpr int RG = 8;                                 // record padding group (lanes read records 8 apart)
    using RecT = typename PrimRec<SURF>::T;
    constexpr int RW = PrimRec<SURF>::RW;                 // float4 per record
    __shared__ float4 srec4[3][RW * FK + FK / RG];
    __shared__ uint32_t sg[3][FK];
    constexpr int NFT = FS ? 3 : 1;                       // feature tiles: h (+ m, l)
    constexpr int NFR = FS ? 2 * NIT : NIT;               // 16-byte registers of one chunk's feature items
    constexpr int FROW = 2 * DS + 32, FT = FK * FROW;     // bytes of a position's row, and of a feature tile
    __shared__ __attribute__((aligned(16))) unsigned char sft[2][NFT * FT];
    __shared__ uint32_t smax[ROWS], sodd;
    __shared__ __attribute__((aligned(16))) uint8_t sbusy[2][16];   // per wave: a pixel still walking
    if (a.counters->inst_overflow) return;
    constexpr int NG = TILE / ROWS;                      // row groups per tile
    const int t = a.tile_order ? (int)a.tile_order[blockIdx.x] : (int)blockIdx.x;
    const int grp = blockIdx.y % NG, slice = blockIdx.y / NG, d0 = slice * DS;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int q = lane >> 4, xi = lane & 15;
    const int v = view_of_tile(vt, t);
    const int lt = t - vt.tile_off[v];
    const int tx = lt % vt.tiles_x[v], ty = lt / vt.tiles_x[v];
    const int px = tx * TILE + xi, py = ty * TILE + grp * ROWS + w;
    const bool inside = px < vt.width[v] && py < vt.height[v];
    const float x = (float)px + 0.5f, y = (float)py + 0.5f;
    const uint32_t s = a.ranges[2 * t], e = a.ranges[2 * t + 1];
    const uint32_t len = e - s;
    const uint16_t* feat = static_cast<const uint16_t*>(a.feat);
    // the tile's list as a range-checked buffer: positions past its end read 0
    // (rank 0, a valid index; such positions become padding when stored)
    const uint32_t* list = a.packed ? a.keys : a.vals;
    const __amdgpu_buffer_rsrc_t list_rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t*>(list + s), (short)0, (int)(len < 0x1fffffffu ? len * 4u : 0x7ffffffcu), BUF_DWORD3);
    const uint32_t rmask = a.packed ? ((1u << a.rank_bits) - 1u) : 0xFFFFFFFFu;
    const int k = (int)threadIdx.x;   // list position within a chunk (threads 0..FK-1)

    auto put_rec = [&](int buf, uint32_t pos, const RecT& r, uint32_t g) {
        const bool real = pos < len;
        // padding: opacity 0 never blends
        RecT o = real ? r : pad_rec<SURF>();
        // (an infinite colour enters the branch-free sums as zero, 0 * inf must not
        // reach the pixels that do not blend it, and is added at the end; the
        // projection leaves no NaN and nothing negative)
        const float INF = __builtin_inff();
        if (fmaxf(fmaxf(o.r2.y, o.r2.z), o.r2.w) == INF) {
            sodd = 1u;
            o.r2.y = o.r2.y == INF ? 0.0f : o.r2.y;
            o.r2.z = o.r2.z == INF ? 0.0f : o.r2.z;
            o.r2.w = o.r2.w == INF ? 0.0f : o.r2.w;
        }
        lds_put_prec<SURF, RG>(srec4[buf], k, o);
        sg[buf][k] = real ? g : 0u;
    };
    // e: a raw list entry (masked here, where it is used, so that its load is
    // not waited for where it is issued)
    auto get_rec = [&](uint32_t e, RecT& r, uint32_t& g) {
        const uint32_t j = e & rmask;
        r = load_rec<SURF>(a.rrec, j);
        g = a.order[j];
    };
    // feature items of one chunk, 8 channels each, the channels of a position
    // consecutive; padding positions read Gaussian 0 and are zeroed when stored
    auto load_feats = [&](const uint32_t* gl, u32x4* fr) {
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int idx = (int)threadIdx.x + NT * it;
            if ((it + 1) * NT <= FK * (DS / 8) || idx < FK * (DS / 8)) {
                const int kk = idx / (DS / 8), dg = idx % (DS / 8);
                const uint64_t row = (uint64_t)gl[kk] * (uint32_t)a.d;
                if constexpr (FS) {
                    const u32x4* src =
                        reinterpret_cast<const u32x4*>(static_cast<const float*>(a.feat) + row + (d0 + dg * 8));
                    fr[2 * it] = src[0];
                    fr[2 * it + 1] = src[1];
                } else {
                    fr[it] = *reinterpret_cast<const u32x4*>(feat + row + (d0 + dg * 8));
                }
            }
        }
    };
    auto store_items = [&](auto whole, uint32_t pos, const u32x4* fr, unsigned char* dst) {
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int idx = (int)threadIdx.x + NT * it;
            if ((it + 1) * NT <= FK * (DS / 8) || idx < FK * (DS / 8)) {
                const int kk = idx / (DS / 8), dg = idx % (DS / 8);
                const bool pad = !decltype(whole)::value && pos + (uint32_t)kk >= len;
                unsigned char* row = dst + feat_row(kk) * FROW + 16 * dg;
                const u32x4 none = u32x4{0u, 0u, 0u, 0u};
                if constexpr (FS) {
                    u32x4 h, m, l;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const u32x4 f = pad ? none : fr[2 * it + e / 2];
                        const float x0 = __uint_as_float(f[2 * (e % 2)]), x1 = __uint_as_float(f[2 * (e % 2) + 1]);
                        h[e] = pack_bf16(x0, x1);
                        const float r0 = x0 - lo_f32(h[e]), r1 = x1 - hi_f32(h[e]);
                        m[e] = pack_bf16(r0, r1);
                        l[e] = pack_bf16(r0 - lo_f32(m[e]), r1 - hi_f32(m[e]));
                    }
                    *reinterpret_cast<u32x4*>(row) = h;
                    *reinterpret_cast<u32x4*>(row + FT) = m;
                    *reinterpret_cast<u32x4*>(row + 2 * FT) = l;
                } else {
                    *reinterpret_cast<u32x4*>(row) = pad ? none : fr[it];
                }
            }
        }
    };

    // (pos: the chunk's first list position; only the last chunk holds padding)
    auto store_feats = [&](uint32_t pos, const u32x4* fr, unsigned char* dst) {
        if (pos + FK <= len)
            store_items(std::true_type{}, pos, fr, dst);
        else
            store_items(std::false_type{}, pos, fr, dst);
    };

    // prologue: chunks 0 and 1 into LDS, chunk 2's ranks into registers, then chunk 0's features
    uint32_t rk2 = 0u;
    if (threadIdx.x == 0) sodd = 0u;   // (set by the same wave)
    if (k < FK && len > 0) {
        const uint32_t j0 = list_load(list_rs, (uint32_t)k);
        const uint32_t j1 = list_load(list_rs, (uint32_t)(FK + k));
        rk2 = list_load(list_rs, (uint32_t)(2 * FK + k));
        RecT r0, r1;
        uint32_t g0, g1;
        get_rec(j0, r0, g0);
        get_rec(j1, r1, g1);
        put_rec(0, (uint32_t)k, r0, g0);
        put_rec(1, (uint32_t)(FK + k), r1, g1);
    }
    if (threadIdx.x < 32) reinterpret_cast<uint8_t*>(sbusy)[threadIdx.x] = 0;
    __syncthreads();
    if (len > 0) {   // (an empty list stages nothing: sg holds no Gaussians then)
        u32x4 fr[NFR];
        load_feats(sg[0], fr);
        store_feats(0u, fr, sft[0]);
    }
    __syncthreads();

    f32x4 acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float T = 1.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
    bool done = !inside;
    uint32_t last = 0;

    int b3 = 0, b2 = 0;   // chunk index mod 3 and mod 2
    for (uint32_t cpos = 0; cpos < len; cpos += FK) {
        const int n3 = b3 == 2 ? 0 : b3 + 1, nn3 = n3 == 2 ? 0 : n3 + 1;
        // chunk c+2's records and Gaussians, chunk c+3's ranks, chunk c+1's features: all in flight now
        RecT r2;
        uint32_t g2 = 0u, rk3 = 0u;
        if (k < FK) {
            get_rec(rk2, r2, g2);
            rk3 = list_load(list_rs, cpos + (uint32_t)(3 * FK + k));
        }
        u32x4 fr[NFR];
        load_feats(sg[n3], fr);

        // alpha of this lane's eight Gaussians (zero where they do not blend, and in
        // a pixel that has stopped) and their transmittance product
        const float least = done ? 2.0f : ALPHA_MIN;
        float al[8];
        float P = 1.0f;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const float alpha = prim_alpha<SURF>(lds_prec<SURF, RG>(srec4[b3], 8 * q + m), x, y);
            al[m] = alpha >= least ? alpha : 0.0f;
            P *= (1.0f - al[m]);
        }
        const Rows4 Pr = rows4(P);
        float excl = q > 0 ? Pr.r0 : 1.0f;
        excl = q > 1 ? excl * Pr.r1 : excl;
        excl = q > 2 ? excl * Pr.r2 : excl;
        // The walk.  Tv runs on past the stop (it never rises again), so that a
        // Gaussian blends exactly where Tv behind it is at least T_MIN; Tl stays at
        // the last such value.  W (this lane's 8 weights) goes straight into its
        // MFMA A operand as BF16 hi + lo (FS: three terms).
        float Tl = T * excl, Tv = Tl;
        const bool open = Tl >= T_MIN;
        uint32_t mylast = 0;
        u32x4 whi, wlo, wmid;
        auto colour = [&](int m) { return srec4[b3][prec_slot<SURF, RG>(8 * q + m) + 2]; };   // (opacity, r, g, b)
        float4 col[2] = {colour(0), colour(1)};
#pragma unroll
        for (int m = 0; m < 8; m += 2) {
            float4 next[2];
            if (m < 6) {
                next[0] = colour(m + 2);
                next[1] = colour(m + 3);
            }
            float wv[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const float Tn = Tv * (1.0f - al[m + e]);
                const bool on = Tn >= T_MIN;
                wv[e] = on ? al[m + e] * Tv : 0.0f;
                Tl = on ? Tn : Tl;
                Tv = Tn;
                c0 = __builtin_fmaf(wv[e], col[e].y, c0);
                c1 = __builtin_fmaf(wv[e], col[e].z, c1);
                c2 = __builtin_fmaf(wv[e], col[e].w, c2);
                mylast = wv[e] > 0.0f ? cpos + 8 * q + m + e + 1 : mylast;
            }
            uint32_t h = pack_bf16(wv[0], wv[1]);
            const float r0 = wv[0] - lo_f32(h), r1 = wv[1] - hi_f32(h);
            uint32_t r = pack_bf16(r0, r1);
            if constexpr (FS) {
                wmid[m / 2] = r;
                r = pack_bf16(r0 - lo_f32(r), r1 - hi_f32(r));
            }
            // (in order: the next pair's colours in flight, no more held)
            asm volatile("" : "+v"(Tv), "+v"(c0), "+v"(c1), "+v"(c2), "+v"(h), "+v"(r), "+v"(mylast)::"memory");
            whi[m / 2] = h;
            wlo[m / 2] = r;
            col[0] = next[0];
            col[1] = next[1];
        }
        const bf16x8 ahi = __builtin_bit_cast(bf16x8, whi), alo = __builtin_bit_cast(bf16x8, wlo);
        // pixel state after the chunk: the first lane that stopped (its sign), else lane 3
        const Rows4 Tr = rows4(open && Tv < T_MIN ? -Tl : Tl);
        if (!done) {
            T = fabsf(Tr.r0 < 0.0f ? Tr.r0 : (Tr.r1 < 0.0f ? Tr.r1 : (Tr.r2 < 0.0f ? Tr.r2 : Tr.r3)));
            done = fminf(fminf(Tr.r0, Tr.r1), fminf(Tr.r2, Tr.r3)) < 0.0f;
            // A lane starts from T times the product of the lanes before it, which
            // may round below T_MIN where the lane before ended at or above it by its
            // own sequence of products.  Then no lane carries the stop's sign: the
            // pixel stopped there, with the T of the last open lane.  (One pixel in 10
            // to 100 million; its T came out as a product over Gaussians that never
            // blended, 0 to 1e-32 for 1e-4, and with it gradients off by 1e-3 of their
            // norm at 800x800.)
            if (T < T_MIN) {
                T = Tr.r2 >= T_MIN ? Tr.r2 : (Tr.r1 >= T_MIN ? Tr.r1 : Tr.r0);
                done = true;
            }
        }
        const Rows4 Lr = rows4(__uint_as_float(mylast));
        const uint32_t lm = max(max(__float_as_uint(Lr.r0), __float_as_uint(Lr.r1)),
                                max(__float_as_uint(Lr.r2), __float_as_uint(Lr.r3)));
        last = max(last, lm);

        // W times the feature chunk (channel blocks in pairs, so that the hi and
        // lo products of one block are not issued back to back)
#pragma unroll
        for (int j = 0; j < NB; j += 2) {
            if (j % 4 == 0) asm volatile("" ::: "memory");
            const unsigned char* fb = sft[b2] + (4 * q + (xi >> 2)) * FROW + 32 * j + 8 * (xi & 3);
            const bf16x8 bv0 = read_tr(fb, 16 * FROW), bv1 = read_tr(fb + 32, 16 * FROW);
            if constexpr (FS) {
                // the six products, smallest first: lh, hl, mm, mh, hm, hh
                const bf16x8 amid = __builtin_bit_cast(bf16x8, wmid);
                const bf16x8 bm0 = read_tr(fb + FT, 16 * FROW), bm1 = read_tr(fb + FT + 32, 16 * FROW);
                const bf16x8 bl0 = read_tr(fb + 2 * FT, 16 * FROW), bl1 = read_tr(fb + 2 * FT + 32, 16 * FROW);
                f32x4 s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo, bv0, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                f32x4 s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo, bv1, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, bl0, s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, bl1, s1, 0, 0, 0);
                s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(amid, bm0, s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(amid, bm1, s1, 0, 0, 0);
                s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(amid, bv0, s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(amid, bv1, s1, 0, 0, 0);
                s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, bm0, s0, 0, 0, 0);
                s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, bm1, s1, 0, 0, 0);
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, bv0, acc[j] + s0, 0, 0, 0);
                acc[j + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, bv1, acc[j + 1] + s1, 0, 0, 0);
            } else {
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, bv0, acc[j], 0, 0, 0);
                acc[j + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, bv1, acc[j + 1], 0, 0, 0);
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo, bv0, acc[j], 0, 0, 0);
                acc[j + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo, bv1, acc[j + 1], 0, 0, 0);
            }
        }
        // chunk c+1's features and chunk c+2's records to LDS
        store_feats(cpos + FK, fr, sft[b2 ^ 1]);
        if (k < FK) {
            put_rec(nn3, cpos + (uint32_t)(2 * FK + k), r2, g2);
            rk2 = rk3;
        }
        // leave when every pixel of the workgroup has stopped (flags double-buffered by chunk parity)
        const bool wave_busy = ballot64(!done) != 0;   // (all lanes vote, outside the lane-0 store)
        if (lane == 0) sbusy[b2][w] = wave_busy ? 1 : 0;
        __syncthreads();
        const uint4 bz = *reinterpret_cast<const uint4*>(sbusy[b2]);
        if ((bz.x | bz.y | bz.z | bz.w) == 0u) break;
        b3 = n3;
        b2 ^= 1;
    }

    // colour: the four lanes of a pixel hold partial sums
    c0 += __shfl_xor(c0, 16, 64);
    c0 += __shfl_xor(c0, 32, 64);
    c1 += __shfl_xor(c1, 16, 64);
    c1 += __shfl_xor(c1, 32, 64);
    c2 += __shfl_xor(c2, 16, 64);
    c2 += __shfl_xor(c2, 32, 64);
    const int64_t rowp = vt.pix_off[v] + (int64_t)py * vt.width[v];
    // F: lane holds F[pixel 4q + r of this row][channel 16 j + xi]
    if (py < vt.height[v]) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int pxr = tx * TILE + 4 * q + r;
            if (pxr < vt.width[v]) {
                float* fo = a.F + (rowp + pxr) * a.d + d0 + xi;
#pragma unroll
                for (int j = 0; j < NB; ++j) fo[16 * j] = acc[j][r];
            }
        }
    }
    if (slice == 0 && q == 0 && inside) {
        if (sodd != 0u) {   // (rare: infinite colours, by a second walk; up to the last blend every alpha of 1/255 blends)
            for (uint32_t pos = 0; pos < last; ++pos) {
                const RecT r = load_rec<SURF>(a.rrec, list[s + pos] & rmask);
                if (prim_alpha<SURF>(r, x, y) < ALPHA_MIN) continue;
                c0 = r.r2.y == __builtin_inff() ? r.r2.y : c0;
                c1 = r.r2.z == __builtin_inff() ? r.r2.z : c1;
                c2 = r.r2.w == __builtin_inff() ? r.r2.w : c2;
            }
        }
        const int64_t p = rowp + px;
        a.C[3 * p] = c0;
        a.C[3 * p + 1] = c1;
        a.C[3 * p + 2] = c2;
        a.T[p] = T;
        a.n_iter[p] = last;
    }
    if (slice == 0) {
        // the tile's traversal length: max over its row groups (tile_niter is
        // zeroed before the launch)
        const uint32_t m = wave_max_u32(last);
        if (lane == 0) smax[w] = m;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t mm = 0;
            for (int k = 0; k < ROWS; ++k) mm = smax[k] > mm ? smax[k] : mm;
            if (NG == 1)
                a.tile_niter[t] = mm;
            else
                atomicMax(&a.tile_niter[t], mm);
        }
    }
}

bool render_fwd_bf16_shape_ok(int d, int slice, int rows) {
    if (rows == 16) return (slice == 32 || slice == 64 || slice == 96 || slice == 128) && d % slice == 0;
    if (rows == 8) return (slice == 64 || slice == 128 || slice == 256) && d % slice == 0;
    if (rows == 4) return (slice == 128 || slice == 256) && d % slice == 0;
    return false;
}

template <bool FS, bool SURF>
static void launch_fwd_mfma(const RenderArgs& a, const ViewTable& vt, int n_tiles, int slice, int rows, hipStream_t s) {
    // slice and rows form a valid shape for d (checked by the caller)
    const unsigned ns = (unsigned)(a.d / slice);
    const dim3 g16(n_tiles, ns), g8(n_tiles, 2 * ns), g4(n_tiles, 4 * ns);
    if (rows == 4) {
        // (BF16-stored features only)
        if constexpr (!FS) {
            if (slice == 128)
                hipLaunchKernelGGL((k_render_fwd_bf16<128, 4, false, SURF>), g4, dim3(256), 0, s, a, vt);
            else
                hipLaunchKernelGGL((k_render_fwd_bf16<256, 4, false, SURF>), g4, dim3(256), 0, s, a, vt);
        }
        return;
    }
    if (rows == 8) {
        switch (slice) {
            case 64: hipLaunchKernelGGL((k_render_fwd_bf16<64, 8, FS, SURF>), g8, dim3(512), 0, s, a, vt); break;
            case 128: hipLaunchKernelGGL((k_render_fwd_bf16<128, 8, FS, SURF>), g8, dim3(512), 0, s, a, vt); break;
            default:
                // (BF16 features: two workgroups of four rows instead of one of eight, three
                // a CU instead of one: 0.79 against 1.02 ms at 500k, 1920x1080; FP32
                // features, three LDS tiles of 17 KB each, stay at eight)
                if constexpr (FS)
                    hipLaunchKernelGGL((k_render_fwd_bf16<256, 8, true, SURF>), g8, dim3(512), 0, s, a, vt);
                else
                    hipLaunchKernelGGL((k_render_fwd_bf16<256, 4, false, SURF>), g4, dim3(256), 0, s, a, vt);
                break;
        }
        return;
    }
    // 16 rows: one workgroup at 128 channels; narrower slices in four of four rows,
    // whose records and features are cheap to stage four times and whose list
    // latencies overlap (32 channels at 637x479 95 -> 72 us, 64 FP32 channels at
    // 800x800 243 -> 202 us against one workgroup of 16 waves)
    switch (slice) {
        case 32: hipLaunchKernelGGL((k_render_fwd_bf16<32, 4, FS, SURF>), g4, dim3(256), 0, s, a, vt); break;
        case 64: hipLaunchKernelGGL((k_render_fwd_bf16<64, 4, FS, SURF>), g4, dim3(256), 0, s, a, vt); break;
        case 96: hipLaunchKernelGGL((k_render_fwd_bf16<96, 4, FS, SURF>), g4, dim3(256), 0, s, a, vt); break;
        default:
            // (16 rows of 128 channels is not an FP32-feature shape: it would spill)
            if constexpr (!FS) hipLaunchKernelGGL((k_render_fwd_bf16<128, 16, false, SURF>), g16, dim3(1024), 0, s, a, vt);
            break;
    }
}

// BF16 features enter the MFMA as stored; FP32 features (fsplit) as three terms.
// Surfels (a.prim): BF16 features only.
void launch_render_fwd_bf16(const RenderArgs& a, const ViewTable& vt, int n_tiles, int slice, int rows, bool fsplit,
                            hipStream_t s) {
    if (a.prim == FH_PRIM_SURFEL)
        launch_fwd_mfma<false, true>(a, vt, n_tiles, slice, rows, s);
    else if (fsplit)
        launch_fwd_mfma<true, false>(a, vt, n_tiles, slice, rows, s);
    else
        launch_fwd_mfma<false, false>(a, vt, n_tiles, slice, rows, s);
}

}  // namespace fh
