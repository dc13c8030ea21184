// Adjoint of the compositing pass, both arithmetic forms (gfx950).
//
// Per tile, back to front over the tile's visited list (Appendix A.2:
// dL/dalpha_k = T_k g_k - (S_k + T_final dT)/(1 - alpha_k), S_k = sum_{i>k} w_i
// g_i, g_k = rgb_k . dC + f_k . dF), in chunks of 16 positions.  One workgroup
// of four waves per tile; a wave owns four pixel rows and runs on its own (its
// records, features and weights never leave it), except for one barrier a
// chunk where the four waves' sums per position are added.  Per chunk:
//   1. g for the wave's 64 pixels is a contraction over channels and colour,
//      G^T[16 x 64] = [Feat | rgb][16 x (D + 3)] . [dF | dC]^T[(D + 3) x 64], with
//      dF resident in registers for the whole tile.  FP32 form: FP32 operands on
//      v_mfma_f32_16x16x4_f32.  BF16 form: BF16 features as stored, dF as two
//      BF16 terms hi + lo (about 16 significant bits) on
//      v_mfma_f32_16x16x32_bf16; the colour part in FP32 in both.  The result
//      is turned from (position, pixel row) to (pixel, position) order by lane
//      swaps, so that
//   2. each lane walks its own pixel sequentially: T and S need no scan over
//      lanes.  The chunk's records live one position per lane and reach the walk
//      as DPP row broadcasts inside its arithmetic instructions, without loads;
//   3. (w, dL/dpower) pairs cross through LDS of the wave, and a pass with one
//      position per lane sums the screen-space terms over the wave's pixels
//      (dC again by row broadcast).
//
// Order of the arithmetic.  The moments of a Gaussian near the camera cancel to
// 1e-4 of their size, so that its scale and rotation gradients show every
// rounding of these sums.  The BF16 form keeps one fixed order whatever the
// split over lanes: T divided by products of four (1 - alpha), row sums left to
// right, rows in pairs, the eight pairs in order; its gradients are bit for bit
// those of a walk split over four lanes a pixel.
//
// What bounds it: VALU work per (pixel, position), about 45 instructions (a
// walk split over four lanes per pixel with scans took 90 in the BF16 form and
// 131 in the FP32 form); at 256 channels in the FP32 form also the matrix rate.
// Measured against that walk: BF16 form, 128 channels, 1M Gaussians, 16 views,
// 10.82 -> 6.67 ms; 256 channels, 500k, 1920x1080, 1.49 -> 1.27 ms (k_dot 0.71);
// FP32 form there, fusion included, 25.6 -> 2.23 ms; no features, 987x657,
// 914 -> 180 us.
//
// SURF: the surfel primitive (Section 3.1): four-float4 records, the density at
// the ray-plane intersection, 14 terms per instance in rows of 16 floats.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "kernels.hpp"

namespace fh {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int CK = 16;          // positions per chunk
// (w, dL/dpower) pairs of a wave, pixel-major in rows of 17 pairs: the walk's
// stores (34 dwords apart) and the position-parallel reads both fall in
// distinct banks
constexpr int WST = CK + 1;

// Value of lane K of the lane's 16-lane row, for use as a DPP operand.
template <int K>
__device__ __forceinline__ float row_bcast(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + K, 0xf, 0xf, true));
}
template <int K>
__device__ __forceinline__ Rec bcast_rec(const Rec& r) {
    Rec o;
    o.r0 = make_float4(row_bcast<K>(r.r0.x), row_bcast<K>(r.r0.y), row_bcast<K>(r.r0.z), row_bcast<K>(r.r0.w));
    o.r1 = make_float4(row_bcast<K>(r.r1.x), row_bcast<K>(r.r1.y), row_bcast<K>(r.r1.z), row_bcast<K>(r.r1.w));
    o.r2 = make_float4(row_bcast<K>(r.r2.x), 0.f, 0.f, 0.f);   // (the colour enters through the contraction)
    return o;
}
template <int K>
__device__ __forceinline__ SRec bcast_rec(const SRec& r) {
    SRec o;
    o.r0 = make_float4(row_bcast<K>(r.r0.x), row_bcast<K>(r.r0.y), row_bcast<K>(r.r0.z), row_bcast<K>(r.r0.w));
    o.r1 = make_float4(row_bcast<K>(r.r1.x), row_bcast<K>(r.r1.y), row_bcast<K>(r.r1.z), row_bcast<K>(r.r1.w));
    o.r2 = make_float4(row_bcast<K>(r.r2.x), 0.f, 0.f, 0.f);
    o.r3 = make_float4(row_bcast<K>(r.r3.x), row_bcast<K>(r.r3.y), row_bcast<K>(r.r3.z), 0.f);
    return o;
}

template <int... Ks, typename Fn>
__device__ __forceinline__ void unroll_seq(std::integer_sequence<int, Ks...>, Fn f) {
    (f(std::integral_constant<int, Ks>{}), ...);
}

struct Pair {
    float a, b;
};
// upper half of a with lower half of b: (a0 a1 b0 b1), (a2 a3 b2 b3) by lane rows
__device__ __forceinline__ Pair swap32(float a, float b) {
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return Pair{__uint_as_float(s[0]), __uint_as_float(s[1])};
}
// odd rows of a with even rows of b: (a0 b0 a2 b2), (a1 b1 a3 b3)
__device__ __forceinline__ Pair swap16(float a, float b) {
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return Pair{__uint_as_float(s[0]), __uint_as_float(s[1])};
}
// Four values summed over the four lane rows at once: lane row q returns the
// sum of value (0, 2, 1, 3)[q].
__device__ __forceinline__ float reduce4(float a, float b, float c, float d) {
    const Pair ab = swap32(a, b), cd = swap32(c, d);
    const Pair x = swap16(ab.a + ab.b, cd.a + cd.b);
    return x.a + x.b;
}

// Two values summed over pairs of lane rows: lane row q returns value q % 2 of
// rows 2 (q / 2) and 2 (q / 2) + 1.
__device__ __forceinline__ float reduce2(float a, float b) {
    const Pair x = swap16(a, b);
    return x.a + x.b;
}

// 1 / x to within one rounding (one Newton step): the FP32 form carries T from
// position to position by it, so that its error is summed along a pixel's walk.
__device__ __forceinline__ float rcp1(float x) {
    const float r = __builtin_amdgcn_rcpf(x);
    return __builtin_fmaf(__builtin_fmaf(-x, r, 1.0f), r, r);
}

// Rows of four channels from c (zeros past d): one load where the rows allow
// it (vec), else element by element.
__device__ __forceinline__ float4 load_row4(const float* p, int c, int d, bool vec) {
    if (vec) return c < d ? *reinterpret_cast<const float4*>(p + c) : make_float4(0.f, 0.f, 0.f, 0.f);
    return make_float4(c < d ? p[c] : 0.f, c + 1 < d ? p[c + 1] : 0.f, c + 2 < d ? p[c + 2] : 0.f,
                       c + 3 < d ? p[c + 3] : 0.f);
}
__device__ __forceinline__ uint2 load_row4h(const uint16_t* p, int c, int d, bool vec) {
    if (vec) return c < d ? *reinterpret_cast<const uint2*>(p + c) : make_uint2(0u, 0u);
    const uint32_t e0 = c < d ? p[c] : 0u, e1 = c + 1 < d ? p[c + 1] : 0u;
    const uint32_t e2 = c + 2 < d ? p[c + 2] : 0u, e3 = c + 3 < d ? p[c + 3] : 0u;
    return make_uint2(e0 | (e1 << 16), e2 | (e3 << 16));
}

// Operands of the feature contraction.  FP32 form: NS slabs of 16 channels,
// lane (q, xi) holding channels 16 s + 4 q .. + 3 of pixel or position xi; FB:
// features stored in BF16.  BF16 form: NS slabs of 32, channels 32 s + 8 q .. + 7.
template <bool BF16, bool FB, int NS>
struct Operands;

template <bool FB, int NS>
struct Operands<false, FB, NS> {
    static constexpr int DC = 16 * NS;
    using FT = typename std::conditional<FB, uint2, float4>::type;
    FT f[NS];
    float4 df[4][NS];
    __device__ __forceinline__ void load_df(int h, const float* row, bool inside, int c0, int q, int d, int vec) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
            df[h][s] = inside ? load_row4(row, c0 + 16 * s + 4 * q, d, vec != 0) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __device__ __forceinline__ void load_feat(const void* feat, int64_t g, int c0, int q, int d, int vec) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int c = c0 + 16 * s + 4 * q;
            if constexpr (FB)
                f[s] = load_row4h(static_cast<const uint16_t*>(feat) + g * d, c, d, vec != 0);
            else
                f[s] = load_row4(static_cast<const float*>(feat) + g * d, c, d, vec != 0);
        }
    }
    __device__ __forceinline__ void contract(f32x4* gk) const {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            float4 a;
            if constexpr (FB)
                a = make_float4(__uint_as_float(f[s].x << 16), __uint_as_float(f[s].x & 0xFFFF0000u),
                                __uint_as_float(f[s].y << 16), __uint_as_float(f[s].y & 0xFFFF0000u));
            else
                a = f[s];
#pragma unroll
            for (int h = 0; h < 4; ++h) gk[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, df[h][s].x, gk[h], 0, 0, 0);
#pragma unroll
            for (int h = 0; h < 4; ++h) gk[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, df[h][s].y, gk[h], 0, 0, 0);
#pragma unroll
            for (int h = 0; h < 4; ++h) gk[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, df[h][s].z, gk[h], 0, 0, 0);
#pragma unroll
            for (int h = 0; h < 4; ++h) gk[h] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, df[h][s].w, gk[h], 0, 0, 0);
        }
    }
};
template <bool FB, int NS>
struct Operands<true, FB, NS> {
    static constexpr int DC = 32 * NS;
    uint4 f[NS];
    bf16x8 hi[4][NS], lo[4][NS];
    __device__ __forceinline__ void load_df(int h, const float* row, bool inside, int c0, int q, int, int) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a;
            if (inside) {
                const float4* src = reinterpret_cast<const float4*>(row + c0 + 32 * s + 8 * q);
                a = src[0];
                b = src[1];
            }
            const float v[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                const __bf16 hb = (__bf16)v[m];
                hi[h][s][m] = hb;
                lo[h][s][m] = (__bf16)(v[m] - (float)hb);
            }
        }
    }
    __device__ __forceinline__ void load_feat(const void* feat, int64_t g, int c0, int q, int d, int) {
        const uint16_t* row = static_cast<const uint16_t*>(feat) + g * d + c0 + 8 * q;
#pragma unroll
        for (int s = 0; s < NS; ++s) f[s] = *reinterpret_cast<const uint4*>(row + 32 * s);
    }
    __device__ __forceinline__ void contract(f32x4* gk) const {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const bf16x8 a = __builtin_bit_cast(bf16x8, f[s]);
#pragma unroll
            for (int h = 0; h < 4; ++h) gk[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, hi[h][s], gk[h], 0, 0, 0);
#pragma unroll
            for (int h = 0; h < 4; ++h) gk[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, lo[h][s], gk[h], 0, 0, 0);
        }
    }
};
struct NoOperands {
    static constexpr int DC = 16;
    __device__ __forceinline__ void load_df(int, const float*, bool, int, int, int, int) {}
    __device__ __forceinline__ void load_feat(const void*, int64_t, int, int, int, int) {}
    __device__ __forceinline__ void contract(f32x4*) const {}
};

template <bool BF16, bool FB, int NS>
struct OperandsOf {
    using T = Operands<BF16, FB, NS>;
};
template <bool BF16, bool FB>
struct OperandsOf<BF16, FB, 0> {
    using T = NoOperands;
};

enum { G_WHOLE = 0, G_CARRY = 1 };

// Waves per SIMD the registers of dF leave room for.
constexpr int min_waves(bool bf16, int ns, bool surf) {
    const int dc = (bf16 ? 32 : 16) * ns;
    return dc > 128 ? 1 : (dc > (surf || bf16 ? 32 : 64) ? 2 : 3);
}

// MODE: G_WHOLE the whole width at once; G_CARRY the feature part of g read
// from a.g (k_dot wrote it; NS = 0).
// SEG: T at the segment ends goes to a.tseg.
template <bool BF16, int NS, bool FB, bool SURF, int MODE, bool SEG>
__global__ __launch_bounds__(256, min_waves(BF16, NS, SURF)) void k_bwd(BwdArgs a, ViewTable vt, int vec_f, int vec_df) {
    using RecT = typename PrimRec<SURF>::T;
    using Ops = typename OperandsOf<BF16, FB, NS>::T;
    constexpr int RW = PrimRec<SURF>::RW, NQ = PrimRec<SURF>::NQ, GP = PrimRec<SURF>::GP;
    __shared__ float2 swd[4][64 * WST];                                         // per wave: [pixel][position] (w, dL/dpower)
    constexpr int NP = BF16 ? 8 : 4;   // partial sums a position: pairs of pixel rows, or waves
    __shared__ __attribute__((aligned(16))) float sred[2][NP][CK * GP];         // [position][term], by chunk parity
    if (a.counters->inst_overflow || a.counters->visit_overflow) return;
    const int t = a.tile_order ? (int)a.tile_order[blockIdx.x] : (int)blockIdx.x;
    const int nt = __builtin_amdgcn_readfirstlane((int)a.tile_niter[t]);
    if (nt == 0) return;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int q = lane >> 4, xi = lane & 15;
    const int v = view_of_tile(vt, t);
    const int lt = t - vt.tile_off[v];
    const int tx = lt % vt.tiles_x[v], ty = lt / vt.tiles_x[v];
    const int W = vt.width[v], H = vt.height[v];
    const int64_t voff = a.tile_voff[t];
    const bool has_df = NS > 0 && a.dF != nullptr;
    const float LN2 = 0.69314718055994531f;
    const int px = tx * TILE + xi, py = ty * TILE + 4 * w + q;
    const float x = (float)px + 0.5f, y = (float)py + 0.5f;
    const bool inside = px < W && py < H;
    const int64_t p = vt.pix_off[v] + (int64_t)(inside ? py : 0) * W + (inside ? px : 0);
    const int n = (4 * w + q) * TILE + xi;

    // the lane's pixel
    const int nit = inside ? (int)a.n_iter[p] : 0;
    float T = inside ? a.T_final[p] : 1.0f;
    const float TdT = T * ((inside && a.dT) ? a.dT[p] : 0.0f);
    float U = BF16 ? 0.0f : TdT;   // FP32 form: S + T_final dT; BF16 form: S
    float dC0 = 0.f, dC1 = 0.f, dC2 = 0.f;
    if (inside && a.dC) {
        dC0 = a.dC[3 * p];
        dC1 = a.dC[3 * p + 1];
        dC2 = a.dC[3 * p + 2];
    }
    const uint64_t odd_dc = ballot64(!(isfinite(dC0) && isfinite(dC1) && isfinite(dC2)));   // (see the colour sums)
    // B operands: pixel (row 4 w + h, column xi), dF and one dC component (the BF16
    // form adds green, red, blue in this order, the FP32 form red, green, blue)
    const int comp = BF16 && q < 2 ? 1 - q : q;
    Ops ops;
    float dcb[4];
    int64_t prow[4];
    bool in_h[4];
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const int hy = ty * TILE + 4 * w + h;
        in_h[h] = px < W && hy < H;
        prow[h] = vt.pix_off[v] + (int64_t)(in_h[h] ? hy : 0) * W + (in_h[h] ? px : 0);
        dcb[h] = (in_h[h] && a.dC && q < 3) ? a.dC[3 * prow[h] + comp] : 0.0f;
    }
    // (dC0, dC1, dC2, 1)[xi % 4] of the pixels of row 4 w + q: the B operand of
    // the colour and weight sums
    float cw[TILE];
    unroll_seq(std::make_integer_sequence<int, TILE>{}, [&](auto mc) {
        constexpr int m = decltype(mc)::value;
        const float d0 = row_bcast<m>(dC0), d1 = row_bcast<m>(dC1), d2 = row_bcast<m>(dC2);
        const int j = xi & 3;
        cw[m] = j == 0 ? d0 : (j == 1 ? d1 : (j == 2 ? d2 : 1.0f));
        cw[m] = isfinite(cw[m]) ? cw[m] : 0.0f;
    });
    auto load_df = [&](int c0) {
#pragma unroll
        for (int h = 0; h < 4; ++h) ops.load_df(h, a.dF + prow[h] * a.d, in_h[h], c0, q, a.d, vec_df);
    };
    if (has_df) load_df(0);

    // chunk of positions cs .. cs + 15 (the first ones of the list: cnt of them
    // not yet walked); lane xi holds position xi's record and features
    auto at = [&](int cs) { return voff + (cs + xi < nt ? cs + xi : nt - 1); };
    // The BF16 form divides T by a product of four (1 - alpha) at a time, so its
    // result depends on where the chunks lie: pairs of 16 from the end of the
    // list, the first positions (fewer than 32) split at 16.
    auto start_of = [&](int ce) {
        if (BF16 && ce > CK && ce < 2 * CK && ((nt - ce) & (2 * CK - 1)) == 0) return CK;
        return ce - CK > 0 ? ce - CK : 0;
    };
    int cs = start_of(nt);
    RecT rc = load_rec<SURF>(a.vrec, at(cs));
    uint32_t gid_next = 0u;
    if (has_df) {
        ops.load_feat(a.feat, a.vgid[at(cs)], 0, q, a.d, vec_f);
        gid_next = a.vgid[at(start_of(cs))];
    }
    // the pixel's feature part of g for the chunk (a.g: [visit][pixel]); rows of
    // positions the chunk does not hold are not read
    float gn[MODE == G_CARRY ? CK : 1];
    auto load_g = [&](int c0, int cnt) {
        const float* gi = a.g + (voff + c0) * TILE_PIX + n;
#pragma unroll
        for (int k = 0; k < CK; ++k) gn[k] = k < cnt ? gi[k * TILE_PIX] : 0.0f;
    };
    if constexpr (MODE == G_CARRY) load_g(cs, nt - cs);
    int buf = 0;
    float2* wd = swd[w];
    for (int ce = nt; ce > 0; ce = cs, cs = start_of(cs), buf ^= 1) {
        const int cnt = ce - cs, ncs = start_of(cs);
        if constexpr (SEG)   // (thread = pixel of the tile)
            if (ce < nt && (nt - ce) % T_SEG == 0)
                a.tseg[(voff / T_SEG + t + (nt - ce) / T_SEG - 1) * TILE_PIX + threadIdx.x] = T;
        // 1. G: lane (q, xi) gets positions 4 q + r of pixel (row 4 w + h, column xi)
        f32x4 gk[4];
        {
            const float col = comp == 0 ? rc.r2.y : (comp == 1 ? rc.r2.z : (comp == 2 ? rc.r2.w : 0.0f));
            const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int h = 0; h < 4; ++h)
                gk[h] = BF16 && has_df ? zero : __builtin_amdgcn_mfma_f32_16x16x4f32(col, dcb[h], zero, 0, 0, 0);
            if (has_df) ops.contract(gk);
            if constexpr (BF16)   // (the channels in a chain of their own, and the colour added)
                if (has_df)
#pragma unroll
                    for (int h = 0; h < 4; ++h) gk[h] += __builtin_amdgcn_mfma_f32_16x16x4f32(col, dcb[h], zero, 0, 0, 0);
        }
        if (has_df) {
            // the next chunk's features, in flight during the walk
            ops.load_feat(a.feat, gid_next, 0, q, a.d, vec_f);
            gid_next = a.vgid[at(start_of(ncs))];
        }
        const RecT rn = load_rec<SURF>(a.vrec, at(ncs));   // (and its records)
        // to the lane's own pixel: g[4 p + r] from lane row p (a 4 x 4 transpose
        // of lane rows against registers)
        float g[CK];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const Pair a02 = swap32(gk[0][r], gk[2][r]), a13 = swap32(gk[1][r], gk[3][r]);
            const Pair lo = swap16(a02.a, a13.a), hi = swap16(a02.b, a13.b);
            g[r] = lo.a;
            g[4 + r] = lo.b;
            g[8 + r] = hi.a;
            g[12 + r] = hi.b;
        }
        if constexpr (MODE == G_CARRY) {
#pragma unroll
            for (int k = 0; k < CK; ++k) g[k] += gn[k];
            if (cs > 0) load_g(ncs, cs - ncs);   // (in flight during the walk)
        }
        // 2. back to front; positions past rem lie behind the pixel's last one
        //    or were walked before
        const int rem = nit - cs < cnt ? nit - cs : cnt;
        if constexpr (BF16) {
            // four positions at a time: their alphas, the product P of (1 - alpha)
            // and the sum R of w g relative to the T behind them; then their
            // terms; then T and S in front of them
            float al[4], gg[4], iv[4], P = 1.0f, R = 0.0f, trel = 1.0f;
            unroll_seq(std::make_integer_sequence<int, CK>{}, [&](auto kc) {
                constexpr int k = CK - 1 - decltype(kc)::value, r = k & 3;
                const float alpha = prim_alpha<SURF>(bcast_rec<k>(rc), x, y);
                const bool on = alpha >= ALPHA_MIN && k < rem;
                // (a position that does not blend: alpha 0 leaves T and S as they are)
                al[r] = on ? alpha : 0.0f;
                gg[r] = on ? g[k] : 0.0f;
                const float om = 1.0f - al[r];
                iv[r] = __builtin_amdgcn_rcpf(om);
                trel = r == 3 ? iv[r] : trel * iv[r];
                P = r == 3 ? om : P * om;
                R = r == 3 ? al[r] * trel * gg[r] : __builtin_fmaf(al[r] * trel, gg[r], R);
                if constexpr (r == 0) {
                    float Tc = T, Sc = U;
#pragma unroll
                    for (int e = 3; e >= 0; --e) {
                        Tc = Tc * iv[e];
                        const float wv = al[e] * Tc;
                        const float dalpha = __builtin_fmaf(Tc, gg[e], -((Sc + TdT) * iv[e]));
                        // alpha < ALPHA_MAX exactly when o G was not clamped
                        const float dpow = (al[e] > 0.0f && al[e] < ALPHA_MAX) ? dalpha * al[e] : 0.0f;
                        Sc = __builtin_fmaf(wv, gg[e], Sc);
                        wd[lane * WST + k + e] = make_float2(wv, dpow);
                    }
                    U = __builtin_fmaf(T, R, U);
                    T = T * __builtin_amdgcn_rcpf(P);
                }
            });
        } else {
            unroll_seq(std::make_integer_sequence<int, CK>{}, [&](auto kc) {
                constexpr int k = CK - 1 - decltype(kc)::value;
                const float alpha = prim_alpha<SURF>(bcast_rec<k>(rc), x, y);
                const bool on = alpha >= ALPHA_MIN && k < rem;
                // (a position that does not blend: alpha 0 leaves T and S as they are)
                const float al = on ? alpha : 0.0f, gg = on ? g[k] : 0.0f;
                const float inv = rcp1(1.0f - al);
                T = T * inv;
                const float wv = al * T;
                const float dalpha = __builtin_fmaf(T, gg, -(U * inv));
                U = __builtin_fmaf(wv, gg, U);
                // alpha < ALPHA_MAX exactly when o G was not clamped
                const float dpow = (on && alpha < ALPHA_MAX) ? dalpha * al : 0.0f;
                wd[lane * WST + k] = make_float2(wv, dpow);
            });
        }
        // 3. lane (q, xi): position xi, the 16 pixels of row 4 w + q.  The
        //    screen-space terms are moments of dL/dpower along the row: with a =
        //    e.d and b = e x d linear in d = (dx, dy), dy fixed,
        //      sum dp (q1 a e_x - q2 b e_y) = A Sx + B dy S0,
        //      sum dp (q1 a e_y + q2 b e_x) = B Sx + C dy S0,
        //    A = q1 e_x^2 + q2 e_y^2, B = (q1 - q2) e_x e_y, C = q1 e_y^2 + q2 e_x^2,
        //    S0 = sum dp, Sx = sum dp dx, Sxx = sum dp dx^2.  For a long thin splat
        //    A Sx and B dy S0 nearly cancel (q1, of the short axis, dwarfs q2, and its part
        //    is a, small beside dx and dy), so the FP32 form sums a itself, Sa, and combines
        //    q1 e_x Sa - q2 e_y Sb and q1 e_y Sa + q2 e_x Sb, Sb = e_x dy S0 - e_y Sx: two
        //    instructions more a pixel and position (476 -> 487 us of 500k Gaussians, 256
        //    channels, 1920x1080); axes of 60 and 1.5 pixels: error of dL/d(u, v) over the
        //    terms' sizes 1.0e-7 -> 1.0e-8, of terms formed pixel by pixel 0.9e-8.
        //    A surfel's nine record terms are linear in dL/dk = dp (-u/k2, -v/k2,
        //    (u^2 + v^2)/k2) = (l0, l1, l2) with coefficients from the record and (dx, dy):
        //      dx_c: -b1 L0 + b0 L1 + e2 L2,  dy_c: a1 L0 - a0 L1 + e1 L2,
        //      a0: dy L1, a1: -dy L0, b0: -L1x, b1: L0x, D: L2, e1: -dy L2, e2: -L2x.
        //    The colour and weight sums are contractions over the pixels, W^T . [dC | 1]
        //    (v_mfma_f32_4x4x1_16b_f32: block b = 4 positions of one pixel row).
        constexpr int NR = NQ - 4;          // terms summed on the VALU
        constexpr int NR4 = (NR + 3) / 4 * 4;
        float qv[NR4];
#pragma unroll
        for (int m = 0; m < NR4; ++m) qv[m] = 0.0f;
        f32x4 col[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
        const float2* wr = wd + q * TILE * WST + xi;
        {
            const float dy = (y - rc.r0.y) - rc.r0.w;
            float x0 = (float)(tx * TILE) + 0.5f;
            asm volatile("" : "+v"(x0));   // (x0 + m is formed here: not sixteen registers held across the chunks)
            float s0 = 0.0f, sx = 0.0f, sxx = 0.0f, sa = 0.0f;
            const float eydy = rc.r1.y * dy;   // (Gaussians)
            float L0 = 0.0f, L1 = 0.0f, L2 = 0.0f, L0x = 0.0f, L1x = 0.0f, L2x = 0.0f;
#pragma unroll
            for (int m = 0; m < TILE; ++m) {
                if (m % 4 == 0) asm volatile("" ::: "memory");   // (four pairs in flight, not all sixteen)
                const float2 e = wr[m * WST];
                col[BF16 ? 0 : m & 1] = __builtin_amdgcn_mfma_f32_4x4x1f32(e.x, cw[m], col[BF16 ? 0 : m & 1], 0, 0, 0);
                const float dx = BF16 && !SURF ? ((x0 - rc.r0.x) - rc.r0.z) + (float)m : ((x0 + (float)m) - rc.r0.x) - rc.r0.z;
                if constexpr (SURF) {
                    SurfPlane sp = surfel_plane(rc, dx, dy);
                    // (a ray nearly parallel to the plane, which does not blend: u or v may not be finite)
                    if (e.y == 0.0f) sp.u = sp.v = sp.ik2 = 0.0f;
                    const float pk = e.y * sp.ik2;
                    const float l0 = -(pk * sp.u), l1 = -(pk * sp.v);
                    const float l2 = pk * __builtin_fmaf(sp.u, sp.u, sp.v * sp.v);
                    L0 += l0;
                    L1 += l1;
                    L2 += l2;
                    L0x = __builtin_fmaf(l0, dx, L0x);
                    L1x = __builtin_fmaf(l1, dx, L1x);
                    L2x = __builtin_fmaf(l2, dx, L2x);
                } else {
                    if constexpr (!BF16) sa = __builtin_fmaf(e.y, __builtin_fmaf(rc.r1.x, dx, eydy), sa);
                    const float pdx = e.y * dx;
                    sx += pdx;
                    sxx = __builtin_fmaf(pdx, dx, sxx);
                }
                s0 += e.y;
            }
            if constexpr (SURF) {
                const float a0 = rc.r1.x, a1 = rc.r1.y, b0 = rc.r1.z, b1 = rc.r1.w, e1 = rc.r3.y, e2 = rc.r3.z;
                qv[0] = __builtin_fmaf(-b1, L0, __builtin_fmaf(b0, L1, e2 * L2));
                qv[1] = __builtin_fmaf(a1, L0, __builtin_fmaf(-a0, L1, e1 * L2));
                qv[2] = dy * L1;
                qv[3] = -dy * L0;
                qv[4] = -L1x;
                qv[5] = L0x;
                qv[6] = L2;
                qv[7] = -dy * L2;
                qv[8] = -L2x;
            } else {
                const float ex = rc.r1.x, ey = rc.r1.y, q1 = rc.r1.z, q2 = rc.r1.w;
                const float A = q1 * ex * ex + q2 * ey * ey, B = (q1 - q2) * ex * ey, C = q1 * ey * ey + q2 * ex * ex;
                const float sy = dy * s0;
                if constexpr (BF16) {
                    qv[0] = -2.0f * LN2 * (A * sx + B * sy);
                    qv[1] = -2.0f * LN2 * (B * sx + C * sy);
                } else {
                    const float sb = __builtin_fmaf(ex, sy, -(ey * sx));
                    qv[0] = -2.0f * LN2 * (q1 * ex * sa - q2 * ey * sb);
                    qv[1] = -2.0f * LN2 * (q1 * ey * sa + q2 * ex * sb);
                }
                qv[2] = -0.5f * sxx;
                qv[3] = -dy * sx;
                qv[4] = -0.5f * dy * sy;
            }
            qv[NR - 1] = s0;
        }
        float* sr = BF16 ? sred[buf][2 * w + (q >> 1)] : sred[buf][w];
        const int term = BF16 ? q & 1 : (q == 1 ? 2 : (q == 2 ? 1 : q));
        constexpr int RT = BF16 ? 2 : 4;    // terms a reduction
#pragma unroll
        for (int m = 0; m < (NR + RT - 1) / RT * RT; m += RT) {
            const float sum = BF16 ? reduce2(qv[m], qv[m + 1]) : reduce4(qv[m], qv[m + 1], qv[m + 2], qv[m + 3]);
            if (m + term < NR) sr[xi * GP + m + term] = sum;
        }
        if constexpr (!BF16) col[0] += col[1];
        // a component of dC that is not finite enters the contraction as zero (0 *
        // inf must not reach the positions its pixel does not blend) and is added
        // here, pixel by pixel, to those it does
        for (uint64_t odd = odd_dc; odd != 0; odd &= odd - 1) {
            const int l = __builtin_ctzll(odd), j = xi & 3;
            const float d0 = __shfl(dC0, l, 64), d1 = __shfl(dC1, l, 64), d2 = __shfl(dC2, l, 64);
            const float b = j == 0 ? d0 : (j == 1 ? d1 : (j == 2 ? d2 : 0.0f));
            if ((l >> 4) == q && !isfinite(b)) {
                const float2* e = wd + l * WST + (xi & ~3);
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (e[i].x != 0.0f) col[0][i] += e[i].x * b;
            }
        }
        // (lane (q, xi) now holds position 4 (xi / 4) + term, component xi % 4)
        if constexpr (BF16) {
#pragma unroll
            for (int i = 0; i < 4; i += 2)
                sr[((xi & ~3) + i + term) * GP + NR + (xi & 3)] = reduce2(col[0][i], col[0][i + 1]);
        } else {
            sr[((xi & ~3) + term) * GP + NR + (xi & 3)] = reduce4(col[0][0], col[0][1], col[0][2], col[0][3]);
        }
        __syncthreads();
        // the partial sums, in order (terms NQ .. GP - 1 are padding: zero)
        if ((int)threadIdx.x < cnt * GP) {
            float sum = sred[buf][0][threadIdx.x];
#pragma unroll
            for (int k = 1; k < NP; ++k) sum += sred[buf][k][threadIdx.x];
            a.part_geom[(voff + cs) * GP + threadIdx.x] = (int)threadIdx.x % GP < NQ ? sum : 0.0f;
        }
        // No second barrier: the next chunk writes the other buffer, whose last
        // readers all passed the barrier above; the pairs are the wave's own.
        rc = rn;
    }
}

// ---------------------------------------------------------------------------
// f_k . dF for widths whose dF does not fit beside the walk (256 channels and
// up), written as g[visit][pixel] for every visited position (a.d0 > 0: added
// to it) and read back by the walk (G_CARRY), 1 KB a visit.  At 256 channels a
// tile's dF fills half a CU's registers: one workgroup a CU would load it (26k
// cycles at the HBM rate) with nothing else to run.  Here eight waves of one
// pixel row each hold their dF, a 32 NS channel slice at a time, two workgroups
// a CU, and share the features of DK positions through LDS: most tiles pay the
// chain list -> Gaussian -> features once or twice (chunks of 32 paid it five
// times: 1.39 ms at 500k, 1920x1080).  Bound: HBM (dF read once, g written once).
//
// TERMS: dF as that many BF16 terms on v_mfma_f32_16x16x32_bf16, BF16 features
// as stored: 2 in the BF16 form; 3 in the FP32 form, where x = h + m + l is exact
// (three roundings to 8 bits cover 24), so that only the FP32 accumulation
// rounds.  0: FP32 features, FP32 operands on v_mfma_f32_16x16x4_f32.
// VEC: 16-byte feature loads, the slice wholly inside the width.
// PARTS: a workgroup takes every gridDim.y-th chunk of the list (images of few tiles).
template <int TERMS, int NS, bool VEC, bool PARTS>
__global__ __launch_bounds__(512, TERMS == 2 && VEC ? 4 : 2) void k_dot(BwdArgs a, ViewTable vt, int n_tiles, int vec_df) {
    constexpr int DK = TERMS > 0 ? 128 : 64;                 // positions per chunk
    constexpr int EB = TERMS > 0 ? 2 : 4;                    // bytes per feature element
    constexpr int ROW = 32 * NS * EB + 32;                   // LDS row, an odd multiple of 32 bytes
    constexpr int NI = 32 * NS * EB / 16, IT = DK * NI / 512;   // 16-byte items per row and per thread
    __shared__ __attribute__((aligned(16))) unsigned char sf[DK * ROW];
    if (a.counters->inst_overflow || a.counters->visit_overflow) return;
    // (workgroups go to the eight XCDs in turn: the two halves of a tile to the
    // same one, which then reads the tile's features into its L2 once)
    const int j = (int)blockIdx.x >> 3, t = (j >> 1) * 8 + ((int)blockIdx.x & 7);
    if (t >= n_tiles) return;
    const int nt = __builtin_amdgcn_readfirstlane((int)a.tile_niter[t]);
    const int c0 = PARTS ? (int)blockIdx.y * DK : 0, step = PARTS ? (int)gridDim.y * DK : DK;
    if (c0 >= nt) return;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int q = lane >> 4, xi = lane & 15;
    const int v = view_of_tile(vt, t);
    const int lt = t - vt.tile_off[v];
    const int row = 8 * (j & 1) + w;
    const int px = (lt % vt.tiles_x[v]) * TILE + xi, py = (lt / vt.tiles_x[v]) * TILE + row;
    if (py - w >= vt.height[v]) return;   // (no row of this half is inside the image: its g is not used)
    const bool inside = px < vt.width[v] && py < vt.height[v];
    const int64_t voff = a.tile_voff[t];
    const float* drow = a.dF + (inside ? vt.pix_off[v] + (int64_t)py * vt.width[v] + px : 0) * a.d;
    float* out = a.g + voff * TILE_PIX + row * TILE + xi;
    const bool add = a.d0 > 0;

    // staging: item it of this thread is 16 bytes of position (threadIdx.x + 512 it) / NI
    auto load_gid = [&](int cs, uint32_t* gid) {
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int k = cs + ((int)threadIdx.x + 512 * it) / NI;
            gid[it] = a.vgid[voff + (k < nt ? k : nt - 1)];
        }
    };
    auto load = [&](const uint32_t* gid, u32x4* raw) {
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int c = (((int)threadIdx.x + 512 * it) % NI) * (16 / EB);
            if constexpr (VEC) {
                raw[it] = *reinterpret_cast<const u32x4*>(static_cast<const unsigned char*>(a.feat) +
                                                          ((int64_t)gid[it] * a.d + a.d0 + c) * EB);
            } else if constexpr (TERMS > 0) {
                const uint16_t* fr = static_cast<const uint16_t*>(a.feat) + (int64_t)gid[it] * a.d;
                const uint2 lo = load_row4h(fr, a.d0 + c, a.d, false), hi = load_row4h(fr, a.d0 + c + 4, a.d, false);
                raw[it] = u32x4{lo.x, lo.y, hi.x, hi.y};
            } else {
                raw[it] = __builtin_bit_cast(
                    u32x4, load_row4(static_cast<const float*>(a.feat) + (int64_t)gid[it] * a.d, a.d0 + c, a.d, false));
            }
        }
    };
    auto run = [&](auto mul) {
        for (int cs = c0; cs < nt; cs += step) {
            uint32_t gid[IT];
            u32x4 raw[IT];
            load_gid(cs, gid);
            load(gid, raw);
            if (cs > c0) __syncthreads();   // (the previous chunk's readers are done)
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int idx = (int)threadIdx.x + 512 * it;
                *reinterpret_cast<u32x4*>(sf + (idx / NI) * ROW + (idx % NI) * 16) = raw[it];
            }
            __syncthreads();
            const int end = nt - cs < DK ? nt - cs : DK;
            for (int k0 = 0; k0 < end; k0 += CK) {
                const f32x4 g = mul(sf + (k0 + xi) * ROW + 16 * q);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int k = k0 + 4 * q + r;
                    if (k < end) {
                        float* o = out + (int64_t)(cs + k) * TILE_PIX;
                        *o = add ? *o + g[r] : g[r];
                    }
                }
            }
        }
    };
    if constexpr (TERMS > 0) {
        bf16x8 d[TERMS][NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            float4 u = make_float4(0.f, 0.f, 0.f, 0.f), x = u;
            if (inside) {
                u = load_row4(drow, a.d0 + 32 * s + 8 * q, a.d, vec_df != 0);
                x = load_row4(drow, a.d0 + 32 * s + 8 * q + 4, a.d, vec_df != 0);
            }
            const float vals[8] = {u.x, u.y, u.z, u.w, x.x, x.y, x.z, x.w};
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                float rest = vals[m];
#pragma unroll
                for (int c = 0; c < TERMS; ++c) {
                    // (all terms but the last stay finite: values above the largest BF16 would
                    // round to an infinity; an infinity or NaN is the last term)
                    const float top = 3.38953139e38f;
                    const __bf16 b = (__bf16)(c < TERMS - 1 ? __builtin_amdgcn_fmed3f(rest, -top, top) : rest);
                    d[c][s][m] = b;
                    rest -= (float)b;
                }
            }
        }
        run([&](const unsigned char* f) {
            f32x4 g[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
            // (three terms: two chains, a slab's small terms first; two: one chain,
            // as the widths contracted beside the walk)
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const bf16x8 fa = *reinterpret_cast<const bf16x8*>(f + 64 * s);
#pragma unroll
                for (int c = 0; c < TERMS; ++c) {
                    const int e = TERMS == 3 ? 2 - c : c, ch = TERMS == 3 ? s & 1 : 0;
                    g[ch] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, d[e][s], g[ch], 0, 0, 0);
                }
            }
            return TERMS == 3 ? g[0] + g[1] : g[0];
        });
    } else {
        float4 d[2 * NS];
#pragma unroll
        for (int s = 0; s < 2 * NS; ++s)
            d[s] = inside ? load_row4(drow, a.d0 + 16 * s + 4 * q, a.d, vec_df != 0) : make_float4(0.f, 0.f, 0.f, 0.f);
        run([&](const unsigned char* f) {
            f32x4 g[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int s = 0; s < 2 * NS; ++s) {
                const float4 fa = *reinterpret_cast<const float4*>(f + 64 * s);
                f32x4& c = g[s & 1];
                c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa.x, d[s].x, c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa.y, d[s].y, c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa.z, d[s].z, c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa.w, d[s].w, c, 0, 0, 0);
            }
            return g[0] + g[1];
        });
    }
}

template <bool BF16, int NS, bool FB, bool SURF, int MODE>
void launch(const BwdArgs& a, const ViewTable& vt, int n_tiles, hipStream_t s) {
    // 16-byte (FP32 form with BF16 storage: 8-byte) feature and dF loads where every row is aligned to them
    const int vec_f = a.d % 4 == 0 && reinterpret_cast<uintptr_t>(a.feat) % (FB ? 8 : 16) == 0;
    const int vec_df = a.d % 4 == 0 && reinterpret_cast<uintptr_t>(a.dF) % 16 == 0;
    if constexpr (BF16)
        if (a.tseg) {
            hipLaunchKernelGGL((k_bwd<BF16, NS, FB, SURF, MODE, true>), dim3(n_tiles), dim3(256), 0, s, a, vt, vec_f, vec_df);
            return;
        }
    hipLaunchKernelGGL((k_bwd<BF16, NS, FB, SURF, MODE, false>), dim3(n_tiles), dim3(256), 0, s, a, vt, vec_f, vec_df);
}

// the feature part of g in slices of 256 channels into a.g, then the walk
template <int TERMS, bool SURF>
void launch_dot(const BwdArgs& a0, const ViewTable& vt, int n_tiles, hipStream_t s) {
    const bool vec_f = a0.d % (TERMS > 0 ? 8 : 4) == 0 && reinterpret_cast<uintptr_t>(a0.feat) % 16 == 0;
    const int vec_df = a0.d % 4 == 0 && reinterpret_cast<uintptr_t>(a0.dF) % 16 == 0;
    BwdArgs a = a0;
    const unsigned parts = (unsigned)std::max(list_parts(n_tiles) / 2, 1);   // (two workgroups a tile already)
    const dim3 grid((unsigned)(((n_tiles + 7) / 8) * 16), parts);
    auto slice = [&](auto p) {
        constexpr bool PARTS = decltype(p)::value;
        const int rest = a.d - a.d0;
        if (vec_f && rest >= 256)
            hipLaunchKernelGGL((k_dot<TERMS, 8, true, PARTS>), grid, dim3(512), 0, s, a, vt, n_tiles, vec_df);
        else if (vec_f && rest == 128)
            hipLaunchKernelGGL((k_dot<TERMS, 4, true, PARTS>), grid, dim3(512), 0, s, a, vt, n_tiles, vec_df);
        else
            hipLaunchKernelGGL((k_dot<TERMS, 8, false, PARTS>), grid, dim3(512), 0, s, a, vt, n_tiles, vec_df);
    };
    for (a.d0 = 0; a.d0 < a.d; a.d0 += 256) {
        if (parts > 1)
            slice(std::true_type{});
        else
            slice(std::false_type{});
    }
    launch<TERMS == 2, 0, false, SURF, G_CARRY>(a, vt, n_tiles, s);
}

template <bool FB, bool SURF>
void launch_f32(const BwdArgs& a, const ViewTable& vt, int n_tiles, hipStream_t s) {
    const int ns = a.dF ? (a.d + 15) / 16 : 0;
    if (ns == 0) launch<false, 0, false, SURF, G_WHOLE>(a, vt, n_tiles, s);
    else if (ns == 1) launch<false, 1, FB, SURF, G_WHOLE>(a, vt, n_tiles, s);
    else if (ns == 2) launch<false, 2, FB, SURF, G_WHOLE>(a, vt, n_tiles, s);
    else if (ns <= 4) launch<false, 4, FB, SURF, G_WHOLE>(a, vt, n_tiles, s);
    else if (ns <= 8) launch<false, 8, FB, SURF, G_WHOLE>(a, vt, n_tiles, s);
    else if (a.d < 256) launch<false, 16, FB, SURF, G_WHOLE>(a, vt, n_tiles, s);   // (no room for g: see a.g)
    else launch_dot<FB ? 3 : 0, SURF>(a, vt, n_tiles, s);
}

template <bool SURF>
void launch_bf16(const BwdArgs& a, const ViewTable& vt, int n_tiles, hipStream_t s) {
    const int ns = a.dF ? a.d / 32 : 0;
    if (ns == 0) launch<true, 0, false, SURF, G_WHOLE>(a, vt, n_tiles, s);
    else if (ns == 1) launch<true, 1, true, SURF, G_WHOLE>(a, vt, n_tiles, s);
    else if (ns == 2) launch<true, 2, true, SURF, G_WHOLE>(a, vt, n_tiles, s);
    else if (ns == 3) launch<true, 3, true, SURF, G_WHOLE>(a, vt, n_tiles, s);
    else if (ns == 4) launch<true, 4, true, SURF, G_WHOLE>(a, vt, n_tiles, s);
    else launch_dot<2, SURF>(a, vt, n_tiles, s);
}

}  // namespace

void launch_render_grad(const BwdArgs& a, const ViewTable& vt, int n_tiles, bool bf16, hipStream_t s) {
    const bool surf = a.prim == FH_PRIM_SURFEL;
    if (bf16) {
        if (surf) launch_bf16<true>(a, vt, n_tiles, s);
        else launch_bf16<false>(a, vt, n_tiles, s);
    } else if (a.feat_bf16) {
        if (surf) launch_f32<true, true>(a, vt, n_tiles, s);
        else launch_f32<true, false>(a, vt, n_tiles, s);
    } else {
        if (surf) launch_f32<false, true>(a, vt, n_tiles, s);
        else launch_f32<false, false>(a, vt, n_tiles, s);
    }
}

}  // namespace fh
