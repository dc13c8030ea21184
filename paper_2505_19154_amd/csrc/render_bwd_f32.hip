// Adjoint and feature fusion of the compositing pass in the FP32 form, on the
// FP32 matrix unit (v_mfma_f32_16x16x4_f32, gfx950): FP32 operands and FP32
// accumulation throughout, no split and no narrower type.
//
// Gradient kernel, per tile, back to front over the tile's visited list in
// chunks of 32 positions (Appendix A.2: dL/dalpha_k = T_k g_k - (S_k + T_final
// dT)/(1 - alpha_k), S_k = sum_{i>k} w_i g_i, g_k = rgb_k . dC + f_k . dF):
//   1. g for all (pixel, position) pairs of the chunk is one contraction over
//      the channels and the colour, G^T[k x px] = [Feat | rgb][k x (D + 3)] .
//      [dF | dC]^T[(D + 3) x px]; its result lands in the lanes that walk
//      those pairs;
//   2. wave w walks pixel row w: each pixel's four lanes take four consecutive
//      positions, and the back-to-front transmittance division and the suffix
//      sum S are combined across the lanes with a scan;
//   3. (w, dL/dpower) per (pixel, position) go to LDS, and a position-parallel
//      pass sums the screen-space terms over the tile's pixels in a fixed
//      order into one partial per instance: no atomics.
//
// What bounds it: VALU work per (pixel, position) (alpha, the walk, the
// moments), the FP32 matrix rate (157 TFLOP/s) only at 256 channels.  Sixteen
// waves of one row each keep four waves per SIMD, with the row's dF (64
// registers at 256 channels) resident for the whole tile.
//
// Measured against a VALU form (each pixel's dot products as FMAs over features
// broadcast from LDS, ten wave-wide sums per (row of pixels, position)):
// 1k Gaussians, 128x128, D = 16: 386 -> 55 us; 200k, 800x800, D = 64: 1383 ->
// 489 us; 150k, 987x657, D = 0: 914 -> 354 us; 500k, 1920x1080, D = 256 with
// fusion: 25.6 -> 5.8 ms (both kernels).
//
// Fusion kernel: the same walk needs only w = alpha T; the per-instance partial
// sum_p w(p) target(p) is the contraction W^T[k x px] . Target[px x D], the
// tile's target held in registers (one 16-channel block per wave).
//
// Both take the surfel primitive (SURF): four-float4 records, the density at
// the ray-plane intersection, 14 terms per instance in rows of 16 floats.
#include "kernels.hpp"

namespace fh {

typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int BK = 32;          // positions per chunk
// (w, dL/dpower) pairs, pixel-major, in rows of 33 pairs: the walk's stores
// (lane xi = pixel) start 66 dwords apart, the position-parallel reads are
// consecutive
constexpr int SKW = BK + 1;
constexpr int RG = 4;           // record padding group: the walk's lane rows read records 4 apart
template <bool SURF>
constexpr int rslots() {
    return PrimRec<SURF>::RW * BK + BK / RG;
}

// 1 / x to within one rounding: the hardware reciprocal (1 ulp) and one Newton step.
__device__ __forceinline__ float rcp_nr(float x) {
    const float r = __builtin_amdgcn_rcpf(x);
    return __builtin_fmaf(__builtin_fmaf(-x, r, 1.0f), r, r);
}

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// Sum over the lanes xi, xi + 16, xi + 32, xi + 48 (the same bits in each).
__device__ __forceinline__ float sum_rows(float v) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    const unsigned s = __float_as_uint(__uint_as_float(a[0]) + __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(s, s, false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Rows of four channels from c (zeros past d): a 16-byte load where the rows
// allow it (vec), else element by element.
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

// NS: 16-channel slabs resident (dF registers) and staged (features); STREAM:
// widths above 256 channels, where each chunk takes the slabs NS at a time,
// its dF read again from memory.  FB: features stored in BF16.
template <int NS, bool FB, bool SURF, bool STREAM>
__global__ __launch_bounds__(1024) void k_bwd_f32(BwdArgs a, ViewTable vt, int vec_f, int vec_df) {
    using RecT = typename PrimRec<SURF>::T;
    constexpr int RW = PrimRec<SURF>::RW, NQ = PrimRec<SURF>::NQ, GP = PrimRec<SURF>::GP;
    constexpr int RSLOTS = rslots<SURF>();
    constexpr int DC = 16 * NS;                       // channels staged at a time
    // feature rows in LDS, an odd multiple of 8 dwords apart (the 16-byte reads
    // of lanes served together then fall in distinct banks)
    constexpr int DP = FB ? DC + 16 : DC + 8;         // in elements
    constexpr int FBYTES = FB ? 2 : 4;
    constexpr int NFB = STREAM ? 1 : 2;               // feature buffers
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    float2* swd = reinterpret_cast<float2*>(smem);                              // [256][SKW] (w, dL/dpower)
    float4* sdc = reinterpret_cast<float4*>(swd + TILE_PIX * SKW);              // [256] dC of the tile
    float* sred = reinterpret_cast<float*>(sdc + TILE_PIX);                     // [8 row pairs][NQ][BK]
    unsigned char* sfeat2 = reinterpret_cast<unsigned char*>(sred + 8 * NQ * BK);   // [NFB][BK][DP]
    __shared__ float4 srecb[3][RSLOTS];   // chunk records and Gaussians, triple-buffered:
    __shared__ uint32_t sgb[3][BK];       // those two chunks ahead arrive during this one

    if (a.counters->inst_overflow || a.counters->visit_overflow) return;
    const int t = blockIdx.x;
    const uint32_t nt = a.tile_niter[t];
    if (nt == 0) return;
    const int D = a.d;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int q = lane >> 4, xi = lane & 15;
    const int v = view_of_tile(vt, t);
    const int lt = t - vt.tile_off[v];
    const int tx = lt % vt.tiles_x[v], ty = lt / vt.tiles_x[v];
    const int W = vt.width[v], H = vt.height[v];
    const uint32_t voff = a.tile_voff[t];
    const bool has_df = NS > 0 && a.dF != nullptr;
    const float LN2 = 0.69314718055994531f;
    const int px = tx * TILE + xi, py = ty * TILE + w;
    const float x = (float)px + 0.5f, y = (float)py + 0.5f;
    const bool inside = px < W && py < H;
    const int64_t p = vt.pix_off[v] + (int64_t)(inside ? py : 0) * W + (inside ? px : 0);
    const int n = w * TILE + xi;

    // the pixel's state (identical in its four lanes)
    const uint32_t nit = inside ? a.n_iter[p] : 0u;
    float T = inside ? a.T_final[p] : 1.0f, S = 0.0f;
    const float TdT = T * ((inside && a.dT) ? a.dT[p] : 0.0f);   // T_final dT
    float dC0 = 0.f, dC1 = 0.f, dC2 = 0.f;
    if (inside && a.dC) {
        dC0 = a.dC[3 * p];
        dC1 = a.dC[3 * p + 1];
        dC2 = a.dC[3 * p + 2];
    }
    if (q == 0) sdc[n] = make_float4(dC0, dC1, dC2, 0.f);
    // a pixel whose dC is not finite must not reach the positions it does not
    // blend (0 * inf): such tiles select the colour products
    const bool odd_dc = __syncthreads_or(!(isfinite(dC0) && isfinite(dC1) && isfinite(dC2))) != 0;
    const float dcq = q == 0 ? dC0 : (q == 1 ? dC1 : (q == 2 ? dC2 : 0.0f));   // B operand of the colour step
    // dF of the pixel, channels 16 s + 4 q + i
    float4 df[NS > 0 ? NS : 1];
    auto load_df = [&](int c0) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
            df[s] = inside ? load_row4(a.dF + p * D, c0 + 16 * s + 4 * q, D, vec_df != 0)
                           : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    if (has_df && !STREAM) load_df(0);

    // feature rows of a chunk, four channels an item; padding positions read
    // Gaussian 0 (a record that never blends)
    constexpr int NG = NS > 0 ? 4 * NS : 1;            // items per row
    constexpr int ITEMS = NS > 0 ? BK * NG : 0, NI = NS > 0 ? (ITEMS + 1023) / 1024 : 1;
    auto load_feats = [&](const uint32_t* gl, int c0, uint4* raw) {
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const int idx = (int)threadIdx.x + 1024 * it;
            raw[it] = make_uint4(0, 0, 0, 0);
            if (idx < ITEMS) {
                const int k = idx / NG, c = c0 + 4 * (idx % NG);
                const uint32_t g = gl[k];
                const int64_t ga = g != 0xFFFFFFFFu ? g : 0u;
                if constexpr (FB) {
                    const uint2 u = load_row4h(static_cast<const uint16_t*>(a.feat) + ga * D, c, D, vec_f != 0);
                    raw[it].x = u.x;
                    raw[it].y = u.y;
                } else {
                    raw[it] = __builtin_bit_cast(
                        uint4, load_row4(static_cast<const float*>(a.feat) + ga * D, c, D, vec_f != 0));
                }
            }
        }
    };
    auto store_feats = [&](const uint4* raw, unsigned char* dst) {
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const int idx = (int)threadIdx.x + 1024 * it;
            if (idx < ITEMS) {
                const int k = idx / NG, c = 4 * (idx % NG);
                if constexpr (FB)
                    *reinterpret_cast<uint2*>(dst + (k * DP + c) * 2) = make_uint2(raw[it].x, raw[it].y);
                else
                    *reinterpret_cast<uint4*>(dst + (k * DP + c) * 4) = raw[it];
            }
        }
    };
    // A operand: feature row k, channels 16 s + 4 q .. + 3
    auto feat_a = [&](const unsigned char* sf, int k, int s) -> float4 {
        if constexpr (FB) {
            const uint2 u = *reinterpret_cast<const uint2*>(sf + (k * DP + 16 * s + 4 * q) * 2);
            return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xFFFF0000u),
                               __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xFFFF0000u));
        } else {
            return *reinterpret_cast<const float4*>(sf + (k * DP + 16 * s + 4 * q) * 4);
        }
    };
    auto contract = [&](const unsigned char* sf, f32x4* gk) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const float4 f0 = feat_a(sf, xi, s), f1 = feat_a(sf, 16 + xi, s);
            gk[0] = mfma4(f0.x, df[s].x, gk[0]);
            gk[1] = mfma4(f1.x, df[s].x, gk[1]);
            gk[0] = mfma4(f0.y, df[s].y, gk[0]);
            gk[1] = mfma4(f1.y, df[s].y, gk[1]);
            gk[0] = mfma4(f0.z, df[s].z, gk[0]);
            gk[1] = mfma4(f1.z, df[s].z, gk[1]);
            gk[0] = mfma4(f0.w, df[s].w, gk[0]);
            gk[1] = mfma4(f1.w, df[s].w, gk[1]);
        }
    };

    // prologue: records and Gaussians of the first two chunks, features of the first
    {
        const int cs0 = (int)nt - BK > 0 ? (int)nt - BK : 0;
        const int cs1 = cs0 - BK > 0 ? cs0 - BK : 0;
        const int c = (int)threadIdx.x / BK, k = (int)threadIdx.x % BK;
        if (c < 2) {
            const int cs = c ? cs1 : cs0, cnt = c ? cs0 - cs1 : (int)nt - cs0;
            RecT r = pad_rec<SURF>();
            uint32_t g = 0xFFFFFFFFu;
            if (k < cnt) {
                r = load_rec<SURF>(a.vrec, (int64_t)voff + cs + k);
                g = a.vgid[(int64_t)voff + cs + k];
            }
            lds_put_prec<SURF, RG>(srecb[c], k, r);
            sgb[c][k] = g;
        }
    }
    __syncthreads();
    if (has_df && !STREAM) {
        uint4 raw[NI];
        load_feats(sgb[0], 0, raw);
        store_feats(raw, sfeat2);
    }
    __syncthreads();
    int b3 = 0, f2 = 0;   // this chunk's record buffer (mod 3) and feature buffer (mod 2)
    for (int ce = (int)nt; ce > 0; ce -= BK) {
        const int cs = ce - BK > 0 ? ce - BK : 0;
        const int cnt = ce - cs;
        const int n3 = b3 == 2 ? 0 : b3 + 1, nn3 = n3 == 2 ? 0 : n3 + 1;
        const float4* srec = srecb[b3];
        // records (RD dwords each) and Gaussians of the chunk after next, one
        // dword per thread, stored after this chunk's walk; padding positions
        // get the padding record.  (Positions nncs .. nncs + BK - 1 all lie in
        // this tile's visits: that chunk exists only when this one and the next
        // are full.)
        constexpr int RD = 4 * RW;
        const int ncs = cs - BK > 0 ? cs - BK : 0;
        const int nncs = ncs - BK > 0 ? ncs - BK : 0;
        const int nncnt = ncs - nncs;
        const bool pre_on = ncs > 0 && threadIdx.x < (RD + 1) * BK;
        const bool pre_g = threadIdx.x >= RD * BK;
        const int pre_k = pre_g ? (int)threadIdx.x - RD * BK : (int)threadIdx.x / RD;
        uint32_t pre = 0u;
        if (pre_on) {
            const uint32_t* src = pre_g ? a.vgid + ((int64_t)voff + nncs)
                                        : reinterpret_cast<const uint32_t*>(a.vrec) + ((int64_t)voff + nncs) * RD;
            pre = src[pre_g ? pre_k : (int)threadIdx.x];
        }
        // the next chunk's features, stored after this chunk's walk
        uint4 fnext[NI];
        const bool fnext_on = has_df && !STREAM && cs > 0;
        if (fnext_on) load_feats(sgb[n3], 0, fnext);

        // 1. G^T[k][px]: lane gets k = 16 kb + 4 q + r for its pixel; the colour
        //    part first (channels r, g, b, 0 of the records)
        f32x4 gk[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
        if constexpr (STREAM) {
            if (has_df) {
                for (int c0 = 0; c0 < D; c0 += DC) {
                    if (c0 > 0) __syncthreads();   // (the first slice's buffer was released by the chunk's last barrier)
                    uint4 raw[NI];
                    load_feats(sgb[b3], c0, raw);
                    load_df(c0);
                    store_feats(raw, sfeat2);
                    __syncthreads();
                    contract(sfeat2, gk);
                }
            }
        }
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
            const float col = reinterpret_cast<const float*>(srec + prec_slot<SURF, RG>(16 * kb + xi) + 2)[q < 3 ? q + 1 : 0];
            gk[kb] = mfma4(q < 3 ? col : 0.0f, dcq, gk[kb]);
        }
        if constexpr (!STREAM) {
            if (has_df) contract(sfeat2 + f2 * BK * DP * FBYTES, gk);
        }
        // 2. back to front: half-chunk kb = 1 (positions 16..31), then kb = 0
#pragma unroll
        for (int kb = 1; kb >= 0; --kb) {
            asm volatile("" ::: "memory");
            float al[4], gg[4], iv[4];   // iv = 1 / (1 - alpha)
            bool on[4];
            float P = 1.0f, R = 0.0f, trel = 1.0f;
#pragma unroll
            for (int r = 3; r >= 0; --r) {
                const int k = 16 * kb + 4 * q + r;
                // (slot of k = 16 kb + 4 q + r: (16 RW + 4) kb + (4 RW + 1) q + RW r)
                const float4* rp = srec + (4 * RW + 1) * q + (16 * RW + 4) * kb + RW * r;
                RecT rc;
                rc.r0 = rp[0];
                rc.r1 = rp[1];
                rc.r2.x = rp[2].x;
                if constexpr (SURF) rc.r3 = rp[3];
                const float alpha = prim_alpha<SURF>(rc, x, y);
                on[r] = k < cnt && (uint32_t)(cs + k) < nit && alpha >= ALPHA_MIN;
                al[r] = alpha;
                gg[r] = gk[kb][r];
                iv[r] = rcp_nr(1.0f - al[r]);
                // (branch-free: a position that does not blend leaves the state as is)
                const float tn = trel * iv[r];
                R = on[r] ? __builtin_fmaf(al[r] * tn, gg[r], R) : R;
                P = on[r] ? P * (1.0f - al[r]) : P;
                trel = on[r] ? tn : trel;
            }
            // entry state of every lane, scanning from the back (lane q = 3 first)
            const Rows4 Pr = rows4(P), Rr = rows4(R);
            const float Te3 = T, Se3 = S;
            const float Te2 = Te3 * rcp_nr(Pr.r3), Se2 = Se3 + Te3 * Rr.r3;
            const float Te1 = Te2 * rcp_nr(Pr.r2), Se1 = Se2 + Te2 * Rr.r2;
            const float Te0 = Te1 * rcp_nr(Pr.r1), Se0 = Se1 + Te1 * Rr.r1;
            float Tc = q == 3 ? Te3 : (q == 2 ? Te2 : (q == 1 ? Te1 : Te0));
            float Sc = q == 3 ? Se3 : (q == 2 ? Se2 : (q == 1 ? Se1 : Se0));
            T = Te0 * rcp_nr(Pr.r0);
            S = Se0 + Te0 * Rr.r0;
#pragma unroll
            for (int r = 3; r >= 0; --r) {
                const int k = 16 * kb + 4 * q + r;
                const float inv = iv[r];
                const float Tk = Tc * inv;
                const float wb = al[r] * Tk;
                const float dalpha = Tk * gg[r] - (Sc + TdT) * inv;
                const float wv = on[r] ? wb : 0.0f;
                // alpha < ALPHA_MAX exactly when o G was not clamped
                const float dpow = (on[r] && al[r] < ALPHA_MAX) ? dalpha * al[r] : 0.0f;
                Sc = on[r] ? __builtin_fmaf(wb, gg[r], Sc) : Sc;
                Tc = on[r] ? Tk : Tc;
                swd[n * SKW + k] = make_float2(wv, dpow);
            }
        }
        // the prefetches go to LDS before this chunk's partial stores are
        // issued (a wait for them placed later would also wait for the stores)
        if (pre_on) {
            // padding dwords: the padding record (opacity 0; a Gaussian's unit
            // eigenframe, a surfel's D = 1) and no Gaussian
            const int j = (int)threadIdx.x % RD;
            const uint32_t pad = pre_g ? 0xFFFFFFFFu
                                 : SURF ? (j == 12 ? 0x3f800000u : 0u)
                                        : (j == 4 ? 0x3f800000u : ((j == 6 || j == 7) ? 0xbf800000u : 0u));
            const uint32_t val = pre_k < nncnt ? pre : pad;
            if (pre_g)
                sgb[nn3][pre_k] = val;
            else
                reinterpret_cast<uint32_t*>(srecb[nn3])[4 * prec_slot<SURF, RG>(pre_k) + j] = val;
        }
        if (fnext_on) store_feats(fnext, sfeat2 + (f2 ^ 1) * BK * DP * FBYTES);
        __syncthreads();

        // 3. position-parallel sums over the tile's pixels: wave w takes the
        //    positions 16 (w & 1) + xi and the rows 2 (w / 2), 2 (w / 2) + 1,
        //    lane row q the 8 pixels 8 (q & 1) .. of row q / 2 of the two.
        //    The screen-space terms are moments of dL/dpower along a row: with
        //    a = e.d and b = e x d linear in d = (dx, dy), dy fixed,
        //      sum dp (q1 a e_x - q2 b e_y) = A Sx + B dy S0,
        //      sum dp (q1 a e_y + q2 b e_x) = B Sx + C dy S0,
        //    A = q1 e_x^2 + q2 e_y^2, B = (q1 - q2) e_x e_y, C = q1 e_y^2 + q2 e_x^2,
        //    S0 = sum dp, Sx = sum dp dx, Sxx = sum dp dx^2.  A surfel's nine
        //    record terms are linear in dL/dk = dp (-u/k2, -v/k2, (u^2 + v^2)/k2)
        //    = (l0, l1, l2) with coefficients from the record and (dx, dy):
        //      dx_c: -b1 L0 + b0 L1 + e2 L2,  dy_c: a1 L0 - a0 L1 + e1 L2,
        //      a0: dy L1, a1: -dy L0, b0: -L1x, b1: L0x, D: L2, e1: -dy L2, e2: -L2x.
        {
            const int k = 16 * (w & 1) + xi, row = 2 * (w >> 1) + (q >> 1), m0 = 8 * (q & 1);
            const RecT rc = lds_prec<SURF, RG>(srec, k);
            const float dy = (((float)(ty * TILE + row) + 0.5f) - rc.r0.y) - rc.r0.w;
            const float xb = (float)(tx * TILE + m0) + 0.5f;
            const float2* wd = swd + (row * TILE + m0) * SKW + k;
            const float4* dcp = sdc + row * TILE + m0;
            float qv[NQ];
            float s0 = 0.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f, ws = 0.0f;
            if constexpr (!SURF) {
                float sx = 0.0f, sxx = 0.0f;
#pragma unroll 2
                for (int m = 0; m < 8; ++m) {
                    const float2 e = wd[m * SKW];
                    const float4 dc = dcp[m];
                    const float dx = ((xb + (float)m) - rc.r0.x) - rc.r0.z;
                    const float pdx = e.y * dx;
                    s0 += e.y;
                    sx += pdx;
                    sxx = __builtin_fmaf(pdx, dx, sxx);
                    if (!odd_dc || e.x != 0.0f) {
                        c0 = __builtin_fmaf(e.x, dc.x, c0);
                        c1 = __builtin_fmaf(e.x, dc.y, c1);
                        c2 = __builtin_fmaf(e.x, dc.z, c2);
                    }
                    ws += e.x;
                }
                const float ex = rc.r1.x, ey = rc.r1.y, q1 = rc.r1.z, q2 = rc.r1.w;
                const float A = q1 * ex * ex + q2 * ey * ey, B = (q1 - q2) * ex * ey, C = q1 * ey * ey + q2 * ex * ex;
                const float sy = dy * s0;
                qv[0] = -2.0f * LN2 * (A * sx + B * sy);
                qv[1] = -2.0f * LN2 * (B * sx + C * sy);
                qv[2] = -0.5f * sxx;
                qv[3] = -dy * sx;
                qv[4] = -0.5f * dy * sy;
            } else {
                float L0 = 0.0f, L1 = 0.0f, L2 = 0.0f, L0x = 0.0f, L1x = 0.0f, L2x = 0.0f;
#pragma unroll 2
                for (int m = 0; m < 8; ++m) {
                    const float2 e = wd[m * SKW];
                    const float4 dc = dcp[m];
                    const float dx = ((xb + (float)m) - rc.r0.x) - rc.r0.z;
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
                    s0 += e.y;
                    if (!odd_dc || e.x != 0.0f) {
                        c0 = __builtin_fmaf(e.x, dc.x, c0);
                        c1 = __builtin_fmaf(e.x, dc.y, c1);
                        c2 = __builtin_fmaf(e.x, dc.z, c2);
                    }
                    ws += e.x;
                }
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
            }
            qv[NQ - 5] = s0;
            qv[NQ - 4] = c0;
            qv[NQ - 3] = c1;
            qv[NQ - 2] = c2;
            qv[NQ - 1] = ws;
#pragma unroll
            for (int m = 0; m < NQ; ++m) {
                const float sum = sum_rows(qv[m]);
                if (q == 0) sred[((w >> 1) * NQ + m) * BK + k] = sum;
            }
        }
        __syncthreads();
        if (threadIdx.x < GP * BK) {
            // terms NQ..GP-1 of a partial are padding: written as zero
            const int k = threadIdx.x % BK, m = threadIdx.x / BK;
            float sum = 0.0f;
            if (m < NQ) {
#pragma unroll
                for (int ww = 0; ww < 8; ++ww) sum += sred[(ww * NQ + m) * BK + k];
            }
            if (k < cnt) a.part_geom[((int64_t)voff + cs + k) * GP + m] = sum;
        }
        // No barrier here: the next chunk's LDS writes before its first barrier
        // (the pairs, the chunk after next's records and Gaussians, the next
        // features) go to arrays whose last readers all passed the barrier
        // above, and the row sums are written only after that next barrier,
        // which these threads reach last.
        b3 = n3;
        f2 ^= 1;
    }
}

// ---------------------------------------------------------------------------
// Fusion kernel: wave w walks pixel row w for the weights, W^T goes to LDS
// (double-buffered by chunk parity, one barrier per chunk), and the waves
// contract it with the tile's target, 16 channels a wave (NB blocks; with 8 or
// fewer, two waves share a block, one half-chunk each).  Above 256 channels one
// workgroup per (tile, 256-channel slice).  WS: also the weight sums (fusion
// without the gradient kernel).
//
// W^T rows (FP32) are 264 dwords apart, so the 16-byte operand reads of lanes
// served together fall in distinct banks; position 4 q + r of a half-chunk is
// row 4 r + q, which keeps the walk's stores (lanes q apart, same r) in
// neighbouring rows (two-way conflicts instead of four-way).
template <int NB, bool WS, bool SURF>
__global__ __launch_bounds__(1024) void k_fuse_f32(BwdArgs a, ViewTable vt) {
    using RecT = typename PrimRec<SURF>::T;
    constexpr int RW = PrimRec<SURF>::RW, RD = 4 * RW;
    constexpr int PP = TILE_PIX + 8;
    constexpr bool HALF = NB <= 8;        // two waves per channel block
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    float* sw2 = reinterpret_cast<float*>(smem);     // [2][BK][PP] W^T
    __shared__ float swsum2[2][16][BK];   // per wave (pixel row): sum over its pixels of w, per position
    __shared__ float4 srecb[3][rslots<SURF>()];

    if (a.counters->inst_overflow || a.counters->visit_overflow) return;
    const int t = blockIdx.x;
    const uint32_t nt = a.tile_niter[t];
    if (nt == 0) return;
    const int D = a.d;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int q = lane >> 4, xi = lane & 15;
    const int v = view_of_tile(vt, t);
    const int lt = t - vt.tile_off[v];
    const int tx = lt % vt.tiles_x[v], ty = lt / vt.tiles_x[v];
    const int W = vt.width[v], H = vt.height[v];
    const uint32_t voff = a.tile_voff[t];
    const int px = tx * TILE + xi, py = ty * TILE + w;
    const bool inside = px < W && py < H;
    const float x = (float)px + 0.5f, y = (float)py + 0.5f;
    const int64_t p = vt.pix_off[v] + (int64_t)(inside ? py : 0) * W + (inside ? px : 0);
    const uint32_t nit = inside ? a.n_iter[p] : 0u;
    float T = inside ? a.T_final[p] : 1.0f;
    const int d0 = (int)blockIdx.y * 256;

    // target[px = 16 s + 4 q + i][channel]: the B operands of this wave's block
    // (pixels outside the image and channels past the width as zero)
    const int blk = HALF ? w >> 1 : w, ch = d0 + 16 * blk + xi;
    const bool mine = blk < NB && d0 + 16 * blk < D;
    float4 tg[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) tg[s] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (mine) {
        const int chc = ch < D ? ch : D - 1;
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            const int qy = ty * TILE + s;
            float e[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int qx = tx * TILE + 4 * q + i;
                const int64_t at = (vt.pix_off[v] + (int64_t)(qy < H ? qy : H - 1) * W + (qx < W ? qx : W - 1)) * D + chc;
                e[i] = a.target_bf16 ? bf16_to_f32(static_cast<const uint16_t*>(a.target)[at])
                                     : static_cast<const float*>(a.target)[at];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (qy >= H || tx * TILE + 4 * q + i >= W || ch >= D) e[i] = 0.0f;
            tg[s] = make_float4(e[0], e[1], e[2], e[3]);
        }
    }
    {
        const int cs0 = (int)nt - BK > 0 ? (int)nt - BK : 0;
        const int cs1 = cs0 - BK > 0 ? cs0 - BK : 0;
        const int c = (int)threadIdx.x / BK, k = (int)threadIdx.x % BK;
        if (c < 2) {
            const int cs = c ? cs1 : cs0, cnt = c ? cs0 - cs1 : (int)nt - cs0;
            RecT r = pad_rec<SURF>();
            if (k < cnt) r = load_rec<SURF>(a.vrec, (int64_t)voff + cs + k);
            lds_put_prec<SURF, RG>(srecb[c], k, r);
        }
    }
    __syncthreads();
    int b3 = 0, b2 = 0;
    for (int ce = (int)nt; ce > 0; ce -= BK) {
        const int cs = ce - BK > 0 ? ce - BK : 0;
        const int cnt = ce - cs;
        const int n3 = b3 == 2 ? 0 : b3 + 1, nn3 = n3 == 2 ? 0 : n3 + 1;
        const float4* srec = srecb[b3];
        float* sw = sw2 + b2 * BK * PP;
        // the records of the chunk after next, one dword per thread (as in the
        // gradient kernel)
        const int ncs = cs - BK > 0 ? cs - BK : 0;
        const int nncs = ncs - BK > 0 ? ncs - BK : 0;
        const int nncnt = ncs - nncs;
        const bool pre_on = ncs > 0 && threadIdx.x < RD * BK;
        uint32_t pre = 0u;
        if (pre_on) pre = (reinterpret_cast<const uint32_t*>(a.vrec) + ((int64_t)voff + nncs) * RD)[threadIdx.x];
        const int n = w * TILE + xi;
#pragma unroll
        for (int kb = 1; kb >= 0; --kb) {
            float al[4];
            bool on[4];
            float P = 1.0f;
#pragma unroll
            for (int r = 3; r >= 0; --r) {
                const int k = 16 * kb + 4 * q + r;
                const float4* rp = srec + (4 * RW + 1) * q + (16 * RW + 4) * kb + RW * r;   // slot of k
                RecT rc;
                rc.r0 = rp[0];
                rc.r1 = rp[1];
                rc.r2.x = rp[2].x;
                if constexpr (SURF) rc.r3 = rp[3];
                const float alpha = prim_alpha<SURF>(rc, x, y);
                on[r] = k < cnt && (uint32_t)(cs + k) < nit && alpha >= ALPHA_MIN;
                al[r] = alpha;
                P = on[r] ? P * (1.0f - al[r]) : P;
            }
            const Rows4 Pr = rows4(P);
            const float Te3 = T, Te2 = Te3 * rcp_nr(Pr.r3), Te1 = Te2 * rcp_nr(Pr.r2), Te0 = Te1 * rcp_nr(Pr.r1);
            float Tc = q == 3 ? Te3 : (q == 2 ? Te2 : (q == 1 ? Te1 : Te0));
            T = Te0 * rcp_nr(Pr.r0);
#pragma unroll
            for (int r = 3; r >= 0; --r) {
                const float Tk = Tc * rcp_nr(1.0f - al[r]);
                const float wv = on[r] ? al[r] * Tk : 0.0f;
                Tc = on[r] ? Tk : Tc;
                sw[(16 * kb + 4 * r + q) * PP + n] = wv;
                if (WS && d0 == 0) {
                    // the row's weight sum of the position: butterfly over the 16 pixels
                    float rs = wv;
#pragma unroll
                    for (int off = 1; off < 16; off <<= 1) rs += __shfl_xor(rs, off, 64);
                    if (xi == 0) swsum2[b2][w][16 * kb + 4 * q + r] = rs;
                }
            }
        }
        if (pre_on) {
            const int j = (int)threadIdx.x % RD, k = (int)threadIdx.x / RD;
            const uint32_t pad = SURF ? (j == 12 ? 0x3f800000u : 0u)
                                      : (j == 4 ? 0x3f800000u : ((j == 6 || j == 7) ? 0xbf800000u : 0u));
            reinterpret_cast<uint32_t*>(srecb[nn3])[4 * prec_slot<SURF, RG>(k) + j] = k < nncnt ? pre : pad;
        }
        __syncthreads();
        // weight sums per instance: the 16 rows in order
        if (WS && d0 == 0 && threadIdx.x < BK) {
            const int k = threadIdx.x;
            float ws = 0.0f;
#pragma unroll
            for (int ww = 0; ww < 16; ++ww) ws += swsum2[b2][ww][k];
            if (k < cnt) a.part_geom[((int64_t)voff + cs + k) * PrimRec<SURF>::GP + PrimRec<SURF>::WSLOT] = ws;
        }
        // out[k][c] = sum_px W^T[k][px] target[px][c]
        auto contract = [&](int kb) {
            f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 16; s += 2) {
                const float4 a0 = *reinterpret_cast<const float4*>(&sw[(16 * kb + xi) * PP + 16 * s + 4 * q]);
                const float4 a1 = *reinterpret_cast<const float4*>(&sw[(16 * kb + xi) * PP + 16 * (s + 1) + 4 * q]);
                acc0 = mfma4(a0.x, tg[s].x, acc0);
                acc1 = mfma4(a1.x, tg[s + 1].x, acc1);
                acc0 = mfma4(a0.y, tg[s].y, acc0);
                acc1 = mfma4(a1.y, tg[s + 1].y, acc1);
                acc0 = mfma4(a0.z, tg[s].z, acc0);
                acc1 = mfma4(a1.z, tg[s + 1].z, acc1);
                acc0 = mfma4(a0.w, tg[s].w, acc0);
                acc1 = mfma4(a1.w, tg[s + 1].w, acc1);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int k = 16 * kb + 4 * r + q;   // (row 4 q + r holds position 4 r + q)
                if (k < cnt && ch < D) a.part_fuse[((int64_t)voff + cs + k) * D + ch] = acc0[r] + acc1[r];
            }
        };
        if (mine) {
            if constexpr (HALF) {
                contract(w & 1);
            } else {
                contract(0);
                contract(1);
            }
        }
        // No barrier here: before its barrier the next chunk writes the other
        // W^T and weight-sum buffers and a record buffer whose last readers all
        // passed the barrier above.
        b3 = n3;
        b2 ^= 1;
    }
}

// ---------------------------------------------------------------------------
template <int NS, bool FB, bool SURF, bool STREAM>
void launch_grad(const BwdArgs& a, const ViewTable& vt, int n_tiles, hipStream_t s) {
    constexpr int DC = 16 * NS, DP = FB ? DC + 16 : DC + 8;
    const size_t lds = sizeof(float2) * TILE_PIX * SKW + sizeof(float4) * TILE_PIX +
                       sizeof(float) * 8 * PrimRec<SURF>::NQ * BK +
                       (NS > 0 ? (size_t)(STREAM ? 1 : 2) * BK * DP * (FB ? 2 : 4) : 0);
    // 16-byte (BF16: 8-byte) feature and dF loads where every row is aligned to them
    const int vec_f = a.d % 4 == 0 && reinterpret_cast<uintptr_t>(a.feat) % (FB ? 8 : 16) == 0;
    const int vec_df = a.d % 4 == 0 && reinterpret_cast<uintptr_t>(a.dF) % 16 == 0;
    hipLaunchKernelGGL((k_bwd_f32<NS, FB, SURF, STREAM>), dim3(n_tiles), dim3(1024), lds, s, a, vt, vec_f, vec_df);
}

template <bool FB, bool SURF>
void launch_grad_d(const BwdArgs& a, const ViewTable& vt, int n_tiles, hipStream_t s) {
    const int ns = a.dF ? (a.d + 15) / 16 : 0;
    if (ns == 0) launch_grad<0, FB, SURF, false>(a, vt, n_tiles, s);
    else if (ns == 1) launch_grad<1, FB, SURF, false>(a, vt, n_tiles, s);
    else if (ns == 2) launch_grad<2, FB, SURF, false>(a, vt, n_tiles, s);
    else if (ns <= 4) launch_grad<4, FB, SURF, false>(a, vt, n_tiles, s);
    else if (ns <= 8) launch_grad<8, FB, SURF, false>(a, vt, n_tiles, s);
    else if (ns <= 16) launch_grad<16, FB, SURF, false>(a, vt, n_tiles, s);
    else launch_grad<16, FB, SURF, true>(a, vt, n_tiles, s);
}

template <int NB, bool SURF>
void launch_fuse(const BwdArgs& a, const ViewTable& vt, int n_tiles, bool grads, hipStream_t s) {
    const size_t lds = sizeof(float) * 2 * BK * (TILE_PIX + 8);
    const dim3 grid(n_tiles, (a.d + 255) / 256);
    if (grads)
        hipLaunchKernelGGL((k_fuse_f32<NB, false, SURF>), grid, dim3(1024), lds, s, a, vt);
    else
        hipLaunchKernelGGL((k_fuse_f32<NB, true, SURF>), grid, dim3(1024), lds, s, a, vt);
}

template <bool SURF>
void launch_f32(const BwdArgs& a, const ViewTable& vt, int n_tiles, bool grads, bool fuse, hipStream_t s) {
    if (grads) {
        if (a.feat_bf16)
            launch_grad_d<true, SURF>(a, vt, n_tiles, s);
        else
            launch_grad_d<false, SURF>(a, vt, n_tiles, s);
    }
    if (fuse) {
        if (a.d <= 128)
            launch_fuse<8, SURF>(a, vt, n_tiles, grads, s);
        else
            launch_fuse<16, SURF>(a, vt, n_tiles, grads, s);
    }
}

}  // namespace

// grads: the gradient kernel (needs dC); fuse: the fusion kernel (needs the target)
void launch_render_bwd_f32(const BwdArgs& a, const ViewTable& vt, int n_tiles, bool grads, bool fuse, hipStream_t s) {
    if (a.prim == FH_PRIM_SURFEL)
        launch_f32<true>(a, vt, n_tiles, grads, fuse, s);
    else
        launch_f32<false>(a, vt, n_tiles, grads, fuse, s);
}

}  // namespace fh
