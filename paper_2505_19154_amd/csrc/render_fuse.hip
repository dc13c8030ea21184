// Feature fusion: per visited instance the partial sum_p w(p) target(p) over the
// tile's pixels (gfx950), both arithmetic forms.
//
// Per tile, back to front over the visited list in chunks of 16 positions: one
// workgroup, four waves of which walk 64 pixels each, one per lane (w =
// alpha T, T recovered by division as in the gradient kernel; the chunk's
// records, one position per lane, reach the walk as DPP row broadcasts).  W^T
// goes to LDS (double-buffered, one barrier a chunk) and the waves contract it
// with the tile's target, W^T[16 x 256 px] . Target[256 px x channels], each wave
// with its share of the channels held in registers for the whole tile.
//
// BF16 targets: W as BF16 terms on v_mfma_f32_16x16x32_bf16, two (hi + lo, about
// 16 significant bits) in the BF16 form, three in the FP32 form (exact: three
// roundings to 8 bits cover 24), the target as stored.  The target comes
// through LDS in rows of pixels and is read transposed (ds_read_b64_tr_b16)
// into operands, instead of one 2-byte load per element.  FP32 targets (FP32
// form): k_fuse_f32 below, FP32 operands on v_mfma_f32_16x16x4_f32.
//
// WS: also the weight sums (fusion without the gradient kernel, which writes
// them otherwise).  SURF: the surfel primitive.
//
// Bound: VALU of the walk (alpha and T, about 25 instructions a position) beside
// the target's one read.  Reading weights recorded by the gradient kernel
// instead costs 1 KB written and read a visit: 128 channels, 1M Gaussians in 16
// views 4.14 ms with, 3.36 ms without; 256 channels, 500k at 1920x1080 0.66 and
// 0.72 ms, but 0.2 ms of recording in the gradient kernel.  Images of few tiles are
// bound by the chain of the walk instead (PARTS, BF16 form): the gradient kernel
// leaves T at every 128th position (8 bytes a visit), and the segments of a list run
// side by side (lists of 7,900 positions in 16 tiles: 1.00 ms for the whole walk).
#include <type_traits>
#include <utility>

#include "kernels.hpp"

namespace fh {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace {

constexpr int CK = 16;                   // positions per chunk
// W^T rows and staged target rows: 544 bytes apart, an odd multiple of 32, so
// that the rows read together fall in distinct banks
constexpr int PP = TILE_PIX + 16;

template <int K>
__device__ __forceinline__ float row_bcast(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x150 + K, 0xf, 0xf, true));
}
template <int K>
__device__ __forceinline__ Rec bcast_rec(const Rec& r) {
    Rec o;
    o.r0 = make_float4(row_bcast<K>(r.r0.x), row_bcast<K>(r.r0.y), row_bcast<K>(r.r0.z), row_bcast<K>(r.r0.w));
    o.r1 = make_float4(row_bcast<K>(r.r1.x), row_bcast<K>(r.r1.y), row_bcast<K>(r.r1.z), row_bcast<K>(r.r1.w));
    o.r2 = make_float4(row_bcast<K>(r.r2.x), 0.f, 0.f, 0.f);
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
// 1 / x to within one rounding (one Newton step): T is carried from position
// to position by it, so its error is summed along a pixel's walk.
__device__ __forceinline__ float rcp1(float x) {
    const float r = __builtin_amdgcn_rcpf(x);
    return __builtin_fmaf(__builtin_fmaf(-x, r, 1.0f), r, r);
}
template <int CTRL>
__device__ __forceinline__ float add_dpp(float v) {
    return v + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
// sum over the lane's 16-lane row
__device__ __forceinline__ float row_sum(float v) {
    v = add_dpp<0xB1>(v);          // quad_perm 1 0 3 2
    v = add_dpp<0x4E>(v);          // quad_perm 2 3 0 1
    v = add_dpp<0x141>(v);         // row_half_mirror
    return add_dpp<0x140>(v);      // row_mirror
}

// NB: 16-channel blocks per wave (16 NB WAVES channels a workgroup, blockIdx.y
// slices).  WAVES = 8, above 128 channels: the first four waves walk, all eight
// contract 32 channels each.  With four waves of 64 channels the target alone
// held 128 registers a lane, two waves a SIMD; the barriers at the chunk ends
// and the MFMA chains showed: 500k Gaussians at 1920x1080, D = 256, three terms
// 0.78 -> 0.70 ms, two terms 0.71 -> 0.69.  Up to 128 channels four waves fit.
template <int TERMS, int NB, int WAVES, bool WS, bool SURF, bool PARTS>
__global__ __launch_bounds__(64 * WAVES, WAVES == 8 ? 4 : 3) void k_fuse(BwdArgs a, ViewTable vt, int vec) {
    using RecT = typename PrimRec<SURF>::T;
    constexpr int DS = 16 * NB * WAVES;               // channels of this workgroup
    constexpr int TST = DS + 16;                      // staged target row stride (an odd multiple of 32 bytes)
    constexpr int WEL = 2 * TERMS * CK * PP, TEL = 2 * 32 * TST;
    // W^T [2 buffers][terms][CK][PP]; before the walk, two slabs of 32 target pixels
    __shared__ __attribute__((aligned(16))) uint16_t smem[WEL > TEL ? WEL : TEL];
    __shared__ float swsum[WS ? 2 : 1][CK][16];       // weight sum of every pixel row per position
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
    const int d0 = (int)blockIdx.y * DS;
    const int px = tx * TILE + xi, prow = 4 * w + q, py = ty * TILE + prow;
    const float x = (float)px + 0.5f, y = (float)py + 0.5f;
    const bool walks = WAVES == 4 || w < 4;           // (the waves that hold the tile's pixels)
    const bool inside = walks && px < W && py < H;
    const int64_t p = vt.pix_off[v] + (int64_t)(inside ? py : 0) * W + (inside ? px : 0);
    const int nit = inside ? (int)a.n_iter[p] : 0;
    float T = inside ? a.T_final[p] : 1.0f;
    auto at = [&](int cs) { return voff + (cs + xi < nt ? cs + xi : nt - 1); };
    // PARTS: segments blockIdx.z, blockIdx.z + gridDim.z, ... of the list, counted
    // from its end, each from the T that the gradient walk left there
    const int len = PARTS ? T_SEG : nt;
    int end = nt - (PARTS ? (int)blockIdx.z * len : 0);
    if (PARTS && end <= 0) return;
    int first = PARTS && end > len ? end - len : 0;
    int cs = end - CK > first ? end - CK : first;
    RecT rc = load_rec<SURF>(a.vrec, at(cs));

    // target operands of this wave's channels d0 + 16 (NB w + j) + xi: slab s, lane
    // row q, elements m: pixels 32 s + 4 q + m and (m >= 4) 32 s + 16 + 4 q + m - 4
    bf16x8 tg[NB][8];
    {
        constexpr int IT = 32 * (DS / 8) / (64 * WAVES);   // 8-channel items per thread and slab
        uint4 raw[IT];
        const uint16_t* src = static_cast<const uint16_t*>(a.target);
        auto load = [&](int s) {
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int idx = (int)threadIdx.x + 64 * WAVES * it, k = idx / (DS / 8), c = d0 + 8 * (idx % (DS / 8));
                const int qy = ty * TILE + 2 * s + (k >> 4), qx = tx * TILE + (k & 15);
                raw[it] = make_uint4(0u, 0u, 0u, 0u);
                if (qy < H && qx < W) {
                    const uint16_t* e = src + (vt.pix_off[v] + (int64_t)qy * W + qx) * a.d + c;
                    if (vec) {
                        if (c < a.d) raw[it] = *reinterpret_cast<const uint4*>(e);
                    } else {
                        uint32_t h[8];
#pragma unroll
                        for (int m = 0; m < 8; ++m) h[m] = c + m < a.d ? e[m] : 0u;
                        raw[it] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
                    }
                }
            }
        };
        load(0);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            uint16_t* st = smem + (s & 1) * 32 * TST;
#pragma unroll
            for (int it = 0; it < IT; ++it) {
                const int idx = (int)threadIdx.x + 64 * WAVES * it, k = idx / (DS / 8), c = 8 * (idx % (DS / 8));
                *reinterpret_cast<uint4*>(st + k * TST + c) = raw[it];
            }
            if (s < 7) load(s + 1);
            __syncthreads();
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                // (transposed read: lanes 4 r .. 4 r + 3 of a lane row give row r's 16
                // columns, lane i gets column i of the four rows)
                const uint16_t* b = st + (4 * q + (xi >> 2)) * TST + 16 * (NB * w + j) + 4 * (xi & 3);
                typedef __attribute__((address_space(3))) s16x4 lds4;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)(b));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)(b + 16 * TST));
                const uint2 l2 = __builtin_bit_cast(uint2, lo), h2 = __builtin_bit_cast(uint2, hi);
                tg[j][s] = __builtin_bit_cast(bf16x8, make_uint4(l2.x, l2.y, h2.x, h2.y));
            }
        }
        __syncthreads();   // (the staging area becomes W^T)
    }
    // column of the lane's pixel in a W^T row, in the order of the target operands
    const int col = 32 * (prow >> 1) + 8 * (xi >> 2) + 4 * (prow & 1) + (xi & 3);
    int buf = 0;
    for (;;) {
        if constexpr (PARTS)
            if (end < nt && inside)
                T = a.tseg[(voff / T_SEG + t + (nt - end) / T_SEG - 1) * TILE_PIX + prow * TILE + xi];
        for (int ce = end; ce > first; ce -= CK, buf ^= 1) {
            const int cnt = ce - cs, ncs = cs - CK > first ? cs - CK : first;
            const RecT rn = load_rec<SURF>(a.vrec, at(ncs));
            uint16_t* sw = smem + buf * TERMS * CK * PP;
            const int rem = nit - cs < cnt ? nit - cs : cnt;
            if (walks) unroll_seq(std::make_integer_sequence<int, CK>{}, [&](auto kc) {
                constexpr int k = CK - 1 - decltype(kc)::value;
                const float alpha = prim_alpha<SURF>(bcast_rec<k>(rc), x, y);
                const float al = (alpha >= ALPHA_MIN && k < rem) ? alpha : 0.0f;
                T = T * rcp1(1.0f - al);
                const float wv = al * T;
                float rest = wv;
#pragma unroll
                for (int c = 0; c < TERMS; ++c) {
                    const __bf16 b = (__bf16)rest;
                    sw[(c * CK + k) * PP + col] = __builtin_bit_cast(uint16_t, b);
                    rest -= (float)b;
                }
                if constexpr (WS) {
                    const float rs = row_sum(wv);
                    if (xi == 0) swsum[buf][k][prow] = rs;
                }
            });
            __syncthreads();
            if (WS && d0 == 0 && (int)threadIdx.x < cnt) {
                float ws = 0.0f;
#pragma unroll
                for (int r = 0; r < 16; ++r) ws += swsum[buf][threadIdx.x][r];
                a.part_geom[(voff + cs + threadIdx.x) * PrimRec<SURF>::GP + PrimRec<SURF>::WSLOT] = ws;
            }
            if (d0 + 16 * NB * w < a.d) {
                f32x4 acc[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int c = TERMS - 1; c >= 0; --c) {      // (small terms first)
#pragma unroll
                    for (int s = 0; s < 8; ++s) {
                        const bf16x8 av = *reinterpret_cast<const bf16x8*>(sw + (c * CK + xi) * PP + 32 * s + 8 * q);
#pragma unroll
                        for (int j = 0; j < NB; ++j)
                            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, tg[j][s], acc[j], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int k = 4 * q + r;
                    if (k < cnt) {
                        float* o = a.part_fuse + (voff + cs + k) * a.d + d0 + 16 * NB * w + xi;
#pragma unroll
                        for (int j = 0; j < NB; ++j)
                            if (d0 + 16 * (NB * w + j) + xi < a.d) o[16 * j] = acc[j][r];
                    }
                }
            }
            // No second barrier: the next chunk writes the other buffers, whose last
            // readers all passed the barrier above.
            rc = rn;
            cs = ncs;
        }
        end -= PARTS ? (int)gridDim.z * len : nt;
        if (end <= 0) break;
        first = end > len ? end - len : 0;
        cs = end - CK > first ? end - CK : first;
        rc = load_rec<SURF>(a.vrec, at(cs));
    }
}

constexpr int BK = 32;          // positions per chunk of k_fuse_f32
constexpr int RG = 4;           // record padding group: the walk's lane rows read records 4 apart
template <bool SURF>
constexpr int rslots() {
    return PrimRec<SURF>::RW * BK + BK / RG;
}
__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// FP32 targets: wave w walks pixel row w for the weights (each pixel's four lanes
// take four consecutive positions each, their transmittance combined by a
// scan), chunks of 32 positions; W^T goes to LDS
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
    constexpr int PPF = TILE_PIX + 8;
    constexpr bool HALF = NB <= 8;        // two waves per channel block
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    float* sw2 = reinterpret_cast<float*>(smem);     // [2][BK][PPF] W^T
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
        float* sw = sw2 + b2 * BK * PPF;
        // the records of the chunk after next, one dword per thread
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
            const float Te3 = T, Te2 = Te3 * rcp1(Pr.r3), Te1 = Te2 * rcp1(Pr.r2), Te0 = Te1 * rcp1(Pr.r1);
            float Tc = q == 3 ? Te3 : (q == 2 ? Te2 : (q == 1 ? Te1 : Te0));
            T = Te0 * rcp1(Pr.r0);
#pragma unroll
            for (int r = 3; r >= 0; --r) {
                const float Tk = Tc * rcp1(1.0f - al[r]);
                const float wv = on[r] ? al[r] * Tk : 0.0f;
                Tc = on[r] ? Tk : Tc;
                sw[(16 * kb + 4 * r + q) * PPF + n] = wv;
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
                const float4 a0 = *reinterpret_cast<const float4*>(&sw[(16 * kb + xi) * PPF + 16 * s + 4 * q]);
                const float4 a1 = *reinterpret_cast<const float4*>(&sw[(16 * kb + xi) * PPF + 16 * (s + 1) + 4 * q]);
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
template <int TERMS, int NB, int WAVES, bool SURF>
void launch_nb(const BwdArgs& a, const ViewTable& vt, int n_tiles, bool ws, hipStream_t s) {
    // 16-byte target loads where every row is aligned to them
    const int vec = a.d % 8 == 0 && reinterpret_cast<uintptr_t>(a.target) % 16 == 0;
    constexpr int DS = 16 * NB * WAVES;
    const dim3 grid(n_tiles, (a.d + DS - 1) / DS), block(64 * WAVES);
    if (ws)
        hipLaunchKernelGGL((k_fuse<TERMS, NB, WAVES, true, SURF, false>), grid, block, 0, s, a, vt, vec);
    else if (TERMS == 2 && a.tseg)
        hipLaunchKernelGGL((k_fuse<2, NB, WAVES, false, SURF, true>), dim3(grid.x, grid.y, list_parts(n_tiles)), block, 0, s, a,
                           vt, vec);
    else
        hipLaunchKernelGGL((k_fuse<TERMS, NB, WAVES, false, SURF, false>), grid, block, 0, s, a, vt, vec);
}

template <int TERMS, bool SURF>
void launch_terms(const BwdArgs& a, const ViewTable& vt, int n_tiles, bool ws, hipStream_t s) {
    if (a.d <= 64) launch_nb<TERMS, 1, 4, SURF>(a, vt, n_tiles, ws, s);
    else if (a.d <= 128) launch_nb<TERMS, 2, 4, SURF>(a, vt, n_tiles, ws, s);
    else launch_nb<TERMS, 2, 8, SURF>(a, vt, n_tiles, ws, s);
}

template <int NB, bool SURF>
void launch_f32(const BwdArgs& a, const ViewTable& vt, int n_tiles, bool ws, hipStream_t s) {
    const size_t lds = sizeof(float) * 2 * BK * (TILE_PIX + 8);
    const dim3 grid(n_tiles, (a.d + 255) / 256);
    if (ws)
        hipLaunchKernelGGL((k_fuse_f32<NB, true, SURF>), grid, dim3(1024), lds, s, a, vt);
    else
        hipLaunchKernelGGL((k_fuse_f32<NB, false, SURF>), grid, dim3(1024), lds, s, a, vt);
}

template <bool SURF>
void launch_fuse(const BwdArgs& a, const ViewTable& vt, int n_tiles, bool bf16, bool ws, hipStream_t s) {
    if (bf16) launch_terms<2, SURF>(a, vt, n_tiles, ws, s);
    else if (a.target_bf16) launch_terms<3, SURF>(a, vt, n_tiles, ws, s);
    else if (a.d <= 128) launch_f32<8, SURF>(a, vt, n_tiles, ws, s);
    else launch_f32<16, SURF>(a, vt, n_tiles, ws, s);
}

}  // namespace

void launch_render_fuse(const BwdArgs& a, const ViewTable& vt, int n_tiles, bool bf16, bool ws, hipStream_t s) {
    if (a.prim == FH_PRIM_SURFEL)
        launch_fuse<true>(a, vt, n_tiles, bf16, ws, s);
    else
        launch_fuse<false>(a, vt, n_tiles, bf16, ws, s);
}

}  // namespace fh
