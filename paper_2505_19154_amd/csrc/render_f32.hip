// Front-to-back compositing in the FP32 form, for the widths and storage types
// that the split-BF16 forward (render_bf16.hip) does not take, and small
// kernels around it.
//
// Forward (Section 3.1): for every pixel, walk its tile's depth-sorted list;
//   alpha = min(0.99, o G), skip if alpha < 1/255, stop before T drops below
//   1e-4, w = alpha T, C += w rgb, F += w f, T *= (1 - alpha).
//
#include <type_traits>

#include "kernels.hpp"

namespace fh {

__device__ __forceinline__ uint32_t inst_rank(const uint32_t* keys, const uint32_t* vals, int64_t i, int rank_bits,
                                              int packed) {
    return packed ? (keys[i] & ((1u << rank_bits) - 1u)) : vals[i];
}

__device__ __forceinline__ float load_feat(const void* f, int bf16, int64_t idx) {
    return bf16 ? bf16_to_f32(static_cast<const uint16_t*>(f)[idx]) : static_cast<const float*>(f)[idx];
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ float lo_f32(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float hi_f32(uint32_t p) { return __uint_as_float(p & 0xFFFF0000u); }

// One 256-thread workgroup per (tile, slice of 16 NB channels); wave w owns the
// pixel rows 4 w .. 4 w + 3, one pixel per lane.  The walk is sequential per
// pixel (the transmittance is the product in list order); the alphas of four
// positions are evaluated ahead of it, so that their latency overlaps.  The
// weights of 16 positions go to LDS that only this wave reads, and the wave
// contracts them with the staged features on the FP32 matrix unit,
//   F[64 px x 16 NB] += W[64 px x 16] . Feat[16 x 16 NB]
// (v_mfma_f32_16x16x4_f32; BF16-stored features: FB below), so a slice of 128
// channels walks once where FMAs from LDS took slices of 16 to 64.  Records, Gaussians and
// features are staged a chunk of 32 positions at a time, requested one to three
// chunks ahead (as in render_bf16.hip).  Bound: VALU work of the walk (about 30
// instructions per pixel and position), then the FP32 matrix rate at 256
// channels.  Against the VALU form: 500k, 1920x1080, D = 256 (BF16 storage)
// 5.57 -> 2.50 ms; 150k, 987x657, D = 0 123 -> 86 us; 1k, 128x128, D = 16 69 ->
// 45 us.
//
// FB: features stored in BF16.  They enter v_mfma_f32_16x16x32_bf16 as stored and
// W as three BF16 terms (h + m + l: exact, three roundings to 8 bits cover 24), 32
// positions at once, so that only the FP32 accumulation rounds: 48 cycles for 32
// positions of a 16 x 16 block where the FP32 instruction takes 256 (D = 256 above
// 2.50 -> 1.36 ms).  Features stay in rows of positions in LDS (32 (NB | 1) bytes
// apart, position 8 q + m in row 4 q + m or 16 + 4 q + m - 4) and are read transposed.
template <int NB, bool FB, bool SURF>
__global__ __launch_bounds__(256, 2) void k_render_fwd_f32(RenderArgs a, ViewTable vt, int vec) {
    using RecT = typename PrimRec<SURF>::T;
    constexpr int FK = 32;                               // positions per chunk
    constexpr int DS = 16 * NB;
    constexpr int FST = DS % 32 == 0 ? DS + 16 : DS;     // feature row stride: lanes q (rows apart) 16 dwords apart mod 64
    constexpr int WST = FB ? 66 : 64 + 16;               // weight row stride, the same (FB: lanes q are 8 rows apart)
    constexpr int WROWS = FB ? FK : 16;
    constexpr int FROW = 32 * (NB | 1);                  // FB: bytes of a feature row
    constexpr int GE = 4;                                // positions evaluated ahead of the walk
    constexpr int NG = NB > 0 ? 4 * NB : 1;              // four-channel items per feature row
    constexpr int ITEMS = NB > 0 ? FK * NG : 0, NI = NB > 0 ? (ITEMS + 255) / 256 : 1;
    __shared__ RecT srec[3][FK];
    __shared__ uint32_t sg[3][FK];
    __shared__ __attribute__((aligned(16))) float sft[NB > 0 ? (FB ? 2 * FK * FROW / 4 : 2 * FK * FST) : 4];
    __shared__ float sw[NB > 0 ? 4 * WROWS * WST : 4];
    __shared__ uint32_t smax[4], sodd;
    __shared__ __attribute__((aligned(4))) uint8_t sbusy[2][4];   // per wave: a pixel still walking (read as one word)
    static_assert(__alignof__(sbusy) >= 4, "the four flags are read as one word");
    if (a.counters->inst_overflow) return;
    const int t = blockIdx.x, slice = blockIdx.y, d0 = slice * DS;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int q = lane >> 4, xi = lane & 15;
    const int v = view_of_tile(vt, t);
    const int lt = t - vt.tile_off[v];
    const int tx = lt % vt.tiles_x[v], ty = lt / vt.tiles_x[v];
    const int px = tx * TILE + xi, py = ty * TILE + 4 * w + q;
    const bool inside = px < vt.width[v] && py < vt.height[v];
    const float x = (float)px + 0.5f, y = (float)py + 0.5f;
    const uint32_t s = a.ranges[2 * t], len = a.ranges[2 * t + 1] - s;
    const int k = (int)threadIdx.x;   // list position within a chunk (threads 0..FK-1)

    auto rank_at = [&](uint32_t pos) { return pos < len ? inst_rank(a.keys, a.vals, (int64_t)s + pos, a.rank_bits, a.packed) : 0u; };
    auto get_rec = [&](uint32_t j, RecT& r, uint32_t& g) {
        r = load_rec<SURF>(a.rrec, j);
        g = a.order[j];
    };
    auto put_rec = [&](int buf, uint32_t pos, const RecT& r, uint32_t g) {
        const bool real = pos < len;
        srec[buf][k] = real ? r : pad_rec<SURF>();   // padding: opacity 0 never blends
        sg[buf][k] = real ? g : 0xFFFFFFFFu;
    };
    using Item = typename std::conditional<FB, uint2, float4>::type;   // four channels as stored
    auto load_feats = [&](const uint32_t* gl, Item* fr) {
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const int idx = (int)threadIdx.x + 256 * it;
            fr[it] = Item{};
            if (idx < ITEMS) {
                const uint32_t g = gl[idx / NG];
                const int c = d0 + 4 * (idx % NG);
                if (g != 0xFFFFFFFFu) {
                    if constexpr (FB) {
                        const uint16_t* f = static_cast<const uint16_t*>(a.feat) + (int64_t)g * a.d;
                        if (vec) {
                            if (c < a.d) fr[it] = *reinterpret_cast<const uint2*>(f + c);
                        } else {
                            const uint32_t e0 = c < a.d ? f[c] : 0u, e1 = c + 1 < a.d ? f[c + 1] : 0u;
                            const uint32_t e2 = c + 2 < a.d ? f[c + 2] : 0u, e3 = c + 3 < a.d ? f[c + 3] : 0u;
                            fr[it] = make_uint2(e0 | (e1 << 16), e2 | (e3 << 16));
                        }
                    } else {
                        const float* f = static_cast<const float*>(a.feat) + (int64_t)g * a.d;
                        if (vec) {
                            if (c < a.d) fr[it] = *reinterpret_cast<const float4*>(f + c);
                        } else {
                            fr[it] = make_float4(c < a.d ? f[c] : 0.f, c + 1 < a.d ? f[c + 1] : 0.f,
                                                 c + 2 < a.d ? f[c + 2] : 0.f, c + 3 < a.d ? f[c + 3] : 0.f);
                        }
                    }
                }
            }
        }
    };
    // (a feature that is not finite enters the contraction as zero, 0 * inf must
    // not reach the pixels that do not blend it, and is added at the end)
    auto store_feats = [&](const Item* fr, int buf) {
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const int idx = (int)threadIdx.x + 256 * it;
            if (idx < ITEMS) {
                const int kk = idx / NG, cg = idx % NG;
                if constexpr (FB) {
                    uint2 f = fr[it];
                    const uint32_t EXP = 0x7F80u;
                    const bool o0 = (f.x & EXP) == EXP, o1 = ((f.x >> 16) & EXP) == EXP;
                    const bool o2 = (f.y & EXP) == EXP, o3 = ((f.y >> 16) & EXP) == EXP;
                    if (o0 || o1 || o2 || o3) {
                        sodd = 1u;
                        f.x &= (o0 ? 0u : 0xFFFFu) | (o1 ? 0u : 0xFFFF0000u);
                        f.y &= (o2 ? 0u : 0xFFFFu) | (o3 ? 0u : 0xFFFF0000u);
                    }
                    const int row = (kk & 3) | ((kk >> 1) & 12) | ((kk & 4) << 2);
                    *reinterpret_cast<uint2*>(reinterpret_cast<unsigned char*>(sft) + (buf * FK + row) * FROW + 8 * cg) = f;
                } else {
                    float4 f = fr[it];
                    if (!(isfinite(f.x) && isfinite(f.y) && isfinite(f.z) && isfinite(f.w))) {
                        sodd = 1u;
                        f.x = isfinite(f.x) ? f.x : 0.0f;
                        f.y = isfinite(f.y) ? f.y : 0.0f;
                        f.z = isfinite(f.z) ? f.z : 0.0f;
                        f.w = isfinite(f.w) ? f.w : 0.0f;
                    }
                    *reinterpret_cast<float4*>(&sft[buf * FK * FST + kk * FST + 4 * cg]) = f;
                }
            }
        }
    };

    // prologue: chunks 0 and 1 into LDS, chunk 2's ranks into registers, then chunk 0's features
    uint32_t rk2 = 0u;
    if (threadIdx.x == 0) sodd = 0u;
    if (threadIdx.x < 8) reinterpret_cast<uint8_t*>(sbusy)[threadIdx.x] = 0;
    if (k < FK && len > 0) {
        RecT r0, r1;
        uint32_t g0, g1;
        const uint32_t j0 = rank_at((uint32_t)k), j1 = rank_at((uint32_t)(FK + k));
        rk2 = rank_at((uint32_t)(2 * FK + k));
        get_rec(j0, r0, g0);
        get_rec(j1, r1, g1);
        put_rec(0, (uint32_t)k, r0, g0);
        put_rec(1, (uint32_t)(FK + k), r1, g1);
    }
    __syncthreads();
    if (NB > 0 && len > 0) {
        Item fr[NI];
        load_feats(sg[0], fr);
        store_feats(fr, 0);
    }
    __syncthreads();

    f32x4 acc[4][NB > 0 ? NB : 1];
#pragma unroll
    for (int pb = 0; pb < 4; ++pb)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[pb][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Tv runs on past the stop (it never rises again), so that a Gaussian blends
    // exactly where Tv behind it is at least T_MIN; T stays at the last such value
    float T = 1.0f, Tv = inside ? 1.0f : 0.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
    bool wave_done = ballot64(inside) == 0;
    uint32_t last = 0;
    float* wsw = sw + w * WROWS * WST;

    int b3 = 0, b2 = 0;   // chunk index mod 3 and mod 2
    for (uint32_t cpos = 0; cpos < len; cpos += FK) {
        const int n3 = b3 == 2 ? 0 : b3 + 1, nn3 = n3 == 2 ? 0 : n3 + 1;
        RecT r2;
        uint32_t g2 = 0u, rk3 = 0u;
        if (k < FK) {
            get_rec(rk2, r2, g2);
            rk3 = rank_at(cpos + (uint32_t)(3 * FK + k));
        }
        Item fr[NI];
        if constexpr (NB > 0) load_feats(sg[n3], fr);

        if (!wave_done) {
#pragma unroll 1
            for (int half = 0; half < 2; ++half) {
#pragma unroll 1
                for (int grp = 0; grp < 16; grp += GE) {
                    const RecT* rp = srec[b3] + 16 * half + grp;
                    float al[GE];
#pragma unroll
                    for (int m = 0; m < GE; ++m) al[m] = prim_alpha<SURF>(rp[m], x, y);
                    asm volatile("" ::: "memory");   // (the colours are read again, not held from above)
#pragma unroll
                    for (int m = 0; m < GE; ++m) {
                        const float4 col = rp[m].r2;   // (opacity, r, g, b)
                        float Tn, wv;
                        bool on, blend;
                        if constexpr (NB == 0) {   // (flags cost less than the extra selects: 90 against 97 us)
                            const bool act = Tv >= T_MIN && !(al[m] < ALPHA_MIN);
                            Tn = Tv * (1.0f - al[m]);
                            on = blend = act && !(Tn < T_MIN);
                            wv = al[m] * Tv;
                            Tn = act ? Tn : Tv;
                        } else {
                            const float am = al[m] < ALPHA_MIN ? 0.0f : al[m];
                            Tn = Tv * (1.0f - am);
                            on = Tn >= T_MIN;
                            wv = on ? am * Tv : 0.0f;
                            blend = wv > 0.0f;
                        }
                        if (blend) {
                            c0 = __builtin_fmaf(wv, col.y, c0);
                            c1 = __builtin_fmaf(wv, col.z, c1);
                            c2 = __builtin_fmaf(wv, col.w, c2);
                        }
                        T = on ? Tn : T;
                        Tv = Tn;
                        last = blend ? cpos + (uint32_t)(16 * half + grp + m + 1) : last;
                        if constexpr (NB > 0) wsw[((FB ? 16 * half : 0) + grp + m) * WST + lane] = wv;
                    }
                }
                if constexpr (NB > 0 && !FB) {
                    const float* sf = sft + b2 * FK * FST + 16 * half * FST;
#pragma unroll
                    for (int st = 0; st < 4; ++st) {
                        float aw[4];
#pragma unroll
                        for (int pb = 0; pb < 4; ++pb) aw[pb] = wsw[(4 * st + q) * WST + 16 * pb + xi];
#pragma unroll
                        for (int j = 0; j < NB; ++j) {
                            const float f = sf[(4 * st + q) * FST + 16 * j + xi];
#pragma unroll
                            for (int pb = 0; pb < 4; ++pb)
                                acc[pb][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(aw[pb], f, acc[pb][j], 0, 0, 0);
                        }
                    }
                }
            }
            if constexpr (NB > 0 && FB) {
                bf16x8 aw[3][4];   // W of pixel (row 4 w + pb, column xi), positions 8 q .. 8 q + 7
#pragma unroll
                for (int pb = 0; pb < 4; ++pb) {
                    u32x4 h, m, l;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float* wp = wsw + (8 * q + 2 * e) * WST + 16 * pb + xi;
                        const float x0 = wp[0], x1 = wp[WST];
                        h[e] = pack_bf16(x0, x1);
                        const float r0 = x0 - lo_f32(h[e]), r1 = x1 - hi_f32(h[e]);
                        m[e] = pack_bf16(r0, r1);
                        l[e] = pack_bf16(r0 - lo_f32(m[e]), r1 - hi_f32(m[e]));
                    }
                    aw[0][pb] = __builtin_bit_cast(bf16x8, h);
                    aw[1][pb] = __builtin_bit_cast(bf16x8, m);
                    aw[2][pb] = __builtin_bit_cast(bf16x8, l);
                }
                const unsigned char* fb = reinterpret_cast<const unsigned char*>(sft) +
                                          (b2 * FK + 4 * q + (xi >> 2)) * FROW + 8 * (xi & 3);
                typedef __attribute__((address_space(3))) s16x4 lds4;
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)(fb + 32 * j)));
                    const uint2 hi =
                        __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds4*)(fb + 16 * FROW + 32 * j)));
                    const bf16x8 f = __builtin_bit_cast(bf16x8, u32x4{lo.x, lo.y, hi.x, hi.y});
#pragma unroll
                    for (int c = 2; c >= 0; --c)   // (small terms first)
#pragma unroll
                        for (int pb = 0; pb < 4; ++pb)
                            acc[pb][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw[c][pb], f, acc[pb][j], 0, 0, 0);
                }
            }
            wave_done = ballot64(Tv >= T_MIN) == 0;
        }
        // chunk c+1's features and chunk c+2's records to LDS
        if constexpr (NB > 0) store_feats(fr, b2 ^ 1);
        if (k < FK) {
            put_rec(nn3, cpos + (uint32_t)(2 * FK + k), r2, g2);
            rk2 = rk3;
        }
        // leave when every pixel has stopped (flags double-buffered by chunk parity)
        if (lane == 0) sbusy[b2][w] = wave_done ? 0 : 1;
        __syncthreads();
        if (*reinterpret_cast<const uint32_t*>(sbusy[b2]) == 0u) break;
        b3 = n3;
        b2 ^= 1;
    }

    const int64_t rowp = vt.pix_off[v];
    if (inside && slice == 0) {
        const int64_t p = rowp + (int64_t)py * vt.width[v] + px;
        a.C[3 * p] = c0;
        a.C[3 * p + 1] = c1;
        a.C[3 * p + 2] = c2;
        a.T[p] = T;
        a.n_iter[p] = last;
    }
    // F: lane holds F[pixel 4 q + r of row 4 w + pb][channel 16 j + xi]
    if constexpr (NB > 0) {
#pragma unroll
        for (int pb = 0; pb < 4; ++pb) {
            const int fy = ty * TILE + 4 * w + pb;
            if (fy < vt.height[v]) {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int fx = tx * TILE + 4 * q + r;
                    if (fx < vt.width[v]) {
                        float* fo = a.F + (rowp + (int64_t)fy * vt.width[v] + fx) * a.d + d0 + xi;
#pragma unroll
                        for (int j = 0; j < NB; ++j)
                            if (d0 + 16 * j + xi < a.d) fo[16 * j] = acc[pb][j][r];
                    }
                }
            }
        }
    }
    if constexpr (NB > 0) {
        // features that are not finite, added to the pixels that blend them by a
        // second walk (rare: nothing to do for finite features)
        __syncthreads();
        if (sodd != 0u) {
            __threadfence();   // (this pixel's F was stored by other lanes)
            __syncthreads();
            float Tw = 1.0f;
            for (uint32_t pos = 0; pos < last; ++pos) {
                const uint32_t j = inst_rank(a.keys, a.vals, (int64_t)s + pos, a.rank_bits, a.packed);
                const float alpha = prim_alpha<SURF>(load_rec<SURF>(a.rrec, j), x, y);
                if (alpha < ALPHA_MIN) continue;
                const float wv = alpha * Tw;
                Tw = Tw * (1.0f - alpha);
                const int64_t g = a.order[j];
                float* fo = a.F + (rowp + (int64_t)py * vt.width[v] + px) * a.d;
                for (int c = d0; c < a.d && c < d0 + DS; ++c) {
                    const float f = load_feat(a.feat, a.feat_bf16, g * a.d + c);
                    if (!isfinite(f)) fo[c] += wv * f;
                }
            }
        }
    }
    if (slice == 0) {
        const uint32_t m = wave_max_u32(last);
        if (lane == 0) smax[w] = m;
        __syncthreads();
        if (threadIdx.x == 0) a.tile_niter[t] = max(max(smax[0], smax[1]), max(smax[2], smax[3]));
    }
}

// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_fuse_finalize(const float* sum, const float* comp, const float* wsum,
                                                       const float* wcomp, int64_t n, int d, const void* feat_in,
                                                       void* feat_out, int bf16) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n * d) return;
    const int64_t g = i / d;
    const float W = wsum[g] + wcomp[g];
    float val;
    if (W > 0.0f)
        val = (sum[i] + comp[i]) / W;
    else
        val = feat_in ? load_feat(feat_in, bf16, i) : 0.0f;
    if (bf16) {
        // round to nearest even
        uint32_t u = __float_as_uint(val);
        u += 0x7FFFu + ((u >> 16) & 1u);
        static_cast<uint16_t*>(feat_out)[i] = (uint16_t)(u >> 16);
    } else {
        static_cast<float*>(feat_out)[i] = val;
    }
}

// The same for rows of a multiple of four channels, aligned to four of them:
// L lanes a row (a power of two), four channels a lane, so a row's weight is
// tested once and only rows with weight read their sums.  Bound: HBM; 300k rows
// of 512 BF16 channels 435 -> 106 us (a 64-bit division and one element a thread
// before).
template <bool BF16>
__global__ __launch_bounds__(256) void k_fuse_finalize_rows(const float* __restrict__ sum, const float* __restrict__ comp,
                                                            const float* __restrict__ wsum,
                                                            const float* __restrict__ wcomp, int64_t n, int d, int L,
                                                            const void* __restrict__ feat_in, void* __restrict__ feat_out) {
    const int64_t rows = (int64_t)gridDim.x * (256 / L);
    const int l = (int)threadIdx.x % L;
    for (int64_t g = (int64_t)blockIdx.x * (256 / L) + threadIdx.x / L; g < n; g += rows) {
        const float W = wsum[g] + wcomp[g];
        for (int c = 4 * l; c < d; c += 4 * L) {
            const int64_t i = g * d + c;
            if (!(W > 0.0f)) {
                if constexpr (BF16)
                    *reinterpret_cast<uint2*>(static_cast<uint16_t*>(feat_out) + i) =
                        feat_in ? *reinterpret_cast<const uint2*>(static_cast<const uint16_t*>(feat_in) + i)
                                : make_uint2(0u, 0u);
                else
                    *reinterpret_cast<float4*>(static_cast<float*>(feat_out) + i) =
                        feat_in ? *reinterpret_cast<const float4*>(static_cast<const float*>(feat_in) + i)
                                : make_float4(0.f, 0.f, 0.f, 0.f);
                continue;
            }
            const float4 a = *reinterpret_cast<const float4*>(sum + i), b = *reinterpret_cast<const float4*>(comp + i);
            const float v[4] = {(a.x + b.x) / W, (a.y + b.y) / W, (a.z + b.z) / W, (a.w + b.w) / W};
            if constexpr (BF16) {
                uint32_t u[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    u[k] = __float_as_uint(v[k]);
                    u[k] = (u[k] + 0x7FFFu + ((u[k] >> 16) & 1u)) >> 16;   // round to nearest even
                }
                *reinterpret_cast<uint2*>(static_cast<uint16_t*>(feat_out) + i) =
                    make_uint2((u[0] & 0xFFFFu) | (u[1] << 16), (u[2] & 0xFFFFu) | (u[3] << 16));
            } else {
                *reinterpret_cast<float4*>(static_cast<float*>(feat_out) + i) = make_float4(v[0], v[1], v[2], v[3]);
            }
        }
    }
}

// ---------------------------------------------------------------------------
template <bool FB, bool SURF>
static void launch_fwd_f32(const RenderArgs& a, const ViewTable& vt, int n_tiles, hipStream_t s) {
    // 16-byte (BF16: 8-byte) feature loads where every row is aligned to them
    const int vec = a.d % 4 == 0 && reinterpret_cast<uintptr_t>(a.feat) % (FB ? 8 : 16) == 0;
    const unsigned ns = (unsigned)((a.d + 127) / 128);
    if (a.d <= 16)
        hipLaunchKernelGGL((k_render_fwd_f32<1, FB, SURF>), dim3(n_tiles, 1), dim3(256), 0, s, a, vt, vec);
    else if (a.d <= 32)
        hipLaunchKernelGGL((k_render_fwd_f32<2, FB, SURF>), dim3(n_tiles, 1), dim3(256), 0, s, a, vt, vec);
    else if (a.d <= 64)
        hipLaunchKernelGGL((k_render_fwd_f32<4, FB, SURF>), dim3(n_tiles, 1), dim3(256), 0, s, a, vt, vec);
    else
        hipLaunchKernelGGL((k_render_fwd_f32<8, FB, SURF>), dim3(n_tiles, ns), dim3(256), 0, s, a, vt, vec);
}

template <bool SURF>
static void launch_fwd_f32(const RenderArgs& a, const ViewTable& vt, int n_tiles, hipStream_t s) {
    if (a.d == 0)
        hipLaunchKernelGGL((k_render_fwd_f32<0, false, SURF>), dim3(n_tiles, 1), dim3(256), 0, s, a, vt, 0);
    else if (a.feat_bf16)
        launch_fwd_f32<true, SURF>(a, vt, n_tiles, s);
    else
        launch_fwd_f32<false, SURF>(a, vt, n_tiles, s);
}

void launch_render_fwd_f32(const RenderArgs& a, const ViewTable& vt, int n_tiles, hipStream_t s) {
    if (a.prim == FH_PRIM_SURFEL)
        launch_fwd_f32<true>(a, vt, n_tiles, s);
    else
        launch_fwd_f32<false>(a, vt, n_tiles, s);
}

void launch_fuse_finalize(const float* sum, const float* comp, const float* wsum, const float* wcomp, int64_t n, int d,
                          const void* feat_in, void* feat_out, int bf16, hipStream_t s) {
    const int64_t tot = n * d;
    if (tot <= 0) return;
    const uintptr_t at = reinterpret_cast<uintptr_t>(sum) | reinterpret_cast<uintptr_t>(comp);
    const uintptr_t ft = reinterpret_cast<uintptr_t>(feat_in) | reinterpret_cast<uintptr_t>(feat_out);
    if (d % 4 == 0 && at % 16 == 0 && ft % (bf16 ? 8 : 16) == 0) {
        int L = 1;
        while (L < 64 && 4 * L < d) L *= 2;
        const int64_t nb = (n + 256 / L - 1) / (256 / L);
        const dim3 grid((unsigned)(nb < 16384 ? nb : 16384));
        if (bf16)
            hipLaunchKernelGGL(k_fuse_finalize_rows<true>, grid, dim3(256), 0, s, sum, comp, wsum, wcomp, n, d, L, feat_in,
                               feat_out);
        else
            hipLaunchKernelGGL(k_fuse_finalize_rows<false>, grid, dim3(256), 0, s, sum, comp, wsum, wcomp, n, d, L, feat_in,
                               feat_out);
        return;
    }
    hipLaunchKernelGGL(k_fuse_finalize, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, sum, comp, wsum, wcomp, n, d,
                       feat_in, feat_out, bf16);
}

}  // namespace fh
