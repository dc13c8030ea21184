// Front-to-back compositing (FP32 VALU form) and its adjoint.
//
// Forward (Section 3.1): for every pixel, walk its tile's depth-sorted list;
//   alpha = min(0.99, o G), skip if alpha < 1/255, stop before T drops below
//   1e-4, w = alpha T, C += w rgb, F += w f, T *= (1 - alpha).
// One 256-thread workgroup per (tile, feature slice); records and feature rows
// of 256 instances at a time are staged in LDS and read by every pixel.
//
// Backward (Appendix A.2): per tile, back to front from the tile's longest
// traversal, transmittance recovered by division from T_final,
//   dL/dalpha_k = T_k g_k - (S_k + T_final dT) / (1 - alpha_k),
//   g_k = rgb_k . dC + f_k . dF,  S_k = sum_{i>k} w_i g_i,
// reduced over the tile's pixels into per-instance partials (no atomics);
// optionally the fusion partials sum_p w(p) target(p) in the same sweep.
//
// Both kernels also take the surfel primitive (Section 3.1; SURF = true):
// four-float4 records (see k_project_surfel), the density at the ray-plane
// intersection, and 14 per-instance partials (the nine record entries' terms,
// sum dL/dpower, rgb, sum w) in rows of 16 floats.
#include "kernels.hpp"

namespace fh {


__device__ __forceinline__ uint32_t inst_rank(const uint32_t* keys, const uint32_t* vals, int64_t i, int rank_bits,
                                              int packed) {
    return packed ? (keys[i] & ((1u << rank_bits) - 1u)) : vals[i];
}

__device__ __forceinline__ float load_feat(const void* f, int bf16, int64_t idx) {
    return bf16 ? bf16_to_f32(static_cast<const uint16_t*>(f)[idx]) : static_cast<const float*>(f)[idx];
}

template <int DS, bool SURF>
__global__ __launch_bounds__(256) void k_render_fwd_f32(RenderArgs a, ViewTable vt) {
    using RecT = typename PrimRec<SURF>::T;
    __shared__ RecT srec[256];
    __shared__ float sfeat[256][DS > 0 ? DS : 1];
    __shared__ uint32_t smax[4];
    if (a.counters->inst_overflow) return;
    const int t = blockIdx.x, slice = blockIdx.y, d0 = slice * DS;
    const int v = view_of_tile(vt, t);
    const int lt = t - vt.tile_off[v];
    const int tx = lt % vt.tiles_x[v], ty = lt / vt.tiles_x[v];
    const int px = tx * TILE + (threadIdx.x % TILE), py = ty * TILE + (threadIdx.x / TILE);
    const bool inside = px < vt.width[v] && py < vt.height[v];
    const float x = (float)px + 0.5f, y = (float)py + 0.5f;
    const uint32_t s = a.ranges[2 * t], e = a.ranges[2 * t + 1];
    const int ds_here = (a.d - d0) < DS ? (a.d - d0) : DS;

    float T = 1.0f, c0 = 0.0f, c1 = 0.0f, c2 = 0.0f;
    float F[DS > 0 ? DS : 1];
#pragma unroll
    for (int c = 0; c < (DS > 0 ? DS : 1); ++c) F[c] = 0.0f;
    bool done = !inside;
    uint32_t last = 0;

    for (uint32_t base = s; base < e; base += 256) {
        const uint32_t cnt = (e - base) < 256u ? (e - base) : 256u;
        if (threadIdx.x < cnt) {
            const int64_t i = base + threadIdx.x;
            const uint32_t j = inst_rank(a.keys, a.vals, i, a.rank_bits, a.packed);
            const uint32_t g = a.order[j];
            srec[threadIdx.x] = load_rec<SURF>(a.rrec, j);
            if (DS > 0) {
#pragma unroll
                for (int c = 0; c < DS; ++c)
                    sfeat[threadIdx.x][c] = c < ds_here ? load_feat(a.feat, a.feat_bf16, (int64_t)g * a.d + d0 + c) : 0.0f;
            }
        }
        __syncthreads();
        if (!done) {
            for (uint32_t k = 0; k < cnt; ++k) {
                const RecT r = srec[k];
                const float alpha = prim_alpha<SURF>(r, x, y);
                if (alpha < ALPHA_MIN) continue;
                const float Tn = T * (1.0f - alpha);
                if (Tn < T_MIN) {
                    done = true;
                    break;
                }
                const float w = alpha * T;
                c0 += w * r.r2.y;
                c1 += w * r.r2.z;
                c2 += w * r.r2.w;
#pragma unroll
                for (int c = 0; c < DS; ++c) F[c] += w * sfeat[k][c];
                T = Tn;
                last = base - s + k + 1;
            }
        }
        if (__syncthreads_count(!done) == 0) break;
    }

    const int64_t p = vt.pix_off[v] + (int64_t)py * vt.width[v] + px;
    if (inside) {
        if (slice == 0) {
            a.C[3 * p] = c0;
            a.C[3 * p + 1] = c1;
            a.C[3 * p + 2] = c2;
            a.T[p] = T;
            a.n_iter[p] = last;
        }
        if (DS > 0) {
#pragma unroll
            for (int c = 0; c < DS; ++c)
                if (c < ds_here) a.F[p * a.d + d0 + c] = F[c];
        }
    }
    if (slice == 0) {
        const uint32_t m = wave_max_u32(last);
        if ((threadIdx.x & 63) == 0) smax[threadIdx.x / 64] = m;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t mm = smax[0];
            for (int k = 1; k < 4; ++k) mm = smax[k] > mm ? smax[k] : mm;
            a.tile_niter[t] = mm;
        }
    }
}

// ---------------------------------------------------------------------------
// Per-tile traversal bookkeeping after the forward pass.
__global__ void k_check_visits(const uint32_t* tile_voff, int n_tiles, Counters* c, int64_t cap) {
    if (threadIdx.x == 0) {
        const unsigned long long tot = tile_voff[n_tiles];
        c->n_visited = tot;
        c->visit_overflow = tot > (unsigned long long)cap ? 1u : 0u;
    }
}

// Per depth rank j (view v = j / n): the rank of each (view, Gaussian) and the
// screen records in rank order, so that a tile list entry (a rank) reaches its
// record with one load.
__global__ __launch_bounds__(256) void k_rank_tables(const uint32_t* __restrict__ order, const float4* __restrict__ rec,
                                                     int64_t n, int64_t total, uint32_t* __restrict__ rank_of,
                                                     float4* __restrict__ rrec, int rw) {
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= total) return;
    const int64_t v = j / n;
    const int64_t i = v * n + order[j];
    rank_of[i] = (uint32_t)(j - v * n);
    for (int k = 0; k < rw; ++k) rrec[rw * j + k] = rec[rw * i + k];
}

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

// ---------------------------------------------------------------------------
template <bool SURF>
static void launch_fwd_f32(const RenderArgs& a, const ViewTable& vt, int n_tiles, int slice, hipStream_t s) {
    if (a.d == 0) {
        hipLaunchKernelGGL((k_render_fwd_f32<0, SURF>), dim3(n_tiles, 1), dim3(256), 0, s, a, vt);
        return;
    }
    const unsigned ns = (unsigned)((a.d + slice - 1) / slice);
    switch (slice) {
        case 8: hipLaunchKernelGGL((k_render_fwd_f32<8, SURF>), dim3(n_tiles, ns), dim3(256), 0, s, a, vt); break;
        case 16: hipLaunchKernelGGL((k_render_fwd_f32<16, SURF>), dim3(n_tiles, ns), dim3(256), 0, s, a, vt); break;
        case 32: hipLaunchKernelGGL((k_render_fwd_f32<32, SURF>), dim3(n_tiles, ns), dim3(256), 0, s, a, vt); break;
        default: hipLaunchKernelGGL((k_render_fwd_f32<64, SURF>), dim3(n_tiles, ns), dim3(256), 0, s, a, vt); break;
    }
}

void launch_render_fwd_f32(const RenderArgs& a, const ViewTable& vt, int n_tiles, int slice, hipStream_t s) {
    if (a.prim == FH_PRIM_SURFEL)
        launch_fwd_f32<true>(a, vt, n_tiles, slice, s);
    else
        launch_fwd_f32<false>(a, vt, n_tiles, slice, s);
}

void launch_check_visits(const uint32_t* tile_voff, int n_tiles, Counters* c, int64_t cap, hipStream_t s) {
    hipLaunchKernelGGL(k_check_visits, dim3(1), dim3(64), 0, s, tile_voff, n_tiles, c, cap);
}

void launch_rank_tables(const uint32_t* order, const float4* rec, int64_t n, int64_t total, uint32_t* rank_of,
                        float4* rrec, int rw, hipStream_t s) {
    hipLaunchKernelGGL(k_rank_tables, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, order, rec, n, total,
                       rank_of, rrec, rw);
}

void launch_fuse_finalize(const float* sum, const float* comp, const float* wsum, const float* wcomp, int64_t n, int d,
                          const void* feat_in, void* feat_out, int bf16, hipStream_t s) {
    const int64_t tot = n * d;
    if (tot > 0)
        hipLaunchKernelGGL(k_fuse_finalize, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, sum, comp, wsum,
                           wcomp, n, d, feat_in, feat_out, bf16);
}

}  // namespace fh
