// The training step around the rasterizer (Algorithm 1: photometric loss,
// Adam update, adaptive density control), on the GPU.
//
// Parameters are held raw and activated for rendering: scale = exp(log-scale),
// opacity = sigmoid(logit); means, the raw quaternion and the SH coefficients
// are rendered as stored.  Every kernel here is elementwise over pixels or
// Gaussians (HBM-bound); reductions run in a fixed order (bitwise
// reproducible), and the densification decisions are taken in float32 on
// float32 values, so they are integers that any float32 evaluation in the same
// order reproduces.
#include <cmath>

#include "kernels.hpp"

namespace fh {

constexpr int TB = 256;

// ---------------------------------------------------------------------------
// Adam (Kingma and Ba) on one parameter group, with the activation's chain
// rule folded in: the raw gradient is g * dact/draw, evaluated at the
// activated value used for rendering (act), and the new activated value is
// written back.  kind: 0 identity, 1 exp (log-scales), 2 sigmoid (logits).
struct AdamGroup {
    float* x;
    float* m;
    float* v;
    const float* g;
    float* act;       // kinds 1, 2: activated values (read: rendering value; written: the updated one)
    int64_t count;
    float lr;
    int kind;
};
struct AdamArgs {
    AdamGroup grp[5];
    float b1, b2, eps, bc1, bc2;   // bc1 = 1 / (1 - b1^t), bc2 = 1 / (1 - b2^t)
};

__global__ __launch_bounds__(TB) void k_adam(AdamArgs a) {
    const AdamGroup& G = a.grp[blockIdx.y];
    const int64_t stride = (int64_t)gridDim.x * TB;
    for (int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x; i < G.count; i += stride) {
        float g = G.g[i];
        float act = 0.0f;
        if (G.kind == 1) {
            act = G.act[i];
            g *= act;                       // d exp(l) / dl = exp(l)
        } else if (G.kind == 2) {
            act = G.act[i];
            g *= act * (1.0f - act);        // d sigmoid(z) / dz = o (1 - o)
        }
        const float m = a.b1 * G.m[i] + (1.0f - a.b1) * g;
        const float v = a.b2 * G.v[i] + (1.0f - a.b2) * (g * g);
        const float mh = m * a.bc1, vh = v * a.bc2;
        const float x = G.x[i] - G.lr * mh / (sqrtf(vh) + a.eps);
        G.m[i] = m;
        G.v[i] = v;
        G.x[i] = x;
        if (G.kind == 1)
            G.act[i] = expf(x);
        else if (G.kind == 2)
            G.act[i] = 1.0f / (1.0f + expf(-x));
    }
}

// Activations of raw values: scales = exp(log-scales), opacity = sigmoid(logit).
__global__ __launch_bounds__(TB) void k_activate(int64_t n, const float* __restrict__ log_scales,
                                                 const float* __restrict__ logit, float* __restrict__ scales,
                                                 float* __restrict__ opacity) {
    const int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x;
    if (i < 3 * n) scales[i] = expf(log_scales[i]);
    if (i < n) opacity[i] = 1.0f / (1.0f + expf(-logit[i]));
}

// ---------------------------------------------------------------------------
// Densification statistics: per Gaussian, over the views that binned it (at
// least one tile instance), the norm of the screen-space mean gradient
// |dL/d(u, v)| is added (in view order) and the views counted.
__global__ __launch_bounds__(TB) void k_densify_stats(const float* __restrict__ grad2d, const int4* __restrict__ rect,
                                                      const Counters* c, int64_t n, int n_views,
                                                      float* __restrict__ gsum, int32_t* __restrict__ cnt) {
    const int64_t g = (int64_t)blockIdx.x * TB + threadIdx.x;
    if (g >= n) return;
    // after an instance or visit overflow the screen-space adjoints are stale
    if (c->inst_overflow || c->visit_overflow) return;
    float s = gsum[g];
    int k = cnt[g];
    for (int v = 0; v < n_views; ++v) {
        const int64_t j = (int64_t)v * n + g;
        const int4 r = rect[j];
        if (r.x > r.z || r.y > r.w) continue;
        const float du = grad2d[j * 12], dv = grad2d[j * 12 + 1];
        s += sqrtf(du * du + dv * dv);
        ++k;
    }
    gsum[g] = s;
    cnt[g] = k;
}

// ---------------------------------------------------------------------------
// Densification decisions: 0 keep, 1 clone (small and hot), 2 split (large and
// hot); a Gaussian below the opacity threshold is pruned together with its
// copies (they share its logit).  keep[g] = 1 if it survives (its first copy
// stays at its place in index order), extra[g] = 1 if it also appends one.
struct DensifyCfg {
    float grad_thr, log_scale_thr, prune_logit;
};

__global__ __launch_bounds__(TB) void k_densify_classify(int64_t n, const float* __restrict__ gsum,
                                                         const int32_t* __restrict__ cnt,
                                                         const float* __restrict__ log_scales,
                                                         const float* __restrict__ logit, DensifyCfg cfg,
                                                         uint32_t* __restrict__ action, uint32_t* __restrict__ keep,
                                                         uint32_t* __restrict__ extra) {
    const int64_t g = (int64_t)blockIdx.x * TB + threadIdx.x;
    if (g >= n) return;
    const int32_t k = cnt[g];
    const float avg = k > 0 ? gsum[g] / (float)k : 0.0f;
    const float lmax = fmaxf(fmaxf(log_scales[3 * g], log_scales[3 * g + 1]), log_scales[3 * g + 2]);
    const bool hot = avg >= cfg.grad_thr;
    const uint32_t act = hot ? (lmax <= cfg.log_scale_thr ? 1u : 2u) : 0u;
    const bool kept = logit[g] >= cfg.prune_logit;
    action[g] = act;
    keep[g] = kept ? 1u : 0u;
    extra[g] = (kept && act != 0u) ? 1u : 0u;
}

// counts[0] = kept + appended (the two scans' totals), counts[1] = kept
__global__ void k_densify_total(const uint32_t* keep_off, const uint32_t* extra_off, int64_t n, int64_t* counts) {
    if (threadIdx.x == 0) {
        counts[0] = (int64_t)keep_off[n] + (int64_t)extra_off[n];
        counts[1] = (int64_t)keep_off[n];
    }
}

// Rotation matrix of the normalised quaternion (w, x, y, z), row-major.
__device__ __forceinline__ void quat_rot(const float* q, float R[9]) {
    const float nn = rsqrtf(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    const float w = q[0] * nn, x = q[1] * nn, y = q[2] * nn, z = q[3] * nn;
    R[0] = 1.0f - 2.0f * (y * y + z * z);
    R[1] = 2.0f * (x * y - w * z);
    R[2] = 2.0f * (x * z + w * y);
    R[3] = 2.0f * (x * y + w * z);
    R[4] = 1.0f - 2.0f * (x * x + z * z);
    R[5] = 2.0f * (y * z - w * x);
    R[6] = 2.0f * (x * z - w * y);
    R[7] = 2.0f * (y * z + w * x);
    R[8] = 1.0f - 2.0f * (x * x + y * y);
}

// Where every parent's rows go: the kept original (or first child) at
// keep_off[g], the clone or second child at n_keep + extra_off[g].
struct DensifyMap {
    int64_t n, n_keep;
    const uint32_t *action, *keep_off, *extra_off, *keep;
};
struct DensifyApplyArgs {
    DensifyMap map;
    const float *means, *log_scales, *quats, *logit;
    const float* z;             // [n, 2, 3] standard normal draws (used by split Gaussians)
    float *means_out, *log_scales_out, *logit_out, *scales_out, *opacity_out;
};

// One thread per parent, the values densification computes: split children's
// means mu + R(q) diag(s) z_j and log-scales log s - ln 1.6, and the activated
// scales and opacity of every copy.  (Rows that are only copied, quaternions,
// SH, moments and features, go through k_densify_rows.)
__device__ __forceinline__ void densify_apply(const DensifyApplyArgs& a) {
    const int64_t g = (int64_t)blockIdx.x * TB + threadIdx.x;
    if (g >= a.map.n || !a.map.keep[g]) return;
    const uint32_t act = a.map.action[g];
    const int64_t dst[2] = {(int64_t)a.map.keep_off[g], a.map.n_keep + (int64_t)a.map.extra_off[g]};
    const int ncopy = act != 0u ? 2 : 1;
    const float mu[3] = {a.means[3 * g], a.means[3 * g + 1], a.means[3 * g + 2]};
    float ls[3] = {a.log_scales[3 * g], a.log_scales[3 * g + 1], a.log_scales[3 * g + 2]};
    float mean[2][3];
    for (int j = 0; j < 2; ++j)
        for (int r = 0; r < 3; ++r) mean[j][r] = mu[r];
    if (act == 2u) {
        float R[9];
        const float q[4] = {a.quats[4 * g], a.quats[4 * g + 1], a.quats[4 * g + 2], a.quats[4 * g + 3]};
        quat_rot(q, R);
        const float s[3] = {expf(ls[0]), expf(ls[1]), expf(ls[2])};
        for (int j = 0; j < 2; ++j) {
            const float* zj = a.z + 6 * g + 3 * j;
            const float t[3] = {s[0] * zj[0], s[1] * zj[1], s[2] * zj[2]};
            for (int r = 0; r < 3; ++r)
                mean[j][r] = mu[r] + (R[3 * r] * t[0] + R[3 * r + 1] * t[1] + R[3 * r + 2] * t[2]);
        }
        const float ln16 = 0.47000362924573558f;   // ln 1.6
        for (int r = 0; r < 3; ++r) ls[r] = ls[r] - ln16;
    }
    const float logit = a.logit[g], op = 1.0f / (1.0f + expf(-logit));
    const float sc[3] = {expf(ls[0]), expf(ls[1]), expf(ls[2])};
    for (int c = 0; c < ncopy; ++c) {
        const int64_t o = dst[c];
        for (int r = 0; r < 3; ++r) {
            a.means_out[3 * o + r] = mean[c][r];
            a.log_scales_out[3 * o + r] = ls[r];
            a.scales_out[3 * o + r] = sc[r];
        }
        a.logit_out[o] = logit;
        a.opacity_out[o] = op;
    }
}

// Rows of per-Gaussian arrays carried to the densified set.  A job is one
// array: rows of `units` elements (16, 4 or 1 bytes each, as its row size and
// addresses allow); zero_new: an Adam moment, kept by an original that was not
// split and zero for every other copy.  A workgroup takes 32 parents and its
// threads run over (parent, element), so that neighbouring threads move
// neighbouring elements of a row (370 us for 1.3 GB at 500k Gaussians with 512-byte
// features, 3.5 TB/s; one thread per parent, which stepped through
// its rows alone, took 1.98 ms; bound: HBM).
struct RowJob {
    const uint8_t* in;
    uint8_t* out;
    int64_t units;
    int unit_bytes;
    int zero_new;
};
constexpr int MAX_ROW_JOBS = 12;
struct RowJobs {
    RowJob job[MAX_ROW_JOBS];
    DensifyMap map;
};
constexpr int ROW_PARENTS = 32;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <typename T>
__device__ __forceinline__ void densify_rows(const RowJob& J, const uint32_t* d0, const uint32_t* d1, const uint8_t* how,
                                             int64_t g0, int parents, int64_t n_keep) {
    const T* in = reinterpret_cast<const T*>(J.in) + g0 * J.units;
    T* out = reinterpret_cast<T*>(J.out);
    const T zero = {};
    if (J.units >= 4 * TB) {
        // long rows: one at a time, the workgroup over its elements
        for (int k = 0; k < parents; ++k) {
            const uint8_t h = how[k];
            if (!(h & 1)) continue;
            for (int64_t i = threadIdx.x; i < J.units; i += TB) {
                const T val = in[k * J.units + i];
                out[(int64_t)d0[k] * J.units + i] = (J.zero_new && (h & 4)) ? zero : val;
                if (h & 2) out[(n_keep + (int64_t)d1[k]) * J.units + i] = J.zero_new ? zero : val;
            }
        }
        return;
    }
    const uint32_t U = (uint32_t)J.units, total = (uint32_t)parents * U;
    // four elements a thread requested before any is stored
    for (uint32_t i0 = threadIdx.x; i0 < total; i0 += 4 * TB) {
        T val[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t idx = i0 + e * TB;
            val[e] = idx < total ? in[idx] : zero;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const uint32_t idx = i0 + e * TB;
            if (idx >= total) break;
            const uint32_t k = idx / U, i = idx - k * U;
            const uint8_t h = how[k];
            if (!(h & 1)) continue;                   // pruned
            out[(int64_t)d0[k] * U + i] = (J.zero_new && (h & 4)) ? zero : val[e];
            if (h & 2) out[(n_keep + (int64_t)d1[k]) * U + i] = J.zero_new ? zero : val[e];
        }
    }
}

// APPLY: the last row of workgroups computes the children's values (b), in the
// same launch (a launch of its own cost small scenes 5 us).
template <bool APPLY>
__global__ __launch_bounds__(TB) void k_densify_rows(RowJobs a, DensifyApplyArgs b) {
    if (APPLY && blockIdx.y == gridDim.y - 1) {
        densify_apply(b);
        return;
    }
    __shared__ uint32_t d0[ROW_PARENTS], d1[ROW_PARENTS];
    __shared__ uint8_t how[ROW_PARENTS];              // bit 0 kept, 1 copied, 2 split
    const int64_t g0 = (int64_t)blockIdx.x * ROW_PARENTS;
    const int parents = (int)(a.map.n - g0 < ROW_PARENTS ? a.map.n - g0 : ROW_PARENTS);
    if ((int)threadIdx.x < parents) {
        const int64_t g = g0 + threadIdx.x;
        const uint32_t act = a.map.action[g];
        d0[threadIdx.x] = a.map.keep_off[g];
        d1[threadIdx.x] = a.map.extra_off[g];
        how[threadIdx.x] = a.map.keep[g] ? (uint8_t)(1u | (act != 0u ? 2u : 0u) | (act == 2u ? 4u : 0u)) : 0;
    }
    __syncthreads();
    // (selected with constant indices, field by field: the argument stays out of scratch memory)
    const uint8_t* in = a.job[0].in;
    uint8_t* out = a.job[0].out;
    int64_t units = a.job[0].units;
    int unit_bytes = a.job[0].unit_bytes, zero_new = a.job[0].zero_new;
#pragma unroll
    for (int k = 1; k < MAX_ROW_JOBS; ++k) {
        const bool me = (int)blockIdx.y == k;
        in = me ? a.job[k].in : in;
        out = me ? a.job[k].out : out;
        units = me ? a.job[k].units : units;
        unit_bytes = me ? a.job[k].unit_bytes : unit_bytes;
        zero_new = me ? a.job[k].zero_new : zero_new;
    }
    const RowJob J{in, out, units, unit_bytes, zero_new};
    if (J.unit_bytes == 16)
        densify_rows<u32x4>(J, d0, d1, how, g0, parents, a.map.n_keep);
    else if (J.unit_bytes == 4)
        densify_rows<uint32_t>(J, d0, d1, how, g0, parents, a.map.n_keep);
    else
        densify_rows<uint8_t>(J, d0, d1, how, g0, parents, a.map.n_keep);
}

// ---------------------------------------------------------------------------
// Photometric loss (mean squared error over pixels and channels) and its
// gradient dC = 2 (C - C_target) / (3 P).  Block b sums elements
// [b * LOSS_CHUNK, (b + 1) * LOSS_CHUNK) by a fixed tree; one block then adds
// the partials in block order.
constexpr int LOSS_CHUNK = 8192;
constexpr int LOSS_TB = 1024;   // eight elements a thread

__device__ __forceinline__ float block_sum_256(float v, float* sh) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) sh[w] = v;
    __syncthreads();
    float t = 0.0f;
    if (threadIdx.x == 0) t = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    __syncthreads();
    return t;
}

// One pass, 1024 threads a chunk with two 16-byte loads of each map in flight
// (256 threads stepping through 32 scalar elements: 26 us at 1297x841 and
// 18 at 987x657, latency-bound at one block a CU).  vec: every map 16-byte
// aligned; else, and at the end of the maps, element by element.
__global__ __launch_bounds__(LOSS_TB) void k_loss_partial(const float* __restrict__ C, const float* __restrict__ Ct,
                                                          int64_t count, float scale, float* __restrict__ dC,
                                                          float* __restrict__ part, int vec) {
    __shared__ float sh[LOSS_TB / 64];
    const int64_t b0 = (int64_t)blockIdx.x * LOSS_CHUNK;
    const float s2 = 2.0f * scale;
    float acc = 0.0f;
    if (vec && b0 + LOSS_CHUNK <= count) {
        float4 c[2], t[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int64_t i = b0 / 4 + threadIdx.x + LOSS_TB * k;
            c[k] = reinterpret_cast<const float4*>(C)[i];
            t[k] = reinterpret_cast<const float4*>(Ct)[i];
        }
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const float4 e = make_float4(c[k].x - t[k].x, c[k].y - t[k].y, c[k].z - t[k].z, c[k].w - t[k].w);
            acc += (e.x * e.x + e.y * e.y) + (e.z * e.z + e.w * e.w);
            reinterpret_cast<float4*>(dC)[b0 / 4 + threadIdx.x + LOSS_TB * k] =
                make_float4(s2 * e.x, s2 * e.y, s2 * e.z, s2 * e.w);
        }
    } else {
        for (int64_t i = b0 + threadIdx.x; i < count && i < b0 + LOSS_CHUNK; i += LOSS_TB) {
            const float e = C[i] - Ct[i];
            acc += e * e;
            dC[i] = s2 * e;
        }
    }
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        float t = 0.0f;
        for (int k = 0; k < LOSS_TB / 64; ++k) t += sh[k];
        part[blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(TB) void k_loss_final(const float* __restrict__ part, int nb, float scale,
                                                   float* __restrict__ loss) {
    __shared__ float sh[4];
    float acc = 0.0f;
    for (int i = threadIdx.x; i < nb; i += TB) acc += part[i];
    const float t = block_sum_256(acc, sh);
    if (threadIdx.x == 0) loss[0] = t * scale;
}

// ---------------------------------------------------------------------------
static unsigned grid_for(int64_t n) {
    const int64_t b = (n + TB - 1) / TB;
    return (unsigned)(b < 1 ? 1 : b);
}

void launch_adam(const AdamArgs& a, int64_t max_count, hipStream_t s) {
    int64_t b = (max_count + TB - 1) / TB;
    if (b > 8192) b = 8192;
    if (b < 1) b = 1;
    hipLaunchKernelGGL(k_adam, dim3((unsigned)b, 5), dim3(TB), 0, s, a);
}

void launch_densify_stats(const float* grad2d, const int4* rect, const Counters* c, int64_t n, int n_views,
                          float* gsum, int32_t* cnt, hipStream_t s) {
    if (n == 0) return;
    hipLaunchKernelGGL(k_densify_stats, dim3(grid_for(n)), dim3(TB), 0, s, grad2d, rect, c, n, n_views, gsum, cnt);
}

}  // namespace fh

using namespace fh;

namespace {
// densify workspace: action, keep, extra [n]; keep_off, extra_off [n + 1]; scan scratch
struct DensifyWs {
    uint32_t *action, *keep, *extra, *keep_off, *extra_off, *scratch;
};
size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }
size_t densify_ws_layout(int64_t n, char* base, DensifyWs* w) {
    const size_t u = sizeof(uint32_t);
    const size_t sizes[6] = {n * u, n * u, n * u, (n + 1) * u, (n + 1) * u, scan_scratch_u32(n + 1) * u};
    size_t off = 0;
    uint32_t* at[6];
    for (int i = 0; i < 6; ++i) {
        at[i] = base ? reinterpret_cast<uint32_t*>(base + off) : nullptr;
        off += al256(sizes[i]);
    }
    if (w) *w = DensifyWs{at[0], at[1], at[2], at[3], at[4], at[5]};
    return off;
}
bool params_ok(const fh_params* p) {
    return p && p->means && p->log_scales && p->quats && p->logit_opacity && p->sh;
}
RowJob row_job(const void* in, void* out, int64_t row_bytes, int zero_new) {
    const uintptr_t at = reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out) | (uintptr_t)row_bytes;
    const int ub = at % 16 == 0 ? 16 : (at % 4 == 0 ? 4 : 1);
    return RowJob{static_cast<const uint8_t*>(in), static_cast<uint8_t*>(out), row_bytes / ub, ub, zero_new};
}
template <bool APPLY>
void launch_rows(const RowJobs& r, int jobs, const DensifyApplyArgs& b, hipStream_t s) {
    const unsigned nb = (unsigned)((r.map.n + ROW_PARENTS - 1) / ROW_PARENTS);
    if (nb > 0) hipLaunchKernelGGL(k_densify_rows<APPLY>, dim3(nb, jobs + (APPLY ? 1 : 0)), dim3(TB), 0, s, r, b);
}
fh_status status_of_launch() { return hipGetLastError() == hipSuccess ? FH_OK : FH_E_HIP; }
}  // namespace

extern "C" {

fh_status fh_adam_step(int64_t n, int32_t sh_degree, const fh_params* param, const fh_params* m, const fh_params* v,
                       const fh_grads* grads, const fh_adam* cfg, float* scales, float* opacity, hipStream_t s) {
    if (n < 0 || sh_degree < 0 || sh_degree > 3) return FH_E_INVALID;
    if (!params_ok(param) || !params_ok(m) || !params_ok(v) || !grads || !cfg || !scales || !opacity)
        return FH_E_INVALID;
    if (!grads->means || !grads->scales || !grads->quats || !grads->opacity || !grads->sh) return FH_E_INVALID;
    if (cfg->step < 1 || !(cfg->beta1 >= 0.0f && cfg->beta1 < 1.0f) || !(cfg->beta2 >= 0.0f && cfg->beta2 < 1.0f) ||
        !(cfg->eps >= 0.0f))
        return FH_E_INVALID;
    if (n == 0) return FH_OK;
    const int64_t nsh = 3 * (int64_t)(sh_degree + 1) * (sh_degree + 1);
    AdamArgs a;
    a.b1 = cfg->beta1;
    a.b2 = cfg->beta2;
    a.eps = cfg->eps;
    a.bc1 = (float)(1.0 / (1.0 - std::pow((double)cfg->beta1, (double)cfg->step)));
    a.bc2 = (float)(1.0 / (1.0 - std::pow((double)cfg->beta2, (double)cfg->step)));
    a.grp[0] = AdamGroup{param->means, m->means, v->means, grads->means, nullptr, 3 * n, cfg->lr[0], 0};
    a.grp[1] = AdamGroup{param->log_scales, m->log_scales, v->log_scales, grads->scales, scales, 3 * n, cfg->lr[1], 1};
    a.grp[2] = AdamGroup{param->quats, m->quats, v->quats, grads->quats, nullptr, 4 * n, cfg->lr[2], 0};
    a.grp[3] = AdamGroup{param->logit_opacity, m->logit_opacity, v->logit_opacity, grads->opacity, opacity, n,
                         cfg->lr[3], 2};
    a.grp[4] = AdamGroup{param->sh, m->sh, v->sh, grads->sh, nullptr, nsh * n, cfg->lr[4], 0};
    launch_adam(a, nsh * n > 4 * n ? nsh * n : 4 * n, s);
    return status_of_launch();
}

fh_status fh_activate(int64_t n, const float* log_scales, const float* logit_opacity, float* scales, float* opacity,
                      hipStream_t s) {
    if (n < 0) return FH_E_INVALID;
    if (n == 0) return FH_OK;
    if (!log_scales || !logit_opacity || !scales || !opacity) return FH_E_INVALID;
    hipLaunchKernelGGL(k_activate, dim3(grid_for(3 * n)), dim3(TB), 0, s, n, log_scales, logit_opacity, scales,
                       opacity);
    return status_of_launch();
}

fh_status fh_densify_stats(const fh_plan* p, const void* ws, float* grad_sum, int32_t* count, hipStream_t s) {
    if (!p || !ws || !grad_sum || !count) return FH_E_INVALID;
    const char* b = static_cast<const char*>(ws);
    launch_densify_stats(reinterpret_cast<const float*>(b + p->off[WS_GRAD2D]),
                         reinterpret_cast<const int4*>(b + p->off[WS_RECT]),
                         reinterpret_cast<const Counters*>(b + p->off[WS_COUNTERS]), p->n, p->n_views, grad_sum, count,
                         s);
    return status_of_launch();
}

size_t fh_densify_workspace_size(int64_t n) { return n < 0 ? 0 : densify_ws_layout(n, nullptr, nullptr); }

fh_status fh_densify_plan(int64_t n, const float* grad_sum, const int32_t* count, const float* log_scales,
                          const float* logit_opacity, const fh_densify_config* cfg, void* dws, int64_t* counts,
                          hipStream_t s) {
    if (n < 0 || !cfg || !dws || !counts) return FH_E_INVALID;
    if (n > 0 && (!grad_sum || !count || !log_scales || !logit_opacity)) return FH_E_INVALID;
    DensifyWs w;
    densify_ws_layout(n, static_cast<char*>(dws), &w);
    if (n > 0) {
        const DensifyCfg c{cfg->grad_threshold, cfg->log_scale_threshold, cfg->prune_logit};
        hipLaunchKernelGGL(k_densify_classify, dim3(grid_for(n)), dim3(TB), 0, s, n, grad_sum, count, log_scales,
                           logit_opacity, c, w.action, w.keep, w.extra);
        device_exclusive_scan(w.keep, w.keep_off, n, w.scratch, 1, s);
        device_exclusive_scan(w.extra, w.extra_off, n, w.scratch, 1, s);
    } else {
        launch_fill_u32(w.keep_off, 1, 0u, s);
        launch_fill_u32(w.extra_off, 1, 0u, s);
    }
    hipLaunchKernelGGL(k_densify_total, dim3(1), dim3(64), 0, s, w.keep_off, w.extra_off, n, counts);
    return status_of_launch();
}

fh_status fh_densify_apply(int64_t n, int32_t sh_degree, const void* dws, const fh_params* in, const fh_params* m_in,
                           const fh_params* v_in, const float* z, int64_t n_out, int64_t n_keep, const fh_params* out,
                           const fh_params* m_out, const fh_params* v_out, float* scales_out, float* opacity_out,
                           hipStream_t s) {
    if (n < 0 || n_keep < 0 || n_keep > n || n_out < n_keep || n_out > n_keep + n || sh_degree < 0 ||
        sh_degree > 3 || !dws)
        return FH_E_INVALID;
    if (n_out == 0) return FH_OK;   // every Gaussian pruned: nothing to write
    if (!params_ok(in) || !params_ok(m_in) || !params_ok(v_in) || !z || !params_ok(out) || !params_ok(m_out) ||
        !params_ok(v_out) || !scales_out || !opacity_out)
        return FH_E_INVALID;
    DensifyWs w;
    densify_ws_layout(n, static_cast<char*>(const_cast<void*>(dws)), &w);
    const DensifyMap map{n, n_keep, w.action, w.keep_off, w.extra_off, w.keep};
    DensifyApplyArgs a;
    a.map = map;
    a.means = in->means;
    a.log_scales = in->log_scales;
    a.quats = in->quats;
    a.logit = in->logit_opacity;
    a.z = z;
    a.means_out = out->means;
    a.log_scales_out = out->log_scales;
    a.logit_out = out->logit_opacity;
    a.scales_out = scales_out;
    a.opacity_out = opacity_out;
    const int64_t nsh = 4 * 3 * (int64_t)(sh_degree + 1) * (sh_degree + 1);
    RowJobs r;
    r.map = map;
    int k = 0;
    r.job[k++] = row_job(in->quats, out->quats, 16, 0);
    r.job[k++] = row_job(in->sh, out->sh, nsh, 0);
    const fh_params* mi[2] = {m_in, v_in};
    const fh_params* mo[2] = {m_out, v_out};
    for (int c = 0; c < 2; ++c) {
        r.job[k++] = row_job(mi[c]->means, mo[c]->means, 12, 1);
        r.job[k++] = row_job(mi[c]->log_scales, mo[c]->log_scales, 12, 1);
        r.job[k++] = row_job(mi[c]->quats, mo[c]->quats, 16, 1);
        r.job[k++] = row_job(mi[c]->logit_opacity, mo[c]->logit_opacity, 4, 1);
        r.job[k++] = row_job(mi[c]->sh, mo[c]->sh, nsh, 1);
    }
    launch_rows<true>(r, k, a, s);
    return status_of_launch();
}

fh_status fh_densify_copy_rows(int64_t n, const void* dws, const void* in, void* out, int64_t row_bytes,
                               int64_t n_out, int64_t n_keep, hipStream_t s) {
    if (n < 0 || row_bytes < 0 || n_keep < 0 || n_keep > n || n_out < n_keep || n_out > n_keep + n || !dws)
        return FH_E_INVALID;
    if (n_out == 0 || row_bytes == 0) return FH_OK;
    if (!in || !out) return FH_E_INVALID;
    DensifyWs w;
    densify_ws_layout(n, static_cast<char*>(const_cast<void*>(dws)), &w);
    RowJobs r;
    r.map = DensifyMap{n, n_keep, w.action, w.keep_off, w.extra_off, w.keep};
    r.job[0] = row_job(in, out, row_bytes, 0);
    launch_rows<false>(r, 1, DensifyApplyArgs{}, s);
    return status_of_launch();
}

size_t fh_loss_workspace_size(int64_t n_pixels) {
    if (n_pixels < 0) return 0;
    const int64_t nb = (3 * n_pixels + LOSS_CHUNK - 1) / LOSS_CHUNK;
    return al256((size_t)(nb < 1 ? 1 : nb) * sizeof(float));
}

fh_status fh_photometric_loss(int64_t n_pixels, const float* C, const float* C_target, float* dC, float* loss,
                              void* lws, hipStream_t s) {
    if (n_pixels < 1 || !C || !C_target || !dC || !loss || !lws) return FH_E_INVALID;
    const int64_t count = 3 * n_pixels;
    const int64_t nb = (count + LOSS_CHUNK - 1) / LOSS_CHUNK;
    if (nb > 0x7fffffff) return FH_E_UNSUPPORTED;
    const float scale = (float)(1.0 / (double)count);
    float* part = static_cast<float*>(lws);
    const int vec = (reinterpret_cast<uintptr_t>(C) | reinterpret_cast<uintptr_t>(C_target) |
                     reinterpret_cast<uintptr_t>(dC)) % 16 == 0;
    hipLaunchKernelGGL(k_loss_partial, dim3((unsigned)nb), dim3(LOSS_TB), 0, s, C, C_target, count, scale, dC, part, vec);
    hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(TB), 0, s, (const float*)part, (int)nb, scale, loss);
    return status_of_launch();
}

}  // extern "C"
