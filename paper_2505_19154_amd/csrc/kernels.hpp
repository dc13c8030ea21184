// Kernel argument structs and launchers shared by the HIP translation units.
#pragma once

#include "common.hpp"

namespace fh {
// project.hip
struct ProjectArgs {
    const float *means, *scales, *quats, *opacity, *sh;
    int n, sh_degree;
    int bin_rule;       // fh_bin_rule
    int prim;           // fh_primitive (surfel records: 4 float4)
    float4* rec;
    uint32_t* depth_key;
    int4* rect;
    Counters* counters;
};
struct ProjectBwdArgs {
    const float *means, *scales, *quats, *opacity, *sh;
    int n, sh_degree;
    const float* grad2d;
    const uint32_t* visited;    // [n] bit v: view v visited an instance of the Gaussian (after no overflow)
    const Counters* counters;   // an instance or visit overflow leaves the (zero-filled) outputs zero
    float *g_means, *g_scales, *g_quats, *g_opacity, *g_sh;
    int prim;                   // fh_primitive (surfel adjoint rows: 16 floats)
};
void launch_project(const ProjectArgs&, const CamTable&, const ViewTable&, int, hipStream_t);
void launch_project_bwd(const ProjectBwdArgs&, const CamTable&, hipStream_t);
// sort.hip
size_t scan_scratch_u32(int64_t n);
void device_exclusive_scan(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* scratch, int write_total,
                           hipStream_t s);
int radix_sort(const uint32_t* keys_src, const uint32_t* vals_src, uint32_t* ka, uint32_t* va, uint32_t* kb,
               uint32_t* vb, bool with_vals, int64_t segs, int64_t seg_len, const unsigned long long* dev_len,
               int64_t cap, int lo, int hi, uint32_t* hist, Counters* reset, hipStream_t s);
size_t radix_hist_u32(int64_t segs, int64_t span);
// rank tables, tiles per rank and their scan (sums and starts are set by the launch)
struct RankArgs {
    const uint32_t* order;
    const int4* rect;
    const float4* rec;
    int64_t n, total, cap;
    uint32_t *ntiles, *inst_off, *rank_of;
    float4* rrec;
    int rw;
    Counters* counters;
    uint32_t* ranges;          // nullable: cleared
    int64_t n_ranges;
    uint32_t *sums, *starts;
    uint32_t n_starts;
};
void launch_ranks(const RankArgs& a, uint32_t* hist, uint32_t* scan_tmp, hipStream_t s);
// first rank of k_duplicate's workgroups, as launch_ranks left them in hist
inline const uint32_t* dup_starts(const uint32_t* hist, int64_t total) { return hist + (total + 1023) / 1024; }
// voff = exclusive scan of the tiles' traversal lengths; the visit count and its overflow flag
void launch_scan_visits(const uint32_t* niter, uint32_t* voff, int64_t n_tiles, uint32_t* scratch, Counters* c, int64_t cap,
                        hipStream_t s);
struct DupArgs {
    const uint32_t* inst_off;
    const uint32_t* starts;
    const uint32_t* order;
    const int4* rect;
    int64_t n, total_ranks;
    int64_t cap;
    const Counters* counters;
    uint32_t* keys;
    uint32_t* vals;
    int rank_bits;
    int packed;
    ViewTable vt;
};
void launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t s);
// tile schedule keys: 0xFFFF - min(cost, 0xFFFF), cost = the list length
// (ranges) or the traversal length (tile_niter)
void launch_tile_cost_keys(const uint32_t* ranges, const uint32_t* tile_niter, int64_t n_tiles, uint32_t* keys,
                           hipStream_t s);
void launch_duplicate(const DupArgs& a, hipStream_t s);
void launch_ranges(const uint32_t* keys, const Counters* c, int64_t cap, int rank_bits, int packed, uint32_t* ranges,
                   hipStream_t s);
void launch_bin_keys(const uint32_t* keys, const uint32_t* vals, const uint32_t* order, const uint32_t* depth_key,
                     int64_t n_inst, int64_t n, int rank_bits, int packed, uint64_t* ko, uint32_t* go, hipStream_t s);
// render_f32.hip
struct RenderArgs {
    const float4* rec;
    const float4* rrec;       // [V*N*3] records in depth-rank order
    const uint32_t* order;
    const uint32_t* keys;
    const uint32_t* vals;
    const uint32_t* ranges;
    const Counters* counters;
    int rank_bits, packed;
    int64_t n;
    const void* feat;
    int d, feat_bf16;
    float* C;
    float* F;
    float* T;
    uint32_t* n_iter;
    uint32_t* tile_niter;
    const uint32_t* tile_order;   // nullable: work item i takes tile tile_order[i]
    int prim;                     // fh_primitive
};
struct BwdArgs {
    const float4* rec;
    const uint32_t* order;
    const uint32_t* keys;
    const uint32_t* vals;
    const uint32_t* ranges;
    const uint32_t* tile_niter;
    const uint32_t* tile_voff;
    const Counters* counters;
    int rank_bits, packed;
    int64_t n;
    const void* feat;
    int d, feat_bf16;
    const float* T_final;
    const uint32_t* n_iter;
    const float* dC;
    const float* dF;
    const float* dT;
    const void* target;
    int target_bf16;
    const float4* vrec;        // [visits * 3] staged records, in visit order
    const uint32_t* vgid;      // [visits] staged Gaussians
    float* part_geom;
    float* part_fuse;
    const uint32_t* tile_order;   // nullable: work item i takes tile tile_order[i]
    // widths of 256 channels and up: [visits][256] f . dF of every visited
    // (position, pixel), written by the contraction kernel a slice at a time
    // (from channel d0) and read by the walk
    float* g;
    int d0;
    // nullable: T of every pixel at the segment ends of its tile's list, counted
    // from the list's end ([voff / T_SEG + tile + segment - 1][256]), left by the walk
    // of the gradients for the fusion of the same call
    float* tseg;
    int prim;                     // fh_primitive
};
constexpr int T_SEG = 128;        // positions a segment
struct VisitStageArgs {
    const uint32_t* ranges;
    const uint32_t* tile_niter;
    const uint32_t* tile_voff;
    const uint32_t* keys;
    const uint32_t* vals;
    int rank_bits, packed;
    const uint32_t* order;
    const float4* rrec;
    Counters* counters;
    uint32_t* vkey;     // [visits] rank of the visited instance
    uint32_t* vgid;     // [visits] its Gaussian
    float4* vrec;       // [visits * rw] its screen record
    int rw;             // float4 per record: 3 (Gaussians) or 4 (surfels)
    uint32_t* vseg;            // nullable: cleared (n_vseg words)
    int64_t n_vseg;
    uint32_t* visited;         // nullable: cleared (n words)
    int64_t n;
    float4* grad2d;            // nullable: cleared after no overflow (n_grad2d float4)
    int64_t n_grad2d;
    int n_tiles;
};
struct ReduceArgs {
    const uint32_t* order;
    const uint32_t* vseg;      // [V*N][2] per-rank [start, end) into vsorted
    const uint32_t* vsorted;   // visit indices sorted by rank (stable: row-major tiles)
    Counters* counters;
    uint32_t* long_list;       // [total] ranks (geometry), [n] long Gaussians (fusion), [n] their first unit,
                               // [n] short Gaussians (fusion)
    uint32_t* unit_owner;      // [unit_cap] long-fusion slot of each unit
    float* upart;              // [unit_cap][2 d + 2] unit partials (sum, compensation per channel; weight pair)
    int64_t unit_cap;
    int64_t n, total;
    const float* part_geom;
    float* grad2d;
    const uint32_t* visited;   // [n] bit v set for every visited (view v, Gaussian)
    const uint32_t* rank_of;
    const float* part_fuse;
    int d;
    int n_views;
    float *acc_sum, *acc_comp, *acc_wsum, *acc_wcomp;
    int wslot;                 // per-instance partial row (12 floats, surfels 16): weight sum at entry 9 (surfels 13)
};
void launch_render_fwd_f32(const RenderArgs& a, const ViewTable& vt, int n_tiles, hipStream_t s);
// slice: channels per workgroup; rows: pixel rows per workgroup (16 or 8)
bool render_fwd_bf16_shape_ok(int d, int slice, int rows);
void launch_render_fwd_bf16(const RenderArgs& a, const ViewTable& vt, int n_tiles, int slice, int rows, bool fsplit,
                            hipStream_t s);
// render_bwd.hip: the gradient kernel (needs dC); bf16: the BF16 form.  With dF
// and d >= 256 it needs a.g
void launch_render_grad(const BwdArgs& a, const ViewTable& vt, int n_tiles, bool bf16, hipStream_t s);
// Workgroups that share a tile's list where the list can be cut (the fusion with
// a.tseg, f . dF): with one a tile images of few tiles leave the chip idle, each a
// chain of a few hundred cycles a position.  About 1024 in all, four a CU.  Steps with
// fusion, 4,000 Gaussians, 128 channels: 12 tiles 926 -> 696 us, 48 tiles 538 -> 440,
// 320 tiles 372 -> 344, 432 tiles 373 -> 355; 100,000 of 256 channels 432 tiles 595 ->
// 589, 512 tiles 592 -> 602.
inline int list_parts(int64_t n_tiles) { return n_tiles <= 448 ? (int)(n_tiles <= 64 ? 16 : 1024 / n_tiles) : 1; }
// render_fuse.hip: the fusion partials (needs the target); ws: also the weight
// sums, which the gradient kernel of the same call writes otherwise
void launch_render_fuse(const BwdArgs& a, const ViewTable& vt, int n_tiles, bool bf16, bool ws, hipStream_t s);
void launch_visit_stage(const VisitStageArgs& a, hipStream_t s);
void launch_vseg(const uint32_t* skeys, const Counters* c, int64_t cap, uint32_t* vseg, const uint32_t* order, int64_t n,
                 uint32_t* visited, hipStream_t s);
// gp: floats per partial row, 12 (Gaussians: 10 used) or 16 (surfels: 14 used)
void launch_reduce_geom(const ReduceArgs& a, int gp, hipStream_t s);
void launch_reduce_fuse(const ReduceArgs& a, hipStream_t s);
// units available for the long fusion reduction at a visit capacity (see reduce.hip)
int64_t fuse_unit_capacity(int64_t visit_capacity);
// ndfd.hip
struct NdfdArgs {
    const uint32_t* tile_niter;
    const uint32_t* tile_voff;
    const Counters* counters;
    const float4* vrec;         // [visits * rw] staged records, in visit order
    const uint32_t* vgid;       // [visits] staged Gaussians
    const uint16_t* feat;       // [n, d] BF16 features
    int d;
    const float* T_final;
    const uint32_t* n_iter;
    const uint16_t* gt;         // [P, d] BF16 ground-truth feature map
    const float* a;             // [P] dL/dL_gt (nullable: 0)
    const float* b;             // [P] dL/dL_cf (nullable: 0)
    float lam, kk;              // sigmoid threshold and slope
    float* Lgt;                 // [P] (nullable)
    float* Lcf;                 // [P] (nullable)
    float* part;                // [visits][2 halves][ndfd_part_floats] screen-space partials (gradient)
    float2* sc;                 // [visits][256 pixels] (sigma, prefix term) of the forward sweep (gradient)
    int prim;                   // fh_primitive (surfel records: 4 float4)
};
bool ndfd_supported(int d);
int ndfd_part_floats(int prim);   // floats per (visit, half) partial: 8 (Gaussians), 16 (surfels)
void launch_ndfd(const NdfdArgs& a, const ViewTable& vt, int n_tiles, bool grad, hipStream_t s);
void launch_ndfd_combine(const float* part, float* part_geom, const Counters* c, int64_t cap, int prim,
                         hipStream_t s);
void launch_fuse_finalize(const float* sum, const float* comp, const float* wsum, const float* wcomp, int64_t n, int d,
                          const void* feat_in, void* feat_out, int bf16, hipStream_t s);

}  // namespace fh
