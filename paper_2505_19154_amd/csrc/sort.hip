// Tile binning: depth sort, instance generation, radix sort by tile, ranges.
//
// The paper's method (Appendix A, "Details of the Rasterizer"; Algorithm 2)
// duplicates every Gaussian once per overlapped tile, keys each copy with
// (tile << 32 | depth bits) and radix-sorts the keys.  This implementation
// reaches the same order with less traffic: the visible Gaussians of each view
// are first sorted by (depth, index) -- N keys instead of M instances -- and
// the instances are then generated in that order, so that a stable sort on
// the tile bits alone yields (tile, depth, index) order.  The instance key is
// (tile << rank_bits | rank), one u32 when it fits, else a u32 tile key with
// a u32 rank payload.
//
// Radix sort: LSD, digits of at most 8 bits, stable, by size of a segment:
// up to 16384 keys one workgroup sorts it in LDS, all passes in one launch;
// above that each pass counts the digits of every workgroup's keys (upsweep),
// turns them into positions and scatters (downsweep).  Waves rank their keys
// with ballot-based digit matching (positions are visited in order: stable,
// no LDS atomics).  See radix_sort for where the lines lie and why.  Against one
// size of tile (4096 keys, four waves) and four launches a pass: 1,000 keys 120
// -> 10 us (a launch takes 4 to 5 us of the stream, whatever it
// does); 500k pairs, 32 bits, 122 -> 74 us; 23M keys, 13
// bits, 251 -> 183 us; 430M pairs, 16 bits, 6.9 -> 5.0 ms (2.6 ms the pass that
// scatters each view over all 256 digits in runs of 32, 4.2 TB/s the other).
#include "kernels.hpp"

namespace fh {

constexpr int SCAN_BLOCK = 256;
constexpr int SCAN_ITEMS = 16;
constexpr int SCAN_TILE = SCAN_BLOCK * SCAN_ITEMS;   // 4096
constexpr int RADIX_TILE = 4096;    // the smallest tile of keys: the digit counts are sized for it
constexpr int SMALL_SORT = 16384;   // keys one workgroup sorts
constexpr int64_t MAX_SUM_ROWS = 48 * 1024;
constexpr int WAVE = 64;

// ---------------------------------------------------------------------------
// Block-wide exclusive scan of one u32 per thread (256 threads = 4 waves).
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t x, uint32_t* total, uint32_t* sh_wave) {
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    uint32_t incl = x;
#pragma unroll
    for (int off = 1; off < WAVE; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, WAVE);
        if (lane >= off) incl += y;
    }
    if (lane == WAVE - 1) sh_wave[w] = incl;
    __syncthreads();
    uint32_t wbase = 0, tot = 0;
    for (int k = 0; k < SCAN_BLOCK / WAVE; ++k) {
        const uint32_t s = sh_wave[k];
        if (k < w) wbase += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return wbase + incl - x;
}

__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_reduce(const uint32_t* __restrict__ in, int64_t n,
                                                            uint32_t* __restrict__ block_sums) {
    __shared__ uint32_t sh_wave[SCAN_BLOCK / WAVE];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i)
        if (base + i < n) s += in[base + i];
    uint32_t tot;
    block_exclusive_scan(s, &tot, sh_wave);
    if (threadIdx.x == 0) block_sums[blockIdx.x] = tot;
}

// out[i] = offsets[block] + exclusive prefix within the block; optionally
// out[n] = total (when total_out is set, written by the last block).
__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_down(const uint32_t* __restrict__ in, int64_t n,
                                                          const uint32_t* __restrict__ block_offsets,
                                                          uint32_t* __restrict__ out, int write_total) {
    __shared__ uint32_t sh_wave[SCAN_BLOCK / WAVE];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    uint32_t v[SCAN_ITEMS];
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        v[i] = (base + i < n) ? in[base + i] : 0u;
        s += v[i];
    }
    uint32_t tot;
    uint32_t run = block_exclusive_scan(s, &tot, sh_wave) + (block_offsets ? block_offsets[blockIdx.x] : 0u);
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        if (base + i < n) out[base + i] = run;
        run += v[i];
    }
    if (write_total && blockIdx.x == gridDim.x - 1 && threadIdx.x == SCAN_BLOCK - 1) out[n] = run;
}

// The same, with the block's offset formed in place: the sum of the block sums
// before it (integer sums, so the order of the additions does not matter).
__global__ __launch_bounds__(SCAN_BLOCK) void k_scan_down_sums(const uint32_t* __restrict__ in, int64_t n,
                                                               const uint32_t* __restrict__ block_sums,
                                                               uint32_t* __restrict__ out, int write_total) {
    __shared__ uint32_t sh_wave[SCAN_BLOCK / WAVE];
    uint32_t part = 0;
    for (int k = threadIdx.x; k < (int)blockIdx.x; k += SCAN_BLOCK) part += block_sums[k];
    uint32_t offset;
    block_exclusive_scan(part, &offset, sh_wave);
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    uint32_t v[SCAN_ITEMS];
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        v[i] = (base + i < n) ? in[base + i] : 0u;
        s += v[i];
    }
    uint32_t tot;
    uint32_t run = block_exclusive_scan(s, &tot, sh_wave) + offset;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        if (base + i < n) out[base + i] = run;
        run += v[i];
    }
    if (write_total && blockIdx.x == gridDim.x - 1 && threadIdx.x == SCAN_BLOCK - 1) out[n] = run;
}

// Scratch (in u32) needed by device_exclusive_scan for n items.
size_t scan_scratch_u32(int64_t n) {
    size_t tot = 0;
    int64_t m = n;
    while (m > SCAN_TILE) {
        m = (m + SCAN_TILE - 1) / SCAN_TILE;
        tot += (size_t)m + 64;
        tot += (size_t)m + 64;  // offsets of that level
    }
    return tot + 64;
}

// Exclusive scan of n u32 into out (out[n] = total if write_total).
void device_exclusive_scan(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* scratch, int write_total,
                           hipStream_t s) {
    if (n <= 0) return;
    const int64_t nb = (n + SCAN_TILE - 1) / SCAN_TILE;
    if (nb == 1) {
        hipLaunchKernelGGL(k_scan_down, dim3(1), dim3(SCAN_BLOCK), 0, s, in, n, (const uint32_t*)nullptr, out,
                           write_total);
        return;
    }
    uint32_t* sums = scratch;
    uint32_t* offs = scratch + nb + 64;
    uint32_t* next = offs + nb + 64;
    hipLaunchKernelGGL(k_scan_reduce, dim3((unsigned)nb), dim3(SCAN_BLOCK), 0, s, in, n, sums);
    if (nb <= 16 * SCAN_BLOCK) {
        // few blocks: each adds up the sums before it (two launches instead of three)
        hipLaunchKernelGGL(k_scan_down_sums, dim3((unsigned)nb), dim3(SCAN_BLOCK), 0, s, in, n, (const uint32_t*)sums,
                           out, write_total);
        return;
    }
    device_exclusive_scan(sums, offs, nb, next, 0, s);
    hipLaunchKernelGGL(k_scan_down, dim3((unsigned)nb), dim3(SCAN_BLOCK), 0, s, in, n, (const uint32_t*)offs, out,
                       write_total);
}

// The visits before every tile (out[n] = all of them), with the visit count and
// its overflow flag.  One workgroup takes up to 16384 tiles, in one launch
// instead of three.
__global__ __launch_bounds__(1024) void k_scan_visits(const uint32_t* __restrict__ in, int n, uint32_t* __restrict__ out,
                                                      Counters* c, int64_t cap) {
    __shared__ uint32_t sh[16];
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE, base = (int)threadIdx.x * SCAN_ITEMS;
    uint32_t v[SCAN_ITEMS], s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        v[i] = base + i < n ? in[base + i] : 0u;
        s += v[i];
    }
    uint32_t incl = s;
#pragma unroll
    for (int off = 1; off < WAVE; off <<= 1) {
        const uint32_t y = __shfl_up(incl, off, WAVE);
        if (lane >= off) incl += y;
    }
    if (lane == WAVE - 1) sh[w] = incl;
    __syncthreads();
    uint32_t run = incl - s;
    for (int k = 0; k < w; ++k) run += sh[k];
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        if (base + i < n) out[base + i] = run;
        run += v[i];
    }
    if (threadIdx.x == 1023) {
        out[n] = run;
        c->n_visited = run;
        c->visit_overflow = (unsigned long long)run > (unsigned long long)cap ? 1u : 0u;
    }
}
__global__ void k_check_visits(const uint32_t* total, Counters* c, int64_t cap) {
    if (threadIdx.x == 0) {
        c->n_visited = *total;
        c->visit_overflow = (unsigned long long)*total > (unsigned long long)cap ? 1u : 0u;
    }
}
void launch_scan_visits(const uint32_t* niter, uint32_t* voff, int64_t n_tiles, uint32_t* scratch, Counters* c, int64_t cap,
                        hipStream_t s) {
    if (n_tiles <= 1024 * SCAN_ITEMS) {
        hipLaunchKernelGGL(k_scan_visits, dim3(1), dim3(1024), 0, s, niter, (int)n_tiles, voff, c, cap);
        return;
    }
    device_exclusive_scan(niter, voff, n_tiles, scratch, 1, s);
    hipLaunchKernelGGL(k_check_visits, dim3(1), dim3(64), 0, s, (const uint32_t*)(voff + n_tiles), c, cap);
}

// ---------------------------------------------------------------------------
// Radix sort pass over equal-length segments laid out back to back.
// The valid length of every segment is seg_len, or min(*dev_len, cap) for a
// single segment whose length is only known on the device.
struct RadixPass {
    const uint32_t* keys_in;
    const uint32_t* vals_in;   // nullptr: payload = position within the segment
    uint32_t* keys_out;
    uint32_t* vals_out;
    uint32_t* hist;            // [seg * blocks_per_seg + block][256] digit counts; then [seg][256] totals (see below)
    Counters* reset;           // nullable: bin counters cleared by the launch
    const unsigned long long* dev_len;
    int64_t seg_len;
    int64_t cap;
    int segs, blocks_per_seg;
    int tiles_per_block;       // consecutive tiles one workgroup handles, in order
    int tile;                  // keys per tile
    int shift, bits;
};

__device__ __forceinline__ int64_t seg_valid_len(const RadixPass& p) {
    if (p.dev_len) {
        const unsigned long long m = *p.dev_len;
        return (int64_t)(m < (unsigned long long)p.cap ? m : (unsigned long long)p.cap);
    }
    return p.seg_len;
}
// workgroups of a segment that hold keys
__device__ __forceinline__ int valid_blocks(const RadixPass& p, int64_t len) {
    const int64_t per = (int64_t)p.tiles_per_block * p.tile;
    return (int)((len + per - 1) / per);
}

// Lanes of this wave whose digit equals mine (among lanes with valid = true).
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool valid, int bits) {
    const uint64_t v = ballot64(valid);
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
    for (int b = 0; b < bits; ++b) {
        const uint32_t x = (uint32_t)((int32_t)(d << (31 - b)) >> 31);   // all ones where the bit is set
        const uint64_t bb = ballot64(x != 0u);
        lo &= ~((uint32_t)bb ^ x);
        hi &= ~((uint32_t)(bb >> 32) ^ x);
    }
    return ((uint64_t)hi << 32) | lo;
}

// Stable ranks of a wave's ITEMS x 64 keys among the wave's keys of the same
// digit (in position order); cnt[256] (zeroed) receives the wave's digit counts.
template <int ITEMS>
__device__ __forceinline__ void rank_wave(const uint32_t* key, uint32_t* rank, int64_t first, int64_t len, int shift,
                                          int bits, uint32_t* cnt) {
    const uint32_t mask = (1u << bits) - 1u;
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const bool valid = first + i * WAVE < len;
        const uint32_t d = (key[i] >> shift) & mask;
        const uint64_t m = match_digit(d, valid, bits);
        const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
        uint32_t before = 0;
        if (valid) before = cnt[d];
        rank[i] = before + below;
        if (valid && below == 0u) cnt[d] = before + (uint32_t)__builtin_popcountll(m);
    }
}

// Counts per wave and digit -> the waves' exclusive prefixes in place; *lstart
// (thread d < 256): the tile's first position of digit d.  Returns the tile's
// count of digit d.  Ends with a barrier.
template <int WAVES>
__device__ __forceinline__ uint32_t digit_starts(uint32_t (*cnt)[256], uint32_t* lstart, uint32_t* wsum) {
    uint32_t tot = 0;
    if (threadIdx.x < 256) {
#pragma unroll
        for (int k = 0; k < WAVES; ++k) {
            const uint32_t c = cnt[k][threadIdx.x];
            cnt[k][threadIdx.x] = tot;
            tot += c;
        }
    }
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    uint32_t incl = tot;
#pragma unroll
    for (int off = 1; off < WAVE; off <<= 1) {
        const uint32_t t = (uint32_t)__shfl_up((int)incl, off, WAVE);
        if (lane >= off) incl += t;
    }
    if (w < 4 && lane == WAVE - 1) wsum[w] = incl;
    __syncthreads();
    if (threadIdx.x < 256) {
        uint32_t before = 0;
        for (int k = 0; k < w; ++k) before += wsum[k];
        lstart[threadIdx.x] = before + incl - tot;
    }
    __syncthreads();
    return tot;
}

__device__ __forceinline__ void reset_bin_counters(Counters* c) {
    c->n_instances = 0;
    c->inst_overflow = 0;
    c->n_visited = 0;
    c->visit_overflow = 0;
}

// A whole sort of one segment of at most 1024 ITEMS keys, all passes in one
// launch: the keys stay in registers and change places through LDS.  Bound:
// latency (one workgroup; about 4 us a pass of 4096 keys), against two or
// three launches a pass of 4 us each at least.
template <int ITEMS, bool VALS>
__global__ __launch_bounds__(1024) void k_sort_small(RadixPass p, int lo, int hi, int width) {
    constexpr int WAVES = 16;
    __shared__ uint32_t cnt[WAVES][256];
    __shared__ uint32_t lstart[256];
    __shared__ uint32_t wsum[4];
    __shared__ uint32_t skey[1024 * ITEMS];
    __shared__ uint32_t sval[VALS ? 1024 * ITEMS : 1];
    if (p.reset && blockIdx.x == 0 && threadIdx.x == 0) reset_bin_counters(p.reset);
    const int64_t len = seg_valid_len(p);
    const int64_t base = (int64_t)blockIdx.x * p.seg_len;
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    const int first = w * (ITEMS * WAVE) + lane;
    uint32_t key[ITEMS], val[VALS ? ITEMS : 1], rank[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int pos = first + i * WAVE;
        const bool valid = pos < len;
        key[i] = valid ? p.keys_in[base + pos] : 0u;
        if constexpr (VALS) val[i] = valid ? (p.vals_in ? p.vals_in[base + pos] : (uint32_t)pos) : 0u;
    }
    for (int shift = lo; shift < hi; shift += width) {
        const int bits = hi - shift < width ? hi - shift : width;
        for (int t = threadIdx.x; t < WAVES * 256; t += 1024) (&cnt[0][0])[t] = 0u;
        __syncthreads();
        rank_wave<ITEMS>(key, rank, first, len, shift, bits, cnt[w]);
        __syncthreads();
        digit_starts<WAVES>(cnt, lstart, wsum);
        const uint32_t mask = (1u << bits) - 1u;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            if (first + i * WAVE < len) {
                const uint32_t d = (key[i] >> shift) & mask;
                const uint32_t lp = lstart[d] + cnt[w][d] + rank[i];
                skey[lp] = key[i];
                if constexpr (VALS) sval[lp] = val[i];
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int pos = first + i * WAVE;
            if (pos < len) {
                key[i] = skey[pos];
                if constexpr (VALS) val[i] = sval[pos];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        const int pos = first + i * WAVE;
        if (pos < len) {
            p.keys_out[base + pos] = key[i];
            if constexpr (VALS) p.vals_out[base + pos] = val[i];
        }
    }
}

// Digit counts of a workgroup's keys, one row of 256 per workgroup.  Two
// copies in LDS by wave parity (equal digits of neighbouring keys serialise).
__global__ __launch_bounds__(512) void k_radix_upsweep(RadixPass p) {
    __shared__ uint32_t cnt[2][256];
    const int seg = blockIdx.x / p.blocks_per_seg, blk = blockIdx.x % p.blocks_per_seg;
    if (p.reset && blockIdx.x == 0 && threadIdx.x == 0) reset_bin_counters(p.reset);
    const uint32_t mask = (1u << p.bits) - 1u;
    (&cnt[0][0])[threadIdx.x] = 0u;
    __syncthreads();
    const int64_t len = seg_valid_len(p);
    const int64_t per = (int64_t)p.tiles_per_block * p.tile;
    const int64_t b0 = blk * per, b1 = b0 + per < len ? b0 + per : len;
    const uint32_t* in = p.keys_in + (int64_t)seg * p.seg_len;
    uint32_t* c = cnt[(threadIdx.x >> 6) & 1];
    for (int64_t pos = b0 + threadIdx.x; pos < b1; pos += 8 * 512) {
        uint32_t k[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) k[e] = pos + e * 512 < b1 ? in[pos + e * 512] : 0u;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (pos + e * 512 < b1) atomicAdd(&c[(k[e] >> p.shift) & mask], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 256)
        p.hist[((int64_t)seg * p.blocks_per_seg + blk) * 256 + threadIdx.x] = cnt[0][threadIdx.x] + cnt[1][threadIdx.x];
}

// Counts -> exclusive prefixes over a segment's workgroups, per digit, and the
// segment's totals.  One workgroup per (segment, 16 digits): 4 lanes of four
// digits by 256 runs of rows, then a wave a digit over the runs.  (64 digits a
// workgroup, 64 runs and a serial sum over them took 14 us of 1468 rows, this 8.5;
// the nine scans of a 16-view step 131 -> 83 us.)
__global__ __launch_bounds__(1024) void k_radix_scan(RadixPass p) {
    __shared__ uint32_t part[256][17];
    const int seg = blockIdx.x >> 4, d0 = (blockIdx.x & 15) * 16, dl = (threadIdx.x & 3) * 4, run = threadIdx.x >> 2;
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    const int rows = valid_blocks(p, seg_valid_len(p));
    const int per = (rows + 255) / 256, r0 = run * per, r1 = r0 + per < rows ? r0 + per : rows;
    uint32_t* h = p.hist + (int64_t)seg * p.blocks_per_seg * 256 + d0 + dl;
    uint32_t a0 = 0, a1 = 0, a2 = 0, a3 = 0;
#pragma unroll 8
    for (int r = r0; r < r1; ++r) {
        const uint4 c = *reinterpret_cast<const uint4*>(h + (int64_t)r * 256);
        a0 += c.x;
        a1 += c.y;
        a2 += c.z;
        a3 += c.w;
    }
    uint32_t* pr = &part[run][dl];
    pr[0] = a0;
    pr[1] = a1;
    pr[2] = a2;
    pr[3] = a3;
    __syncthreads();
    {
        uint32_t c[4], sum = 0;   // digit d0 + w, runs 4 lane .. + 3
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            c[e] = part[4 * lane + e][w];
            sum += c[e];
        }
        uint32_t incl = sum;
#pragma unroll
        for (int off = 1; off < WAVE; off <<= 1) {
            const uint32_t t = (uint32_t)__shfl_up((int)incl, off, WAVE);
            if (lane >= off) incl += t;
        }
        uint32_t before = incl - sum;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            part[4 * lane + e][w] = before;
            before += c[e];
        }
        if (lane == WAVE - 1) p.hist[((int64_t)p.segs * p.blocks_per_seg + seg) * 256 + d0 + w] = incl;
    }
    __syncthreads();
    a0 = pr[0];
    a1 = pr[1];
    a2 = pr[2];
    a3 = pr[3];
#pragma unroll 8
    for (int r = r0; r < r1; ++r) {
        uint4* at = reinterpret_cast<uint4*>(h + (int64_t)r * 256);
        const uint4 c = *at;
        *at = make_uint4(a0, a1, a2, a3);
        a0 += c.x;
        a1 += c.y;
        a2 += c.z;
        a3 += c.w;
    }
}

// Scatter of a workgroup's tiles, in order.  Per tile: stable ranks within
// each wave, per-digit prefixes over the waves and over the digits, the keys
// placed in LDS in digit order, then written out so that consecutive threads
// write consecutive positions of each digit's run; the next tile's keys are
// requested before.  SUM: the rows before this workgroup's and all of them
// are added up here (few rows, see radix_sort), else k_radix_scan did.
template <int THREADS, int ITEMS, bool VALS, bool SUM>
__global__ __launch_bounds__(THREADS) void k_radix_downsweep(RadixPass p) {
    constexpr int WAVES = THREADS / WAVE, TILE_KEYS = THREADS * ITEMS;
    static_assert(TILE_KEYS >= 8 * 2 * 256 && WAVES >= 8, "the row sums of eight waves alias the keys");
    __shared__ uint32_t cnt[WAVES][256];
    __shared__ uint32_t gbase[256];     // global position of the next key of each digit
    __shared__ uint32_t lstart[256];    // tile position of the tile's first key of each digit
    __shared__ uint32_t wsum[4];
    __shared__ __attribute__((aligned(16))) uint32_t skey[TILE_KEYS];
    __shared__ uint32_t sval[VALS ? TILE_KEYS : 1];
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    const int seg = blockIdx.x / p.blocks_per_seg, blk = blockIdx.x % p.blocks_per_seg;
    const int64_t len = seg_valid_len(p);
    const int64_t base = (int64_t)seg * p.seg_len;
    const int64_t b0 = (int64_t)blk * p.tiles_per_block * TILE_KEYS;
    if (b0 >= len) return;                                             // nothing to move (uniform)
    const int64_t b1 = b0 + (int64_t)p.tiles_per_block * TILE_KEYS < len ? b0 + (int64_t)p.tiles_per_block * TILE_KEYS : len;
    uint32_t key[ITEMS], val[VALS ? ITEMS : 1], rank[ITEMS];
    auto load = [&](int64_t first) {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const int64_t pos = first + i * WAVE;
            const bool valid = pos < b1;
            key[i] = valid ? p.keys_in[base + pos] : 0u;
            if constexpr (VALS) val[i] = valid ? (p.vals_in ? p.vals_in[base + pos] : (uint32_t)pos) : 0u;
        }
    };
    int64_t first = b0 + (int64_t)w * (ITEMS * WAVE) + lane;
    load(first);
    {
        const uint32_t* h = p.hist + (int64_t)seg * p.blocks_per_seg * 256;
        uint32_t before = 0, tot = 0;
        if constexpr (SUM) {
            uint32_t(*part)[2][256] = reinterpret_cast<uint32_t(*)[2][256]>(skey);
            if (w < 8) {
                const int rows = valid_blocks(p, len);
                uint32_t s[4] = {0, 0, 0, 0}, t[4] = {0, 0, 0, 0};
#pragma unroll 8
                for (int r = w; r < rows; r += 8) {
                    const uint4 c = *reinterpret_cast<const uint4*>(h + (int64_t)r * 256 + 4 * lane);
                    const bool prior = r < blk;
                    t[0] += c.x;
                    t[1] += c.y;
                    t[2] += c.z;
                    t[3] += c.w;
                    s[0] += prior ? c.x : 0u;
                    s[1] += prior ? c.y : 0u;
                    s[2] += prior ? c.z : 0u;
                    s[3] += prior ? c.w : 0u;
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    part[w][0][4 * lane + e] = s[e];
                    part[w][1][4 * lane + e] = t[e];
                }
            }
            __syncthreads();
            if (threadIdx.x < 256) {
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    before += part[k][0][threadIdx.x];
                    tot += part[k][1][threadIdx.x];
                }
            }
        } else if (threadIdx.x < 256) {
            before = h[(int64_t)blk * 256 + threadIdx.x];
            tot = p.hist[((int64_t)p.segs * p.blocks_per_seg + seg) * 256 + threadIdx.x];
        }
        // segment start + keys of smaller digits + this digit's keys of earlier workgroups
        uint32_t incl = tot;
#pragma unroll
        for (int off = 1; off < WAVE; off <<= 1) {
            const uint32_t t = (uint32_t)__shfl_up((int)incl, off, WAVE);
            if (lane >= off) incl += t;
        }
        if (w < 4 && lane == WAVE - 1) wsum[w] = incl;
        __syncthreads();
        if (threadIdx.x < 256) {
            uint32_t smaller = incl - tot;
            for (int k = 0; k < w; ++k) smaller += wsum[k];
            gbase[threadIdx.x] = (uint32_t)base + smaller + before;
        }
    }
    const uint32_t mask = (1u << p.bits) - 1u;
    for (int64_t tb = b0; tb < b1; tb += TILE_KEYS) {
        for (int t = threadIdx.x; t < WAVES * 256; t += THREADS) (&cnt[0][0])[t] = 0u;
        __syncthreads();
        rank_wave<ITEMS>(key, rank, first, b1, p.shift, p.bits, cnt[w]);
        __syncthreads();
        const uint32_t tot = digit_starts<WAVES>(cnt, lstart, wsum);
        // keys to LDS in digit order (stable: waves, then items and lanes, in order)
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            if (first + i * WAVE < b1) {
                const uint32_t d = (key[i] >> p.shift) & mask;
                const uint32_t lp = lstart[d] + cnt[w][d] + rank[i];
                skey[lp] = key[i];
                if constexpr (VALS) sval[lp] = val[i];
            }
        }
        __syncthreads();
        first += TILE_KEYS;
        if (tb + TILE_KEYS < b1) load(first);
        const int nb = (int)(b1 - tb < TILE_KEYS ? b1 - tb : TILE_KEYS);
        for (int lp = threadIdx.x; lp < nb; lp += THREADS) {
            const uint32_t k = skey[lp];
            const uint32_t d = (k >> p.shift) & mask;
            const int64_t dst = (int64_t)(gbase[d] + ((uint32_t)lp - lstart[d]));
            p.keys_out[dst] = k;
            if constexpr (VALS) p.vals_out[dst] = sval[lp];
        }
        __syncthreads();
        if (threadIdx.x < 256) gbase[threadIdx.x] += tot;
    }
}

template <int THREADS, int ITEMS>
static void launch_downsweep(const RadixPass& p, bool vals, bool sum, hipStream_t s) {
    const dim3 grid((unsigned)(p.segs * p.blocks_per_seg)), block(THREADS);
    if (vals && sum) hipLaunchKernelGGL((k_radix_downsweep<THREADS, ITEMS, true, true>), grid, block, 0, s, p);
    else if (vals) hipLaunchKernelGGL((k_radix_downsweep<THREADS, ITEMS, true, false>), grid, block, 0, s, p);
    else if (sum) hipLaunchKernelGGL((k_radix_downsweep<THREADS, ITEMS, false, true>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((k_radix_downsweep<THREADS, ITEMS, false, false>), grid, block, 0, s, p);
}

template <int ITEMS>
static void launch_sort_small(const RadixPass& p, bool vals, int lo, int hi, int width, hipStream_t s) {
    if (vals) hipLaunchKernelGGL((k_sort_small<ITEMS, true>), dim3((unsigned)p.segs), dim3(1024), 0, s, p, lo, hi, width);
    else hipLaunchKernelGGL((k_sort_small<ITEMS, false>), dim3((unsigned)p.segs), dim3(1024), 0, s, p, lo, hi, width);
}

// Sort `segs` segments of seg_len keys (or one segment of min(*dev_len, cap)
// keys) by bits [lo, hi).  Buffers alternate (a -> b -> a ...); returns the
// number of passes (the result is in b if odd, in a if even, except that the
// first pass reads from keys_src/vals_src).  reset (nullable): the bin
// counters, cleared on the way.
int radix_sort(const uint32_t* keys_src, const uint32_t* vals_src, uint32_t* ka, uint32_t* va, uint32_t* kb,
               uint32_t* vb, bool with_vals, int64_t segs, int64_t seg_len, const unsigned long long* dev_len,
               int64_t cap, int lo, int hi, uint32_t* hist, Counters* reset, hipStream_t s) {
    const int64_t span = dev_len ? cap : seg_len;
    if (span <= 0 || segs == 0) return 0;
    // digits of at most 8 bits, as even as the bit count allows (13 bits: 7 + 6,
    // so that each digit's run per tile is long enough to fill whole lines)
    const int npass = (hi - lo + 7) / 8;
    if (npass <= 0) return 0;
    const int width = (hi - lo + npass - 1) / npass;
    RadixPass p;
    p.hist = hist;
    p.reset = reset;
    p.dev_len = dev_len;
    p.seg_len = seg_len;
    p.cap = cap;
    p.segs = (int)segs;
    if (span <= SMALL_SORT) {
        p.keys_in = keys_src;
        p.vals_in = with_vals ? vals_src : nullptr;
        p.keys_out = npass % 2 ? kb : ka;
        p.vals_out = with_vals ? (npass % 2 ? vb : va) : nullptr;
        if (span <= 2048) launch_sort_small<2>(p, with_vals, lo, hi, width, s);
        else if (span <= 8192) launch_sort_small<8>(p, with_vals, lo, hi, width, s);
        else launch_sort_small<16>(p, with_vals, lo, hi, width, s);
        return npass;
    }
    // Tiles of 8192 keys fill the chip from about 1.5M keys on and write runs of
    // 32 keys a digit; below, 4096 keys over 16 waves have half the chain.
    const int64_t rows4 = (span + RADIX_TILE - 1) / RADIX_TILE;
    const bool big = segs * span > ((int64_t)3 << 19) || segs * rows4 * rows4 > MAX_SUM_ROWS;
    p.tile = big ? 8192 : RADIX_TILE;
    const int64_t tiles = (span + p.tile - 1) / p.tile;
    // several tiles per workgroup once there are more than ~2048 workgroups' worth
    p.tiles_per_block = (int)std::min<int64_t>(16, std::max<int64_t>(1, (segs * tiles + 2047) / 2048));
    p.blocks_per_seg = (int)((tiles + p.tiles_per_block - 1) / p.tiles_per_block);
    // Every workgroup adding up all rows of 1 KB itself saves a launch (5 us at
    // least) and costs segs * rows^2 KB of L2 reads: up to 48 MB.
    const bool sum = segs * p.blocks_per_seg * (int64_t)p.blocks_per_seg <= MAX_SUM_ROWS;
    int pass = 0;
    for (int shift = lo; shift < hi; shift += width, ++pass) {
        const bool first = (pass == 0), to_b = (pass % 2 == 0);
        p.keys_in = first ? keys_src : (to_b ? ka : kb);
        p.vals_in = with_vals ? (first ? vals_src : (to_b ? va : vb)) : nullptr;
        p.keys_out = to_b ? kb : ka;
        p.vals_out = with_vals ? (to_b ? vb : va) : nullptr;
        p.shift = shift;
        p.bits = (hi - shift) < width ? (hi - shift) : width;
        hipLaunchKernelGGL(k_radix_upsweep, dim3((unsigned)(segs * p.blocks_per_seg)), dim3(512), 0, s, p);
        p.reset = nullptr;
        if (!sum) hipLaunchKernelGGL(k_radix_scan, dim3((unsigned)(16 * segs)), dim3(1024), 0, s, p);
        if (big) launch_downsweep<512, 16>(p, with_vals, sum, s);
        else launch_downsweep<1024, 4>(p, with_vals, sum, s);
    }
    return pass;
}

// (a row per 4096 keys, or at most a row per 8192 of them and one of totals)
size_t radix_hist_u32(int64_t segs, int64_t span) {
    const int64_t bps = (span + RADIX_TILE - 1) / RADIX_TILE;
    return (size_t)(segs * 256 * (bps > 0 ? bps : 1)) + 64;
}

// ---------------------------------------------------------------------------
// Ranks.  k_rank_count: for j = v*N + r, the r-th Gaussian of view v in depth
// order, its tiles (0 when culled), their sum per 1024 ranks and the u64 total;
// the rank of each (view, Gaussian) and the screen records in rank order, so
// that a list entry (a rank) reaches its record with one load.  Bound: the
// gathers through the order (four ranks a thread in flight).
constexpr int RANKS_BLOCK = 1024;
__global__ __launch_bounds__(256) void k_rank_count(RankArgs a) {
    __shared__ unsigned long long red[4];
    uint32_t total = (uint32_t)a.total, n = (uint32_t)a.n;
    const uint32_t j0 = blockIdx.x * (uint32_t)RANKS_BLOCK + threadIdx.x;
    uint32_t i[4];
    int4 r[4];
    bool on[4];
    unsigned long long s = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint32_t j = j0 + e * 256u;
        on[e] = j < total && j >= j0;
        i[e] = on[e] ? j / n * n + a.order[j] : 0u;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] = on[e] ? a.rect[i[e]] : make_int4(0, 0, -1, -1);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const uint32_t j = j0 + e * 256u;
        if (!on[e]) continue;
        const uint32_t c = (r[e].x <= r[e].z && r[e].y <= r[e].w) ? (uint32_t)((r[e].z - r[e].x + 1) * (r[e].w - r[e].y + 1)) : 0u;
        a.ntiles[j] = c;
        if (c == 0u) continue;   // (no list holds it: its record and rank are not read)
        s += c;
        a.rank_of[i[e]] = j - j / n * n;
        for (int k = 0; k < a.rw; ++k) a.rrec[a.rw * (int64_t)j + k] = a.rec[a.rw * (int64_t)i[e] + k];
    }
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned long long t = red[0] + red[1] + red[2] + red[3];
        a.sums[blockIdx.x] = (uint32_t)t;
        if (t) atomicAdd(&a.counters->n_instances, t);
    }
}

// k_rank_scan: the first instance of every rank, the rank that owns every
// DUP_TILE-th instance (where k_duplicate's workgroups start), the overflow
// flag, and the tiles' ranges cleared.  Each workgroup adds up the sums before
// it (scanned: they are prefixes already).
constexpr int DUP_TILE = 2048;
__global__ __launch_bounds__(SCAN_BLOCK) void k_rank_scan(RankArgs a, int scanned) {
    __shared__ uint32_t sh_wave[SCAN_BLOCK / WAVE];
    uint32_t offset;
    const int before = (int)blockIdx.x * (SCAN_TILE / RANKS_BLOCK);
    if (scanned) {
        offset = a.sums[before];
    } else {
        uint32_t part = 0;
        for (int k = threadIdx.x; k < before; k += SCAN_BLOCK) part += a.sums[k];
        block_exclusive_scan(part, &offset, sh_wave);
    }
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    uint32_t v[SCAN_ITEMS];
    uint32_t s = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        v[i] = (base + i < a.total) ? a.ntiles[base + i] : 0u;
        s += v[i];
    }
    uint32_t tot;
    uint32_t run = block_exclusive_scan(s, &tot, sh_wave) + offset;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        if (base + i < a.total) {
            a.inst_off[base + i] = run;
            for (uint32_t m = (run + DUP_TILE - 1) / DUP_TILE; v[i] && m < a.n_starts && m * DUP_TILE - run < v[i]; ++m)
                a.starts[m] = (uint32_t)(base + i);
        }
        run += v[i];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == SCAN_BLOCK - 1) {
        a.inst_off[a.total] = run;
        a.counters->inst_overflow = a.counters->n_instances > (unsigned long long)a.cap ? 1u : 0u;
    }
    if (a.ranges)
        for (int64_t k = (int64_t)blockIdx.x * SCAN_BLOCK + threadIdx.x; k < a.n_ranges; k += (int64_t)gridDim.x * SCAN_BLOCK)
            a.ranges[k] = 0u;
}

// sums and starts share the digit counts' buffer, which is free between the sorts
void launch_ranks(const RankArgs& a0, uint32_t* hist, uint32_t* scan_tmp, hipStream_t s) {
    RankArgs a = a0;
    const int64_t ns = (a.total + RANKS_BLOCK - 1) / RANKS_BLOCK;
    a.sums = hist;
    a.starts = const_cast<uint32_t*>(dup_starts(hist, a.total));
    a.n_starts = (uint32_t)((a.cap + DUP_TILE - 1) / DUP_TILE);
    hipLaunchKernelGGL(k_rank_count, dim3((unsigned)ns), dim3(256), 0, s, a);
    // (up to 16384 sums, 64 a thread; beyond, a scan of their own)
    const int scanned = ns > 16384;
    if (scanned) device_exclusive_scan(a.sums, a.sums, ns, scan_tmp, 0, s);
    hipLaunchKernelGGL(k_rank_scan, dim3((unsigned)((a.total + SCAN_TILE - 1) / SCAN_TILE)), dim3(SCAN_BLOCK), 0, s, a, scanned);
}

// Instance generation.  Each workgroup writes a fixed range of 2048 output
// instances (so that the few huge Gaussians at the front of the depth order
// spread over many workgroups).  The ranks covering the range are staged in
// LDS with their first instance; every rank marks the position where its
// instances start (the largest rank wins: a rank with no instance starts where
// the next one does), and a prefix maximum over the range gives every
// instance its rank.  A range that spans more ranks than the window holds (most
// splats in one tile each, or a view boundary with culled ranks, which own none)
// searches the scan in global memory, an instance a thread.
constexpr int DUP_WIN = 1024;

// largest r in [lo, hi] with off[r] <= i (off non-decreasing, off[lo] <= i)
__device__ __forceinline__ int64_t last_le(const uint32_t* off, int64_t lo, int64_t hi, uint32_t i) {
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (off[mid] <= i) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// The same search by all 256 threads of a workgroup (uniform arguments): each
// round probes 256 evenly spaced entries and keeps the interval after the last
// one <= i (the probes' test is true for a prefix of the threads), so a search
// over R entries takes log_256(R) rounds of parallel loads instead of log2(R)
// dependent ones.
__device__ __forceinline__ int64_t block_last_le(const uint32_t* off, int64_t lo, int64_t hi, uint32_t i) {
    while (hi - lo >= 256) {
        const int64_t step = (hi - lo + 256) / 256;
        const int64_t pr = lo + (int64_t)threadIdx.x * step;
        const int cnt = __syncthreads_count(pr <= hi && off[pr] <= i);
        lo += (int64_t)(cnt - 1) * step;
        hi = lo + step - 1 < hi ? lo + step - 1 : hi;
    }
    const int64_t pr = lo + (int64_t)threadIdx.x;
    const int cnt = __syncthreads_count(pr <= hi && off[pr] <= i);
    return lo + cnt - 1;
}

// q = a / b, r = a % b for a < 2^22, 1 <= b < 2^12: the float estimate is
// within one of the quotient (relative error below 2^-22), then corrected.
__device__ __forceinline__ void divmod_small(uint32_t a, uint32_t b, uint32_t& q, uint32_t& r) {
    uint32_t qq = (uint32_t)((float)a * __builtin_amdgcn_rcpf((float)b));
    int32_t rr = (int32_t)a - (int32_t)(qq * b);
    if (rr < 0) {
        qq -= 1u;
        rr += (int32_t)b;
    }
    if (rr >= (int32_t)b) {
        qq += 1u;
        rr -= (int32_t)b;
    }
    q = qq;
    r = (uint32_t)rr;
}

__global__ __launch_bounds__(256) void k_duplicate(DupArgs a) {
    constexpr int PER = DUP_TILE / 256;   // positions per thread in the prefix maximum
    // (20 KB of LDS per workgroup, so that eight are resident per CU)
    __shared__ uint32_t offs[DUP_WIN + 1];
    __shared__ uint2 rects[DUP_WIN];      // tile rect origin (x0 | y0 << 16: views are at most 1024 tiles wide) and width
    __shared__ uint32_t owner[DUP_TILE];  // window index + 1 of the rank owning each position
    __shared__ uint32_t wmax[4];
    __shared__ long long s_r0;
    __shared__ int s_win;
    if (a.counters->inst_overflow) return;   // uniform over the block
    const int64_t m = (int64_t)a.counters->n_instances;
    const int64_t ib = (int64_t)blockIdx.x * DUP_TILE;
    if (ib >= m) return;                      // uniform over the block
    const int64_t ie = ib + DUP_TILE < m ? ib + DUP_TILE : m;
    {
        // (the owners of this range's first instance and of the next range's, from
        // the scan: a search took six dependent loads, most of the workgroup's time)
        const int64_t q0 = a.starts[blockIdx.x];
        const int64_t q1 = ib + DUP_TILE < m ? (int64_t)a.starts[blockIdx.x + 1]
                                             : block_last_le(a.inst_off, q0, a.total_ranks - 1, (uint32_t)(ie - 1));
        if (threadIdx.x == 0) {
            s_r0 = q0;
            s_win = (q1 - q0 + 1 <= DUP_WIN) ? (int)(q1 - q0 + 1) : -1;
        }
    }
    for (int k = threadIdx.x; k < DUP_TILE; k += 256) owner[k] = 0u;
    __syncthreads();
    const int64_t r0 = s_r0;
    const int win = s_win;
    if (win > 0) {
        for (int k = threadIdx.x; k <= win; k += 256) offs[k] = a.inst_off[r0 + k];
        for (int k = threadIdx.x; k < win; k += 256) {
            const int64_t j = r0 + k;
            const int4 rc = a.rect[(j / a.n) * a.n + a.order[j]];
            rects[k] = make_uint2((uint32_t)rc.x | ((uint32_t)rc.y << 16), (uint32_t)(rc.z - rc.x + 1));
        }
        __syncthreads();
        for (int k = threadIdx.x; k < win; k += 256) {
            const uint32_t st = offs[k];
            if (st >= (uint64_t)ib && st < (uint64_t)ie) atomicMax(&owner[st - (uint32_t)ib], (uint32_t)k + 1u);
        }
        if (threadIdx.x == 0) atomicMax(&owner[0], 1u);   // the first rank owns the range's first instance
        __syncthreads();
        // inclusive prefix maximum: PER consecutive positions per thread, then over threads
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        uint32_t run = 0;
#pragma unroll
        for (int e = 0; e < PER; ++e) run = max(run, owner[threadIdx.x * PER + e]);
        uint32_t incl = run;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t t = (uint32_t)__shfl_up((int)incl, off, 64);
            if (lane >= off) incl = max(incl, t);
        }
        if (lane == 63) wmax[w] = incl;
        uint32_t excl = (uint32_t)__shfl_up((int)incl, 1, 64);
        if (lane == 0) excl = 0u;
        __syncthreads();
        for (int k = 0; k < w; ++k) excl = max(excl, wmax[k]);
        uint32_t cur = excl;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            cur = max(cur, owner[threadIdx.x * PER + e]);
            owner[threadIdx.x * PER + e] = cur;
        }
    }
    __syncthreads();
    for (int64_t ii = ib + threadIdx.x; ii < ie; ii += 256) {
        const uint32_t i = (uint32_t)ii;
        int64_t j;
        uint32_t x0, y0, wdt, local;
        if (win > 0) {
            const int wi = (int)owner[ii - ib] - 1;
            j = r0 + wi;
            const uint2 r = rects[wi];
            x0 = r.x & 0xFFFFu;
            y0 = r.x >> 16;
            wdt = r.y;
            local = i - offs[wi];
        } else {
            j = last_le(a.inst_off, r0, a.total_ranks - 1, i);
            const int4 r = a.rect[(j / a.n) * a.n + a.order[j]];
            x0 = (uint32_t)r.x;
            y0 = (uint32_t)r.y;
            wdt = (uint32_t)(r.z - r.x + 1);
            local = i - a.inst_off[j];
        }
        const int v = (int)(j / a.n);
        uint32_t qy, qx;
        divmod_small(local, wdt, qy, qx);
        const uint32_t tx = x0 + qx;
        const uint32_t ty = y0 + qy;
        const uint32_t tile = (uint32_t)a.vt.tile_off[v] + ty * (uint32_t)a.vt.tiles_x[v] + tx;
        if (a.packed) {
            a.keys[i] = (tile << a.rank_bits) | (uint32_t)j;
        } else {
            a.keys[i] = tile;
            a.vals[i] = (uint32_t)j;
        }
    }
}

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* p, int64_t n, uint32_t v) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = v;
}

// the same for a 16-byte aligned p, four values per thread
__global__ __launch_bounds__(256) void k_fill_u32x4(uint32_t* p, int64_t n, uint32_t v) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i + 4 <= n) {
        *reinterpret_cast<uint4*>(p + i) = make_uint4(v, v, v, v);
    } else {
        for (int64_t k = i; k < n; ++k) p[k] = v;
    }
}

__device__ __forceinline__ uint32_t inst_tile(const uint32_t* keys, int64_t i, int rank_bits, int packed) {
    return packed ? (keys[i] >> rank_bits) : keys[i];
}

// [start, end) of every non-empty tile's run in the sorted instances; each
// thread checks 8 consecutive instances against their neighbours.
__global__ __launch_bounds__(256) void k_ranges(const uint32_t* __restrict__ keys, const Counters* counters,
                                                int64_t cap, int rank_bits, int packed, uint32_t* ranges) {
    if (counters->inst_overflow) return;
    const int64_t n_inst = (int64_t)counters->n_instances;
    const int64_t m = n_inst < cap ? n_inst : cap;
    const int64_t i0 = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
    if (i0 >= m) return;
    uint32_t t[8];
    if (i0 + 8 <= m) {
        const uint4 a0 = *reinterpret_cast<const uint4*>(keys + i0);
        const uint4 a1 = *reinterpret_cast<const uint4*>(keys + i0 + 4);
        t[0] = a0.x; t[1] = a0.y; t[2] = a0.z; t[3] = a0.w;
        t[4] = a1.x; t[5] = a1.y; t[6] = a1.z; t[7] = a1.w;
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) t[e] = i0 + e < m ? keys[i0 + e] : 0u;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) t[e] = packed ? (t[e] >> rank_bits) : t[e];
    uint32_t prev = i0 > 0 ? inst_tile(keys, i0 - 1, rank_bits, packed) : 0xFFFFFFFFu;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int64_t i = i0 + e;
        if (i >= m) break;
        if (i == 0 || prev != t[e]) ranges[2 * t[e]] = (uint32_t)i;
        const uint32_t next = e < 7 ? (i + 1 < m ? t[e + 1] : 0xFFFFFFFFu)
                                    : (i + 1 < m ? inst_tile(keys, i + 1, rank_bits, packed) : 0xFFFFFFFFu);
        if (i == m - 1 || next != t[e]) ranges[2 * t[e] + 1] = (uint32_t)(i + 1);
        prev = t[e];
    }
}

// The paper's 64-bit keys of the sorted instances.
__global__ __launch_bounds__(256) void k_bin_keys(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ vals,
                                                  const uint32_t* __restrict__ order,
                                                  const uint32_t* __restrict__ depth_key, int64_t n_inst, int64_t n,
                                                  int rank_bits, int packed, uint64_t* keys_out, uint32_t* gid_out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n_inst) return;
    const uint32_t tile = packed ? (keys[i] >> rank_bits) : keys[i];
    const uint32_t j = packed ? (keys[i] & ((1u << rank_bits) - 1u)) : vals[i];
    const int64_t v = (int64_t)j / n;
    const uint32_t g = order[j];
    if (keys_out) keys_out[i] = ((uint64_t)tile << 32) | (uint64_t)depth_key[v * n + g];
    if (gid_out) gid_out[i] = g;
}

// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_tile_cost_keys(const uint32_t* __restrict__ ranges,
                                                      const uint32_t* __restrict__ tile_niter, int64_t n_tiles,
                                                      uint32_t* __restrict__ keys) {
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= n_tiles) return;
    const uint32_t cost = ranges ? ranges[2 * t + 1] - ranges[2 * t] : tile_niter[t];
    keys[t] = 0xFFFFu - (cost < 0xFFFFu ? cost : 0xFFFFu);
}

void launch_tile_cost_keys(const uint32_t* ranges, const uint32_t* tile_niter, int64_t n_tiles, uint32_t* keys,
                           hipStream_t s) {
    if (n_tiles <= 0) return;
    hipLaunchKernelGGL(k_tile_cost_keys, dim3((unsigned)((n_tiles + 255) / 256)), dim3(256), 0, s, ranges, tile_niter,
                       n_tiles, keys);
}

void launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t s) {
    if (n <= 0) return;
    if (reinterpret_cast<uintptr_t>(p) % 16 == 0) {
        const int64_t threads = (n + 3) / 4;
        hipLaunchKernelGGL(k_fill_u32x4, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, p, n, v);
    } else {
        hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    }
}

void launch_duplicate(const DupArgs& a, hipStream_t s) {
    if (a.cap <= 0 || a.total_ranks <= 0) return;
    hipLaunchKernelGGL(k_duplicate, dim3((unsigned)((a.cap + DUP_TILE - 1) / DUP_TILE)), dim3(256), 0, s, a);
}

void launch_ranges(const uint32_t* keys, const Counters* c, int64_t cap, int rank_bits, int packed, uint32_t* ranges,
                   hipStream_t s) {
    const int64_t threads = (cap + 7) / 8;
    if (threads > 0)
        hipLaunchKernelGGL(k_ranges, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, keys, c, cap, rank_bits,
                           packed, ranges);
}

void launch_bin_keys(const uint32_t* keys, const uint32_t* vals, const uint32_t* order, const uint32_t* depth_key,
                     int64_t n_inst, int64_t n, int rank_bits, int packed, uint64_t* ko, uint32_t* go,
                     hipStream_t s) {
    if (n_inst <= 0) return;
    hipLaunchKernelGGL(k_bin_keys, dim3((unsigned)((n_inst + 255) / 256)), dim3(256), 0, s, keys, vals, order, depth_key,
                       n_inst, n, rank_bits, packed, ko, go);
}

}  // namespace fh
