// Gaussian-tile pair binning on gfx950: exclusive scans, the pairs of every Gaussian, their order
// (tile, depth, index) and the per-tile ranges.  All integer work; results are unique and reproducible
// bit for bit.
//
// FastGS Sec. 3 blends "Gaussians sorted by depth" per pixel; Sec. 4.4 names the Gaussian-tile pairs that
// the 3-sigma rule (or the Compact Box) produces.  A pair's key is tile_id << 32 | bits(depth).  Two ways
// to the same order live here: the tile-bucketed one (count per tile, place, sort each tile's segment in
// LDS), used whenever the lists are short enough, and a global stable LSD radix sort of index-ordered keys.
//
// Times "at 500k Gaussians" and the like are of the scenes of perf/cases.py, those at 10 M and 27 M pairs of bench.py's largest.
#include <algorithm>
#include <type_traits>

#include "common.hpp"

namespace fs {

namespace {

// The render kernels take the tiles longest list first, by buckets of list lengths; the last bucket takes all longer ones.
constexpr int ORDER_BUCKETS = 512;
constexpr uint32_t ORDER_STEP = 8;

constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_BLOCK = SCAN_THREADS * SCAN_ITEMS;  // 2048 values per workgroup

// Exclusive scan over the 256 threads of a workgroup; returns the thread's exclusive prefix and
// the workgroup total.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* total, uint32_t* smem /*[4]*/)
{
    const uint32_t inc = wave_inclusive_scan(v);
    const int wave = threadIdx.x >> 6;
    __syncthreads();
    if (lane_id() == 63) smem[wave] = inc;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < 4; w++) {
        const uint32_t s = smem[w];
        if (w < wave) base += s;
        tot += s;
    }
    *total = tot;
    return base + inc - v;
}

// Pass 1: per-workgroup sums (64-bit, so that a total beyond 2^32 is detected by the caller).
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_block_sums(const uint32_t* __restrict__ in, int64_t n,
                                                                 uint64_t* __restrict__ block_sums)
{
    __shared__ uint32_t smem[4];
    const int64_t base = (int64_t)blockIdx.x * SCAN_BLOCK + threadIdx.x * SCAN_ITEMS;
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++)
        if (base + k < n) s += in[base + k];
    uint32_t tot;
    block_exclusive_scan(s, &tot, smem);
    if (threadIdx.x == 0) block_sums[blockIdx.x] = tot;
}

// Pass 2: one workgroup turns the block sums into exclusive block offsets (sequential chunks).
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_block_offsets(uint64_t* __restrict__ block_sums,
                                                                    int64_t num_blocks,
                                                                    uint64_t* __restrict__ total_out)
{
    __shared__ uint64_t wave_tot[4];
    __shared__ uint64_t carry_s;
    if (threadIdx.x == 0) carry_s = 0;
    __syncthreads();
    for (int64_t c = 0; c < num_blocks; c += SCAN_THREADS) {
        const int64_t i = c + threadIdx.x;
        const uint64_t v = i < num_blocks ? block_sums[i] : 0;
        // 64-bit inclusive scan within the wave
        uint64_t inc = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t lo = __shfl_up((uint32_t)inc, d, 64);
            const uint32_t hi = __shfl_up((uint32_t)(inc >> 32), d, 64);
            if ((int)lane_id() >= d) inc += ((uint64_t)hi << 32) | lo;
        }
        const int wave = threadIdx.x >> 6;
        if (lane_id() == 63) wave_tot[wave] = inc;
        __syncthreads();
        uint64_t base = carry_s;
        for (int w = 0; w < wave; w++) base += wave_tot[w];
        if (i < num_blocks) block_sums[i] = base + inc - v;
        __syncthreads();
        if (threadIdx.x == SCAN_THREADS - 1) carry_s = base + inc;
        __syncthreads();
    }
    if (threadIdx.x == 0) *total_out = carry_s;
}

// Pass 3: exclusive scan inside each workgroup plus its block offset.
// `in` and `out` may be the same array (each thread reads its values before writing them).
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_apply(const uint32_t* in, uint32_t* out, int64_t n,
                                                            const uint64_t* __restrict__ block_offsets)
{
    __shared__ uint32_t smem[4];
    const int64_t base = (int64_t)blockIdx.x * SCAN_BLOCK + threadIdx.x * SCAN_ITEMS;
    uint32_t v[SCAN_ITEMS];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) {
        v[k] = base + k < n ? in[base + k] : 0u;
        s += v[k];
    }
    uint32_t tot;
    uint32_t run = block_exclusive_scan(s, &tot, smem) + (uint32_t)block_offsets[blockIdx.x];
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; k++) {
        if (base + k < n) out[base + k] = run;
        run += v[k];
    }
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int d)
{
    return (uint64_t)(uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), d, 64) << 32 | (uint32_t)__shfl_xor((int)(uint32_t)v, d, 64);
}

// The 64-byte record the render kernels gather for Gaussian i (see SPLAT_REC).
__device__ __forceinline__ void pack_splat(float4* __restrict__ splats, int64_t i, const float2& m, const float4& co,
                                           const float* __restrict__ rgb, uint32_t first_record, const ushort4& r, const CfgDev& cfg)
{
    float4* rec = splats + (size_t)i * (SPLAT_REC / 4);
    rec[0] = make_float4(m.x, m.y, co.x, co.y);
    rec[1] = make_float4(co.z, co.w, rgb[3 * i], rgb[3 * i + 1]);
    rec[2] = make_float4(rgb[3 * i + 2], __uint_as_float(first_record | (is_needle(co) ? NEEDLE : 0u)), __uint_as_float((uint32_t)r.x | (uint32_t)r.y << 16),
                         __uint_as_float((uint32_t)r.z | (uint32_t)r.w << 16));
    rec[3] = support_strips(co, cfg);
}

// One key per tile of each Gaussian's rectangle, rows then columns, starting at offsets[i].  A
// wavefront takes 64 consecutive Gaussians; their pairs occupy one contiguous run of the output, and
// the wavefront writes that run 64 pairs at a time (lane j of a round finds the Gaussian that owns
// output slot j by a binary search over the lanes' running counts), so a Gaussian that touches
// hundreds of tiles does not stall its 63 neighbours and every store is coalesced.  Each lane also
// packs its own Gaussian's projected splat, rectangle and pair offset into one 64-byte record, so
// that the render kernels gather one cache line per (Gaussian, tile) pair instead of five.
__global__ __launch_bounds__(256) void k_emit_pairs(int64_t n, const ushort4* __restrict__ rect,
                                                    const float* __restrict__ depth,
                                                    const float2* __restrict__ mean2d,
                                                    const float4* __restrict__ conic_opacity,
                                                    const float* __restrict__ rgb, CfgDev cfg,
                                                    const uint32_t* __restrict__ offsets, int tiles_x,
                                                    uint64_t* __restrict__ keys, uint32_t* __restrict__ vals,
                                                    float4* __restrict__ splats)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < n;
    const uint32_t lane = lane_id();
    const ushort4 r = valid ? rect[i] : make_ushort4(0, 0, 0, 0);
    const uint32_t w = r.z > r.x ? (uint32_t)(r.z - r.x) : 0u, h = r.w > r.y ? (uint32_t)(r.w - r.y) : 0u;
    const uint32_t cnt = w * h;
    const uint32_t off = valid ? offsets[i] : 0u;
    const uint32_t dbits = cnt ? __float_as_uint(depth[i]) : 0u;
    if (cnt) {
        const float2 m = mean2d[i];
        const float4 co = conic_opacity[i];
        pack_splat(splats, i, m, co, rgb, off, r, cfg);
    }
    const uint32_t inc = wave_inclusive_scan(cnt);
    const uint32_t excl = inc - cnt;                       // this lane's first slot within the wave's run
    const uint32_t total = (uint32_t)__shfl((int)inc, 63, 64);
    const uint32_t run_start = (uint32_t)__shfl((int)off, 0, 64);  // offsets[] of the wave's first Gaussian
    const uint32_t rect_xy = (uint32_t)r.x | (uint32_t)r.y << 16;
    for (uint32_t j0 = 0; j0 < total; j0 += 64) {
        const uint32_t j = min(j0 + lane, total - 1);     // clamped: every lane takes part in the shuffles
        // owner = last lane whose first slot is <= j (lanes without pairs share their successor's first slot)
        uint32_t s = 0;
#pragma unroll
        for (uint32_t step = 32; step >= 1; step >>= 1) {
            const uint32_t t = s + step;
            const uint32_t e = (uint32_t)__shfl((int)excl, (int)t, 64);
            s = e <= j ? t : s;
        }
        const uint32_t k = j - (uint32_t)__shfl((int)excl, (int)s, 64);  // place in the owner's rectangle, row-major
        const uint32_t ow = (uint32_t)__shfl((int)w, (int)s, 64);
        const uint32_t oxy = (uint32_t)__shfl((int)rect_xy, (int)s, 64);
        const uint32_t od = (uint32_t)__shfl((int)dbits, (int)s, 64);
        const uint32_t row = rect_row(k, ow);
        const uint32_t col = k - row * ow;
        const uint32_t tx = (oxy & 0xffffu) + col, ty = (oxy >> 16) + row;
        if (j0 + lane < total) {
            const size_t o = (size_t)run_start + j0 + lane;
            keys[o] = ((uint64_t)(ty * (uint32_t)tiles_x + tx) << 32) | od;
            vals[o] = (uint32_t)(i - lane + s);
        }
    }
}

// Compact Box: tiles in each Gaussian's box (the candidates of the ellipse test).
__global__ __launch_bounds__(256) void k_rect_area(int64_t n, const ushort4* __restrict__ rect,
                                                   uint32_t* __restrict__ area)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const ushort4 r = rect[i];
    area[i] = r.z > r.x && r.w > r.y ? (uint32_t)(r.z - r.x) * (uint32_t)(r.w - r.y) : 0u;
}

// Compact Box emission.  Same wave-cooperative walk as k_emit_pairs, but over the candidates (all tiles of
// each box): the lane that takes a candidate runs the ellipse-tile test; a hit becomes a key at
// offsets[owner] + (hits of the same Gaussian before it, in row-major order).  Hits of one Gaussian before a
// candidate = those of earlier rounds (kept by the owner lane in `emitted`) + those on lower lanes of this
// round (one ballot, masked to the owner's lanes).
__global__ __launch_bounds__(256) void k_emit_pairs_cb(int64_t n, const ushort4* __restrict__ rect,
                                                       const float* __restrict__ depth,
                                                       const float2* __restrict__ mean2d,
                                                       const float4* __restrict__ conic_opacity,
                                                       const float* __restrict__ rgb, CfgDev cfg,
                                                       const uint32_t* __restrict__ offsets,
                                                       const uint32_t* __restrict__ rec_offsets, int tiles_x,
                                                       uint32_t P, uint64_t* __restrict__ keys,
                                                       uint32_t* __restrict__ vals,
                                                       float4* __restrict__ splats)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < n;
    const uint32_t lane = lane_id();
    const ushort4 r = valid ? rect[i] : make_ushort4(0, 0, 0, 0);
    const uint32_t w = r.z > r.x ? (uint32_t)(r.z - r.x) : 0u, h = r.w > r.y ? (uint32_t)(r.w - r.y) : 0u;
    const uint32_t cnt = w * h;                              // candidates
    const uint32_t off = valid ? offsets[i] : 0u;           // first pair
    const uint32_t roff = valid ? rec_offsets[i] : 0u;      // first gradient record
    const uint32_t dbits = cnt ? __float_as_uint(depth[i]) : 0u;
    float mx = 0.f, my = 0.f, A = 1.f, B = 0.f, C = 1.f, Q = 0.f;
    if (cnt) {
        const float2 m = mean2d[i];
        const float4 co = conic_opacity[i];
        mx = m.x; my = m.y; A = co.x; B = co.y; C = co.z;
        Q = cb_threshold(co.w, cfg);
        pack_splat(splats, i, m, co, rgb, roff, r, cfg);
    }
    const uint32_t inc = wave_inclusive_scan(cnt);
    const uint32_t excl = inc - cnt;
    const uint32_t total = (uint32_t)__shfl((int)inc, 63, 64);
    const uint32_t rect_xy = (uint32_t)r.x | (uint32_t)r.y << 16;
    uint32_t emitted = 0;                                    // hits of this lane's own Gaussian so far
    for (uint32_t j0 = 0; j0 < total; j0 += 64) {
        const bool live = j0 + lane < total;
        const uint32_t j = min(j0 + lane, total - 1);
        uint32_t s = 0;
#pragma unroll
        for (uint32_t step = 32; step >= 1; step >>= 1) {
            const uint32_t t = s + step;
            const uint32_t e = (uint32_t)__shfl((int)excl, (int)t, 64);
            s = e <= j ? t : s;
        }
        const uint32_t oexcl = (uint32_t)__shfl((int)excl, (int)s, 64);
        const uint32_t k = j - oexcl;
        const uint32_t ow = (uint32_t)__shfl((int)w, (int)s, 64);
        const uint32_t oxy = (uint32_t)__shfl((int)rect_xy, (int)s, 64);
        const uint32_t od = (uint32_t)__shfl((int)dbits, (int)s, 64);
        const uint32_t ooff = (uint32_t)__shfl((int)off, (int)s, 64);
        const uint32_t oem = (uint32_t)__shfl((int)emitted, (int)s, 64);
        const float omx = __shfl(mx, (int)s, 64), omy = __shfl(my, (int)s, 64);
        const float oA = __shfl(A, (int)s, 64), oB = __shfl(B, (int)s, 64), oC = __shfl(C, (int)s, 64);
        const float oQ = __shfl(Q, (int)s, 64);
        const uint32_t row = rect_row(k, ow);
        const uint32_t col = k - row * ow;
        const uint32_t tx = (oxy & 0xffffu) + col, ty = (oxy >> 16) + row;
        const bool hit = live && cb_tile_hit(omx, omy, oA, oB, oC, oQ, (int)tx, (int)ty);
        const uint64_t hb = __ballot(hit);
        // lanes of this round that belong to the same Gaussian and come before this one
        const uint32_t seg0 = oexcl > j0 ? oexcl - j0 : 0u;                 // first lane of the owner's run
        const uint64_t below = (lane ? (~0ull >> (64 - lane)) : 0ull) & (~0ull << seg0);
        if (hit) {
            const size_t o = (size_t)ooff + oem + (uint32_t)__popcll(hb & below);
            if (o < P) {   // always true when tiles_touched came from k_preprocess with the same configuration
                keys[o] = ((uint64_t)(ty * (uint32_t)tiles_x + tx) << 32) | od;
                vals[o] = (uint32_t)(i - lane + s);
            }
        }
        // each owner adds the hits of its own run in this round
        const uint32_t a0 = excl > j0 ? excl - j0 : 0u;                      // run of this lane's Gaussian: [a0, a1)
        const uint32_t a1 = inc > j0 ? min(inc - j0, 64u) : 0u;
        if (a1 > a0) {
            const uint64_t mine = (a1 >= 64 ? ~0ull : ((1ull << a1) - 1ull)) & (~0ull << a0);
            emitted += (uint32_t)__popcll(hb & mine);
        }
    }
}

// ---- tile-bucketed ordering ----------------------------------------------------------------
// The order wanted is (tile, depth, Gaussian index): instead of one global sort on 45 live key bits, the
// pairs are (1) counted per tile, (2) placed into their tile's segment in arrival order, and (3) every
// tile's segment is sorted in LDS on the 64-bit word depth_bits << 32 | Gaussian index.  Those words are
// unique within a tile, so the result does not depend on the arrival order and equals what a stable global
// sort of index-ordered keys gives.  The per-tile ranges fall out of step (1).

// Steps (1) and (2) are launched as TILE_COPIES workgroups, each keeping its own counter per tile in LDS
// (so num_tiles * 4 bytes must fit there) and walking the same Gaussians in both steps; step (1) ends by
// writing its counters as one row of a [TILE_COPIES, num_tiles] table, which k_tile_layout turns into each
// workgroup's start within every tile's segment, and step (2) starts from that row.  Global atomics reach
// about 45 G/s on this chip whatever the contention; LDS atomics are an order of magnitude cheaper.
//
// First and last + 1 place of the pairs of band [t0, t0 + BAND_TILES) ({~0, 0}: there are none); lane l looks at tile t0 + l.
__device__ __forceinline__ uint2 band_bounds(const uint2* __restrict__ ranges, int t0, int num_tiles, uint32_t lane)
{
    static_assert(BAND_TILES == 64, "a tile for each lane");
    const uint2 r = t0 + (int)lane < num_tiles ? ranges[t0 + lane] : make_uint2(0u, 0u);
    const uint32_t above = wave_inclusive_max(r.y > r.x ? ~r.x : 0u), last = wave_inclusive_max(r.y > r.x ? r.y : 0u);
    return make_uint2(~(uint32_t)__builtin_amdgcn_readlane((int)above, 63), (uint32_t)__builtin_amdgcn_readlane((int)last, 63));
}

// Steps (1) and (2) walk the candidate tiles of 64 consecutive Gaussians per wavefront the way k_emit_pairs
// does.  SCATTER = false: count[tile] += 1 per pair.  SCATTER = true: slot = first[tile] + counter[tile]++
// (k_tile_layout has turned each copy's counter into that copy's start within the tile's segment, or those of a band into one),
// bucket[slot] = depth_bits << 32 | index.  In this mode `P` is the number of words the buffers hold: nothing is written at or
// beyond it (the kernel may be enqueued before the host has seen the real totals).
//
// Step (1) also hands every Gaussian the place of its backward records (one per tile of its rectangle), counted from the
// first record of its workgroup: inside a workgroup the wavefronts, their rounds and the 64 Gaussians of a round follow each
// other.  k_tile_layout adds what the workgroups before have (wg_totals).  The places are disjoint, each Gaussian's are
// contiguous and so are those of 64 consecutive Gaussians, which is all their users need -- no prefix sum over the Gaussians.
// (Reserved with adds on global counters, which take about 10 ns on one address, the 256 workgroups waited for one another.  Without
// them and with the Gaussians dealt out evenly, counting and k_tile_layout together, before and after: 21.2 and 18.4 us at 100k
// Gaussians, 44.8 and 41.2 at 500k, 38.3 and 30.5 at 300k with the Compact Box, 105.8 and 108.5 at 3 M, where placement gains more.)
// The sums of tiles_touched are there for the host, which compares them with the number of pairs counted per tile.
struct RecAlloc {
    const uint32_t* tiles_touched;   // [n]
    uint32_t* rec_offsets;           // [n] out: first record of each Gaussian
    uint32_t* rec_counts;            // [n] out (may be null): records of each Gaussian = area of its rectangle
    uint64_t* wg_totals;             // [2][TILE_COPIES] out: each workgroup's records, and its sum of tiles_touched
};

// BANDS (placement): the words go into their band of tiles instead, and `places` gets the first place of every tile and the bands'
// bounds (see k_band_split).
template <bool CB, bool SCATTER, bool BANDS>
__global__ __launch_bounds__(TILE_PAIR_THREADS) void k_tile_pairs(int64_t n, const ushort4* __restrict__ rect,
                                                    const float* __restrict__ depth,
                                                    const float2* __restrict__ mean2d,
                                                    const float4* __restrict__ conic_opacity, CfgDev cfg, int tiles_x,
                                                    int num_tiles, uint32_t* __restrict__ tile_counter,
                                                    const uint2* __restrict__ ranges, uint32_t P,
                                                    uint64_t* __restrict__ bucket, RecAlloc ra, BandPlaces places)
{
    static_assert(SCATTER || !BANDS, "a variant of the placement");
    extern __shared__ uint32_t s_tile[];   // this workgroup's counter per tile (BANDS: per band)
    uint32_t* const my_row = tile_counter + (size_t)blockIdx.x * num_tiles;
    // placement: the counter starts at the absolute position of this workgroup's first pair of the tile
    const uint32_t lane = lane_id();
    if (BANDS) {
        for (int t0 = (int)(threadIdx.x & ~63u); t0 < num_tiles; t0 += TILE_PAIR_THREADS) {
            const uint2 bounds = band_bounds(ranges, t0, num_tiles, lane);
            if (lane == 0) s_tile[t0 / BAND_TILES] = bounds.x + my_row[t0];
            if (lane == 0 && blockIdx.x == 0) places.band[t0 / BAND_TILES] = bounds;
        }
        for (int t = (int)(blockIdx.x * TILE_PAIR_THREADS + threadIdx.x); t < num_tiles; t += (int)gridDim.x * TILE_PAIR_THREADS)
            places.tile[t] = ranges[t].x;
    } else {
        for (int t = threadIdx.x; t < num_tiles; t += TILE_PAIR_THREADS) s_tile[t] = SCATTER ? ranges[t].x + my_row[t] : 0u;
    }
    __syncthreads();
    __shared__ uint32_t s_mark[TILE_PAIR_THREADS / 64][128];
    uint32_t* const mark = s_mark[threadIdx.x >> 6];   // this wavefront's own
    // Wavefront w of workgroup b takes the 64 Gaussians from 64 (w gridDim + b) on in its first round, so that every workgroup has as
    // much to do as the next, also where there are fewer Gaussians than threads.
    const int64_t i_first = ((int64_t)(threadIdx.x >> 6) * gridDim.x + blockIdx.x) * 64 + lane;
    uint32_t rec_next = 0;   // (counting) where the records of this wavefront's next round start
    if (!SCATTER) {
        __shared__ uint32_t s_wave_recs[TILE_PAIR_THREADS / 64];
        __shared__ uint32_t s_tt[TILE_PAIR_THREADS / 64];
        uint32_t recs = 0, tt = 0;
        // (four rounds' loads are requested together: with one wavefront's worth of loads in flight per round the
        // loop would take one memory latency per round)
        const int64_t stride = (int64_t)gridDim.x * TILE_PAIR_THREADS;
        for (int64_t i = i_first; i < n; i += 4 * stride) {
            ushort4 r[4];
            uint32_t t4[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const bool in = i + q * stride < n;
                r[q] = in ? rect[i + q * stride] : make_ushort4(0, 0, 0, 0);
                t4[q] = in ? ra.tiles_touched[i + q * stride] : 0u;
            }
#pragma unroll
            for (int q = 0; q < 4; q++) {
                recs += (r[q].z > r[q].x ? (uint32_t)(r[q].z - r[q].x) : 0u) * (r[q].w > r[q].y ? (uint32_t)(r[q].w - r[q].y) : 0u);
                tt += t4[q];
            }
        }
        recs = wave_inclusive_scan(recs);
        tt = wave_inclusive_scan(tt);
        if (lane == 63) { s_wave_recs[threadIdx.x >> 6] = recs; s_tt[threadIdx.x >> 6] = tt; }
        __syncthreads();
        if (threadIdx.x == 0) {
            uint64_t all = 0, all_tt = 0;
            for (int w = 0; w < TILE_PAIR_THREADS / 64; w++) { all += s_wave_recs[w]; all_tt += s_tt[w]; }
            ra.wg_totals[blockIdx.x] = all;
            ra.wg_totals[TILE_COPIES + blockIdx.x] = all_tt;
        }
        // (32 bits: the host rejects a call whose records do not fit them)
        for (int w = 0; w < (int)(threadIdx.x >> 6); w++) rec_next += s_wave_recs[w];
    }
    // (every wavefront of the workgroup walks its own 64 Gaussians per round; no barrier inside the rounds)
    // (the next round's rectangle and depth are requested before this round's candidates are walked)
    const int64_t round_stride = (int64_t)gridDim.x * TILE_PAIR_THREADS;
    ushort4 r_next = i_first < n ? rect[i_first] : make_ushort4(0, 0, 0, 0);
    uint32_t dbits_next = (SCATTER && i_first < n) ? __float_as_uint(depth[i_first]) : 0u;
    for (int64_t i = i_first; i - lane < n; i += round_stride) {
        const bool valid = i < n;
        const ushort4 r = r_next;
        const uint32_t w = r.z > r.x ? (uint32_t)(r.z - r.x) : 0u, h = r.w > r.y ? (uint32_t)(r.w - r.y) : 0u;
        const uint32_t cnt = w * h;
        const uint32_t dbits = cnt ? dbits_next : 0u;
        {
            const int64_t i2 = i + round_stride;
            const bool in = i2 < n;
            r_next = in ? rect[i2] : make_ushort4(0, 0, 0, 0);
            if (SCATTER) dbits_next = in ? __float_as_uint(depth[i2]) : 0u;
        }
        float mx = 0.f, my = 0.f, A = 1.f, B = 0.f, C = 1.f, Q = 0.f;
        if (CB && cnt) {
            const float2 m = mean2d[i];
            const float4 co = conic_opacity[i];
            mx = m.x; my = m.y; A = co.x; B = co.y; C = co.z;
            Q = cb_threshold(co.w, cfg);
        }
        const uint32_t inc = wave_inclusive_scan(cnt);
        const uint32_t excl = inc - cnt;
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        const uint32_t rect_xy = (uint32_t)r.x | (uint32_t)r.y << 16;
        if (!SCATTER) {
            if (valid) {
                ra.rec_offsets[i] = rec_next + excl;
                if (ra.rec_counts) ra.rec_counts[i] = cnt;
            }
            rec_next += total;
        }
        uint32_t carry = 0;   // 1 + the lane whose rectangle holds candidate j0 - 1 (uniform)
        // Candidates j0 + 64 q + lane, whose owners are lanes owners[q].  Two windows of 64 at a time where there are two: a window is a
        // chain of some ten LDS operations (owner, its rectangle, the tile's counter) with four wavefronts on a SIMD to hide it.
        // Counting with k_tile_layout, and placement with the sorts, one window at a time and two, in us: 155.6 and 147.2, 610 and
        // 602 at 27 M pairs; 109.4 and 107.2, 236 and 234 at 10 M; 41.5 and 40.3, 70.6 and 68.6 at 500k Gaussians.
        auto candidates = [&](uint32_t j0, auto& owners) {
            constexpr int W = sizeof(owners) / sizeof(owners[0]);
            uint32_t tile[W], od[W];
            bool hit[W];
#pragma unroll
            for (int q = 0; q < W; q++) {
                const uint32_t j1 = j0 + 64 * q + lane, j = min(j1, total - 1), s = owners[q];
                const uint32_t k = j - (uint32_t)__shfl((int)excl, (int)s, 64);
                const uint32_t ow = (uint32_t)__shfl((int)w, (int)s, 64);
                const uint32_t oxy = (uint32_t)__shfl((int)rect_xy, (int)s, 64);
                const uint32_t row = rect_row(k, ow);
                const uint32_t col = k - row * ow;
                const uint32_t tx = (oxy & 0xffffu) + col, ty = (oxy >> 16) + row;
                hit[q] = j1 < total;
                if (CB) {
                    const float omx = __shfl(mx, (int)s, 64), omy = __shfl(my, (int)s, 64);
                    const float oA = __shfl(A, (int)s, 64), oB = __shfl(B, (int)s, 64), oC = __shfl(C, (int)s, 64);
                    const float oQ = __shfl(Q, (int)s, 64);
                    hit[q] = hit[q] && cb_tile_hit(omx, omy, oA, oB, oC, oQ, (int)tx, (int)ty);
                }
                tile[q] = ty * (uint32_t)tiles_x + tx;
                hit[q] = hit[q] && tile[q] < (uint32_t)num_tiles;   // (always true for a rect made for this camera)
                if (SCATTER) od[q] = (uint32_t)__shfl((int)dbits, (int)s, 64);
            }
            if (!SCATTER) {
#pragma unroll
                for (int q = 0; q < W; q++)
                    if (hit[q]) atomicAdd(&s_tile[tile[q]], 1u);
                return;
            }
            uint32_t slot[W];
#pragma unroll
            for (int q = 0; q < W; q++) slot[q] = hit[q] ? atomicAdd(&s_tile[BANDS ? tile[q] / BAND_TILES : tile[q]], 1u) : P;
#pragma unroll
            for (int q = 0; q < W; q++) {
                if (hit[q]) {
                    const uint32_t of = BANDS ? tile[q] % BAND_TILES << BAND_SHIFT : 0u;
                    if (slot[q] < P) bucket[slot[q]] = ((uint64_t)od[q] << 32) | of | (uint32_t)(i - lane + owners[q]);
                }
            }
        };
        for (uint32_t j0 = 0; j0 < total; j0 += 128) {
            if (total - j0 > 64) {
                uint32_t owners[2];
                wave_run_owner2(mark, cnt, excl, j0, carry, owners);
                candidates(j0, owners);
            } else {
                uint32_t owners[1] = {wave_run_owner(mark, cnt, excl, j0, carry)};
                candidates(j0, owners);
            }
        }
    }
    if (!SCATTER) {
        __syncthreads();
        for (int t = threadIdx.x; t < num_tiles; t += TILE_PAIR_THREADS) my_row[t] = s_tile[t];
    }
}

// Between steps (1) and (2), in one launch:
//
// The first `sum_blocks` workgroups, per tile: its count summed over the workgroups' rows; each row's counter is replaced
// by the number of the tile's pairs in the rows before it (where that workgroup's pairs start within the tile's
// segment).  A workgroup takes 64 tiles; its wavefront g takes rows [16 g, 16 g + 16) of each.  Where the placement goes by
// bands, these 64 tiles are one, and only the counter of its first tile is replaced, by the number of the band's pairs in the rows before.
//
// Whichever of them is done last then turns the tile totals into ranges [first, last), by an exclusive scan in rounds of 1024
// tiles, a thread each; totals[2] = sum, totals[3] = longest list; and the order in which
// the render kernels take the tiles (longest list first, bucketed by length / 8, as k_tile_order).
//
// The other workgroups pack the projected splats into the records the render kernels gather (SPLAT_REC); the first of them also
// stores totals[0..1], the sums of the counting workgroups' totals (wg_totals).  The placement
// kernel did this on the way, with one workgroup per compute unit; here it has the whole chip and hides the chain of the
// two steps above, and the records no longer drive the placement's half-filled lines out of the L2.
// Placement, sums and scan together, before and after: 222 and 185 us at 3 M Gaussians / 10 M pairs, 18.3 and 16.8 at 4k.
// They also complete the record places of all Gaussians (4 bytes read and written for each): this launch went from 20.7 to 21.8 us at
// 500k Gaussians and from 64 to 69 at 3 M with it, the counting kernel from 18.1 to 12.6 and from 43.5 to 39.
//
// Up to 500k Gaussians the chain of the first two is what the launch takes: the rows' loads (1.5 us), the totals' way past the L2 and
// the count of arrivals (1.5), the totals' loads (0.6 to 0.9), sums and maximum (1), places and stores (0.5 to 4).  So a round is 1024
// neighbouring tiles, a thread each (whole lines), the store that is waited for comes ahead of the table's, and the maximum goes through
// the wavefronts: all threads on one LDS address took 2 to 3.5 us.  Counting and this launch, before and after, us: 14.8 and 12.4 at 4k
// Gaussians, 18.5 and 15.5 at 100k, 27.5 and 23.5 at 300k, 36.0 and 30.7 at 500k.  (Two workgroups to a compute unit, at 64 registers:
// 5 % slower at 300k; nearly empty tiles counted a wavefront at a time: 3 to 11 % slower.)
constexpr int LAYOUT_THREADS = 1024;
constexpr int LAYOUT_WAVES = LAYOUT_THREADS / 64;
__global__ __launch_bounds__(LAYOUT_THREADS) void k_tile_layout(uint32_t* __restrict__ count, int num_tiles, int sum_blocks,
                                                                uint32_t* __restrict__ tile_total, uint2* __restrict__ ranges,
                                                                uint32_t* __restrict__ order, uint64_t* __restrict__ totals,
                                                                unsigned long long* __restrict__ arrivals,
                                                                const uint64_t* __restrict__ wg_totals, int64_t n,
                                                                const ushort4* __restrict__ rect, const float2* __restrict__ mean2d,
                                                                const float4* __restrict__ conic_opacity, const float* __restrict__ rgb,
                                                                CfgDev cfg, uint32_t* __restrict__ rec_offsets,
                                                                float4* __restrict__ splats, int bands)
{
    if ((int)blockIdx.x >= sum_blocks) {
        const int64_t i = (int64_t)((int)blockIdx.x - sum_blocks) * LAYOUT_THREADS + threadIdx.x;
        // the records of the workgroups before the one that counted these 64 Gaussians (see k_tile_pairs)
        const uint32_t wg = (uint32_t)(i >> 6) % TILE_COPIES;
        uint32_t before = 0;
#pragma unroll
        for (uint32_t k = 0; k < TILE_COPIES; k += 64) before += k + lane_id() < wg ? (uint32_t)wg_totals[k + lane_id()] : 0u;
        before = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(before), 63);
        if ((int)blockIdx.x == sum_blocks && threadIdx.x < 64) {
            uint64_t recs = 0, tt = 0;
#pragma unroll
            for (uint32_t k = 0; k < TILE_COPIES; k += 64) { recs += wg_totals[k + lane_id()]; tt += wg_totals[TILE_COPIES + k + lane_id()]; }
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) { recs += shfl_xor_u64(recs, d); tt += shfl_xor_u64(tt, d); }
            // (the host looks at the totals while the kernel runs: past every cache)
            if (lane_id() == 0) {
                __hip_atomic_store(&totals[0], tt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                __hip_atomic_store(&totals[1], recs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
        if (i >= n) return;
        const uint32_t first_record = rec_offsets[i] + before;
        rec_offsets[i] = first_record;
        const ushort4 r = rect[i];
        if (r.z <= r.x || r.w <= r.y) return;   // (no pair names it)
        pack_splat(splats, i, mean2d[i], conic_opacity[i], rgb, first_record, r, cfg);
        return;
    }
    // Order of the workgroups' shares within a tile's segment: workgroups are handed to the 8 XCDs in turn, so
    // those with the same index mod 8 share an L2; putting their shares next to each other lets the 8-byte words
    // they scatter into a segment fill whole lines in one L2 before they are written back.
    auto row_at = [](int pos) { return (pos % (TILE_COPIES / 8)) * 8 + pos / (TILE_COPIES / 8); };
    constexpr int PER_WAVE = TILE_COPIES / LAYOUT_WAVES;
    __shared__ uint32_t gsum[LAYOUT_WAVES][64];
    __shared__ uint32_t bsum[TILE_COPIES];
    __shared__ bool s_last;
    {
        const int g = threadIdx.x >> 6, lane = threadIdx.x & 63;
        const int t = blockIdx.x * 64 + lane;
        uint32_t part[PER_WAVE];
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < PER_WAVE; k++) {
            part[k] = t < num_tiles ? count[(size_t)row_at(g * PER_WAVE + k) * num_tiles + t] : 0u;
            sum += part[k];
        }
        gsum[g][lane] = sum;
        if (bands) {
            // the rows' sums over the whole band, by their position in the order of shares
#pragma unroll
            for (int k = 0; k < PER_WAVE; k++) {
                const uint32_t s = wave_inclusive_scan(part[k]);
                if (lane == 63) bsum[g * PER_WAVE + k] = s;
            }
        }
        __syncthreads();
        uint32_t run = 0, all = 0;
#pragma unroll
        for (int q = 0; q < LAYOUT_WAVES; q++) {
            run += q < g ? gsum[q][lane] : 0u;
            all += gsum[q][lane];
        }
        if (g == 0) {
            // (ahead of the table's stores, which nothing in this launch waits for)
            // (another compute die may read these: they go past this one's L2, and have arrived before the workgroup counts
            // as done.  A release fence would do the same, and write the whole L2 back each time: the launch took 15 us instead
            // of 11 at 100k Gaussians.  The reader needs no acquire fence for its part: it loads them with agent-scope atomics,
            // which do not look for them in its own L2 either, and only after the branch on the count.  This is the cache policy of
            // this chip's agent-scope accesses, not an ordering of the language's memory model.)
            if (t < num_tiles) __hip_atomic_store(&tile_total[t], all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            if (lane == 0) s_last = atomicAdd(arrivals, 1ull) + 1 == (unsigned long long)sum_blocks;
        }
        if (bands) {
            // only where a workgroup's pairs start within the band is wanted, in the place of its first tile's counter
            uint32_t before = 0;
#pragma unroll
            for (int k = 0; k < TILE_COPIES; k += 64) before += k + lane < g * PER_WAVE ? bsum[k + lane] : 0u;
            before = (uint32_t)__builtin_amdgcn_readlane((int)wave_inclusive_scan(before), 63);
            const uint32_t own = lane < PER_WAVE ? bsum[g * PER_WAVE + lane] : 0u;
            const uint32_t start = before + wave_inclusive_scan(own) - own;
            if (lane < PER_WAVE) count[(size_t)row_at(g * PER_WAVE + lane) * num_tiles + blockIdx.x * BAND_TILES] = start;
        } else if (t < num_tiles) {
#pragma unroll
            for (int k = 0; k < PER_WAVE; k++) {
                count[(size_t)row_at(g * PER_WAVE + k) * num_tiles + t] = run;
                run += part[k];
            }
        }
    }
    __syncthreads();
    if (!s_last) return;

    // Round q of thread t: tile 1024 q + t.
    constexpr int NB = ORDER_BUCKETS;
    constexpr int PER_MAX = (TILE_LDS_MAX_TILES + LAYOUT_THREADS - 1) / LAYOUT_THREADS;   // this path is only taken up to that many tiles
    static_assert(PER_MAX * LAYOUT_WAVES <= 256 && NB == 512, "four of the sums, eight of the buckets for a lane");
    __shared__ __align__(16) uint32_t wsum[256];   // pairs of each round's wavefronts
    __shared__ uint32_t wmax[LAYOUT_WAVES];
    __shared__ __align__(16) uint32_t cnt[NB];
    const int t = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
    const int per = (num_tiles + LAYOUT_THREADS - 1) / LAYOUT_THREADS;
    auto bucket = [](uint32_t len) { return (int)(NB - 1 - min(len / ORDER_STEP, (uint32_t)NB - 1)); };
    uint32_t c[PER_MAX], inc[PER_MAX];   // this thread's tile totals, and those of its wavefront's tiles up to them
#pragma unroll
    for (int q = 0; q < PER_MAX; q++)
        c[q] = q * LAYOUT_THREADS + t < num_tiles ? __hip_atomic_load(&tile_total[q * LAYOUT_THREADS + t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    if (t < NB) cnt[t] = 0u;
    if (t >= per * LAYOUT_WAVES && t < 256) wsum[t] = 0u;
    __syncthreads();
    uint32_t most = 0;
#pragma unroll
    for (int q = 0; q < PER_MAX; q++) {
        if (q >= per) continue;
        inc[q] = wave_inclusive_scan(c[q]);
        if (lane == 63) wsum[q * LAYOUT_WAVES + wave] = inc[q];
        most = max(most, c[q]);
        if (q * LAYOUT_THREADS + t < num_tiles) atomicAdd(&cnt[bucket(c[q])], 1u);
    }
    // (one LDS address for 1024 threads' maximum took 2 us of the launch)
    most = wave_inclusive_max(most);
    if (lane == 63) wmax[wave] = most;
    __syncthreads();
    // tile order: exclusive prefix over the 512 length buckets by one wavefront, then a counting placement
    if (wave == 0) {
        uint4* const mine = reinterpret_cast<uint4*>(cnt) + 2 * lane;
        const uint4 a = mine[0], b = mine[1];
        const uint32_t sum = a.x + a.y + a.z + a.w + b.x + b.y + b.z + b.w;
        const uint32_t pre = wave_inclusive_scan(sum) - sum, mid = pre + a.x + a.y + a.z + a.w;
        mine[0] = make_uint4(pre, pre + a.x, pre + a.x + a.y, pre + a.x + a.y + a.z);
        mine[1] = make_uint4(mid, mid + b.x, mid + b.x + b.y, mid + b.x + b.y + b.z);
    }
    // the pairs before this wavefront's tiles of each round: in lane 4 q + wave / 4
    const uint4 w4 = reinterpret_cast<const uint4*>(wsum)[lane];
    const uint32_t upto = wave_inclusive_scan(w4.x + w4.y + w4.z + w4.w);
    const int w3 = wave & 3;
    const uint32_t start = upto - (w4.w + (w3 < 3 ? w4.z : 0u) + (w3 < 2 ? w4.y : 0u) + (w3 < 1 ? w4.x : 0u));
    if (t == LAYOUT_THREADS - 1) {
        // totals: sum of tiles_touched, backward records, pairs counted per tile, longest list; the arrivals start the
        // next call at zero
#pragma unroll
        for (int w = 0; w < LAYOUT_WAVES; w++) most = max(most, wmax[w]);
        __hip_atomic_store(&totals[2], (uint64_t)upto, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        __hip_atomic_store(&totals[3], (uint64_t)most, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        *arrivals = 0ull;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < PER_MAX; q++) {
        if (q >= per) continue;
        const int tile = q * LAYOUT_THREADS + t;
        const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)start, 4 * q + wave / 4) + inc[q] - c[q];
        if (tile < num_tiles) {
            ranges[tile] = c[q] ? make_uint2(first, first + c[q]) : make_uint2(0u, 0u);
            order[atomicAdd(&cnt[bucket(c[q])], 1u)] = (uint32_t)tile;
        }
    }
}

// Step (2), second half, where the first one has placed the words by bands: a workgroup takes SPLIT_WORDS of a band's words at a time,
// orders them by tile in LDS, reserves a place for each tile's share and writes the shares, as words without their tile.
// Memory traffic bounds the placement at millions of pairs.  With a share of some five words for each workgroup and tile, the 32
// workgroups of a compute die keep a half-filled line open for each of 8160 tiles, 33 MB where its L2 holds four: 345 MB
// were written for 80 at 10 M pairs, 849 for 219 at 27 M.  A band's share is 64 times as long and all open lines fit; the second
// step reads and writes every word once more, in whole lines (a tile's share of 4096 words is 64 of them).
// Kernel durations in one step and in two, us: 193 and 68 + 39 at 12 M pairs (3 M Gaussians, 1920x1080), 486 and 155 + 142 at 36 M.
// Taking 2048 words with 256 threads, 4096 with 1024 or 8192 with 1024: order and placement 158, 161, 162 instead of 157 at 10 M
// pairs, 446, 434, 433 instead of 432 at 27 M.
// The chunks of all bands are dealt out as one row, so that bands of any lengths keep the chip busy.  With as many workgroups for each
// band as for the next, those of the longest one went on alone; before and after, us: 5 M pairs with nine tenths of them in 6 of 128
// bands 42.1 and 21.8, half in 4 bands 38.3 and 20.8, 10 M pairs with half in 6 bands 39.7 and 35.3; even bands 40.9 and 38.8 at 12 M
// pairs, 153 and 142 at 36 M, 9.8 and 10.4 at 2.5 M.
constexpr int SPLIT_THREADS = 512;
constexpr int SPLIT_WORDS = 4096;
__global__ __launch_bounds__(SPLIT_THREADS) void k_band_split(int num_tiles, uint32_t limit, BandPlaces places,
                                                              const uint64_t* __restrict__ by_band, uint64_t* __restrict__ by_tile)
{
    constexpr int PER = SPLIT_WORDS / SPLIT_THREADS;
    constexpr int BANDS = (TILE_LDS_MAX_TILES + 64 * BAND_TILES - 1) / (64 * BAND_TILES);   // of a lane: BANDS lane ... BANDS lane + BANDS - 1
    __shared__ uint64_t k[SPLIT_WORDS];
    __shared__ uint32_t cnt[BAND_TILES], first[BAND_TILES], to[BAND_TILES];   // words of each tile, the first one's place in k; from there to by_tile
    const int t = threadIdx.x, lane = (int)lane_id();
    // (every wavefront for itself)
    uint32_t begin[BANDS], end[BANDS], chunks[BANDS], mine = 0;
#pragma unroll
    for (int q = 0; q < BANDS; q++) {
        const int b = BANDS * lane + q;
        const uint2 bounds = b * BAND_TILES < num_tiles ? places.band[b] : make_uint2(~0u, 0u);
        begin[q] = bounds.x;
        end[q] = min(bounds.y, limit);   // (nothing was placed beyond the limit)
        chunks[q] = begin[q] < end[q] ? (end[q] - begin[q] - 1) / SPLIT_WORDS + 1 : 0u;
        mine += chunks[q];
    }
    const uint32_t upto = wave_inclusive_scan(mine);
    const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
    for (uint32_t c = blockIdx.x; c < all; c += gridDim.x) {
        uint32_t before = upto - mine, p = 0, last = 0;
        int band = -1;
#pragma unroll
        for (int q = 0; q < BANDS; q++) {
            if (c >= before && c - before < chunks[q]) {
                band = BANDS * lane + q;
                p = begin[q] + (c - before) * SPLIT_WORDS;
                last = end[q];
            }
            before += chunks[q];
        }
        const int owner = __builtin_ctzll(__ballot(band >= 0));   // (c < all: there is one)
        p = (uint32_t)__builtin_amdgcn_readlane((int)p, owner);
        last = (uint32_t)__builtin_amdgcn_readlane((int)last, owner);
        const int t0 = __builtin_amdgcn_readlane(band, owner) * BAND_TILES;
        const uint64_t* const src = by_band + p;
        const int m = (int)min((uint32_t)SPLIT_WORDS, last - p);
        uint64_t w[PER];
#pragma unroll
        for (int u = 0; u < PER; u++) w[u] = t + u * SPLIT_THREADS < m ? src[t + u * SPLIT_THREADS] : 0ull;
        if (t < BAND_TILES) cnt[t] = 0u;
        __syncthreads();
        uint32_t rank[PER];
#pragma unroll
        for (int u = 0; u < PER; u++)
            if (t + u * SPLIT_THREADS < m) rank[u] = atomicAdd(&cnt[(uint32_t)w[u] >> BAND_SHIFT], 1u);
        __syncthreads();
        if (t < BAND_TILES) {
            const uint32_t c = cnt[t], at = wave_inclusive_scan(c) - c;
            first[t] = at;
            to[t] = (c != 0u && t0 + t < num_tiles ? atomicAdd(&places.tile[t0 + t], c) : limit) - at;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; u++)
            if (t + u * SPLIT_THREADS < m) k[first[(uint32_t)w[u] >> BAND_SHIFT] + rank[u]] = w[u];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < PER; u++) {
            const uint32_t i = (uint32_t)(t + u * SPLIT_THREADS);
            if ((int)i < m) {
                const uint64_t word = k[i];
                const uint32_t place = to[(uint32_t)word >> BAND_SHIFT] + i;
                if (place < limit) by_tile[place] = word & ~((uint64_t)(BAND_TILES - 1) << BAND_SHIFT);
            }
        }
        __syncthreads();
    }
}

// Step (3): one workgroup sorts one tile's segment in LDS on the 64-bit words and writes the final keys
// tile << 32 | depth_bits and the Gaussian indices.
//
// First the network that the few lists take which the buckets below do not suit: bitonic, on the words padded to a power
// of two with all-ones words.  The steps at distances 4, 2, 1 of a stage -- which stay inside aligned groups of 8 words
// -- are done in registers: a thread loads a group, runs the three steps (all of the stages 2, 4, 8 at the start) and
// stores it back; the steps at larger distances are taken three at a time as well, on groups of 8 words the right
// distance apart.
__device__ __forceinline__ void cmpx(uint64_t& a, uint64_t& b, bool up)
{
    const bool sw = (a > b) == up;
    const uint64_t x = sw ? b : a, y = sw ? a : b;
    a = x;
    b = y;
}

// GG words at distance 2^a from each other through registers: the GG/2 .. 1 steps of stage k2 at distances
// 2^a GG/2 .. 2^a.  The words of a group agree in every index bit outside [a, a + log2 GG), the stage's bit
// among them, so one direction serves the group.  Ends with a workgroup barrier.
template <int GG, int THREADS>
__device__ __forceinline__ void network_strided(uint64_t* k, int N, int a, int k2)
{
    constexpr int LGG = GG == 2 ? 1 : GG == 4 ? 2 : 3;
    for (int g = threadIdx.x; g < N / GG; g += THREADS) {
        const int e0 = ((g >> a) << (a + LGG)) | (g & ((1 << a) - 1));
        const bool up = (e0 & k2) == 0;
        uint64_t v[GG];
#pragma unroll
        for (int q = 0; q < GG; q++) v[q] = k[e0 + (q << a)];
#pragma unroll
        for (int jj = GG / 2; jj > 0; jj >>= 1)
#pragma unroll
            for (int q = 0; q < GG; q++)
                if ((q & jj) == 0) cmpx(v[q], v[q | jj], up);
#pragma unroll
        for (int q = 0; q < GG; q++) k[e0 + (q << a)] = v[q];
    }
    __syncthreads();
}

// k[0, n) <- the words in order (word(u) is word t + u THREADS of thread t); k holds N words, N >= 16 a power of two, N >= n.
template <int THREADS, int PER, typename Word>
__device__ __forceinline__ void network_sort(uint64_t* k, int N, int n, Word word)
{
#pragma unroll
    for (int u = 0; u < PER; u++) {
        const int i = (int)threadIdx.x + u * THREADS;
        if (i < N) k[i] = i < n ? word(u) : ~0ull;
    }
    __syncthreads();
    for (int g = threadIdx.x; g < N / 8; g += THREADS) {   // the complete stages 2, 4, 8
        uint64_t v[8];
#pragma unroll
        for (int q = 0; q < 8; q++) v[q] = k[8 * g + q];
#pragma unroll
        for (int k2 = 2; k2 <= 8; k2 <<= 1)
#pragma unroll
            for (int j = k2 >> 1; j > 0; j >>= 1)
#pragma unroll
                for (int e = 0; e < 8; e++)
                    if ((e & j) == 0) cmpx(v[e], v[e | j], k2 == 8 ? (g & 1) == 0 : (e & k2) == 0);
#pragma unroll
        for (int q = 0; q < 8; q++) k[8 * g + q] = v[q];
    }
    __syncthreads();
    for (int k2 = 16, m = 4; k2 <= N; k2 <<= 1, m++) {   // m = log2 k2: the stage has steps 2^(m-1) .. 1
        int top = m;
        if (m % 3 == 1) network_strided<2, THREADS>(k, N, top - 1, k2);
        if (m % 3 == 2) network_strided<4, THREADS>(k, N, top - 2, k2);
        top -= m % 3;
        for (; top > 0; top -= 3) network_strided<8, THREADS>(k, N, top - 3, k2);
    }
}

// A list is ordered by spreading it over about as many buckets as it has words, monotonically in the depth bits, and
// ranking every word among the few words of its own bucket: a constant number of trips through LDS and a handful of
// comparisons per word, where the network needs log2(N)^2 / 2 of them per word (91 at 8 192).  The bucket function is
// linear between the list's smallest and largest depth for short lists; longer ones (depths that cluster, an outlier
// that stretches the range) go through a histogram of COARSE equal parts first and then interpolate its running sum,
// which gives every word a bucket share whatever the distribution between the parts.  A list with more than
// BUCKET_LIMIT words in one bucket (hundreds of equal depths) is left to the network above.
// What is left is the segments' loads and stores (20 bytes per pair) and, for the shortest lists, the chain of six
// barriers.  Against the network for everything: 27 M pairs (lists of 3 350 on average) 830 -> 259 us in four launches
// (<= 2 048, <= 4 096, <= 8 192, <= 16 384 words),
// 10 M pairs 177 -> 75 us, 300k Gaussians at 1332x876 55 -> 23 us, 100k at 980x545 16.4 -> 8.4 us.
constexpr int COARSE = 256;
constexpr int BUCKET_LIMIT = 256;

template <int CAP, int THREADS, int NB>
struct SortMem {
    uint64_t k[CAP + NB / 2 + 1];   // the words in bucket order, and behind them the buckets' counts, then first places ([NB + 1])
    float2 part[COARSE];            // words before a part, words in it
    uint32_t red[3][THREADS / 64];
};

// One workgroup orders a tile's n <= CAP words: word t + u THREADS is w[u] of thread t (anything beyond the n-th), and again(u) once more
// for the few lists that the network takes.  place() is called by all threads, between barriers, and says where the tile's segment
// starts, or (not SURE) ~0u to write nothing.
template <int CAP, int THREADS, int NB, bool SURE, typename Again, typename Place>
__device__ __forceinline__ void sort_list(SortMem<CAP, THREADS, NB>& mem, const uint64_t (&w)[CAP / THREADS], int n, uint32_t tile, Again again,
                                          Place place, uint64_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out)
{
    constexpr int PER = CAP / THREADS, WAVES = THREADS / 64, NBT = NB / THREADS;
    static_assert(CAP % THREADS == 0 && NB % THREADS == 0 && THREADS >= COARSE, "whole words and buckets per thread");
    uint64_t* const k = mem.k;
    uint32_t* const start = reinterpret_cast<uint32_t*>(k + CAP);
    float2* const part = mem.part;
    uint32_t (*const red)[WAVES] = mem.red;
    const int t = threadIdx.x, wave = t >> 6;
    uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
    for (int u = 0; u < PER; u++) {
        if (t + u * THREADS < n) {
            const uint32_t d = (uint32_t)(w[u] >> 32);
            lo = min(lo, d);
            hi = max(hi, d);
        }
    }
    const bool two_level = n > 2 * COARSE;
    uint32_t* const coarse = start;   // (the parts' counters sit where the buckets' will)
    if (two_level) {
        if (t < COARSE) coarse[t] = 0u;
    } else {
#pragma unroll
        for (int q = 0; q < NBT; q++) start[t + q * THREADS] = 0u;
    }
    const uint32_t nlo = wave_inclusive_max(~lo);   // (zero is the neutral element of this maximum)
    hi = wave_inclusive_max(hi);
    if ((t & 63) == 63) { red[0][wave] = nlo; red[1][wave] = hi; }
    __syncthreads();
    uint32_t all_nlo = 0u, all_hi = 0u;
#pragma unroll
    for (int q = 0; q < WAVES; q++) { all_nlo = max(all_nlo, red[0][q]); all_hi = max(all_hi, red[1][q]); }
    const uint32_t first = ~all_nlo;
    const float range = (float)(all_hi - first);
    // every step (conversion, product, sum of exactly representable counts, truncation) is monotone in the depth bits
    const float scale = range > 0.f ? (two_level ? (float)COARSE : (float)NB) / range : 0.f;
    const float per_word = (float)NB / (float)n;
    if (two_level) {
#pragma unroll
        for (int u = 0; u < PER; u++) {
            if (t + u * THREADS < n) {
                const float x = (float)((uint32_t)(w[u] >> 32) - first) * scale;
                atomicAdd(&coarse[min((uint32_t)x, (uint32_t)COARSE - 1u)], 1u);
            }
        }
        __syncthreads();
        uint32_t c = 0, inc = 0;
        if (t < COARSE) {
            c = coarse[t];
            inc = wave_inclusive_scan(c);
            if ((t & 63) == 63) red[2][wave] = inc;
        }
        __syncthreads();
        if (t < COARSE) {
            uint32_t before = inc - c;
            for (int q = 0; q < wave; q++) before += red[2][q];
            part[t] = make_float2((float)before, (float)c);
        }
#pragma unroll
        for (int q = 0; q < NBT; q++) start[t + q * THREADS] = 0u;
        __syncthreads();
    }
    auto bucket_of = [&](uint64_t word) {
        float x = (float)((uint32_t)(word >> 32) - first) * scale;
        if (two_level) {
            const uint32_t c = min((uint32_t)x, (uint32_t)COARSE - 1u);
            const float2 p = part[c];
            x = (p.x + fminf(x - (float)c, 1.0f) * p.y) * per_word;
        }
        return min((uint32_t)x, (uint32_t)NB - 1u);
    };
    uint32_t at[PER];   // a word's bucket and its place of arrival in it (each below 65 536)
#pragma unroll
    for (int u = 0; u < PER; u++) {
        if (t + u * THREADS < n) {
            const uint32_t b = bucket_of(w[u]);
            at[u] = b << 16 | atomicAdd(&start[b], 1u);
        }
    }
    __syncthreads();
    {
        // thread t turns the counts of buckets [t NBT, t NBT + NBT) into first places
        uint32_t c[NBT], sum = 0, most = 0;
#pragma unroll
        for (int q = 0; q < NBT; q++) { c[q] = start[t * NBT + q]; sum += c[q]; most = max(most, c[q]); }
        const uint32_t inc = wave_inclusive_scan(sum);
        most = wave_inclusive_max(most);
        if ((t & 63) == 63) { red[0][wave] = inc; red[1][wave] = most; }
        __syncthreads();
        uint32_t run = inc - sum;
        most = 0u;
#pragma unroll
        for (int q = 0; q < WAVES; q++) { run += q < wave ? red[0][q] : 0u; most = max(most, red[1][q]); }
        if (most > (uint32_t)BUCKET_LIMIT) {   // (uniform over the workgroup)
            int N = 16;
            while (N < n) N <<= 1;
            network_sort<THREADS, PER>(k, N, n, again);
            const uint32_t to = place();
            if (!SURE && to == ~0u) return;
            for (int i = t; i < n; i += THREADS) {
                keys_out[to + i] = ((uint64_t)tile << 32) | (k[i] >> 32);
                vals_out[to + i] = (uint32_t)k[i];
            }
            return;
        }
#pragma unroll
        for (int q = 0; q < NBT; q++) { start[t * NBT + q] = run; run += c[q]; }
        if (t == 0) start[NB] = (uint32_t)n;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; u++)
        if (t + u * THREADS < n) k[start[at[u] >> 16] + (at[u] & 0xffffu)] = w[u];
    __syncthreads();
    const uint32_t to = place();
    if (!SURE && to == ~0u) return;
    // (words are taken in bucket order now, so that neighbouring lanes write neighbouring places)
#pragma unroll
    for (int u = 0; u < PER; u++) {
        const int i = t + u * THREADS;
        if (i < n) {
            const uint64_t word = k[i];
            const uint32_t b = bucket_of(word);
            const uint32_t s = start[b], e = start[b + 1];
            uint32_t rank = s;
            if (e - s > 1u)
                for (uint32_t q = s; q < e; q++) rank += k[q] < word ? 1u : 0u;
            keys_out[to + rank] = ((uint64_t)tile << 32) | (word >> 32);
            vals_out[to + rank] = (uint32_t)word;
        }
    }
}

// Handles the tiles whose length is in (len_lo, CAP]; the others are left to another launch.
template <int CAP, int THREADS, int NB>
__global__ __launch_bounds__(THREADS, CAP == TILE_SORT_MAX ? 8 : 4) void k_tile_sort(const uint2* __restrict__ ranges,
                                                   const uint32_t* __restrict__ tile_order,
                                                   const uint64_t* __restrict__ bucket, int len_lo, uint32_t limit,
                                                   uint64_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out)
{
    __shared__ __align__(16) SortMem<CAP, THREADS, NB> mem;
    const uint32_t tile = tile_order[blockIdx.x];
    const uint2 r = ranges[tile];
    const int n = (int)(r.y - r.x);
    // (uniform over the workgroup; `limit` = the words the buffers hold: a segment that reaches beyond it is left alone)
    if (n <= len_lo || n > CAP || r.y > limit) return;
    uint64_t w[CAP / THREADS];
#pragma unroll
    for (int u = 0; u < CAP / THREADS; u++) {
        const int i = (int)threadIdx.x + u * THREADS;
        w[u] = i < n ? bucket[r.x + i] : 0ull;
    }
    sort_list<CAP, THREADS, NB, true>(mem, w, n, tile, [&](int u) { return bucket[r.x + threadIdx.x + u * THREADS]; }, [&] { return r.x; }, keys_out, vals_out);
}

// The whole ordering of a small frame in one launch, where the four of the general way take some 5 us each and have little to do.
//
// Workgroups [0, num_tiles), one for each tile: it looks at every Gaussian's rectangle itself, keeps those that hold the tile (and meet
// it, with the Compact Box), says how many they are, orders them in LDS, and writes them behind the pairs of the tiles before it once
// all of those have said theirs.  Workgroup num_tiles waits for all tiles and leaves their order and two totals.  The others, 256
// Gaussians each, sum the areas before theirs and pack records and record places; the last one leaves the other two totals.
// What the workgroups say to each other is in small_words.hpp: words with the call's number in them, past all caches, so that nothing has
// to be cleared or fenced.  A workgroup waits only for workgroups of lower numbers that wait for nothing before they speak, so the
// lowest silent one is always under way or next in line; and no wait is longer than SMALL_POLLS looks (a second, in which another
// stream's kernel may hold the place that the silent one is meant for).  After that the totals stay unset, or this workgroup's pairs and
// range are whole all the same; unset totals make the host order the frame with the general launches.
// A list longer than TILE_SORT_SMALL is left unordered in `bucket` for the launches that take longer ones.
// What bounds it are its chains: the rectangles' loads (n / 256 of a thread, 16 at a time), list and sort in LDS, and the wait.
// fs_bin_sort, back to back, in four launches and in this one, us: 4k at 128x128 19.6 -> 12, 3k at 509x337 20.5 -> 15.6, 9k at 400x300 20.1 -> 17.8,
// with splats of twelve tiles 24.8 -> 17.3; a new context's first render at 4k 147 -> 98.  Lists of up to 128 ordered by comparing each word
// with all others instead of the sort: no difference (within 2 %).
constexpr int SMALL_PER = 16;          // rectangles a thread has in flight
constexpr int SMALL_POLLS = 1 << 20;
struct SmallFrame {
    int64_t n;
    const ushort4* rect;
    const float* depth;
    const float2* mean2d;
    const float4* conic_opacity;
    const float* rgb;
    const uint32_t* tiles_touched;
    int tiles_x, num_tiles;
    uint32_t limit;                  // words the buffers hold
    uint32_t* said;                  // [SMALL_MAX_TILES], and the state
    uint32_t call;                   // (16 bits)
    uint2* ranges;
    uint32_t* order;
    uint64_t* totals;                // (null: only the pairs are still to be written, into the ranges of the launch before)
    uint32_t* rec_offsets;
    uint32_t* rec_counts;
    float4* splats;
    uint64_t* bucket;
    uint64_t* keys_out;
    uint32_t* vals_out;
};

__device__ __forceinline__ uint32_t rect_area(const ushort4& r)
{
    return r.z > r.x && r.w > r.y ? (uint32_t)(r.z - r.x) * (uint32_t)(r.w - r.y) : 0u;
}

static_assert(SMALL_MAX_N < 65536, "16 bits for a tile's pairs");
struct SmallMemory {
    uint32_t* said;
    __device__ __forceinline__ unsigned long long pair(int i) const
    {
        return __hip_atomic_load(reinterpret_cast<const unsigned long long*>(said) + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ uint32_t state() const { return __hip_atomic_load(said + SMALL_MAX_TILES, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
    __device__ __forceinline__ uint32_t swap(uint32_t was, uint32_t now) const
    {
        __hip_atomic_compare_exchange_strong(said + SMALL_MAX_TILES, &was, now, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return was;
    }
    __device__ __forceinline__ void rest() const { __builtin_amdgcn_s_sleep(1); }
};

template <bool CB>
__global__ __launch_bounds__(SMALL_THREADS) void k_small_frame(SmallFrame f, CfgDev cfg)
{
    constexpr int T = SMALL_THREADS, WAVES = T / 64;
    constexpr int PER_TILE = SMALL_TILES_PER;
    constexpr int NB = ORDER_BUCKETS;
    union Mem {
        SortMem<TILE_SORT_SMALL, T, 1024> sort;
        uint16_t list[SMALL_MAX_N];     // Gaussians of the tile
        uint32_t buckets[NB];
    };
    __shared__ __align__(16) Mem mem;
    __shared__ uint32_t s_count, s_wave[2][WAVES], s_late, s_decided;
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const int n = (int)f.n;
    const SmallMemory mem_words = {f.said};
    auto said_tile = [&](int q) { return small_tile(t, q); };
    auto pairs_said = [&](int end, uint32_t (&c)[PER_TILE]) { return small_look(mem_words, t, end, f.call, SMALL_POLLS, c); };
    auto below = [](uint64_t bal) { return __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u)); };

    if ((int)blockIdx.x > f.num_tiles) {
        const int first = ((int)blockIdx.x - f.num_tiles - 1) * T, i = first + t;
        const ushort4 r = i < n ? f.rect[i] : make_ushort4(0, 0, 0, 0);
        const uint32_t area = rect_area(r);
        uint32_t before = 0;
        for (int j0 = 0; j0 < first; j0 += SMALL_PER * T) {
            ushort4 q[SMALL_PER];
#pragma unroll
            for (int u = 0; u < SMALL_PER; u++) q[u] = f.rect[min(j0 + u * T + t, n - 1)];
#pragma unroll
            for (int u = 0; u < SMALL_PER; u++) before += j0 + u * T < first ? rect_area(q[u]) : 0u;
        }
        const uint32_t inc = wave_inclusive_scan(area), all_before = wave_inclusive_scan(before);
        if (lane == 63) { s_wave[0][wave] = inc; s_wave[1][wave] = all_before; }
        __syncthreads();
        uint32_t at = inc - area, total = 0;
#pragma unroll
        for (int w = 0; w < WAVES; w++) {
            at += s_wave[1][w] + (w < wave ? s_wave[0][w] : 0u);
            total += s_wave[1][w] + s_wave[0][w];
        }
        if (i < n) {
            f.rec_offsets[i] = at;
            if (f.rec_counts) f.rec_counts[i] = area;
            if (area) pack_splat(f.splats, i, f.mean2d[i], f.conic_opacity[i], f.rgb, at, r, cfg);
        }
        if (blockIdx.x + 1 == gridDim.x) {
            // (below 2^31 both: at most 2^14 Gaussians in at most 2^10 tiles)
            uint32_t touched = 0;
            for (int j0 = 0; j0 < n; j0 += SMALL_PER * T) {
                uint32_t q[SMALL_PER];
#pragma unroll
                for (int u = 0; u < SMALL_PER; u++) q[u] = f.tiles_touched[min(j0 + u * T + t, n - 1)];
#pragma unroll
                for (int u = 0; u < SMALL_PER; u++) touched += j0 + u * T + t < n ? q[u] : 0u;
            }
            touched = wave_inclusive_scan(touched);
            __syncthreads();
            if (lane == 63) s_wave[0][wave] = touched;
            __syncthreads();
            if (t == 0) {
                uint64_t tt = 0;
                for (int w = 0; w < WAVES; w++) tt += s_wave[0][w];
                __hip_atomic_store(&f.totals[0], tt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
                __hip_atomic_store(&f.totals[1], (uint64_t)total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
        return;
    }

    if (t == 0) { s_count = 0u; s_late = 0u; }
    if ((int)blockIdx.x == f.num_tiles) {
        // the order: as in k_tile_layout
        auto bucket = [](uint32_t len) { return (int)(NB - 1 - min(len / ORDER_STEP, (uint32_t)NB - 1)); };
        uint32_t* const cnt = mem.buckets;
#pragma unroll
        for (int q = 0; q < NB / T; q++) cnt[t + q * T] = 0u;
        uint32_t c[PER_TILE], sum = 0, most = 0;
        const uint32_t state = t == T - 1 ? mem_words.state() : 0u;   // (requested here: only the swap follows the looks)
        const bool late = !pairs_said(f.num_tiles, c);
#pragma unroll
        for (int q = 0; q < PER_TILE; q++) {
            sum += c[q];
            most = max(most, c[q]);
        }
        __syncthreads();
        if (late) s_late = 1u;
#pragma unroll
        for (int q = 0; q < PER_TILE; q++)
            if (said_tile(q) < f.num_tiles) atomicAdd(&cnt[bucket(c[q])], 1u);
        sum = wave_inclusive_scan(sum);
        most = wave_inclusive_max(most);
        if (lane == 63) { s_wave[0][wave] = sum; s_wave[1][wave] = most; }
        __syncthreads();
        if (s_late) {   // (the totals stay unset; sorts of long lists that are enqueued already take what is here as tiles)
            for (int k = t; k < f.num_tiles; k += T) f.order[k] = (uint32_t)k;
            return;
        }
        if (wave == 0) {
            uint32_t v[NB / 64], all = 0;
#pragma unroll
            for (int q = 0; q < NB / 64; q++) { v[q] = cnt[lane * (NB / 64) + q]; all += v[q]; }
            uint32_t run = wave_inclusive_scan(all) - all;
#pragma unroll
            for (int q = 0; q < NB / 64; q++) { cnt[lane * (NB / 64) + q] = run; run += v[q]; }
        }
        if (t == T - 1 && small_decide(mem_words, f.call, state, SMALL_PUBLISHED) == SMALL_PUBLISHED) {
            uint64_t pairs = 0, longest = 0;
            for (int w = 0; w < WAVES; w++) { pairs += s_wave[0][w]; longest = max(longest, (uint64_t)s_wave[1][w]); }
            __hip_atomic_store(&f.totals[2], pairs, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(&f.totals[3], longest, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < PER_TILE; q++)
            if (said_tile(q) < f.num_tiles) f.order[atomicAdd(&cnt[bucket(c[q])], 1u)] = (uint32_t)said_tile(q);
        return;
    }

    const uint32_t tile = blockIdx.x;
    const uint32_t tx = tile % (uint32_t)f.tiles_x, ty = tile / (uint32_t)f.tiles_x;
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    struct Rect { u16x2 first, last; };   // (one past the last)
    const u16x2 me = {(unsigned short)tx, (unsigned short)ty};
    const Rect* const rects = reinterpret_cast<const Rect*>(f.rect);
    __syncthreads();
    auto scan = [&](int i0, auto whole) {
        Rect r[SMALL_PER];
#pragma unroll
        for (int u = 0; u < SMALL_PER; u++) r[u] = rects[min(i0 + u * T + t, n - 1)];   // (all requested at once: no branches between them)
        uint64_t in[SMALL_PER];
        uint32_t count = 0;
#pragma unroll
        for (int u = 0; u < SMALL_PER; u++) {
            // first <= me < last, both coordinates at once: a place before the first wraps round to beyond any size, and a rectangle
            // that ends before it starts has the size 0
            const u16x2 at = me - r[u].first, size = __builtin_elementwise_sub_sat(r[u].last, r[u].first);
            in[u] = __ballot((at.x < size.x) & (at.y < size.y) & (decltype(whole)::value || i0 + u * T + t < n));
            count += (uint32_t)__popcll(in[u]);
        }
        if (count == 0) return;
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&s_count, count);
        at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
        for (int u = 0; u < SMALL_PER; u++) {
            if (in[u] >> lane & 1ull) mem.list[at + below(in[u])] = (uint16_t)(i0 + u * T + t);
            at += (uint32_t)__popcll(in[u]);
        }
    };
    int i0 = 0;
    for (; i0 + SMALL_PER * T <= n; i0 += SMALL_PER * T) scan(i0, std::true_type{});
    if (i0 < n) scan(i0, std::false_type{});
    __syncthreads();
    int len = (int)s_count;
    if (CB) {
        // those that the ellipse leaves, packed to the front of the list: a round's places are read before any is written, and no later
        // one's is
        __syncthreads();
        if (t == 0) s_count = 0u;
        __syncthreads();
        constexpr int PER = 4;
        for (int i0 = 0; i0 < len; i0 += PER * T) {
            uint32_t g[PER];
            float2 m[PER];
            float4 co[PER];
#pragma unroll
            for (int u = 0; u < PER; u++) g[u] = i0 + u * T + t < len ? mem.list[i0 + u * T + t] : ~0u;
            __syncthreads();
#pragma unroll
            for (int u = 0; u < PER; u++) {
                const uint32_t at = g[u] != ~0u ? g[u] : 0u;
                m[u] = f.mean2d[at];
                co[u] = f.conic_opacity[at];
            }
            uint64_t in[PER];
            uint32_t count = 0;
#pragma unroll
            for (int u = 0; u < PER; u++) {
                if (i0 + u * T >= len) { in[u] = 0ull; continue; }
                in[u] = __ballot(g[u] != ~0u && cb_tile_hit(m[u].x, m[u].y, co[u].x, co[u].y, co[u].z, cb_threshold(co[u].w, cfg), (int)tx, (int)ty));
                count += (uint32_t)__popcll(in[u]);
            }
            uint32_t at = 0;
            if (lane == 0 && count) at = atomicAdd(&s_count, count);
            at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
#pragma unroll
            for (int u = 0; u < PER; u++) {
                if (in[u] >> lane & 1ull) mem.list[at + below(in[u])] = (uint16_t)g[u];
                at += (uint32_t)__popcll(in[u]);
            }
        }
        __syncthreads();
        len = (int)s_count;
    }
    if (t == 0 && f.totals)
        __hip_atomic_store(&f.said[tile], f.call << 16 | (uint32_t)len, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

    // where the tile's segment starts, ~0u where nothing is to be written; its range
    auto place = [&]() -> uint32_t {
        if (!f.totals) {
            const uint2 r = f.ranges[tile];
            return r.y <= f.limit ? r.x : ~0u;
        }
        uint32_t first = 0;
        for (bool again = false;; again = true) {
            uint32_t c[PER_TILE], sum = 0;
            if (!pairs_said((int)tile, c)) s_late = 1u;
#pragma unroll
            for (int q = 0; q < PER_TILE; q++) sum += c[q];
            sum = wave_inclusive_scan(sum);
            if (lane == 63) s_wave[0][wave] = sum;
            __syncthreads();
            first = 0;
#pragma unroll
            for (int w = 0; w < WAVES; w++) first += s_wave[0][w];
            if (!s_late) break;
            if (t == 0) s_decided = small_decide(mem_words, f.call, mem_words.state(), SMALL_GIVEN_UP);
            __syncthreads();
            if (s_decided != SMALL_PUBLISHED || again) {
                if (t == 0) f.ranges[tile] = make_uint2(0u, 0u);   // (for sorts of long lists that are enqueued already)
                return ~0u;
            }
            if (t == 0) s_late = 0u;   // (all words are there by now: the next look finds them)
            __syncthreads();
        }
        if (t == 0) f.ranges[tile] = make_uint2(first, first + (uint32_t)len);
        return first + (uint32_t)len <= f.limit ? first : ~0u;
    };
    auto word = [&](int i) {   // (any i: the first one stands in for those past the list's end)
        const uint32_t g = mem.list[i < len ? i : 0];
        return (uint64_t)__float_as_uint(f.depth[g]) << 32 | g;
    };
    if (len == 0) {   // (its range is the same wherever the other tiles' pairs lie: it waits for none)
        if (t == 0 && f.totals) f.ranges[tile] = make_uint2(0u, 0u);
        return;
    }
    if (len > TILE_SORT_SMALL) {
        const uint32_t to = place();
        if (to != ~0u)
            for (int i = t; i < len; i += T) f.bucket[to + i] = word(i);
        return;
    }
    uint64_t w[TILE_SORT_SMALL / T];
#pragma unroll
    for (int u = 0; u < TILE_SORT_SMALL / T; u++) w[u] = u * T < len ? word(t + u * T) : 0ull;
    __syncthreads();   // (the list has been read: the sort's memory is the same)
    sort_list<TILE_SORT_SMALL, T, 1024, false>(mem.sort, w, len, tile, [&](int u) { return w[u]; }, place, f.keys_out, f.vals_out);
}

// ---- radix sort -------------------------------------------------------------------------
// One pass ranks RADIX_BLOCK_KEYS keys per workgroup on a digit of up to RADIX_BITS bits (the live key
// bits are split into the fewest such digits, of equal width).  Wave w of the workgroup owns the
// contiguous chunk [w*512, w*512+512) of the block's keys and walks it in 8 rounds of 64 consecutive
// keys, so (wave, round, lane) order is the input order and the ranking is stable.

constexpr int RADIX_ROUNDS = RADIX_BLOCK_KEYS / 256;  // rounds per wave

// Per-workgroup digit histogram, stored digit-major: hist[digit * num_blocks + block].
__global__ __launch_bounds__(256) void k_radix_hist(const uint64_t* __restrict__ keys, uint32_t P, int shift,
                                                    uint32_t mask, uint32_t num_blocks,
                                                    uint32_t* __restrict__ hist)
{
    __shared__ uint32_t cnt[RADIX_DIGITS];
    for (int d = threadIdx.x; d < RADIX_DIGITS; d += 256) cnt[d] = 0;
    __syncthreads();
    const uint32_t base = blockIdx.x * RADIX_BLOCK_KEYS;
#pragma unroll
    for (int r = 0; r < RADIX_ROUNDS; r++) {
        const uint32_t i = base + r * 256 + threadIdx.x;
        if (i < P) atomicAdd(&cnt[(uint32_t)(keys[i] >> shift) & mask], 1u);
    }
    __syncthreads();
    for (uint32_t d = threadIdx.x; d <= mask; d += 256) hist[d * num_blocks + blockIdx.x] = cnt[d];
}

__global__ __launch_bounds__(256) void k_radix_scatter(const uint64_t* __restrict__ kin,
                                                       const uint32_t* __restrict__ vin,
                                                       uint64_t* __restrict__ kout, uint32_t* __restrict__ vout,
                                                       const uint32_t* __restrict__ hist_scanned, uint32_t P,
                                                       int shift, int bits, uint32_t num_blocks)
{
    __shared__ uint32_t cnt[4][RADIX_DIGITS];
    const int wave = threadIdx.x >> 6;
    const uint32_t lane = lane_id();
    const uint32_t mask = (1u << bits) - 1u;
#pragma unroll
    for (int w = 0; w < 4; w++)
        for (int d = threadIdx.x; d < RADIX_DIGITS; d += 256) cnt[w][d] = 0;
    __syncthreads();

    const uint32_t wave_start = blockIdx.x * RADIX_BLOCK_KEYS + wave * (RADIX_ROUNDS * 64);
    uint64_t key[RADIX_ROUNDS];
    uint32_t val[RADIX_ROUNDS], rank[RADIX_ROUNDS];
#pragma unroll
    for (int r = 0; r < RADIX_ROUNDS; r++) {
        const uint32_t i = wave_start + r * 64 + lane;
        const bool valid = i < P;
        key[r] = valid ? kin[i] : 0ull;
        val[r] = valid ? vin[i] : 0u;
    }
#pragma unroll
    for (int r = 0; r < RADIX_ROUNDS; r++) {
        const uint32_t i = wave_start + r * 64 + lane;
        const bool valid = i < P;
        const uint32_t d = (uint32_t)(key[r] >> shift) & mask;
        // lanes of this wave holding the same digit
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < bits; b++) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bal = __ballot(valid && bit);
            peers &= bit ? bal : ~bal;
        }
        const uint32_t below = __popcll(peers & ((1ull << lane) - 1ull));
        const uint32_t count = __popcll(peers);
        uint32_t prev = 0;
        if (valid) prev = cnt[wave][d];
        __builtin_amdgcn_wave_barrier();
        if (valid && below == 0) cnt[wave][d] = prev + count;
        __builtin_amdgcn_wave_barrier();
        rank[r] = prev + below;
    }
    __syncthreads();
    // per digit: global start of this block's run of that digit, then per-wave starts
    for (uint32_t d = threadIdx.x; d <= mask; d += 256) {
        uint32_t run = hist_scanned[d * num_blocks + blockIdx.x];
#pragma unroll
        for (int w = 0; w < 4; w++) {
            const uint32_t c = cnt[w][d];
            cnt[w][d] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RADIX_ROUNDS; r++) {
        const uint32_t i = wave_start + r * 64 + lane;
        if (i < P) {
            const uint32_t d = (uint32_t)(key[r] >> shift) & mask;
            const uint32_t pos = cnt[wave][d] + rank[r];
            kout[pos] = key[r];
            vout[pos] = val[r];
        }
    }
}

// ranges[t] = [first,last) for every tile present in the sorted keys (ranges pre-filled with 0).
__global__ __launch_bounds__(256) void k_tile_ranges(const uint64_t* __restrict__ keys, uint32_t P,
                                                     uint32_t* __restrict__ ranges)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= P) return;
    const uint32_t t = (uint32_t)(keys[i] >> 32);
    if (i == 0 || (uint32_t)(keys[i - 1] >> 32) != t) ranges[2 * t] = i;
    if (i + 1 == P || (uint32_t)(keys[i + 1] >> 32) != t) ranges[2 * t + 1] = i + 1;
}

// Order in which the render kernels take the tiles: longest list first (bucketed by length / 8), so
// that the last workgroups of a launch are the cheapest ones.  One workgroup; any order is valid.
__global__ __launch_bounds__(1024) void k_tile_order(const uint2* __restrict__ ranges, int num_tiles,
                                                     uint32_t* __restrict__ order)
{
    constexpr int NB = ORDER_BUCKETS;
    __shared__ uint32_t cnt[NB];
    for (int b = threadIdx.x; b < NB; b += 1024) cnt[b] = 0;
    __syncthreads();
    auto bucket = [](uint2 r) { const uint32_t len = r.y - r.x; return (int)(NB - 1 - min(len / ORDER_STEP, (uint32_t)NB - 1)); };
    for (int t = threadIdx.x; t < num_tiles; t += 1024) atomicAdd(&cnt[bucket(ranges[t])], 1u);
    __syncthreads();
    if (threadIdx.x < 64) {  // exclusive prefix over the 512 buckets by one wavefront, 8 buckets per lane
        uint32_t c[8], sum = 0;
#pragma unroll
        for (int k = 0; k < 8; k++) { c[k] = cnt[threadIdx.x * 8 + k]; sum += c[k]; }
        uint32_t run = wave_inclusive_scan(sum) - sum;
#pragma unroll
        for (int k = 0; k < 8; k++) { cnt[threadIdx.x * 8 + k] = run; run += c[k]; }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < num_tiles; t += 1024) order[atomicAdd(&cnt[bucket(ranges[t])], 1u)] = (uint32_t)t;
}

constexpr int FILL_BLOCKS = 2048;   // eight for each compute unit
// Bound by memory: four words for each store (where p is on a 16-byte boundary), as many workgroups as the chip holds at a time.  The
// records of 1.5 M candidate tiles (72 MB, which stay in the last-level cache) 11.9 us, 19.1 with a word for each thread; 960 MB 206 and 203.
__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* __restrict__ p, uint32_t v, int64_t count, int64_t fours)
{
    const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = first; i < fours; i += stride) reinterpret_cast<uint4*>(p)[i] = make_uint4(v, v, v, v);
    for (int64_t i = 4 * fours + first; i < count; i += stride) p[i] = v;
}

}  // namespace

size_t scan_tmp_bytes(int64_t n)
{
    const int64_t nb = (n + SCAN_BLOCK - 1) / SCAN_BLOCK;
    return (size_t)(nb > 0 ? nb : 1) * sizeof(uint64_t);
}

hipError_t launch_exclusive_scan(hipStream_t st, const uint32_t* in, uint32_t* out, int64_t n, void* tmp,
                                 uint64_t* total_dev)
{
    const int64_t nb = (n + SCAN_BLOCK - 1) / SCAN_BLOCK;
    uint64_t* bs = static_cast<uint64_t*>(tmp);
    if (nb > 0) hipLaunchKernelGGL(k_scan_block_sums, dim3((unsigned)nb), dim3(SCAN_THREADS), 0, st, in, n, bs);
    hipLaunchKernelGGL(k_scan_block_offsets, dim3(1), dim3(SCAN_THREADS), 0, st, bs, nb, total_dev);
    if (nb > 0) hipLaunchKernelGGL(k_scan_apply, dim3((unsigned)nb), dim3(SCAN_THREADS), 0, st, in, out, n, bs);
    return hipGetLastError();
}

hipError_t launch_emit_pairs(hipStream_t st, int64_t n, const fs_projected& proj, const CfgDev& cfg, const uint32_t* offsets,
                             int tiles_x, uint64_t* keys, uint32_t* vals, float* splats)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_emit_pairs, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n,
                       reinterpret_cast<const ushort4*>(proj.rect), proj.depth,
                       reinterpret_cast<const float2*>(proj.mean2d), reinterpret_cast<const float4*>(proj.conic_opacity),
                       proj.rgb, cfg, offsets, tiles_x, keys, vals, reinterpret_cast<float4*>(splats));
    return hipGetLastError();
}

hipError_t launch_rect_area(hipStream_t st, int64_t n, const uint16_t* rect, uint32_t* rec_counts)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_rect_area, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n,
                       reinterpret_cast<const ushort4*>(rect), rec_counts);
    return hipGetLastError();
}

hipError_t launch_emit_pairs_cb(hipStream_t st, int64_t n, const fs_projected& proj, const CfgDev& cfg,
                                const uint32_t* offsets, const uint32_t* rec_offsets, int tiles_x, int64_t P,
                                uint64_t* keys, uint32_t* vals, float* splats)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_emit_pairs_cb, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n,
                       reinterpret_cast<const ushort4*>(proj.rect), proj.depth,
                       reinterpret_cast<const float2*>(proj.mean2d), reinterpret_cast<const float4*>(proj.conic_opacity),
                       proj.rgb, cfg, offsets, rec_offsets, tiles_x, (uint32_t)P, keys, vals,
                       reinterpret_cast<float4*>(splats));
    return hipGetLastError();
}

hipError_t launch_tile_count(hipStream_t st, int64_t n, const fs_projected& proj, const CfgDev& cfg, int tiles_x,
                             int num_tiles, uint32_t* tile_count, uint32_t* tile_total, uint2* ranges,
                             uint32_t* tile_order, uint64_t* totals, uint32_t* rec_offsets, uint32_t* rec_counts,
                             uint64_t* counters, float* splats, bool bands)
{
    uint64_t* const wg_totals = counters + 1;
    const RecAlloc ra = {proj.tiles_touched, rec_offsets, rec_counts, wg_totals};
    {
        const dim3 grid(TILE_COPIES), block(TILE_PAIR_THREADS);
        const size_t lds = (size_t)num_tiles * sizeof(uint32_t);
        const ushort4* rect = reinterpret_cast<const ushort4*>(proj.rect);
        const float2* m2 = reinterpret_cast<const float2*>(proj.mean2d);
        const float4* co = reinterpret_cast<const float4*>(proj.conic_opacity);
        if (cfg.compact_box)
            hipLaunchKernelGGL((k_tile_pairs<true, false, false>), grid, block, lds, st, n, rect, proj.depth, m2, co, cfg,
                               tiles_x, num_tiles, tile_count, nullptr, 0u, nullptr, ra, BandPlaces{});
        else
            hipLaunchKernelGGL((k_tile_pairs<false, false, false>), grid, block, lds, st, n, rect, proj.depth, m2, co,
                               cfg, tiles_x, num_tiles, tile_count, nullptr, 0u, nullptr, ra, BandPlaces{});
    }
    const int sum_blocks = (num_tiles + 63) / 64;
    hipLaunchKernelGGL(k_tile_layout, dim3((unsigned)(sum_blocks + std::max<int64_t>(1, (n + LAYOUT_THREADS - 1) / LAYOUT_THREADS))), dim3(LAYOUT_THREADS), 0, st,
                       tile_count, num_tiles, sum_blocks, tile_total, ranges, tile_order, totals,
                       reinterpret_cast<unsigned long long*>(counters), wg_totals, n, reinterpret_cast<const ushort4*>(proj.rect),
                       reinterpret_cast<const float2*>(proj.mean2d), reinterpret_cast<const float4*>(proj.conic_opacity), proj.rgb,
                       cfg, rec_offsets, reinterpret_cast<float4*>(splats), bands ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_tile_scatter(hipStream_t st, int64_t n, const fs_projected& proj, const CfgDev& cfg,
                               int tiles_x, int num_tiles, uint32_t pair_limit, const uint2* ranges, uint32_t* cursor, uint64_t* bucket,
                               const BandPlaces& places)
{
    if (n <= 0) return hipSuccess;
    const dim3 grid(TILE_COPIES), block(TILE_PAIR_THREADS);
    const size_t lds = (size_t)num_tiles * sizeof(uint32_t);
    const ushort4* rect = reinterpret_cast<const ushort4*>(proj.rect);
    const float2* m2 = reinterpret_cast<const float2*>(proj.mean2d);
    const float4* co = reinterpret_cast<const float4*>(proj.conic_opacity);
    auto launch = [&](auto kernel, size_t bytes) {
        hipLaunchKernelGGL(kernel, grid, block, bytes, st, n, rect, proj.depth, m2, co, cfg, tiles_x, num_tiles, cursor, ranges, pair_limit,
                           bucket, RecAlloc{}, places);
    };
    if (places.band) {
        const size_t bytes = (size_t)(num_tiles + BAND_TILES - 1) / BAND_TILES * sizeof(uint32_t);
        if (cfg.compact_box) launch(k_tile_pairs<true, true, true>, bytes);
        else launch(k_tile_pairs<false, true, true>, bytes);
    } else if (cfg.compact_box) launch(k_tile_pairs<true, true, false>, lds);
    else launch(k_tile_pairs<false, true, false>, lds);
    return hipGetLastError();
}

hipError_t launch_small_frame(hipStream_t st, int64_t n, const fs_projected& proj, const CfgDev& cfg, int tiles_x, int num_tiles,
                              uint32_t pair_limit, uint32_t* said, uint32_t call, uint2* ranges, uint32_t* tile_order, uint64_t* totals,
                              uint32_t* rec_offsets, uint32_t* rec_counts, float* splats, uint64_t* bucket, uint64_t* keys_out, uint32_t* vals_out)
{
    const SmallFrame f = {n, reinterpret_cast<const ushort4*>(proj.rect), proj.depth, reinterpret_cast<const float2*>(proj.mean2d),
                          reinterpret_cast<const float4*>(proj.conic_opacity), proj.rgb, proj.tiles_touched, tiles_x, num_tiles, pair_limit,
                          said, call, ranges, tile_order, totals, rec_offsets, rec_counts,
                          reinterpret_cast<float4*>(splats), bucket, keys_out, vals_out};
    const dim3 grid((unsigned)(totals ? num_tiles + 1 + (n + SMALL_THREADS - 1) / SMALL_THREADS : num_tiles));
    if (cfg.compact_box) hipLaunchKernelGGL(k_small_frame<true>, grid, dim3(SMALL_THREADS), 0, st, f, cfg);
    else hipLaunchKernelGGL(k_small_frame<false>, grid, dim3(SMALL_THREADS), 0, st, f, cfg);
    return hipGetLastError();
}

int tile_sort_variants(int64_t max_len, bool long_lists, int have)
{
    // which length classes still need a launch: (0, SMALL], (SMALL, MID], (MID, MAX], (MAX, HUGE]
    int v = 0;
    if (!(have & TS_SMALL)) v |= TS_SMALL;
    const bool need_mid = max_len > TILE_SORT_SMALL && !(have & (TS_MID | TS_MIDMAX));
    const bool need_max = max_len > TILE_SORT_MID && !(have & (TS_MAX | TS_MIDMAX));
    if (need_mid && need_max) v |= long_lists ? (TS_MID | TS_MAX) : TS_MIDMAX;
    else if (need_mid) v |= long_lists || (have & TS_MAX) ? TS_MID : TS_MIDMAX;
    else if (need_max) v |= TS_MAX;
    if (max_len > TILE_SORT_MAX && !(have & TS_HUGE)) v |= TS_HUGE;
    return v;
}

hipError_t launch_tile_sorts(hipStream_t st, int num_tiles, int variants, uint32_t pair_limit, const uint2* ranges,
                             const uint32_t* tile_order, uint64_t* bucket, uint64_t* keys_out, uint32_t* vals_out,
                             const BandPlaces& places)
{
    if (num_tiles <= 0) return hipSuccess;
    // Lists longer than len_lo stand at the front of the order: it is sorted by buckets of ORDER_STEP lengths (the last one
    // open), so only the lists of their bucket or a longer one stand before them, and no more of those fit into the pairs.
    // (A workgroup per tile, almost all of which left at once, took 2 to 4 us per launch: placement and sorts 75.3 -> 72.6 us at
    // 500k Gaussians and 1600x1064, 242 -> 238 at 3 M and 1920x1080.)
    auto grid = [&](uint32_t len_lo) {
        const uint32_t least = ORDER_STEP * std::min((len_lo + 1) / ORDER_STEP, (uint32_t)ORDER_BUCKETS - 1);
        return dim3(std::min((uint32_t)num_tiles, std::max(1u, pair_limit / least)));
    };
    if (variants & TS_SPLIT) {
        // (no more chunks than these; a capacity far beyond the pairs would give workgroups that leave at once)
        const uint32_t bands = (uint32_t)((num_tiles + BAND_TILES - 1) / BAND_TILES);
        hipLaunchKernelGGL(k_band_split, dim3(std::min(pair_limit / SPLIT_WORDS, 4096u) + bands), dim3(SPLIT_THREADS), 0, st, num_tiles,
                           pair_limit, places, keys_out, bucket);
    }
    // the long lists first: few workgroups, each a long chain of steps, which more threads shorten
    if (variants & TS_HUGE)
        hipLaunchKernelGGL((k_tile_sort<TILE_SORT_HUGE, 1024, 4096>), grid(TILE_SORT_MAX), dim3(1024), 0, st, ranges, tile_order,
                           bucket, TILE_SORT_MAX, pair_limit, keys_out, vals_out);
    if (variants & (TS_MAX | TS_MIDMAX)) {
        const int len_lo = (variants & TS_MIDMAX) ? TILE_SORT_SMALL : TILE_SORT_MID;
        hipLaunchKernelGGL((k_tile_sort<TILE_SORT_MAX, 1024, 2048>), grid(len_lo), dim3(1024), 0, st, ranges, tile_order,
                           bucket, len_lo, pair_limit, keys_out, vals_out);
    }
    if (variants & TS_MID)
        hipLaunchKernelGGL((k_tile_sort<TILE_SORT_MID, 512, 1536>), grid(TILE_SORT_SMALL), dim3(512), 0, st, ranges, tile_order,
                           bucket, TILE_SORT_SMALL, pair_limit, keys_out, vals_out);
    if (variants & TS_SMALL)
        hipLaunchKernelGGL((k_tile_sort<TILE_SORT_SMALL, 256, 1024>), dim3(num_tiles), dim3(256), 0, st, ranges, tile_order, bucket,
                           0, pair_limit, keys_out, vals_out);
    return hipGetLastError();
}

hipError_t launch_radix_sort(hipStream_t st, int64_t P, int total_bits, uint64_t* keys[2], uint32_t* vals[2],
                             uint32_t* hist, void* scan_tmp, uint64_t* scan_total_dev, int* result_index)
{
    int cur = 0;
    if (P > 0) {
        const uint32_t nb = (uint32_t)radix_num_blocks(P);
        const int passes = (total_bits + RADIX_BITS - 1) / RADIX_BITS;
        const int bits = (total_bits + passes - 1) / passes;  // equal-width digits, at most RADIX_BITS
        for (int p = 0; p < passes; p++) {
            const int shift = bits * p;
            const uint32_t mask = (1u << bits) - 1u;
            hipLaunchKernelGGL(k_radix_hist, dim3(nb), dim3(256), 0, st, keys[cur], (uint32_t)P, shift, mask, nb,
                               hist);
            hipError_t e = launch_exclusive_scan(st, hist, hist, (int64_t)(mask + 1) * nb, scan_tmp, scan_total_dev);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(k_radix_scatter, dim3(nb), dim3(256), 0, st, keys[cur], vals[cur], keys[cur ^ 1],
                               vals[cur ^ 1], hist, (uint32_t)P, shift, bits, nb);
            cur ^= 1;
        }
    }
    *result_index = cur;
    return hipGetLastError();
}

hipError_t launch_tile_ranges(hipStream_t st, int64_t P, const uint64_t* keys_sorted, int num_tiles,
                              uint32_t* ranges, uint32_t* tile_order)
{
    hipError_t e = launch_fill_u32(st, ranges, 0u, (int64_t)2 * num_tiles);
    if (e != hipSuccess) return e;
    if (P > 0)
        hipLaunchKernelGGL(k_tile_ranges, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, st, keys_sorted,
                           (uint32_t)P, ranges);
    if (num_tiles > 0)
        hipLaunchKernelGGL(k_tile_order, dim3(1), dim3(1024), 0, st, reinterpret_cast<const uint2*>(ranges), num_tiles,
                           tile_order);
    return hipGetLastError();
}

hipError_t launch_fill_u32(hipStream_t st, uint32_t* p, uint32_t v, int64_t count)
{
    if (count <= 0) return hipSuccess;
    // (a launch of 2^32 threads or more is refused, and a dense backward pass with the Compact Box clears up to 2^31 records)
    const int64_t fours = reinterpret_cast<uintptr_t>(p) % 16 == 0 ? count / 4 : 0;
    const int64_t threads = std::max(fours, count - 4 * fours);
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)std::min<int64_t>((threads + 255) / 256, FILL_BLOCKS)), dim3(256), 0, st, p, v, count, fours);
    return hipGetLastError();
}

}  // namespace fs
