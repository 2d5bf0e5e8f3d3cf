// Per-tile alpha compositing (forward), its gradient (backward) and the high-error-pixel count
// (score) on gfx950.
//
// FastGS Sec. 3, Eq. (4): C(p) = sum_i c_i alpha_i prod_{j<i} (1 - alpha_j), alpha_i = sigma_i G'_i(p),
// Eq. (5): G'_i(p) = exp(-1/2 (p - mu_2D)^T Sigma_2D^-1 (p - mu_2D)).
// Sec. 4.2, Eq. for s_d: per Gaussian, the number of high-error pixels in its footprint.
//
// One workgroup (4 wavefronts) per 16x16 tile, one pixel per lane.  Wavefront w owns the 8x8
// quadrant (w&1, w>>1); each of its four rows of 16 lanes (the unit of the DPP row operations) owns
// one 4x4 sub-tile of that quadrant.  The tile's depth-ordered Gaussians are staged through LDS in
// batches of 255 (k_render_bwd: 231, with the absolute gradient 207).  Every Gaussian's support
// {alpha >= alpha_min} is bounded by its ellipse (conservatively, support_strips; it comes with the splat
// record) and each of the 16 sub-tiles gets its own order-preserving list of the staged Gaussians
// whose ellipse meets it.  In the inner loops the four
// rows of a wavefront walk their own lists side by side, so one wavefront iteration evaluates
// four different Gaussians on 16 pixels each.  A wavefront stops as soon as all of its 64 pixels
// have terminated.
//
// alpha, T and the blend weights follow a fixed fp32 operation order (fused multiply-adds only
// where written as __builtin_fmaf; the file is compiled with -ffp-contract=off) so that the
// integer outputs they decide (n_contrib, counts) can be reproduced bit for bit on a CPU.  The
// ellipse only ever drops (Gaussian, pixel) pairs that this arithmetic would reject as well.
//
// Times "at 500k Gaussians and 1600x1064" and the like are of the scenes of perf/cases.py.  They have other pairs than those of
// bench.py with the same sizes: 6 k against 11 k at 4k Gaussians and 128x128, 0.4 M to 0.5 M against 0.5 M at 100k, 2.1 M to 2.9 M
// against 1.4 M at 500k, 11 M to 13 M against 10 M at 3 M (wide: 30 M to 37 M against 27 M).
#include <type_traits>

#include "common.hpp"

namespace fs {

namespace {

constexpr int SLOTS = 256;        // records a workgroup holds in LDS: one per thread (k_render_bwd: fewer)
constexpr int BATCH = SLOTS - 1;  // list entries staged at a time; the last record is the empty one that pads the sub-tile lists
constexpr int GROUP = 4;          // entries of a sub-tile list that a lane evaluates side by side (one 32-bit word of slots)

// exp(x) for x <= 0, with t = x*log2(e) (exponent_of): n = rint(t); r = t - n; 2^r by a degree-5 polynomial (Horner,
// fused), scaled by 2^n.  No range clamp: the scaling underflows to zero by itself where t is finite; t = -infinity, which
// conics at the end of the single-precision range give, would leave a NaN and is what takes_part keeps out.
__device__ __forceinline__ float exponent_of(float x) { return x * 0x1.715476p+0f; }
__device__ constexpr float EXP_C[5] = {0x1.5bba14p-10f, 0x1.3cea88p-7f, 0x1.c6b752p-5f, 0x1.ebf9bcp-3f, 0x1.62e42ap-1f};
__device__ __forceinline__ float exp_c(float t)
{
    const float n = __builtin_rintf(t);
    const float r = t - n;
    float p = EXP_C[0];
    p = __builtin_fmaf(p, r, EXP_C[1]);
    p = __builtin_fmaf(p, r, EXP_C[2]);
    p = __builtin_fmaf(p, r, EXP_C[3]);
    p = __builtin_fmaf(p, r, EXP_C[4]);
    p = __builtin_fmaf(p, r, 1.0f);
    return __builtin_ldexpf(p, (int)n);
}
// Neither positive nor -infinity.  Class bits: 0, 1 NaNs; 3, 4 negative numbers; 5, 6 zeros.
constexpr int TAKES_PART = 0x003 | 0x018 | 0x060;
__device__ __forceinline__ bool takes_part(float t) { return __builtin_amdgcn_classf(t, TAKES_PART); }
// The same as one bit per lane, in one instruction like the comparison with zero that it stands for (the compiler makes three
// of a ballot of the above: the render kernels 1 to 2 % slower).
__device__ __forceinline__ uint64_t takes_part_mask(float t)
{
    uint64_t mask;
    asm("v_cmp_class_f32_e64 %0, %1, %2" : "=s"(mask) : "v"(t), "s"(TAKES_PART));
    return mask;
}

// One step of four entries' chains of arithmetic: nothing moves into it or out of it.
#define FS_STEP __builtin_amdgcn_sched_barrier(0); _Pragma("unroll") for (int u = 0; u < GROUP; u++)

// 16-byte streaming (non-temporal) store / load
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void nt_store(const uint4& v, uint4* dst)
{
    u32x4 t;
    t.x = v.x; t.y = v.y; t.z = v.z; t.w = v.w;
    __builtin_nontemporal_store(t, reinterpret_cast<u32x4*>(dst));
}
__device__ __forceinline__ uint4 nt_load(const uint4* src)
{
    const u32x4 t = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src));
    return make_uint4(t.x, t.y, t.z, t.w);
}

struct Pixel {
    int x, y;
    bool inside;
    float px, py;
};

__device__ __forceinline__ Pixel pixel_of_thread(const CamDev& cam, int tile, int thread)
{
    const int wave = thread >> 6, lane = thread & 63;
    const int tx = tile % cam.tiles_x, ty = tile / cam.tiles_x;
    const int row = lane >> 4;  // 4x4 sub-tile (row & 1, row >> 1) of the quadrant
    Pixel p;
    p.x = tx * TILE + (wave & 1) * 8 + (row & 1) * 4 + (lane & 3);
    p.y = ty * TILE + (wave >> 1) * 8 + (row >> 1) * 4 + ((lane >> 2) & 3);
    p.inside = p.x < cam.width && p.y < cam.height;
    p.px = (float)p.x + 0.5f;
    p.py = (float)p.y + 0.5f;
    return p;
}

__device__ __forceinline__ Pixel pixel_of_thread(const CamDev& cam, int tile)
{
    return pixel_of_thread(cam, tile, (int)threadIdx.x);
}

// LDS image of one batch of a tile's list, shared by the kernels.  A staged Gaussian is one 16-byte word in each of two
// or (WITH_RGB) three arrays, so that one slot number, shifted once, addresses all of them:
//   r0 = (mu_x, mu_y, -a/2, -b)   r1 = (-c/2, sigma, r, g)   r2 = (r, g, b, bits of the pair's gradient record number + NEEDLE)
// The factors make the quadratic form come out as the exponent -1/2 (a dx^2 + 2 b dx dy + c dy^2) itself: halving and
// negating commute with every rounding on the way, so the exponent is the same to the bit.
template <bool WITH_RGB, int N = SLOTS>
struct Stage {
    static_assert(N <= 256 && N % 8 == 0, "one byte names a slot, one thread fills it");
    static constexpr int EMPTY = N - 1;
    float4 r0[N], r1[N];
    float4 r2[WITH_RGB ? N : 1];
    __align__(16) uint32_t list[16][N / 4];  // per sub-tile (index wave*4 + row): batch slots to visit, in list order, one byte each
    __align__(16) uint32_t sub[128];  // per slot, 16 bits: the sub-tiles that visit it (see sub_place)
    int len[16];                   // length of each sub-tile's list
    // Slot EMPTY is the empty record (sigma = 0: alpha = 0, nothing is ever blended); the others must hold finite numbers
    // before they are filled for the first time.
    __device__ __forceinline__ void clear(int t)
    {
        const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
        if (N < 256 && t >= N) return;
        r0[t] = z;
        r1[t] = z;
        if (WITH_RGB) r2[t] = z;
    }
    // where slot t's 16 bits sit in `sub` (in units of 16 bits): word 8 (t / 16) + t % 8, upper half for t % 16 >= 8, so
    // that the eight words of 16 slots turn into one sub-tile's 16 bits with a shift, a mask and an insertion each
    static __device__ __forceinline__ int sub_place(int t) { return ((t >> 4) * 8 + (t & 7)) * 2 + ((t >> 3) & 1); }
    __device__ __forceinline__ int slot(int st, int k) const { return reinterpret_cast<const uint8_t*>(list[st])[N == 256 ? k & 255 : k]; }
};

// Sub-tile st = wave*4 + row of a tile sits at column kx = (wave&1)*2 + (row&1), line ky = (wave>>1)*2 + (row>>1).
struct SubTiles {
    // bits 4 ky + kx to bits st: the two middle bits of the bit's number change places
    static __device__ __forceinline__ uint32_t from_grid(uint32_t m) { return (m & 0xc3c3u) | (m & 0x0c0cu) << 2 | (m >> 2 & 0x0c0cu); }
};

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_shr_add(uint32_t v)
{
    return v + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xF, 0xF, false);
}

// Loads m entries of the tile's list into `s` (slot t <- Gaussian g of thread t) and builds
// the 16 per-sub-tile slot lists.  Returns the length of the list of the calling lane's sub-tile.
// Contains one workgroup barrier; every thread of the workgroup must call it, after a barrier behind the previous
// batch's walk.  A wavefront's own four lists are complete when it returns (the others' only behind another barrier).
//
// Which sub-tiles may blend a Gaussian: those its support's ellipse meets (support_strips, part of the splat record).
//
// Lists: every thread leaves its entry's 16 sub-tile bits in LDS; then the 16 lanes that own a sub-tile in the render
// loops gather that sub-tile's bit of 16 slots each and expand them into slot numbers with a prefix sum over the row.
// The rest of a list is filled with the empty slot, so that the loops may run past a list's end.
// REVERSED: the lists run from the last entry to the first, and the calling lane's row leaves out slots from row_end on.
// ID_MODE: 0 = nothing, 1 = s_id[t] <- Gaussian index, 2 = r2[t].w <- index of the pair's
// gradient record (where the pair was emitted before the sort: offset + place in the rectangle), 3 = r2[t].w <- Gaussian index.
// GIVEN: the sub-tiles come as an argument (bit st).
template <int ID_MODE, bool REVERSED = false, bool GIVEN = false, bool WITH_RGB, int N>
__device__ __forceinline__ int stage_batch(Stage<WITH_RGB, N>& s, uint32_t* s_id, const CamDev& cam,
                                           int tile, const float4* __restrict__ splats, uint32_t g, int m, int row_end = N, uint32_t given = 0)
{
    const int t = threadIdx.x;
    const int swave = t >> 6, lane = t & 63;
    uint32_t sub_mask = 0;  // bit (wave*4 + row) of every sub-tile the ellipse meets
    if (t < m) {
        const float4* rec = splats + (size_t)g * (SPLAT_REC / 4);  // one 64-byte line
        const float4 r0 = rec[0], r1 = rec[1], r2 = rec[2];
        const float2 xy = make_float2(r0.x, r0.y);
        const float4 co = make_float4(r0.z, r0.w, r1.x, r1.y);
        s.r0[t] = make_float4(xy.x, xy.y, -0.5f * co.x, -co.y);
        s.r1[t] = make_float4(-0.5f * co.z, co.w, r1.z, r1.w);
        float id = 0.f;
        if (ID_MODE == 1) s_id[t] = g;
        if (ID_MODE == 3) id = __uint_as_float(g);
        if (ID_MODE == 2) {
            const uint32_t r01 = __float_as_uint(r2.z), r23 = __float_as_uint(r2.w);
            const uint32_t x0 = r01 & 0xffffu, y0 = r01 >> 16, x1 = r23 & 0xffffu;
            id = __uint_as_float(__float_as_uint(r2.y) + ((uint32_t)(tile / cam.tiles_x) - y0) * (x1 - x0) +
                                 ((uint32_t)(tile % cam.tiles_x) - x0));
        }
        if (WITH_RGB) s.r2[t] = make_float4(r1.z, r1.w, r2.x, id);
        if (GIVEN) {
            sub_mask = given;
        } else {
            const float4 ell = rec[3];
            sub_mask = SubTiles::from_grid(strip_mask(ell, xy.x - (float)((tile % cam.tiles_x) * TILE), xy.y - (float)((tile / cam.tiles_x) * TILE)));
        }
    }
    reinterpret_cast<uint16_t*>(s.sub)[s.sub_place(t)] = (uint16_t)sub_mask;
    uint32_t pad = 0x01010101u * (uint32_t)(N - 1);
    asm volatile("" : "+v"(pad));   // (formed here: kept for the next batch, four copies of it spill registers of k_render_bwd)
    if (N == 256 || t < N) reinterpret_cast<uint4*>(s.list)[t] = make_uint4(pad, pad, pad, pad);
    __syncthreads();
    // lane i of the row that owns sub-tile st expands slots [16 i, 16 i + 16)
    const int st = swave * 4 + (lane >> 4);
    const int i = lane & 15;
    const uint4 lo = *reinterpret_cast<const uint4*>(&s.sub[8 * i]), hi = *reinterpret_cast<const uint4*>(&s.sub[8 * i + 4]);
    auto bits_of = [&](uint32_t word, int q) { return ((word >> st) & 0x00010001u) << q; };
    const uint32_t both = bits_of(lo.x, 0) | bits_of(lo.y, 1) | bits_of(lo.z, 2) | bits_of(lo.w, 3) | bits_of(hi.x, 4) |
                          bits_of(hi.y, 5) | bits_of(hi.z, 6) | bits_of(hi.w, 7);
    uint32_t b16 = (both & 0xffu) | (both >> 16) << 8;
    if (REVERSED && !GIVEN) b16 &= (1u << min(max(row_end - 16 * i, 0), 16)) - 1u;
    const uint32_t cnt = __popc(b16);
    uint32_t inc = cnt;
    inc = dpp_shr_add<0x111>(inc);  // row_shr:1
    inc = dpp_shr_add<0x112>(inc);  // row_shr:2
    inc = dpp_shr_add<0x114>(inc);  // row_shr:4
    inc = dpp_shr_add<0x118>(inc);  // row_shr:8
    const int mine = __shfl((int)inc, (lane & 48) | 15, 64);
    uint8_t* dst = reinterpret_cast<uint8_t*>(s.list[st]) + (REVERSED ? mine - 1 - (int)(inc - cnt) : (int)(inc - cnt));
    while (b16) {
        *dst = (uint8_t)(16 * i + __builtin_ctz(b16));
        dst += REVERSED ? -1 : 1;
        b16 &= b16 - 1u;
    }
    if (i == 15) s.len[st] = mine;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    return mine;
}

// One step of a sum (three doubles) and a minimum / maximum (bit patterns of non-negative floats, which order like
// unsigned integers) over the lanes of a wavefront: every lane combines its values with those of the lane the DPP
// control names; a lane without such a source (the start of a row, a row the mask leaves out) adds zero and keeps
// its extrema.  SHIFT: a shift within the rows (all rows take part, a missing source reads as zero).
template <int CTRL, int ROW_MASK, bool SHIFT>
__device__ __forceinline__ void wave_step(double& a, double& b, double& c, uint32_t& lo, uint32_t& hi)
{
    auto moved = [](double v) {
        const long long bits = __double_as_longlong(v);
        const int l = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)bits, CTRL, ROW_MASK, 0xF, SHIFT);
        const int h = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)((unsigned long long)bits >> 32), CTRL, ROW_MASK, 0xF, SHIFT);
        return __longlong_as_double((long long)(((unsigned long long)(uint32_t)h << 32) | (uint32_t)l));
    };
    a += moved(a);
    b += moved(b);
    c += moved(c);
    // (the minimum must not meet the zero a missing source reads as: its own value stands in)
    lo = min(lo, (uint32_t)__builtin_amdgcn_update_dpp((int)lo, (int)lo, CTRL, ROW_MASK, 0xF, false));
    hi = max(hi, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, CTRL, ROW_MASK, 0xF, SHIFT));
}

// Conditions are kept as one bit per lane of the wavefront (the scalar unit combines them).
__device__ __forceinline__ uint64_t ballot(bool v) { return __builtin_amdgcn_ballot_w64(v); }
__device__ __forceinline__ bool lane_of(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

// One list entry in the lanes of `mask`: those that it leaves at Tn >= T_min blend it (C += w c, T = Tn, last = at), the others come
// back in `stop`.  HITS: returns the lanes that blended with w > hit_above.  Under the lane mask this is six (seven) vector
// instructions, where selects would take more, with no branch in the way of the instructions around them; the comparison narrows
// the mask itself, so that no scalar instruction stands between it and what depends on it.  Whichever lanes are active stay so:
// the mask is taken out of them and they are put back.  (Outputs are written before all inputs have been read: they share no
// registers.  `hits` is read by a vector instruction behind at least two others: it is written early.)
// BLENDS: `history` moves up by one bit, and its lowest says whether the lane blended (whatever lanes are active).
template <bool HITS, bool BLENDS>
__device__ __forceinline__ uint64_t blend_under_mask(uint64_t mask, float& C0, float& C1, float& C2, float& T, int& last, float c0, float c1,
                                                     float c2, float w, float Tn, float T_min, float hit_above, int at, uint64_t& stop, uint32_t& history)
{
    uint64_t active, hits;
#define FS_BLEND(COUNT, SHIFT)                                                                                                        \
    asm("s_and_saveexec_b64 %[active], %[m]\n\t"                                                                               \
        "v_cmpx_ngt_f32_e32 vcc, %[T_min], %[Tn]\n\t"                                                                          \
        "v_mov_b32_e32 %[T], %[Tn]\n\t" COUNT                                                                                  \
        "v_fmac_f32_e32 %[C0], %[c0], %[w]\n\t"                                                                                \
        "v_fmac_f32_e32 %[C1], %[c1], %[w]\n\t"                                                                                \
        "v_fmac_f32_e32 %[C2], %[c2], %[w]\n\t"                                                                                \
        "v_mov_b32_e32 %[l], %[at]\n\t"                                                                                        \
        "s_andn2_b64 %[stop], %[m], vcc\n\t"                                                                                   \
        "s_mov_b64 exec, %[active]" SHIFT                                                                                      \
        : [C0] "+&v"(C0), [C1] "+&v"(C1), [C2] "+&v"(C2), [T] "+&v"(T), [l] "+&v"(last), [active] "=&s"(active), [stop] "=&s"(stop), \
          [hits] "=&s"(hits), [h] "+&v"(history)                                                                               \
        : [m] "s"(mask), [c0] "v"(c0), [c1] "v"(c1), [c2] "v"(c2), [w] "v"(w), [Tn] "v"(Tn), [T_min] "s"(T_min), [at] "s"(at), \
          [hit_above] "v"(hit_above)                                                                                           \
        : "scc", "vcc");
#define FS_HISTORY "\n\tv_addc_co_u32_e32 %[h], vcc, %[h], %[h], vcc"
    if (HITS && BLENDS) { FS_BLEND("v_cmp_gt_f32_e64 %[hits], %[w], %[hit_above]\n\t", FS_HISTORY) }
    else if (HITS) { FS_BLEND("v_cmp_gt_f32_e64 %[hits], %[w], %[hit_above]\n\t", "") }
    else if (BLENDS) { FS_BLEND("", FS_HISTORY) }
    else { FS_BLEND("", "") }
#undef FS_HISTORY
#undef FS_BLEND
    return hits;
}

// v with `value` (uniform) in lane `at`: the instruction v_writelane_b32, for which this compiler has no builtin.
extern "C" __device__ uint32_t fs_write_lane(uint32_t value, uint32_t at, uint32_t v) __asm("llvm.amdgcn.writelane.i32");

// Longest of the four sub-tile lists of the calling wavefront (`mine` is uniform within a row).
__device__ __forceinline__ int wave_max_of_rows(int mine)
{
    const int a = __builtin_amdgcn_readlane(mine, 0), b = __builtin_amdgcn_readlane(mine, 16);
    const int c = __builtin_amdgcn_readlane(mine, 32), d = __builtin_amdgcn_readlane(mine, 48);
    // (read back through a scalar register: a loop bound the compiler knows to be uniform is counted by the scalar unit)
    return __builtin_amdgcn_readfirstlane(max(max(a, b), max(c, d)));
}

// FUSED: the epilogue also does, per pixel, what the L1 term (FastGS Sec. 4.5) and the error map of the
// multi-view score (Sec. 4.2) need from the finished colour -- dL/dC = sign(C - target) * scale, the error
// e = ((|d0| + |d1|) + |d2|) / 3 -- and leaves this tile's partial sums (sum of |d|; sum, min, max and sum of squares
// of e) at tile_partial[q * num_tiles + tile], so that the image is not read again for them.
//
// BITS: the kernel also records, for every pair of the tile's list (by its position in the sorted order), at which
// of the tile's 256 pixels the Gaussian is counted by the multi-view score (Sec. 4.2): where it is blended and, in
// FS_SCORE_WEIGHT mode, alpha T > alpha_min.  32 bytes per pair: 16 sub-tiles (index wave*4 + row) x 16 bits (lane
// within the row); only the rows with a bit set are written, packed at the start of the tile's segment, each with its Gaussian.
// With these the count pass is a population count per pair instead of a second walk over the lists (k_score_bits).
//
// BLENDS: the kernel notes the pairs it blends anywhere, and in which sub-tiles, for k_render_bwd (BlendRecord).  Each lane shifts one
// bit per entry into a register; every 32 places the 16 lanes of a row put theirs together and name the slots (history_to_slots).
// It costs 4 to 7 us at 300k and 500k Gaussians, 14 at 3 M, and saves k_render_bwd more: see there.
//
// (80 registers: with two more, where the compiler goes by itself, a SIMD holds five wavefronts instead of six, and the kernel with the
// record takes 129 us instead of 119 at 500k Gaussians and 1600x1064.)
template <bool FUSED, bool BITS, bool BLENDS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_num_vgpr(80))) void k_render_fwd(CamDev cam, CfgDev cfg, const uint2* __restrict__ ranges,
                                                    const uint32_t* __restrict__ tile_order,
                                                    const uint32_t* __restrict__ gauss_sorted,
                                                    const float4* __restrict__ splats, float* __restrict__ image,
                                                    float* __restrict__ final_T, uint32_t* __restrict__ n_contrib,
                                                    const float* __restrict__ target, float scale,
                                                    float* __restrict__ dL, float* __restrict__ err,
                                                    double* __restrict__ tile_partial, ScoreRecord record, BlendRecord blends)
{
    __shared__ Stage<true> s;
    __shared__ __align__(16) uint16_t s_pb[BITS ? SLOTS : 1][16];  // this batch's bits, [slot][sub-tile]
    __shared__ uint32_t s_blend[BLENDS ? 2 : 1][BLENDS ? SLOTS / 2 : 1];   // sub-tiles that blended a slot's pair (16 bits), this batch's and the one's before
    __shared__ uint32_t s_rows;                                    // rows of the record this tile has written so far
    __shared__ __align__(16) int s_alive[4];                       // whether a wavefront has pixels that go on

    const int tile = (int)tile_order[blockIdx.x];  // longest lists first
    const int sub = (threadIdx.x >> 6) * 4 + ((threadIdx.x & 63) >> 4);  // this lane's sub-tile list
    const Pixel p = pixel_of_thread(cam, tile);
    const uint2 range = ranges[tile];
    const int total = (int)(range.y - range.x);

    uint64_t done = ballot(!p.inside);   // the wavefront's pixels that have terminated
    float T = 1.0f, C0 = 0.f, C1 = 0.f, C2 = 0.f;
    uint32_t last = 0;

    s.clear(threadIdx.x);

    // BITS: row t of s_pb is zeroed and written out by thread t alone; the other wavefronts set bits in it between
    // a batch's staging barriers and the barrier at the top of the next batch
    const float hit_above = cfg.score_mode == FS_SCORE_ALPHA ? 0.0f : cfg.alpha_min;
    int pending_m = 0;  // length of the batch whose bits are in s_pb and not yet in memory (uniform; 0: none)
    if (BITS && threadIdx.x == 0) s_rows = 0;   // (the first use lies behind the barrier at the top of the second batch)
    auto entry = [&](int start) {   // the Gaussian of this thread's slot of the batch that starts there
        const int i = start + (int)threadIdx.x;
        return i < total && threadIdx.x < BATCH ? gauss_sorted[range.x + i] : 0u;
    };
    uint32_t g_next = entry(0);
    auto g_here = [&](uint32_t t) { return __float_as_uint(s.r2[t].w); };   // the Gaussian of slot t, until the next batch is staged
    auto write_bits = [&](int count) {
        // A pair that is counted nowhere (at 500k Gaussians half of them: the rectangle's corners, entries behind the
        // last blended one) leaves nothing.  The others' rows are packed at the start of the tile's segment: a
        // wavefront reserves as many places as it has rows with one LDS atomic, so the order of the rows within the
        // tile depends on which wavefront comes first (the count pass adds integers: its result does not).
        uint4 lo = make_uint4(0u, 0u, 0u, 0u), hi = lo;
        if ((int)threadIdx.x < count) {
            const uint4* row = reinterpret_cast<const uint4*>(s_pb[threadIdx.x]);
            lo = row[0];
            hi = row[1];
        }
        const bool any = ((lo.x | lo.y) | (lo.z | lo.w) | (hi.x | hi.y) | (hi.z | hi.w)) != 0u;
        const uint64_t bal = __ballot(any);
        if (bal != 0) {   // (uniform over the wavefront)
            uint32_t base = 0;
            if ((threadIdx.x & 63) == 0) base = atomicAdd(&s_rows, (uint32_t)__popcll(bal));
            base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
            if (any) {
                const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
                const size_t at = (size_t)range.x + base + below;
                // (streaming stores: the record is read once, by the count pass, and should not displace the step's
                // other arrays from the caches)
                nt_store(lo, record.rows + at * 2);
                nt_store(hi, record.rows + at * 2 + 1);
                record.row_gauss[at] = g_here(threadIdx.x);
            }
        }
    };
    // BLENDS: the pairs of the batch before that were blended, in order behind those of earlier batches: every wavefront looks at all
    // slots' words, so that it knows how many stand before its own.
    int blended = 0, batch = 0;
    auto write_blends = [&](int batch_start) {
        const uint16_t* const words = reinterpret_cast<const uint16_t*>(s_blend[(batch & 1) ^ 1]);
        uint32_t t = threadIdx.x;
        asm volatile("" : "+v"(t));   // (as in history_to_slots)
        const uint32_t mine = words[t];
        int before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < SLOTS / 64; w++) {
            const int count = __popcll(ballot(words[64 * w + ((int)t & 63)] != 0));
            before += w < (int)(t >> 6) ? count : 0;
            all += count;
        }
        const uint64_t bal = ballot(mine != 0u);
        if (mine != 0u) {
            const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            blends.entries[(size_t)range.x + (uint32_t)(blended + before) + below] = make_uint2(g_here(t), (uint32_t)(batch_start + (int)t) | mine << 16);
        }
        blended += all;
    };
    int start = 0;
    for (; start < total; start += BATCH) {
        // (before the first batch nothing has been written that another thread reads; __syncthreads_or is two barriers and a reduction for
        // any shape of workgroup)
        int alive = 1;
        if (start > 0) {
            if ((threadIdx.x & 63) == 0) s_alive[threadIdx.x >> 6] = done != ~0ull;
            __syncthreads();
            const int4 a = *reinterpret_cast<const int4*>(s_alive);
            alive = __builtin_amdgcn_readfirstlane((a.x | a.y) | (a.z | a.w));
        }
        if (BITS && pending_m > 0) {
            write_bits(pending_m);
            pending_m = 0;
        }
        if (BLENDS) {
            // (the words about to be cleared were read behind the barrier before the one inside the batch before)
            if (start > 0) write_blends(start - BATCH);
            if (threadIdx.x < SLOTS / 2) s_blend[batch & 1][threadIdx.x] = 0u;
        }
        if (alive == 0) break;
        const int m = min(BATCH, total - start);
        if (BITS) {
            uint4* row = reinterpret_cast<uint4*>(s_pb[threadIdx.x]);
            row[0] = make_uint4(0u, 0u, 0u, 0u);
            row[1] = make_uint4(0u, 0u, 0u, 0u);
            pending_m = m;
        }
        const int mine = stage_batch<BITS || BLENDS ? 3 : 0>(s, nullptr, cam, tile, splats, g_next, m);
        g_next = entry(start + BATCH);   // (its latency passes during the walk)
        // a row whose 16 pixels have all finished does not lengthen the wavefront's loop
        const bool row_alive = ((~done >> (threadIdx.x & 48)) & 0xffffull) != 0;
        const int longest = wave_max_of_rows(row_alive ? mine : 0);
        // What weighs in the loop is the number of vector instructions where the chip is full (a SIMD takes one of this mixture in
        // 2.3 cycles at best; over the whole kernel one takes 3.3 to 4.0 at bench.py's 3 M and 500k Gaussians), and the latency of one trip where the longest tiles are left
        // alone (4.5 to 6 cycles for every instruction, scalar ones included).  Four
        // entries' alphas are formed side by side from one word of slots -- four independent chains -- and only the
        // transmittance runs through them one after the other; conditions are lane masks in the scalar unit and blending
        // happens under the mask instead of through selects: a trip of four entries has 125 vector and 35 scalar instructions, the
        // loop's own included, and six waits; 138 and 41 with the record of counted pixels, 130 and 37 with that of blended pairs, 143
        // and 41 with both.  Lanes past their list's end evaluate the empty record.  The four records are requested ahead of all arithmetic, in the order of their use: with both
        // records the compiler by itself places each request before its use (100k Gaussians: 60 us instead of 49, 3 M: 292 and 271).
        // The record: each entry's 64 bits go into one lane of two registers, and 64 entries later to the slots' rows; stored
        // entry by entry they took a 64-bit shift, an address, an LDS store and a change of the lane mask each.  Both steps together,
        // before and after, kernel durations in us, with the record: 4k Gaussians at 128x128 18.7 and 16.9, 100k at 980x545 54.8 and
        // 50.0, 500k at 1600x1064 124.5 and 117.3, 3 M at 1920x1080 276 and 265; without it: 4k 13.4 and 12.2, 12k at 509x337 17.7 and
        // 17.3, 300k at 1332x876 (two scenes) 68.3 and 68.6, 64.3 and 65.7, 500k 88.4 and 88.4.
        // (Skipping an entry when no lane passes the range test does not pay: four rows look at four different
        // Gaussians, so all of them missing is rare.)
        int lastk = -1;   // place on the row's list of the last Gaussian this pixel blended in this batch
        uint32_t next = s.list[sub][0];
        uint32_t hits_lo = 0, hits_hi = 0;   // BITS: lane l holds the pixels counted for place l of the four rows' lists, 64 places at a time
        // the pixels counted for places [k0, k0 + 64), to their slots' rows
        auto hits_to_rows = [&](int k0) {
            const int k = k0 + ((int)threadIdx.x & 63), first = sub & 12;
            if (k < longest) {
#pragma unroll
                for (int r = 0; r < 4; r++) s_pb[s.slot(first + r, k)][first + r] = (uint16_t)((r < 2 ? hits_lo : hits_hi) >> (16 * (r & 1)));
            }
            hits_lo = hits_hi = 0;
        };
        // BLENDS: bit 31 - j of `history` says whether this lane blended place k0 + j of its row's list (places being how many it holds);
        // the row's 16 lanes together name the places, two for each lane, whose slots its sub-tile blended
        uint32_t history = 0;
        auto history_to_slots = [&](int k0, int places) {
            uint32_t h = history << (32 - places);
            h |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h, 0x128, 0xF, 0xF, true);   // row_ror:8, 4, 2, 1
            h |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h, 0x124, 0xF, 0xF, true);
            h |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h, 0x122, 0xF, 0xF, true);
            h |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h, 0x121, 0xF, 0xF, true);
            uint32_t t = threadIdx.x;
            asm volatile("" : "+v"(t));   // (what follows from it is formed here: kept through the trips it takes registers, and with them a wavefront)
            const int i = (int)(t & 15u), st = (int)(t >> 4);
            const int j0 = s.slot(st, k0 + i), j1 = s.slot(st, k0 + 16 + i);
            if (h >> (31 - i) & 1u) atomicOr(&s_blend[batch & 1][j0 >> 1], 1u << (st + 16 * (j0 & 1)));
            if (h >> (15 - i) & 1u) atomicOr(&s_blend[batch & 1][j1 >> 1], 1u << (st + 16 * (j1 & 1)));
            history = 0;
        };
        auto trip = [&](uint32_t k) {
            const uint32_t word = next;
            float alpha[GROUP], cb[GROUP];
            float4 r0[GROUP], r1[GROUP];
            uint64_t ok[GROUP];
#pragma unroll
            for (int u = 0; u < GROUP; u++) {
                const int j = (word >> (8 * u)) & 0xffu;
                r0[u] = s.r0[j];
                r1[u] = s.r1[j];
                cb[u] = s.r2[j].z;
                if (BITS) __builtin_amdgcn_sched_barrier(0);
            }
            next = s.list[sub][k / GROUP + 1];   // (one past the list's end is still in `s`, and not looked at)
            if (BITS) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < GROUP; u++) {
                const float dx = p.px - r0[u].x, dy = p.py - r0[u].y;
                const float h = __builtin_fmaf(r0[u].w, dy, r0[u].z * dx);
                const float t = exponent_of(__builtin_fmaf(dx, h, (r1[u].x * dy) * dy));
                alpha[u] = fminf(cfg.alpha_max, r1[u].y * exp_c(t));
                ok[u] = takes_part_mask(t) & ballot(alpha[u] >= cfg.alpha_min);
            }
#pragma unroll
            for (int u = 0; u < GROUP; u++) {
                const float Tn = T * (1.0f - alpha[u]), w = alpha[u] * T;
                // w is alpha T with the transmittance in front of this Gaussian: where it is blended, w > alpha_min
                // (FS_SCORE_WEIGHT) or w > 0 (FS_SCORE_ALPHA, always) decides
                uint64_t stop;
                const uint64_t hb = blend_under_mask<BITS, BLENDS>(ok[u] & ~done, C0, C1, C2, T, lastk, r1[u].z, r1[u].w, cb[u], w, Tn, cfg.T_min,
                                                                   hit_above, (int)k + u, stop, history);
                done |= stop;
                if (BITS) {
                    hits_lo = fs_write_lane((uint32_t)hb, (k + u) & 63u, hits_lo);
                    hits_hi = fs_write_lane((uint32_t)(hb >> 32), (k + u) & 63u, hits_hi);
                }
            }
        };
        // places [k, end), or until all of the wavefront's pixels have terminated; returns where the next trip would start
        auto trips = [&](int k, int end) {
            do {
                trip((uint32_t)k);
                k += GROUP;
                if (done == ~0ull) break;
            } while (k < end);
            return k;
        };
        if (BLENDS || BITS) {
            // as many places at a time as the record's registers hold
            constexpr int SPAN = BLENDS ? 32 : 64;
            int k = 0;
            while (k < longest && done != ~0ull) {
                const int k0 = k;
                k = trips(k0, min(longest, k0 + SPAN));
                if (BLENDS) history_to_slots(k0, k - k0);
                if (BITS && (SPAN == 64 || (k0 & 32))) hits_to_rows(k0 & ~63);
            }
            if (BITS && SPAN == 32 && k != 0 && ((k - 1) & 32) == 0) hits_to_rows((k - 1) & ~63);
            batch++;
        } else if (longest > 0 && done != ~0ull) {
            trips(0, longest);
        }
        last = lastk >= 0 ? (uint32_t)(start + s.slot(sub, lastk) + 1) : last;
    }
    if (BLENDS) {
        if (start >= total && total > 0) {   // (the last batch has been walked; a break above comes behind its words)
            __syncthreads();
            write_blends(start - BATCH);
        }
        if (threadIdx.x == 0) blends.tile_count[tile] = blended;
    }
    if (BITS) {
        if (pending_m > 0) {
            if (!BLENDS) __syncthreads();
            write_bits(pending_m);
        }
        // (pairs the loop never reached -- every pixel had finished -- are blended nowhere and leave no row)
        __syncthreads();
        if (threadIdx.x == 0) record.tile_rows[tile] = (int32_t)s_rows;
    }
    double l1 = 0.0, esum = 0.0, esq = 0.0, emin = 1.0e300, emax = -1.0e300;
    if (p.inside) {
        const size_t hw = (size_t)cam.width * cam.height;
        const size_t pix = (size_t)p.y * cam.width + p.x;
        const float c0 = __builtin_fmaf(T, cfg.bg[0], C0), c1 = __builtin_fmaf(T, cfg.bg[1], C1);
        const float c2 = __builtin_fmaf(T, cfg.bg[2], C2);
        image[pix] = c0;
        image[hw + pix] = c1;
        image[2 * hw + pix] = c2;
        final_T[pix] = T;
        n_contrib[pix] = last;
        if (FUSED) {
            const float d0 = c0 - target[pix], d1 = c1 - target[hw + pix], d2 = c2 - target[2 * hw + pix];
            if (dL) {
                dL[pix] = d0 > 0.f ? scale : (d0 < 0.f ? -scale : 0.f);
                dL[hw + pix] = d1 > 0.f ? scale : (d1 < 0.f ? -scale : 0.f);
                dL[2 * hw + pix] = d2 > 0.f ? scale : (d2 < 0.f ? -scale : 0.f);
            }
            const float e = ((fabsf(d0) + fabsf(d1)) + fabsf(d2)) / 3.0f;
            err[pix] = e;
            l1 = ((double)fabsf(d0) + (double)fabsf(d1)) + (double)fabsf(d2);
            esum = emin = emax = (double)e;
            esq = (double)e * (double)e;
        }
    }
    if (FUSED) {
        // per-wavefront partials (sums in double, extrema of the fp32 errors in float: exact) by DPP moves -- four
        // shifts within the rows of 16 lanes, lane 15 of rows 0 and 2 into the row after it, lane 31 into rows 2 and
        // 3 -- which leave the totals in lane 63; combined across the four wavefronts through LDS with a single barrier
        // (errors are >= 0: threads outside the image carry +3e38 for the minimum and 0 for the maximum)
        uint32_t lo_e = __float_as_uint((float)emin == (float)emin && emin < 1.0e299 ? (float)emin : 3.0e38f);
        uint32_t hi_e = __float_as_uint(emax > -1.0e299 ? (float)emax : 0.0f);
        wave_step<0x111, 0xF, true>(l1, esum, esq, lo_e, hi_e);
        wave_step<0x112, 0xF, true>(l1, esum, esq, lo_e, hi_e);
        wave_step<0x114, 0xF, true>(l1, esum, esq, lo_e, hi_e);
        wave_step<0x118, 0xF, true>(l1, esum, esq, lo_e, hi_e);
        wave_step<0x142, 0xA, false>(l1, esum, esq, lo_e, hi_e);
        wave_step<0x143, 0xC, false>(l1, esum, esq, lo_e, hi_e);
        const float fmin_e = __uint_as_float(lo_e), fmax_e = __uint_as_float(hi_e);
        // (the staging masks serve as the 4 x 5 doubles of scratch: they are only live inside stage_batch)
        static_assert(sizeof(s.sub) >= 4 * 5 * sizeof(double), "scratch for the per-wavefront partials");
        __syncthreads();
        double (*s_part)[5] = reinterpret_cast<double (*)[5]>(s.sub);
        if ((threadIdx.x & 63) == 63) {
            double* w = s_part[threadIdx.x >> 6];
            w[0] = l1; w[1] = esum; w[2] = (double)fmin_e; w[3] = (double)fmax_e; w[4] = esq;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            const size_t nt = (size_t)cam.tiles_x * cam.tiles_y;
            tile_partial[tile] = (s_part[0][0] + s_part[1][0]) + (s_part[2][0] + s_part[3][0]);
            tile_partial[nt + tile] = (s_part[0][1] + s_part[1][1]) + (s_part[2][1] + s_part[3][1]);
            tile_partial[2 * nt + tile] = fmin(fmin(s_part[0][2], s_part[1][2]), fmin(s_part[2][2], s_part[3][2]));
            tile_partial[3 * nt + tile] = fmax(fmax(s_part[0][3], s_part[1][3]), fmax(s_part[2][3], s_part[3][3]));
            tile_partial[4 * nt + tile] = (s_part[0][4] + s_part[1][4]) + (s_part[2][4] + s_part[3][4]);
        }
    }
}

// ---- backward ---------------------------------------------------------------------------------
// Walks each sub-tile's list back to front from the furthest blended Gaussian.  Per (Gaussian, pixel) two numbers are left:
// w = alpha T and v = G dL/dalpha.  Everything a Gaussian receives from a sub-tile is a sum over its 16 pixels of one of
// them times something that belongs to the pixel alone: w times the pixel's dL/dC (3 sums), and v times the pixel's place,
// {1, x, y, x^2, x y, y^2} (dL/dsigma, and the moments from which dL/dconic and dL/dmu_2D follow).
//
// Vector instructions weigh most in this kernel, and forming nine products per pixel and adding them up
// across a row's 16 lanes took half of them.  So the numbers change places first: after eight entries of every row's list a
// wavefront writes its 8 x 64 w's (then its v's) to LDS and reads them back with the 32 (entry, row) combinations across its
// lanes, two lanes to a combination and eight pixels to a lane.  The sums over pixels are then plain additions within a
// lane -- separable ones for the moments, since x and y take four values each -- plus one exchange between the two lanes:
// 12 instructions per entry instead of 41.  (The matrix cores do not help: v_mfma_f32_16x16x4_f32 keeps the vector unit
// from issuing for its 32 cycles, and forms many sums nobody wants; measured between the two.)
// Before and after, in us: 4k Gaussians at 128x128 41 and 30, 100k at 980x545 119 and 82, 500k at 1600x1064 308 and 245 (with
// ABS 336 and 262), 3 M at 1920x1080 730 and 565.
//
// Places are relative to mu itself, as one subtraction per column and line: a line's sums of v, v dx, v dx^2, then dy and dy^2
// times those.  (Sums about the sub-tile's centre, shifted to mu afterwards, take 8 of the 48 instructions per exchange less
// and cancel: 3 to 9 times the rounding error for splats below two pixels.)  The flush works in double and rounds once.
// Measured against exact sums on splats with a tile to themselves, dL/dconic: 8.2e-8 at the low-pass floor (5.6e-7 with the
// shift, 8.6e-8 with products per pixel added over 16 lanes), 8.8e-8 at eigenvalues 2 and 4 (1.6e-7, 9.5e-8).
//
// Every Gaussian-tile pair owns one record of PAIR_REC floats in `pair_grad`, at the position the
// pair had when it was emitted (pair_offsets[g] + its place in g's tile rectangle): the flush is a
// plain store (rgb 3, sigma, conic 3, mu_2D 2), every pair of the tile is written exactly once (zeros
// for the ones nothing blended), and the per-Gaussian sum over its contiguous records is left to the
// projection's backward kernel.  No global atomics.  The only sums whose order depends on scheduling are those of a
// Gaussian's (up to 16) sub-tile totals within a tile, taken in double precision in LDS: the record is the same from
// run to run unless the exponents of those terms span more than 29 bits.
//
// What else shapes the inner loop is what this chip's vector unit and LDS do with an instruction (measured, in cycles of one SIMD):
// it takes them from two wavefronts at a time, 2.2 to 2.6 each, as long as one in two is a plain addition, product or multiply-add of
// vector registers (4.4 in an unbroken run of comparisons, minima, selects, shifts, conversions or operations with a scalar
// operand); an exponential or a reciprocal (8.4), a data-parallel move, a permutation of the lanes or a read of one lane (4.3) ends that
// for some sixteen instructions after it (one in 16: 4.2 on average, one in 32: 3.6), wherever it stands: so they stand
// together (the reciprocals of four entries, the exchange between
// the two lanes).  An LDS add of doubles takes 8 cycles of its compute unit where all lanes name places of their own, 44 where
// four lanes name each: the adds were a seventh of the kernel, and now rows take turns (see there).  ABS needs no more exchanges:
// its sums are formed behind the one of the v's.  Together, before and after, kernel durations in us: 500k Gaussians at 1600x1064 224
// and 207, 3 M at 1920x1080 512 and 484, 100k at 980x545 74.5 and 70.5; with ABS 245 and 216 (500k, Compact Box), 170 and 152 (300k at
// 1332x876).
// PACKED: the walk goes over the pairs that the forward pass noted as blended, each with its exact sub-tiles (BlendRecord), instead of the
// whole list with every sub-tile that a pair's support reaches.  That leaves out pairs behind opaque ones or beside all pixels, half of
// the list up to the furthest blended pair at 3 M Gaussians and three quarters with a tail of large splats: fewer batches to stage, a tenth to two
// fifths fewer trips.  Kernel durations, whole lists and PACKED, us: 500k Gaussians at 1600x1064 188 and 165, 3 M at 1920x1080 460 and 380,
// 100k at 980x545 61 and 50, 12k at 509x337 33 and 28, 300k at 1332x876 140 and 131, 4k at 128x128 22.3 and 20.8.
//
// A trip of eight entries has about 415 vector instructions (without needles), which at these rates would take a SIMD 1 050
// cycles, 2.55 for each; over the whole kernel one takes 4.1 to 4.8 at bench.py's 3 M (wide) and 500k Gaussians.  What the other two
// fifths are spent on (the LDS adds and exchanges, their waits, wavefronts that end early) has not been taken apart.
//
// ABS adds the absolute positional gradient (used by FastGS for the split decision): per pixel the
// magnitudes |dL/dmu_x|, |dL/dmu_y| of its own contribution, summed like the other values and stored
// in the record's floats 9 and 10.
template <bool ABS, bool SPARSE, bool PACKED>
__global__ __launch_bounds__(256, 4) void k_render_bwd(
    CamDev cam, CfgDev cfg, const uint2* __restrict__ ranges, const uint32_t* __restrict__ tile_order,
    const uint32_t* __restrict__ gauss_sorted,
    const float4* __restrict__ splats, const float* __restrict__ final_T, const uint32_t* __restrict__ n_contrib,
    const float* __restrict__ dL_dimage, float4* __restrict__ pair_grad, uint8_t* __restrict__ rec_valid, BlendRecord blends)
{
    // (as many slots as four workgroups of a compute unit's 160 KB of LDS leave room for)
    constexpr int N = ABS ? 208 : 232, B = N - 1;
    constexpr int NV = ABS ? 11 : 9;
    constexpr int HALF = ABS ? 6 : 4;   // sums 0 .. HALF - 1 are added by the first lane of a combination, the others by the second
    enum { DR, DG, DB, DSIGMA, DABS_X, DABS_Y, DX = HALF, DY, DXX, DYY, DXY };
    constexpr int SPAN = 2 * GROUP;     // entries per exchange
    // The sub-tiles' sums of a Gaussian meet in double precision: on this chip the LDS atomic add of a double is
    // markedly cheaper than that of a float, and the
    // sum of up to 16 single-precision terms is then exact unless their exponents span more than 29 bits.
    typedef double acc_t;
    __shared__ Stage<true, N> s;
    __shared__ acc_t s_acc[N][NV];
    __shared__ __align__(16) float s_turn[4][SPAN][64];   // per wavefront: one value of SPAN entries, [entry][lane]
    __shared__ uint16_t s_pos[PACKED ? N : 1];            // the slots' positions in the tile's list
    static_assert(sizeof(s) + sizeof(s_acc) + sizeof(s_turn) + sizeof(s_pos) <= 40960, "four workgroups per compute unit");

    const int tile = (int)tile_order[blockIdx.x];  // longest lists first
    const Pixel p = pixel_of_thread(cam, tile);
    const uint2 range = ranges[tile];
    const size_t hw = (size_t)cam.width * cam.height;
    const size_t pix = (size_t)p.y * cam.width + p.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sub = wave * 4 + (lane >> 4);

    const int last = p.inside ? (int)n_contrib[pix] : 0;
    float T = p.inside ? final_T[pix] : 0.f;
    float dC0 = 0.f, dC1 = 0.f, dC2 = 0.f;
    if (p.inside) {
        dC0 = dL_dimage[pix];
        dC1 = dL_dimage[hw + pix];
        dC2 = dL_dimage[2 * hw + pix];
    }
    // dC . (colour composited behind the Gaussian at hand): all that dL/dalpha = T (dC . c - S) needs of it
    float S = __builtin_fmaf(dC2, cfg.bg[2], __builtin_fmaf(dC1, cfg.bg[1], dC0 * cfg.bg[0]));

    // After the exchange this lane has entry `ent` of row `row`: lines q1 and q2 (of four pixels each) of the row's sub-tile;
    // the lane 8 places on in its group of 16 has the other two.  Which lane takes which lines is laid out so
    // that any eight neighbouring lanes' 16-byte reads fall into different banks.
    const int row = lane & 3, ent = (lane >> 2 & 1) | (lane >> 4) << 1;
    const bool second = lane & 8;
    const int q1 = ((lane >> 3 ^ lane >> 2) & 1) + (row & 2), q2 = q1 ^ 2;
    const int sub_x = (tile % cam.tiles_x) * TILE + (wave & 1) * 8 + (row & 1) * 4;
    const int sub_y = (tile / cam.tiles_x) * TILE + (wave >> 1) * 8 + (row >> 1) * 4;
    float g1[3][4], g2[3][4];   // the lines' dL/dC
#pragma unroll
    for (int ch = 0; ch < 3; ch++)
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const int x = sub_x + c;
            g1[ch][c] = x < cam.width && sub_y + q1 < cam.height ? dL_dimage[ch * hw + (size_t)(sub_y + q1) * cam.width + x] : 0.f;
            g2[ch][c] = x < cam.width && sub_y + q2 < cam.height ? dL_dimage[ch * hw + (size_t)(sub_y + q2) * cam.width + x] : 0.f;
        }
    const float px0 = (float)sub_x + 0.5f;   // centres of the first column, of the lines
    const float py1 = (float)(sub_y + q1) + 0.5f, py2 = (float)(sub_y + q2) + 0.5f;
    const uint8_t* const ent_list = reinterpret_cast<const uint8_t*>(s.list[wave * 4 + row]) + ent;
    float* const turn = &s_turn[wave][0][lane];
    const float4* const turned = reinterpret_cast<const float4*>(&s_turn[wave][0][0]) + ent * 16 + row * 4;
    // (a wavefront's LDS operations complete in the order they were issued)
    auto exchange = [&](const float (&v)[SPAN], float4& l1, float4& l2) {
#pragma unroll
        for (int u = 0; u < SPAN; u++) turn[u * 64] = v[u];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        l1 = turned[q1];
        l2 = turned[q2];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    auto column = [&](int c) {   // (formed where it is used: kept, the four of them spill registers of the ABS kernel)
        float x = px0;
        asm volatile("" : "+v"(x));
        return x + (float)c;
    };
    auto other = [](float v) {   // what the other lane of the combination has
        constexpr int ROR8 = 0x128;
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ROR8, 0xF, 0xF, true));
    };
    auto both = [&](float v) { return v + other(v); };   // the sum of the two lanes, in both

    s.clear(threadIdx.x);
    int row_last = last, total;
    if (PACKED) {
        total = blends.tile_count[tile];
    } else {
        // the furthest position any pixel of this lane's row of 16 reaches (by rotations of the row: every lane has it)
        auto rotated_max = [&](auto ctrl) {
            row_last = max(row_last, __builtin_amdgcn_update_dpp(0, row_last, decltype(ctrl)::value, 0xF, 0xF, true));
        };
        rotated_max(std::integral_constant<int, 0x121>{});
        rotated_max(std::integral_constant<int, 0x122>{});
        rotated_max(std::integral_constant<int, 0x124>{});
        rotated_max(std::integral_constant<int, 0x128>{});
        // (With exchanges through LDS, a maximum added up by LDS atomics and a second barrier for it: 22.9 us instead of 22.3 at 4k Gaussians,
        // 54.6 and 53.8 at 100k, 174.6 and 172.6 at 500k.  s_turn is not in use before the first batch's barriers.)
        int* const wave_last = reinterpret_cast<int*>(&s_turn[0][0][0]);
        const int wave_max = wave_max_of_rows(row_last);
        if (lane == 0) wave_last[wave] = wave_max;
        __syncthreads();
        const int4 furthest = *reinterpret_cast<const int4*>(wave_last);
        total = max(max(furthest.x, furthest.y), max(furthest.z, furthest.w));  // entries at positions >= total are blended by no pixel of the tile
    }

    // batches from the back: batch b covers positions [b*B, min(total,(b+1)*B))
    const int final_start = total > 0 ? ((total - 1) / B) * B : -1;
    // PACKED: of the pairs that the forward pass blended, which come with their sub-tiles and positions
    auto entry = [&](int start) {   // the Gaussian of this thread's slot of the batch that starts there
        const int i = start + (int)threadIdx.x;
        const bool in = start >= 0 && i < total && threadIdx.x < B;
        if constexpr (PACKED) return in ? blends.entries[range.x + i] : make_uint2(0u, 0u);
        else return make_uint2(in ? gauss_sorted[range.x + i] : 0u, 0u);
    };
    uint2 next = entry(final_start);
    for (int start = final_start; start >= 0; start -= B) {
        const int m = min(B, total - start);
        if (start != final_start) __syncthreads();  // the previous batch's flush has read s_acc / s.r2
        if ((int)threadIdx.x < N) {
#pragma unroll
            for (int k = 0; k < NV; k++) s_acc[threadIdx.x][k] = (acc_t)0;
        }
        // (entries behind a row's furthest one are left out of its list)
        if (PACKED && (int)threadIdx.x < N) s_pos[threadIdx.x] = (uint16_t)next.y;
        const int mine = stage_batch<2, true, PACKED>(s, nullptr, cam, tile, splats, next.x, m, row_last - start, next.y >> 16);
        next = entry(start - B);   // (its latency passes during the walk)
        const int longest = wave_max_of_rows(mine);
        uint32_t last_here = (uint32_t)max(last - start, 0);   // slots below this one hold entries this pixel blended (or examined)
        if (PACKED) {
            // (positions ascend with the slots)
            last_here = (uint32_t)m;
            if (ballot((int)s_pos[m - 1] >= last) != 0) {
                last_here = 0;
#pragma unroll
                for (uint32_t step = 128; step > 0; step >>= 1) {
                    const uint32_t to = last_here + step;
                    last_here = to <= (uint32_t)m && (int)s_pos[min(to, (uint32_t)m) - 1] < last ? to : last_here;
                }
            }
        }
        uint64_t acted = 0;   // lanes that blend any of the trip's entries
        // the records of a word's four slots
        float4 r0[GROUP], r1[GROUP];
        float cb[GROUP];
        uint32_t js[GROUP];
        auto fetch = [&](uint32_t word) {
#pragma unroll
            for (int u = 0; u < GROUP; u++) {
                js[u] = (word >> (8 * u)) & 0xffu;
                r0[u] = s.r0[js[u]];
                r1[u] = s.r1[js[u]];
                cb[u] = s.r2[js[u]].z;   // (16 bytes twice and 4 are read faster than 16, 8 and 12)
            }
        };
        float alpha[GROUP], G[GROUP], cd[GROUP], inv[GROUP];
        // The four entries' alphas and what else does not depend on the transmittance, one step of all four after the other: a result
        // is read 8.4 cycles after its instruction was issued, the next independent one is issued after 5.2.  The compiler by itself
        // forms one alpha after the other, each behind the wait for its own record.  Kernel durations before and after, in us: 4k Gaussians
        // at 128x128 23.6 and 22.4, 100k at 980x545 57.5 and 54.4, 12k at 509x337 28.3 and 26.7; where the chip is full 1 to 2 % (500k at
        // 1600x1064 175 and 173): there the LDS takes as long as the vector units do (three of four fetches left out: 0.85 of the time).
        auto evaluate = [&]() {
            float dx[GROUP], dy[GROUP], tx[GROUP], ty[GROUP], t[GROUP], n[GROUP], sG[GROUP], al[GROUP];
            uint64_t act[GROUP], capped[GROUP];
            FS_STEP { dx[u] = p.px - r0[u].x; dy[u] = p.py - r0[u].y; }
            FS_STEP { tx[u] = r0[u].z * dx[u]; ty[u] = r1[u].x * dy[u]; }
            FS_STEP { tx[u] = __builtin_fmaf(r0[u].w, dy[u], tx[u]); ty[u] = ty[u] * dy[u]; }
            FS_STEP { t[u] = __builtin_fmaf(dx[u], tx[u], ty[u]); cd[u] = r1[u].z * dC0; }
            FS_STEP { t[u] = exponent_of(t[u]); cd[u] = __builtin_fmaf(r1[u].w, dC1, cd[u]); }
            FS_STEP { n[u] = __builtin_rintf(t[u]); cd[u] = __builtin_fmaf(cb[u], dC2, cd[u]); }   // dC . c
            FS_STEP { act[u] = takes_part_mask(t[u]); t[u] = t[u] - n[u]; }
            FS_STEP { G[u] = __builtin_fmaf(EXP_C[0], t[u], EXP_C[1]); }
            FS_STEP { G[u] = __builtin_fmaf(G[u], t[u], EXP_C[2]); }
            FS_STEP { G[u] = __builtin_fmaf(G[u], t[u], EXP_C[3]); act[u] &= ballot(js[u] < last_here); }
            FS_STEP { G[u] = __builtin_fmaf(G[u], t[u], EXP_C[4]); }
            FS_STEP { G[u] = __builtin_fmaf(G[u], t[u], 1.0f); }
            FS_STEP { G[u] = __builtin_ldexpf(G[u], (int)n[u]); }
            FS_STEP { sG[u] = r1[u].y * G[u]; }
            FS_STEP { al[u] = fminf(cfg.alpha_max, sG[u]); }
            FS_STEP { capped[u] = ballot(sG[u] > cfg.alpha_max); act[u] &= ballot(al[u] >= cfg.alpha_min); }
            // lanes that do not blend this Gaussian run the same arithmetic with alpha = G = 0: w and v are
            // exact zeros (and T / (1 - 0) leaves T as it is); a capped alpha is a constant: G = 0
            FS_STEP { acted |= act[u]; alpha[u] = lane_of(act[u]) ? al[u] : 0.f; }
            FS_STEP { G[u] = lane_of(act[u] & ~capped[u]) ? G[u] : 0.f; inv[u] = 1.0f - alpha[u]; }
            FS_STEP { inv[u] = __builtin_amdgcn_rcpf(inv[u]); }
            __builtin_amdgcn_sched_barrier(0);
        };
        for (int k = 0; k < longest; k += SPAN) {
            const uint2 words = *reinterpret_cast<const uint2*>(&s.list[sub][k / 4]);
            float w[SPAN], v[SPAN];
            acted = 0;
            auto chain = [&](int g) {
#pragma unroll
                for (int u = 0; u < GROUP; u++) {
                    T = T * inv[u];                                  // transmittance in front of this Gaussian
                    w[g + u] = alpha[u] * T;
                    const float diff = cd[u] - S;
                    v[g + u] = G[u] * (T * diff);                    // G dL/dalpha: d/d sigma
                    S = __builtin_fmaf(alpha[u], diff, S);
                }
            };
            fetch(words.x);
            evaluate();
            const uint32_t slot = ent_list[k];
            if (k + GROUP < longest) {
                fetch(words.y);   // (on its way during the chain)
                __builtin_amdgcn_sched_barrier(0);
                chain(0);
                evaluate();
                chain(GROUP);
            } else {
                chain(0);
#pragma unroll
                for (int u = 0; u < GROUP; u++) w[GROUP + u] = v[GROUP + u] = 0.f;
            }
            if (acted == 0) continue;
            const float mu_x = s.r0[slot].x, mu_y = s.r0[slot].y;
            const bool needle = __float_as_uint(s.r2[slot].w) & NEEDLE;
            float sums0[6], sums1[6];   // the first lane's, the second one's
            float4 wa, wb, a, b;
            exchange(w, wa, wb);
            exchange(v, a, b);   // (its writes need not wait for the reads before them)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ch = 0; ch < 3; ch++)
                sums0[ch] = (__builtin_fmaf(wb.w, g2[ch][3], __builtin_fmaf(wb.z, g2[ch][2], __builtin_fmaf(wb.y, g2[ch][1],
                                   __builtin_fmaf(wb.x, g2[ch][0], __builtin_fmaf(wa.w, g1[ch][3], __builtin_fmaf(wa.z, g1[ch][2],
                                   __builtin_fmaf(wa.y, g1[ch][1], wa.x * g1[ch][0]))))))));
            {
                const float dx[4] = {px0 - mu_x, column(1) - mu_x, column(2) - mu_x, column(3) - mu_x}, dy1 = py1 - mu_y, dy2 = py2 - mu_y;
                const float dxx[4] = {dx[0] * dx[0], dx[1] * dx[1], dx[2] * dx[2], dx[3] * dx[3]};
                auto along = [](const float4& l, const float (&d)[4]) {
                    return __builtin_fmaf(l.w, d[3], __builtin_fmaf(l.z, d[2], __builtin_fmaf(l.y, d[1], l.x * d[0])));
                };
                const float a0 = (a.x + a.y) + (a.z + a.w), b0 = (b.x + b.y) + (b.z + b.w);
                const float a1 = along(a, dx), b1 = along(b, dx);
                const float ya = dy1 * a0, yb = dy2 * b0;
                sums0[DSIGMA] = a0 + b0;
                sums1[DX - HALF] = a1 + b1;
                sums1[DY - HALF] = ya + yb;
                sums1[DXX - HALF] = along(a, dxx) + along(b, dxx);
                sums1[DYY - HALF] = __builtin_fmaf(dy1, ya, dy2 * yb);
                sums1[DXY - HALF] = __builtin_fmaf(dy1, a1, dy2 * b1);
                if (ABS) {
                    // |v| times half of |dq/dmu| = |a dx + b dy|, |b dx + c dy|, pixel by pixel
                    const float4 r0 = s.r0[slot];
                    const float qa = r0.z + r0.z, qb = r0.w, qc = 2.0f * s.r1[slot].x;
                    auto sizes = [&](const float4& l, float dy, float& x, float& y) {
                        const float v4[4] = {l.x, l.y, l.z, l.w}, bx = qb * dy, by = qc * dy;
#pragma unroll
                        for (int c = 0; c < 4; c++) {
                            const float hx = __builtin_fmaf(qa, dx[c], bx), hy = __builtin_fmaf(qb, dx[c], by);
                            x = c == 0 ? fabsf(v4[c]) * fabsf(hx) : __builtin_fmaf(fabsf(v4[c]), fabsf(hx), x);
                            y = c == 0 ? fabsf(v4[c]) * fabsf(hy) : __builtin_fmaf(fabsf(v4[c]), fabsf(hy), y);
                        }
                    };
                    float x1, y1, x2, y2;
                    sizes(a, dy1, x1, y1);
                    sizes(b, dy2, x2, y2);
                    sums0[DABS_X] = x1 + x2;
                    sums0[DABS_Y] = y1 + y2;
                }
            }
            // the two lanes of a combination: the first one gets the whole of sums0, the second one that of sums1
            float sum[6];
            __builtin_amdgcn_sched_barrier(0);   // (side by side)
#pragma unroll
            for (int f = 0; f < (ABS ? 6 : 5); f++) {
                const float s0 = f < HALF ? sums0[f] : 0.f, s1 = f < NV - HALF ? sums1[f] : 0.f;
                const float keep = second ? s1 : s0, give = second ? s0 : s1;
                sum[f] = keep + other(give);
            }
            __builtin_amdgcn_sched_barrier(0);
            // needles: dL/dq times dx^2, dx dy, dy^2 pixel by pixel, added in the order of a balanced tree over the lines and
            // their pixels (500k Gaussians: one exchange in ten has one).  The v's are read from LDS once more, so that the common
            // path does not hold them in registers.
            if (ballot(needle) != 0) {
                float xx = 0.f, xy = 0.f, yy = 0.f;
                const float gq = -0.5f * s.r1[slot].y;
#pragma unroll
                for (int l = 0; l < 2; l++) {
                    const float4 v4 = turned[l ? q2 : q1];
                    const float dy = (l ? py2 : py1) - mu_y;
                    const float vv[4] = {v4.x, v4.y, v4.z, v4.w};
                    float pxx[4], pxy[4], pyy[4];
#pragma unroll
                    for (int c = 0; c < 4; c++) {
                        const float dx = column(c) - mu_x;
                        const float gv = gq * vv[c], gx = gv * dx, gy = gv * dy;
                        pxx[c] = gx * dx;
                        pxy[c] = gx * dy;
                        pyy[c] = gy * dy;
                    }
                    // (lines 0 and 1, then 2 and 3, or the other way round)
                    xx = xx + both((pxx[0] + pxx[1]) + (pxx[2] + pxx[3]));
                    xy = xy + both((pxy[0] + pxy[1]) + (pxy[2] + pxy[3]));
                    yy = yy + both((pyy[0] + pyy[1]) + (pyy[2] + pyy[3]));
                }
                const bool mine = needle & second;
                sum[DXX - HALF] = mine ? xx : sum[DXX - HALF];
                sum[DYY - HALF] = mine ? yy : sum[DYY - HALF];
                sum[DXY - HALF] = mine ? xy : sum[DXY - HALF];
            }
            // The four rows of a quadrant often have the same Gaussian in the same exchange, and an LDS atomic takes one round for every
            // lane that names the same place: so each row takes the first four sums in an order of its own (number i ^ row in
            // round i), and neighbouring lanes name neighbouring places.
            const uint32_t acc = slot * (uint32_t)(NV * sizeof(acc_t)) + (second ? HALF * (uint32_t)sizeof(acc_t) : 0u);
            auto add = [&](uint32_t place, float u) {
                if (u != 0.f) atomicAdd(reinterpret_cast<acc_t*>(reinterpret_cast<char*>(&s_acc[0][0]) + place), (acc_t)u);
            };
            {
                static_assert(sizeof(acc_t) == 8, "places of the sums");
                const float p0 = row & 1 ? sum[1] : sum[0], p1 = row & 1 ? sum[0] : sum[1], p2 = row & 1 ? sum[3] : sum[2], p3 = row & 1 ? sum[2] : sum[3];
                const float mine[4] = {row & 2 ? p2 : p0, row & 2 ? p3 : p1, row & 2 ? p0 : p2, row & 2 ? p1 : p3};
#pragma unroll
                for (int f = 0; f < 4; f++) add(acc + 8u * (uint32_t)(f ^ row), mine[f]);
#pragma unroll
                for (int f = 4; f < (ABS ? 6 : 5); f++) add(acc + 8u * f, sum[f]);
            }
        }
        __syncthreads();
        if ((int)threadIdx.x < m) {
            acc_t a[NV];
#pragma unroll
            for (int k = 0; k < NV; k++) a[k] = s_acc[threadIdx.x][k];
            // SPARSE: a pair that received nothing (blended at no pixel of the tile) leaves no record; its flag stays 0
            // and k_preprocess_bwd does not read the record's place
            bool any = !SPARSE;
            if (SPARSE) {
#pragma unroll
                for (int k = 0; k < NV; k++) any = any | (a[k] != (acc_t)0);
            }
            if (any) {
                const float4 f0 = s.r0[threadIdx.x];
                const float2 f1 = make_float2(s.r1[threadIdx.x].x, s.r1[threadIdx.x].y);
                const float3 co = make_float3(-2.0f * f0.z, -2.0f * f0.w, -2.0f * f1.x);  // (a, 2b, c)
                const acc_t sigma = f1.y, gq = -0.5 * sigma;                              // dL/dq = -1/2 sigma G dL/dalpha
                const float mx = (float)(gq * a[DX]), my = (float)(gq * a[DY]);
                const uint32_t idx = __float_as_uint(s.r2[threadIdx.x].w) & ~NEEDLE;
                float4* rec = pair_grad + (size_t)idx * (PAIR_REC / 4);
                rec[0] = make_float4((float)a[DR], (float)a[DG], (float)a[DB], (float)a[DSIGMA]);
                // d = p - mu  =>  dq/dmu = -(2 a dx + 2b dy, 2b dx + 2 c dy)
                const acc_t second = __float_as_uint(s.r2[threadIdx.x].w) & NEEDLE ? 1.0 : gq;   // (a needle's come times dL/dq)
                rec[1] = make_float4((float)(second * a[DXX]), (float)(2.0 * second * a[DXY]), (float)(second * a[DYY]),
                                     -(2.0f * co.x * mx + co.y * my));
                rec[2] = make_float4(-(co.y * mx + 2.0f * co.z * my), ABS ? (float)(sigma * a[DABS_X]) : 0.f,
                                     ABS ? (float)(sigma * a[DABS_Y]) : 0.f, 0.f);
                if (SPARSE) rec_valid[idx] = 1;
            }
        }
    }
    // pairs behind the furthest blended Gaussian of the tile received nothing (SPARSE: their flags stay 0); PACKED: so did those in between
    if (!SPARSE) {
        uint32_t* const in_record = reinterpret_cast<uint32_t*>(&s_turn[0][0][0]);   // a bit for each place on the tile's list (the walks are over)
        const uint32_t n = range.y - range.x;
        if (PACKED) {
            static_assert(sizeof(s_turn) * 8 >= 65536, "a bit for every place that a record names");
            for (uint32_t w = threadIdx.x; w < (n + 31) / 32; w += 256) in_record[w] = 0u;
            __syncthreads();
            for (int i = (int)threadIdx.x; i < total; i += 256) {
                const uint32_t at = blends.entries[range.x + i].y & 0xffffu;
                atomicOr(&in_record[at / 32], 1u << (at & 31));
            }
            __syncthreads();
        }
        for (uint32_t at = (PACKED ? 0u : (uint32_t)total) + threadIdx.x; at < n; at += 256) {
            if (PACKED && (in_record[at / 32] >> (at & 31) & 1u)) continue;
            const float4 r2 = splats[(size_t)gauss_sorted[range.x + at] * (SPLAT_REC / 4) + 2];
            const uint32_t r01 = __float_as_uint(r2.z), r23 = __float_as_uint(r2.w);
            const uint32_t x0 = r01 & 0xffffu, y0 = r01 >> 16, x1 = r23 & 0xffffu;
            const uint32_t idx = (__float_as_uint(r2.y) & ~NEEDLE) + ((uint32_t)(tile / cam.tiles_x) - y0) * (x1 - x0) +
                                 ((uint32_t)(tile % cam.tiles_x) - x0);
            float4* rec = pair_grad + (size_t)idx * (PAIR_REC / 4);
            rec[0] = make_float4(0.f, 0.f, 0.f, 0.f);
            rec[1] = make_float4(0.f, 0.f, 0.f, 0.f);
            rec[2] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
}

// ---- per-splat-parallel backward (the mapping of Taming-3DGS that the paper's baseline uses) -------------
// Alternative to k_render_bwd with the same inputs, outputs and record layout; kept for comparison.
// A wavefront owns one 8x8 quadrant of the tile.  Per batch it forms the quadrant's list (the staged entries
// whose ellipse meets any of its four sub-tiles), takes it in chunks of 64 entries from the back, one entry per
// lane (lane 0 = the entry furthest back), and passes the quadrant's 64 pixels by one after the other.  For a
// pixel p every lane evaluates its own Gaussian; what the per-pixel kernel carries from entry to entry becomes
// two scans over the lanes:
//   T in front of entry l    = T_behind_chunk / prod_{k <= l} (1 - alpha_k)
//   S behind entry l         = the maps  S -> alpha_k (dC . c_k) + (1 - alpha_k) S  of the entries k < l applied,
//                              furthest first, to S_behind_chunk, where S = dC . (colour composited behind),
//                              which is all that dL/dalpha = T (dC . c - S) needs.
// The 9 (11) sums of a Gaussian over the pixels are then plain per-lane accumulators: no reduction across
// lanes.  Pixel p's state (T, S behind the part of the list already done) lives in lane p and is fetched with
// readlane.  The four quadrants' sums of a Gaussian meet in LDS as in k_render_bwd.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_from(float identity, float v)
{
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(identity), __float_as_int(v), CTRL, ROW_MASK, 0xF, false));
}

// Inclusive scan over the lanes of the composition of the maps S -> b + m S, lane 0 applied first:
// afterwards (m, b) of lane l is the composition of the maps of lanes 0 .. l.
__device__ __forceinline__ void wave_scan_affine(float& m, float& b)
{
#define FS_AFFINE_STEP(CTRL, ROW_MASK)                                  \
    {                                                                   \
        const float mo = dpp_from<CTRL, ROW_MASK>(1.0f, m);             \
        const float bo = dpp_from<CTRL, ROW_MASK>(0.0f, b);             \
        b = __builtin_fmaf(m, bo, b);                                   \
        m = m * mo;                                                     \
    }
    FS_AFFINE_STEP(0x111, 0xF)   // row_shr:1
    FS_AFFINE_STEP(0x112, 0xF)   // row_shr:2
    FS_AFFINE_STEP(0x114, 0xF)   // row_shr:4
    FS_AFFINE_STEP(0x118, 0xF)   // row_shr:8
    FS_AFFINE_STEP(0x142, 0xA)   // row_bcast:15 into rows 1 and 3
    FS_AFFINE_STEP(0x143, 0xC)   // row_bcast:31 into rows 2 and 3
#undef FS_AFFINE_STEP
}

template <bool ABS, bool SPARSE>
__global__ __launch_bounds__(256) void k_render_bwd_splat(
    CamDev cam, CfgDev cfg, const uint2* __restrict__ ranges, const uint32_t* __restrict__ tile_order,
    const uint32_t* __restrict__ gauss_sorted,
    const float4* __restrict__ splats, const float* __restrict__ final_T, const uint32_t* __restrict__ n_contrib,
    const float* __restrict__ dL_dimage, float4* __restrict__ pair_grad, uint8_t* __restrict__ rec_valid)
{
    __shared__ Stage<true> s;
    constexpr int NV = ABS ? 11 : 9;
    __shared__ double s_acc[SLOTS][NV];   // (double: the cheaper LDS atomic add on this chip, see k_render_bwd)
    __shared__ uint8_t s_qlist[4][SLOTS];   // per quadrant: the batch slots on its list, in list order
    __shared__ int s_max;

    const int tile = (int)tile_order[blockIdx.x];
    const Pixel p = pixel_of_thread(cam, tile);
    const uint2 range = ranges[tile];
    const size_t hw = (size_t)cam.width * cam.height;
    const size_t pix = (size_t)p.y * cam.width + p.x;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;

    // this lane's pixel: constants and the state behind the part of the list already done
    const int last = p.inside ? (int)n_contrib[pix] : 0;
    float T_st = p.inside ? final_T[pix] : 0.f;
    float dC0 = 0.f, dC1 = 0.f, dC2 = 0.f;
    if (p.inside) {
        dC0 = dL_dimage[pix];
        dC1 = dL_dimage[hw + pix];
        dC2 = dL_dimage[2 * hw + pix];
    }
    float S_st = __builtin_fmaf(dC2, cfg.bg[2], __builtin_fmaf(dC1, cfg.bg[1], dC0 * cfg.bg[0]));

    s.clear(threadIdx.x);
    if (threadIdx.x == 0) s_max = 0;
    __syncthreads();
    atomicMax(&s_max, last);
    __syncthreads();
    const int total = s_max;
    // the furthest position any pixel of this quadrant reaches (uniform in the wavefront)
    int wave_last = last;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) wave_last = max(wave_last, __shfl_xor(wave_last, d, 64));

    for (int start = ((total - 1) / BATCH) * BATCH; start >= 0 && total > 0; start -= BATCH) {
        const int m = min(BATCH, total - start);
        __syncthreads();  // the previous batch's flush has read s_acc, its walk s_qlist
#pragma unroll
        for (int k = 0; k < NV; k++) s_acc[threadIdx.x][k] = 0.0;
        stage_batch<2>(s, nullptr, cam, tile, splats, (int)threadIdx.x < m ? gauss_sorted[range.x + start + threadIdx.x] : 0u, m);
        // the quadrant's list: lane l looks at slots 4 l .. 4 l + 3 of the union of its four sub-tiles' masks
        uint32_t b4 = 0;
        {
            const uint16_t* of = reinterpret_cast<const uint16_t*>(s.sub);
#pragma unroll
            for (int k = 0; k < 4; k++) b4 |= (of[s.sub_place(4 * lane + k)] >> (wave * 4) & 0xfu) != 0u ? 1u << k : 0u;
        }
        const int cnt = __popc(b4);
        int inc = cnt;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(inc, d, 64);
            if (lane >= d) inc += o;
        }
        const int qlen = __shfl(inc, 63, 64);
        {
            int pos = inc - cnt;
            uint32_t b = b4;
            while (b) {
                s_qlist[wave][pos++] = (uint8_t)(4 * lane + __builtin_ctz(b));
                b &= b - 1u;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();

        if (start < wave_last) {
            for (int c_end = qlen; c_end > 0; c_end -= 64) {
                // lane 0 takes the entry furthest back of the chunk
                const int idx = c_end - 1 - lane;
                const bool have = idx >= 0;
                const int j = have ? (int)s_qlist[wave][idx] : 0;
                const float4 f0 = s.r0[j], f1 = s.r1[j], f2 = s.r2[j];
                const float2 xy = make_float2(f0.x, f0.y);
                const float4 co = make_float4(f0.z, f0.w, f1.x, f1.y);    // (-a/2, -b, -c/2, sigma)
                const float4 col = make_float4(f2.x, f2.y, f2.z, 0.f);
                const int pos_j = start + j;
                float acc[NV];
#pragma unroll
                for (int k = 0; k < NV; k++) acc[k] = 0.f;
                bool any = false;
                for (int q = 0; q < 64; q++) {
                    const int last_q = __builtin_amdgcn_readlane(last, q);
                    if (last_q <= start) continue;   // this pixel blends nothing of this batch
                    const float px = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(p.px), q));
                    const float py = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(p.py), q));
                    const float dx = px - xy.x, dy = py - xy.y;
                    const float h = __builtin_fmaf(co.y, dy, co.x * dx);
                    const float t = exponent_of(__builtin_fmaf(dx, h, (co.z * dy) * dy));
                    bool act = have & (pos_j < last_q) & takes_part(t);
                    if (__ballot(act) == 0) continue;
                    float G = exp_c(act ? t : 0.0f);
                    const float sG = co.w * G;
                    float alpha = fminf(cfg.alpha_max, sG);
                    act = act & (alpha >= cfg.alpha_min);
                    if (__ballot(act) == 0) continue;
                    any = true;
                    alpha = act ? alpha : 0.f;
                    G = act ? G : 0.f;
                    const float d0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dC0), q));
                    const float d1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dC1), q));
                    const float d2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dC2), q));
                    const float T_behind = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(T_st), q));
                    const float S_behind = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(S_st), q));
                    const float cd = __builtin_fmaf(col.z, d2, __builtin_fmaf(col.y, d1, col.x * d0));   // dC . c
                    float M = 1.0f - alpha, Bc = alpha * cd;
                    wave_scan_affine(M, Bc);
                    // maps of the lanes before this one (the entries behind it)
                    float Mx = __shfl_up(M, 1, 64), Bx = __shfl_up(Bc, 1, 64);
                    if (lane == 0) { Mx = 1.0f; Bx = 0.0f; }
                    const float T = T_behind * __builtin_amdgcn_rcpf(M);   // in front of this entry
                    const float S = __builtin_fmaf(Mx, S_behind, Bx);      // dC . (colour behind this entry)
                    const float w = alpha * T;
                    acc[0] = __builtin_fmaf(w, d0, acc[0]);
                    acc[1] = __builtin_fmaf(w, d1, acc[1]);
                    acc[2] = __builtin_fmaf(w, d2, acc[2]);
                    float dL_dalpha = T * (cd - S);
                    dL_dalpha = sG > cfg.alpha_max ? 0.f : dL_dalpha;   // capped alpha is a constant
                    acc[3] = __builtin_fmaf(G, dL_dalpha, acc[3]);
                    const float gq = -0.5f * (co.w * G) * dL_dalpha;
                    const float gx = gq * dx, gy = gq * dy;
                    acc[4] = __builtin_fmaf(gx, dx, acc[4]);
                    acc[5] = __builtin_fmaf(gx, dy, acc[5]);
                    acc[6] = __builtin_fmaf(gy, dy, acc[6]);
                    acc[7] += gx;
                    acc[8] += gy;
                    if (ABS) {
                        const float ag = 2.0f * fabsf(gq);
                        acc[NV - 2] = __builtin_fmaf(ag, fabsf(__builtin_fmaf(co.y, dy, 2.0f * co.x * dx)), acc[NV - 2]);
                        acc[NV - 1] = __builtin_fmaf(ag, fabsf(__builtin_fmaf(co.y, dx, 2.0f * co.z * dy)), acc[NV - 1]);
                    }
                    // pixel q moves in front of the chunk: the last lane holds the composition of all its maps
                    const float M_all = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(M), 63));
                    const float B_all = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(Bc), 63));
                    const float T_new = T_behind * __builtin_amdgcn_rcpf(M_all);
                    const float S_new = __builtin_fmaf(M_all, S_behind, B_all);
                    T_st = lane == q ? T_new : T_st;
                    S_st = lane == q ? S_new : S_st;
                }
                if (any && have) {
#pragma unroll
                    for (int k = 0; k < NV; k++)
                        if (acc[k] != 0.f) atomicAdd(&s_acc[j][k], (double)acc[k]);
                }
            }
        }
        __syncthreads();
        if ((int)threadIdx.x < m) {
            float a[NV];
#pragma unroll
            for (int k = 0; k < NV; k++) a[k] = (float)s_acc[threadIdx.x][k];
            // SPARSE: a pair that received nothing (blended at no pixel of the tile) leaves no record; its flag stays 0
            // and k_preprocess_bwd does not read the record's place
            bool any = !SPARSE;
            if (SPARSE) {
#pragma unroll
                for (int k = 0; k < NV; k++) any = any | (a[k] != 0.f);
            }
            if (any) {
                const float4 f0 = s.r0[threadIdx.x];
                const float3 co = make_float3(-2.0f * f0.z, -2.0f * f0.w, -2.0f * s.r1[threadIdx.x].x);  // (a, 2b, c)
                const uint32_t idx = __float_as_uint(s.r2[threadIdx.x].w) & ~NEEDLE;
                float4* rec = pair_grad + (size_t)idx * (PAIR_REC / 4);
                rec[0] = make_float4(a[0], a[1], a[2], a[3]);
                // d = p - mu  =>  dq/dmu = -(2 a dx + 2b dy, 2b dx + 2 c dy)
                rec[1] = make_float4(a[4], 2.0f * a[5], a[6], -(2.0f * co.x * a[7] + co.y * a[8]));
                rec[2] = make_float4(-(co.y * a[7] + 2.0f * co.z * a[8]), ABS ? a[NV - 2] : 0.f, ABS ? a[NV - 1] : 0.f, 0.f);
                if (SPARSE) rec_valid[idx] = 1;
            }
        }
    }
    // pairs behind the furthest blended Gaussian of the tile received nothing (SPARSE: their flags stay 0)
    if (!SPARSE) {
        for (uint32_t pos = range.x + total + threadIdx.x; pos < range.y; pos += 256) {
            const float4 r2 = splats[(size_t)gauss_sorted[pos] * (SPLAT_REC / 4) + 2];
            const uint32_t r01 = __float_as_uint(r2.z), r23 = __float_as_uint(r2.w);
            const uint32_t x0 = r01 & 0xffffu, y0 = r01 >> 16, x1 = r23 & 0xffffu;
            const uint32_t idx = (__float_as_uint(r2.y) & ~NEEDLE) + ((uint32_t)(tile / cam.tiles_x) - y0) * (x1 - x0) +
                                 ((uint32_t)(tile % cam.tiles_x) - x0);
            float4* rec = pair_grad + (size_t)idx * (PAIR_REC / 4);
            rec[0] = make_float4(0.f, 0.f, 0.f, 0.f);
            rec[1] = make_float4(0.f, 0.f, 0.f, 0.f);
            rec[2] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }
}

// Count pass: re-walks the forward loop for the mask pixels only (other pixels cannot add to a
// count) up to each pixel's n_contrib, and counts per Gaussian the pixels where it is blended
// (and, in weight mode, alpha*T > alpha_min).  A ballot + population count gives each sub-tile's
// count without any cross-lane arithmetic.
__global__ __launch_bounds__(256) void k_score(CamDev cam, CfgDev cfg, const uint2* __restrict__ ranges,
                                               const uint32_t* __restrict__ tile_order,
                                               const uint32_t* __restrict__ gauss_sorted,
                                               const float4* __restrict__ splats,
                                               const uint32_t* __restrict__ n_contrib,
                                               const uint8_t* __restrict__ mask, int32_t* __restrict__ counts)
{
    __shared__ Stage<false> s;
    __shared__ uint32_t s_id[SLOTS];
    __shared__ int s_cnt[SLOTS];
    __shared__ int s_max;

    const int tile = (int)tile_order[blockIdx.x];  // longest lists first
    const Pixel p = pixel_of_thread(cam, tile);
    const uint2 range = ranges[tile];
    const size_t pix = (size_t)p.y * cam.width + p.x;
    const int lane = threadIdx.x & 63;
    const int sub = (threadIdx.x >> 6) * 4 + (lane >> 4);
    int last = 0;
    if (p.inside && mask[pix]) last = (int)n_contrib[pix];
    s.clear(threadIdx.x);
    if (threadIdx.x == 0) s_max = 0;
    __syncthreads();
    atomicMax(&s_max, last);
    __syncthreads();
    const int total = s_max;
    float T = 1.0f;

    // The walking pixels (mask pixels with at least one blended Gaussian) are usually a small part of the
    // tile.  When at most half of it walks, they are packed into the first lanes of the workgroup: lane c
    // takes over the c-th walking pixel, with that pixel's own sub-tile list, so that one or two wavefronts
    // run the loop instead of four mostly idle ones.  The per-pixel arithmetic is the same either way.
    __shared__ int s_wave_cnt[4];
    __shared__ uint8_t s_walker[256];
    const bool walks = last > 0;
    const uint64_t wb = __ballot(walks);
    if (lane == 0) s_wave_cnt[threadIdx.x >> 6] = __popcll(wb);
    __syncthreads();
    int before = 0, nwalk = 0;
#pragma unroll
    for (int w = 0; w < 4; w++) {
        before += w < (int)(threadIdx.x >> 6) ? s_wave_cnt[w] : 0;
        nwalk += s_wave_cnt[w];
    }
    if (walks) s_walker[before + __popcll(wb & ((1ull << lane) - 1ull))] = (uint8_t)threadIdx.x;
    __syncthreads();

    if (nwalk <= 128) {
        // Which wavefront takes the first 64 walkers rotates with the workgroup index: wavefront w of every
        // workgroup runs on the same SIMD of its CU, and the walk is the expensive part.
        const int c = (int)((((threadIdx.x >> 6) - blockIdx.x) & 3u) * 64u) + lane;
        const bool on = c < nwalk;
        const int me = on ? (int)s_walker[c] : 0;
        const Pixel pw = pixel_of_thread(cam, tile, me);
        const int my_sub = (me >> 6) * 4 + ((me & 63) >> 4);
        const int my_last = on ? (int)n_contrib[(size_t)pw.y * cam.width + pw.x] : 0;
        const bool wave_on = (c - lane) < nwalk;   // uniform per wavefront
        for (int start = 0; start < total; start += BATCH) {
            const int m = min(BATCH, total - start);
            __syncthreads();  // the previous batch's flush has read s_cnt / s_id
            s_cnt[threadIdx.x] = 0;
            stage_batch<1>(s, s_id, cam, tile, splats, (int)threadIdx.x < m ? gauss_sorted[range.x + start + threadIdx.x] : 0u, m);
            __syncthreads();  // (a walker follows the list of its own sub-tile, whichever wavefront made it)
            if (wave_on) {
                const int len = start < my_last ? s.len[my_sub] : 0;
                // two list entries per trip: their alphas are independent, only the transmittance chains
                for (int k = 0; __ballot(k < len) != 0; k += 2) {
                    const int j0 = s.slot(my_sub, k), j1 = s.slot(my_sub, k + 1);
                    const float4 a0 = s.r0[j0], b0 = s.r1[j0], a1 = s.r0[j1], b1 = s.r1[j1];
                    const float dx0 = pw.px - a0.x, dy0 = pw.py - a0.y;
                    const float dx1 = pw.px - a1.x, dy1 = pw.py - a1.y;
                    const float t0 = exponent_of(__builtin_fmaf(dx0, __builtin_fmaf(a0.w, dy0, a0.z * dx0), (b0.x * dy0) * dy0));
                    const float t1 = exponent_of(__builtin_fmaf(dx1, __builtin_fmaf(a1.w, dy1, a1.z * dx1), (b1.x * dy1) * dy1));
                    bool act0 = (k < len) & (start + j0 < my_last) & takes_part(t0);
                    bool act1 = (k + 1 < len) & (start + j1 < my_last) & takes_part(t1);
                    if (__ballot(act0 | act1) == 0) continue;
                    // (an inactive entry's exponent may be anything: clamp it so that exp_c stays in range)
                    const float alpha0 = fminf(cfg.alpha_max, b0.y * exp_c(act0 ? t0 : 0.0f));
                    const float alpha1 = fminf(cfg.alpha_max, b1.y * exp_c(act1 ? t1 : 0.0f));
                    act0 = act0 & (alpha0 >= cfg.alpha_min);
                    act1 = act1 & (alpha1 >= cfg.alpha_min);
                    const bool hit0 = act0 & (cfg.score_mode == FS_SCORE_ALPHA || alpha0 * T > cfg.alpha_min);
                    T = act0 ? T * (1.0f - alpha0) : T;
                    const bool hit1 = act1 & (cfg.score_mode == FS_SCORE_ALPHA || alpha1 * T > cfg.alpha_min);
                    T = act1 ? T * (1.0f - alpha1) : T;
                    if (hit0) atomicAdd(&s_cnt[j0], 1);
                    if (hit1) atomicAdd(&s_cnt[j1], 1);
                }
            }
            __syncthreads();
            if ((int)threadIdx.x < m && s_cnt[threadIdx.x] != 0)
                atomicAdd(&counts[s_id[threadIdx.x]], s_cnt[threadIdx.x]);
        }
        return;
    }

    for (int start = 0; start < total; start += BATCH) {
        const int m = min(BATCH, total - start);
        __syncthreads();  // the previous batch's flush has read s_cnt / s_id
        s_cnt[threadIdx.x] = 0;
        const int mine = stage_batch<1>(s, s_id, cam, tile, splats, (int)threadIdx.x < m ? gauss_sorted[range.x + start + threadIdx.x] : 0u, m);
        // a row none of whose pixels is still walking (no mask pixel, or all past their last Gaussian)
        // has nothing to count in this batch
        const uint64_t walking = __ballot(start < last);
        if (walking != 0) {
            const bool row_walks = ((walking >> (lane & 48)) & 0xffffull) != 0;
            const int longest = wave_max_of_rows(row_walks ? mine : 0);
            for (int k = 0; k < longest; k++) {
                const int j = s.slot(sub, k);
                const float4 a0 = s.r0[j], b0 = s.r1[j];
                const float dx = p.px - a0.x, dy = p.py - a0.y;
                const float t = exponent_of(__builtin_fmaf(dx, __builtin_fmaf(a0.w, dy, a0.z * dx), (b0.x * dy) * dy));
                bool act = (k < mine) & (start + j < last) & takes_part(t);
                if (__ballot(act) == 0) continue;
                const float alpha = fminf(cfg.alpha_max, b0.y * exp_c(t));
                act = act & (alpha >= cfg.alpha_min);
                const float w = alpha * T;
                const bool hit = act & (cfg.score_mode == FS_SCORE_ALPHA || w > cfg.alpha_min);
                T = act ? T * (1.0f - alpha) : T;
                const uint32_t b = (uint32_t)(__ballot(hit) >> (lane & 48)) & 0xffffu;  // this row's pixels
                if (b != 0 && (lane & 15) == 0) atomicAdd(&s_cnt[j], (int)__popc(b));
            }
        }
        __syncthreads();
        if ((int)threadIdx.x < m && s_cnt[threadIdx.x] != 0) atomicAdd(&counts[s_id[threadIdx.x]], s_cnt[threadIdx.x]);
    }
}

// Count pass from the record a k_render_fwd<., true> launch left: per tile, the mask of its 256 pixels in the same
// layout as a row's bits, then one population count per row of the tile.  Tiles without rows or without mask pixels
// read nothing else.  Workgroup (x, y) takes rows [y * chunk, (y + 1) * chunk) of tile x (the last one whatever is
// left), so that thousands of rows are not one workgroup's chain of dependent rounds; a workgroup past the tile's last
// row leaves at once.  (Tiles in plain order: a tile's rows are few, and the detour over the order array would be one
// more dependent load.)
// FROM_ERR: the mask is not read but made here, mask[p] = err[p] > threshold (Sec. 4.2), by the first workgroup of
// every tile, which also stores it (mask_out) -- the mask kernel's launch saved.
template <bool FROM_ERR>
__global__ __launch_bounds__(256) void k_score_bits(CamDev cam, const uint2* __restrict__ ranges, ScoreRecord record,
                                                    const uint8_t* __restrict__ mask, int32_t* __restrict__ counts,
                                                    uint32_t chunk, const float* __restrict__ err,
                                                    const double* __restrict__ stats, int rule, float k,
                                                    uint8_t* __restrict__ mask_out, float* __restrict__ thr_out)
{
    __shared__ __align__(16) uint16_t s_m[16];
    const int tile = (int)blockIdx.x;
    const uint32_t rows = (uint32_t)record.tile_rows[tile];
    uint32_t first = blockIdx.y * chunk;
    if (rows <= first && !(FROM_ERR && blockIdx.y == 0)) return;   // (uniform over the workgroup)
    uint32_t end = blockIdx.y + 1 == gridDim.y ? rows : min(rows, first + chunk);
    const uint32_t seg = ranges[tile].x;
    first += seg;
    end += seg;
    const Pixel p = pixel_of_thread(cam, tile);
    const int lane = threadIdx.x & 63;
    const size_t pix = (size_t)p.y * cam.width + p.x;
    // the first 256 rows are requested before the tile's mask is known, so that the two latencies overlap
    uint32_t pos = first + threadIdx.x;
    uint4 a = make_uint4(0u, 0u, 0u, 0u), c = a;
    uint32_t g = 0;
    if (pos < end) {
        a = nt_load(record.rows + (size_t)pos * 2);
        c = nt_load(record.rows + (size_t)pos * 2 + 1);
        g = record.row_gauss[pos];
    }
    bool on;
    if (FROM_ERR) {
        const float thr = threshold_from_stats(stats[0], stats[1], stats[2], stats[3], (int64_t)cam.width * cam.height, rule, k);
        on = p.inside && err[pix] > thr;
        if (blockIdx.y == 0) {
            if (tile == 0 && threadIdx.x == 0) *thr_out = thr;
            if ((cam.width & 3) == 0 && (reinterpret_cast<uintptr_t>(mask_out) & 3) == 0) {
                // four neighbouring pixels of a line are four neighbouring lanes: one 4-byte store for them
                const uint32_t four = (uint32_t)(__ballot(on) >> (lane & 60)) & 0xfu;
                if ((lane & 3) == 0 && p.inside)
                    *reinterpret_cast<uint32_t*>(mask_out + pix) = (four & 1u) | (four & 2u) << 7 | (four & 4u) << 14 | (four & 8u) << 21;
            } else if (p.inside) {
                mask_out[pix] = on ? 1 : 0;
            }
        }
    } else {
        on = p.inside && mask[pix] != 0;
    }
    const uint64_t b = __ballot(on);
    if ((lane & 15) == 0) s_m[(threadIdx.x >> 6) * 4 + (lane >> 4)] = (uint16_t)((b >> (lane & 48)) & 0xffffull);
    if (__syncthreads_or(on) == 0 || first >= end) return;
    const uint4 m0 = reinterpret_cast<const uint4*>(s_m)[0], m1 = reinterpret_cast<const uint4*>(s_m)[1];
    for (;;) {
        // (the next round's rows are requested before this round's are counted)
        const uint32_t next = pos + 256;
        uint4 a2 = make_uint4(0u, 0u, 0u, 0u), c2 = a2;
        uint32_t g2 = 0;
        if (next < end) {
            a2 = nt_load(record.rows + (size_t)next * 2);
            c2 = nt_load(record.rows + (size_t)next * 2 + 1);
            g2 = record.row_gauss[next];
        }
        const int n = __popc(a.x & m0.x) + __popc(a.y & m0.y) + __popc(a.z & m0.z) + __popc(a.w & m0.w) +
                      __popc(c.x & m1.x) + __popc(c.y & m1.y) + __popc(c.z & m1.z) + __popc(c.w & m1.w);
        if (n != 0) atomicAdd(&counts[g], n);   // (all zeros for a thread past the last row)
        if (next >= end) break;
        pos = next; a = a2; c = c2; g = g2;
    }
}

__global__ __launch_bounds__(256) void k_record_rows(int tiles, const int32_t* __restrict__ tile_rows, int32_t* __restrict__ rows)
{
    const int tile = (int)(blockIdx.x * 256 + threadIdx.x);
    if (tile < tiles) rows[tile] = tile_rows[tile];
}

}  // namespace

hipError_t launch_render_fwd(hipStream_t st, const CamDev& cam, const CfgDev& cfg, const uint32_t* ranges,
                             const uint32_t* tile_order, const uint32_t* gauss_sorted, const float* splats, float* image, float* final_T,
                             uint32_t* n_contrib, const ScoreRecord& record, const BlendRecord& blends)
{
    const int tiles = cam.tiles_x * cam.tiles_y;
    if (tiles == 0) return hipSuccess;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(tiles), dim3(256), 0, st, cam, cfg, reinterpret_cast<const uint2*>(ranges), tile_order, gauss_sorted,
                           reinterpret_cast<const float4*>(splats), image, final_T, n_contrib, nullptr, 0.f, nullptr, nullptr, nullptr, record, blends);
    };
    if (record.rows && blends.entries) launch(k_render_fwd<false, true, true>);
    else if (record.rows) launch(k_render_fwd<false, true, false>);
    else if (blends.entries) launch(k_render_fwd<false, false, true>);
    else launch(k_render_fwd<false, false, false>);
    return hipGetLastError();
}

hipError_t launch_render_fwd_fused(hipStream_t st, const CamDev& cam, const CfgDev& cfg, const uint32_t* ranges,
                                   const uint32_t* tile_order, const uint32_t* gauss_sorted, const float* splats,
                                   float* image, float* final_T, uint32_t* n_contrib, const float* target, float* dL,
                                   float* err, double* tile_partial, const ScoreRecord& record, const BlendRecord& blends)
{
    const int tiles = cam.tiles_x * cam.tiles_y;
    if (tiles == 0) return hipSuccess;
    const float scale = 1.0f / (float)((int64_t)3 * cam.width * cam.height);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(tiles), dim3(256), 0, st, cam, cfg, reinterpret_cast<const uint2*>(ranges), tile_order, gauss_sorted,
                           reinterpret_cast<const float4*>(splats), image, final_T, n_contrib, target, scale, dL, err, tile_partial, record, blends);
    };
    if (record.rows && blends.entries) launch(k_render_fwd<true, true, true>);
    else if (record.rows) launch(k_render_fwd<true, true, false>);
    else if (blends.entries) launch(k_render_fwd<true, false, true>);
    else launch(k_render_fwd<true, false, false>);
    return hipGetLastError();
}

namespace {
// a workgroup of k_score_bits takes SCORE_CHUNK rows (the last one of a tile whatever is left); the longest list bounds
// the rows of any tile (0: not known)
constexpr uint32_t SCORE_CHUNK = 4096;
unsigned score_chunks(int64_t longest_list)
{
    int64_t chunks = longest_list > 0 ? (longest_list + SCORE_CHUNK - 1) / SCORE_CHUNK : 4;
    return (unsigned)(chunks > 64 ? 64 : chunks);
}
}  // namespace

hipError_t launch_score_bits(hipStream_t st, const CamDev& cam, const uint32_t* ranges, const ScoreRecord& record,
                             const uint8_t* mask, int32_t* counts, int64_t longest_list)
{
    const int tiles = cam.tiles_x * cam.tiles_y;
    if (tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(k_score_bits<false>, dim3(tiles, score_chunks(longest_list)), dim3(256), 0, st, cam,
                       reinterpret_cast<const uint2*>(ranges), record, mask, counts, SCORE_CHUNK, nullptr, nullptr, 0, 0.f,
                       nullptr, nullptr);
    return hipGetLastError();
}

hipError_t launch_mask_score_bits(hipStream_t st, const CamDev& cam, const uint32_t* ranges, const ScoreRecord& record,
                                  const float* err, const double* stats, int rule, float k, uint8_t* mask, float* thr_out,
                                  int32_t* counts, int64_t longest_list)
{
    const int tiles = cam.tiles_x * cam.tiles_y;
    if (tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(k_score_bits<true>, dim3(tiles, score_chunks(longest_list)), dim3(256), 0, st, cam,
                       reinterpret_cast<const uint2*>(ranges), record, nullptr, counts, SCORE_CHUNK, err, stats, rule, k, mask,
                       thr_out);
    return hipGetLastError();
}

hipError_t launch_record_rows(hipStream_t st, int tiles, const ScoreRecord& record, int32_t* rows)
{
    if (tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(k_record_rows, dim3((tiles + 255) / 256), dim3(256), 0, st, tiles, record.tile_rows, rows);
    return hipGetLastError();
}

hipError_t launch_render_bwd(hipStream_t st, const CamDev& cam, const CfgDev& cfg, const uint32_t* ranges,
                             const uint32_t* tile_order, const uint32_t* gauss_sorted, const float* splats, const float* final_T,
                             const uint32_t* n_contrib, const float* dL_dimage, float* pair_grad, uint8_t* rec_valid,
                             bool abs_grad, bool per_splat, const BlendRecord& blends)
{
    const int tiles = cam.tiles_x * cam.tiles_y;
    if (tiles == 0) return hipSuccess;
    const uint2* r2 = reinterpret_cast<const uint2*>(ranges);
    const float4* sp = reinterpret_cast<const float4*>(splats);
    float4* pg = reinterpret_cast<float4*>(pair_grad);
    auto launch = [&](auto kernel, auto... more) {
        hipLaunchKernelGGL(kernel, dim3(tiles), dim3(256), 0, st, cam, cfg, r2, tile_order, gauss_sorted, sp, final_T, n_contrib, dL_dimage, pg, rec_valid,
                           more...);
    };
    // rec_valid: null = dense records, else the flags of the sparse records
    auto choose = [&](auto abs, auto sparse) {
        constexpr bool ABS = decltype(abs)::value, SPARSE = decltype(sparse)::value;
        if (per_splat) launch(k_render_bwd_splat<ABS, SPARSE>);
        else if (blends.entries) launch(k_render_bwd<ABS, SPARSE, true>, blends);
        else launch(k_render_bwd<ABS, SPARSE, false>, blends);
    };
    if (abs_grad && rec_valid) choose(std::true_type{}, std::true_type{});
    else if (abs_grad) choose(std::true_type{}, std::false_type{});
    else if (rec_valid) choose(std::false_type{}, std::true_type{});
    else choose(std::false_type{}, std::false_type{});
    return hipGetLastError();
}

hipError_t launch_score(hipStream_t st, const CamDev& cam, const CfgDev& cfg, const uint32_t* ranges,
                        const uint32_t* tile_order, const uint32_t* gauss_sorted, const float* splats, const uint32_t* n_contrib,
                        const uint8_t* mask, int32_t* counts)
{
    const int tiles = cam.tiles_x * cam.tiles_y;
    if (tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(k_score, dim3(tiles), dim3(256), 0, st, cam, cfg, reinterpret_cast<const uint2*>(ranges),
                       tile_order, gauss_sorted, reinterpret_cast<const float4*>(splats), n_contrib, mask, counts);
    return hipGetLastError();
}

}  // namespace fs
