// Steps a5 and a7: per-pixel forward compositing (Eq. 1-5) and its adjoint,
// over the masked pixels only.
//
// Work decomposition: a work item is a pack of up to 64 masked pixels of one
// (frame, tile), compacted so that sparse masks do not idle lanes.  Each
// wave64 of a persistent grid takes items either round-robin (items_per_pop
// = 0: item k goes to wave k mod waves, so the packs of one tile land on the
// waves of one workgroup, i.e. one CU and one XCD L2) or in chunks of
// items_per_pop consecutive items from an atomic queue head.
//
// Records come in list order from the 64-byte pair-order copy written by the
// per-tile sort, 64 per batch, one per lane, with one coalesced load level;
// the next batch is prefetched into registers while the current one is
// composited.  Each batch is pack-culled (records that cannot reach any pixel
// of the pack are dropped, lane-parallel; about 95 % of those kept reach one)
// and the survivors are compacted into the wave's own LDS slice, from which
// every lane reads the same record (an LDS broadcast) with one lane per
// pixel.  Culling follows the pixels that are still open (forward: colour or
// hit outstanding; backward: entries left below their last): where a few
// pixels of a pack keep compositing through a long list, its later batches
// shrink to what reaches those.  (A path of its own for them, one entry per
// lane and pixel after pixel, took 106 of the 120 thousand cycles of a frame's
// longest pack; without it the forward of one masked 1200x680 frame went from
// 61 to 45 us, of 16 keyframes from 679 to 632 us.)  A ballot ends the walk once
// every lane has finished its colour and found its depth hit.
//
// Decisions (footprint, depth hit) use the fixed binary32 sequence on the
// rounded centre; the values (f, gradients) use offsets from the centre
// including its residual.
//
// The backward pass re-walks each pixel's list back to front, recovering the
// transmission in front of each Gaussian from the stored final value
// (T_i = T_{i+1} / (1 - f_i); nothing per pair is stored).  The nine
// colour-path gradients of the unstable Gaussians are summed over the wave's
// pixels eight records at a time, the five depth-path terms once per pack
// and hit, and added with float atomics into the Gaussian's per-frame
// camera-space accumulator.
//
// Both kernels are bound by vector issue where the items outnumber the waves
// (batches of keyframes) and by the longest packs' serial walks where they do
// not (one frame).  What a record costs on every lane was cut to: decision 8
// operations, value 2 more and the exponential, blend 7 (forward), and the
// one gradient sum g . (c - A) in place of three colour recursions (backward).
// Measured on MI355X, forward / backward: 16 keyframes of 1200x680 with 2.6M
// masked pixels 914 / 1050 to 630 / 650 us, 8 keyframes 632 / 930 to 499 /
// 650 us, one masked 1200x680 frame 63 / 103 to 44 / 59 us, one full 640x480
// frame 28 / 68 to 27 / 49 us.
#include <type_traits>

#include "rtg_common.h"

// Compile-time tuning knobs of the compositing kernels: records whose
// loads and independent parts are taken together before the sequential blend
// (instruction-level parallelism against register pressure), and the
// minimum number of resident waves per SIMD each kernel is compiled for
// (occupancy; 0 = compiler's choice).  Measured on gfx950, us per launch over
// 16 / 8 keyframes: forward groups of four (110 VGPRs, four waves) 793 / 582,
// of two (five waves) 912 / 589, of four held to five waves 900 / 593;
// backward groups of two (127 VGPRs, four waves) 705 / 715, single records
// 725 / 734.
#ifndef RTG_FWD_GROUP
#define RTG_FWD_GROUP 4
#endif
#ifndef RTG_FWD_WAVES_PER_EU
#define RTG_FWD_WAVES_PER_EU 0
#endif
#ifndef RTG_BWD_GROUP
#define RTG_BWD_GROUP 2
#endif
#ifndef RTG_BWD_WAVES_PER_EU
#define RTG_BWD_WAVES_PER_EU 4
#endif
#if RTG_FWD_WAVES_PER_EU > 0
#define RTG_FWD_BOUNDS __launch_bounds__(256, RTG_FWD_WAVES_PER_EU)
#else
#define RTG_FWD_BOUNDS __launch_bounds__(256)
#endif
#if RTG_BWD_WAVES_PER_EU > 0
#define RTG_BWD_BOUNDS __launch_bounds__(256, RTG_BWD_WAVES_PER_EU)
#else
#define RTG_BWD_BOUNDS __launch_bounds__(256)
#endif

namespace rtg {

struct PixelOfItem {
    uint32_t ft, r;     // (frame, tile) and rank of the pixel in the tile
    int f, px, py;
    bool act;
    float ux, uy;
    uint32_t rs, re;    // pair range of the tile
};

__device__ __forceinline__ PixelOfItem decode_item(const Dims& d, const WS& w, uint32_t it, int lane) {
    PixelOfItem p;
    uint32_t code = w.items[it];
    p.ft = code / (uint32_t)d.ppt;
    uint32_t pack = code - p.ft * (uint32_t)d.ppt;
    uint32_t npx = w.tile_npx[p.ft];
    p.r = pack * 64u + (uint32_t)lane;
    p.act = p.r < npx;
    // (loaded beside the count: the list has room for every rank of a pack)
    const int lp = (int)w.pix[(size_t)p.ft * d.tarea + p.r];
    const int l = p.act ? lp : 0;
    p.f = (int)(p.ft / (uint32_t)d.ntiles);
    int t = (int)(p.ft - (uint32_t)p.f * (uint32_t)d.ntiles);
    p.px = (t % d.tx) * d.tw + (l & (d.tw - 1));
    p.py = (t / d.tx) * d.th + (l >> d.lg_tw);
    p.ux = (float)p.px + 0.5f;
    p.uy = (float)p.py + 0.5f;
    p.rs = w.tile_start[p.ft];
    p.re = w.tile_end[p.ft];
    return p;
}

// Bounding box of pixels of one pack (inclusive pixel indices).
struct PackBox {
    int x0, x1, y0, y1;
};

// Wave minimum: DPP within the rows, then the permlane swaps across them.
template <int CTRL>
__device__ __forceinline__ int dpp_mov_i(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}
__device__ __forceinline__ int wave_min_i(int v) {
    v = min(v, dpp_mov_i<0xB1>(v));
    v = min(v, dpp_mov_i<0x4E>(v));
    v = min(v, dpp_mov_i<0x141>(v));
    v = min(v, dpp_mov_i<0x140>(v));
    auto a = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
    v = min((int)a[0], (int)a[1]);
    auto b = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
    return min((int)b[0], (int)b[1]);
}
__device__ __forceinline__ int wave_max_i(int v) { return ~wave_min_i(~v); }

// (`on`: the lanes whose pixels count)
__device__ __forceinline__ PackBox pack_box(const PixelOfItem& p, bool on) {
    PackBox b;
    b.x0 = readfirstlane(wave_min_i(on ? p.px : 0x7fffffff));
    b.x1 = readfirstlane(wave_max_i(on ? p.px : -1));
    b.y0 = readfirstlane(wave_min_i(on ? p.py : 0x7fffffff));
    b.y1 = readfirstlane(wave_max_i(on ? p.py : -1));
    return b;
}

// Conservative pack culling of one record.  For conics with condition
// number below ~1000 -- where both the binary32 decision and this binary32
// test err by well under 0.1 % -- a record is dropped when the box of the
// pack's pixel centres lies outside the cut-off ellipse's bounding box (with
// 1 % and one pixel of margin) or when the minimum of the quadratic form over
// that box (0 with the centre inside, else the clamped minimum on each edge)
// exceeds the cut-off by more than 1 %.  A dropped record has d^2 > cut-off
// at every pixel of the pack, so culling changes no output.  Records with
// worse conditioning are always kept.
__device__ __forceinline__ bool pack_keeps(float4 h0, float qc, const PackBox& b, float cut) {
    float a = h0.z, bq = 0.5f * h0.w, c = qc;
    float det = a * c - bq * bq;
    float tr = a + c;
    if (!(det > 0.f) || tr * tr >= 1000.f * det) return true;
    float idet = __builtin_amdgcn_rcpf(det);
    float ex = __builtin_sqrtf(1.01f * cut * c * idet) + 1.f;
    float ey = __builtin_sqrtf(1.01f * cut * a * idet) + 1.f;
    float lx = ((float)b.x0 + 0.5f) - h0.x, hx = ((float)b.x1 + 0.5f) - h0.x;
    float ly = ((float)b.y0 + 0.5f) - h0.y, hy = ((float)b.y1 + 0.5f) - h0.y;
    if (lx > ex || hx < -ex || ly > ey || hy < -ey) return false;
    if (lx <= 0.f && hx >= 0.f && ly <= 0.f && hy >= 0.f) return true;
    float ia = __builtin_amdgcn_rcpf(a), ic = __builtin_amdgcn_rcpf(c);
    auto q = [&](float x, float y) { return a * x * x + 2.f * bq * x * y + c * y * y; };
    float y0 = fminf(fmaxf(-bq * lx * ic, ly), hy), y1 = fminf(fmaxf(-bq * hx * ic, ly), hy);
    float x0 = fminf(fmaxf(-bq * ly * ia, lx), hx), x1 = fminf(fmaxf(-bq * hy * ia, lx), hx);
    float m = fminf(fminf(q(lx, y0), q(hx, y1)), fminf(q(x0, ly), q(x1, hy)));
    return m <= 1.01f * cut;
}

// One batch of up to 64 pair-order records, one per lane, held in registers
// (prefetched while the previous batch is composited).  Callers guarantee
// j0 < j1, so lanes past the end re-load record j0 instead of branching
// (keeps the batch in registers).  {n^c, h} is left out: the compositing
// passes read it only for the depth-hit record of a pixel.
struct Batch {
    float4 r0, r1, r2;
    bool ok;
};

__device__ __forceinline__ Batch load_batch(const WS& w, uint32_t j0, uint32_t j1, int lane) {
    Batch B;
    uint32_t j = j0 + (uint32_t)lane;
    B.ok = j < j1;
    const float4* src = w.prec + 4ull * (B.ok ? j : j0);
    B.r0 = src[0];
    B.r1 = src[1];
    B.r2 = src[2];
    return B;
}

// A record's depth-hit test dd <= cut && dd < tau as one comparison,
// dd < min(tau, the next float above cut).
__device__ __forceinline__ float hit_bound(float tau, float cut) {
    return fminf(tau, __uint_as_float(__float_as_uint(cut) + 1u));
}

// Iterates the work items of one wave: round-robin over the first n_static
// items (item k to wave k mod waves), then chunks of items_per_pop
// consecutive items from an atomic queue head over the rest.  n_static is
// every item with items_per_pop = 0, none with static_share = 0, else
// static_share percent of them (a whole number of rounds).  Only as many waves
// as there are chunks pop: each chunk is one successful pop, and with few
// items the pops of thousands of waves that find nothing queue up on the one
// counter (55 us of a launch over 50 items).  A launch leaves the head at zero
// for the next; with a launch of its own to clear it before each, a step of
// 4,239 Gaussians in three frames took 70 us, 66 so.
struct ItemIter {
    uint32_t it, end, n_items, n_static, ipp, stride, last;
    uint32_t* queue;
    int lane;
    bool dyn, pops;
    __device__ __forceinline__ bool next(uint32_t& out) {
        if (!dyn) {
            if (it < n_static) {
                out = it;
                it += stride;
                return true;
            }
            if (!pops) return false;
            dyn = true;
            it = end = 0;
        }
        if (it >= end) {
            uint32_t it0 = 0;
            if (lane == 0) {
                it0 = atomicAdd(queue, ipp);
                if (it0 == last) *queue = 0u;
            }
            it0 = n_static + (uint32_t)readfirstlane((int)it0);
            if (it0 >= n_items) return false;
            it = it0;
            end = min(it0 + ipp, n_items);
        }
        out = it;
        it += 1u;
        return true;
    }
};

__device__ __forceinline__ ItemIter make_iter(int items_per_pop, int static_share, uint32_t n_items,
                                             uint32_t* queue, int lane) {
    ItemIter I;
    I.n_items = n_items;
    I.ipp = (uint32_t)items_per_pop;
    I.queue = queue;
    I.lane = lane;
    I.stride = gridDim.x * 4u;
    I.it = (uint32_t)readfirstlane((int)(blockIdx.x * 4u + (threadIdx.x >> 6)));
    I.end = 0;
    I.dyn = false;
    const uint32_t wave = I.it;
    I.n_static = I.ipp == 0 ? n_items
                            : (uint32_t)((uint64_t)n_items * (uint32_t)static_share / 100u / I.stride * I.stride);
    // (as many waves as there are chunks, each of which ends on one pop too
    // many: the last of all pops finds the head at `last` and clears it)
    const uint32_t chunks = I.ipp ? (n_items - I.n_static + I.ipp - 1u) / I.ipp : 0u;
    I.pops = wave < chunks;
    I.last = (chunks + min(chunks, I.stride) - 1u) * I.ipp;
    return I;
}

// Cross-lane sums.  swap32 / swap16: the gfx950 permlane swaps followed by
// one add leave each half (of the wave, of a row pair) with its own value's
// partial sum.  mirror_sum<CTRL>: lane pairs that differ in a lane bit `hi`;
// the lane with the bit clear keeps a, the other b, each with the
// partner's share added.
__device__ __forceinline__ float swap32_sum(float a, float b) {
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_sum(float a, float b) {
    auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
template <int CTRL>
__device__ __forceinline__ float mirror_sum(float a, float b, bool hi) {
    float send = hi ? a : b;
    float keep = hi ? b : a;
    return keep + dpp_mov<CTRL>(send);
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kHalfMirror = 0x141, kMirror = 0x140;   // DPP controls

// Wave totals of five values: lane l returns that of slot b5 + 2 b4 + 4 b3
// (b_k = bit k of l), slots 5-7 zero.
__device__ __forceinline__ float reduce_scatter5(const float (&v)[5], int lane) {
    const float r0 = swap32_sum(v[0], v[1]), r1 = swap32_sum(v[2], v[3]), r2 = swap32_sum(v[4], 0.f);
    const float q0 = swap16_sum(r0, r1), q1 = swap16_sum(r2, 0.f);
    float t = mirror_sum<kMirror>(q0, q1, (lane >> 3) & 1);
    t += dpp_mov<kHalfMirror>(t);
    t += dpp_mov<kXor2>(t);
    return t + dpp_mov<kXor1>(t);
}

// Totals of eight values over each group of eight lanes: lane l returns
// that of slot b2 + 2 b1 + 4 b0.
__device__ __forceinline__ float oct_scatter8(const float (&v)[8], int lane) {
    const bool b2 = (lane >> 2) & 1, b1 = (lane >> 1) & 1, b0 = lane & 1;
    float t[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = mirror_sum<kHalfMirror>(v[2 * j], v[2 * j + 1], b2);
    const float u0 = mirror_sum<kXor2>(t[0], t[1], b1), u1 = mirror_sum<kXor2>(t[2], t[3], b1);
    return mirror_sum<kXor1>(u0, u1, b0);
}
__device__ __forceinline__ float oct_sum(float t) {
    t += dpp_mov<kHalfMirror>(t);
    t += dpp_mov<kXor2>(t);
    return t + dpp_mov<kXor1>(t);
}

// The Gaussian weight exp(-d^2 / 2) of both compositing kernels, as one
// multiply and the hardware base-2 exponential (the forward and the
// backward must evaluate it identically: the backward recovers the
// transmission by dividing out the forward's factors).
__device__ __forceinline__ float gauss_weight(float dd) {
    return __builtin_amdgcn_exp2f(dd * -0.72134752044448170f);   // -log2(e) / 2
}

// Lane k's value (k the same on every lane).
__device__ __forceinline__ uint32_t rdl_u(uint32_t v, int k) { return (uint32_t)__builtin_amdgcn_readlane((int)v, k); }

// What the value path takes from a record's centre residual lo = mu -
// fl32(mu): with d the offsets from the binary32 centre, (d - lo)^T Q (d -
// lo) = dd + e . d + q(lo), e = -2 Q lo, so the value distance is the
// decision distance plus two multiply-adds, and q(lo) goes into the opacity,
// alpha' = alpha exp(-q(lo) / 2).  (A second evaluation of the form took
// eight operations per pixel and record.)  Precise records take neither:
// their value distance comes from the whitened offsets.
struct Resid {
    float e0, e1, alpha;
};
__device__ __forceinline__ Resid resid_of(const float4& A, const float4& Bq, const float4& Cc) {
    if (rec_precise(Cc)) return Resid{0.f, 0.f, Bq.y};
    float lx, ly;
    mu_lo(Cc.w, lx, ly);
    const float e0 = -__builtin_fmaf(2.f * A.z, lx, A.w * ly), e1 = -__builtin_fmaf(2.f * Bq.x, ly, A.w * lx);
    return Resid{e0, e1, Bq.y * gauss_weight(-0.5f * __builtin_fmaf(e0, lx, e1 * ly))};
}

// Decision distance dd (the fixed sequence) and the offsets d.
__device__ __forceinline__ float eval_dd(const float4& A, float qyy, float ux, float uy, float& dx, float& dy) {
    dx = ux - A.x;
    dy = uy - A.y;
    return __builtin_fmaf(qyy * dy, dy, __builtin_fmaf(A.w * dx, dy, (A.z * dx) * dx));
}

// Value opacity f = min(alpha exp(-d_v^2 / 2), 0.99) of a record that is
// not precise; every compositing path takes the same sequence.
__device__ __forceinline__ float eval_f(float dd, float dx, float dy, const Resid& r) {
    return fminf(r.alpha * gauss_weight(__builtin_fmaf(r.e0, dx, __builtin_fmaf(r.e1, dy, dd))), 0.99f);
}

// The same of a precise record (its row of recp at r).
__device__ __forceinline__ float eval_f_precise(const float4& A, float alpha, const float* r, float ux, float uy,
                                                float dx, float dy) {
    float e0, e1;
    precise_offsets(r, ux, uy, A.x, A.y, dx, dy, e0, e1);
    return fminf(alpha * gauss_weight(e0 * e0 + e1 * e1), 0.99f);
}

// One wave's compacted batch in LDS: {mu.x, mu.y, Q.xx, 2 Q.xy}, {Q.yy,
// alpha', hit bound, c.r}, {c.g, c.b, e0, e1} per surviving record in list
// order, then kPad records whose d^2 is NaN at every pixel (no comparison
// holds), so that the passes work in whole groups.  In the alpha-blended depth
// mode they carry the index of a record of the list: the depth that the passes
// read by it, with weight zero, must be a number, and the word of a Gaussian
// that the frame does not see is never written.
constexpr int kPad = 3;
struct Slice {
    float4 r[3][64 + kPad];
    uint32_t pos[64];         // absolute pair position (forward), residual word (backward)
    uint32_t gid[64 + kPad];  // index word
};

// Pack-cull the batch and compact the survivors into the wave's slice;
// returns the lanes that hold one.
template <bool BWD, int DM>
__device__ __forceinline__ uint64_t compact_batch(const Batch& B, uint32_t j0, Slice& S, int lane, const PackBox& pb,
                                                  float cut) {
    const bool keep = B.ok && pack_keeps(B.r0, B.r1.x, pb, cut);
    const uint64_t m = ballot(keep);
    const uint32_t n = (uint32_t)__builtin_popcountll(m);
    if (keep) {
        const uint32_t q = (uint32_t)__builtin_popcountll(m & ((1ull << lane) - 1ull));
        const Resid r = resid_of(B.r0, B.r1, B.r2);
        S.r[0][q] = B.r0;
        S.r[1][q] = make_float4(B.r1.x, r.alpha, hit_bound(B.r1.z, cut), B.r1.w);
        S.r[2][q] = make_float4(B.r2.x, B.r2.y, r.e0, r.e1);
        S.pos[q] = BWD ? __float_as_uint(B.r2.w) : j0 + (uint32_t)lane;
        S.gid[q] = __float_as_uint(B.r2.z);
    }
    // (lane 0 holds a record of the list, kept or not)
    const uint32_t listed = DM == 1 ? rdl_u(__float_as_uint(B.r2.z), 0) & kGidMask : 0u;
    if (lane < kPad) {
        S.r[0][n + lane] = make_float4(__builtin_nanf(""), 0.f, 1.f, 0.f);
        S.r[1][n + lane] = make_float4(0.f, 0.f, -1.f, 0.f);
        S.r[2][n + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
        S.gid[n + lane] = listed;
    }
    return m;
}

// DM = 0: the depth of Eq. 4-5 (first hit, disc plane or centre); DM = 1:
// the alpha-blended depth sum_i z_i f_i T_i of the depth-rendering ablation
// (z_i the record's binary32 camera depth, -1 where nothing blends), with
// the index map still by the first hit.  ONCE: for a threshold t_eps above 1,
// where a pixel blends the first record that reaches it and stops, whatever its
// transmission then is (a variant, since the test costs the others registers).
template <int DM, bool ONCE>
__global__ RTG_FWD_BOUNDS void k_raster_fwd(Dims d, WS w, float* __restrict__ out_c,
                                                 float* __restrict__ out_d, float* __restrict__ out_t,
                                                 int* __restrict__ out_i) {
    __shared__ Slice slices[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    Slice& S = slices[wv];
    ItemIter iter = make_iter(d.fwd_items_per_pop, d.fwd_static_share, w.hdr->n_items, &w.hdr->q_fwd, lane);
    // (read beside the item count: later it would meet the queue on its line)
    const uint32_t blend_row = w.hdr->part_row == 1u ? 3u : 1u;
    float cnt_eval = 0.f;
    unsigned long long cnt_blend = 0;   // of the whole wave
    const float cut = d.cutoff2, teps = d.t_eps;
    uint32_t it;
    while (iter.next(it)) {
        PixelOfItem p = decode_item(d, w, it, lane);
        PackBox pb = pack_box(p, p.act);
        uint64_t boxed = ballot(p.act);   // the pixels pb holds
        // a pixel is done with its colour once T < t_eps; lanes without one
        // start there
        float T = p.act ? 1.f : -1.f, C0 = 0.f, C1 = 0.f, C2 = 0.f, Da = 0.f;
        uint32_t last = p.rs, hitpos = 0;
        int hitk = -1, lastk = -1;
        bool ddone = !p.act, blended = false;
        Batch B = {};
        if (p.rs < p.re) B = load_batch(w, p.rs, p.re, lane);
        // the frame is the same for every lane of the pack: a scalar base
        const float* rpf = w.recp + 6 * ((int64_t)readfirstlane(p.f) * d.N);
        const float* zf = w.zkey + (int64_t)readfirstlane(p.f) * d.N;
        for (uint32_t b = p.rs; b < p.re; b += 64) {
            const bool prec = B.ok && rec_precise(B.r2);
            const uint64_t kept = compact_batch<false, DM>(B, b, S, lane, pb, cut);
            const uint32_t nb = (uint32_t)__builtin_popcountll(kept);
            const bool anyp = (ballot(prec) & kept) != 0;
            wave_lds_sync();
            if (b + 64 < p.re) B = load_batch(w, b + 64, p.re, lane);
            // groups of G records, specialised on whether the batch holds a
            // precise record (the value distance of those comes from the
            // factored form); the slice is padded to whole groups with
            // records that reach no pixel
            auto groups = [&](auto prec) -> bool {
                constexpr bool PR = decltype(prec)::value;
                constexpr int G = PR ? 1 : RTG_FWD_GROUP;
                for (uint32_t k0 = 0; k0 < nb; k0 += G) {
                    float4 A[G], Bq[G], Cc[G];
#pragma unroll
                    for (int u = 0; u < G; ++u) {
                        A[u] = S.r[0][k0 + u];
                        Bq[u] = S.r[1][k0 + u];
                        Cc[u] = S.r[2][k0 + u];
                    }
                    // independent part: decision, value, opacity
                    float fvq[G], ddq[G];
#pragma unroll
                    for (int u = 0; u < G; ++u) {
                        float dx, dy;
                        ddq[u] = eval_dd(A[u], Bq[u].x, p.ux, p.uy, dx, dy);
                        fvq[u] = eval_f(ddq[u], dx, dy, Resid{Cc[u].z, Cc[u].w, Bq[u].y});
                        if constexpr (PR) {
                            const uint32_t gw = (uint32_t)readfirstlane((int)S.gid[k0 + u]);
                            if (gw & kPreciseBit)
                                fvq[u] = eval_f_precise(A[u], Bq[u].y, rpf + 6 * (int64_t)(gw & kGidMask), p.ux, p.uy,
                                                        dx, dy);
                        }
                    }
                    // sequential part: compositing in list order
#pragma unroll
                    for (int u = 0; u < G; ++u) {
                        bool take = ddq[u] <= cut && !(T < teps);
                        if constexpr (ONCE) take = ddq[u] <= cut && p.act && last == p.rs && lastk < 0;
                        lastk = take ? (int)(k0 + u) : lastk;
                        const float fv = take ? fvq[u] : 0.f;
                        const float wgt = fv * T;
                        C0 = __builtin_fmaf(Bq[u].w, wgt, C0);
                        C1 = __builtin_fmaf(Cc[u].x, wgt, C1);
                        C2 = __builtin_fmaf(Cc[u].y, wgt, C2);
                        if constexpr (DM == 1) {
                            // the record is the same on every lane: a scalar load
                            const float z = zf[readfirstlane((int)(S.gid[k0 + u] & kGidMask))];
                            Da = __builtin_fmaf(z, wgt, Da);
                            blended = blended || take;
                        }
                        T = __builtin_fmaf(-fv, T, T);
                        cnt_blend += (unsigned long long)__builtin_popcountll(ballot(take));
                    }
                    // (a uniform branch: a pixel's depth hit comes once)
                    bool h = false;
#pragma unroll
                    for (int u = 0; u < G; ++u) h = h || ddq[u] < Bq[u].z;
                    h = h && !ddone;
                    if (ballot(h) != 0) {
#pragma unroll
                        for (int u = G - 1; u >= 0; --u)
                            if (h && ddq[u] < Bq[u].z) hitk = (int)(k0 + u);
                        ddone = ddone || h;
                    }
                    if (((k0 + G) & 7) == 0 && ballot(!(T < teps && ddone)) == 0) return true;
                }
                return false;
            };
            bool all_done;
            if constexpr (ONCE) all_done = groups(std::true_type{});
            else all_done = anyp ? groups(std::true_type{}) : groups(std::false_type{});
            // list positions of this batch's last blend and depth hit, and the
            // hit's normal and plane offset, before the slice is reused
            if (lastk >= 0) {
                last = S.pos[lastk] + 1;
                lastk = -1;
            }
            if (hitk >= 0) {
                hitpos = S.pos[hitk] + 1;
                hitk = -1;
            }
            wave_lds_sync();
            const uint64_t live = ballot(!(T < teps && ddone));
            if (all_done || live == 0) break;
            // culling the rest of the list for the pixels still open only
            if (live != boxed) {
                pb = pack_box(p, !(T < teps && ddone));
                boxed = live;
            }
        }
        const uint32_t cterm = T < teps ? last : p.re;
        cnt_eval += p.act ? (float)(max(cterm, hitpos ? hitpos : p.re) - p.rs) : 0.f;
        if (p.act) {
            size_t pix = ((size_t)p.f * d.H + p.py) * d.W + p.px;
            out_c[3 * pix + 0] = C0;
            out_c[3 * pix + 1] = C1;
            out_c[3 * pix + 2] = C2;
            out_t[pix] = T;
            const float4* hr = w.prec + 4ull * (hitpos ? hitpos - 1u : 0u);
            const int hit = hitpos ? rec_gid(hr[2]) : -1;
            float D = -1.f;
            if constexpr (DM == 1) {
                D = blended ? Da : -1.f;
            } else if (hit >= 0) {
                const float4 hn = hr[3];
                if (plane_branch(d, hn.x, hn.y, hn.z, p.ux, p.uy)) {
                    double d0 = ((double)p.ux - d.cx) / d.fx, d1 = ((double)p.uy - d.cy) / d.fy;
                    double dn = ((double)hn.x * d0 + (double)hn.y * d1) + (double)hn.z;
                    D = (float)((double)hn.w / dn);
                } else {
                    D = w.zkey[(int64_t)p.f * d.N + hit];
                }
            }
            out_d[pix] = D;
            out_i[pix] = hit;
            reinterpret_cast<uint2*>(w.px_aux)[(size_t)p.ft * d.tarea + p.r] = make_uint2(last, hitpos);
        }
    }
    // per-wave counters: no shared-address atomics
    {
        float se = wave_sum(cnt_eval);
        uint32_t gw = blockIdx.x * 4u + (uint32_t)wv;
        if (lane == 0 && gw < (uint32_t)kMaxWaves) {
            w.wcount[gw] = (unsigned long long)se;
            w.wcount[blend_row * kMaxWaves + gw] = cnt_blend;
        }
        if (lane == 0 && gw == 0) {
            w.hdr->fwd_waves = gridDim.x * 4u;
            w.hdr->blend_row = blend_row;
        }
    }
}

// The upstream gradients come from gC / gD, or, with `l1` set, are the L1
// loss of Eq. 7-8 at unit scale: sign(C - C*) per channel and, on pixels
// with a hit and a valid target, sign(D - D*) (out_c, tgt_c, tgt_d the
// rendered colour and the targets).  Both gradient paths are linear in
// their upstream, so the projection backward applies w_c / (3 |M|) to the
// colour slots and w_d / |M_D| to the depth slots; each workgroup leaves its
// sums of |C - C*|, |D - D*| and its count of M_D pixels in lwave for that.
struct L1Up {
    const float* out_c;
    const float* tgt_c;
    const float* tgt_d;
    int l1;
};

// Gradients of the unstable records, kQ at a time.  Walking a pixel's list
// is serial, so there the wave has one pixel per lane and only leaves two
// numbers per record and pixel in LDS: e = dL/df g and w = f T (zero where the
// pixel takes no part).  Once kQ records are held, the wave turns round: eight
// lanes per record, each adding up eight pixels' moments of e about the
// record's centre and their colour sums in registers, then one
// reduce-scatter over the eight lanes and one float atomic per value.  That
// takes about 23 vector operations per record, where reducing nine values
// across the wave for every record took about 60.
constexpr int kQ = 8, kQLanes = 64 / kQ;
struct GradQueue {
    float2 ew[kQ][64 + 8];      // e, w per pixel (rows staggered over the banks)
    float4 px[64];              // ux, uy, g0, g1 per pixel
    float2 px2[64];             // g2, gD
    float4 ra[kQ], rb[kQ];      // {mu, Q.xx, 2 Q.xy}, {Q.yy, alpha', residual word, index word}
};

// Parameters of the records held since the last call (their places in the
// slice one byte each in qk), before the slice is reused or they are summed.
__device__ __forceinline__ void queue_records(GradQueue& G, const Slice& S, int lane, int n0, int n, uint64_t qk) {
    if (lane >= n0 && lane < n) {
        const int k = (int)((qk >> (8 * lane)) & 63u);
        G.ra[lane] = S.r[0][k];
        const float4 b = S.r[1][k];
        G.rb[lane] = make_float4(b.x, b.y, __uint_as_float(S.pos[k]), __uint_as_float(S.gid[k]));
    }
}

// The held records' sums into their gradient rows (slots 0-8, and 13 with
// the alpha-blended depth); grad is the frame's first row, rpf its recp.
template <int DM>
__device__ __forceinline__ void queue_sums(const GradQueue& G, int lane, int n, bool anyp, const float* rpf,
                                           float* grad) {
    const int r = lane / kQLanes, s = lane % kQLanes;
    const int rr = r < n ? r : 0;
    const float4 a = G.ra[rr], b = G.rb[rr];
    const uint32_t gw = __float_as_uint(b.w);
    const bool prec = (gw & kPreciseBit) != 0u;
    float lx, ly;
    mu_lo(b.z, lx, ly);
    float s0 = 0.f, sx = 0.f, sy = 0.f, sxx = 0.f, sxy = 0.f, syy = 0.f, w0 = 0.f, w1 = 0.f, w2 = 0.f, wd = 0.f;
    struct Px {
        float2 ew, p2;
        float4 p;
    };
    auto load = [&](int i) {
        const int k = s + kQLanes * i;
        return Px{G.ew[rr][k], G.px2[k], G.px[k]};
    };
    auto add = [&](const Px& q, float dx, float dy) {
        const float ex = q.ew.x * dx, ey = q.ew.x * dy;
        s0 += q.ew.x;
        sx = __builtin_fmaf(q.ew.x, dx, sx);
        sy = __builtin_fmaf(q.ew.x, dy, sy);
        sxx = __builtin_fmaf(ex, dx, sxx);
        sxy = __builtin_fmaf(ex, dy, sxy);
        syy = __builtin_fmaf(ey, dy, syy);
        w0 = __builtin_fmaf(q.p.z, q.ew.y, w0);
        w1 = __builtin_fmaf(q.p.w, q.ew.y, w1);
        w2 = __builtin_fmaf(q.p2.x, q.ew.y, w2);
        if constexpr (DM == 1) wd = __builtin_fmaf(q.p2.y, q.ew.y, wd);   // dL/dz of the blended depth
    };
    if (!anyp) {
        Px q = load(0);
#pragma unroll
        for (int i = 0; i < 64 / kQLanes; ++i) {
            // (one pixel ahead, no more: registers)
            const Px nx = load(i + 1 < 64 / kQLanes ? i + 1 : i);
            __builtin_amdgcn_sched_barrier(0);
            add(q, (q.p.x - a.x) - lx, (q.p.y - a.y) - ly);
            q = nx;
        }
    } else {
        // precise records: the whitened offsets e = U (u - mu), Q = U^T U;
        // their slots hold sum g e and sum g e e^T, which the projection
        // backward maps back through U
#pragma unroll 1
        for (int i = 0; i < 64 / kQLanes; ++i) {
            const Px q = load(i);
            const float dxd = q.p.x - a.x, dyd = q.p.y - a.y;
            float dx = dxd - lx, dy = dyd - ly;
            if (prec) precise_offsets(rpf + 6 * (int64_t)(gw & kGidMask), q.p.x, q.p.y, a.x, a.y, dxd, dyd, dx, dy);
            add(q, dx, dy);
        }
    }
    // d^2 enters f as exp(-d^2 / 2): h = -alpha' / 2; alpha' = alpha q0
    const float h = -0.5f * b.y, h2 = -2.f * h;
    const float qxx = a.z, qxy = 0.5f * a.w, qyy = b.x;
    const float q0 = prec ? 1.f : gauss_weight(__builtin_fmaf(__builtin_fmaf(qxx, lx, a.w * ly), lx, (qyy * ly) * ly));
    float v[8];
    v[0] = prec ? h * sx : h2 * __builtin_fmaf(qxx, sx, qxy * sy);
    v[1] = prec ? h * sy : h2 * __builtin_fmaf(qyy, sy, qxy * sx);
    v[2] = h * sxx;
    v[3] = -h2 * sxy;
    v[4] = h * syy;
    v[5] = q0 * s0;
    v[6] = w0;
    v[7] = w1;
    const float t = oct_scatter8(v, lane), t8 = oct_sum(w2);
    float t13 = 0.f;
    if constexpr (DM == 1) t13 = oct_sum(wd);
    if (r >= n) return;
    float* row = grad + 16 * (int64_t)(gw & kGidMask);
    atomic_add_f32(row + (((s >> 2) & 1) + 2 * ((s >> 1) & 1) + 4 * (s & 1)), t);
    if (s == 0) atomic_add_f32(row + 8, t8);
    if constexpr (DM == 1)
        if (s == 1) atomic_add_f32(row + 13, t13);
}

// Depth-path terms (Eq. 4-5) of the pixels whose depth hit is an unstable
// Gaussian, slots 9-13 of its row: the pixels that share a hit are summed
// over the wave, one round per distinct hit.
__device__ __forceinline__ void depth_hits(const Dims& d, const WS& w, const PixelOfItem& p, int lane, uint32_t hitpos,
                                           float gd, float D, float* grad) {
    uint32_t gw = 0u;
    float v[5] = {0.f, 0.f, 0.f, 0.f, 0.f};
    if (hitpos) {
        const float4* hr = w.prec + 4ull * (hitpos - 1u);
        gw = __float_as_uint(hr[2].z);
        if (gw & kUnstableBit) {
            const float4 nh = hr[3];
            if (plane_branch(d, nh.x, nh.y, nh.z, p.ux, p.uy)) {
                const float rx = (float)(((double)p.ux - d.cx) / d.fx);
                const float ry = (float)(((double)p.uy - d.cy) / d.fy);
                const float dn = (nh.x * rx + nh.y * ry) + nh.z;
                v[0] = gd / dn;
                const float aD = v[0] * D;
                v[1] = aD * rx;
                v[2] = aD * ry;
                v[3] = aD;
            } else {
                v[4] = gd;
            }
        }
    }
    for (uint64_t m = ballot((gw & kUnstableBit) != 0u); m != 0;) {
        const uint32_t hw = rdl_u(gw, __builtin_ctzll(m));
        const bool mine = gw == hw;
        m &= ~ballot(mine);
        float u[5];
#pragma unroll
        for (int k = 0; k < 5; ++k) u[k] = mine ? v[k] : 0.f;
        const float t = reduce_scatter5(u, lane);
        const int slot = ((lane >> 5) & 1) + 2 * ((lane >> 4) & 1) + 4 * ((lane >> 3) & 1);
        if ((lane & 7) == 0 && slot < 5) atomic_add_f32(grad + 16 * (int64_t)(hw & kGidMask) + 9 + slot, t);
    }
}

// The records of the slice (bit k) that reach a pixel of the pack before its
// last entry: the first kl of this lane's.
__device__ __forceinline__ uint64_t reached(const Slice& S, const PixelOfItem& p, int kl, float cut) {
    uint64_t m = 0;
#pragma unroll 1
    for (int k = 0; ballot(k < kl) != 0; ++k) {
        float dx, dy;
        const float dd = eval_dd(S.r[0][k], S.r[1][k].x, p.ux, p.uy, dx, dy);
        if (ballot(dd <= cut && k < kl) != 0) m |= 1ull << k;
    }
    return m;
}

template <int DM>
__global__ RTG_BWD_BOUNDS void k_raster_bwd(Dims d, WS w, const float* __restrict__ out_d,
                                                 const float* __restrict__ out_t,
                                                 const int* __restrict__ out_i,
                                                 const float* __restrict__ gC,
                                                 const float* __restrict__ gD, L1Up up) {
    __shared__ Slice slices[4];
    __shared__ GradQueue queues[4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    Slice& S = slices[wv];
    GradQueue& GQ = queues[wv];
    ItemIter iter = make_iter(d.items_per_pop, d.static_share, w.hdr->n_items, &w.hdr->q_bwd, lane);
    float l1 = 0.f;   // the wave's L1 sums: colour in lane 0, depth in lane 1, depth count in lane 2
    const float cut = d.cutoff2;
    float cnt_walk = 0.f;
    (void)out_i;   // the depth hit is identified by its list position
    uint32_t it;
    while (iter.next(it)) {
        PixelOfItem p = decode_item(d, w, it, lane);
        size_t pix = ((size_t)p.f * d.H + p.py) * d.W + p.px;
        float Tc = 1.f, g0 = 0.f, g1 = 0.f, g2 = 0.f, gd = 0.f, D = -1.f;
        float ec = 0.f, ed = 0.f, nd = 0.f;
        uint32_t last = p.rs, hitpos = 0;
        if (p.act) {
            Tc = out_t[pix];
            D = out_d[pix];
            if (up.l1) {
                const float e0 = up.out_c[3 * pix] - up.tgt_c[3 * pix];
                const float e1 = up.out_c[3 * pix + 1] - up.tgt_c[3 * pix + 1];
                const float e2 = up.out_c[3 * pix + 2] - up.tgt_c[3 * pix + 2];
                g0 = sgn(e0);
                g1 = sgn(e1);
                g2 = sgn(e2);
                const float dt = up.tgt_d[pix];
                const bool vd = D != -1.f && dt > 0.f;
                gd = vd ? sgn(D - dt) : 0.f;
                ec = fabsf(e0) + fabsf(e1) + fabsf(e2);
                ed = vd ? fabsf(D - dt) : 0.f;
                nd = vd ? 1.f : 0.f;
            } else {
                g0 = gC[3 * pix];
                g1 = gC[3 * pix + 1];
                g2 = gC[3 * pix + 2];
                gd = gD[pix];
            }
            uint2 aux = reinterpret_cast<const uint2*>(w.px_aux)[(size_t)p.ft * d.tarea + p.r];
            last = aux.x;
            hitpos = gd != 0.f ? aux.y : 0u;
        }
        if (up.l1) {
            const float tc = wave_sum(ec), td = wave_sum(ed), tn = wave_sum(nd);
            l1 += lane == 0 ? tc : lane == 1 ? td : lane == 2 ? tn : 0.f;
        }
        // the frame is the same for every lane of the pack: scalar bases
        const int64_t f0 = (int64_t)readfirstlane(p.f) * d.N;
        const float* rpf = w.recp + 6 * f0;
        const float* zf = w.zkey + f0;
        float* grad = w.grad + 16 * f0;
        const uint32_t jend = (uint32_t)wave_max_i((int)last);   // (pair positions are below 2^31)
        Batch B = {};
        if (jend > p.rs) B = load_batch(w, jend - p.rs > 64u ? jend - 64u : p.rs, jend, lane);
        GQ.px[lane] = make_float4(p.ux, p.uy, g0, g1);
        GQ.px2[lane] = make_float2(g2, gd);
        // an upstream that is no number times a weight of zero is none either:
        // then a record that reaches no pixel must not be summed
        const float big = fmaxf(fmaxf(fabsf(g0), fabsf(g1)), fmaxf(fabsf(g2), fabsf(gd)));
        const bool wild = ballot(!(big <= 3.4028235e38f) || g0 != g0 || g1 != g1 || g2 != g2 || gd != gd) != 0;
        // alpha-blended depth: the depth path follows the colour's
        if constexpr (DM == 0) depth_hits(d, w, p, lane, hitpos, gd, D, grad);
        // the upstream-weighted colour (and blended depth) behind: only g . A
        // enters the gradients, so one sum replaces one per channel
        float Ag = 0.f;
        int nq = 0, nq0 = 0;   // records held, and those whose parameters are
        uint64_t qk = 0;
        bool qprec = false;
        PackBox pb = {};
        uint64_t boxed = 0;   // the pixels pb holds
        for (uint32_t top = jend; top > p.rs;) {
            uint32_t b0 = top - p.rs > 64u ? top - 64u : p.rs;
            // this lane's records: the first kl of the slice lie before `last`;
            // the batch is culled for the pixels that have any
            const uint32_t lim = last > b0 ? last - b0 : 0u;
            const uint64_t open = ballot(lim != 0u);
            if (open != boxed) {
                pb = pack_box(p, lim != 0u);
                boxed = open;
            }
            const uint64_t kept = compact_batch<true, DM>(B, b0, S, lane, pb, cut);
            const int nk = __builtin_popcountll(kept);
            const int kl = __builtin_popcountll(lim >= 64u ? kept : kept & ((1ull << lim) - 1ull));
            wave_lds_sync();
            const uint32_t gwl = lane < nk ? S.gid[lane] : 0u;
            uint64_t um = ballot((gwl & kUnstableBit) != 0u);
            const uint64_t pm = ballot((gwl & kPreciseBit) != 0u);
            if (wild) um &= reached(S, p, kl, cut);
            qprec = qprec || pm != 0;
            if (b0 > p.rs) B = load_batch(w, b0 - p.rs > 64u ? b0 - 64u : p.rs, b0, lane);
            // groups of G records, specialised on whether the batch holds a
            // precise record; the next group is read from LDS while the
            // sequential part of this one runs
            auto groups = [&](auto prec) {
                constexpr bool PR = decltype(prec)::value;
                constexpr int G = RTG_BWD_GROUP;
                int k0 = nk > 0 ? (nk - 1) / G * G : -1;
                float4 A[G], Bq[G], Cc[G];
                auto load = [&](int kb) {
#pragma unroll
                    for (int u = 0; u < G; ++u) {
                        A[u] = S.r[0][kb + u];
                        Bq[u] = S.r[1][kb + u];
                        Cc[u] = S.r[2][kb + u];
                    }
                };
                if (nk > 0) load(k0);
                for (; k0 >= 0; k0 -= G) {
                    // independent part: decision, weight, 1 / (1 - f), upstream . colour
                    float gw[G], fv[G], ro[G], gc[G];
                    bool part[G], free[G];
#pragma unroll
                    for (int u = 0; u < G; ++u) {
                        const int k = k0 + u;
                        float dx, dy;
                        const float dd = eval_dd(A[u], Bq[u].x, p.ux, p.uy, dx, dy);
                        part[u] = dd <= cut && k < kl;
                        float ddv = __builtin_fmaf(Cc[u].z, dx, __builtin_fmaf(Cc[u].w, dy, dd));
                        if constexpr (PR) {
                            const uint32_t gi = (uint32_t)readfirstlane((int)S.gid[k]);
                            if (gi & kPreciseBit) {
                                float e0, e1;
                                precise_offsets(rpf + 6 * (int64_t)(gi & kGidMask), p.ux, p.uy, A[u].x, A[u].y, dx, dy,
                                                e0, e1);
                                ddv = e0 * e0 + e1 * e1;
                            }
                        }
                        gw[u] = gauss_weight(ddv);
                        const float fa = Bq[u].y * gw[u];
                        free[u] = !(fa > 0.99f);   // not clamped
                        fv[u] = fminf(fa, 0.99f);
                        // 1 / (1 - f) to binary32: one step on the hardware
                        // reciprocal, with the residual from f itself (the
                        // transmission recovered over a long list is a product
                        // of these: without the step d_pos was 5 % further from
                        // 64 bits than with per-record sums, with it 2 % nearer)
                        const float r0 = __builtin_amdgcn_rcpf(1.f - fv[u]);
                        ro[u] = __builtin_fmaf(__builtin_fmaf(fv[u], r0, 1.f - r0), r0, r0);
                        gc[u] = __builtin_fmaf(g2, Cc[u].y, __builtin_fmaf(g1, Cc[u].x, g0 * Bq[u].w));
                        if constexpr (DM == 1)
                            gc[u] = __builtin_fmaf(gd, zf[readfirstlane((int)(S.gid[k] & kGidMask))], gc[u]);
                    }
                    load(max(k0 - G, 0));
                    // (without this the compiler moves each record's
                    // evaluation behind the branch of the one before, and the
                    // chains no longer overlap)
#pragma unroll
                    for (int u = 0; u < G; ++u) asm volatile("" : "+v"(ro[u]), "+v"(gc[u]));
                    // sequential part, back to front
#pragma unroll
                    for (int u = G - 1; u >= 0; --u) {
                        const float Tb = Tc * ro[u];
                        const float gsum = gc[u] - Ag;
                        const float fp = part[u] ? fv[u] : 0.f;
                        if ((um >> (k0 + u)) & 1ull) {
                            // a stable one only moves T and the colour behind
                            const float e = part[u] && free[u] ? (gsum * Tb) * gw[u] : 0.f;
                            GQ.ew[nq][lane] = make_float2(e, fp * Tb);
                            qk |= (uint64_t)(uint32_t)(k0 + u) << (8 * nq);
                            ++nq;
                        }
                        Ag = __builtin_fmaf(fp, gsum, Ag);
                        Tc = part[u] ? Tb : Tc;
                    }
                    if (nq > kQ - G) {   // no room for another group
                        queue_records(GQ, S, lane, nq0, nq, qk);
                        wave_lds_sync();
                        queue_sums<DM>(GQ, lane, nq, qprec, rpf, grad);
                        wave_lds_sync();
                        nq = nq0 = 0;
                        qk = 0;
                        qprec = pm != 0;
                    }
                }
            };
            if (pm != 0) groups(std::true_type{});
            else groups(std::false_type{});
            if (nq > nq0) queue_records(GQ, S, lane, nq0, nq, qk);
            nq0 = nq;
            wave_lds_sync();
            top = b0;
        }
        if (nq) {
            queue_sums<DM>(GQ, lane, nq, qprec, rpf, grad);
            wave_lds_sync();
        }
        cnt_walk += (float)(last - p.rs);
    }
    {
        float sw = wave_sum(cnt_walk);
        uint32_t gw = blockIdx.x * 4u + (uint32_t)wv;
        if (lane == 0 && gw < (uint32_t)kMaxWaves) {
            w.wcount[2 * kMaxWaves + gw] = (unsigned long long)sw;
        }
        if (up.l1) {
            // one triple per workgroup (every wave reaches this point)
            __shared__ float l1red[3][4];
            if (lane < 3) l1red[lane][wv] = l1;
            __syncthreads();
            if (threadIdx.x < 3 && blockIdx.x < (uint32_t)kMaxWaves) {
                const float* t = l1red[threadIdx.x];
                w.lwave[threadIdx.x * kMaxWaves + blockIdx.x] = (t[0] + t[1]) + (t[2] + t[3]);
            }
        }
        // A record takes part in a pixel here exactly where the forward blended
        // it (the same decision, up to the same last entry): this launch's
        // contributions are that render's blends, a row that the next render
        // leaves alone.  (Counted per record they cost 5 % of the kernel: 645
        // to 675 us over 8 keyframes.)
        if (lane == 0 && gw == 0) {
            w.hdr->bwd_waves = gridDim.x * 4u;
            w.hdr->part_row = w.hdr->blend_row;
        }
    }
}

}  // namespace rtg
