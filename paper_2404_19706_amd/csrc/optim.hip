// The steps of the mapping iteration either side of the backward (Sec. 3.2
// "Gaussian optimization", Eq. 8-9, and "Keyframes and global
// optimization"): the L2 regulariser of the transparent Gaussians, the
// confidence-weighted fusion of a window's result (Eq. 9), and the
// selection of a keyframe's pixels with the largest colour errors.
#include "rtg_common.h"

namespace rtg {

// L_reg = sum over transparent Gaussians of |p - p0|^2 + |q - q0|^2 +
// |s - s0|^2, weighted by w_reg: each workgroup (at most 1024, striding over
// the Gaussians) adds its binary64 partial sum of the weighted loss to
// loss_out[0] (one atomic per workgroup), and
// the gradient 2 w_reg (x - x0) goes onto the gradient rows of the unstable
// transparent Gaussians.
__global__ __launch_bounds__(256) void k_reg_l2(int64_t n, double w_reg, const uint8_t* __restrict__ transparent,
                                                const uint8_t* __restrict__ unstable,
                                                const float* __restrict__ pos, const float* __restrict__ scale,
                                                const float* __restrict__ rot, const float* __restrict__ pos0,
                                                const float* __restrict__ scale0, const float* __restrict__ rot0,
                                                float* __restrict__ d_pos, float* __restrict__ d_scale,
                                                float* __restrict__ d_rot, double* __restrict__ loss_out) {
    __shared__ double part[4];
    double l = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        if (!transparent[i]) continue;
        const bool un = unstable[i] != 0;
        auto term = [&](const float* x, const float* x0, float* g, int w) {
            for (int c = 0; c < w; ++c) {
                const double dx = (double)x[w * i + c] - (double)x0[w * i + c];
                l += dx * dx;
                if (un) g[w * i + c] += (float)(2.0 * w_reg * dx);
            }
        };
        term(pos, pos0, d_pos, 3);
        term(scale, scale0, d_scale, 3);
        term(rot, rot0, d_rot, 4);
    }
    for (int o = 32; o > 0; o >>= 1) l += __shfl_xor(l, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = l;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double t = (part[0] + part[1]) + (part[2] + part[3]);
        if (t != 0.0) atomicAdd(loss_out, w_reg * t);
    }
}

// Eq. 9 per Gaussian: w = (eta' - eta_prev) / eta' (a binary32 division of
// the two counts; 1 when eta' = 0), G = fl32(fl32((1 - w) G_prev) +
// fl32(w G')) for every optimised value, written over G'.  A workgroup forms
// the weights of 256 rows once and then walks each array's part of them by
// elements (V4: 16-byte aligned arrays, four per access), so that wide SH
// rows are read contiguously; a thread per row read 48 floats at a stride
// of 192 bytes.  Bound by memory: 12 bytes per value.
struct FuseArrays {
    const float* prev[4];
    float* cur[4];
    int32_t width[4];
};

template <bool V4>
__global__ __launch_bounds__(256) void k_fuse(int64_t n, const int32_t* __restrict__ eta_prev,
                                              const int32_t* __restrict__ eta_cur, FuseArrays A) {
    __shared__ float wt[256];
    const int64_t i0 = (int64_t)blockIdx.x * 256;
    const uint32_t rows = (uint32_t)(n - i0 < 256 ? n - i0 : 256);
    if (threadIdx.x < rows) {
        const int32_t ec = eta_cur[i0 + threadIdx.x];
        wt[threadIdx.x] = ec != 0 ? (float)(ec - eta_prev[i0 + threadIdx.x]) / (float)ec : 1.f;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t W = (uint32_t)A.width[k], tot = rows * W;
        // e / W for e < 256 W, W <= 48: the reciprocal is above 1 / W by less
        // than 2^-20, e times that by less than 1 / W
        const uint32_t inv = (1u << 20) / W + 1u;
        const float* __restrict__ g0 = A.prev[k] + i0 * W;
        float* __restrict__ g1 = A.cur[k] + i0 * W;
        auto mix = [&](uint32_t e, float a, float b) {
            const float w = wt[(e * inv) >> 20];
            const float x = (1.f - w) * a, y = w * b;
            return x + y;
        };
        if constexpr (V4) {
            for (uint32_t e = 4u * threadIdx.x; e + 4u <= tot; e += 1024u) {
                const float4 a = *reinterpret_cast<const float4*>(g0 + e);
                float4 b = *reinterpret_cast<const float4*>(g1 + e);
                b.x = mix(e, a.x, b.x);
                b.y = mix(e + 1u, a.y, b.y);
                b.z = mix(e + 2u, a.z, b.z);
                b.w = mix(e + 3u, a.w, b.w);
                *reinterpret_cast<float4*>(g1 + e) = b;
            }
            const uint32_t e = (tot & ~3u) + threadIdx.x;
            if (e < tot) g1[e] = mix(e, g0[e], g1[e]);
        } else {
            for (uint32_t e = threadIdx.x; e < tot; e += 256u) g1[e] = mix(e, g0[e], g1[e]);
        }
    }
}

// ---- top colour-error selection ---------------------------------------------
//
// Per frame: the colour error e = (|dC0| + |dC1|) + |dC2| of every pixel
// (binary32, as Eq. 6), its bits as an order-preserving key (e >= 0), and
// the k-th largest key found by four 8-bit radix passes (per-frame
// 256-bin histograms of the keys that share the prefix found so far; the
// frame's last workgroup to add its counts picks the bin holding the k-th
// largest); the mask takes every pixel whose key is at least that value.
//
// Bound by memory: 24 bytes per pixel of images once, then the 4-byte keys
// (52 MB for 16 frames of 1200x680, in the last-level cache) for three
// histograms and the mask.  The first histogram is taken while the keys are
// made, four pixels per thread and load where the frame size keeps frames
// 16-byte aligned; it counts into 32 interleaved copies of the bins (a lane's
// copy is its bank), since the leading digits of the errors fall into a few
// bins; the later digits spread, and one copy does.  16 frames of 1200x680:
// keys and first histogram 88 to 72 us (5.1 TB/s, the rate of a copy), a later
// histogram with its pick 33 to 12 us, the mask 26 to 11 us.

struct SelState {
    uint32_t prefix;   // high bits of the k-th largest key found so far
    uint32_t rem;      // its rank among the keys with that prefix (1-based)
    uint32_t none;     // k = 0: nothing selected
    uint32_t done;     // workgroups that have added their counts
};

constexpr int kSelCopies = 32;

// The bin b (counting from the top) whose keys hold the rem-th largest: the
// prefix gains b, rem drops by the keys in higher bins, and the histogram is
// cleared for the next digit.  256 threads or more, thread t holding bin t;
// `suf` is 257 words of LDS.
__device__ __forceinline__ void sel_pick(int shift, uint32_t* suf, uint32_t* hist, SelState* st) {
    const int t = threadIdx.x;
    const bool bin = t < 256;
    // read where the other workgroups' adds were made, past this XCD's L2
    const uint32_t c = bin ? __hip_atomic_load(&hist[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    const SelState s = *st;
    // suffix sums: suf[b] = keys in bins >= b
    if (bin) suf[t] = c;
    if (t == 0) suf[256] = 0u;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
        const uint32_t add = t + o < 256 ? suf[t + o] : 0u;
        __syncthreads();
        if (bin) suf[t] += add;
        __syncthreads();
    }
    if (!bin) return;
    // the bin with suf[b + 1] < rem <= suf[b] (exactly one when rem <= suf[0])
    if (!s.none && suf[t + 1] < s.rem && s.rem <= suf[t]) {
        st->prefix = s.prefix | ((uint32_t)t << shift);
        st->rem = s.rem - suf[t + 1];
    }
    hist[t] = 0u;
    if (t == 0) st->done = 0u;
}

// The workgroup's counts (COPIES interleaved copies of 256 bins) onto the
// frame's (thread t: bin t; the copies are read from a staggered start, a
// different bank per lane; at least 258 words, used again for the pick, since
// more than 32 KB would let a workgroup less onto a CU).  The frame's last
// workgroup then picks the digit: with a launch of its own for it, ten in
// all, one frame of 512x384 took 40 us and 16 of 1200x680 124, now 31 and 120.
template <int COPIES>
__device__ __forceinline__ void sel_flush(int shift, uint32_t* h, uint32_t* hist, SelState* st) {
    __syncthreads();
    uint32_t c = 0;
    if (threadIdx.x < 256) {
#pragma unroll
        for (int k = 0; k < COPIES; ++k) c += h[threadIdx.x * COPIES + ((k + threadIdx.x) & (COPIES - 1))];
    }
    if (c) __hip_atomic_fetch_add(&hist[threadIdx.x], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    // Every wave waits until its adds have been made in memory, then the ticket
    // is drawn: all that the last workgroup reads are those sums, so no cache
    // has to be written back (a releasing ticket writes the keys back once per
    // workgroup: 276 us).
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0)
        h[257] = __hip_atomic_fetch_add(&st->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
    __syncthreads();
    if (h[257]) sel_pick(shift, h, hist, st);
}

__device__ __forceinline__ uint32_t sel_key(float r0, float r1, float r2, float i0, float i1, float i2) {
    return __float_as_uint((fabsf(r0 - i0) + fabsf(r1 - i1)) + fabsf(r2 - i2));
}

// Keys, the histogram of their first digit and its pick.  Grid (blocks per frame,
// frames).  V4: hw a multiple of 4 and 16-byte aligned arrays, four pixels
// per thread and step.
template <bool V4>
__global__ __launch_bounds__(256) void k_sel_keys(int64_t hw, const float* __restrict__ color_r,
                                                  const float* __restrict__ color_in, uint32_t* __restrict__ keys,
                                                  uint32_t* __restrict__ hist, SelState* __restrict__ st) {
    __shared__ __attribute__((aligned(16))) uint32_t h[256 * kSelCopies];
    for (int i = threadIdx.x; i < 64 * kSelCopies; i += 256) reinterpret_cast<uint4*>(h)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    auto count = [&](uint32_t key) {
        atomicAdd(&h[(key >> 24) * kSelCopies + (threadIdx.x & (kSelCopies - 1))], 1u);
    };
    const int f = blockIdx.y;
    const int64_t t0 = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
    if constexpr (V4) {
        const float4* r = reinterpret_cast<const float4*>(color_r + 3 * hw * f);
        const float4* s = reinterpret_cast<const float4*>(color_in + 3 * hw * f);
        uint4* k4 = reinterpret_cast<uint4*>(keys + hw * f);
        for (int64_t p = t0; p < hw / 4; p += step) {
            const float4 a = r[3 * p], b = r[3 * p + 1], c = r[3 * p + 2];
            const float4 d = s[3 * p], e = s[3 * p + 1], g = s[3 * p + 2];
            uint4 k;
            k.x = sel_key(a.x, a.y, a.z, d.x, d.y, d.z);
            k.y = sel_key(a.w, b.x, b.y, d.w, e.x, e.y);
            k.z = sel_key(b.z, b.w, c.x, e.z, e.w, g.x);
            k.w = sel_key(c.y, c.z, c.w, g.y, g.z, g.w);
            k4[p] = k;
            count(k.x);
            count(k.y);
            count(k.z);
            count(k.w);
        }
    } else {
        const float* r = color_r + 3 * hw * f;
        const float* s = color_in + 3 * hw * f;
        for (int64_t p = t0; p < hw; p += step) {
            const uint32_t k = sel_key(r[3 * p], r[3 * p + 1], r[3 * p + 2], s[3 * p], s[3 * p + 1], s[3 * p + 2]);
            keys[hw * f + p] = k;
            count(k);
        }
    }
    sel_flush<kSelCopies>(24, h, hist + 256 * f, st + f);
}

__global__ __launch_bounds__(256) void k_sel_init(int32_t frames, uint32_t k, uint32_t* __restrict__ hist,
                                                  SelState* __restrict__ st) {
    const int f = blockIdx.x;
    if (f >= frames) return;
    hist[256 * f + threadIdx.x] = 0u;
    if (threadIdx.x == 0) st[f] = SelState{0u, k, k == 0u ? 1u : 0u, 0u};
}

// The histogram of a later digit, over the keys with the prefix found so
// far, and its pick.  Grid (blocks per frame, frames); 1024 threads, so that
// few workgroups add their 256 counts and draw tickets (16 frames of 1200x680:
// 17.5 us with workgroups of 256, 11.9 so).
template <bool V4>
__global__ __launch_bounds__(1024) void k_sel_hist(int64_t hw, int shift, const uint32_t* __restrict__ keys,
                                                   uint32_t* __restrict__ hist, SelState* __restrict__ st) {
    __shared__ uint32_t h[258];
    const int f = blockIdx.y;
    const uint32_t prefix = st[f].prefix;
    if (threadIdx.x < 256) h[threadIdx.x] = 0u;
    __syncthreads();
    const uint32_t hi = 0xffffffffu << (shift + 8);
    auto count = [&](uint32_t key) {
        if ((key & hi) == prefix) atomicAdd(&h[(key >> shift) & 255u], 1u);
    };
    const uint32_t* kf = keys + (int64_t)f * hw;
    const int64_t t0 = (int64_t)blockIdx.x * 1024 + threadIdx.x, step = (int64_t)gridDim.x * 1024;
    if constexpr (V4) {
        const uint4* k4 = reinterpret_cast<const uint4*>(kf);
        for (int64_t p = t0; p < hw / 4; p += step) {
            const uint4 k = k4[p];
            count(k.x);
            count(k.y);
            count(k.z);
            count(k.w);
        }
    } else {
        for (int64_t p = t0; p < hw; p += step) count(kf[p]);
    }
    sel_flush<1>(shift, h, hist + 256 * f, st + f);
}

// Grid (blocks per frame, frames).
template <bool V4>
__global__ __launch_bounds__(256) void k_sel_mask(int64_t hw, const uint32_t* __restrict__ keys,
                                                  const SelState* __restrict__ st, uint8_t* __restrict__ mask) {
    const int f = blockIdx.y;
    const SelState s = st[f];
    const uint32_t* kf = keys + (int64_t)f * hw;
    uint8_t* mf = mask + (int64_t)f * hw;
    auto on = [&](uint32_t key) { return !s.none && key >= s.prefix ? 1u : 0u; };
    const int64_t t0 = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
    if constexpr (V4) {
        const uint4* k4 = reinterpret_cast<const uint4*>(kf);
        uint32_t* m4 = reinterpret_cast<uint32_t*>(mf);
        for (int64_t p = t0; p < hw / 4; p += step) {
            const uint4 k = k4[p];
            m4[p] = on(k.x) | on(k.y) << 8 | on(k.z) << 16 | on(k.w) << 24;
        }
    } else {
        for (int64_t p = t0; p < hw; p += step) mf[p] = (uint8_t)on(kf[p]);
    }
}

}  // namespace rtg
