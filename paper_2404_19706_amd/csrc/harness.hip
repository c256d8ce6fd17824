// Steps a6 and a10: the L1 loss of Eq. 7-8 with its upstream gradients,
// and Adam on the unstable rows (supp. Sec. C learning rates).  Both walk
// only what the iteration touches: the rendered pixel lists and the rows of
// unstable Gaussians.
#include "rtg_common.h"

namespace rtg {

// Bytes to v: 16 per store between the first and last aligned address.
__global__ __launch_bounds__(256) void k_fill_u8(uint8_t* p, size_t n, uint8_t v) {
    const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x, stride = (size_t)gridDim.x * 256;
    const size_t head = min((size_t)(-(intptr_t)p & 15), n), body = (n - head) / 16, tail = head + 16 * body;
    const uint32_t q = 0x01010101u * v;
    uint4* p4 = reinterpret_cast<uint4*>(p + head);
    for (size_t i = t; i < body; i += stride) p4[i] = make_uint4(q, q, q, q);
    if (t < head) p[t] = v;
    if (t < n - tail) p[tail + t] = v;
}

// Up to kClearMax arrays of 32-bit words, each to a value of its own: workgroup
// b writes up to kClearWords words of the array whose workgroups [first[a],
// first[a + 1]) hold it, 16 bytes per store between aligned addresses.  Bound
// by the stores; one launch, where a fill per array took as long as its launch
// (9 us a call with 5 us on the device, four of them around a view).
constexpr int kClearMax = 5;
constexpr int64_t kClearWords = 4096;
struct ClearArrays {
    uint32_t* p[kClearMax];
    int64_t n[kClearMax];
    uint32_t v[kClearMax];
    uint32_t first[kClearMax + 1];
};

__global__ __launch_bounds__(256) void k_clear(ClearArrays A) {
    int a = 0;
#pragma unroll
    for (int k = 1; k < kClearMax; ++k) a += blockIdx.x >= A.first[k];
    uint32_t* p = A.p[0];
    int64_t n = A.n[0];
    uint32_t v = A.v[0], first = 0;
#pragma unroll
    for (int k = 1; k < kClearMax; ++k)
        if (a == k) {
            p = A.p[k];
            n = A.n[k];
            v = A.v[k];
            first = A.first[k];
        }
    const int64_t b = kClearWords * (int64_t)(blockIdx.x - first);
    p += b;
    const int64_t m = min(n - b, kClearWords), t = threadIdx.x;
    const int64_t head = min((int64_t)((-(reinterpret_cast<intptr_t>(p) >> 2)) & 3), m), body = (m - head) / 4,
                  tail = head + 4 * body;
    uint4* p4 = reinterpret_cast<uint4*>(p + head);
    for (int64_t i = t; i < body; i += 256) p4[i] = make_uint4(v, v, v, v);
    if (t < head) p[t] = v;
    if (t < m - tail) p[tail + t] = v;
}

// Status of the calls on a workspace as an rtg_status value, written on the
// device (for callers that do not synchronise to read the header).
__global__ void k_status_out(WS w, int32_t* out) {
    if (threadIdx.x == 0) *out = w.hdr->overflow ? -2 : (w.hdr->err ? -5 : 0);
}

// Sums of the per-wave work counters of the last render and backward
// launches, and the count of the last binning's blocks that fell back to a
// second enumeration (nbb blocks), into the header (one workgroup; no
// host-side reduction).  The contributions of a backward launch are the blends
// of the render it followed.
__global__ __launch_bounds__(1024) void k_sum_counters(WS w, uint32_t nbb) {
    __shared__ unsigned long long part[4][16];
    __shared__ uint32_t nfail[16];
    const uint32_t fw = min(w.hdr->fwd_waves, (uint32_t)kMaxWaves), bw = min(w.hdr->bwd_waves, (uint32_t)kMaxWaves);
    const uint32_t rb = w.hdr->blend_row, rp = w.hdr->part_row;
    const uint32_t row[4] = {0u, rb, 2u, rp}, nw[4] = {fw, rb ? fw : 0u, bw, rp ? fw : 0u};
    for (int c = 0; c < 4; ++c) {
        unsigned long long v = 0;
        for (uint32_t k = threadIdx.x; k < nw[c]; k += blockDim.x) v += w.wcount[(size_t)row[c] * kMaxWaves + k];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
        if ((threadIdx.x & 63) == 0) part[c][threadIdx.x >> 6] = v;
    }
    {
        uint32_t v = 0;
        for (uint32_t k = threadIdx.x; k < nbb; k += blockDim.x) v += w.bfail[k] ? 1u : 0u;
        for (int o = 32; o > 0; o >>= 1) v += (uint32_t)__shfl_xor((int)v, o);
        if ((threadIdx.x & 63) == 0) nfail[threadIdx.x >> 6] = v;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        unsigned long long t = 0;
        for (int k = 0; k < 16; ++k) t += part[threadIdx.x][k];
        w.hdr->sums[threadIdx.x] = t;
    }
    if (threadIdx.x == 4) {
        uint32_t t = 0;
        for (int k = 0; k < 16; ++k) t += nfail[k];
        w.hdr->n_restaged = t;
    }
}

__device__ __forceinline__ bool pixel_of_rank(const Dims& d, const WS& w, int64_t idx, int& f, size_t& pix) {
    int64_t ft = idx / d.tarea;
    uint32_t r = (uint32_t)(idx - ft * d.tarea);
    if (ft >= (int64_t)d.F * d.ntiles) return false;
    if (r >= w.tile_npx[ft]) return false;
    int l = w.pix[idx];
    f = (int)(ft / d.ntiles);
    int t = (int)(ft % d.ntiles);
    int px = (t % d.tx) * d.tw + (l & (d.tw - 1));
    int py = (t / d.tx) * d.th + (l >> d.lg_tw);
    pix = ((size_t)f * d.H + py) * d.W + px;
    return true;
}

// Per-block partial sums of |C - C*| over the rendered pixels, |D - D*| and
// the count over pixels with a hit and a valid target (no shared-address
// atomics: one partial triple per block).
__global__ __launch_bounds__(256) void k_loss_partials(Dims d, WS w, const float* __restrict__ C,
                                                       const float* __restrict__ D,
                                                       const float* __restrict__ Cgt,
                                                       const float* __restrict__ Dgt, float* __restrict__ part) {
    __shared__ float red[3][4];
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int f;
    size_t pix;
    float sc = 0.f, sd = 0.f, nd = 0.f;
    if (pixel_of_rank(d, w, idx, f, pix)) {
        sc = fabsf(C[3 * pix] - Cgt[3 * pix]) + fabsf(C[3 * pix + 1] - Cgt[3 * pix + 1]) +
             fabsf(C[3 * pix + 2] - Cgt[3 * pix + 2]);
        if (D[pix] != -1.f && Dgt[pix] > 0.f) {
            sd = fabsf(D[pix] - Dgt[pix]);
            nd = 1.f;
        }
    }
    sc = wave_sum(sc);
    sd = wave_sum(sd);
    nd = wave_sum(nd);
    int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][wv] = sc;
        red[1][wv] = sd;
        red[2][wv] = nd;
    }
    __syncthreads();
    if (threadIdx.x < 3)
        part[3 * blockIdx.x + threadIdx.x] =
            (red[threadIdx.x][0] + red[threadIdx.x][1]) + (red[threadIdx.x][2] + red[threadIdx.x][3]);
}

// One workgroup: totals of the partials, the loss value.
__global__ __launch_bounds__(1024) void k_loss_final(WS w, const float* __restrict__ part, uint32_t nparts,
                                                     float w_c, float w_d, float* __restrict__ loss_out) {
    __shared__ float red[3][16];
    float a = 0.f, b = 0.f, c = 0.f;
    for (uint32_t k = threadIdx.x; k < nparts; k += 1024) {
        a += part[3 * k];
        b += part[3 * k + 1];
        c += part[3 * k + 2];
    }
    a = wave_sum(a);
    b = wave_sum(b);
    c = wave_sum(c);
    int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[0][wv] = a;
        red[1][wv] = b;
        red[2][wv] = c;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float ta = 0.f, tb = 0.f, tc = 0.f;
        for (int q = 0; q < 16; ++q) {
            ta += red[0][q];
            tb += red[1][q];
            tc += red[2][q];
        }
        uint32_t nmd = (uint32_t)tc;
        w.hdr->loss_c = ta;
        w.hdr->loss_d = tb;
        w.hdr->cnt_md = nmd;
        float nm = (float)max(w.hdr->n_px, 1u);
        loss_out[0] = w_c * ta / (3.f * nm) + w_d * tb / (float)max(nmd, 1u);
    }
}

__global__ __launch_bounds__(256) void k_loss_grad(Dims d, WS w, const float* __restrict__ C,
                                                   const float* __restrict__ D,
                                                   const float* __restrict__ Cgt,
                                                   const float* __restrict__ Dgt, float w_c, float w_d,
                                                   float* __restrict__ gC, float* __restrict__ gD) {
    int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int f;
    size_t pix;
    if (!pixel_of_rank(d, w, idx, f, pix)) return;
    float nm = (float)max(w.hdr->n_px, 1u);
    float nmd = (float)max(w.hdr->cnt_md, 1u);
    float kc = w_c / (3.f * nm);
    for (int c = 0; c < 3; ++c) gC[3 * pix + c] = kc * sgn(C[3 * pix + c] - Cgt[3 * pix + c]);
    gD[pix] = (D[pix] != -1.f && Dgt[pix] > 0.f) ? (w_d / nmd) * sgn(D[pix] - Dgt[pix]) : 0.f;
}

__global__ void k_step_inc(int32_t* step) {
    if (threadIdx.x == 0 && blockIdx.x == 0) step[0] += 1;
}

struct AdamArgs {
    float lr_pos, lr_scale, lr_rot, lr_col, lr_rest, b1, b2, eps;
    int32_t K;   // colour parameters per channel: 1 (RGB) or (D+1)^2 (SH)
};

// A workgroup lists the unstable ones of its 256 rows and walks their values
// by elements, neighbouring lanes neighbouring values of a row, so that the
// moments and wide SH rows are read contiguously (a thread per row read them
// at a stride of 52 to 232 bytes).  Bound by memory: seven accesses per value,
// whole lines where the unstable rows are scattered.
__global__ __launch_bounds__(256) void k_adam(int64_t N, float* __restrict__ pos, float* __restrict__ scale,
                                              float* __restrict__ rot, float* __restrict__ col,
                                              const uint8_t* __restrict__ unstable,
                                              const float* __restrict__ gpos, const float* __restrict__ gscale,
                                              const float* __restrict__ grot, const float* __restrict__ gcol,
                                              float* __restrict__ m, float* __restrict__ v,
                                              const int32_t* __restrict__ step, AdamArgs a) {
    __shared__ uint16_t list[256];
    __shared__ uint32_t wc[4];
    const int64_t i0 = (int64_t)blockIdx.x * 256;
    const bool un = i0 + threadIdx.x < N && unstable[i0 + threadIdx.x] != 0;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const uint64_t bits = ballot(un);
    if (lane == 0) wc[wv] = (uint32_t)__builtin_popcountll(bits);
    __syncthreads();
    uint32_t at = 0;
    for (int k = 0; k < wv; ++k) at += wc[k];
    if (un) list[at + (uint32_t)__builtin_popcountll(bits & ((1ull << lane) - 1ull))] = (uint16_t)threadIdx.x;
    const uint32_t rows = (wc[0] + wc[1]) + (wc[2] + wc[3]);
    __syncthreads();
    if (rows == 0) return;
    const float t = (float)step[0];
    const float bc1 = 1.f - powf(a.b1, t), bc2 = 1.f - powf(a.b2, t);
    const uint32_t K3 = 3u * (uint32_t)a.K, W = 10u + K3, tot = rows * W;
    // e / W for e < 256 W, W <= 58: as for a 2^-20 reciprocal above 1 / W
    const uint32_t inv = (1u << 20) / W + 1u;
    for (uint32_t e = threadIdx.x; e < tot; e += 256u) {
        const uint32_t r = (e * inv) >> 20, k = e - r * W;
        const int64_t i = i0 + list[r];
        float* __restrict__ p;
        const float* __restrict__ g;
        float lr;
        if (k < 3u) {
            p = pos + 3 * i + k;
            g = gpos + 3 * i + k;
            lr = a.lr_pos;
        } else if (k < 6u) {
            p = scale + 3 * i + (k - 3u);
            g = gscale + 3 * i + (k - 3u);
            lr = a.lr_scale;
        } else if (k < 10u) {
            p = rot + 4 * i + (k - 6u);
            g = grot + 4 * i + (k - 6u);
            lr = a.lr_rot;
        } else {
            p = col + (int64_t)K3 * i + (k - 10u);
            g = gcol + (int64_t)K3 * i + (k - 10u);
            lr = k < 13u ? a.lr_col : a.lr_rest;
        }
        const int64_t q = (int64_t)W * i + k;
        const bool log_scale = k >= 3u && k < 6u;   // scales move in their logarithm
        const float x = *p, gx = log_scale ? x * *g : *g;
        const float mk = a.b1 * m[q] + (1.f - a.b1) * gx;
        const float vk = a.b2 * v[q] + (1.f - a.b2) * gx * gx;
        m[q] = mk;
        v[q] = vk;
        const float u = (mk / bc1) / (sqrtf(vk / bc2) + a.eps);
        *p = log_scale ? x * __expf(-lr * u) : x - lr * u;
    }
}

}  // namespace rtg
