// Frame-to-model tracking (Sec. 3.2 "Camera tracking", Eq. 10) on the
// rasterizer's outputs: the rendered normal map (Sec. 3.1, the hit
// Gaussian's normal per pixel) and a multi-level projective point-to-plane
// ICP of an input depth frame against the rendered depth and normals.
//
// One launch per iteration: each workgroup first adds the partial normal
// equations of the iteration before in a fixed order, solves the 6x6 system
// by Cholesky and applies the SE(3) update; then its lanes form the pairs of
// Eq. 10 for their input pixels (binary64, a fixed operation sequence), their
// residuals and Jacobians, and the workgroup sums the 29 terms of the normal
// equations (A upper triangle, b, r^2, count) in a fixed tree.  A last launch
// solves for the result, so the whole iteration schedule is enqueued without
// a host round trip.
//
// The order of the sums is part of the result: a view that does not fix all
// six degrees (one wall fills the image) has a singular system, whose last
// pivots are rounding noise, and the sign of that noise decides whether the
// pose moves.  Products and sums are separate operations.  A level's pixels
// are dealt to B = min(ceil(pixels / 256), 512) blocks of 256 threads, pixel p
// to thread p mod 256 of block (p / 256) mod B; a thread adds its kept pairs
// in pixel order; a block's waves add their lanes that differ in bit 5, then 4,
// 3, 2, 1, 0, and the block (w0 + w1) + (w2 + w3).  The blocks' rows are added
// by 256 threads, thread s rows s and s + 256, in the same tree.
#include "rtg_common.h"

namespace rtg {

constexpr int kIcpTerms = 29;     // 21 (A, upper triangle) + 6 (b) + r^2 + count
constexpr int kIcpTrace = 48;     // doubles per trace row

// Normal map: the hit Gaussian's camera-frame normal {n^c} per rendered
// pixel, turned to face the camera (flipped when its dot product with the
// pixel's ray direction ((x + 0.5 - cx) / fx, (y + 0.5 - cy) / fy, 1) is
// positive, binary64); 0 on rendered pixels without a hit.
__global__ __launch_bounds__(256) void k_render_normals(Dims d, WS w, float* __restrict__ out_n) {
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int f;
    size_t pix;
    if (!pixel_of_rank(d, w, idx, f, pix)) return;
    const uint32_t hitpos = reinterpret_cast<const uint2*>(w.px_aux)[idx].y;
    float n0 = 0.f, n1 = 0.f, n2 = 0.f;
    if (hitpos) {
        const float4 hn = w.prec[4ull * (hitpos - 1u) + 3];
        const int64_t r = (int64_t)(pix % ((size_t)d.W * d.H));
        const int x = (int)(r % d.W), y = (int)(r / d.W);
        const double rx = (((double)x + 0.5) - d.cx) / d.fx, ry = (((double)y + 0.5) - d.cy) / d.fy;
        const double s = ((double)hn.x * rx + (double)hn.y * ry) + (double)hn.z;
        const float sg = s > 0.0 ? -1.f : 1.f;
        n0 = sg * hn.x;
        n1 = sg * hn.y;
        n2 = sg * hn.z;
    }
    out_n[3 * pix] = n0;
    out_n[3 * pix + 1] = n1;
    out_n[3 * pix + 2] = n2;
}

// Pyramid levels 1 and 2 of the input depth, the model depth and the model
// normals in one launch.  Depth of a coarser pixel: the binary32 mean of the
// valid (> 0) depths of its 2 x 2 block, ((d00 + d01) + d10) + d11 over the
// valid ones / their count; model normal: that of the block's first pixel
// (raster order) with a valid depth.  A thread makes a 2 x 2 block of level-1
// pixels (fewer at an odd edge) and the level-2 pixel they form, so level 2
// is built from registers; the six single-map launches this replaces were
// bound by their launches (28 us together at 1200x680 against 6 us).
struct IcpPyr {
    const float *D, *Dm, *Nm;            // level 0
    float *D1, *Dm1, *Nm1;               // level 1
    float *D2, *Dm2, *Nm2;               // level 2 (unused with two levels)
    int W, W1, H1, W2, H2;               // W2 = H2 = 0 with two levels
};

__device__ __forceinline__ float mean_valid(const float (&q)[4]) {
    float s = 0.f, c = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (q[k] > 0.f) {
            s = s + q[k];
            c = c + 1.f;
        }
    return c > 0.f ? s / c : 0.f;
}

__global__ __launch_bounds__(256) void k_icp_pyramid(IcpPyr P) {
    const int cw = (P.W1 + 1) >> 1, ch = (P.H1 + 1) >> 1;
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= (int64_t)cw * ch) return;
    const int bx = (int)(c % cw), by = (int)(c / cw);
    float d1[4] = {0.f, 0.f, 0.f, 0.f}, m1[4] = {0.f, 0.f, 0.f, 0.f}, n1[4][3];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int x = 2 * bx + (k & 1), y = 2 * by + (k >> 1);
        n1[k][0] = n1[k][1] = n1[k][2] = 0.f;
        if (x >= P.W1 || y >= P.H1) continue;
        const int64_t q = (int64_t)(2 * y) * P.W + 2 * x;
        const float d[4] = {P.D[q], P.D[q + 1], P.D[q + P.W], P.D[q + P.W + 1]};
        const float m[4] = {P.Dm[q], P.Dm[q + 1], P.Dm[q + P.W], P.Dm[q + P.W + 1]};
        d1[k] = mean_valid(d);
        m1[k] = mean_valid(m);
        const int64_t qn = m[0] > 0.f ? q : m[1] > 0.f ? q + 1 : m[2] > 0.f ? q + P.W : q + P.W + 1;
        if (m[0] > 0.f || m[1] > 0.f || m[2] > 0.f || m[3] > 0.f) {
            n1[k][0] = P.Nm[3 * qn];
            n1[k][1] = P.Nm[3 * qn + 1];
            n1[k][2] = P.Nm[3 * qn + 2];
        }
        const int64_t o = (int64_t)y * P.W1 + x;
        P.D1[o] = d1[k];
        P.Dm1[o] = m1[k];
        P.Nm1[3 * o] = n1[k][0];
        P.Nm1[3 * o + 1] = n1[k][1];
        P.Nm1[3 * o + 2] = n1[k][2];
    }
    if (bx >= P.W2 || by >= P.H2) return;
    const int64_t o = (int64_t)by * P.W2 + bx;
    P.D2[o] = mean_valid(d1);
    P.Dm2[o] = mean_valid(m1);
    float n0 = 0.f, nx = 0.f, nz = 0.f;
#pragma unroll
    for (int k = 3; k >= 0; --k)
        if (m1[k] > 0.f) {
            n0 = n1[k][0];
            nx = n1[k][1];
            nz = n1[k][2];
        }
    P.Nm2[3 * o] = n0;
    P.Nm2[3 * o + 1] = nx;
    P.Nm2[3 * o + 2] = nz;
}

struct IcpLevel {
    int W, H;
    double fx, fy, cx, cy;
    const float* D;    // input depth
    const float* Dm;   // model depth
    const float* Nm;   // model normals (camera frame of the model pose)
};

// Ray of a pixel column / row: vertex = D * (ray_x, ray_y, 1).
__device__ __forceinline__ double ray_x(const IcpLevel& L, int x) { return (((double)x + 0.5) - L.cx) / L.fx; }
__device__ __forceinline__ double ray_y(const IcpLevel& L, int y) { return (((double)y + 0.5) - L.cy) / L.fy; }

__device__ __forceinline__ void mat_vec(const double* R, const double* v, double* o) {
    for (int i = 0; i < 3; ++i) o[i] = (R[3 * i] * v[0] + R[3 * i + 1] * v[1]) + R[3 * i + 2] * v[2];
}

__device__ __forceinline__ void cross3(const double* a, const double* b, double* o) {
    o[0] = a[1] * b[2] - a[2] * b[1];
    o[1] = a[2] * b[0] - a[0] * b[2];
    o[2] = a[0] * b[1] - a[1] * b[0];
}

__device__ __forceinline__ double dot3(const double* a, const double* b) {
    return (a[0] * b[0] + a[1] * b[1]) + a[2] * b[2];
}

// SE(3) exponential of xi = (omega, v): R = I + a [w] + b [w]^2,
// t = (I + b [w] + c [w]^2) v, a = sin th / th, b = (1 - cos th) / th^2,
// c = (th - sin th) / th^3 (R = I + [w], V = I + [w] / 2 below th = 1e-12).
__device__ void se3_exp(const double* xi, double* R, double* t) {
    const double w0 = xi[0], w1 = xi[1], w2 = xi[2];
    const double th = sqrt((w0 * w0 + w1 * w1) + w2 * w2);
    const double Wx[9] = {0.0, -w2, w1, w2, 0.0, -w0, -w1, w0, 0.0};
    double W2[9];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) W2[3 * i + j] = (Wx[3 * i] * Wx[j] + Wx[3 * i + 1] * Wx[3 + j]) + Wx[3 * i + 2] * Wx[6 + j];
    double a, b, bv, c;   // bv: the [w] coefficient of V
    if (th < 1e-12) {
        a = 1.0;
        b = 0.0;
        bv = 0.5;
        c = 0.0;
    } else {
        a = sin(th) / th;
        b = (1.0 - cos(th)) / (th * th);
        bv = b;
        c = (th - sin(th)) / (th * th * th);
    }
    double Vm[9];
    for (int k = 0; k < 9; ++k) {
        const double id = (k % 4 == 0) ? 1.0 : 0.0;
        R[k] = id + a * Wx[k] + b * W2[k];
        Vm[k] = id + bv * Wx[k] + c * W2[k];
    }
    for (int i = 0; i < 3; ++i) t[i] = (Vm[3 * i] * xi[3] + Vm[3 * i + 1] * xi[4]) + Vm[3 * i + 2] * xi[5];
}

// Reduce-scatters of 2^m binary64 values over the wave, in the tree of a
// butterfly that adds lanes differing in bit 5, then 4, 3, 2, 1, 0: while
// several values are left, each half keeps its own one's partial sum after
// one add (lane bits 5 and 4 by the permlane swaps, 3 and below by DPP moves).
// 31 exchanges for 32 values where a butterfly per value takes 174 for the
// 29 terms; the same additions, so the same bits.
__device__ __forceinline__ double f64_of(uint32_t lo, uint32_t hi) {
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ void f64_to(double v, uint32_t& lo, uint32_t& hi) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    lo = (uint32_t)b;
    hi = (uint32_t)(b >> 32);
}
__device__ __forceinline__ double swap32_sum64(double a, double b) {
    uint32_t al, ah, bl, bh;
    f64_to(a, al, ah);
    f64_to(b, bl, bh);
    auto l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
    auto h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    return f64_of(l[0], h[0]) + f64_of(l[1], h[1]);
}
__device__ __forceinline__ double swap16_sum64(double a, double b) {
    uint32_t al, ah, bl, bh;
    f64_to(a, al, ah);
    f64_to(b, bl, bh);
    auto l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
    auto h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    return f64_of(l[0], h[0]) + f64_of(l[1], h[1]);
}
template <int CTRL>
__device__ __forceinline__ double dpp_mov64(double v) {
    uint32_t lo, hi;
    f64_to(v, lo, hi);
    lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, CTRL, 0xf, 0xf, false);
    hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, CTRL, 0xf, 0xf, false);
    return f64_of(lo, hi);
}
// The value of lane ^ 8 (row rotation by 8), ^ 4 (half-row mirror, then the
// quad reversed), ^ 2 and ^ 1.
template <int BIT>
__device__ __forceinline__ double lane_xor64(double v) {
    if constexpr (BIT == 8) return dpp_mov64<0x128>(v);
    else if constexpr (BIT == 4) return dpp_mov64<0x1B>(dpp_mov64<0x141>(v));
    else if constexpr (BIT == 2) return dpp_mov64<0x4E>(v);
    else return dpp_mov64<0xB1>(v);
}
template <int BIT>
__device__ __forceinline__ double pair_sum64(double a, double b, int lane) {
    const bool hi = (lane & BIT) != 0;
    const double send = hi ? a : b, keep = hi ? b : a;
    return keep + lane_xor64<BIT>(send);
}
// Every lane returns the wave total of value icp_slot(lane) of 32.
__device__ __forceinline__ double reduce_scatter32(double (&t)[32], int lane) {
#pragma unroll
    for (int j = 0; j < 16; ++j) t[j] = swap32_sum64(t[2 * j], t[2 * j + 1]);
#pragma unroll
    for (int j = 0; j < 8; ++j) t[j] = swap16_sum64(t[2 * j], t[2 * j + 1]);
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = pair_sum64<8>(t[2 * j], t[2 * j + 1], lane);
#pragma unroll
    for (int j = 0; j < 2; ++j) t[j] = pair_sum64<4>(t[2 * j], t[2 * j + 1], lane);
    const double r = pair_sum64<2>(t[0], t[1], lane);
    return r + lane_xor64<1>(r);
}
// The same of 16: value icp_slot(lane) & 15.
__device__ __forceinline__ double reduce_scatter16(double (&t)[16], int lane) {
#pragma unroll
    for (int j = 0; j < 8; ++j) t[j] = swap32_sum64(t[2 * j], t[2 * j + 1]);
#pragma unroll
    for (int j = 0; j < 4; ++j) t[j] = swap16_sum64(t[2 * j], t[2 * j + 1]);
#pragma unroll
    for (int j = 0; j < 2; ++j) t[j] = pair_sum64<8>(t[2 * j], t[2 * j + 1], lane);
    double r = pair_sum64<4>(t[0], t[1], lane);
    r += lane_xor64<2>(r);
    return r + lane_xor64<1>(r);
}
__device__ __forceinline__ int icp_slot(int lane) {
    return ((lane >> 5) & 1) + 2 * ((lane >> 4) & 1) + 4 * ((lane >> 3) & 1) + 8 * ((lane >> 2) & 1) +
           16 * ((lane >> 1) & 1);
}

// What a pass starts from: the normal equations of the pass before it (partial
// sums, `rows` (at most 256) per term) and the pose that pass used, or, for the
// first one (part == nullptr), the initial pose itself.
struct IcpPrev {
    const double* part;
    int rows;
    const double* T;
    double* trace;   // trace row of the pass before, or nullptr
};

// The pose after the previous pass, into T (LDS) for the whole workgroup of
// kIcpThreads: the partial sums added in their fixed order (every workgroup
// gets the same bits; the first four waves take terms 0-14, the others 15-28),
// the 6x6 solve by Cholesky (no update with fewer than 6 pairs or a
// non-positive pivot) and T <- exp(xi) T.  `write`: this workgroup also writes
// the trace row (pose used, r^2, count, A, b).
constexpr int kIcpThreads = 512;   // two blocks of 256
constexpr int kIcpHalf = 15;

__device__ void icp_next_pose(const IcpPrev& v, bool write, double (&red)[8][32], double (&T)[12]) {
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (!v.part) {
        if (tid < 12) T[tid] = v.T[tid];
        __syncthreads();
        return;
    }
    double s[16];
    const int slot = tid & 255;
    const double* p = v.part + (int64_t)(wv < 4 ? 0 : kIcpHalf) * v.rows + slot;
    const int terms = wv < 4 ? kIcpHalf : kIcpTerms - kIcpHalf;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = slot < v.rows && i < terms ? p[i * v.rows] : 0.0;
    const double sum = reduce_scatter16(s, lane);
    if ((lane & 3) == 0) red[wv][icp_slot(lane)] = sum;
    __syncthreads();
    if (wv == 0) {
        const int k = min(lane, kIcpTerms - 1), w = k < kIcpHalf ? 0 : 4, kk = k < kIcpHalf ? k : k - kIcpHalf;
        const double t = (red[w][kk] + red[w + 1][kk]) + (red[w + 2][kk] + red[w + 3][kk]);
        double tot[kIcpTerms];
#pragma unroll
        for (int i = 0; i < kIcpTerms; ++i) tot[i] = __shfl(t, i);
        double T0[12];
#pragma unroll
        for (int i = 0; i < 12; ++i) T0[i] = v.T[i];
        if (write && v.trace && lane < kIcpTrace) {
            double o = 0.0;
            if (lane < 12) o = v.T[lane];
            const int src = lane == 12 ? 27 : lane == 13 ? 28 : lane - 14;
            const double ts = __shfl(t, src & 31);
            if (lane >= 12 && lane < 41) o = ts;
            v.trace[lane] = o;
        }
        // Cholesky A = L L^T; the upper triangle of A is tot[0..20] row by row
        double Lc[6][6], yv[6], xi[6];
        bool good = tot[28] >= 6.0;
#pragma unroll
        for (int j = 0; j < 6; ++j)
#pragma unroll
            for (int i = j; i < 6; ++i) {
                double acc = tot[j * 6 - (j * (j - 1)) / 2 + (i - j)];
#pragma unroll
                for (int m = 0; m < j; ++m) acc -= Lc[i][m] * Lc[j][m];
                if (i == j) {
                    good = good && acc > 0.0;
                    Lc[j][j] = sqrt(acc);
                } else {
                    Lc[i][j] = acc / Lc[j][j];
                }
            }
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            double acc = tot[21 + i];
#pragma unroll
            for (int m = 0; m < i; ++m) acc -= Lc[i][m] * yv[m];
            yv[i] = acc / Lc[i][i];
        }
#pragma unroll
        for (int i = 5; i >= 0; --i) {
            double acc = yv[i];
#pragma unroll
            for (int m = i + 1; m < 6; ++m) acc -= Lc[m][i] * xi[m];
            xi[i] = acc / Lc[i][i];
        }
#pragma unroll
        for (int i = 0; i < 6; ++i) xi[i] = -xi[i];
        double dR[9], dt[3], Tn[12];
        se3_exp(xi, dR, dt);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
#pragma unroll
            for (int j = 0; j < 3; ++j)
                Tn[3 * i + j] = (dR[3 * i] * T0[j] + dR[3 * i + 1] * T0[3 + j]) + dR[3 * i + 2] * T0[6 + j];
            Tn[9 + i] = ((dR[3 * i] * T0[9] + dR[3 * i + 1] * T0[10]) + dR[3 * i + 2] * T0[11]) + dt[i];
        }
        if (lane == 0)
#pragma unroll
            for (int i = 0; i < 12; ++i) T[i] = good ? Tn[i] : T0[i];
    }
    __syncthreads();
}

// The same value on every lane, held in scalar registers.
__device__ __forceinline__ double uniform64(double v) {
    uint32_t lo, hi;
    f64_to(v, lo, hi);
    return f64_of((uint32_t)readfirstlane((int)lo), (uint32_t)readfirstlane((int)hi));
}

// Rays of the level's columns and rows, from a table in LDS (TAB) or formed
// where they are needed.
constexpr int kIcpTable = 7168;   // entries (56 KB): columns, then rows

template <bool TAB>
struct IcpRays {
    const double* tab;
    __device__ __forceinline__ double x(const IcpLevel& L, int i) const {
        if constexpr (TAB) return tab[i];
        else return ray_x(L, i);
    }
    __device__ __forceinline__ double y(const IcpLevel& L, int i) const {
        if constexpr (TAB) return tab[L.W + i];
        else return ray_y(L, i);
    }
};

// The pair of one input pixel up to the model's depth and normal (in flight
// while the pixel before it is summed).
struct IcpCand {
    double P[3], Nn[3];   // world point, input normal (camera frame, not normalised)
    float Dm, n0, n1, n2;
    int ui, vi;
    bool ok;
};

// One pass: the pose from the pass before (each workgroup solves for it
// itself: about 2 us once the rows are there, where a launch of its own cost
// 19 us, most of it one thread working from scratch memory), then the
// input pixels' pairs (Eq. 10, projective association) under that estimate
// T of the input frame's camera-to-world pose against the model rendered at
// Tm.  Workgroup b holds blocks b and b + 256 of the order above, so that the
// sum of the two is one of the rows' first additions.  The lanes take their
// pixels two at a time, staggered: the depths of the pixel after next and the
// model's entries of the next one are loaded while the present one is summed
// (two waves per SIMD, all that the order leaves, do not hide those two
// dependent loads).  The rays come from a table in LDS where image width +
// height fit it, which takes the binary64 divisions per pixel from ten to two.
// The partial sums of consecutive passes and the poses alternate between two
// places, so no workgroup overwrites what another still reads.
//
// A level-0 pass at 1200x680 takes 17.0 us.  4.8 of them are the launch, the
// sums of the rows and the solve (a launch that does only these takes as long).
// Vector instructions are issued for 9 of the other 12 (5.3M wave instructions,
// 3.2M of them binary64, by counters); the rest is latency that two waves per
// SIMD leave open.  With three (balanced strips, other sums) a pass took 19 us.
// The call: 245 us, 298 with the strips, 720 with a solve launch per iteration.
template <bool TAB>
__global__ __launch_bounds__(kIcpThreads) void k_icp_pass(IcpLevel L, IcpPrev prev, const double* __restrict__ Tm,
                                                          double dist, double sin_a, int blocks,
                                                          double* __restrict__ T_out, double* __restrict__ partials) {
    __shared__ double red[8][32];
    __shared__ double sT[12];
    extern __shared__ double ray_tab[];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if constexpr (TAB)
        for (int i = threadIdx.x; i < L.W + L.H; i += kIcpThreads)
            ray_tab[i] = i < L.W ? ray_x(L, i) : ray_y(L, i - L.W);
    const IcpRays<TAB> rays{ray_tab};
    icp_next_pose(prev, blockIdx.x == 0, red, sT);   // (ends with a barrier)
    double T[12], M[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        T[k] = uniform64(sT[k]);
        M[k] = Tm[k];
    }
    if (blockIdx.x == 0 && threadIdx.x < 12) T_out[threadIdx.x] = sT[threadIdx.x];
    double t[32];
#pragma unroll
    for (int k = 0; k < 32; ++k) t[k] = 0.0;
    // this wave's block, its first pixel and its number of pixels per lane
    const int block = (int)blockIdx.x + (wv < 4 ? 0 : 256), np = L.W * L.H, step = blocks * 256;
    const int first = readfirstlane(block * 256 + (wv & 3) * 64);
    const int n = block < blocks && first < np ? (np - 1 - first) / step + 1 : 0;
    // pixel of the next load: its depths are read in advance (the last row and
    // column have no forward difference; past the image: nothing)
    const int sx = step % L.W, sy = step / L.W;
    int qy = (first + lane) / L.W, qx = first + lane - qy * L.W;
    struct Row {
        float D, Dr, Dd;
        int x, y;
    };
    auto load_row = [&]() {
        const bool in = qx < L.W - 1 && qy < L.H - 1;
        Row r;
        r.x = in ? qx : 0;
        r.y = in ? qy : 0;
        const float* p = L.D + (r.y * L.W + r.x);
        r.D = in ? p[0] : 0.f;
        r.Dr = p[1];
        r.Dd = p[L.W];
        qx += sx;
        qy += sy;
        if (qx >= L.W) {
            qx -= L.W;
            ++qy;
        }
        return r;
    };
    auto candidate = [&](const Row& rw) {
        IcpCand c;
        c.ok = rw.D > 0.f && rw.Dr > 0.f && rw.Dd > 0.f;
        const double D = rw.D, Dr = rw.Dr, Dd = rw.Dd;
        const double rx = rays.x(L, rw.x), rxr = rays.x(L, rw.x + 1), ry = rays.y(L, rw.y), ryd = rays.y(L, rw.y + 1);
        const double V[3] = {D * rx, D * ry, D};
        const double a[3] = {Dr * rxr - V[0], Dr * ry - V[1], Dr - V[2]};
        const double b[3] = {Dd * rx - V[0], Dd * ryd - V[1], Dd - V[2]};
        double dm[3], pm[3];
        cross3(a, b, c.Nn);
        mat_vec(T, V, c.P);
        for (int i = 0; i < 3; ++i) c.P[i] = c.P[i] + T[9 + i];
        for (int i = 0; i < 3; ++i) dm[i] = c.P[i] - M[9 + i];
        for (int i = 0; i < 3; ++i) pm[i] = (M[i] * dm[0] + M[3 + i] * dm[1]) + M[6 + i] * dm[2];
        const double u = floor(L.fx * pm[0] / pm[2] + L.cx);
        const double v = floor(L.fy * pm[1] / pm[2] + L.cy);
        c.ok = c.ok && pm[2] > 0.0 && u >= 0.0 && u < (double)L.W && v >= 0.0 && v < (double)L.H;
        c.ui = c.ok ? (int)u : 0;
        c.vi = c.ok ? (int)v : 0;
        const int64_t q = (int64_t)c.vi * L.W + c.ui;
        c.Dm = L.Dm[q];
        c.n0 = L.Nm[3 * q];
        c.n1 = L.Nm[3 * q + 1];
        c.n2 = L.Nm[3 * q + 2];
        return c;
    };
    auto add_pair = [&](const IcpCand& c) {
        const double Dmq = c.Dm, nm[3] = {c.n0, c.n1, c.n2};
        if (!(c.ok && Dmq > 0.0 && dot3(nm, nm) > 0.0)) return;
        const double Vm[3] = {Dmq * rays.x(L, c.ui), Dmq * rays.y(L, c.vi), Dmq};
        double Q[3], n[3], m[3], dd[3], cr[3];
        mat_vec(M, Vm, Q);
        for (int i = 0; i < 3; ++i) Q[i] = Q[i] + M[9 + i];
        mat_vec(M, nm, n);
        mat_vec(T, c.Nn, m);
        for (int i = 0; i < 3; ++i) dd[i] = c.P[i] - Q[i];
        cross3(m, n, cr);
        if (!(dot3(dd, dd) <= dist * dist && dot3(cr, cr) <= (sin_a * sin_a) * (dot3(m, m) * dot3(n, n)))) return;
        const double r = dot3(dd, n);
        double J[6];
        cross3(c.P, n, J);
        J[3] = n[0];
        J[4] = n[1];
        J[5] = n[2];
        int k = 0;
#pragma unroll
        for (int i = 0; i < 6; ++i)
#pragma unroll
            for (int j = i; j < 6; ++j, ++k) t[k] += J[i] * J[j];
#pragma unroll
        for (int i = 0; i < 6; ++i) t[21 + i] += J[i] * r;
        t[27] += r * r;
        t[28] += 1.0;
    };
    if (n > 0) {
        Row rw = load_row();
        IcpCand c = candidate(rw);
        rw = load_row();
        for (int u = 0; u < n; ++u) {
            IcpCand nx = candidate(rw);   // pixel u + 1 (past the end: dropped)
            rw = load_row();
            add_pair(c);
            c = nx;
        }
    }
    // the wave's reduce-scatter, the four waves of each block, the two blocks
    // (a block or wave without pixels adds zeros)
    const double s = reduce_scatter32(t, lane);
    if ((lane & 1) == 0) red[wv][icp_slot(lane)] = s;
    __syncthreads();
    if (threadIdx.x < kIcpTerms) {
        const int k = threadIdx.x;
        partials[(int64_t)k * gridDim.x + blockIdx.x] = ((red[0][k] + red[1][k]) + (red[2][k] + red[3][k])) +
                                                        ((red[4][k] + red[5][k]) + (red[6][k] + red[7][k]));
    }
}

// The pose after the last pass (one workgroup; T_out may be the place of the
// pose that the pass used).
__global__ __launch_bounds__(kIcpThreads) void k_icp_finish(IcpPrev prev, double* T_out) {
    __shared__ double red[8][32];
    __shared__ double sT[12];
    icp_next_pose(prev, true, red, sT);
    if (threadIdx.x < 12) T_out[threadIdx.x] = sT[threadIdx.x];
}

}  // namespace rtg
