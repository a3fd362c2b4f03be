// Point-to-plane ICP camera tracking (Sec. 3.2.1, "Camera tracking", Eq. 5).
//   k_depth_down   one level of the depth hierarchy: mean of the valid depths of
//                  each 2x2 block (binary64 sum and division, rounded once)
//   k_icp_pairs    per pixel of the current level: back-projection, projective
//                  association into the previous frame's raycast depth, the
//                  model vertex and vertex-map normal there, the point-to-plane
//                  residual r and its Jacobian J = (N, p x N) for a left
//                  perturbation of the camera-to-world pose; at most 1024
//                  blocks of 256 lanes, each lane taking every (256 x blocks)-th
//                  pixel; per block the 29 sums (upper triangle of J J^T, J r,
//                  r^2, count) in a fixed order
//   k_icp_total    one block: the block sums in binary64, in a fixed order
//   k_icp_solve    one wavefront: solution of H xi = -g in binary64 and the
//                  update T_{g,k} <- Exp(xi) T_{g,k} of the device pose
// No atomics: the system is bitwise reproducible.  Every stage reads the pose
// from device memory, so a tracking loop can be replayed as a graph.
#include <cmath>
#include <mutex>

#include "gps_internal.h"
#include "launch.h"
#include "prof.h"
#include "se3.h"

namespace gps {

constexpr int kIcpTerms = 29;  // 21 (H, upper triangle, row-major) + 6 (g) + E + count
constexpr int kIcpMaxBlocks = 1024;  // widest grid of k_icp_pairs (four blocks per compute unit)

// Block sums of the allocation-free reduce (gps_icp_reduce_noalloc): room for the
// widest grid, so every level size fits.  One copy per GPU, held until the process
// ends; each call overwrites the entries it reads, so nothing is cleared.  Host code
// takes its address from icp_scratch(), never from this name.
static __device__ __align__(256) float scratch[kIcpTerms * kIcpMaxBlocks];
static_assert(sizeof(scratch) == GPS_ICP_SCRATCH_BYTES, "the header states the scratch size");

__global__ void __launch_bounds__(256) k_depth_down(const float* __restrict__ in, int W, int H,
                                                    float* __restrict__ out, int Wo, int Ho)
{
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= Wo * Ho) return;
    const int i = p % Wo, j = p / Wo;
    const float* r0 = in + (size_t)(2 * j) * W + 2 * i;
    const float* r1 = r0 + W;
    const float v[4] = {r0[0], r0[1], r1[0], r1[1]};
    double s = 0.0;
    int n = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (v[k] > 0.0f) {
            s += (double)v[k];
            ++n;
        }
    out[p] = n > 0 ? (float)(s / (double)n) : 0.0f;
}

struct IcpArgs {
    // previous frame: intrinsics, pose (world -> camera), raycast depth
    float pfx, pfy, pcx, pcy;
    float pR[9], pt[3];
    int pW, pH;
    const float* pdepth;
    // current level: intrinsics, depth; the pose comes from `pose`
    float fx, fy, cx, cy;
    int W, H;
    const float* depth;
    const float* pose;  // [12]: R row-major, t (world -> camera)
    float dist2;
    float* part;        // [kIcpTerms][nblk]
    int nblk;
    int step_x, step_y;  // a lane's next pixel: 256 nblk = step_y W + step_x
};

// x + (x of lane ^ 8, 4, 2, 1 in turn): the sum over a row of 16 lanes in every lane.  After the
// first step the values repeat every 8 lanes, so the rotation by 4 is the exchange with lane ^ 4, and so on.
__device__ __forceinline__ float row_sum(float x)
{
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x128, 0xf, 0xf, true));  // row_ror:8
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x124, 0xf, 0xf, true));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x122, 0xf, 0xf, true));
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x121, 0xf, 0xf, true));
    return x;
}

// Sums of 32 values over the wavefront: row r (lanes 16 r .. 16 r + 15) gets in out[q] that of value
// 4 q + 2 (r & 1) + (r >> 1), summed as x + (x of lane ^ 32, 16, 8, 4, 2, 1).  Across halves and
// rows a lane keeps one of two values and sends the other, so an exchange serves both: 24
// shuffles through LDS, where one per step and value took 174 and most of the kernel's time.
__device__ __forceinline__ float exchange_sum(float a, float b, bool second, int mask)
{
    const float keep = second ? b : a, send = second ? a : b;
    return keep + __shfl_xor(send, mask, 64);
}

__device__ __forceinline__ void wave_sums32(const float (&v)[32], float (&out)[8])
{
    const int lane = threadIdx.x & 63;
    float h[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) h[k] = exchange_sum(v[2 * k], v[2 * k + 1], (lane & 32) != 0, 32);
#pragma unroll
    for (int k = 0; k < 8; ++k) out[k] = row_sum(exchange_sum(h[2 * k], h[2 * k + 1], (lane & 16) != 0, 16));
}

// n / d, correctly rounded, from r = 1 / d correctly rounded: the first correction leaves the
// quotient less than a unit off, and the second then rounds it as the division does (Markstein).  For
// divisors that many quotients share; 5 operations instead of 10.  Exponents far from the ends
// of the range (focal_sane).
template <bool SANE>
__device__ __forceinline__ float div_shared(float n, float d, float r)
{
    if (!SANE) return n / d;
    float q = n * r;
    q = __builtin_fmaf(__builtin_fmaf(-q, d, n), r, q);
    return __builtin_fmaf(__builtin_fmaf(-q, d, n), r, q);
}

// Focal lengths and principal points of ordinary size: a pixel's offset is then 0 or at least 2^-44,
// and quotients and remainders stay far from the smallest numbers.
static bool focal_sane(float f, float c)
{
    const float m = std::fabs(f);
    return m > 0x1p-40f && m < 0x1p40f && std::fabs(c) < 0x1p20f && (c == 0.0f || std::fabs(c) > 0x1p-20f);
}

// Bound by its instructions and by the latency of two dependent loads a pixel: the next pixel's
// depth is loaded ahead.  Mean of a 14-step tracking of a 1280x720 frame over three levels: 8.0 us,
// with sums by shuffles, divisions throughout and no load ahead 14.8.
template <bool SANE>
__global__ void __launch_bounds__(256) k_icp_pairs(IcpArgs a)
{
    __shared__ float red[32][4];
    // Relative pose current camera -> previous camera, formed in binary64 from the
    // two world-to-camera poses so that the association and the residual are
    // computed without world coordinates: q = R_rel X + t_rel.
    double Rc[9], tc[3];
#pragma unroll
    for (int k = 0; k < 9; ++k) Rc[k] = (double)a.pose[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) tc[k] = (double)a.pose[9 + k];
    float Rrel[9], trel[3], Rct[9];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        double tr = (double)a.pt[r];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            // (R_p R_c^T)[r][c] = sum_k R_p[r][k] R_c[c][k]
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < 3; ++k) s += (double)a.pR[3 * r + k] * Rc[3 * c + k];
            Rrel[3 * r + c] = (float)s;
            tr -= s * tc[c];
            Rct[3 * r + c] = (float)Rc[3 * c + r];
        }
        trel[r] = (float)tr;
    }
    float v[32];  // (three more than there are terms)
#pragma unroll
    for (int k = 0; k < 32; ++k) v[k] = 0.0f;
    const float rfx = 1.0f / a.fx, rfy = 1.0f / a.fy, rpfx = 1.0f / a.pfx, rpfy = 1.0f / a.pfy;
    // each lane takes the pixels p, p + 256 * gridDim.x, ... (a fixed assignment, so
    // the sums have a fixed order)
    const int n = a.W * a.H, stride = 256 * (int)gridDim.x;
    int p = blockIdx.x * 256 + threadIdx.x, i = p % a.W, j = p / a.W;
    float d_next = p < n ? a.depth[p] : 0.0f;
    for (bool more = p < n; more;) {
        const float d = d_next;
        const float fi = (float)i, fj = (float)j;
        more = p < n - stride;
        if (more) {
            p += stride;
            d_next = a.depth[p];
            i += a.step_x;
            j += a.step_y;
            if (i >= a.W) {
                i -= a.W;
                ++j;
            }
        }
        bool ok = d > 0.0f;
        float X[3] = {div_shared<SANE>(fi - a.cx, a.fx, rfx) * d, div_shared<SANE>(fj - a.cy, a.fy, rfy) * d, d};
        float q[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int r = 0; r < 3; ++r) q[r] = Rrel[3 * r] * X[0] + Rrel[3 * r + 1] * X[1] + Rrel[3 * r + 2] * X[2] + trel[r];
        ok = ok && q[2] > 0.0f;
        int ua = 0, vb = 0;
        if (ok) {
            const float u = a.pfx * q[0] / q[2] + a.pcx, w = a.pfy * q[1] / q[2] + a.pcy;
            ok = u >= 0.5f && u < (float)a.pW - 1.5f && w >= 0.5f && w < (float)a.pH - 1.5f;  // neighbours in the image
            ua = (int)floorf(u + 0.5f);
            vb = (int)floorf(w + 0.5f);
            ok = ok && ua >= 1 && ua <= a.pW - 2 && vb >= 1 && vb <= a.pH - 2;
        }
        float Xs[3], Nc[3];
        if (ok) {
            const int s = vb * a.pW + ua;
            const float dc = a.pdepth[s], dl = a.pdepth[s - 1], dr = a.pdepth[s + 1], du = a.pdepth[s - a.pW],
                        dd = a.pdepth[s + a.pW];
            ok = dc > 0.0f && dl > 0.0f && dr > 0.0f && du > 0.0f && dd > 0.0f;
            if (ok) {
                // vertices of the pixel and its neighbours: x = ((u - cx) / fx d, (v - cy) / fy d, d)
                const float fu = (float)ua, fv = (float)vb;
                const float gx = div_shared<SANE>(fu - a.pcx, a.pfx, rpfx), gy = div_shared<SANE>(fv - a.pcy, a.pfy, rpfy);
                const float gl = div_shared<SANE>(fu - 1.0f - a.pcx, a.pfx, rpfx);
                const float gr = div_shared<SANE>(fu + 1.0f - a.pcx, a.pfx, rpfx);
                const float gu = div_shared<SANE>(fv - 1.0f - a.pcy, a.pfy, rpfy);
                const float gd = div_shared<SANE>(fv + 1.0f - a.pcy, a.pfy, rpfy);
                Xs[0] = gx * dc, Xs[1] = gy * dc, Xs[2] = dc;
                const float xl[3] = {gl * dl, gy * dl, dl}, xr[3] = {gr * dr, gy * dr, dr};
                const float xu[3] = {gx * du, gu * du, du}, xd[3] = {gx * dd, gd * dd, dd};
                const float ex[3] = {xr[0] - xl[0], xr[1] - xl[1], xr[2] - xl[2]};
                const float ey[3] = {xd[0] - xu[0], xd[1] - xu[1], xd[2] - xu[2]};
                Nc[0] = ex[1] * ey[2] - ex[2] * ey[1];
                Nc[1] = ex[2] * ey[0] - ex[0] * ey[2];
                Nc[2] = ex[0] * ey[1] - ex[1] * ey[0];
                const float nn = Nc[0] * Nc[0] + Nc[1] * Nc[1] + Nc[2] * Nc[2];
                ok = nn > 0.0f;
                const float inv = ok ? 1.0f / sqrtf(nn) : 0.0f;
                // the sign of N cancels in J J^T and J r: no turn towards the camera is needed
                Nc[0] *= inv;
                Nc[1] *= inv;
                Nc[2] *= inv;
            }
        }
        if (ok) {
            const float df[3] = {q[0] - Xs[0], q[1] - Xs[1], q[2] - Xs[2]};
            ok = df[0] * df[0] + df[1] * df[1] + df[2] * df[2] <= a.dist2;
            if (ok) {
                const float r = df[0] * Nc[0] + df[1] * Nc[1] + df[2] * Nc[2];
                // world normal N = R_p^T N_c; world point p = R_c^T (X - t_c)
                float Nw[3], P[3];
                const float xt[3] = {X[0] - a.pose[9], X[1] - a.pose[10], X[2] - a.pose[11]};
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    Nw[k] = a.pR[k] * Nc[0] + a.pR[3 + k] * Nc[1] + a.pR[6 + k] * Nc[2];
                    P[k] = Rct[3 * k] * xt[0] + Rct[3 * k + 1] * xt[1] + Rct[3 * k + 2] * xt[2];
                }
                const float J[6] = {Nw[0], Nw[1], Nw[2], P[1] * Nw[2] - P[2] * Nw[1], P[2] * Nw[0] - P[0] * Nw[2],
                                    P[0] * Nw[1] - P[1] * Nw[0]};
                int k = 0;
#pragma unroll
                for (int r0 = 0; r0 < 6; ++r0)
#pragma unroll
                    for (int c0 = r0; c0 < 6; ++c0) v[k++] += J[r0] * J[c0];
#pragma unroll
                for (int r0 = 0; r0 < 6; ++r0) v[21 + r0] += J[r0] * r;
                v[27] += r * r;
                v[28] += 1.0f;
            }
        }
    }
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    float sums[8];
    wave_sums32(v, sums);
    if ((lane & 15) == 0) {
        const int r = lane >> 4;
#pragma unroll
        for (int q = 0; q < 8; ++q) red[4 * q + 2 * (r & 1) + (r >> 1)][wid] = sums[q];
    }
    __syncthreads();
    if (threadIdx.x < kIcpTerms) {
        const int k = threadIdx.x;
        a.part[(size_t)k * a.nblk + blockIdx.x] = ((red[k][0] + red[k][1]) + red[k][2]) + red[k][3];
    }
}

// Sums of two terms over the blocks: lane l takes blocks l, l + 64, ... in binary64 (the loads of 8 are
// in flight together), then a fixed butterfly across the lanes.
__device__ __forceinline__ void block_totals(const float* p0, const float* p1, int nblk, int lane, double& s0, double& s1)
{
    constexpr int kAhead = 8;
#pragma unroll 1
    for (int b0 = lane; b0 < nblk; b0 += 64 * kAhead) {
        float x0[kAhead], x1[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const int b = b0 + 64 * k;
            x0[k] = p0[b < nblk ? b : 0];
            x1[k] = p1[b < nblk ? b : 0];
        }
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const bool has = b0 + 64 * k < nblk;
            s0 += has ? (double)x0[k] : 0.0;
            s1 += has ? (double)x1[k] : 0.0;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        s0 += __shfl_xor(s0, o, 64);
        s1 += __shfl_xor(s1, o, 64);
    }
}

// Wavefront w sums the terms w and w + 16 over the block partials (both in one
// pass, so their loads overlap): lane l takes blocks l, l + 64, ... in binary64,
// then a fixed butterfly across the lanes.
__global__ void __launch_bounds__(1024) k_icp_total(const float* __restrict__ part, int nblk, double* __restrict__ sys)
{
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int k0 = wid, k1 = wid + 16;
    const bool two = k1 < kIcpTerms;
    const float* p0 = part + (size_t)k0 * nblk;
    const float* p1 = part + (size_t)(two ? k1 : k0) * nblk;
    double s0 = 0.0, s1 = 0.0;
    block_totals(p0, p1, nblk, lane, s0, s1);
    if (lane == 0) {
        sys[k0] = s0;
        if (two) sys[k1] = s1;
    }
}

// The Gauss-Newton step, by one wavefront: H xi = -g, then res = (new pose (12), xi (6)).  The pose is
// kept when fewer than 6 pairs remain or H is not positive definite (xi = 0 then).
// It runs once a launch, so what bounds it is the latency of its chain and the fetch of its
// instructions: the lanes share the work in short loops (a form for one lane with everything
// unrolled took 11 us with the sums, the rolled one 6.3, this 5.3).
struct IcpSolve {
    double sys[kIcpTerms];
    double recip[3][10];  // 1 / ((2 k + 2 + o) (2 k + 3 + o)) of the three series o
    double xi[6], Rx[9], V[9], Rg[9], tg[3];
    float pose[12], res[18];
};

// What does not depend on the system (called while its sums are in flight; 64 lanes).
__device__ __forceinline__ void icp_solve_begin(IcpSolve& s, const float* pose, int lane)
{
    if (lane < 12) s.pose[lane] = pose[lane];
    if (lane < 30) {
        const int o = lane / 10, k = lane % 10;
        s.recip[o][k] = 1.0 / (double)((2 * k + 2 + o) * (2 * k + 3 + o));
    }
}

__device__ __forceinline__ void icp_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void icp_solve_wave(IcpSolve& s, int lane)
{
    // Gauss-Jordan elimination of (H | -g), entry (r, c) in lane 8 r + c; the pivots are those of
    // the Cholesky factorisation squared, and as there all are positive or H is not definite.
    const int r = lane >> 3, c = lane & 7;
    const int lo = min(r, c), hi = max(r, c);
    double e = 0.0, inv = 1.0;
    if (r < 6 && c < 6) e = s.sys[lo * 6 - lo * (lo - 1) / 2 + hi - lo];
    else if (r < 6 && c == 6) e = -s.sys[21 + r];
    bool ok = s.sys[28] >= 6.0;
#pragma unroll 1
    for (int j = 0; j < 6; ++j) {
        double pivot = __shfl(e, 9 * j, 64);
        if (!(pivot > 0.0)) {  // (finish harmlessly)
            ok = false;
            pivot = 1.0;
        }
        const double ip = 1.0 / pivot;
        const double f = __shfl(e, 8 * r + j, 64) * ip, p = __shfl(e, 8 * j + c, 64);
        if (r == j) inv = ip;
        else if (c > j) e -= f * p;
    }
    if (r < 6 && c == 6) s.xi[r] = ok ? e * inv : 0.0;
    icp_lds_order();
    if (ok) {
        // Exp(xi): Rodrigues' formula for the rotation, the left Jacobian of SO(3) for the
        // translation, with sin(th)/th, (1 - cos th)/th^2, (th - sin th)/th^3 by lanes 0, 1, 2: below
        // 1 their series (the next term is under 2^-60 of the sum), above by the functions.
        const double w[3] = {s.xi[3], s.xi[4], s.xi[5]};
        const double th2 = w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
        const int o = min(lane, 2);
        double q = 0.0;
        if (th2 < 1.0) {
#pragma unroll 1
            for (int k = 9; k >= 0; --k) q = 1.0 - th2 * q * s.recip[o][k];
            q *= o == 0 ? 1.0 : (o == 1 ? 0.5 : 1.0 / 6.0);
        } else {
            const double th = sqrt(th2), sn = sin(th);
            q = o == 0 ? sn / th : (o == 1 ? (1.0 - cos(th)) / th2 : (th - sn) / (th2 * th));
        }
        const double A = __shfl(q, 0, 64), B = __shfl(q, 1, 64), C = __shfl(q, 2, 64);
        if (lane < 9) {
            // row i, column k of I + A K + B K^2 and I + B K + C K^2, K the cross-product matrix of
            // w: K^2 = w w^T - th^2 I
            const int i = lane / 3, k = lane % 3;
            const double wi = s.xi[3 + i], wk = s.xi[3 + k], one = i == k ? 1.0 : 0.0;
            double K = 0.0;
            if (i != k) {
                const double wo = s.xi[6 - i - k];
                K = (k - i + 3) % 3 == 1 ? -wo : wo;
            }
            const double K2 = wi * wk - one * th2;
            s.Rx[lane] = one + A * K + B * K2;
            s.V[lane] = one + B * K + C * K2;
        }
        icp_lds_order();
        // camera to world: R_g = R_c^T, t_g = -R_c^T t_c; then R_g' = Rx R_g, t_g' = Rx t_g + V rho
        if (lane < 9) {
            const int i = lane / 3, k = lane % 3;
            s.Rg[lane] = s.Rx[3 * i] * (double)s.pose[3 * k] + s.Rx[3 * i + 1] * (double)s.pose[3 * k + 1] +
                         s.Rx[3 * i + 2] * (double)s.pose[3 * k + 2];
        }
        icp_lds_order();
        if (lane < 3) {
            // Rx t_g = -(Rx R_g) t_c
            s.tg[lane] = -(s.Rg[3 * lane] * (double)s.pose[9] + s.Rg[3 * lane + 1] * (double)s.pose[10] +
                           s.Rg[3 * lane + 2] * (double)s.pose[11]) +
                         (s.V[3 * lane] * s.xi[0] + s.V[3 * lane + 1] * s.xi[1] + s.V[3 * lane + 2] * s.xi[2]);
        }
        icp_lds_order();
        // back to world to camera: R_c = R_g'^T, t_c = -R_g'^T t_g'
        if (lane < 9) s.res[lane] = (float)s.Rg[3 * (lane % 3) + lane / 3];
        else if (lane < 12)
            s.res[lane] = (float)-(s.Rg[lane - 9] * s.tg[0] + s.Rg[lane - 6] * s.tg[1] + s.Rg[lane - 3] * s.tg[2]);
    } else if (lane < 12) {
        s.res[lane] = s.pose[lane];
    }
    if (lane < 6) s.res[12 + lane] = (float)s.xi[lane];
    icp_lds_order();
}

// One value per lane (vector stores).
__device__ __forceinline__ void icp_solve_store(const IcpSolve& s, float* pose, float* out_xi, int lane)
{
    if (lane < 12) pose[lane] = s.res[lane];
    if (out_xi && lane < 6) out_xi[lane] = s.res[12 + lane];
}

// The same sums (each wavefront's two terms, the same order), kept in LDS as well,
// then the Gauss-Newton step of k_icp_solve by the block's first wavefront: one launch
// for the system and the step instead of two.
__global__ void __launch_bounds__(1024) k_icp_total_solve(const float* __restrict__ part, int nblk,
                                                          double* __restrict__ sys, float* __restrict__ pose,
                                                          float* __restrict__ out_xi)
{
    __shared__ IcpSolve sv;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int k0 = wid, k1 = wid + 16;
    const bool two = k1 < kIcpTerms;
    const float* p0 = part + (size_t)k0 * nblk;
    const float* p1 = part + (size_t)(two ? k1 : k0) * nblk;
    double s0 = 0.0, s1 = 0.0;
    if (wid == 15) icp_solve_begin(sv, pose, lane);
    block_totals(p0, p1, nblk, lane, s0, s1);
    if (lane == 0) {
        sys[k0] = s0;
        sv.sys[k0] = s0;
        if (two) {
            sys[k1] = s1;
            sv.sys[k1] = s1;
        }
    }
    __syncthreads();
    if (wid != 0) return;
    icp_solve_wave(sv, lane);
    icp_solve_store(sv, pose, out_xi, lane);
}

__global__ void __launch_bounds__(64) k_icp_solve(const double* __restrict__ sys, float* __restrict__ pose,
                                                  float* __restrict__ out_xi)
{
    __shared__ IcpSolve sv;
    const int lane = threadIdx.x;
    if (lane < kIcpTerms) sv.sys[lane] = sys[lane];
    icp_solve_begin(sv, pose, lane);
    __syncthreads();
    icp_solve_wave(sv, lane);
    icp_solve_store(sv, pose, out_xi, lane);
}

// Device address of `scratch` on the current device, looked up once per device.
gps_status icp_scratch(char** out, size_t* bytes)
{
    static std::mutex mu;
    static void* addr[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return GPS_ERR_HIP;
    if (dev < 0 || dev >= 64) return GPS_ERR_UNSUPPORTED_DEVICE;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return GPS_ERR_HIP;
        addr[dev] = p;
    }
    *out = static_cast<char*>(addr[dev]);
    *bytes = sizeof(scratch);
    return GPS_OK;
}

// Bytes of block sums k_icp_pairs writes for a level of W x H pixels.
size_t icp_partial_bytes(int W, int H)
{
    const size_t want = ((size_t)W * H + 255) / 256;
    return (size_t)kIcpTerms * sizeof(float) * (want < kIcpMaxBlocks ? want : kIcpMaxBlocks);
}

size_t icp_workspace_bytes(int W, int H)
{
    const size_t nblk = ((size_t)W * H + 255) / 256;
    return ((kIcpTerms * 4 * nblk + 255) & ~(size_t)255) + 256;
}

gps_status launch_depth_downsample(const float* in, int W, int H, float* out, hipStream_t s)
{
    const int Wo = W / 2, Ho = H / 2;
    const int n = Wo * Ho;
    if (n > 0) GPS_LAUNCH(K_ICP, s, k_depth_down, dim3((n + 255) / 256), dim3(256), 0, s, in, W, H, out, Wo, Ho);
    return hipGetLastError() == hipSuccess ? GPS_OK : GPS_ERR_HIP;
}

gps_status launch_icp_reduce(const gps_camera& prev, const float* prev_depth, const gps_camera& lvl,
                             const float* depth, const float* pose, float dist_thresh, double* sys, char* ws,
                             hipStream_t s, float* step_pose, float* step_xi)
{
    IcpArgs a;
    a.pfx = prev.fx, a.pfy = prev.fy, a.pcx = prev.cx, a.pcy = prev.cy;
    for (int k = 0; k < 9; ++k) a.pR[k] = prev.R[k];
    for (int k = 0; k < 3; ++k) a.pt[k] = prev.t[k];
    a.pW = prev.width, a.pH = prev.height;
    a.pdepth = prev_depth;
    a.fx = lvl.fx, a.fy = lvl.fy, a.cx = lvl.cx, a.cy = lvl.cy;
    a.W = lvl.width, a.H = lvl.height;
    a.depth = depth;
    a.pose = pose;
    a.dist2 = dist_thresh * dist_thresh;
    // at most kIcpMaxBlocks blocks; larger levels loop inside the block
    const size_t want = ((size_t)lvl.width * lvl.height + 255) / 256;
    a.nblk = (int)(want < kIcpMaxBlocks ? want : kIcpMaxBlocks);
    a.part = reinterpret_cast<float*>(ws);
    a.step_x = (256 * a.nblk) % lvl.width, a.step_y = (256 * a.nblk) / lvl.width;
    const bool sane = focal_sane(prev.fx, prev.cx) && focal_sane(prev.fy, prev.cy) && focal_sane(lvl.fx, lvl.cx) &&
                      focal_sane(lvl.fy, lvl.cy);
    if (sane) GPS_LAUNCH(K_ICP, s, k_icp_pairs<true>, dim3(a.nblk), dim3(256), 0, s, a);
    else GPS_LAUNCH(K_ICP, s, k_icp_pairs<false>, dim3(a.nblk), dim3(256), 0, s, a);
    if (step_pose)  // the step in the same launch as the system's sum (gps_icp_step)
        GPS_LAUNCH(K_ICP, s, k_icp_total_solve, dim3(1), dim3(1024), 0, s, a.part, a.nblk, sys, step_pose, step_xi);
    else
        GPS_LAUNCH(K_ICP, s, k_icp_total, dim3(1), dim3(1024), 0, s, a.part, a.nblk, sys);
    return hipGetLastError() == hipSuccess ? GPS_OK : GPS_ERR_HIP;
}

gps_status launch_icp_solve(const double* sys, float* pose, float* out_xi, hipStream_t s)
{
    GPS_LAUNCH(K_ICP, s, k_icp_solve, dim3(1), dim3(64), 0, s, sys, pose, out_xi);
    return hipGetLastError() == hipSuccess ? GPS_OK : GPS_ERR_HIP;
}

}  // namespace gps
