// Gaussian removal (Sec. 3.2.2, Eq. 8): a stable compaction of the Gaussian
// set (and of companion arrays such as the Adam moments) that drops the
// Gaussians whose opacity is too low or whose largest scale is too large or
// too small.  The decisions compare stored parameters with thresholds on the
// logit and log-scale axes (binary32), so they are exact and order-free.
//   k_remove_count    per block of 256 Gaussians: how many are kept
//   k_remove_scan     one block: block offsets, kept total (the output row stride)
//   k_remove_scatter  per Gaussian: its rows of every set to its kept position
#include <algorithm>
#include <cmath>

#include "gps_internal.h"
#include "launch.h"
#include "prof.h"
#include "render_common.h"

namespace gps {

constexpr int kRemoveSets = 4;

struct RemovalArgs {
    const float* in[kRemoveSets][6];  // per set: mean, log_scale, quat, opacity_logit, rgb, SH bands
    float* out[kRemoveSets][6];
    int sh_rows;                      // rows of the SH bands (3 K; 0 without)
    int n_sets, M;
    float t_logit, t_hi, t_lo;        // logit(min_opacity), ln(max_scale), ln(min_scale)
    unsigned int* blk_cnt;
    unsigned int* blk_off;
    unsigned int* total;
    int* out_count;
};

__device__ __forceinline__ bool keep_gaussian(const RemovalArgs& a, int g)
{
    const float o = a.in[0][3][g];
    const float* l = a.in[0][1];
    const float lmax = fmaxf(fmaxf(l[g], l[a.M + g]), l[2 * a.M + g]);
    return !(o < a.t_logit) && !(lmax > a.t_hi) && !(lmax < a.t_lo);
}

__global__ void __launch_bounds__(256) k_remove_count(RemovalArgs a)
{
    const int g = blockIdx.x * 256 + threadIdx.x;
    const unsigned int k = (g < a.M && keep_gaussian(a, g)) ? 1u : 0u;
    unsigned int tot;
    block_excl_scan<256>(k, &tot);
    if (threadIdx.x == 0) a.blk_cnt[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(1024) k_remove_scan(RemovalArgs a, int nblk)
{
    __shared__ unsigned int wsum[16];
    __shared__ unsigned int carry_s;
    if (threadIdx.x == 0) carry_s = 0u;
    __syncthreads();
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int base = 0; base < nblk; base += 1024) {
        const int i = base + threadIdx.x;
        const unsigned int c = i < nblk ? a.blk_cnt[i] : 0u;
        unsigned int x = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned int y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[wid] = x;
        __syncthreads();
        unsigned int before = 0u, total = 0u;
        for (int k = 0; k < 16; ++k) {
            if (k < wid) before += wsum[k];
            total += wsum[k];
        }
        const unsigned int carry = carry_s;
        if (i < nblk) a.blk_off[i] = carry + before + x - c;
        __syncthreads();
        if (threadIdx.x == 0) carry_s = carry + total;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *a.total = carry_s;
        if (a.out_count) *a.out_count = (int)carry_s;
    }
}

// One set per grid row.  A Gaussian's values are loaded together before the first is stored: one row
// after the other, each waited for its own round trip (100 k Gaussians and two companion sets:
// 15 us, so 6.6).
__global__ void __launch_bounds__(256) k_remove_scatter(RemovalArgs a)
{
    constexpr int kRows[5] = {3, 3, 4, 1, 3}, kAhead = 8;
    const int g = blockIdx.x * 256 + threadIdx.x, s = blockIdx.y;
    const bool k = g < a.M && keep_gaussian(a, g);
    unsigned int tot;
    const unsigned int excl = block_excl_scan<256>(k ? 1u : 0u, &tot);
    if (!k) return;
    const size_t pos = a.blk_off[blockIdx.x] + excl;
    const size_t nk = *a.total;  // row stride of the outputs
    float v[14];
    int j = 0;
#pragma unroll
    for (int f = 0; f < 5; ++f)
#pragma unroll
        for (int r = 0; r < kRows[f]; ++r) v[j++] = a.in[s][f][(size_t)r * a.M + g];
    j = 0;
#pragma unroll
    for (int f = 0; f < 5; ++f)
#pragma unroll
        for (int r = 0; r < kRows[f]; ++r) a.out[s][f][(size_t)r * nk + pos] = v[j++];
    for (int r0 = 0; r0 < a.sh_rows; r0 += kAhead) {
#pragma unroll
        for (int r = 0; r < kAhead; ++r) v[r] = a.in[s][5][(size_t)min(r0 + r, a.sh_rows - 1) * a.M + g];
#pragma unroll
        for (int r = 0; r < kAhead; ++r)
            if (r0 + r < a.sh_rows) a.out[s][5][(size_t)(r0 + r) * nk + pos] = v[r];
    }
}

size_t removal_workspace_bytes(int M)
{
    const size_t nblk = M > 0 ? (size_t)(M + 255) / 256 : 1;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    return al(4 * nblk) * 2 + 256;
}

gps_status launch_remove_gaussians(const gps_removal_cfg* cfg, const gps_gaussians* sets_in, gps_gaussians* sets_out,
                                   int n_sets, int* out_count, char* ws, hipStream_t s)
{
    RemovalArgs a;
    a.n_sets = n_sets;
    a.M = sets_in[0].count;
    a.t_logit = (float)std::log((double)cfg->min_opacity / (1.0 - (double)cfg->min_opacity));
    a.t_hi = (float)std::log((double)cfg->max_scale);
    a.t_lo = (float)std::log((double)cfg->min_scale);
    for (int k = 0; k < n_sets; ++k) {
        const gps_gaussians& gi = sets_in[k];
        gps_gaussians& go = sets_out[k];
        a.in[k][0] = gi.mean, a.in[k][1] = gi.log_scale, a.in[k][2] = gi.quat, a.in[k][3] = gi.opacity_logit,
        a.in[k][4] = gi.rgb;
        a.out[k][0] = go.mean, a.out[k][1] = go.log_scale, a.out[k][2] = go.quat, a.out[k][3] = go.opacity_logit,
        a.out[k][4] = go.rgb;
        a.in[k][5] = gi.sh;
        a.out[k][5] = go.sh;
    }
    a.sh_rows = 3 * sh_count(sets_in[0].sh_degree);
    const int nblk = a.M > 0 ? (a.M + 255) / 256 : 0;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t nb = nblk > 0 ? (size_t)nblk : 1;
    a.blk_cnt = reinterpret_cast<unsigned int*>(ws);
    a.blk_off = reinterpret_cast<unsigned int*>(ws + al(4 * nb));
    a.total = reinterpret_cast<unsigned int*>(ws + 2 * al(4 * nb));
    a.out_count = out_count;
    if (nblk > 0) GPS_LAUNCH(K_REMOVE, s, k_remove_count, dim3(nblk), dim3(256), 0, s, a);
    GPS_LAUNCH(K_REMOVE, s, k_remove_scan, dim3(1), dim3(1024), 0, s, a, nblk);
    if (nblk > 0) GPS_LAUNCH(K_REMOVE, s, k_remove_scatter, dim3(nblk, n_sets), dim3(256), 0, s, a);
    return hipGetLastError() == hipSuccess ? GPS_OK : GPS_ERR_HIP;
}

// ------------------------------------------------------------------ insertion
// Gaussian insertion (Sec. 3.2.2, Eq. 6; Appendix A).
//   k_insert_flags  per pixel: mask (bit 0) and sample (bit 1) flags and the
//                   mask depth (the depth on mask pixels, 0 elsewhere); per
//                   block of 256 pixels, the number taken
//   k_insert_scan_bits  block 0: block offsets, total taken -> out_count; the others:
//                   per 8x8 pixel block, a 64-bit word of its mask pixels
//   k_insert_place  per taken pixel: its row-major output position
//   k_insert_init   per new Gaussian: its surface point, normal, scale (the
//                   three nearest mask vertices over the whole mask), rotation

struct InsertArgs {
    DevCam cam;
    const float* render_rgb;
    const float* frame_rgb;
    const float* weight;
    const float* depth;
    const float* rnd;
    float* out[6];  // mean, log_scale, quat, opacity_logit, rgb, SH bands: planar [rows][capacity]
    int sh_rows;    // rows of the SH bands (3 K; 0 without): new Gaussians start with zeros there
    int* out_pixel;
    int* out_count;
    int capacity;
    int nbx, nby;  // 8x8 pixel blocks per row and column
    float t_c, t_w, t_frac, scale_cap, flat_ratio, logit_opacity;
    unsigned int* flags;
    unsigned long long* bits;  // per 8x8 block: bit (8 row + column) set on mask pixels
    unsigned int* blk_cnt;
    unsigned int* blk_off;
    unsigned int* total;
    int* list;     // pixel of each output position
    float* mdepth; // depth of the mask pixels, 0 elsewhere
};

__global__ void __launch_bounds__(256) k_insert_flags(InsertArgs a)
{
    const int n = a.cam.W * a.cam.H;
    const int p = blockIdx.x * 256 + threadIdx.x;
    unsigned int f = 0u;
    if (p < n) {
        const size_t HW = (size_t)n;
        const float e = (fabsf(a.render_rgb[p] - a.frame_rgb[p]) + fabsf(a.render_rgb[HW + p] - a.frame_rgb[HW + p])) +
                        fabsf(a.render_rgb[2 * HW + p] - a.frame_rgb[2 * HW + p]);
        const bool mask = a.depth[p] > 0.0f && e > a.t_c && a.weight[p] < a.t_w;
        f = (mask ? 1u : 0u) | ((mask && a.rnd[p] < a.t_frac) ? 2u : 0u);
        a.flags[p] = f;
        a.mdepth[p] = mask ? a.depth[p] : 0.0f;
    }
    unsigned int tot;
    block_excl_scan<256>((f >> 1) & 1u, &tot);
    if (threadIdx.x == 0) a.blk_cnt[blockIdx.x] = tot;
}

// Two things that depend on the flags alone, in one launch: block 0 scans the counts of
// the flag blocks; each wavefront of the others packs one 8x8 pixel block's mask (lane 8 r + c
// holds pixel (8 bx + c, 8 by + r)).
__global__ void __launch_bounds__(1024) k_insert_scan_bits(InsertArgs a, int nblk)
{
    __shared__ unsigned int wsum[16];
    __shared__ unsigned int carry_s;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (blockIdx.x > 0) {
        const int blk = ((int)blockIdx.x - 1) * 16 + wid;
        if (blk >= a.nbx * a.nby) return;  // uniform per wavefront
        const int bx = blk % a.nbx, by = blk / a.nbx;
        const int px = bx * 8 + (lane & 7), py = by * 8 + (lane >> 3);
        const bool m = px < a.cam.W && py < a.cam.H && a.mdepth[(size_t)py * a.cam.W + px] > 0.0f;
        const unsigned long long word = __ballot(m);
        if (lane == 0) a.bits[blk] = word;
        return;
    }
    if (threadIdx.x == 0) carry_s = 0u;
    __syncthreads();
    for (int base = 0; base < nblk; base += 1024) {
        const int i = base + threadIdx.x;
        const unsigned int c = i < nblk ? a.blk_cnt[i] : 0u;
        unsigned int x = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned int y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[wid] = x;
        __syncthreads();
        unsigned int before = 0u, total = 0u;
        for (int k = 0; k < 16; ++k) {
            if (k < wid) before += wsum[k];
            total += wsum[k];
        }
        const unsigned int carry = carry_s;
        if (i < nblk) a.blk_off[i] = carry + before + x - c;
        __syncthreads();
        if (threadIdx.x == 0) carry_s = carry + total;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *a.total = carry_s;
        if (a.out_count) *a.out_count = (int)carry_s;
    }
}

// Camera-frame point of pixel (i, j) at depth d.
__device__ __forceinline__ void cam_point(const DevCam& c, int i, int j, float d, float x[3])
{
    x[0] = ((float)i - c.cx) / c.fx * d;
    x[1] = ((float)j - c.cy) / c.fy * d;
    x[2] = d;
}

// The normal and the neighbour distances are rotation- and translation-free, so
// they are formed from camera-frame differences (no world-coordinate
// cancellation in binary32); only the mean and the normal are rotated to the
// world frame, x_w = R^T (x_c - t).
// Per pixel: the output position of each sampled pixel (row-major order) into
// the list, so that the initialisation runs one lane per new Gaussian.
__global__ void __launch_bounds__(256) k_insert_place(InsertArgs a)
{
    const int n = a.cam.W * a.cam.H;
    const int p = blockIdx.x * 256 + threadIdx.x;
    const bool take = p < n && (a.flags[p] & 2u);
    unsigned int tot;
    const unsigned int excl = block_excl_scan<256>(take ? 1u : 0u, &tot);
    if (!take) return;
    const unsigned int pos = a.blk_off[blockIdx.x] + excl;
    if (pos < (unsigned int)a.capacity) a.list[pos] = p;
}

// The three smallest of two ascending triples, ascending.
__device__ __forceinline__ void merge3(float& a0, float& a1, float& a2, float c0, float c1, float c2)
{
    const float m1 = fminf(fminf(a1, c1), fmaxf(a0, c0));
    const float m2 = fminf(fminf(a2, c2), fminf(fmaxf(a0, c1), fmaxf(a1, c0)));
    a0 = fminf(a0, c0);
    a1 = m1;
    a2 = m2;
}

// New Gaussian `pos` (Appendix A) with first scale s1, by one lane.
__device__ __forceinline__ void write_gaussian(const InsertArgs& a, unsigned int pos, float s1)
{
    const int W = a.cam.W, H = a.cam.H, n = W * H;
    const DevCam& c = a.cam;
    const int p = a.list[pos];
    const int i = p % W, j = p / W;
    float X[3];
    cam_point(c, i, j, a.depth[p], X);
    // normal: central differences of the vertex map, facing the camera (at -X)
    float nc[3] = {-X[0], -X[1], -X[2]};
    if (i > 0 && i < W - 1 && j > 0 && j < H - 1 && a.depth[p - 1] > 0.0f && a.depth[p + 1] > 0.0f &&
        a.depth[p - W] > 0.0f && a.depth[p + W] > 0.0f) {
        float xm[3], xp[3], ym[3], yp[3];
        cam_point(c, i - 1, j, a.depth[p - 1], xm);
        cam_point(c, i + 1, j, a.depth[p + 1], xp);
        cam_point(c, i, j - 1, a.depth[p - W], ym);
        cam_point(c, i, j + 1, a.depth[p + W], yp);
        const float dx[3] = {xp[0] - xm[0], xp[1] - xm[1], xp[2] - xm[2]};
        const float dy[3] = {yp[0] - ym[0], yp[1] - ym[1], yp[2] - ym[2]};
        const float cr[3] = {dx[1] * dy[2] - dx[2] * dy[1], dx[2] * dy[0] - dx[0] * dy[2], dx[0] * dy[1] - dx[1] * dy[0]};
        if (cr[0] * cr[0] + cr[1] * cr[1] + cr[2] * cr[2] > 0.0f) {
            nc[0] = cr[0];
            nc[1] = cr[1];
            nc[2] = cr[2];
        }
    }
    const float inl = 1.0f / sqrtf(nc[0] * nc[0] + nc[1] * nc[1] + nc[2] * nc[2]);
    const float sg = (nc[0] * X[0] + nc[1] * X[1] + nc[2] * X[2]) > 0.0f ? -inl : inl;
#pragma unroll
    for (int k = 0; k < 3; ++k) nc[k] *= sg;
    float nv[3], V[3];
    const float xt[3] = {X[0] - c.t[0], X[1] - c.t[1], X[2] - c.t[2]};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        nv[k] = c.R[k] * nc[0] + c.R[3 + k] * nc[1] + c.R[6 + k] * nc[2];
        V[k] = c.R[k] * xt[0] + c.R[3 + k] * xt[1] + c.R[6 + k] * xt[2];
    }
    // shortest-arc rotation taking the local z axis onto the normal; for a normal
    // near -z the scalar part 1 + n_z is formed as (n_x^2 + n_y^2) / (1 - n_z), its
    // value on the unit sphere, so that the rounding of the normalisation cannot
    // leave a spurious 1 + n_z against vanishing n_x, n_y
    const float nxy2 = nv[0] * nv[0] + nv[1] * nv[1];
    float q[4] = {nv[2] < 0.0f ? nxy2 / (1.0f - nv[2]) : 1.0f + nv[2], -nv[1], nv[0], 0.0f};
    const float qn = sqrtf(q[0] * q[0] + q[1] * q[1] + q[2] * q[2]);
    if (qn > 0.0f) {
        q[0] /= qn;
        q[1] /= qn;
        q[2] /= qn;
    } else {
        q[0] = 0.0f;
        q[1] = 1.0f;
        q[2] = 0.0f;
    }
    const size_t C = (size_t)a.capacity, HW = (size_t)n;
#pragma unroll
    for (int k = 0; k < 3; ++k) a.out[0][k * C + pos] = V[k];
    a.out[1][pos] = logf(s1);
    a.out[1][C + pos] = logf(s1);
    a.out[1][2 * C + pos] = logf(a.flat_ratio * s1);
#pragma unroll
    for (int k = 0; k < 4; ++k) a.out[2][k * C + pos] = q[k];
    a.out[3][pos] = a.logit_opacity;
#pragma unroll
    for (int k = 0; k < 3; ++k) a.out[4][k * C + pos] = a.frame_rgb[k * HW + p];
    for (int r = 0; r < a.sh_rows; ++r) a.out[5][r * C + pos] = 0.0f;
    if (a.out_pixel) a.out_pixel[pos] = p;
}

// Per new Gaussian (position pos < min(sampled, capacity)): NN lanes search its nearest
// mask vertices together, then one lane of the block per Gaussian writes it.
//
// The search is a chain of dependent loads (a block's word, then the depths of its mask
// pixels), so for a keyframe's few thousand it is bound by latency: with one lane per Gaussian (72
// blocks for the 18.4 k Gaussians of a 1280x720 keyframe) it took 170 us, most of the chip idle.  Sixteen
// lanes (a quarter of a wavefront, so that the group's exchanges stay in DPP rows) split each 8x8
// block's 64 pixels four to a lane, read the words of up to 16 blocks of a ring in one round
// trip, and keep a triple of smallest distances per lane that is merged once per ring; the
// three smallest values are the same whatever the order of the search.  Where the whole image is
// new, the groups' exchanges bound it, and eight lanes make fewer.  A 1280x720 frame's insertion with one, 16,
// 8 and 4 lanes, in us: of 20 k 173, 60, 62, 78; of 36 k 118, 72, 70, 74; of 51 k 167, 84, 73, 84; of 203 k
// 191, 233, 160, 143; of 903 k 638, 777, 521, 552.
// The grid is bounded (the number of new Gaussians is only known on the device, and a capacity
// of every pixel would launch 57,600 blocks at 1280x720, most of them empty); blocks stride.
constexpr int kNNFew = 16, kNNMany = 8;
constexpr unsigned int kFewNew = 32768;
constexpr unsigned int kInitGrid = 2048;

// s_scale: one word per Gaussian of the block.
template <int NN>
__device__ __forceinline__ void insert_groups(const InsertArgs& a, unsigned int count, float* s_scale)
{
    const int W = a.cam.W, H = a.cam.H;
    constexpr int kPer = 256 / NN;    // Gaussians per block
    constexpr int kBits = 64 / NN;   // pixels of an 8x8 block per lane
    const DevCam& c = a.cam;
    for (unsigned int pos0 = blockIdx.x * kPer; pos0 < count; pos0 += gridDim.x * kPer) {  // the same for the whole block
        const unsigned int qpos = pos0 + threadIdx.x / NN;
        if (qpos < count) {
            const int l = threadIdx.x % NN;
            const int p = a.list[qpos];
            const int i = p % W, j = p / W;
            float X[3];
            cam_point(c, i, j, a.depth[p], X);
            // The three nearest other mask vertices over the whole mask (Appendix A), by
            // rings of 8x8 blocks around the query's block.  A pixel column c beyond the
            // scanned window holds only points of the half-space fx x - (c - cx) z <= 0
            // (or >= 0), so no unscanned vertex is nearer than the distance from X to the
            // nearest such plane: the search stops once the third distance is within it.
            // A third distance above sqrt(3) scale_cap gives s1 = scale_cap whatever the
            // exact neighbours are, so the rings stop there as well once three are held.
            const float r2max = 3.0f * a.scale_cap * a.scale_cap;
            float l0 = INFINITY, l1 = INFINITY, l2 = INFINITY;  // this lane's squared distances, ascending
            float b0 = INFINITY, b1 = INFINITY, b2 = INFINITY;  // the group's
            int cnt = 0;                                        // vertices scanned by the group
            const int bi = i >> 3, bj = j >> 3;
            // Distance from X (on the ray of pixel column i, depth Z) to the plane through the
            // camera centre holding the rays of column c: |i - c| Z / |(fx, c - cx)| (the
            // integer difference is exact, so the bound has no cancellation); rows alike.
            auto plane_dist = [&](int q, int cq, float f, float cc) {
                const float k = (float)cq - cc;
                return (float)abs(q - cq) * X[2] / sqrtf(f * f + k * k);
            };
            // lower bound of the distance from X to any point of pixel columns [c0, c1], rows [r0, r1]
            auto box_bound = [&](int c0, int c1, int r0, int r1) {
                float lx = 0.0f, ly = 0.0f;
                if (c0 > i) lx = plane_dist(i, c0, c.fx, c.cx);
                else if (c1 < i) lx = plane_dist(i, c1, c.fx, c.cx);
                if (r0 > j) ly = plane_dist(j, r0, c.fy, c.cy);
                else if (r1 < j) ly = plane_dist(j, r1, c.fy, c.cy);
                return fmaxf(lx, ly) * (1.0f - 1e-4f);  // rounding margin: never above the true bound
            };
            for (int r = 0;; ++r) {
                const int bx0 = bi - r, bx1 = bi + r, by0 = bj - r, by1 = bj + r;
                // The ring's blocks in the order top row, bottom row, left and right columns.
                const int ring = r == 0 ? 1 : 8 * r, side = 2 * r + 1;
                for (int q0 = 0; q0 < ring; q0 += NN) {
                    // lane l looks at block q0 + l: in the image, and near enough to matter
                    const int q = q0 + l;
                    int bx, by;
                    if (q < side) bx = bx0 + q, by = by0;
                    else if (q < 2 * side) bx = bx0 + q - side, by = by1;
                    else bx = (q & 1) ? bx1 : bx0, by = by0 + 1 + ((q - 2 * side) >> 1);
                    bool want = q < ring && bx >= 0 && bx < a.nbx && by >= 0 && by < a.nby;
                    if (want && cnt >= 3) {
                        const float lb = box_bound(bx * 8, min(bx * 8 + 7, W - 1), by * 8, min(by * 8 + 7, H - 1));
                        want = !(lb * lb >= b2);
                    }
                    const unsigned long long mine = want ? a.bits[(size_t)by * a.nbx + bx] : 0ull;
                    // blocks of this batch that hold mask pixels, as bits of the group's lanes
                    unsigned int have = (unsigned int)(__ballot(mine != 0ull) >> (threadIdx.x & (64 - NN))) & ((1u << NN) - 1u);
                    const int at = bx | (by << 16);
                    while (have) {
                        const int src = __ffs((int)have) - 1;
                        have &= have - 1u;
                        const unsigned int lo = __shfl((unsigned int)mine, src, NN);
                        const unsigned int hi = __shfl((unsigned int)(mine >> 32), src, NN);
                        const int xy = __shfl(at, src, NN);
                        cnt += __popc(lo) + __popc(hi);
                        // this lane's consecutive pixels of the block
                        unsigned int part = ((l * kBits < 32 ? lo : hi) >> (l * kBits & 31)) & ((1u << kBits) - 1u);
                        while (part) {
                            const int k = l * kBits + __ffs((int)part) - 1;
                            part &= part - 1u;
                            const int ii = (xy & 0xffff) * 8 + (k & 7), jj = (xy >> 16) * 8 + (k >> 3);
                            if (ii == i && jj == j) continue;
                            float U[3];
                            cam_point(c, ii, jj, a.mdepth[(size_t)jj * W + ii], U);
                            const float d2 = (U[0] - X[0]) * (U[0] - X[0]) + (U[1] - X[1]) * (U[1] - X[1]) +
                                             (U[2] - X[2]) * (U[2] - X[2]);
                            if (d2 < l2) {
                                if (d2 < l1) {
                                    l2 = l1;
                                    if (d2 < l0) {
                                        l1 = l0;
                                        l0 = d2;
                                    } else {
                                        l1 = d2;
                                    }
                                } else {
                                    l2 = d2;
                                }
                            }
                        }
                    }
                }
                if (r == 0) --cnt;  // the query is a mask pixel of its own block
                b0 = l0, b1 = l1, b2 = l2;
#pragma unroll
                for (int m = 1; m < NN; m <<= 1) {
                    const float c0 = __shfl_xor(b0, m, NN), c1 = __shfl_xor(b1, m, NN), c2 = __shfl_xor(b2, m, NN);
                    merge3(b0, b1, b2, c0, c1, c2);
                }
                // distance bound of everything outside the scanned window
                const int x0 = max(bx0, 0) * 8, x1 = min(bx1 * 8 + 7, W - 1);
                const int y0 = max(by0, 0) * 8, y1 = min(by1 * 8 + 7, H - 1);
                float bound = INFINITY;
                if (x0 > 0) bound = fminf(bound, box_bound(0, x0 - 1, j, j));
                if (x1 < W - 1) bound = fminf(bound, box_bound(x1 + 1, W - 1, j, j));
                if (y0 > 0) bound = fminf(bound, box_bound(i, i, 0, y0 - 1));
                if (y1 < H - 1) bound = fminf(bound, box_bound(i, i, y1 + 1, H - 1));
                if (bound == INFINITY) break;                       // the whole image is scanned
                if (cnt >= 3 && b2 <= bound * bound) break;         // exact: nothing unscanned is nearer
                if (cnt >= 3 && bound * bound >= r2max) break;      // the third is beyond sqrt(3) cap: capped
            }
            if (l == 0) {
                float s1 = a.scale_cap;
                if (cnt > 0) {
                    const int m = cnt < 3 ? cnt : 3;
                    const float sum = m == 1 ? b0 : (m == 2 ? b0 + b1 : (b0 + b1) + b2);
                    s1 = fminf(a.scale_cap, sqrtf(sum / (float)m));  // root mean square distance
                }
                s_scale[threadIdx.x / NN] = s1;
            }
        }
        __syncthreads();
        const unsigned int pos = pos0 + threadIdx.x;
        if (threadIdx.x < kPer && pos < count) write_gaussian(a, pos, s_scale[threadIdx.x]);
        __syncthreads();
    }
}

__global__ void __launch_bounds__(256) k_insert_init(InsertArgs a)
{
    __shared__ float s_scale[256 / kNNMany];
    const unsigned int count = min(*a.total, (unsigned int)a.capacity);
    if (count <= kFewNew) insert_groups<kNNFew>(a, count, s_scale);
    else insert_groups<kNNMany>(a, count, s_scale);
}

size_t insertion_workspace_bytes(int W, int H)
{
    const size_t n = (size_t)W * H, nblk = n > 0 ? (n + 255) / 256 : 1;
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t nbits = (size_t)((W + 7) / 8) * ((H + 7) / 8);
    return 3 * al(4 * n) + 2 * al(4 * nblk) + 256 + al(8 * nbits);
}

gps_status launch_insert_gaussians(const gps_insert_cfg* cfg, const DevCam& cam, const float* render_rgb,
                                   const float* frame_rgb, const float* weight, const float* sdf_depth,
                                   const float* rnd, gps_gaussians* out, int* out_pixel, int* out_count, char* ws,
                                   hipStream_t s)
{
    InsertArgs a;
    a.cam = cam;
    a.render_rgb = render_rgb;
    a.frame_rgb = frame_rgb;
    a.weight = weight;
    a.depth = sdf_depth;
    a.rnd = rnd;
    a.out[0] = out->mean, a.out[1] = out->log_scale, a.out[2] = out->quat, a.out[3] = out->opacity_logit,
    a.out[4] = out->rgb;
    a.out[5] = out->sh;
    a.sh_rows = 3 * sh_count(out->sh_degree);
    a.out_pixel = out_pixel;
    a.out_count = out_count;
    a.capacity = out->count;
    a.nbx = (cam.W + 7) / 8;
    a.nby = (cam.H + 7) / 8;
    a.t_c = (float)(3.0 * (double)cfg->delta_c);
    a.t_w = cfg->delta_w;
    a.t_frac = cfg->fraction;
    a.scale_cap = cfg->scale_cap;
    a.flat_ratio = cfg->flat_ratio;
    a.logit_opacity = (float)std::log((double)cfg->opacity / (1.0 - (double)cfg->opacity));
    const size_t n = (size_t)cam.W * cam.H;
    const int nblk = (int)((n + 255) / 256);
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const size_t nb = nblk > 0 ? (size_t)nblk : 1;
    a.flags = reinterpret_cast<unsigned int*>(ws);
    a.blk_cnt = reinterpret_cast<unsigned int*>(ws + al(4 * n));
    a.blk_off = reinterpret_cast<unsigned int*>(ws + al(4 * n) + al(4 * nb));
    a.total = reinterpret_cast<unsigned int*>(ws + al(4 * n) + 2 * al(4 * nb));
    a.list = reinterpret_cast<int*>(ws + al(4 * n) + 2 * al(4 * nb) + 256);
    a.mdepth = reinterpret_cast<float*>(ws + 2 * al(4 * n) + 2 * al(4 * nb) + 256);
    a.bits = reinterpret_cast<unsigned long long*>(ws + 3 * al(4 * n) + 2 * al(4 * nb) + 256);
    const int nbits = a.nbx * a.nby;
    if (nblk > 0) GPS_LAUNCH(K_INSERT, s, k_insert_flags, dim3(nblk), dim3(256), 0, s, a);
    GPS_LAUNCH(K_INSERT, s, k_insert_scan_bits, dim3(1 + (nbits + 15) / 16), dim3(1024), 0, s, a, nblk);
    const size_t cap = (size_t)a.capacity < n ? (size_t)a.capacity : n;
    if (nblk > 0 && cap > 0) {
        GPS_LAUNCH(K_INSERT, s, k_insert_place, dim3(nblk), dim3(256), 0, s, a);
        GPS_LAUNCH(K_INSERT, s, k_insert_init, dim3(std::min((unsigned)((cap + 256 / kNNFew - 1) / (256 / kNNFew)), kInitGrid)), dim3(256), 0, s, a);
    }
    return hipGetLastError() == hipSuccess ? GPS_OK : GPS_ERR_HIP;
}

}  // namespace gps
