// TSDF + colour fusion and SDF raycast (Sec. 3.1 first pass, Sec. 3.2.1).
//
// Fusion is one lane per lattice point in view, lanes along x so that the volume
// arrays stream coalesced; only points in the frustum with a valid depth
// sample read and write the volume, so traffic is 8 B/point outside the
// truncation band and 32 B/point inside it (read + write).
//
// The raycast is one lane per pixel.  The march decides the crossing sample in
// binary32 with a fixed evaluation order (the same order every implementation
// of this path uses, so the crossing index is reproducible), and skips samples
// whose 2x2x2 stencil lies in an 8^3 brick whose minimum signed distance is
// positive -- such samples cannot be a crossing, so skipping them does not
// change which sample is found.
#include <algorithm>
#include <cmath>

#include "gps_internal.h"
#include "launch.h"
#include "prof.h"
#include "sdf_common.h"

namespace gps {

// ----------------------------------------------------------------- fusion
// A cell is 2^lx x 2^(6-lx) lattice points of a z plane, one per lane.  A block takes 64 cells from
// all over the lattice (the ones in view are neighbours: consecutive cells give blocks of 64
// and blocks of none): its first wavefront tests, a lane each, whether they lie outside the view, and
// all its wavefronts then fuse the others in turn.  A lane per point executed about 90
// instructions a wavefront for every point of the lattice; what is left is bound by the
// three dependent loads of a point.  256^3 points, 1280x720 frame: 21 us, without the test 39, with
// consecutive cells 35, with 16 wavefronts a block 24.
constexpr int kFuseWaves = 8;

struct FuseArgs {
    FuseCtx ctx;
    int nx, ny;
    unsigned int N;
    int lx;                     // log2 of a cell's width
    unsigned int cx, cy, cells;  // cells along x, along y, in all
    unsigned int first;         // of this launch
    float* tsdf;
    float* w;
    float* col;
    float* cw;
};

// No point of [x0, x1] x [y0, y1] x {z} projects into the image: it is behind the camera, or
// beyond one border of it, at all four corners, by more than the rounding of fuse_point's
// coordinates (below 1e-6 of the sums' magnitude) and of its pixel (below a hundredth and 1e-6 of the
// image): the functions are linear, so all points between are too.  False for anything not finite.
__device__ __forceinline__ bool fuse_outside(const FuseCtx& a, int x0, int x1, int y0, int y1, int z)
{
    const DevCam& c = a.cam;
    const float px[2] = {a.ox + a.voxel * (float)x0, a.ox + a.voxel * (float)x1};
    const float py[2] = {a.oy + a.voxel * (float)y0, a.oy + a.voxel * (float)y1};
    const float pz = a.oz + a.voxel * (float)z;
    float m = 0.0f, tz = 0.0f;
#pragma unroll
    for (int k = 0; k < 9; ++k) m = fmaxf(m, fabsf(c.R[k]));
#pragma unroll
    for (int k = 0; k < 3; ++k) tz = fmaxf(tz, fabsf(c.t[k]));
    const float reach = fmaxf(fabsf(px[0]), fabsf(px[1])) + fmaxf(fabsf(py[0]), fabsf(py[1])) + fabsf(pz) + fabsf(a.ox) +
                        fabsf(a.oy) + fabsf(a.oz);  // (a point's own rounding is relative to its origin's too)
    const float e = 4e-6f * (m * reach + tz);
    const float W = (float)c.W, H = (float)c.H;
    const float du = 0.01f + 1e-6f * (fabsf(c.cx) + W), dv = 0.01f + 1e-6f * (fabsf(c.cy) + H);
    const float kl = c.cx + 0.5f + du, kr = c.cx + 0.5f - W - du, kt = c.cy + 0.5f + dv, kb = c.cy + 0.5f - H - dv;
    const float eu = e * (fabsf(c.fx) + fabsf(c.cx) + W + 2.0f), ev = e * (fabsf(c.fy) + fabsf(c.cy) + H + 2.0f);
    bool behind = true, left = true, right = true, top = true, bottom = true;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float X = px[k & 1], Y = py[k >> 1];
        const float xc = c.R[0] * X + c.R[1] * Y + c.R[2] * pz + c.t[0];
        const float yc = c.R[3] * X + c.R[4] * Y + c.R[5] * pz + c.t[1];
        const float zc = c.R[6] * X + c.R[7] * Y + c.R[8] * pz + c.t[2];
        behind = behind && zc < -e;
        left = left && c.fx * xc + kl * zc < -eu;
        right = right && c.fx * xc + kr * zc > eu;
        top = top && c.fy * yc + kt * zc < -ev;
        bottom = bottom && c.fy * yc + kb * zc > ev;
    }
    return behind || left || right || top || bottom;
}

__global__ void __launch_bounds__(64 * kFuseWaves) k_fuse(FuseArgs a)
{
    __shared__ int4 cell[64];
    __shared__ int n_seen;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int wx = 1 << a.lx, wy = 64 >> a.lx;
    if (wid == 0) {
        const unsigned int c = a.first + lane * gridDim.x + blockIdx.x, r = c / a.cx;
        const int x0 = (int)(c - r * a.cx) << a.lx, z = (int)(r / a.cy);
        const int y0 = (int)(r - (unsigned int)z * a.cy) * wy;
        const bool seen = c < a.cells && !fuse_outside(a.ctx, x0, min(x0 + wx, a.nx) - 1, y0, min(y0 + wy, a.ny) - 1, z);
        const unsigned long long m = __builtin_amdgcn_ballot_w64(seen);
        if (seen)
            cell[__builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, 0u))] =
                make_int4(x0, y0, z, 0);
        if (lane == 0) n_seen = (int)__builtin_popcountll(m);
    }
    __syncthreads();
    const int n = n_seen;
    for (int k = wid; k < n; k += kFuseWaves) {
        const int4 c = cell[k];
        const int x = c.x + (lane & (wx - 1)), y = c.y + (lane >> a.lx);
        if (x < a.nx && y < a.ny) {
            const unsigned int idx = ((unsigned int)c.z * (unsigned int)a.ny + (unsigned int)y) * (unsigned int)a.nx + (unsigned int)x;
            fuse_point(a.ctx, x, y, c.z, idx, a.N, a.tsdf, a.w, a.col, a.cw);
        }
    }
}

gps_status launch_fuse(const gps_volume* vol, const gps_camera* cam, const float* depth, const float* rgb,
                       hipStream_t s)
{
    FuseArgs a;
    a.nx = vol->nx;
    a.ny = vol->ny;
    a.ctx.ox = vol->origin[0];
    a.ctx.oy = vol->origin[1];
    a.ctx.oz = vol->origin[2];
    a.ctx.voxel = vol->voxel;
    a.ctx.mu = vol->trunc;
    a.ctx.wmax = vol->max_weight;
    a.N = (unsigned int)((size_t)vol->nx * vol->ny * vol->nz);
    a.ctx.cam = dev_cam(*cam);
    a.ctx.depth = depth;
    a.ctx.img = rgb;
    a.tsdf = vol->tsdf;
    a.w = vol->weight;
    a.col = vol->rgb;
    a.cw = vol->rgb_weight;
    // The widest cell that leaves at most a quarter of its lanes beyond the rows' ends.
    a.lx = 6;
    while (a.lx > 1 && 4ll * a.nx < 3ll * (((a.nx + (1 << a.lx) - 1) >> a.lx) << a.lx)) --a.lx;
    a.cx = (unsigned int)((a.nx + (1 << a.lx) - 1) >> a.lx);
    a.cy = (unsigned int)((a.ny + (64 >> a.lx) - 1) / (64 >> a.lx));
    a.cells = a.cx * a.cy * (unsigned int)vol->nz;
    // 2^31 lanes a launch (a launch may have up to 2^32 - 1; a lattice 2 points wide and high
    // has a cell for every 4 points)
    constexpr unsigned int kLaunchCells = 64u << 22;
    for (a.first = 0u; a.first < a.cells; a.first += kLaunchCells) {
        const unsigned int n = std::min(a.cells - a.first, kLaunchCells);
        GPS_LAUNCH(K_FUSE, s, k_fuse, dim3((n + 63u) / 64u), dim3(64 * kFuseWaves), 0, s, a);
    }
    return hipGetLastError() == hipSuccess ? GPS_OK : GPS_ERR_HIP;
}

// ------------------------------------------------------------ brick minimum
// bmin[b] = min tsdf over lattice points [8b, 8b+8] (clipped), i.e. every
// 2x2x2 stencil whose base point lies in brick b.
struct BrickArgs {
    int nx, ny, nz, bx, by, bz;
    const float* tsdf;
    float* bmin;
};

// Brick minima over the 9^3 lattice points of each brick (the brick and the first
// plane of its +x, +y, +z neighbours: every 2x2x2 sample stencil based in the brick).
// One block per row of bricks along x: each lane takes lattice columns x (lanes along
// x, so every load of the block reads whole rows of the lattice) and the minimum over
// the 9 x 9 (y, z) points of its column, kept in LDS; then each brick takes the
// minimum over its 9 columns.  Rows of up to kRowCols columns; longer ones use the
// per-brick kernel below.
constexpr int kRowCols = 4096;

__global__ void __launch_bounds__(256) k_brick_min_rows(BrickArgs a)
{
    __shared__ float scol[kRowCols];
    const int byi = (int)blockIdx.x % a.by, bzi = (int)blockIdx.x / a.by;
    const int y0 = byi * kBrick, z0 = bzi * kBrick;
    const int ny = min(kBrick + 1, a.ny - y0), nz = min(kBrick + 1, a.nz - z0);
    for (int x = threadIdx.x; x < a.nx; x += 256) {
        // the 81 loads of a column are issued before the first is used (a point past
        // the lattice edge reads the column's first point again)
        float v[kBrick + 1][kBrick + 1];
#pragma unroll
        for (int dz = 0; dz < kBrick + 1; ++dz)
#pragma unroll
            for (int dy = 0; dy < kBrick + 1; ++dy) {
                const int yy = y0 + (dy < ny ? dy : 0), zz = z0 + (dz < nz ? dz : 0);
                v[dz][dy] = a.tsdf[x + (size_t)a.nx * ((size_t)yy + (size_t)a.ny * (size_t)zz)];
            }
        float m = INFINITY;
#pragma unroll
        for (int dz = 0; dz < kBrick + 1; ++dz)
#pragma unroll
            for (int dy = 0; dy < kBrick + 1; ++dy) m = fminf(m, v[dz][dy]);
        scol[x] = m;
    }
    __syncthreads();
    for (int bxi = threadIdx.x; bxi < a.bx; bxi += 256) {
        const int x0 = bxi * kBrick, x1 = min(x0 + kBrick, a.nx - 1);
        float m = INFINITY;
        for (int x = x0; x <= x1; ++x) m = fminf(m, scol[x]);
        a.bmin[bxi + (size_t)a.bx * (byi + (size_t)a.by * bzi)] = m;
    }
}

// The same minima, one wavefront per 8^3 brick, four bricks per block (rows longer
// than kRowCols).
__global__ void __launch_bounds__(256) k_brick_min(BrickArgs a)
{
    const int b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (b >= a.bx * a.by * a.bz) return;
    const int bxi = b % a.bx, byi = (b / a.bx) % a.by, bzi = b / (a.bx * a.by);
    const int x0 = bxi * kBrick, y0 = byi * kBrick, z0 = bzi * kBrick;
    float m = INFINITY;
    for (int k = lane; k < 9 * 9 * 9; k += 64) {
        const int dx = k % 9, dy = (k / 9) % 9, dz = k / 81;
        const int x = x0 + dx, y = y0 + dy, z = z0 + dz;
        if (x < a.nx && y < a.ny && z < a.nz) m = fminf(m, a.tsdf[x + (size_t)a.nx * (y + (size_t)a.ny * z)]);
    }
    m = -wave_max(-m);
    if (lane == 0) a.bmin[b] = m;
}

// Superbricks of kSuper^3 = 64 bricks: the minimum of their bricks' minima (one
// wavefront each, a lane per brick), so a superbrick above the threshold has
// every sample stencil based in it positive.
constexpr int kSuper = 4;

__global__ void __launch_bounds__(256) k_super_min(const float* __restrict__ bmin, float* __restrict__ smin, int bx,
                                                   int by, int bz, int sx, int sy, int sz)
{
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (t >= sx * sy * sz) return;
    const int jx = t % sx, jy = (t / sx) % sy, jz = t / (sx * sy);
    const int x = jx * kSuper + (lane & 3), y = jy * kSuper + ((lane >> 2) & 3), z = jz * kSuper + (lane >> 4);
    float m = (x < bx && y < by && z < bz) ? bmin[x + bx * (y + by * z)] : INFINITY;
    m = -wave_max(-m);
    if (lane == 0) smin[t] = m;
}

// ---------------------------------------------------------------- raycast
// The dense lattice as a Field of the march: planar arrays indexed
// x + nx (y + ny z); samples based in an 8^3 brick (or a 32^3 superbrick) whose
// minimum is positive are skipped.
// NARROW: the lattice's byte offsets fit 32 bits and its row products 24 (narrow_lattice), which
// makes a stencil's four addresses 8 instructions instead of 22, four of them quarter-rate
// multiplies.
template <bool NARROW>
struct DenseField {
    int n[3];
    size_t N;
    const float* tsdf;
    const float* rgb;
    const float* bmin;  // may be null
    const float* smin;  // superbrick minima (null with bmin)
    int bx, by, sx, sy;
    // The last brick found not positive (and its superbrick not positive), or -1:
    // successive samples of a ray mostly stay in one brick, whose answer does not
    // change during a raycast, so its minima are not read again.
    mutable int cbrick = -1;

    __device__ __forceinline__ void fetch8(int plane, const int b[3], float q[8]) const
    {
        const float* f = plane == 0 ? tsdf : rgb + (size_t)(plane - 1) * N;
        if constexpr (NARROW) {
            const unsigned int row = __umul24((unsigned int)b[2], (unsigned int)n[1]) + (unsigned int)b[1];
            const unsigned int o = (__umul24(row, (unsigned int)n[0]) + (unsigned int)b[0]) * 4u;
            const unsigned int oy = 4u * (unsigned int)n[0], oz = oy * (unsigned int)n[1];
            const char* c = reinterpret_cast<const char*>(f);
            const float* p0 = reinterpret_cast<const float*>(c + o);
            const float* p1 = reinterpret_cast<const float*>(c + (o + oy));
            const float* p2 = reinterpret_cast<const float*>(c + (o + oz));
            const float* p3 = reinterpret_cast<const float*>(c + (o + oz + oy));
            q[0] = p0[0];
            q[1] = p0[1];
            q[2] = p1[0];
            q[3] = p1[1];
            q[4] = p2[0];
            q[5] = p2[1];
            q[6] = p3[0];
            q[7] = p3[1];
        } else {
            const size_t sy_ = (size_t)n[0], sz_ = (size_t)n[0] * n[1];
            const float* p = f + b[0] + sy_ * b[1] + sz_ * b[2];
            q[0] = p[0];
            q[1] = p[1];
            q[2] = p[sy_];
            q[3] = p[sy_ + 1];
            q[4] = p[sz_];
            q[5] = p[sz_ + 1];
            q[6] = p[sz_ + sy_];
            q[7] = p[sz_ + sy_ + 1];
        }
    }

    __device__ __forceinline__ bool depth_range(int, int, int, float*, float*) const { return false; }

    // Edge of the positive box that holds samples based at b: a superbrick's, a brick's, or 0
    // (then kept as the last brick found not positive).
    __device__ __forceinline__ int box_edge(const int b[3]) const
    {
        if (!bmin) return 0;
        const int i0 = b[0] >> 3, i1 = b[1] >> 3, i2 = b[2] >> 3;
        const int bi = i0 + bx * (i1 + by * i2);
        if (bi == cbrick) return 0;
        // the first test takes both minima, so both are read in one round trip
        const float ms = smin[(i0 >> 2) + sx * ((i1 >> 2) + sy * (i2 >> 2))], mb = bmin[bi];
        if (!(fmaxf(ms, mb) > kBrickPositive)) {
            cbrick = bi;
            return 0;
        }
        return ms > kBrickPositive ? kBrick * kSuper : kBrick;
    }

    __device__ __forceinline__ bool skip_box(const int b[3], float lo[3], float* edge) const
    {
        const int e = box_edge(b);
        if (e == 0) return false;
#pragma unroll
        for (int k = 0; k < 3; ++k) lo[k] = (float)(b[k] & -e);
        *edge = (float)e;
        return true;
    }
};

// Bound by instruction issue and the longest rays: a ray of a room view evaluates 16 samples (the
// most of its wavefront; up to 80 where it grazes a wall) and jumps over about as many boxes.
// 8x8 pixels a wavefront keep its rays within about a voxel.  One visit per box (see the slack
// in march_pixel), approximate exits, 32-bit stencil addresses and one bounds test per
// axis took a 1280x720 view of a 256^3 room from 139 to 103 us (4500 -> 2850 instructions a
// wavefront).  Measured and left: jumps and evaluations in loops of their own (fewer
// instructions, but lanes wait for each other twice: 163 us), one wavefront per workgroup (the same time).
template <bool NARROW>
__global__ void __launch_bounds__(256) k_raycast(MarchArgs a, DenseField<NARROW> fld)
{
    const int view = blockIdx.z;
    const DevCam& c = a.cams[view];
    // 16x16 pixels a block, 8x8 a wavefront; 16x4 where every sample is evaluated, which then reads fewer lines a
    // stencil (without brick minima, 8x8 and 16x4 in us: 640x480 view of 400^3 points 466 and 459, of 512^3 605
    // and 587; with them 88 and 92, 100 and 100, a 1280x720 view of 512^3 126 and 133)
    const int wid = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int dx = fld.bmin ? (wid & 1) * 8 + (lane & 7) : lane & 15;
    const int dy = fld.bmin ? (wid >> 1) * 8 + (lane >> 3) : wid * 4 + (lane >> 4);
    const int col = blockIdx.x * 16 + dx, row = blockIdx.y * 16 + dy;
    if (col >= c.W || row >= c.H) return;
    const DenseField<NARROW> f = fld;  // this lane's copy (it keeps the last brick found not positive)
    march_pixel(a, f, view, col, row);
}

// Byte offsets below 2^32 and the factors of an index below 2^24 (DenseField<true>).
static bool narrow_lattice(int nx, int ny, int nz)
{
    return (unsigned long long)nx * ny * nz < (1ull << 30) && nx < (1 << 24) && (unsigned long long)ny * nz < (1ull << 24);
}

gps_status launch_raycast(const gps_volume* vol, const gps_camera* cams, int n_views, float* const* out_depth,
                          float* const* out_rgb, float z_near, float step, hipStream_t s)
{
    MarchArgs a;
    int maxW, maxH;
    march_setup(&a, vol->nx, vol->ny, vol->nz, vol->origin, vol->voxel, z_near, step, cams, n_views, out_depth,
                out_rgb, &maxW, &maxH);
    DenseField<true> f;
    f.n[0] = vol->nx;
    f.n[1] = vol->ny;
    f.n[2] = vol->nz;
    f.N = (size_t)vol->nx * vol->ny * vol->nz;
    f.tsdf = vol->tsdf;
    f.rgb = vol->rgb;
    f.bx = (vol->nx + kBrick - 1) / kBrick;
    f.by = (vol->ny + kBrick - 1) / kBrick;
    const int bz = (vol->nz + kBrick - 1) / kBrick;
    f.sx = (f.bx + kSuper - 1) / kSuper;
    f.sy = (f.by + kSuper - 1) / kSuper;
    const int sz = (bz + kSuper - 1) / kSuper;
    f.bmin = vol->brick_min;
    f.smin = vol->brick_min ? vol->brick_min + (size_t)f.bx * f.by * bz : nullptr;
    if (vol->brick_min) {
        BrickArgs b{vol->nx, vol->ny, vol->nz, f.bx, f.by, bz, vol->tsdf, vol->brick_min};
        if (vol->nx <= kRowCols)
            GPS_LAUNCH(K_BRICK_MIN, s, k_brick_min_rows, dim3(f.by * bz), dim3(256), 0, s, b);
        else
            GPS_LAUNCH(K_BRICK_MIN, s, k_brick_min, dim3((f.bx * f.by * bz + 3) / 4), dim3(256), 0, s, b);
        const int ns = f.sx * f.sy * sz;
        GPS_LAUNCH(K_BRICK_MIN, s, k_super_min, dim3((ns + 3) / 4), dim3(256), 0, s, vol->brick_min,
                   vol->brick_min + (size_t)f.bx * f.by * bz, f.bx, f.by, bz, f.sx, f.sy, sz);
        if (hipGetLastError() != hipSuccess) return GPS_ERR_HIP;
    }
    dim3 grid((maxW + 15) / 16, (maxH + 15) / 16, n_views);
    if (narrow_lattice(vol->nx, vol->ny, vol->nz)) {
        GPS_LAUNCH(K_RAYCAST, s, k_raycast<true>, grid, dim3(256), 0, s, a, f);
    } else {
        const DenseField<false> w{{f.n[0], f.n[1], f.n[2]}, f.N, f.tsdf, f.rgb, f.bmin, f.smin, f.bx, f.by, f.sx, f.sy};
        GPS_LAUNCH(K_RAYCAST, s, k_raycast<false>, grid, dim3(256), 0, s, a, w);
    }
    return hipGetLastError() == hipSuccess ? GPS_OK : GPS_ERR_HIP;
}

}  // namespace gps
