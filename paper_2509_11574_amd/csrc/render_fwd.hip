// Forward render: EWA projection, tile binning, per-tile depth sort and
// compositing over the SDF base image, with the loss fused into the
// compositing epilogue (Sec. 3.1 second pass, Eq. 1-4, Eq. 7).
//
// Kernel sequence (one launch each, all grids sized from host-known shapes,
// so the sequence is graph-capturable):
//   k_upload_views view table and, per screen tile, max of the SDF depth (invalid = +inf);
//                  at an upload, not per forward
//   k_project      per (view, Gaussian): projected record, the number of screen tiles its
//                  support box covers (one slot per tile), and per block and tile the
//                  count of the instances that pass the exact culls
//   k_scan_rows    per tile: each block's first place; one block: the slots' numbers
//   k_scan_tiles   one block: tile ranges (k_scan_small: both in one launch, where they are few)
//   k_emit         (depth, view-Gaussian) keys scattered into tile ranges
//                  (k_project_groups, k_emit_groups: the same where no sort follows)
//   k_tile_sort_large  per tile of >= kLongTile instances: its keys by depth buckets in LDS
//                  (shorter lists: registers of the compositing block's first wavefront)
//   k_composite_fwd<TW,TH,B,PPT>  (composite_fwd.hip) per tile: LDS-staged
//                  batches of B records, wavefronts skip records whose support
//                  misses their pixels, front-to-back compositing, loss
//                  partial per tile
//   k_loss_reduce  one block: per-view and total loss
#include "binning.h"
#include "launch.h"
#include "prof.h"
#include "render_common.h"
#include "se3.h"

namespace gps {

// ---------------------------------------------------------------- project
// EWA projection of one Gaussian into one view (Eq. 3; 3DGS convention):
//   p_c = R mu + t, Sigma_3D = R_q diag(s^2) R_q^T, J the pinhole Jacobian,
//   Sigma_2D = (J R) Sigma_3D (J R)^T + dilation I, conic = Sigma_2D^-1.
// Record of 12 floats: r0 = (m_x, m_y, A', B'), r1 = (C', log2 sigma, z, red),
// r2 = (green, blue, half-width, half-height of the support box), the colour
// being the one seen from this view (rgb plus the SH bands), where
// (A', B', C') = (-0.5 a, -b, -0.5 c) log2(e) for the conic (a, b, c), the
// opacity then being exp2(A' dx^2 + B' dx dy + C' dy^2 + log2 sigma).
// The support ellipse where sigma exp(-q/2) >= alpha_min has the bounding box
// m +- sqrt(kappa Sigma_xx), sqrt(kappa Sigma_yy), kappa = 2 ln(sigma/alpha_min);
// it is padded by one pixel and turned into a tile rectangle.
struct ProjOut {
    float4 r0, r1, r2;
    bool valid;
};

template <bool SH>
__device__ __forceinline__ ProjOut project_one(const DevView& V, const RParams& rp, const GParams& gp, int g)
{
    ProjOut o;
    o.valid = false;
    o.r0 = make_float4(0.f, 0.f, 0.f, 0.f);
    o.r1 = make_float4(0.f, 0.f, 0.f, 0.f);
    o.r2 = make_float4(0.f, 0.f, 0.f, 0.f);
    const int M = rp.M;
    const DevCam& c = V.cam;
    const float m0 = gp.mean[g], m1 = gp.mean[M + g], m2 = gp.mean[2 * M + g];
    const float z = d32_row(c.R, c.t, 2, m0, m1, m2);  // depth key (binary32 decision)
    if (!(z >= rp.znear)) return o;
    const float x = c.R[0] * m0 + c.R[1] * m1 + c.R[2] * m2 + c.t[0];
    const float y = c.R[3] * m0 + c.R[4] * m1 + c.R[5] * m2 + c.t[1];
    float qw = gp.quat[g], qx = gp.quat[M + g], qy = gp.quat[2 * M + g], qz = gp.quat[3 * M + g];
    const float qinv = 1.0f / sqrtf(qw * qw + qx * qx + qy * qy + qz * qz);
    qw *= qinv;
    qx *= qinv;
    qy *= qinv;
    qz *= qinv;
    float Rq[9];
    Rq[0] = 1.f - 2.f * (qy * qy + qz * qz);
    Rq[1] = 2.f * (qx * qy - qw * qz);
    Rq[2] = 2.f * (qx * qz + qw * qy);
    Rq[3] = 2.f * (qx * qy + qw * qz);
    Rq[4] = 1.f - 2.f * (qx * qx + qz * qz);
    Rq[5] = 2.f * (qy * qz - qw * qx);
    Rq[6] = 2.f * (qx * qz - qw * qy);
    Rq[7] = 2.f * (qy * qz + qw * qx);
    Rq[8] = 1.f - 2.f * (qx * qx + qy * qy);
    const float s0 = __expf(gp.log_scale[g]), s1 = __expf(gp.log_scale[M + g]), s2 = __expf(gp.log_scale[2 * M + g]);
    float Mm[9];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        Mm[3 * r + 0] = Rq[3 * r + 0] * s0;
        Mm[3 * r + 1] = Rq[3 * r + 1] * s1;
        Mm[3 * r + 2] = Rq[3 * r + 2] * s2;
    }
    // W = J R (2x3)
    const float iz = 1.0f / z;
    const float J00 = c.fx * iz, J02 = -c.fx * x * iz * iz, J11 = c.fy * iz, J12 = -c.fy * y * iz * iz;
    float W0[3], W1[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        W0[k] = J00 * c.R[k] + J02 * c.R[6 + k];
        W1[k] = J11 * c.R[3 + k] + J12 * c.R[6 + k];
    }
    // U = W Mm (2x3); Sigma_2D = U U^T
    float U0[3], U1[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        U0[k] = W0[0] * Mm[k] + W0[1] * Mm[3 + k] + W0[2] * Mm[6 + k];
        U1[k] = W1[0] * Mm[k] + W1[1] * Mm[3 + k] + W1[2] * Mm[6 + k];
    }
    const float A = U0[0] * U0[0] + U0[1] * U0[1] + U0[2] * U0[2] + rp.dil;
    const float B = U0[0] * U1[0] + U0[1] * U1[1] + U0[2] * U1[2];
    const float C = U1[0] * U1[0] + U1[1] * U1[1] + U1[2] * U1[2] + rp.dil;
    const float det = A * C - B * B;
    if (!(det > 0.0f)) return o;
    const float idet = 1.0f / det;
    const float sig = 1.0f / (1.0f + __expf(-gp.opacity_logit[g]));
    if (!(sig > rp.amin)) return o;
    const float mx = c.fx * x * iz + c.cx, my = c.fy * y * iz + c.cy;
    const float kappa = 2.0f * __logf(sig / rp.amin);
    // support half-extents padded by one pixel (covers the rounding of the opacity test)
    const float rxp = sqrtf(kappa * A) + 1.0f, ryp = sqrtf(kappa * C) + 1.0f;
    if (!(rxp < 1e7f) || !(ryp < 1e7f) || !(fabsf(mx) < 1e7f) || !(fabsf(my) < 1e7f)) return o;
    // conic (a, b, c) = (C, -B, A) / det, pre-scaled for the base-2 exponential
    constexpr float kL2E = 1.4426950408889634f;
    o.r0 = make_float4(mx, my, (-0.5f * kL2E) * (C * idet), kL2E * (B * idet));
    float col[3];
    view_colour<SH>(gp, M, g, c, m0, m1, m2, col);
    o.r1 = make_float4((-0.5f * kL2E) * (A * idet), __log2f(sig), z, col[0]);
    o.r2 = make_float4(col[1], col[2], rxp, ryp);
    o.valid = true;
    return o;
}

// ------------------------------------------------- walk of the tile rectangles
// A wavefront takes PER Gaussians of one view (a lane each) and its lanes then walk the
// concatenation of their tile rectangles together, 64 slots at a time, so a large
// Gaussian, or a run of dense ones, is spread over lanes instead of serialising one.
// The Gaussians that are seen stand in LDS without gaps; the slots at which they start
// are set in a 64-bit word per window, and the owner of a slot is the number of starts
// up to it.  Slots are numbered per wavefront in walking order from seg_off.
template <int PER>
struct WaveWalk {
    unsigned long long starts;
    uint4 c[PER];  // depth bits, first slot, first tile (x | y << 16), width | lane << 16 | big << 31
};

template <int PER>
struct CountWalk : WaveWalk<PER> {
    float4 a[PER];  // mx, my, A, B of the support test
    float4 b[PER];  // C, kx, ky, need
};

template <int PER>
struct EmitWalk : WaveWalk<PER> {
    unsigned int kept[PER];
};

// LDS words of one wavefront, written and read by its own lanes: order without a barrier.
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inclusive sum over the lanes before and at this one.
__device__ __forceinline__ unsigned int wave_incl_sum(unsigned int x)
{
    x += (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);
    x += (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);
    x += (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);
    x += (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);  // row_bcast:15
    x += (unsigned int)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return x;
}

__device__ __forceinline__ unsigned int lanes_before(unsigned long long m)
{
    return __builtin_amdgcn_mbcnt_hi((unsigned int)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned int)m, 0u));
}

// The Gaussian of a lane in iteration i of a wavefront's share (M: none).
template <int PER>
__device__ __forceinline__ int share_gaussian(const BinShape& bs, int chunk, int wid, int lane, int i, int M)
{
    if (lane >= PER) return M;
    const unsigned int per = (unsigned int)(PER / bs.run);  // runs a wavefront takes at a time
    const unsigned long long waves = (unsigned long long)bs.chunks * bs.waves;
    const unsigned long long r = ((unsigned long long)i * per + (unsigned int)(lane / bs.run)) * waves +
                                 (unsigned int)(chunk * bs.waves + wid);
    const unsigned long long g = r * bs.run + (unsigned int)(lane % bs.run);
    return g < (unsigned long long)M ? (int)g : M;
}

// The slots of the window [w0, w0 + 64) of a walk: for this lane's slot its owner in the
// wavefront's list.  n: this lane's slots (0: its Gaussian is not seen), excl: its first;
// before: seen Gaussians that start before the window (advanced by those that start in it).
template <int PER>
__device__ __forceinline__ unsigned int walk_owner(WaveWalk<PER>& ww, unsigned int n, unsigned int excl, unsigned int w0,
                                                   unsigned int& before)
{
    const int lane = threadIdx.x & 63;
    wave_lds_order();
    if (lane == 0) ww.starts = 0ull;
    wave_lds_order();
    if (n > 0u && excl - w0 < 64u) atomicOr(&ww.starts, 1ull << (excl - w0));
    wave_lds_order();
    const unsigned long long st = ww.starts;
    const unsigned int lo = (unsigned int)__builtin_amdgcn_readfirstlane((int)(unsigned int)st);
    const unsigned int hi = (unsigned int)__builtin_amdgcn_readfirstlane((int)(unsigned int)(st >> 32));
    const unsigned long long s = ((unsigned long long)hi << 32) | lo;
    const unsigned int owner = before + lanes_before(s) + (unsigned int)((s >> lane) & 1ull) - 1u;
    before += (unsigned int)__builtin_popcountll(s);
    return owner;
}

// Row and column of slot j in a rectangle `width` tiles wide.  Below 2^21 slots (always with
// counters in LDS: a view then has at most kBinTiles tiles) the product with the reciprocal is
// off by less than j 2^-22 / width < 0.5 / width, so the truncation is exact.
template <bool LDS>
__device__ __forceinline__ unsigned int slot_row(unsigned int j, unsigned int width)
{
    static_assert(kBinTiles <= (1 << 20), "slot numbers are exact in the reciprocal form");
    if (LDS) return (unsigned int)(((float)j + 0.5f) * __builtin_amdgcn_rcpf((float)width));
    return j / width;
}

// One slot of the walk: its tile, and whether the instance passes the culls: the support
// ellipse meets the tile (its box may only overlap it), and the exact tile-level depth cull.
struct Slot {
    unsigned int j, tile;  // in the rectangle, in the view
    bool small;            // of a Gaussian whose culls are kept as bits
};

template <bool LDS>
__device__ __forceinline__ Slot slot_of(const uint4& c, unsigned int i, int tiles_x, int* tx, int* ty)
{
    Slot s;
    s.j = i - c.y;
    const unsigned int width = c.w & 0xffffu, q = slot_row<LDS>(s.j, width);
    *tx = (int)((c.z & 0xffffu) + (s.j - q * width));
    *ty = (int)((c.z >> 16) + q);
    s.tile = (unsigned int)(*ty * tiles_x + *tx);
    s.small = (int)c.w >= 0;
    return s;
}

__device__ __forceinline__ bool slot_passes(const SupportTest& st, float z, int tx, int ty, float tile_max,
                                            const RParams& rp)
{
    return st.meets((float)(tx * rp.tile_w), (float)(ty * rp.tile_h), (float)rp.tile_w, (float)rp.tile_h) &&
           z < tile_max + rp.eps;
}

// Projection of Gaussian g, and what is kept of it: its record, first tile, depth and the tiles of its
// rectangle (span, also of one that is not seen).  Returns its slots: one per covered tile.
template <bool SH>
__device__ __forceinline__ unsigned int project_store(const DevView& V, const RParams& rp, const GParams& gp, const WsPtrs& w,
                                                      int g, size_t vg, ProjOut& p, unsigned int& t0, unsigned int& span)
{
    unsigned int n = 0u;
    p = project_one<SH>(V, rp, gp, g);
    TileRect r;
    if (p.valid && rect_of(p.r0.x, p.r0.y, p.r2.z, p.r2.w, V.cam.W, V.cam.H, rp.tile_w, rp.tile_h, &r)) {
        const unsigned int width = (unsigned int)(r.tx1 - r.tx0 + 1), height = (unsigned int)(r.ty1 - r.ty0 + 1);
        n = width * height;
        span = width | height << 16;
        t0 = (unsigned int)r.tx0 | (unsigned int)r.ty0 << 16;
        w.rec[3 * vg + 0] = p.r0;
        w.rec[3 * vg + 1] = p.r1;
        w.rec[3 * vg + 2] = p.r2;
        w.off[vg] = t0;
        w.depth[vg] = p.r1.z;
    }
    w.span[vg] = span;
    return n;
}

// ---------------------------------------------------------------- project
// Projection of a share of one view's Gaussians (see binning.h), the number of slots of
// each (tiles of its rectangle), and the walk that counts the instances per tile: those that
// pass the culls, kept as a bit per slot for the emission and the backward.  Bound by latency
// for few Gaussians (100 k at 1280x720: 9 us, with a pass of its own for the counts 6 + 5 + 11) and by
// the walk's instructions for many (4 x 1 M: 87 us against 68 + 11 + 370).
template <int WAVES, int PER, bool LDS, bool SH>
__global__ void __launch_bounds__(64 * WAVES, 4) k_project(const ViewTable* __restrict__ vtp, RParams rp, BinShape bs,
                                                     GParams gp, WsPtrs w)
{
    extern __shared__ unsigned int counter[];  // LDS: per tile of the view
    __shared__ CountWalk<PER> walk[WAVES];
    const ViewTable& vt = *vtp;
    const int v = blockIdx.x / bs.chunks, chunk = blockIdx.x - v * bs.chunks;
    const DevView& V = vt.v[v];
    const int n_tiles = V.tiles_x * V.tiles_y, lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    unsigned int* row = w.tile_rows + (size_t)bs.rows * V.tile_base + (size_t)(LDS ? chunk : chunk % bs.rows) * n_tiles;
    CountWalk<PER>& ww = walk[wid];
    const float l2amin = __log2f(rp.amin);
    if (LDS) {
        for (int t = threadIdx.x; t < n_tiles; t += 64 * WAVES) counter[t] = 0u;
        __syncthreads();
    }
    unsigned long long slots = 0ull;
    for (int i = 0; i < bs.iters; ++i) {
        const int g = share_gaussian<PER>(bs, chunk, wid, lane, i, rp.M);
        const size_t vg = (size_t)v * rp.M + g;
        unsigned int n = 0u, t0 = 0u, span = 0u, kept = 0u;
        ProjOut p;
        if (g < rp.M) {
            n = project_store<SH>(V, rp, gp, w, g, vg, p, t0, span);
        }
        const unsigned int excl = wave_incl_sum(n) - n;
        const unsigned int total = (unsigned int)__builtin_amdgcn_readlane((int)(excl + n), 63);
        slots += total;
        if (slots > rp.cap) continue;  // over the capacity: nothing of this forward is used
        const unsigned long long seen = __builtin_amdgcn_ballot_w64(n > 0u);
        const unsigned int at = lanes_before(seen);
        wave_lds_order();
        if (n > 0u) {
            const SupportTest st(p.r0, p.r1, l2amin);  // made once for all slots
            ww.a[at] = make_float4(st.mx, st.my, st.A, st.B);
            ww.b[at] = make_float4(st.C, st.kx, st.ky, st.need);
            ww.c[at] = make_uint4(__float_as_uint(p.r1.z), excl, t0, span & 0xffffu);
        }
        unsigned int before = 0u;
        for (unsigned int w0 = 0u; w0 < total; w0 += 64u) {
            const unsigned int owner = walk_owner(ww, n, excl, w0, before);
            bool pass = false;
            if (w0 + lane < total) {
                const uint4 c = ww.c[owner];
                int tx, ty;
                const Slot s = slot_of<LDS>(c, w0 + lane, V.tiles_x, &tx, &ty);
                const float tile_max = w.tilemax[V.tile_base + s.tile];
                pass = slot_passes(SupportTest(ww.a[owner], ww.b[owner]), __uint_as_float(c.x), tx, ty, tile_max, rp);
                if (pass) atomicAdd(LDS ? &counter[s.tile] : row + s.tile, 1u);
            }
            // this lane's Gaussian takes the bits of its slots in the window
            const unsigned long long passed = __builtin_amdgcn_ballot_w64(pass);
            const unsigned int all = 0xffffffffu >> (kKeptBits - min(n, (unsigned int)kKeptBits) & 31u);
            const int lo = (int)(excl - w0);
            if (lo >= 0 && lo < 64) kept |= (unsigned int)(passed >> lo) & all;
            else if (lo < 0 && lo > -kKeptBits) kept |= (unsigned int)(passed << -lo) & all;
        }
        if (n > 0u) w.kept[vg] = kept;
    }
    if (lane == 0) w.seg_sum[blockIdx.x * WAVES + wid] = (unsigned int)min(slots, 0xffffffffull);
    if (LDS) {
        __syncthreads();
        for (int t = threadIdx.x; t < n_tiles; t += 64 * WAVES) row[t] = counter[t];
    }
}

// The shared rows of tile counts start at zero.
__global__ void __launch_bounds__(kBlk) k_zero_rows(WsPtrs w, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * kBlk + threadIdx.x; i < n; i += (size_t)gridDim.x * kBlk) w.tile_rows[i] = 0u;
}

// ------------------------------------------------------------------- scan
// Per tile: the rows of counts become the first place of each row inside the tile's range,
// and the tile's instances their sum.  kScanCols tiles per block, the rows in as many
// groups of consecutive ones as lanes are left; a lane has its rows in flight together.
constexpr int kScanCols = 16, kScanGroups = kBlk / kScanCols, kScanRows = 32;

// The slots of the projection's wavefronts: their first, and the total against the capacity.
// One block of NT.  The total may pass 32 bits (it is then over the capacity and no place is used).
template <int NT>
__device__ void scan_segments(const RParams& rp, const BinShape& bs, const WsPtrs& w, int n_tiles)
{
    constexpr int kPer = 16;
    __shared__ unsigned long long wsum[NT / 64];
    const int n = rp.V * bs.chunks * bs.waves, lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    unsigned long long carry = 0ull;
    for (int base = 0; base < n; base += NT * kPer) {
        struct alignas(16) Segs {
            unsigned int n[kPer];
        } cv{};
        unsigned int (&c)[kPer] = cv.n;
        unsigned long long sum = 0ull;
        const int t0 = base + threadIdx.x * kPer;
        if (t0 < n) cv = *reinterpret_cast<const Segs*>(w.seg_sum + t0);  // (the array is longer than kMostSegs rounded up)
#pragma unroll
        for (int i = 0; i < kPer; ++i) c[i] = t0 + i < n ? c[i] : 0u;
#pragma unroll
        for (int i = 0; i < kPer; ++i) sum += c[i];
        unsigned long long x = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[wid] = x;
        __syncthreads();
        unsigned long long before = carry;
#pragma unroll
        for (int k = 0; k < NT / 64; ++k) {
            if (k < wid) before += wsum[k];
            carry += wsum[k];
        }
        unsigned int run = (unsigned int)(before + x - sum);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const unsigned int s = c[i];
            c[i] = run;
            run += s;
        }
        if (t0 < n) *reinterpret_cast<Segs*>(w.seg_off + t0) = cv;
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        w.hdr->n_inst = carry;
        w.hdr->cap = rp.cap;
        w.hdr->n_tiles = n_tiles;
        w.hdr->n_views = rp.V;
        w.hdr->n_fallback = 0ull;
        if (carry > rp.cap) atomicCAS(&w.hdr->status, 0, GPS_ERR_CAPACITY);
    }
}

// Block 0 scans the segments, the others the rows of kScanCols tiles each.
__global__ void __launch_bounds__(kBlk) k_scan_rows(const ViewTable* __restrict__ vtp, RParams rp, BinShape bs, WsPtrs w)
{
    const ViewTable& vt = *vtp;
    if (blockIdx.x == 0) {
        scan_segments<kBlk>(rp, bs, w, vt.n_tiles);
        return;
    }
    __shared__ unsigned int sum[kScanGroups][kScanCols + 1];
    const int col = threadIdx.x % kScanCols, grp = threadIdx.x / kScanCols;
    const int tile = (blockIdx.x - 1) * kScanCols + col;
    const bool live = tile < vt.n_tiles;
    const int v = find_view(vt, live ? tile : 0);
    const DevView& V = vt.v[v];
    const size_t n_tiles = (size_t)V.tiles_x * V.tiles_y;
    unsigned int* p = w.tile_rows + (size_t)bs.rows * V.tile_base + (live ? tile - V.tile_base : 0);
    const int per = (bs.rows + kScanGroups - 1) / kScanGroups;
    const int r0 = min(grp * per, bs.rows), r1 = live ? min(r0 + per, bs.rows) : r0;
    unsigned int c[kScanRows], s = 0u;
    for (int r = r0; r < r1; r += kScanRows) {
#pragma unroll
        for (int k = 0; k < kScanRows; ++k) c[k] = r + k < r1 ? p[(size_t)(r + k) * n_tiles] : 0u;
#pragma unroll
        for (int k = 0; k < kScanRows; ++k) s += c[k];
    }
    sum[grp][col] = s;
    __syncthreads();
    unsigned int run = 0u;
    for (int k = 0; k < grp; ++k) run += sum[k][col];
    if (live && grp == kScanGroups - 1) w.tile_cnt[tile] = run + s;
    for (int r = r0; r < r1; r += kScanRows) {
        if (per > kScanRows) {  // not all in registers
#pragma unroll
            for (int k = 0; k < kScanRows; ++k) c[k] = r + k < r1 ? p[(size_t)(r + k) * n_tiles] : 0u;
        }
#pragma unroll
        for (int k = 0; k < kScanRows; ++k) {
            if (r + k < r1) p[(size_t)(r + k) * n_tiles] = run;
            run += c[k];
        }
    }
}

// Position of this lane in its bucket's list: the lanes of one bucket go to the next places of
// cur[bucket] together (one LDS atomic per bucket and wavefront: with one per lane,
// a few buckets hold all tiles and the atomics queue).  Returns the place.
__device__ __forceinline__ unsigned int bucket_add(unsigned int* cur, bool has, int bucket)
{
    const int lane = threadIdx.x & 63;
    unsigned int place = 0u;
    unsigned long long left = __builtin_amdgcn_ballot_w64(has);
    while (left) {
        const int lead = (int)__builtin_ctzll(left);
        const int b = __builtin_amdgcn_readlane(bucket, lead);
        const unsigned long long same = __builtin_amdgcn_ballot_w64(has && bucket == b);
        unsigned int base = 0u;
        if (lane == lead) base = atomicAdd(&cur[b], (unsigned int)__builtin_popcountll(same));
        base = (unsigned int)__builtin_amdgcn_readlane((int)base, lead);
        if (has && bucket == b) place = base + lanes_before(same);
        left &= ~same;
    }
    return place;
}

// One block: the tile ranges, and the tiles in order for the compositing kernels, longest
// first: tiles are bucketed by floor(log2(count + 1)) and the buckets laid out in descending
// order.  The order inside a bucket is arbitrary; it affects only which block processes a
// tile, never a result.  A lane has PER consecutive tiles; with more than 1024 PER tiles the
// block takes them in passes and leaves a tile's place in its bucket in tile_cnt between.
// A lane's tiles are placed one after the other, so it gets as few as one pass allows: with 2, 4 and
// 8 a lane 2160 tiles take 10.1, 9.4 and 14.0 us (with events around), 2539 take 11.4, 11.3 and 16.7, 4000
// 11.8, 9.8 and 14.3, 4520 13.0, 13.0 and 10.7, 7360 19, 19 and 15.
constexpr int kLongBucket = 9;
static_assert(kLongTile == (1u << kLongBucket) - 1u, "the long tiles are whole buckets");

template <int PER>
__device__ __forceinline__ void scan_tiles(const RParams& rp, const WsPtrs& w, int n_tiles)
{
    __shared__ unsigned int wsum[16], hist[33];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    // A lane's tiles are one aligned vector (the arrays are padded to 256 bytes): on one CU the
    // accesses count, and eight of 4 bytes a lane took 18 us over 7360 tiles, this 12.
    struct alignas(PER >= 4 ? 16 : 4 * PER) Tiles {
        unsigned int n[PER];
    };
    Tiles* const cnt = reinterpret_cast<Tiles*>(w.tile_cnt);
    Tiles* const start = reinterpret_cast<Tiles*>(w.tile_start);
    Tiles c, place, begin;
    auto load = [&](int t0) {
        if (t0 < n_tiles) c = cnt[t0 / PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) c.n[i] = t0 + i < n_tiles ? c.n[i] : 0u;
    };
    const unsigned long long n_inst = w.hdr->n_inst;
    load(threadIdx.x * PER);
    if (threadIdx.x < 33) hist[threadIdx.x] = 0u;
    if (n_inst > rp.cap) return;  // below, every sum fits 32 bits
    const bool passes = n_tiles > 1024 * PER;
    unsigned int carry = 0u;
    for (int base = 0; base < n_tiles; base += 1024 * PER) {
        const int t0 = base + threadIdx.x * PER;
        unsigned int s = 0u;
        if (base > 0) load(t0);
#pragma unroll
        for (int i = 0; i < PER; ++i) s += c.n[i];
        const unsigned int x = wave_incl_sum(s);
        __syncthreads();  // hist and wsum are free
        if (lane == 63) wsum[wid] = x;
#pragma unroll
        for (int i = 0; i < PER; ++i) place.n[i] = bucket_add(hist, t0 + i < n_tiles, 31 - __clz(c.n[i] + 1u));
        __syncthreads();
        const unsigned int ws = lane < 16 ? wsum[lane] : 0u;
        const unsigned int wx = wave_incl_sum(ws);  // lane k: sum over wavefronts 0 .. k
        const unsigned int before = wid == 0 ? 0u : (unsigned int)__builtin_amdgcn_readlane((int)wx, wid - 1);
        unsigned int run = carry + before + x - s;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            begin.n[i] = run;
            run += c.n[i];
        }
        if (t0 < n_tiles) {
            start[t0 / PER] = begin;  // (the entry behind the last tile is the end of its range)
            if (passes) cnt[t0 / PER] = place;
        }
        carry += (unsigned int)__builtin_amdgcn_readlane((int)wx, 15);
    }
    // bucket b starts after all longer ones: lane k has the start of bucket 32 - k
    const unsigned int h = lane < 33 ? hist[32 - lane] : 0u;
    const unsigned int first = wave_incl_sum(h) - h;
    const int n_long = __builtin_amdgcn_readlane((int)first, 32 - (kLongBucket - 1));
    if (threadIdx.x == 0) {
        w.tile_start[n_tiles] = carry;
        w.hdr->n_large = (unsigned int)n_long;
    }
    if (!passes) {
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int t = threadIdx.x * PER + i;
            const unsigned int st = (unsigned int)__shfl((int)first, 32 - (31 - __clz(c.n[i] + 1u)), 64);
            if (t < n_tiles) w.tile_queue[st + place.n[i]] = (unsigned int)t;
        }
        return;
    }
    __syncthreads();  // tile_start and tile_cnt of the block's lanes
    for (int base = 0; base < n_tiles; base += 1024) {
        const int t = base + threadIdx.x;
        const unsigned int n = t < n_tiles ? w.tile_start[t + 1] - w.tile_start[t] : 0u;
        const unsigned int st = (unsigned int)__shfl((int)first, 32 - (31 - __clz(n + 1u)), 64);
        if (t < n_tiles) w.tile_queue[st + w.tile_cnt[t]] = (unsigned int)t;
    }
}

template <int PER>
__global__ void __launch_bounds__(1024) k_scan_tiles(RParams rp, WsPtrs w, int n_tiles)
{
    scan_tiles<PER>(rp, w, n_tiles);
}

// Few rows and tiles (kSmallRows, kSmallTiles: up to 4096 Gaussians a view) are scanned by one block
// in one launch: a 160x120 view's 80 tiles take 6.2 us, in two launches 4.0 + 3.6
// and the gap between them; the iteration 65.7 -> 61.4 us.
constexpr int kSmallRows = 16, kSmallTiles = 2048;

__global__ void __launch_bounds__(1024) k_scan_small(const ViewTable* __restrict__ vtp, RParams rp, BinShape bs, WsPtrs w,
                                                    int n_tiles)
{
    const ViewTable& vt = *vtp;
    for (int t = threadIdx.x; t < n_tiles; t += 1024) {
        const DevView& V = vt.v[find_view(vt, t)];
        const size_t n = (size_t)V.tiles_x * V.tiles_y;
        unsigned int* p = w.tile_rows + (size_t)bs.rows * V.tile_base + (t - V.tile_base);
        unsigned int c[kSmallRows], run = 0u;
#pragma unroll
        for (int r = 0; r < kSmallRows; ++r) c[r] = r < bs.rows ? p[r * n] : 0u;
#pragma unroll
        for (int r = 0; r < kSmallRows; ++r) {
            if (r < bs.rows) p[r * n] = run;
            run += c[r];
        }
        w.tile_cnt[t] = run;
    }
    scan_segments<1024>(rp, bs, w, n_tiles);
    __syncthreads();
    scan_tiles<2>(rp, w, n_tiles);
}

// ------------------------------------------------------------------- emit
// The same walk: every instance that passed writes the key (depth bits << 32) |
// view-Gaussian at the next place of its tile in its block's part of the range, and the
// view-Gaussian its first slot.  A tile holds at most one instance of a view-Gaussian, and
// slots grow with the view-Gaussian index inside a wavefront's share, so the keys' order does
// not depend on places; the backward finds the slot from the view-Gaussian's first and the
// tile's place in its rectangle.  The backward reads the slots of a Gaussian by its bits; one
// with more slots than bits is tested again here and the partials of its
// other slots zeroed.  Bound by the scattered 8-byte stores for many instances (8.5 M: 126 us; with every
// slot's partial zeroed and the culls repeated 275).
template <int WAVES, int PER, bool LDS>
__global__ void __launch_bounds__(64 * WAVES, 4) k_emit(const ViewTable* __restrict__ vtp, RParams rp, BinShape bs, WsPtrs w)
{
    extern __shared__ unsigned int counter[];  // LDS: next place per tile of the view
    __shared__ EmitWalk<PER> walk[WAVES];
    const ViewTable& vt = *vtp;
    const int v = blockIdx.x / bs.chunks, chunk = blockIdx.x - v * bs.chunks;
    const DevView& V = vt.v[v];
    const int n_tiles = V.tiles_x * V.tiles_y, lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    unsigned int* row = w.tile_rows + (size_t)bs.rows * V.tile_base + (size_t)(LDS ? chunk : chunk % bs.rows) * n_tiles;
    const unsigned int* start = w.tile_start + V.tile_base;
    EmitWalk<PER>& ww = walk[wid];
    // A Gaussian's loads are issued an iteration ahead.
    unsigned int span = 0u, t0 = 0u, kept = 0u, span1 = 0u, t01 = 0u, kept1 = 0u;
    float z = 0.0f, z1 = 0.0f;
    auto load = [&](int i) {
        const int g = i < bs.iters ? share_gaussian<PER>(bs, chunk, wid, lane, i, rp.M) : rp.M;
        span1 = 0u;
        if (g < rp.M) {
            const size_t vg = (size_t)v * rp.M + g;
            span1 = w.span[vg];
            t01 = w.off[vg];
            kept1 = w.kept[vg];
            z1 = w.depth[vg];
        }
    };
    load(0);
    unsigned int base = w.seg_off[blockIdx.x * WAVES + wid];
    if (w.hdr->n_inst > rp.cap) return;
    if (LDS) {
        for (int t = threadIdx.x; t < n_tiles; t += 64 * WAVES) counter[t] = start[t] + row[t];
        __syncthreads();
    }
    const float l2amin = __log2f(rp.amin);
    for (int i = 0; i < bs.iters; ++i) {
        const size_t vg = (size_t)v * rp.M + share_gaussian<PER>(bs, chunk, wid, lane, i, rp.M);
        span = span1;
        t0 = t01;
        kept = kept1;
        z = z1;
        load(i + 1);
        const unsigned int n = (span & 0xffffu) * (span >> 16);
        const unsigned int excl = wave_incl_sum(n) - n;
        const unsigned int total = (unsigned int)__builtin_amdgcn_readlane((int)(excl + n), 63);
        const unsigned long long seen = __builtin_amdgcn_ballot_w64(n > 0u);
        const unsigned int at = lanes_before(seen);
        const bool big = n > (unsigned int)kKeptBits;
        wave_lds_order();
        if (n > 0u) {
            w.off[vg] = base + excl;
            ww.c[at] = make_uint4(__float_as_uint(z), excl, t0, (span & 0xffffu) | (unsigned int)lane << 16 | (big ? 0x80000000u : 0u));
            ww.kept[at] = kept;
        }
        unsigned int before = 0u;
        for (unsigned int w0 = 0u; w0 < total; w0 += 64u) {
            const unsigned int owner = walk_owner(ww, n, excl, w0, before);
            if (w0 + lane < total) {
                const uint4 c = ww.c[owner];
                int tx, ty;
                const Slot s = slot_of<LDS>(c, w0 + lane, V.tiles_x, &tx, &ty);
                const int owner_g = share_gaussian<PER>(bs, chunk, wid, (c.w >> 16) & 63, i, rp.M);
                bool pass;
                if (s.small) {
                    pass = (ww.kept[owner] >> s.j) & 1u;
                } else {
                    const float4* r = w.rec + 3 * ((size_t)v * rp.M + owner_g);
                    pass = slot_passes(SupportTest(r[0], r[1], l2amin), __uint_as_float(c.x), tx, ty,
                                       w.tilemax[V.tile_base + s.tile], rp);
                    if (!pass) {
                        float* pz = w.partial + (size_t)(base + w0 + lane) * kAdj;
#pragma unroll
                        for (int q = 0; q < kAdj; ++q) pz[q] = 0.0f;
                    }
                }
                if (pass) {
                    const unsigned int pos = LDS ? atomicAdd(&counter[s.tile], 1u) : start[s.tile] + atomicAdd(row + s.tile, 1u);
                    // key: depth bits, then the view-Gaussian
                    if (pos < rp.cap)
                        w.keys[pos] = ((unsigned long long)c.x << 32) | (unsigned int)(v * rp.M + owner_g);
                }
            }
        }
        base += total;
    }
}

// ------------------------------------------------------- lists without a sort
// Projection and emission where no sort follows (see kOrderGroup): a block takes groups of 64 consecutive
// view-Gaussians, numbered over the views, its first wavefront a lane each, and all its lanes then walk the
// concatenation of their tile rectangles, 256 slots at a time; group k adds to shared row k mod
// kCntSplit, which is its part of a tile's range.
struct GroupWalk {
    uint4 c[kOrderGroup];  // as in WaveWalk
    unsigned int kept[kOrderGroup];
    unsigned int seen, total;
};

// The view-Gaussian of a lane of the block's i-th group in its view (M: none).
__device__ __forceinline__ int group_gaussian(const BinShape& bs, int v, int chunk, int lane, int i, int M)
{
    const unsigned int g = ((unsigned int)i * bs.chunks + chunk) * kOrderGroup + lane;
    const unsigned int skew = (unsigned int)(v * M) % kOrderGroup;  // of the view's first group, those of the view before
    return g >= skew && g - skew < (unsigned int)M ? (int)(g - skew) : M;
}

__device__ __forceinline__ unsigned int* group_row(const BinShape& bs, const DevView& V, const WsPtrs& w, int v, int chunk, int M)
{
    const int part = (chunk + v * M / kOrderGroup) % kCntSplit;  // (chunks is a multiple of kCntSplit)
    return w.tile_rows + (size_t)kCntSplit * V.tile_base + (size_t)part * V.tiles_x * V.tiles_y;
}

// The Gaussian in the block's list that slot i belongs to: the last that starts at or before it.
__device__ __forceinline__ unsigned int group_owner(const GroupWalk& gw, unsigned int i)
{
    unsigned int lo = 0u, hi = gw.seen;
#pragma unroll
    for (int step = 0; step < 6; ++step) {
        const unsigned int mid = (lo + hi) >> 1;
        if (gw.c[mid].y <= i) lo = mid;
        else hi = mid;
    }
    return lo;
}

template <bool SH>
__global__ void __launch_bounds__(kBlk) k_project_groups(const ViewTable* __restrict__ vtp, RParams rp, BinShape bs,
                                                         GParams gp, WsPtrs w)
{
    __shared__ GroupWalk gw;
    __shared__ float4 sa[kOrderGroup], sb[kOrderGroup];  // the support tests, as in CountWalk
    const ViewTable& vt = *vtp;
    const int v = blockIdx.x / bs.chunks, chunk = blockIdx.x - v * bs.chunks;
    const DevView& V = vt.v[v];
    const int lane = threadIdx.x & 63;
    const bool first = threadIdx.x < 64;
    unsigned int* row = group_row(bs, V, w, v, chunk, rp.M);
    const float l2amin = __log2f(rp.amin);
    unsigned long long slots = 0ull;
    for (int i = 0; i < bs.iters; ++i) {
        unsigned int n = 0u, at = 0u;
        size_t vg = 0;
        if (first) {
            const int g = group_gaussian(bs, v, chunk, lane, i, rp.M);
            vg = (size_t)v * rp.M + g;
            unsigned int t0 = 0u, span = 0u;
            ProjOut p;
            if (g < rp.M) n = project_store<SH>(V, rp, gp, w, g, vg, p, t0, span);
            const unsigned int excl = wave_incl_sum(n) - n;
            const unsigned long long seen = __builtin_amdgcn_ballot_w64(n > 0u);
            at = lanes_before(seen);
            if (n > 0u) {
                const SupportTest st(p.r0, p.r1, l2amin);
                sa[at] = make_float4(st.mx, st.my, st.A, st.B);
                sb[at] = make_float4(st.C, st.kx, st.ky, st.need);
                gw.c[at] = make_uint4(__float_as_uint(p.r1.z), excl, t0,
                                      (span & 0xffffu) | (n > (unsigned int)kKeptBits ? 0x80000000u : 0u));
                gw.kept[at] = 0u;
            }
            if (lane == 63) {
                gw.seen = (unsigned int)__builtin_popcountll(seen);
                gw.total = excl + n;
            }
        }
        __syncthreads();
        const unsigned int total = gw.total;
        slots += total;
        if (slots <= rp.cap) {  // else nothing of this forward is used
            for (unsigned int k = threadIdx.x; k < total; k += kBlk) {
                const unsigned int owner = group_owner(gw, k);
                const uint4 c = gw.c[owner];
                int tx, ty;
                const Slot s = slot_of<false>(c, k, V.tiles_x, &tx, &ty);
                if (slot_passes(SupportTest(sa[owner], sb[owner]), __uint_as_float(c.x), tx, ty,
                                w.tilemax[V.tile_base + s.tile], rp)) {
                    atomicAdd(row + s.tile, 1u);
                    if (s.small) atomicOr(&gw.kept[owner], 1u << s.j);
                }
            }
        }
        __syncthreads();
        if (n > 0u) w.kept[vg] = gw.kept[at];
    }
    if (threadIdx.x == 0) w.seg_sum[blockIdx.x] = (unsigned int)min(slots, 0xffffffffull);
}

__global__ void __launch_bounds__(kBlk) k_emit_groups(const ViewTable* __restrict__ vtp, RParams rp, BinShape bs, WsPtrs w)
{
    __shared__ GroupWalk gw;
    const ViewTable& vt = *vtp;
    const int v = blockIdx.x / bs.chunks, chunk = blockIdx.x - v * bs.chunks;
    const DevView& V = vt.v[v];
    const int lane = threadIdx.x & 63;
    unsigned int* row = group_row(bs, V, w, v, chunk, rp.M);
    const unsigned int* start = w.tile_start + V.tile_base;
    const float l2amin = __log2f(rp.amin);
    unsigned int base = w.seg_off[blockIdx.x];
    const unsigned long long n_inst = w.hdr->n_inst;
    for (int i = 0; i < bs.iters; ++i) {
        if (threadIdx.x < 64) {
            const int g = group_gaussian(bs, v, chunk, lane, i, rp.M);
            const size_t vg = (size_t)v * rp.M + g;
            unsigned int span = 0u, t0 = 0u, kept = 0u;
            float z = 0.0f;
            if (g < rp.M) {
                span = w.span[vg];
                t0 = w.off[vg];
                kept = w.kept[vg];
                z = w.depth[vg];
            }
            if (n_inst > rp.cap) span = 0u;
            const unsigned int n = (span & 0xffffu) * (span >> 16);
            const unsigned int excl = wave_incl_sum(n) - n;
            const unsigned long long seen = __builtin_amdgcn_ballot_w64(n > 0u);
            const unsigned int at = lanes_before(seen);
            if (n > 0u) {
                w.off[vg] = base + excl;
                gw.c[at] = make_uint4(__float_as_uint(z), excl, t0,
                                      (span & 0xffffu) | (unsigned int)lane << 16 | (n > (unsigned int)kKeptBits ? 0x80000000u : 0u));
                gw.kept[at] = kept;
            }
            if (lane == 63) {
                gw.seen = (unsigned int)__builtin_popcountll(seen);
                gw.total = excl + n;
            }
        }
        __syncthreads();
        const unsigned int total = gw.total;
        for (unsigned int k = threadIdx.x; k < total; k += kBlk) {
            const unsigned int owner = group_owner(gw, k);
            const uint4 c = gw.c[owner];
            int tx, ty;
            const Slot s = slot_of<false>(c, k, V.tiles_x, &tx, &ty);
            const size_t vg = (size_t)v * rp.M + group_gaussian(bs, v, chunk, (c.w >> 16) & 63, i, rp.M);
            bool pass = (gw.kept[owner] >> (s.j & 31u)) & 1u;
            if (!s.small) {
                const float4* r = w.rec + 3 * vg;
                pass = slot_passes(SupportTest(r[0], r[1], l2amin), __uint_as_float(c.x), tx, ty, w.tilemax[V.tile_base + s.tile], rp);
                if (!pass) {
                    float* pz = w.partial + (size_t)(base + k) * kAdj;
#pragma unroll
                    for (int q = 0; q < kAdj; ++q) pz[q] = 0.0f;
                }
            }
            if (pass) {
                const unsigned int pos = start[s.tile] + atomicAdd(row + s.tile, 1u);
                if (pos < rp.cap) w.keys[pos] = ((unsigned long long)c.x << 32) | (unsigned int)vg;
            }
        }
        __syncthreads();
        base += total;
    }
}

// -------------------------------------------------------------- tile sort
// Tiles of fewer than kLongTile keys are sorted in registers by the first
// wavefront of their compositing block (wave_sort_tile, binning.h).
// k_tile_sort_large: one block per longer tile (depth buckets in LDS, or the bitonic network);
// tiles longer than kSortCap use the network in global memory.

__device__ __forceinline__ void cas_lds(unsigned long long* sh, int i, int j)
{
    const unsigned long long a = sh[i], b = sh[j];
    if (a > b) {
        sh[i] = b;
        sh[j] = a;
    }
}

// Lists of kLongTile keys and more are sorted by distributing the keys over as many buckets as
// there are keys, following their depths (a piecewise linear map: 256 equal depth intervals,
// each given as many buckets as it holds keys), after which a bucket holds one or two keys
// and each key counts the smaller ones of its bucket.  About 20 LDS accesses a key, against the
// several hundred of a network (66 steps of 2 reads and 2 writes for 2048 keys).  The map is
// monotone in binary32, so the order is that of the keys, which are distinct.
constexpr int kSortThreads = 512;
constexpr int kSortLds = 4096;             // keys that meet in LDS
constexpr unsigned int kBucketMost = 64;  // a fuller bucket (depths that coincide) sends the list to the network
constexpr int kCoarse = 256;
constexpr int kSortWaves = kSortThreads / 64;

struct SortShared {
    unsigned long long mid[kSortLds];      // keys by bucket
    unsigned int fine[kSortLds / 2 + 2];   // 16-bit counts, then starts, of the n buckets
    unsigned int coarse[kCoarse + 1];
    unsigned int red[2][kSortWaves];
    unsigned int cursor[2];
};

// Depth interval of a key: [z0, z0 + kCoarse / scale] cut into kCoarse.
struct DepthMap {
    float z0, scale;
    __device__ float at(unsigned long long k, int& c) const
    {
        const float t = (__uint_as_float((unsigned int)(k >> 32)) - z0) * scale;
        c = min((int)t, kCoarse - 1);
        return t;
    }
};

// The depth map of the block's keys k[0 .. n) (this lane's every kSortThreads-th) and the starts
// of its intervals in sh.coarse.  Barriers around; sh.coarse must be zero.
template <int PER>
__device__ __forceinline__ DepthMap depth_intervals(const unsigned long long (&k)[PER], int n, SortShared& sh)
{
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    unsigned int lo = 0xffffffffu, hi = 0u;  // depth bits (depths are positive: they order as the depths do)
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (tid + j * kSortThreads < n) {
            lo = min(lo, (unsigned int)(k[j] >> 32));
            hi = max(hi, (unsigned int)(k[j] >> 32));
        }
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, (unsigned int)__shfl_xor((int)lo, o, 64));
        hi = max(hi, (unsigned int)__shfl_xor((int)hi, o, 64));
    }
    if (lane == 0) {
        sh.red[0][wid] = lo;
        sh.red[1][wid] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q) {
        lo = min(lo, sh.red[0][q]);
        hi = max(hi, sh.red[1][q]);
    }
    DepthMap map;
    map.z0 = __uint_as_float(lo);
    const float span = __uint_as_float(hi) - map.z0;
    map.scale = span > 0.0f ? (float)kCoarse / span : 0.0f;
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (tid + j * kSortThreads < n) {
            int c;
            map.at(k[j], c);
            atomicAdd(&sh.coarse[c], 1u);
        }
    __syncthreads();
    if (wid == 0) {  // exclusive scan of the 256 interval counts, four to a lane
        unsigned int v[4], sum = 0u;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[q] = sh.coarse[4 * lane + q];
            sum += v[q];
        }
        unsigned int x = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned int y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        unsigned int run = x - sum;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            sh.coarse[4 * lane + q] = run;
            run += v[q];
        }
        if (lane == 63) sh.coarse[kCoarse] = run;
    }
    __syncthreads();
    return map;
}

// Sorts the n in [1, kSortLds] keys at key; false, with the keys untouched, when a bucket is too full.
__device__ __forceinline__ bool sort_tile_buckets(unsigned long long* __restrict__ key, int n, SortShared& sh)
{
    constexpr int kPer = kSortLds / kSortThreads;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    unsigned long long k[kPer];  // this lane's keys
#pragma unroll
    for (int j = 0; j < kPer; ++j) k[j] = tid + j * kSortThreads < n ? key[tid + j * kSortThreads] : ~0ull;
    for (int i = tid; i <= n / 2; i += kSortThreads) sh.fine[i] = 0u;
    if (tid <= kCoarse) sh.coarse[tid] = 0u;
    const DepthMap map = depth_intervals<kPer>(k, n, sh);
    unsigned int br[kPer];  // bucket << 16 | rank of arrival in it
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        if (j * kSortThreads >= n) break;  // uniform
        if (tid + j * kSortThreads < n) {
            int c;
            const float t = map.at(k[j], c);
            const int c0 = (int)sh.coarse[c], m = (int)sh.coarse[c + 1] - c0;
            const unsigned int b = (unsigned int)(c0 + min((int)((t - (float)c) * (float)m), m - 1));
            const unsigned int half = (b & 1u) * 16u;  // two 16-bit counts a word: n is below 2^16
            const unsigned int old = atomicAdd(&sh.fine[b >> 1], 1u << half);
            br[j] = (b << 16) | ((old >> half) & 0xffffu);
        }
    }
    __syncthreads();
    // exclusive scan of the bucket counts: a run of consecutive words to a lane
    const int words = (n + 1) / 2, per = (words + kSortThreads - 1) / kSortThreads;
    unsigned int sum = 0u, most = 0u;
    for (int q = 0; q < per; ++q) {
        const int i = tid * per + q;
        const unsigned int v = i < words ? sh.fine[i] : 0u;
        sum += (v & 0xffffu) + (v >> 16);
        most = max(most, max(v & 0xffffu, v >> 16));
    }
    unsigned int x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) sh.red[0][wid] = x;
    if (__syncthreads_or(most > kBucketMost)) return false;
    unsigned int run = x - sum;
#pragma unroll
    for (int q = 0; q < kSortWaves; ++q)
        if (q < wid) run += sh.red[0][q];
    for (int q = 0; q < per; ++q) {
        const int i = tid * per + q;
        if (i >= words) break;
        const unsigned int v = sh.fine[i], half = run + (v & 0xffffu);
        sh.fine[i] = run | (half << 16);
        run = half + (v >> 16);
    }
    // the start past the last bucket (an odd n's is the unused half of its last word, scanned to n)
    if (tid == 0 && (n & 1) == 0) sh.fine[n / 2] = (unsigned int)n;
    __syncthreads();
    auto start = [&](unsigned int b) { return (sh.fine[b >> 1] >> ((b & 1u) * 16u)) & 0xffffu; };
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        if (j * kSortThreads >= n) break;
        if (tid + j * kSortThreads < n) sh.mid[start(br[j] >> 16) + (br[j] & 0xffffu)] = k[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        if (j * kSortThreads >= n) break;
        if (tid + j * kSortThreads < n) {
            const unsigned int f0 = start(br[j] >> 16), f1 = start((br[j] >> 16) + 1u);
            unsigned int p = f0;
            for (unsigned int q = f0; q < f1; q += 4) {  // four independent reads at a time
                const unsigned long long m0 = sh.mid[q], m1 = sh.mid[min(q + 1u, f1 - 1u)],
                                         m2 = sh.mid[min(q + 2u, f1 - 1u)], m3 = sh.mid[min(q + 3u, f1 - 1u)];
                p += (m0 < k[j] ? 1u : 0u) + (q + 1u < f1 && m1 < k[j] ? 1u : 0u) +
                     (q + 2u < f1 && m2 < k[j] ? 1u : 0u) + (q + 3u < f1 && m3 < k[j] ? 1u : 0u);
            }
            key[p] = k[j];
        }
    }
    return true;
}

// Splits kSortLds < n <= kSortCap keys in place, at the end of a depth interval, into two lists of at
// most kSortLds; the length of the first, or 0 (keys untouched) when no interval ends there.
__device__ __forceinline__ int split_tile(unsigned long long* __restrict__ key, int n, SortShared& sh)
{
    constexpr int kPer = kSortCap / kSortThreads;
    const int tid = threadIdx.x;
    unsigned long long k[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) k[j] = tid + j * kSortThreads < n ? key[tid + j * kSortThreads] : ~0ull;
    if (tid <= kCoarse) sh.coarse[tid] = 0u;
    if (tid < 2) sh.cursor[tid] = 0u;
    const DepthMap map = depth_intervals<kPer>(k, n, sh);
    // the interval starts ascend: the last one at most kSortLds opens the second list
    int lo = 0, hi = kCoarse;
    while (lo < hi) {
        const int m = (lo + hi + 1) >> 1;
        if (sh.coarse[m] <= (unsigned int)kSortLds) lo = m;
        else hi = m - 1;
    }
    const int first = (int)sh.coarse[lo];
    if (n - first > kSortLds || first == 0) return 0;  // uniform
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        if (tid + j * kSortThreads < n) {
            int c;
            map.at(k[j], c);
            const unsigned int side = c < lo ? 0u : 1u;
            key[(side ? (unsigned int)first : 0u) + atomicAdd(&sh.cursor[side], 1u)] = k[j];
        }
    __syncthreads();
    return first;
}

// Network of the lists that the buckets refuse or that are longer than kSortCap (one block).
__device__ void sort_tile_network(const WsPtrs& w, unsigned long long* key, int n, SortShared& shared)
{
    int P = 1;
    while (P < n) P <<= 1;
    unsigned long long* sh = shared.mid;
    if (n <= kSortLds) {
        for (int i = threadIdx.x; i < P; i += kSortThreads) sh[i] = i < n ? key[i] : ~0ull;
        __syncthreads();
        for (int k = 2; k <= P; k <<= 1) {
            const int half = k >> 1;
            for (int c = threadIdx.x; c < P / 2; c += kSortThreads) {
                const int blk = c / half, wi = c - blk * half;
                cas_lds(sh, blk * k + wi, blk * k + k - 1 - wi);
            }
            __syncthreads();
            for (int jj = k >> 2; jj > 0; jj >>= 1) {
                for (int c = threadIdx.x; c < P / 2; c += kSortThreads) {
                    const int i = (c / jj) * 2 * jj + (c % jj);
                    cas_lds(sh, i, i + jj);
                }
                __syncthreads();
            }
        }
        for (int i = threadIdx.x; i < n; i += kSortThreads) key[i] = sh[i];
    } else {
        // Rare: a tile of more than kSortCap keys (counted), or one whose depths coincide and that
        // the LDS does not hold.  Same network in global memory; elements at or past n
        // act as +inf and are never touched.
        if (threadIdx.x == 0 && n > kSortCap) atomicAdd(&w.hdr->n_fallback, 1ull);
        for (int k = 2; k <= P; k <<= 1) {
            const int half = k >> 1;
            for (int c = threadIdx.x; c < P / 2; c += kSortThreads) {
                const int blk = c / half, wi = c - blk * half;
                const int i = blk * k + wi, j = blk * k + k - 1 - wi;
                if (j < n) {
                    unsigned long long a = key[i], b = key[j];
                    if (a > b) {
                        key[i] = b;
                        key[j] = a;
                    }
                }
            }
            __syncthreads();
            for (int jj = k >> 2; jj > 0; jj >>= 1) {
                for (int c = threadIdx.x; c < P / 2; c += kSortThreads) {
                    const int i = (c / jj) * 2 * jj + (c % jj), j = i + jj;
                    if (j < n) {
                        unsigned long long a = key[i], b = key[j];
                        if (a > b) {
                            key[i] = b;
                            key[j] = a;
                        }
                    }
                }
                __syncthreads();
            }
        }
    }
}

// The tiles of at least kLongTile keys lead the longest-first tile queue (the tile scan counts
// them); blocks stride over those positions.  A list is a chain of nine barriers and as many LDS
// round trips, about 6 us, so what counts is how many are in flight: 42 KB of LDS and 80
// VGPRs put three blocks of 512 lanes on a compute unit (at 151 VGPRs, one block, it took twice as
// long).  8.5 M keys in 7360 lists of about 1150 (four 1280x720 views of 1 M Gaussians): the
// network, with 256 lanes, 64 KB and a block per tile, took 548 us, this takes 87.
constexpr int kSortGrid = 1024;

__global__ void __launch_bounds__(kSortThreads, 6) k_tile_sort_large(RParams rp, WsPtrs w)
{
    __shared__ SortShared sh;
    if (w.hdr->n_inst > rp.cap) return;
    const unsigned int n_large = w.hdr->n_large;
    for (unsigned int q = blockIdx.x; q < n_large; q += gridDim.x) {
        const int tile = (int)w.tile_queue[q];
        const unsigned int s = w.tile_start[tile], e = w.tile_start[tile + 1];
        const int n = (int)(e - s);
        if ((unsigned int)n < kLongTile) continue;  // uniform
        unsigned long long* key = w.keys + s;
        const int first = n > kSortLds && n <= kSortCap ? split_tile(key, n, sh) : 0;
        // the whole list, or its two halves
        for (int at = 0, len = first ? first : n; at < n; at += len, len = n - at) {
            if (len > kSortLds || !sort_tile_buckets(key + at, len, sh)) {
                __syncthreads();
                sort_tile_network(w, key + at, len, sh);
            }
            __syncthreads();  // the next keys take this list's LDS
        }
    }
}

// ------------------------------------------------------------ loss reduce
__global__ void __launch_bounds__(1024) k_loss_reduce(const ViewTable* __restrict__ vtp, RParams rp, WsPtrs w, float* out_loss,
                                                     int has_loss)
{
    const ViewTable& vt = *vtp;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    // Per view: the colour L1 sum, depth L1 sum and |Omega| over its tiles, each
    // summed per lane, then per wavefront (DPP), then over the wavefronts in order
    // by one thread: one barrier for all views.
    __shared__ float4 red[GPS_MAX_VIEWS][16];
    unsigned long long pe = 0ull, pc = 0ull;
    const bool counted = w.hdr->n_inst <= rp.cap;  // else no tile was composited
    for (int v = 0; v < vt.n; ++v) {
        const DevView& V = vt.v[v];
        const int nt = V.tiles_x * V.tiles_y;
        float a = 0.0f, b = 0.0f, c = 0.0f;
#pragma unroll 2
        for (int t = threadIdx.x; t < nt; t += 1024) {
            const float4 q = w.tile_loss[V.tile_base + t];
            const uint2 n = w.tile_pairs[V.tile_base + t];
            pe += n.x;
            pc += n.y;
            a += q.x;
            b += q.y;
            c += q.z;
        }
        a = wave_sum(a);
        b = wave_sum(b);
        c = wave_sum(c);
        if (lane == 0) red[v][wid] = make_float4(a, b, c, 0.0f);
    }
    // Evaluated / composited pair counts of this forward, added to the cumulative
    // counters of the header.
    for (int o = 32; o > 0; o >>= 1) {
        pe += __shfl_xor(pe, o, 64);
        pc += __shfl_xor(pc, o, 64);
    }
    __shared__ unsigned long long spe[16], spc[16];
    if (lane == 0) {
        spe[wid] = pe;
        spc[wid] = pc;
    }
    __syncthreads();
    if (wid != 0) return;
    // one lane per view, then one for all, in order
    float Lv = 0.0f;
    if (lane < vt.n) {
        float a = 0.0f, b = 0.0f, c = 0.0f;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const float4 q = red[lane][k];
            a += q.x;
            b += q.y;
            c += q.z;
        }
        w.hdr->view_stats[lane][0] = a;
        w.hdr->view_stats[lane][1] = b;
        w.hdr->view_stats[lane][2] = c;
        w.hdr->view_stats[lane][3] = 0.0f;
        const float npx = 3.0f * (float)vt.v[lane].cam.W * (float)vt.v[lane].cam.H;
        Lv = a / npx + (c > 0.0f ? rp.lambda * b / c : 0.0f);
    }
    float L = 0.0f;
    for (int v = 0; v < vt.n; ++v) L += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(Lv), v));
    if (lane == 0) {
        unsigned long long te = 0ull, tc = 0ull;
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            te += spe[k];
            tc += spc[k];
        }
        if (counted) {
            w.hdr->pairs_eval += te;
            w.hdr->pairs_contrib += tc;
        }
        L = L / (float)vt.n;
        w.hdr->loss = has_loss ? L : 0.0f;
        if (out_loss && has_loss) *out_loss = L;
    }
}

// ------------------------------------------------------------ view table
// Copies the by-value view table into the workspace (the first block), so that a replayed
// sequence of kernels reads whatever table was uploaded last.  A view with pose_xi is written
// with the camera Exp(xi) T_cw (binary64 composition, rounded once to binary32).
// Then (one block per tile) the tile depth maxima: the maximum of the SDF base depth over each
// screen tile (invalid = +inf; the base images are fixed until the next upload).  They need nothing
// that pose_xi changes, so both are one launch and read the table in the kernel's arguments.
__global__ void __launch_bounds__(256) k_upload_views(ViewTable vt, ViewTable* dst, RParams rp, float* tilemax)
{
    if (blockIdx.x == 0) {
        const unsigned int* src = reinterpret_cast<const unsigned int*>(&vt);
        unsigned int* d = reinterpret_cast<unsigned int*>(dst);
        for (int i = threadIdx.x; i < (int)(sizeof(ViewTable) / 4); i += 256) d[i] = src[i];
        __syncthreads();
        const int v = threadIdx.x;
        if (v < vt.n && vt.v[v].pose_xi) {
            double xi[6], E[9], e[3];
            for (int k = 0; k < 6; ++k) xi[k] = (double)vt.v[v].pose_xi[k];
            se3_exp_d(xi, E, e);
            const DevCam& c = vt.v[v].cam;
            DevCam& o = dst->v[v].cam;
            for (int r = 0; r < 3; ++r) {
                for (int k = 0; k < 3; ++k)
                    o.R[3 * r + k] = (float)(E[3 * r] * c.R[k] + E[3 * r + 1] * c.R[3 + k] + E[3 * r + 2] * c.R[6 + k]);
                o.t[r] = (float)(E[3 * r] * c.t[0] + E[3 * r + 1] * c.t[1] + E[3 * r + 2] * c.t[2] + e[r]);
            }
        }
    }
    if (!tilemax) return;
    const int tile = blockIdx.x;
    const int v = find_view(vt, tile);
    const int W = vt.v[v].cam.W, H = vt.v[v].cam.H, lt = tile - vt.v[v].tile_base, tiles_x = vt.v[v].tiles_x;
    const float* depth = vt.v[v].base_depth;
    const int tx = lt % tiles_x, ty = lt / tiles_x;
    float m = -INFINITY;
    for (int k = threadIdx.x; k < rp.tile_w * rp.tile_h; k += 256) {
        const int x = tx * rp.tile_w + k % rp.tile_w, y = ty * rp.tile_h + k / rp.tile_w;
        if (x < W && y < H) {
            const float d = depth[(size_t)y * W + x];
            m = fmaxf(m, d > 0.0f ? d : INFINITY);
        }
    }
    m = wave_max(m);
    __shared__ float red[4];
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) tilemax[tile] = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// The table upload, with (with_tilemax) the tile depth maxima of its views.
gps_status launch_views_upload(const ViewTable& vt, const RParams& rp, const WsLayout& L, char* ws, int with_tilemax,
                               hipStream_t s)
{
    ViewTable* dvt = reinterpret_cast<ViewTable*>(ws + L.vtab);
    float* tilemax = with_tilemax ? ws_ptrs(ws, L).tilemax : nullptr;
    GPS_LAUNCH(K_UPLOAD, s, k_upload_views, dim3(with_tilemax ? L.n_tiles : 1), dim3(256), 0, s, vt, dvt, rp, tilemax);
    return hipGetLastError() == hipSuccess ? GPS_OK : GPS_ERR_HIP;
}

// ----------------------------------------------------------------- launch
template <int WAVES, int PER, bool LDS>
static void launch_project(const ViewTable* vt, const RParams& rp, const BinShape& bs, const GParams& gp, const WsPtrs& w,
                           hipStream_t s)
{
    const dim3 grid((unsigned int)(bs.chunks * rp.V)), blk(64 * WAVES);
    const size_t lds = 4 * (size_t)bs.lds_words;
    if (gp.sh_k) GPS_LAUNCH(K_PROJECT, s, (k_project<WAVES, PER, LDS, true>), grid, blk, lds, s, vt, rp, bs, gp, w);
    else GPS_LAUNCH(K_PROJECT, s, (k_project<WAVES, PER, LDS, false>), grid, blk, lds, s, vt, rp, bs, gp, w);
}

template <int WAVES, int PER, bool LDS>
static void launch_emit(const ViewTable* vt, const RParams& rp, const BinShape& bs, const WsPtrs& w, hipStream_t s)
{
    const dim3 grid((unsigned int)(bs.chunks * rp.V)), blk(64 * WAVES);
    GPS_LAUNCH(K_EMIT, s, (k_emit<WAVES, PER, LDS>), grid, blk, 4 * (size_t)bs.lds_words, s, vt, rp, bs, w);
}

gps_status launch_render_fwd(const gps_render_cfg* cfg, const RParams& rp, const gps_gaussians* g,
                             const ViewTable& vt, const WsLayout& L, char* ws, float* out_loss, hipStream_t s)
{
    WsPtrs w = ws_ptrs(ws, L);
    GParams gp{g->mean, g->log_scale, g->quat, g->opacity_logit, g->rgb, g->sh_degree > 0 ? g->sh : nullptr,
               sh_count(g->sh_degree)};
    int has_loss = 1;
    for (int v = 0; v < vt.n; ++v)
        if (!vt.v[v].target_rgb) has_loss = 0;
    // the kernels read the view table from the workspace
    const ViewTable* dvt = reinterpret_cast<const ViewTable*>(ws + L.vtab);
    if (!(cfg->flags & GPS_RENDER_VIEWS_PRESET)) {
        const gps_status st = launch_views_upload(vt, rp, L, ws, 1, s);
        if (st != GPS_OK) return st;
    }
    const BinShape& bs = L.bin;
    if (bs.chunks > 0) {
        if (!bs.lds) {
            const size_t n = (size_t)bs.rows * L.n_tiles;
            GPS_LAUNCH(K_SCAN, s, k_zero_rows, dim3((unsigned int)std::min((n + kBlk - 1) / kBlk, (size_t)1024)),
                       dim3(kBlk), 0, s, w, n);
        }
        if (bs.unsorted) {
            const dim3 grid((unsigned int)(bs.chunks * rp.V));
            if (gp.sh_k) GPS_LAUNCH(K_PROJECT, s, k_project_groups<true>, grid, dim3(kBlk), 0, s, dvt, rp, bs, gp, w);
            else GPS_LAUNCH(K_PROJECT, s, k_project_groups<false>, grid, dim3(kBlk), 0, s, dvt, rp, bs, gp, w);
        } else if (bs.per == kFewPer && bs.lds) launch_project<kFewWaves, kFewPer, true>(dvt, rp, bs, gp, w, s);
        else if (bs.per == kFewPer) launch_project<kFewWaves, kFewPer, false>(dvt, rp, bs, gp, w, s);
        else if (bs.lds) launch_project<kManyWaves, kManyPer, true>(dvt, rp, bs, gp, w, s);
        else launch_project<kManyWaves, kManyPer, false>(dvt, rp, bs, gp, w, s);
    }
    if (bs.rows <= kSmallRows && L.n_tiles <= kSmallTiles) {
        GPS_LAUNCH(K_SCAN, s, k_scan_small, dim3(1), dim3(1024), 0, s, dvt, rp, bs, w, L.n_tiles);
    } else {
        GPS_LAUNCH(K_SCAN, s, k_scan_rows, dim3(1 + (L.n_tiles + kScanCols - 1) / kScanCols), dim3(kBlk), 0, s, dvt, rp, bs, w);
        if (L.n_tiles <= 2048) GPS_LAUNCH(K_SCAN_TILES, s, k_scan_tiles<2>, dim3(1), dim3(1024), 0, s, rp, w, L.n_tiles);
        else if (L.n_tiles <= 4096) GPS_LAUNCH(K_SCAN_TILES, s, k_scan_tiles<4>, dim3(1), dim3(1024), 0, s, rp, w, L.n_tiles);
        else GPS_LAUNCH(K_SCAN_TILES, s, k_scan_tiles<8>, dim3(1), dim3(1024), 0, s, rp, w, L.n_tiles);
    }
    if (bs.chunks > 0) {
        if (bs.unsorted) GPS_LAUNCH(K_EMIT, s, k_emit_groups, dim3((unsigned int)(bs.chunks * rp.V)), dim3(kBlk), 0, s, dvt, rp, bs, w);
        else if (bs.per == kFewPer && bs.lds) launch_emit<kFewWaves, kFewPer, true>(dvt, rp, bs, w, s);
        else if (bs.per == kFewPer) launch_emit<kFewWaves, kFewPer, false>(dvt, rp, bs, w, s);
        else if (bs.lds) launch_emit<kManyWaves, kManyPer, true>(dvt, rp, bs, w, s);
        else launch_emit<kManyWaves, kManyPer, false>(dvt, rp, bs, w, s);
    }
    if (rp.mode != 2)  // the unsorted sort-free blend keeps the emission order
        GPS_LAUNCH(K_TILE_SORT_LARGE, s, k_tile_sort_large, dim3(L.n_tiles < kSortGrid ? L.n_tiles : kSortGrid),
                   dim3(kSortThreads), 0, s, rp, w);
    if (!dispatch_cfwd(cfg, dvt, rp, w, L.n_tiles, s)) return GPS_ERR_UNSUPPORTED_CONFIG;
    GPS_LAUNCH(K_LOSS_REDUCE, s, k_loss_reduce, dim3(1), dim3(1024), 0, s, dvt, rp, w, out_loss, has_loss);
    return hipGetLastError() == hipSuccess ? GPS_OK : GPS_ERR_HIP;
}

}  // namespace gps
