// Tuning constants of the instance binning (expansion and per-tile counters).
// Kept apart from the headers of the compositing kernels, which they do not affect.
#pragma once

#include <algorithm>

#include "gps_internal.h"

namespace gps {

// The projection counts the instances of its Gaussians per tile and the emission gives each
// a place, both in blocks over a share of one view's Gaussians.  A block's counters are in LDS and
// its counts a row of their own in memory, so neither pass has an atomic that leaves the CU:
// at four 1280x720 views of 1 M Gaussians (8.5 M instances) the atomics on counters shared by
// all blocks alone took 370 us, and the whole binning 747 against 245 now.
constexpr int kBinTiles = 12288;      // most tiles of a view with counters in LDS (48 KB a block: 64 with the walk)
constexpr int kCntSplit = 4;          // beyond, rows in memory that the blocks of a view share: 1 M Gaussians
                                      // in 12384 tiles 282 us, in 12288 with LDS 222
constexpr int kKeptBits = 32;         // slots of a Gaussian whose culls are kept as bits

// The shapes of a block (wavefronts, Gaussians a wavefront takes at a time), always 256 Gaussians:
//   few Gaussians:  8 of 32.  The walk of the slots is what takes long (up to 20 slots a
//                   Gaussian with 8x8 tiles), so it gets twice the wavefronts although the
//                   projection then uses half their lanes.  The binning of 50 k Gaussians of 14 slots
//                   takes 103 us, of 100 k of 3 slots 28; with 4 of 64 128 and 29, with 16 of 16
//                   87 and 35.
//   many:           4 of 64, which fill the chip: 8 wavefronts a SIMD.  (16 of 64, for fewer
//                   rows, measured the same.)
// Few / many at 40 k, 131 k, 170 k and 380 k (project, scans, emit in us): a 1280x720 view in tiles of 16x32
// 36 / 37, 38 / 39, 46 / 45 and 65 / 61; a 640x480 view in tiles of 8x8 46 / 51, 59 / 62, 68 / 71 and
// 88 / 89; four 640x480 views in tiles of 16x16 36 / 40, 46 / 42, 50 / 50 and 62 / 61.
constexpr int kFewWaves = 8, kFewPer = 32, kManyWaves = 4, kManyPer = 64;
constexpr long long kFewGaussians = 131072;  // over the views
constexpr int kMostWaves = 8192;             // over the views
constexpr int kMostSegs = kMostWaves;
static_assert(kFewGaussians / kFewPer + GPS_MAX_VIEWS * kFewWaves <= kMostSegs, "a view's last block may be short");
constexpr size_t kMostRowWords = 4u << 20;   // of tile counts over all blocks (12288 tiles: 341 blocks)

// Gaussians of a map lie in memory by the surface that they were seeded on, so the ones in view are
// runs of thousands.  A wavefront therefore takes its share from all over the map: with
// consecutive Gaussians the longest walk is five times the mean, and projection and emission of four
// 1280x720 views of 1 M take 116 + 144 us against 87 + 126.  Long runs, whose loads are whole
// lines, where a wavefront takes several anyway.
constexpr int kRunFew = 8, kRunShort = 16, kRunLong = 64, kRunIters = 4;

// Where no sort follows, the places that the emission gives are the order in which every pixel adds its
// Gaussians, so they decide the last bits of the images and, where a residual is within those bits of zero,
// the sign of its L1 adjoint.  The order is this: group k of 64 consecutive view-Gaussians (numbered
// over the views) takes its places in part k mod 4 of each tile's range, in each part as the
// groups arrive.  So the blocks take such groups (the ones in flight together a multiple of kCntSplit), and
// kCntSplit shared rows are the parts.  A pass over 70 k Gaussians at 953x617 takes 160 us, over two views of
// 901x675 and 161x120 and 42 k 213; with the walk by one wavefront a group 163 and 221; with LDS rows
// over the whole map, and so another order, 157 and 202.
constexpr int kOrderGroup = 64;

inline BinShape bin_shape(int M, int V, size_t n_tiles, size_t most_tiles, unsigned long long cap,
                          bool unsorted)
{
    BinShape b{0, kManyWaves, kManyPer, 0, kRunLong, 0, 0, 0, 0};
    if (M == 0) return b;
    if (unsorted) {
        // (a view's first group may begin in the view before)
        const int wanted = (int)(((long long)M + 2 * (kOrderGroup - 1)) / kOrderGroup);
        const int most = std::max(kMostWaves / V / kCntSplit, 1) * kCntSplit;
        b.unsorted = 1;
        b.waves = 1;
        b.per = kOrderGroup;
        b.rows = kCntSplit;
        b.iters = (wanted + most - 1) / most;
        b.chunks = ((wanted + b.iters - 1) / b.iters + kCntSplit - 1) / kCntSplit * kCntSplit;
        return b;
    }
    const bool few = (long long)M * V <= kFewGaussians;
    // The rows lie where the instance capacity has left room.  With much less room than blocks
    // wanted, the shared rows.
    const unsigned long long room = std::min(cap, (unsigned long long)std::max(kMostRowWords, 64 * n_tiles)) / n_tiles;
    b.lds = most_tiles <= (size_t)kBinTiles && room >= (unsigned long long)std::min((M + kBlk - 1) / kBlk, 64);
    if (few) {
        b.waves = kFewWaves;
        b.per = kFewPer;
    }
    const int group = b.waves * b.per, wanted = (M + group - 1) / group;
    int most = few ? wanted : std::max(kMostWaves / b.waves / V, 1);
    if (b.lds) most = (int)std::min((unsigned long long)most, room);
    b.iters = (wanted + most - 1) / most;
    b.chunks = (wanted + b.iters - 1) / b.iters;
    b.run = b.iters >= kRunIters ? kRunLong : kRunShort;
    if (few) b.run = kRunFew;
    b.rows = b.lds ? b.chunks : kCntSplit;
    b.lds_words = b.lds ? (int)most_tiles : 0;
    return b;
}

constexpr int kSmallSort = 512;       // one wavefront sorts up to this many keys in registers
// Tiles of at least kLongTile keys (exactly those whose queue bucket floor(log2(n + 1))
// is log2(kSmallSort) or more, so they lead the longest-first queue) take the block sort.
constexpr unsigned int kLongTile = kSmallSort - 1;


// Bitonic network in which every compare-exchange puts the smaller key at the
// lower index (the first step of each merge compares mirrored pairs: element e
// with e ^ (k - 1) inside its aligned block of k), so padding with +inf keys
// never moves into the sorted range.  wave_sort_regs sorts up to 64 R keys in
// registers of one wavefront: element e = 64 r + lane sits in register r of that
// lane, so a compare-exchange at distance < 64 is a lane exchange (shuffle) and
// one at distance >= 64 a swap between two registers of the same lane.  No LDS
// and no barriers.
__device__ __forceinline__ unsigned long long shfl_xor_u64(unsigned long long v, int m)
{
    const unsigned int lo = __shfl_xor((unsigned int)v, m, 64);
    const unsigned int hi = __shfl_xor((unsigned int)(v >> 32), m, 64);
    return ((unsigned long long)hi << 32) | lo;
}

__device__ __forceinline__ unsigned long long min_u64(unsigned long long a, unsigned long long b) { return a < b ? a : b; }
__device__ __forceinline__ unsigned long long max_u64(unsigned long long a, unsigned long long b) { return a < b ? b : a; }

// Sorts the n <= 64 R keys at key[0..n) ascending; one wavefront, lane `lane`.
template <int R>
__device__ __forceinline__ void wave_sort_regs(unsigned long long* key, int n, int lane)
{
    constexpr int P = 64 * R;
    unsigned long long x[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = 64 * r + lane;
        x[r] = e < n ? key[e] : ~0ull;
    }
#pragma unroll
    for (int k = 2; k <= P; k <<= 1) {
        // mirrored step: e <-> e ^ (k - 1); e is the lower index when bit k/2 of e is clear
        if (k <= 64) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const unsigned long long o = shfl_xor_u64(x[r], k - 1);
                x[r] = (lane & (k >> 1)) == 0 ? min_u64(x[r], o) : max_u64(x[r], o);
            }
        } else {
            const int jr = k / 64 - 1;  // partner: register r ^ jr of lane ^ 63
            unsigned long long o[R];
#pragma unroll
            for (int r = 0; r < R; ++r) o[r] = shfl_xor_u64(x[r ^ jr], 63);
#pragma unroll
            for (int r = 0; r < R; ++r)
                x[r] = ((64 * r) & (k >> 1)) == 0 ? min_u64(x[r], o[r]) : max_u64(x[r], o[r]);
        }
        // half-cleaner steps: e <-> e ^ j, j = k/4 .. 1
#pragma unroll
        for (int j = k >> 2; j > 0; j >>= 1) {
            if (j >= 64) {
                const int jr = j / 64;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if ((r & jr) == 0) {
                        const unsigned long long a = x[r], b = x[r | jr];
                        x[r] = min_u64(a, b);
                        x[r | jr] = max_u64(a, b);
                    }
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const unsigned long long o = shfl_xor_u64(x[r], j);
                    x[r] = (lane & j) == 0 ? min_u64(x[r], o) : max_u64(x[r], o);
                }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = 64 * r + lane;
        if (e < n) key[e] = x[r];
    }
}

// Sorts the n < kLongTile keys at key[0..n) with the smallest register network
// that holds them (one wavefront).
__device__ __forceinline__ void wave_sort_tile(unsigned long long* key, int n, int lane)
{
    if (n <= 64) wave_sort_regs<1>(key, n, lane);
    else if (n <= 128) wave_sort_regs<2>(key, n, lane);
    else if (n <= 256) wave_sort_regs<4>(key, n, lane);
    else wave_sort_regs<8>(key, n, lane);
}

}  // namespace gps
