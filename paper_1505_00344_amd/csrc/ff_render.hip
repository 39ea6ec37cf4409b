// ff_render.hip — particle image (Appendix A "Render Technique"; Appendix A.1:
// the vertex shader applies the model-view matrix, the geometry shader the
// view-projection matrix — orthographic for 2D, perspective for 3D — and
// emits a square sprite; the fragment shader gives each covered pixel an
// intensity that falls off with the distance from the sprite's centre and a
// colour that is fixed or linear in the particle's position; blending adds
// source*alpha into the pixel).
//
// Per particle, all geometry in double precision:
//   c = M (a0, a1, a2, 1) with M = projection * view * model (row-major 4x4);
//   culled if c3 <= 0 or some c_i / c3 (i < 3) is outside [-1, 1] or NaN;
//   px = (c0/c3 + 1) W / 2, py = (1 - c1/c3) H / 2;
//   rgb_k = clamp(base_k + sum_i grad[k][i] (a_i - origin_i), 0, 1);
//   radius 0: pixel (floor px, floor py) gets w = weight; radius R: pixels
//   floor(px - R - 1) .. floor(px + R + 1) (and in y) whose centre is at
//   distance d < R + 1 get w = weight (1 - d / (R + 1))^2;
//   img[(iy W + ix) 3 + k] += rint(256 w rgb_k)   (uint32, modulo 2^32).
// Fixed-point integer accumulation makes the image exact and independent of
// the order in which particles are added, so the two paths below give the
// same image bit for bit.
//
// Tiled path (sprites of radius <= 8, images of <= 4096 tiles of 64 x 32
// pixels, at most 2^29 particles).  Particles projected onto an attractor
// pile onto few pixels, and one global atomic per pixel hit serialises there.
// Instead:
//   1. partition: a block projects its particles, sorts what they draw by
//      tile in LDS and writes it to its own segment, with the start of every
//      tile in it.  A point (radius 0) is its pixel within the tile and its
//      three colour values, packed into 4 bytes (weights below 1/2) or 8; a
//      sprite is its particle's three coordinates (its index in double
//      precision), in the tile of its first pixel
//   2. points: one block owns a tile, gathers the tile's runs from all
//      segments, adds them up in LDS and stores the tile (or adds it to an
//      accumulated image, atomically), the only time the image is written; a
//      tile that holds more than a block's share is listed instead.  Sprites:
//      every tile is listed, in parts
//   3. the listed parts, added up in LDS and merged with one global atomic per
//      non-zero pixel and channel.  A tile of sprites (projected again by the
//      same code) has a margin in LDS on the right and below for what reaches
//      into its neighbours; the partition has cleared the image.
// HBM traffic per point: read 3 coordinates, write and read 4 or 8 B; plus the
// image once.  8,388,608 settled Lorenz particles at 1920 x 1080: 410 -> 99 us
// (partition 55, points 25, their parts 21), of which reading the coordinates
// and writing the image at the 4.6 TB/s of a large copy are 27; the partition
// is bound by VALU issue (70 %), near half of it the double-precision
// projection, the others wait for short gathers (62-71 % of their waves' time).
// 500,009 sprites of radius 2 at 1280 x 720: 137 -> 60 us (partition 12, list
// 5, draw 43); the draw waits two thirds of its waves' time, at barriers and
// for LDS, with VALU issue at 57 % and the LDS at 24 %.  Before, a counting
// sort over the whole image held particle indices: gathering their coordinates
// read a line of memory for each, every chunk of 1024 entries merged its tile
// by atomics, and every pixel took a double-precision square root and division.
// Larger sprites or images, and few points, use the direct path: one thread
// per particle, global atomics per pixel.
#include <algorithm>
#include <cmath>

#include "ff_internal.h"
#include "ff_scan.h"

namespace ff {

namespace {

struct RenderArgs {
    int axis[3];
    double mvp[16];
    int width, height;
    double base[3], grad[9], origin[3];
    double weight;
    int radius;
};

constexpr int kRTileW = 64, kRTileH = 32;
constexpr int kRTilePx = kRTileW * kRTileH;       // 2048 pixels, 24 KB of uint32 RGB
constexpr int kRMaxRadius = 8;                    // sprite <= 19 pixels: <= 2 x 2 tiles
constexpr int kRMaxTiles = 4096;                  // images up to 8M pixels (4K UHD fits)
constexpr int kRSort = 1024;                      // threads of a partition block
constexpr int64_t kRChunk = 4096;
constexpr int64_t kRMaxCounts = (int64_t)1 << 26;  // tiles x chunks of the tiled path
constexpr int64_t kRDirectMax = 8192;              // points drawn by the direct path
constexpr int kRList = 512;                        // sprites a draw block holds at a time
constexpr int kRSprite = 512;                      // threads of such a block
constexpr int64_t kRMaxN = (int64_t)1 << 29;       // 4 n entries stay below 2^31 (uint32 offsets)
constexpr uint32_t kRNone = 0xFFFFFFFFu;

struct Point {
    bool keep;
    double px, py;
    double rgb[3];
};

template <typename R>
__device__ __forceinline__ Point project(R a0, R a1, R a2, const RenderArgs& r) {
    Point P;
    const double a[3] = {(double)a0, (double)a1, (double)a2};
    double c[4];
#pragma unroll
    for (int row = 0; row < 4; ++row) {
        const double* m = r.mvp + 4 * row;
        c[row] = m[0] * a[0] + m[1] * a[1] + m[2] * a[2] + m[3];
    }
    bool keep = c[3] > 0.0;
    double ndc[3];
    if (c[3] > 0x1p-400 && c[3] < 0x1p400) {
        // three quotients by one divisor: its reciprocal (two Newton steps on
        // the hardware estimate), then q = a y and one residual correction,
        // which rounds a / c3 correctly (Markstein, IBM J. Res. Dev. 34, 1990).
        // What over- or underflows on the way is outside [-1, 1] (or NaN, and
        // culled alike) or so small that 1 + q is 1.
        double y = __builtin_amdgcn_rcp(c[3]);
        y = __builtin_fma(y, __builtin_fma(-c[3], y, 1.0), y);
        y = __builtin_fma(y, __builtin_fma(-c[3], y, 1.0), y);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double q = c[k] * y;
            ndc[k] = __builtin_fma(__builtin_fma(-c[3], q, c[k]), y, q);
        }
    } else {
#pragma unroll
        for (int k = 0; k < 3; ++k) ndc[k] = c[k] / c[3];
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) keep = keep && ndc[k] >= -1.0 && ndc[k] <= 1.0;
    P.keep = keep;
    P.px = (ndc[0] + 1.0) * (double)r.width / 2.0;
    P.py = (1.0 - ndc[1]) * (double)r.height / 2.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        double v = r.base[k];
#pragma unroll
        for (int j = 0; j < 3; ++j) v += r.grad[3 * k + j] * (a[j] - r.origin[j]);
        P.rgb[k] = fmin(fmax(v, 0.0), 1.0);
    }
    return P;
}

// Pixel box of a kept particle's sprite (before clipping to the image; the
// image has at most 2^28 pixels and the radius is at most 64).
__device__ __forceinline__ void sprite_box(const Point& P, int radius, int& x0, int& x1, int& y0, int& y1) {
    const double reach = radius + 1.0;
    x0 = (int)floor(P.px);
    x1 = x0;
    y0 = (int)floor(P.py);
    y1 = y0;
    if (radius > 0) {
        x0 = (int)floor(P.px - reach);
        x1 = (int)floor(P.px + reach);
        y0 = (int)floor(P.py - reach);
        y1 = (int)floor(P.py + reach);
    }
}

// The sprite's weight at pixel (ix, iy) of its box; false outside the disc.
__device__ __forceinline__ bool pixel_weight(const Point& P, int ix, int iy, const RenderArgs& r, double& w) {
    w = r.weight;
    if (r.radius > 0) {
        const double reach = r.radius + 1.0;
        const double dx = ((double)ix + 0.5) - P.px, dy = ((double)iy + 0.5) - P.py;
        const double d = sqrt(dx * dx + dy * dy);
        if (!(d < reach)) return false;
        const double f = 1.0 - d / reach;
        w = r.weight * (f * f);
    }
    return true;
}

__device__ __forceinline__ uint32_t quantise(double w, double rgb) { return (uint32_t)rint(256.0 * (w * rgb)); }

// ---------------------------------------------------------------- direct path
template <typename R>
__global__ void __launch_bounds__(256) k_render(const R* a0p, const R* a1p, const R* a2p, int64_t n, RenderArgs r,
                                                uint32_t* img, unsigned long long* culled) {
    __shared__ unsigned int s_cull;
    if (threadIdx.x == 0) s_cull = 0u;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t pix = kRNone, sum[3] = {0u, 0u, 0u};
    if (i < n) {
        const Point P = project<R>(a0p[i], a1p[i], a2p[i], r);
        if (!P.keep) {
            atomicAdd(&s_cull, 1u);
        } else {
            int x0, x1, y0, y1;
            sprite_box(P, r.radius, x0, x1, y0, y1);
            if (r.radius == 0) {
                if (x0 >= 0 && x0 < r.width && y0 >= 0 && y0 < r.height) {
                    pix = (uint32_t)y0 * (uint32_t)r.width + (uint32_t)x0;
#pragma unroll
                    for (int k = 0; k < 3; ++k) sum[k] = quantise(r.weight, P.rgb[k]);
                }
            } else {
                for (int iy = y0; iy <= y1; ++iy) {
                    for (int ix = x0; ix <= x1; ++ix) {
                        if (ix < 0 || ix >= r.width || iy < 0 || iy >= r.height) continue;
                        double w;
                        if (!pixel_weight(P, ix, iy, r, w)) continue;
                        uint32_t* at = img + ((int64_t)iy * r.width + ix) * 3;
#pragma unroll
                        for (int k = 0; k < 3; ++k) {
                            const uint32_t q = quantise(w, P.rgb[k]);
                            if (q) atomicAdd(at + k, q);
                        }
                    }
                }
            }
        }
    }
    // Points: a wave whose points share one pixel (an ensemble sitting on a
    // fixed point) would be served one by one; it adds their sum once (1,000
    // points: 40 -> 14 us).
    const uint64_t hits = __ballot(pix != kRNone);
    if (hits != 0) {
        const int lead = __builtin_ctzll(hits);
        const uint32_t one = (uint32_t)__shfl((int)pix, lead, 64);
        bool add = pix != kRNone;
        if (__ballot(add && pix != one) == 0) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                for (int off = 32; off; off >>= 1) sum[k] += (uint32_t)__shfl_xor((int)sum[k], off, 64);
            add = (int)(threadIdx.x & 63) == lead;
        }
        if (add) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (sum[k]) atomicAdd(img + (int64_t)pix * 3 + k, sum[k]);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0 && culled && s_cull) atomicAdd(culled, (unsigned long long)s_cull);
}

__global__ void k_clear_img(uint32_t* img, int64_t len, unsigned long long* culled) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = i; k < len; k += stride) img[k] = 0u;
    if (i == 0 && culled) *culled = 0ull;
}

// ---------------------------------------------------------------- tiled path
// What a particle leaves in its tile's run.
enum Payload {
    kPack32 = 0,  // point: pixel in the tile (bits 0-10), colour values (7 bits each)
    kPack64 = 1,  // point: pixel in the tile (bits 0-10), colour values (17 bits each)
    kCoords = 2,  // sprite: the three coordinates, single precision
    kIndex = 3    // sprite, or point of a weight beyond kPack64: the particle's index
};

struct Coords {
    float a[3];
};
template <int P> struct Entry { using T = uint32_t; };
template <> struct Entry<kPack64> { using T = unsigned long long; };
template <> struct Entry<kCoords> { using T = Coords; };

// Tile of the first pixel of a kept particle's sprite, clipped to the image;
// kRNone if no pixel of it is inside.
__device__ __forceinline__ uint32_t tile_of(const Point& P, const RenderArgs& r, int ntx) {
    int x0, x1, y0, y1;
    sprite_box(P, r.radius, x0, x1, y0, y1);
    x0 = x0 > 0 ? x0 : 0;
    y0 = y0 > 0 ? y0 : 0;
    if (x0 > x1 || y0 > y1 || x0 >= r.width || y0 >= r.height) return kRNone;
    return (uint32_t)(y0 / kRTileH) * (uint32_t)ntx + (uint32_t)(x0 / kRTileW);
}

// 1. partition: K particles per thread.  Row b of `starts` holds the nt run
// starts of segment b, its entries, and its culled particles.  Clears `clear`
// values of the image, with blocks beyond the particles' where these are too
// few for it.
template <typename R, int K, int P>
__global__ void __launch_bounds__(kRSort) k_render_partition(const R* a0p, const R* a1p, const R* a2p, int64_t n,
                                                             RenderArgs r, int ntx, int nt,
                                                             typename Entry<P>::T* sorted, uint16_t* starts,
                                                             uint32_t* n_items, uint32_t* img, int64_t clear) {
    using E = typename Entry<P>::T;
    constexpr int C = kRSort * K;
    __shared__ uint32_t cnt[kRMaxTiles];
    __shared__ E stage[C];
    __shared__ uint32_t wsum[32];
    __shared__ uint32_t s_cull;
    const int tid = threadIdx.x;
    for (int64_t k = (int64_t)blockIdx.x * kRSort + tid; k < clear; k += (int64_t)gridDim.x * kRSort) img[k] = 0u;
    const int64_t lo = (int64_t)blockIdx.x * C;
    if (lo >= n) return;  // the whole block
    for (int t = tid; t < nt; t += kRSort) cnt[t] = 0u;
    if (tid == 0) s_cull = 0u;
    __syncthreads();
    uint32_t tile[K], rank[K];
    E ent[K];
    uint32_t cull = 0;
    R next[3];
    auto load = [&](int64_t i) {
        const int64_t j = i < n ? i : n - 1;
        next[0] = a0p[j];
        next[1] = a1p[j];
        next[2] = a2p[j];
    };
    load(lo + tid);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t i = lo + k * kRSort + tid;
        tile[k] = kRNone;
        // the next particle is on its way while this one is projected
        const R a0 = next[0], a1 = next[1], a2 = next[2];
        if (k + 1 < K) load(i + kRSort);
        if (i >= n) continue;
        const Point pt = project<R>(a0, a1, a2, r);
        if (!pt.keep) {
            ++cull;
            continue;
        }
        tile[k] = tile_of(pt, r, ntx);
        if constexpr (P == kIndex) {
            ent[k] = (E)i;
        } else if constexpr (P == kCoords) {
            ent[k] = {(float)a0, (float)a1, (float)a2};  // R is float here
        } else {
            const uint32_t x = (uint32_t)(int)floor(pt.px), y = (uint32_t)(int)floor(pt.py);
            E e = (y % kRTileH) * kRTileW + x % kRTileW;
            constexpr int kBits = P == kPack32 ? 7 : 17;
#pragma unroll
            for (int c = 0; c < 3; ++c) e |= (E)quantise(r.weight, pt.rgb[c]) << (11 + kBits * c);
            ent[k] = e;
        }
    }
    if (cull) atomicAdd(&s_cull, cull);
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (tile[k] != kRNone) rank[k] = count_one(cnt, tile[k]);
    __syncthreads();
    // exclusive scan of the counts, four tiles per thread
    uint32_t c[4], sum = 0, kept;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        c[j] = 4 * tid + j < nt ? cnt[4 * tid + j] : 0u;
        sum += c[j];
    }
    uint32_t at = block_scan(sum, wsum, &kept);
    uint16_t* row = starts + (int64_t)blockIdx.x * (nt + 2);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (4 * tid + j < nt) {
            cnt[4 * tid + j] = at;
            row[4 * tid + j] = (uint16_t)at;
            at += c[j];
        }
    }
    if (tid == 0) {
        row[nt] = (uint16_t)kept;
        row[nt + 1] = (uint16_t)s_cull;
        if (blockIdx.x == 0) *n_items = 0u;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (tile[k] != kRNone) stage[cnt[tile[k]] + rank[k]] = ent[k];
    __syncthreads();
    uint32_t* dst = (uint32_t*)(sorted + lo);
    const uint32_t* src = (const uint32_t*)stage;
    for (uint32_t j = tid; j < kept * (uint32_t)(sizeof(E) / 4); j += kRSort) dst[j] = src[j];
}

// The sorted entries and what describes their order.
template <int P> struct RSegments {
    const typename Entry<P>::T* sorted;  // segment b from b * C
    const uint16_t* starts;              // [nblk][ntiles + 2]
    int nblk, C;
};

// Everything the second and third pass need besides the segments.
struct RTiles {
    int ntx, nt;
    bool accumulate;
    uint32_t* img;
};

// Points: LANES threads take a run, 16 bytes each at a time.
template <int P, int LANES>
__device__ __forceinline__ void gather_points(uint32_t* s, const RSegments<P>& g, int nt, int t, int b0, int b1) {
    using E = typename Entry<P>::T;
    constexpr int kPer = 16 / (int)sizeof(E), kBits = P == kPack32 ? 7 : 17;
    constexpr int kGroups = kRSort / LANES;
    auto add = [&](E e, uint32_t times) {
        uint32_t* px = s + 3 * (uint32_t)(e & 2047u);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const uint32_t q = (uint32_t)(e >> (11 + kBits * c)) & ((1u << kBits) - 1);
            if (q) atomicAdd(px + c, q * times);
        }
    };
    const int lane = threadIdx.x % LANES;
    for (int base = b0 + (int)(threadIdx.x / LANES); base < b1; base += 16 * kGroups) {
        // 16 lanes load the bounds of the group's next 16 runs
        const int mine = base + (int)(threadIdx.x & 15) * kGroups;
        uint32_t lo = 0, hi = 0;
        if (mine < b1) {
            const uint16_t* row = g.starts + (int64_t)mine * (nt + 2) + t;
            lo = row[0];
            hi = row[1];
        }
#pragma unroll 2
        for (int q = 0; q < 16; ++q) {
            const uint32_t beg = __shfl(lo, q, 16), end = __shfl(hi, q, 16);
            const E* e = g.sorted + (int64_t)(base + q * kGroups) * g.C;
            for (uint32_t j = (beg & ~(uint32_t)(kPer - 1)) + kPer * lane; j < end; j += kPer * LANES) {
                E v[kPer];
                const uint4 w = *(const uint4*)(e + j);
                __builtin_memcpy(v, &w, 16);
                // lanes that all hold one point (an ensemble on a fixed
                // point) would be served one by one: add their number
                bool same = j >= beg && j + kPer <= end;
#pragma unroll
                for (int k = 1; k < kPer; ++k) same = same && v[k] == v[0];
                const uint32_t f0 = __builtin_amdgcn_readfirstlane((uint32_t)v[0]);
                same = same && (uint32_t)v[0] == f0;
                if (sizeof(E) == 8) same = same && (uint32_t)((unsigned long long)v[0] >> 32) ==
                                                       __builtin_amdgcn_readfirstlane((uint32_t)((unsigned long long)v[0] >> 32));
                if (__ballot(!same) == 0) {
                    const uint64_t live = __ballot(1);
                    if ((threadIdx.x & 63) == (unsigned)__builtin_ctzll(live))
                        add(v[0], (uint32_t)kPer * (uint32_t)__popcll(live));
                } else {
#pragma unroll
                    for (int k = 0; k < kPer; ++k)
                        if (j + k >= beg && j + k < end) add(v[k], 1u);
                }
            }
        }
    }
}

// Segments b0 .. b1 - 1 of a tile with `total` entries in all segments, by 16
// threads a run or, where that takes more rounds of loads, by the whole block:
// few segments (a small ensemble) or an ensemble in few tiles leave few, long
// runs.  9,000 points of weight 1 on a 64 x 48 image (3 runs of 1500 a tile):
// 57 -> 24 us; 200,003 on a line of a 200 x 100 image: 43 -> 27.
template <int P>
__device__ __forceinline__ void gather_runs(uint32_t* s, const RSegments<P>& g, int nt, int t, int b0, int b1,
                                            uint32_t total) {
    constexpr int kPer = 16 / (int)sizeof(typename Entry<P>::T), kGroups = kRSort / 16;
    const int len = (int)(total / (uint32_t)g.nblk) + 1, runs = b1 - b0;
    if (runs * (1 + len / (kPer * kRSort)) < (runs + kGroups - 1) / kGroups * (1 + len / (kPer * 16)))
        gather_points<P, kRSort>(s, g, nt, t, b0, b1);
    else gather_points<P, 16>(s, g, nt, t, b0, b1);
}

// Sprites are worth hundreds of instructions each and their runs are short (a
// block of 1024 particles leaves a few in a tile), so an accumulate block
// first joins the runs into a list, then projects the list's particles, one a
// thread, into these records, and last draws row by row, one row of one
// sprite a thread, so that every lane has work whatever the runs.
// EXACT: the records and the rows in double precision, half as many at a time.
template <bool EXACT> struct SpriteList {
    static constexpr int kN = kRList;
    uint32_t entry[kN];      // position in the segments
    uint32_t box[kN];        // first column (7 bits) and row (6) in the tile, from bit 16 columns and rows less one (5 each)
    float dx0[kN], dy0[kN];  // centre of the first pixel less the sprite's
    float A[3][kN];          // 256 weight rgb
};
template <> struct SpriteList<true> {
    static constexpr int kN = kRList / 2;
    uint32_t entry[kN], box[kN];
    double px[kN], py[kN], rgb[3][kN];  // the sprite's centre and colour
};
constexpr uint32_t kNoRows = 31;  // a sprite has at most 2 (R + 1) = 18 rows

// The particles behind the entries.
template <typename R, int P> struct Particles {
    const R* a0;
    const R* a1;
    const R* a2;
    const typename Entry<P>::T* sorted;
    __device__ __forceinline__ Point at(uint32_t entry, const RenderArgs& r) const {
        if constexpr (P == kCoords) {
            const Coords c = sorted[entry];
            return project<R>(c.a[0], c.a[1], c.a[2], r);
        } else {
            const uint32_t i = sorted[entry];
            return project<R>(a0[i], a1[i], a2[i], r);
        }
    }
};

// A listed particle's record.  Its box holds the image's pixels whose centres
// are nearer than the sprite's reach in either direction (no other can be in
// the disc).
template <bool EXACT>
__device__ __forceinline__ void sprite_record(const Point& P, const RenderArgs& r, int X0, int Y0,
                                              SpriteList<EXACT>& L, uint32_t j) {
    int x0, x1, y0, y1;
    sprite_box(P, r.radius, x0, x1, y0, y1);
    if (r.radius > 0) {
        const double reach = r.radius + 1.0;
        if (((double)x0 + 0.5) - P.px <= -reach) ++x0;
        if (((double)y0 + 0.5) - P.py <= -reach) ++y0;
        if (((double)x1 + 0.5) - P.px >= reach) --x1;
        if (((double)y1 + 0.5) - P.py >= reach) --y1;
    }
    x0 = x0 > X0 ? x0 : X0;
    y0 = y0 > Y0 ? y0 : Y0;
    x1 = x1 < r.width - 1 ? x1 : r.width - 1;
    y1 = y1 < r.height - 1 ? y1 : r.height - 1;
    L.box[j] = x0 > x1 || y0 > y1 ? kNoRows << 21
                                  : (uint32_t)(x0 - X0) | (uint32_t)(y0 - Y0) << 7 | (uint32_t)(x1 - x0) << 16 |
                                        (uint32_t)(y1 - y0) << 21;
    if constexpr (EXACT) {
        L.px[j] = P.px;
        L.py[j] = P.py;
#pragma unroll
        for (int k = 0; k < 3; ++k) L.rgb[k][j] = P.rgb[k];
    } else {
        L.dx0[j] = (float)(((double)x0 + 0.5) - P.px);
        L.dy0[j] = (float)(((double)y0 + 0.5) - P.py);
#pragma unroll
        for (int k = 0; k < 3; ++k) L.A[k][j] = (float)(256.0 * (r.weight * P.rgb[k]));
    }
}

// Row `row` of record j's sprite into the LDS tile (`pitch` values a row).
// The pixel values are rint(256 w rgb_k) of double-precision operations; they
// are found in single precision, whose value differs from that one by less
// than 26 2^-24 times the sprite's largest (with u = 2^-24: dx, dy rounded and
// stepped 2 u (R + 2) each; d 6 u (R + 2); f = 1 - d / (R + 1) 11 u; f^2 23 u;
// the products 26 u), and again in double precision where that could change
// the rounding.
template <typename R, int P>
__device__ __forceinline__ void sprite_row(const SpriteList<false>& L, uint32_t j, uint32_t row, const RenderArgs& r,
                                           int X0, int Y0, uint32_t* s, int pitch, const Particles<R, P>& pa) {
    const uint32_t box = L.box[j], rows = box >> 21;
    if (row > rows || rows == kNoRows) return;
    const int bx = (int)(box & 127u), by = (int)((box >> 7) & 63u), nx = (int)((box >> 16) & 31u);
    const float inv = 1.0f / (float)(r.radius + 1);
    const float dy = L.dy0[j] + (float)row, dy2 = dy * dy, dx0 = L.dx0[j];
    const float A0 = L.A[0][j], A1 = L.A[1][j], A2 = L.A[2][j];
    const float lim = 0.5f - 2e-6f * fmaxf(fmaxf(A0, A1), A2);
    uint32_t* px = s + (by + (int)row) * pitch + 3 * bx;
    for (int ix = 0; ix <= nx; ++ix, px += 3) {
        const float dx = dx0 + (float)ix;
        const float d = __builtin_amdgcn_sqrtf(__builtin_fmaf(dx, dx, dy2));
        const float f = r.radius > 0 ? fmaxf(__builtin_fmaf(-d, inv, 1.0f), 0.0f) : 1.0f;
        const float g = f * f;
        const float v0 = g * A0, v1 = g * A1, v2 = g * A2;
        const float q0 = rintf(v0), q1 = rintf(v1), q2 = rintf(v2);
        if (fmaxf(fmaxf(fabsf(v0 - q0), fabsf(v1 - q1)), fabsf(v2 - q2)) < lim) {
            if (q0 + q1 + q2 > 0.0f) {
                atomicAdd(px, (uint32_t)q0);
                atomicAdd(px + 1, (uint32_t)q1);
                atomicAdd(px + 2, (uint32_t)q2);
            }
        } else {
            const Point pt = pa.at(L.entry[j], r);
            double w;
            if (!pixel_weight(pt, X0 + bx + ix, Y0 + by + (int)row, r, w)) continue;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const uint32_t v = quantise(w, pt.rgb[k]);
                if (v) atomicAdd(px + k, v);
            }
        }
    }
}

// The same by the double-precision operations alone.
template <typename R, int P>
__device__ __forceinline__ void sprite_row(const SpriteList<true>& L, uint32_t j, uint32_t row, const RenderArgs& r,
                                           int X0, int Y0, uint32_t* s, int pitch, const Particles<R, P>&) {
    const uint32_t box = L.box[j], rows = box >> 21;
    if (row > rows || rows == kNoRows) return;
    const int bx = (int)(box & 127u), by = (int)((box >> 7) & 63u), nx = (int)((box >> 16) & 31u);
    const Point pt{true, L.px[j], L.py[j], {L.rgb[0][j], L.rgb[1][j], L.rgb[2][j]}};
    uint32_t* px = s + (by + (int)row) * pitch + 3 * bx;
    for (int ix = 0; ix <= nx; ++ix, px += 3) {
        double w;
        if (!pixel_weight(pt, X0 + bx + ix, Y0 + by + (int)row, r, w)) continue;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t v = quantise(w, pt.rgb[k]);
            if (v) atomicAdd(px + k, v);
        }
    }
}

// Tile t's sprites number e0 .. e1 - 1 (counted over all segments), added to
// the LDS tile.
template <typename R, int P, bool EXACT>
__device__ __forceinline__ void gather_sprites(uint32_t* s, SpriteList<EXACT>& L, uint32_t* wsum, const RSegments<P>& g,
                                               int ntx, int nt, int t, uint32_t e0, uint32_t e1,
                                               const Particles<R, P>& pa, const RenderArgs& r) {
    constexpr uint32_t kList = SpriteList<EXACT>::kN;
    const int X0 = (t % ntx) * kRTileW, Y0 = (t / ntx) * kRTileH;
    const int tid = threadIdx.x;
    const uint32_t margin = r.radius > 0 ? 2u * (uint32_t)(r.radius + 1) : 0u, rows = margin ? margin : 1u;
    const int pitch = 3 * (kRTileW + (int)margin);
    const float per_row = 1.0f / (float)rows;
    uint32_t held = 0;  // entries in the list, uniform over the block
    auto draw = [&]() {
        __syncthreads();
        for (uint32_t j = tid; j < held; j += kRSprite) sprite_record<EXACT>(pa.at(L.entry[j], r), r, X0, Y0, L, j);
        __syncthreads();
        for (uint32_t w = tid; w < held * rows; w += kRSprite) {
            // w / rows: w is below 2^14, so the product is off by far less
            // than the half step
            const uint32_t j = (uint32_t)(((float)w + 0.5f) * per_row);
            sprite_row<R, P>(L, j, w - j * rows, r, X0, Y0, s, pitch, pa);
        }
        __syncthreads();
        held = 0;
    };
    uint32_t seen = 0;  // entries in the segments before `base`
    for (int base = 0; base < g.nblk && seen < e1; base += kRSprite) {
        const int b = base + tid;
        uint32_t lo = 0, len = 0, all;
        if (b < g.nblk) {
            const uint16_t* row = g.starts + (int64_t)b * (nt + 2) + t;
            lo = (uint32_t)b * (uint32_t)g.C + row[0];
            len = row[1] - (uint32_t)row[0];
        }
        uint32_t off = seen + block_scan(len, wsum, &all);
        // what of it lies in e0 .. e1 - 1: `all` entries, this thread's `len`
        // from `off` on
        const uint32_t s0 = max(seen, e0), s1 = min(seen + all, e1);
        seen += all;
        const uint32_t from = max(off, s0), to = min(off + len, s1);
        all = s0 < s1 ? s1 - s0 : 0u;
        len = from < to ? to - from : 0u;
        lo += from - off;
        off = from - s0;
        for (uint32_t done = 0; done < all;) {
            const uint32_t take = all - done < kList - held ? all - done : kList - held;
            // the entries at positions done .. done + take - 1: each thread
            // lists its short run, a wave its long ones together
            if (__ballot(len > 32) == 0) {
                for (uint32_t j = 0; j < len; ++j)
                    if (off + j - done < take) L.entry[held + off + j - done] = lo + j;
            } else {
                for (int q = 0; q < 64; ++q) {
                    const uint32_t qlen = __shfl(len, q, 64), qoff = __shfl(off, q, 64), qlo = __shfl(lo, q, 64);
                    const uint32_t j0 = qoff < done ? done - qoff : 0u;
                    for (uint32_t j = j0 + (tid & 63); j < qlen && qoff + j - done < take; j += 64)
                        L.entry[held + qoff + j - done] = qlo + j;
                }
            }
            held += take;
            done += take;
            if (held == kList) draw();
        }
    }
    if (held) draw();
}

// Entries of tile t in all segments, counted by the whole block.
template <int P>
__device__ __forceinline__ uint32_t tile_total(const RSegments<P>& g, int nt, int t, uint32_t* s_sum) {
    if (threadIdx.x == 0) *s_sum = 0u;
    __syncthreads();
    uint32_t mine = 0;
    for (int b = threadIdx.x; b < g.nblk; b += blockDim.x) {
        const uint16_t* row = g.starts + (int64_t)b * (nt + 2) + t;
        mine += (uint32_t)row[1] - row[0];
    }
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off, 64);
    if ((threadIdx.x & 63) == 0 && mine) atomicAdd(s_sum, mine);
    __syncthreads();
    return *s_sum;
}

// A part of an over-full tile, in four bytes: an image of few tiles leaves
// little more in the caller's workspace beside eight bytes per point.  A tile
// has at most n / per + 1 parts: 411 of points, 822 of sprites (rlayout).
struct RItem {
    uint32_t tile : 12, part : 10, parts : 10;
};
static_assert(sizeof(RItem) == 4 && kRMaxTiles <= 1 << 12, "the fields of a part");

// The culled particles of all segments, by one block.
template <int P>
__device__ __forceinline__ void count_culled(const RSegments<P>& g, int nt, bool accumulate, uint32_t* s_sum,
                                             unsigned long long* culled) {
    if (!culled) return;
    if (threadIdx.x == 0) *s_sum = 0u;
    __syncthreads();
    uint32_t mine = 0;
    for (int b = threadIdx.x; b < g.nblk; b += blockDim.x) mine += g.starts[(int64_t)b * (nt + 2) + nt + 1];
    if (mine) atomicAdd(s_sum, mine);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (accumulate) atomicAdd(culled, (unsigned long long)*s_sum);
        else *culled = *s_sum;
    }
}

// Lists tile t in parts of about `per` entries; called by the whole block.
__device__ __forceinline__ void list_parts(int t, uint32_t total, uint32_t per, RItem* items, uint32_t* n_items,
                                           uint32_t* s_at) {
    const uint32_t parts = (total + per - 1) / per;
    __syncthreads();  // s_at may still be read
    if (threadIdx.x == 0) *s_at = atomicAdd(n_items, parts);
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < parts; k += blockDim.x) items[*s_at + k] = {(uint32_t)t, k, parts};
}

// Hand every image value of an LDS tile with a margin of m pixels to
// put(address, sum).
template <class F>
__device__ __forceinline__ void each_pixel(const uint32_t* s, const RTiles& T, int t, int m, const RenderArgs& r,
                                           F put) {
    const int X0 = (t % T.ntx) * kRTileW, Y0 = (t / T.ntx) * kRTileH;
    const int pitch = 3 * (kRTileW + m);
    const int w = 3 * min(r.width - X0, kRTileW + m), h = min(r.height - Y0, kRTileH + m);
    uint32_t* d = T.img + ((int64_t)Y0 * r.width + X0) * 3;
    for (int y = threadIdx.x >> 6; y < h; y += (int)(blockDim.x >> 6)) {  // a wave per row
        for (int x = threadIdx.x & 63; x < w; x += 64) {
            put(d + (int64_t)y * (3 * r.width) + x, s[y * pitch + x]);
        }
    }
}

// 2. accumulate, points: block t owns tile t; the last block counts the culled
template <int P>
__global__ void __launch_bounds__(kRSort) k_points_accum(RSegments<P> g, RTiles T, uint32_t per, RenderArgs r,
                                                         unsigned long long* culled, RItem* items, uint32_t* n_items) {
    __shared__ uint32_t s[kRTilePx * 3];
    __shared__ uint32_t s_sum;
    const int t = blockIdx.x;
    if (t == T.nt) return count_culled<P>(g, T.nt, T.accumulate, &s_sum, culled);
    const uint32_t total = tile_total<P>(g, T.nt, t, &s_sum);
    if (total > per) {
        list_parts(t, total, per, items, n_items, &s_sum);
        if (!T.accumulate) each_pixel(s, T, t, 0, r, [](uint32_t* d, uint32_t) { *d = 0u; });
        return;
    }
    if (total == 0 && T.accumulate) return;
    for (int k = threadIdx.x; k < kRTilePx * 3; k += kRSort) s[k] = 0u;
    __syncthreads();
    if (total) gather_runs<P>(s, g, T.nt, t, 0, g.nblk, total);
    __syncthreads();
    // no other block has this tile, but calls on other streams may add to the
    // same image
    if (T.accumulate) each_pixel(s, T, t, 0, r, [](uint32_t* d, uint32_t v) { if (v) atomicAdd(d, v); });
    else each_pixel(s, T, t, 0, r, [](uint32_t* d, uint32_t v) { *d = v; });
}

// 3. the listed parts of over-full tiles, points
template <int P>
__global__ void __launch_bounds__(kRSort) k_points_split(RSegments<P> g, RTiles T, uint32_t per, RenderArgs r,
                                                         const RItem* items, const uint32_t* n_items) {
    __shared__ uint32_t s[kRTilePx * 3];
    const uint32_t m = *n_items;
    for (uint32_t k = blockIdx.x; k < m; k += gridDim.x) {  // uniform over the block
        const RItem it = items[k];
        const int tile = (int)it.tile;
        const int b0 = (int)((int64_t)g.nblk * it.part / it.parts);
        const int b1 = (int)((int64_t)g.nblk * (it.part + 1) / it.parts);
        for (int j = threadIdx.x; j < kRTilePx * 3; j += kRSort) s[j] = 0u;
        __syncthreads();
        gather_runs<P>(s, g, T.nt, tile, b0, b1, it.parts * per);
        __syncthreads();
        each_pixel(s, T, tile, 0, r, [](uint32_t* d, uint32_t v) { if (v) atomicAdd(d, v); });
        __syncthreads();
    }
}

// LDS of a sprite block: the list, then the tile with its margins.
template <bool EXACT> size_t sprite_lds(int radius) {
    const size_t m = radius > 0 ? 2 * (size_t)(radius + 1) : 0;
    return sizeof(SpriteList<EXACT>) + (kRTileW + m) * (kRTileH + m) * 12;
}

template <typename R, int P, bool EXACT>
__device__ __forceinline__ void sprite_tile(char* lds, uint32_t* wsum, const RSegments<P>& g, const RTiles& T, int t,
                                            uint32_t e0, uint32_t e1, const Particles<R, P>& pa, const RenderArgs& r) {
    const int m = r.radius > 0 ? 2 * (r.radius + 1) : 0;
    uint32_t* s = (uint32_t*)(lds + sizeof(SpriteList<EXACT>));
    for (int k = threadIdx.x; k < 3 * (kRTileW + m) * (kRTileH + m); k += kRSprite) s[k] = 0u;
    __syncthreads();
    gather_sprites<R, P, EXACT>(s, *(SpriteList<EXACT>*)lds, wsum, g, T.ntx, T.nt, t, e0, e1, pa, r);
    __syncthreads();
}

// 2. sprites: block t lists tile t, the last block counts the culled
template <int P>
__global__ void __launch_bounds__(256) k_sprites_list(RSegments<P> g, RTiles T, uint32_t per,
                                                      unsigned long long* culled, RItem* items, uint32_t* n_items) {
    __shared__ uint32_t s_sum;
    const int t = blockIdx.x;
    if (t == T.nt) return count_culled<P>(g, T.nt, T.accumulate, &s_sum, culled);
    const uint32_t total = tile_total<P>(g, T.nt, t, &s_sum);
    if (total) list_parts(t, total, per, items, n_items, &s_sum);
}

// 3. the listed parts, sprites.  Six waves per SIMD, three blocks of a CU's LDS
// (radius 2): at the 88 VGPRs it takes otherwise two fit (61 -> 69 us for
// 500,009 sprites).
template <typename R, int P, bool EXACT>
__global__ void __launch_bounds__(kRSprite, 6) k_sprites_draw(RSegments<P> g, RTiles T, uint32_t per,
                                                              Particles<R, P> pa, RenderArgs r, const RItem* items,
                                                              const uint32_t* n_items) {
    extern __shared__ __align__(16) char lds[];
    __shared__ uint32_t wsum[32];
    const uint32_t n = *n_items;
    const int m = r.radius > 0 ? 2 * (r.radius + 1) : 0;
    for (uint32_t k = blockIdx.x; k < n; k += gridDim.x) {  // uniform over the block
        const RItem it = items[k];
        // every part but the last is whole; the last ends with the entries
        sprite_tile<R, P, EXACT>(lds, wsum, g, T, (int)it.tile, per * it.part, per * (it.part + 1), pa, r);
        each_pixel((const uint32_t*)(lds + sizeof(SpriteList<EXACT>)), T, (int)it.tile, m, r,
                   [](uint32_t* d, uint32_t v) { if (v) atomicAdd(d, v); });
        __syncthreads();
    }
}

// Heavy sprites are drawn in double precision throughout (EXACT): in single
// precision many of their values are in doubt, and a wave takes the
// double-precision way, which projects the particle again, for any of its lanes
// (1M sprites of radius 4 in 1920 x 1080, single precision against this: weight 1
// 182 to 312 us, 8 319 to 308, 40 563 to 312; radius 1: weight 1 96 to 129, 12 126
// to 129, 20 138 to 128; points by index, weight 600: 8M 581 to 835).
bool exact_sprites(const RenderArgs& r) { return r.radius > 0 && r.weight > (r.radius > 1 ? 8.0 : 16.0); }

struct RLayout {
    bool tiled;      // the call uses scratch (and asks for `total` bytes of it)
    int payload, K;
    int ntx, ntiles, nblk;
    uint32_t per;    // entries a block takes of one tile
    size_t sorted, starts, items, n_items, total;
};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

RLayout rlayout(int64_t n, int width, int height, int radius, double weight, bool f64) {
    RLayout L{};
    const int64_t ntx = (width + kRTileW - 1) / kRTileW, nty = (height + kRTileH - 1) / kRTileH;
    const int64_t chunks = (n + kRChunk - 1) / kRChunk;
    L.tiled = n > 0 && n <= kRMaxN && radius <= kRMaxRadius && ntx * nty <= kRMaxTiles &&
              ntx * nty * chunks <= kRMaxCounts;
    if (!L.tiled) return L;
    L.ntx = (int)ntx;
    L.ntiles = (int)(ntx * nty);
    // what the call asks for does not depend on the payload and split below: 8
    // B per point, 20 per sprite, and 4 per tile and 4096 particles
    L.total = align256((size_t)n * 4) + align256((size_t)L.ntiles * (size_t)chunks * 4) +
              align256((size_t)L.ntiles * 4) + 2 * align256((size_t)(L.ntiles + 1) * 4) +
              align256((size_t)(radius == 0 ? n : 4 * n) * 4);
    auto lay_out = [&](int payload, int K) {
        L.payload = payload;
        L.K = K;
        const int64_t C = (int64_t)kRSort * L.K;
        L.nblk = (int)((n + C - 1) / C);
        // an evenly filled tile stays whole; sprites cost enough to be split finely
        const int64_t least = payload >= kCoords ? 768 : payload == kPack64 && K == 8 ? 12288 : 8192;
        L.per = (uint32_t)std::max<int64_t>(least, 5 * n / (payload >= kCoords ? 4096 : 2048));
        const int size = payload == kCoords ? 12 : payload == kPack64 ? 8 : 4;
        L.sorted = 0;
        L.starts = align256((size_t)n * size);
        L.items = L.starts + ((size_t)L.nblk * (L.ntiles + 2) * 2 + 3) / 4 * 4;
        // at most: each of the listed tiles, of points those over-full, one more
        // than its share of n / per
        const int64_t whole = n / L.per;
        const int64_t parts =
            payload >= kCoords ? std::min<int64_t>(n, whole + L.ntiles) : whole + std::min<int64_t>(whole, L.ntiles);
        L.n_items = L.items + (size_t)parts * sizeof(RItem);
        return L.n_items + 4 + 16 <= L.total;  // 16: room to align the buffers
    };
    // Particles per thread: one block for each of the 256 CUs while the ensemble
    // is too small to fill them otherwise, and few segments (short columns of
    // starts) beyond; bounded by the LDS that sorts them.  Points of eight bytes
    // take twice as many where the starts of more segments would pass the size
    // above, on images of one or two tiles.  A point's largest colour value is
    // that of rgb = 1.
    const int64_t full = 256 * (int64_t)kRSort;
    const double top = std::rint(256.0 * weight);
    const int few = n <= full && L.ntiles <= 2048 ? 1 : 4;
    if (radius == 0 && top <= 127.0 && lay_out(kPack32, n <= full ? 1 : n <= 4 * full ? 4 : 8)) return L;
    if (radius == 0 && top <= 131071.0 && (lay_out(kPack64, 4) || lay_out(kPack64, 8))) return L;
    if (radius > 0 && !f64 && lay_out(kCoords, few)) return L;
    (void)lay_out(kIndex, few);
    return L;
}

struct Target {
    uint32_t* img;
    unsigned long long* culled;
    bool accumulate;
    hipStream_t st;
};

template <typename R, int P>
hipError_t partition(const R* a0, const R* a1, const R* a2, int64_t n, const RenderArgs& r, const RLayout& L, char* ws,
                     const Target& to) {
    auto* sorted = (typename Entry<P>::T*)(ws + L.sorted);
    auto* starts = (uint16_t*)(ws + L.starts);
    auto* n_items = (uint32_t*)(ws + L.n_items);
    const int64_t clear = P >= kCoords && !to.accumulate ? (int64_t)r.width * r.height * 3 : 0;
    // a block for every 64 KB to clear: 10 sprites on a 3840 x 2160 image take
    // 27 us, and 850 with the one block that has particles
    const dim3 grid((unsigned)std::max<int64_t>(L.nblk, std::min<int64_t>(1024, clear / (16 * kRSort)))), block(kRSort);
    if (L.K == 1)
        hipLaunchKernelGGL((k_render_partition<R, 1, P>), grid, block, 0, to.st, a0, a1, a2, n, r, L.ntx, L.ntiles,
                           sorted, starts, n_items, to.img, clear);
    else if (L.K == 4)
        hipLaunchKernelGGL((k_render_partition<R, 4, P>), grid, block, 0, to.st, a0, a1, a2, n, r, L.ntx, L.ntiles,
                           sorted, starts, n_items, to.img, clear);
    else if constexpr (P == kPack32 || P == kPack64)
        hipLaunchKernelGGL((k_render_partition<R, 8, P>), grid, block, 0, to.st, a0, a1, a2, n, r, L.ntx, L.ntiles,
                           sorted, starts, n_items, to.img, clear);
    return hipGetLastError();
}

template <typename R, int P>
hipError_t run_tiles(const R* a0, const R* a1, const R* a2, int64_t n, const RenderArgs& r, const RLayout& L, char* ws,
                     const Target& to) {
    if (hipError_t e = partition<R, P>(a0, a1, a2, n, r, L, ws, to)) return e;
    const RSegments<P> g{(const typename Entry<P>::T*)(ws + L.sorted), (const uint16_t*)(ws + L.starts), L.nblk,
                         L.K * kRSort};
    const RTiles T{L.ntx, L.ntiles, to.accumulate, to.img};
    RItem* items = (RItem*)(ws + L.items);
    uint32_t* n_items = (uint32_t*)(ws + L.n_items);
    if constexpr (P >= kCoords) {
        const Particles<R, P> pa{a0, a1, a2, g.sorted};
        hipLaunchKernelGGL(k_sprites_list<P>, dim3(L.ntiles + 1), dim3(256), 0, to.st, g, T, L.per, to.culled, items,
                           n_items);
        if (hipError_t e = hipGetLastError()) return e;
        const unsigned grid = (unsigned)std::min<int64_t>(1024, n / L.per + L.ntiles);
        if (exact_sprites(r))
            hipLaunchKernelGGL((k_sprites_draw<R, P, true>), dim3(grid), dim3(kRSprite), sprite_lds<true>(r.radius),
                               to.st, g, T, L.per, pa, r, items, n_items);
        else
            hipLaunchKernelGGL((k_sprites_draw<R, P, false>), dim3(grid), dim3(kRSprite), sprite_lds<false>(r.radius),
                               to.st, g, T, L.per, pa, r, items, n_items);
    } else {
        hipLaunchKernelGGL((k_points_accum<P>), dim3(L.ntiles + 1), dim3(kRSort), 0, to.st, g, T, L.per, r, to.culled,
                           items, n_items);
        if (hipError_t e = hipGetLastError()) return e;
        if (n <= L.per) return hipSuccess;  // no tile can be over-full
        const unsigned grid = (unsigned)std::min<int64_t>(512, 2 * n / L.per + 1);
        hipLaunchKernelGGL((k_points_split<P>), dim3(grid), dim3(kRSort), 0, to.st, g, T, L.per, r, items, n_items);
    }
    return hipGetLastError();
}

template <typename R>
hipError_t run_render(const R* a0, const R* a1, const R* a2, int64_t n, const RenderArgs& r, const RLayout& L,
                      char* ws, const Target& to) {
    if (!L.tiled || (r.radius == 0 && n <= kRDirectMax)) {
        if (!to.accumulate) {
            const int64_t len = (int64_t)r.width * r.height * 3;
            const int64_t blocks = std::min<int64_t>((len + 1023) / 1024, 2048);
            hipLaunchKernelGGL(k_clear_img, dim3((unsigned)blocks), dim3(1024), 0, to.st, to.img, len, to.culled);
            if (hipError_t e = hipGetLastError()) return e;
        }
        if (n == 0) return hipSuccess;
        const unsigned grid = (unsigned)((n + 255) / 256);
        hipLaunchKernelGGL((k_render<R>), dim3(grid), dim3(256), 0, to.st, a0, a1, a2, n, r, to.img, to.culled);
        return hipGetLastError();
    }
    ws += (16 - ((uintptr_t)ws & 15)) & 15;  // the 16-byte loads; a caller's workspace may have any alignment
    switch (L.payload) {
        case kPack32: return run_tiles<R, kPack32>(a0, a1, a2, n, r, L, ws, to);
        case kPack64: return run_tiles<R, kPack64>(a0, a1, a2, n, r, L, ws, to);
        case kCoords:
            if constexpr (sizeof(R) == sizeof(float)) return run_tiles<R, kCoords>(a0, a1, a2, n, r, L, ws, to);
            return hipErrorInvalidValue;
        default: return run_tiles<R, kIndex>(a0, a1, a2, n, r, L, ws, to);
    }
}

ff_status check_render(const ff_render* r) {
    if (!r) return fail(FF_E_INVALID, "render description is NULL");
    if (r->width <= 0 || r->height <= 0) return fail(FF_E_INVALID, "image size must be positive");
    if ((int64_t)r->width * r->height > (int64_t)1 << 28) return fail(FF_E_UNSUPPORTED, "image larger than 2^28 pixels");
    if (r->radius < 0 || r->radius > 64) return fail(FF_E_INVALID, "sprite radius must be in [0, 64]");
    return FF_OK;
}

}  // namespace

}  // namespace ff

using namespace ff;

extern "C" {

ff_status ff_render_workspace_size(int64_t n, const ff_render* r, size_t* bytes) {
    set_error("");
    if (!bytes) return fail(FF_E_INVALID, "bytes is NULL");
    if (n < 0) return fail(FF_E_INVALID, "n < 0");
    if (ff_status s = check_render(r)) return s;
    const RLayout L = rlayout(n, r->width, r->height, r->radius, 1.0, false);
    *bytes = L.tiled ? L.total : 0;
    return FF_OK;
}

ff_status ff_render_image(ff_system_t sys, const ff_batch* b, const ff_render* r, uint32_t* img,
                          uint64_t* n_culled, int32_t accumulate, void* workspace, size_t workspace_bytes,
                          void* stream) {
    set_error("");
    if (ff_status s = check_system(sys)) return s;
    if (ff_status s = check_batch(sys, b, false)) return s;
    if (ff_status s = check_render(r)) return s;
    if (b->n > 0 && !b->state) return fail(FF_E_INVALID, "batch.state is NULL");
    auto axis_ok = [&](int a) { return (a >= 0 && a < sys->dim) || (a < 0 && -1 - a < b->n_pp); };
    for (int i = 0; i < 3; ++i)
        if (!axis_ok(r->axis[i])) return fail(FF_E_INVALID, "render axis must be a state component or -1 - k");
    for (int k = 0; k < 16; ++k)
        if (!std::isfinite(r->mvp[k])) return fail(FF_E_INVALID, "matrix entries must be finite");
    if (!std::isfinite(r->weight) || r->weight < 0.0) return fail(FF_E_INVALID, "weight must be finite and >= 0");
    if (!img) return fail(FF_E_INVALID, "img is NULL");
    hipStream_t st = (hipStream_t)stream;
    RenderArgs a;
    for (int i = 0; i < 3; ++i) a.axis[i] = r->axis[i];
    for (int k = 0; k < 16; ++k) a.mvp[k] = r->mvp[k];
    a.width = r->width;
    a.height = r->height;
    for (int k = 0; k < 3; ++k) {
        a.base[k] = r->base[k];
        a.origin[k] = r->origin[k];
    }
    for (int k = 0; k < 9; ++k) a.grad[k] = r->grad[k];
    a.weight = r->weight;
    a.radius = r->radius;
    const RLayout L = rlayout(b->n, r->width, r->height, r->radius, r->weight, b->prec == FF_FP64);
    char* ws = nullptr;
    if (L.tiled) {
        if (workspace) {
            if (workspace_bytes < L.total)
                return fail(FF_E_NOMEM, "render workspace too small: need " + std::to_string(L.total) + " bytes");
            ws = (char*)workspace;
        } else {
            void* p = nullptr;
            if (ff_status s = library_scratch(kScratchRender, L.total, st, &p)) return s;
            ws = (char*)p;
        }
    }
    unsigned long long* cu = (unsigned long long*)n_culled;
    const size_t esz = prec_size(b->prec);
    auto col = [&](int ax) -> const char* {
        return ax >= 0 ? (const char*)b->state + (size_t)ax * b->ld * esz
                       : (const char*)b->pparams + (size_t)(-1 - ax) * b->ld * esz;
    };
    const Target to{img, cu, accumulate != 0, st};
    hipError_t e;
    if (b->prec == FF_FP64)
        e = run_render<double>((const double*)col(r->axis[0]), (const double*)col(r->axis[1]),
                               (const double*)col(r->axis[2]), b->n, a, L, ws, to);
    else
        e = run_render<float>((const float*)col(r->axis[0]), (const float*)col(r->axis[1]),
                              (const float*)col(r->axis[2]), b->n, a, L, ws, to);
    if (e != hipSuccess) return device_fail(e, "ff_render_image launch");
    return FF_OK;
}

}  // extern "C"
