// ff_hist.hip — 2D density projection (Appendix A "Render Technique" and
// Appendix A.1: each particle is a unit-weight point added into the pixel it
// projects to), as exact uint32 counts.
//
// Binning, in double precision whatever the state precision (float values
// convert exactly): vx = (a - x_lo) * sx with sx = nx / (x_hi - x_lo) formed
// on the host; kept iff 0 <= vx < nx and 0 <= vy < ny (NaN fails); bin =
// floor(vy) * nx + floor(vx).
//
// The grids of interest (512^2 and 1024^2 uint32 = 1-4 MB) are far larger
// than one CU's 160 KB of LDS, and particle order in memory is random with
// respect to bins.  Large grids therefore go in two passes over square tiles of
// 32 to 128 bins a side:
//   1. partition: a block bins its particles, sorts their 16-bit indices
//      within the tile by tile in LDS and writes them to its own segment of
//      `sorted`, with the start of every tile in it; it also clears its share
//      of the grid
//   2. accumulate: one block owns a tile, gathers the tile's runs from all
//      segments into an LDS histogram and stores its non-zero bins (or adds
//      them, atomically, to an accumulated grid).  A tile
//      that holds more than a block's share of the particles is listed instead
//      and split over blocks of a third launch, which add theirs with atomics.
// Square tiles keep an attractor, a curve on the grid, spread over many
// tiles; rows of bins would put its flat stretches into one.  HBM traffic per
// particle: read 2 coordinates, write and read 2 B; plus the grid.  8,388,608
// settled Lorenz particles on a 1024 x 1024 (r, y) grid: 146 -> 66 us
// (partition 33, accumulate 15, split 13), of which reading the coordinates at
// the 4.6 TB/s of a large copy is 15; a counting sort over the whole grid
// (count, two scans, scatter, accumulate in chunks of 8192 merged by atomics)
// took the 146.  All three wait (69-75 % of their waves' time): the partition
// for the LDS atomics that return a particle's rank, which take turns in a
// skewed ensemble's tiles (23 us when uniform), the others for short loads.
// Ensembles of at most kDirectMax particles add straight to the grid with
// global atomics, and grids of at most 16384 bins use one LDS histogram per
// block over a stride of particles.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <vector>

#include "ff_internal.h"
#include "ff_scan.h"

namespace ff {

namespace {

constexpr uint32_t kSmallBins = 1u << 14;        // one LDS histogram (64 KB)
constexpr int kBlock = 256;
constexpr int64_t kChunk = 4096;                 // particles that make one more block of the small path worth it
constexpr int kMaxTiles = 4096;                         // grids up to 64M bins
constexpr int kSort = 1024;                             // threads of the partition and accumulate blocks
constexpr int kMaxItems = 1024;                         // splits of over-full tiles (at most 2 * 1024 / 5 arise)
constexpr int64_t kDirectMax = 8192;
constexpr int64_t kMaxBins = (int64_t)kMaxTiles << 14;
constexpr uint32_t kNone = 0xFFFFFFFFu;

struct Geom {
    double xlo, ylo, sx, sy;
    int nx, ny;
};

// Tiles of 2^tw x 2^th bins, ntx of them in a row.  With `linear` the grid is
// taken as one row of nx * ny bins.
struct Tiling {
    int bits;  // tw + th: 10, 12 or 14
    int tw, th, ntx, ntiles;
    bool linear;
};

// Tiles small enough to give each of the 256 CUs one (512^2 bins: 256 of 32 x
// 32; 1024^2: 256 of 64 x 64) and large enough to be at most 1024 (then runs
// of a segment stay long), up to 128 x 128 (64 KB of LDS); runs of 16384 bins
// for grids whose shape leaves too much of the square tiles empty.
Tiling tiling(int nx, int ny) {
    for (int w = 5; w <= 7; ++w) {
        const int64_t tx = (nx + (1 << w) - 1) >> w, t = tx * ((ny + (1 << w) - 1) >> w);
        if (t <= (w == 5 ? 320 : w == 6 ? 1024 : kMaxTiles)) return {2 * w, w, w, (int)tx, (int)t, false};
    }
    const int64_t t = ((int64_t)nx * ny + 16383) >> 14;
    return {14, 14, 0, (int)t, (int)t, true};
}

// Entries a block takes of one tile: a little more than the share of one of
// 256 CUs, so that evenly filled tiles stay whole, and enough to be worth
// merging a tile's bins with atomics.
int64_t per_split(int64_t n, const Tiling& t) { return std::max<int64_t>((int64_t)4 << t.bits, 5 * n / 1024); }

// The cell a particle falls in; false where it is dropped.
template <typename R>
__device__ __forceinline__ bool cell_of(R a, R b, const Geom& g, uint32_t& ix, uint32_t& iy) {
    const double vx = ((double)a - g.xlo) * g.sx;
    const double vy = ((double)b - g.ylo) * g.sy;
    const bool ok = (vx >= 0.0) && (vx < (double)g.nx) && (vy >= 0.0) && (vy < (double)g.ny);
    ix = (uint32_t)(int)(ok ? vx : 0.0);
    iy = (uint32_t)(int)(ok ? vy : 0.0);
    return ok;
}

template <typename R>
__device__ __forceinline__ uint32_t bin_of(R a, R b, const Geom& g) {
    uint32_t ix, iy;
    return cell_of<R>(a, b, g, ix, iy) ? iy * (uint32_t)g.nx + ix : kNone;
}

// Tile (high bits) and index within the tile (low `bits`) of a kept cell.
__device__ __forceinline__ uint32_t tile_code(uint32_t ix, uint32_t iy, const Geom& g, const Tiling& t) {
    if (t.linear) return iy * (uint32_t)g.nx + ix;
    const uint32_t tile = (iy >> t.th) * (uint32_t)t.ntx + (ix >> t.tw);
    const uint32_t local = ((iy & ((1u << t.th) - 1)) << t.tw) | (ix & ((1u << t.tw) - 1));
    return (tile << t.bits) | local;
}

__global__ void k_fill(uint32_t* hist, int64_t nbins, unsigned long long* dropped) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t k = i; k < nbins; k += stride) hist[k] = 0u;
    if (i == 0 && dropped) *dropped = 0ull;
}

__device__ __forceinline__ void add_drops(unsigned long long* dropped, unsigned int mine,
                                          unsigned int* s_drop) {
    if (!dropped) return;
    if (mine) atomicAdd(s_drop, mine);
    __syncthreads();
    if (threadIdx.x == 0 && *s_drop) atomicAdd(dropped, (unsigned long long)*s_drop);
}

// Grids of <= kSmallBins bins: LDS histogram per block, grid-stride over
// particles.  Every block adds its non-zero bins to the grid, so there are no
// more than one per CU.
template <typename R>
__global__ void __launch_bounds__(kSort) k_hist_small(const R* ax, const R* ay, int64_t n, Geom g,
                                                       uint32_t* hist, unsigned long long* dropped) {
    __shared__ uint32_t s[kSmallBins];
    __shared__ unsigned int s_drop;
    const uint32_t nbins = (uint32_t)g.nx * (uint32_t)g.ny;
    for (uint32_t k = threadIdx.x; k < nbins; k += blockDim.x) s[k] = 0u;
    if (threadIdx.x == 0) s_drop = 0u;
    __syncthreads();
    unsigned int drops = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint32_t b = bin_of<R>(ax[i], ay[i], g);
        if (b != kNone) atomicAdd(&s[b], 1u);
        else ++drops;
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < nbins; k += blockDim.x)
        if (s[k]) atomicAdd(&hist[k], s[k]);
    add_drops(dropped, drops, &s_drop);
}

// Few particles: one global atomic each.
template <typename R>
__global__ void __launch_bounds__(kBlock) k_hist_direct(const R* ax, const R* ay, int64_t n, Geom g, uint32_t* hist,
                                                        unsigned long long* dropped) {
    __shared__ unsigned int s_drop;
    if (threadIdx.x == 0) s_drop = 0u;
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned int drops = 0;
    if (i < n) {
        const uint32_t b = bin_of<R>(ax[i], ay[i], g);
        if (b != kNone) (void)count_one(hist, b);
        else drops = 1;
    }
    add_drops(dropped, drops, &s_drop);
}

// 1. partition: K particles per thread
template <typename R, int K>
__global__ void __launch_bounds__(kSort) k_hist_partition(const R* ax, const R* ay, int64_t n, Geom g, Tiling tl,
                                                          uint16_t* sorted, uint16_t* starts, uint32_t* hist,
                                                          int64_t clear, uint32_t* n_items) {
    constexpr int C = kSort * K;
    __shared__ uint32_t cnt[kMaxTiles];
    __shared__ __align__(4) uint16_t stage[C];
    __shared__ uint32_t wsum[32];
    const int tid = threadIdx.x, nt = tl.ntiles;
    for (int64_t k = (int64_t)blockIdx.x * kSort + tid; k < clear; k += (int64_t)gridDim.x * kSort) hist[k] = 0u;
    const int64_t lo = (int64_t)blockIdx.x * C;
    if (lo >= n) return;  // the whole block
    for (int t = tid; t < nt; t += kSort) cnt[t] = 0u;
    __syncthreads();
    uint32_t code[K], rank[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t i = lo + k * kSort + tid;
        code[k] = kNone;
        if (i < n) {
            uint32_t ix, iy;
            if (cell_of<R>(ax[i], ay[i], g, ix, iy)) code[k] = tile_code(ix, iy, g, tl);
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (code[k] != kNone) rank[k] = count_one(cnt, code[k] >> tl.bits);
    __syncthreads();
    // exclusive scan of the counts, four tiles per thread
    uint32_t c[4], sum = 0, kept;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        c[j] = 4 * tid + j < nt ? cnt[4 * tid + j] : 0u;
        sum += c[j];
    }
    uint32_t at = block_scan(sum, wsum, &kept);
    uint16_t* row = starts + (int64_t)blockIdx.x * (nt + 1);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (4 * tid + j < nt) {
            cnt[4 * tid + j] = at;
            row[4 * tid + j] = (uint16_t)at;
            at += c[j];
        }
    }
    if (tid == 0) row[nt] = (uint16_t)kept;
    if (tid == 0 && blockIdx.x == 0) *n_items = 0u;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (code[k] != kNone) stage[cnt[code[k] >> tl.bits] + rank[k]] = (uint16_t)(code[k] & ((1u << tl.bits) - 1));
    __syncthreads();
    // lo is even: pairs are aligned (the last may end one entry past the kept
    // ones, inside the buffer's alignment)
    uint32_t* dst = (uint32_t*)(sorted + lo);
    const uint32_t* src = (const uint32_t*)stage;
    for (uint32_t j = tid; j < (kept + 1) / 2; j += kSort) dst[j] = src[j];
}

// The sorted particles and what describes their order.
struct Segments {
    const uint16_t* sorted;  // segment b from b * C
    const uint16_t* starts;  // [nblk][ntiles + 1], within the segment
    int nblk, C;
};

// Entries of tile t in segments b0 .. b1 - 1, counted by the whole block.
__device__ __forceinline__ uint64_t tile_total(const Segments& g, int nt, int t, int b0, int b1, uint64_t* s_sum) {
    if (threadIdx.x == 0) *s_sum = 0ull;
    __syncthreads();
    unsigned long long mine = 0;
    for (int b = b0 + (int)threadIdx.x; b < b1; b += kSort) {
        const uint16_t* r = g.starts + (int64_t)b * (nt + 1) + t;
        mine += (uint32_t)r[1] - r[0];
    }
    for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off, 64);
    if ((threadIdx.x & 63) == 0 && mine) atomicAdd((unsigned long long*)s_sum, mine);
    __syncthreads();
    return *s_sum;
}

// LDS histogram of tile t's runs in segments b0 .. b1 - 1: LANES threads (16
// or more) take a run, four entries each at a time (8-byte loads; what lies
// before or after the run in them is masked).
template <int BITS, int LANES>
__device__ __forceinline__ void gather_tile(uint32_t* s, const Segments& g, int nt, int t, int b0, int b1) {
    for (int k = threadIdx.x; k < 1 << BITS; k += kSort) s[k] = 0u;
    __syncthreads();
    constexpr int kGroups = kSort / LANES;
    const int lane = threadIdx.x % LANES;
    for (int base = b0 + (int)(threadIdx.x / LANES); base < b1; base += 16 * kGroups) {
        // 16 lanes load the bounds of the group's next 16 runs
        const int mine = base + (int)(threadIdx.x & 15) * kGroups;
        uint32_t lo = 0, hi = 0;
        if (mine < b1) {
            const uint16_t* r = g.starts + (int64_t)mine * (nt + 1) + t;
            lo = r[0];
            hi = r[1];
        }
#pragma unroll 4
        for (int q = 0; q < 16; ++q) {
            const uint32_t beg = __shfl(lo, q, 16), end = __shfl(hi, q, 16);
            const uint16_t* e = g.sorted + (int64_t)(base + q * kGroups) * g.C;
            for (uint32_t j = (beg & ~3u) + 4 * lane; j < end; j += 4 * LANES) {
                const ushort4 v = *(const ushort4*)(e + j);
                if (j >= beg && j + 3 < end) {
                    // lanes that all hold one bin (an ensemble on a fixed
                    // point) would be served one by one: add their number
                    const uint32_t first = __builtin_amdgcn_readfirstlane(v.x);
                    if (__ballot(v.x != first || v.y != first || v.z != first || v.w != first) == 0) {
                        const uint64_t live = __ballot(1);
                        if ((threadIdx.x & 63) == (unsigned)__builtin_ctzll(live))
                            atomicAdd(&s[first], 4u * (uint32_t)__popcll(live));
                    } else {
                        atomicAdd(&s[v.x], 1u);
                        atomicAdd(&s[v.y], 1u);
                        atomicAdd(&s[v.z], 1u);
                        atomicAdd(&s[v.w], 1u);
                    }
                } else {
                    if (j >= beg) atomicAdd(&s[v.x], 1u);
                    if (j + 1 >= beg && j + 1 < end) atomicAdd(&s[v.y], 1u);
                    if (j + 2 >= beg && j + 2 < end) atomicAdd(&s[v.z], 1u);
                    if (j + 3 >= beg && j + 3 < end) atomicAdd(&s[v.w], 1u);
                }
            }
        }
    }
    __syncthreads();
}

// Hand every non-zero bin of tile t to put(address, count).
template <int BITS, class F>
__device__ __forceinline__ void merge_tile(const uint32_t* s, const Geom& g, const Tiling& tl, int t, uint32_t* hist,
                                           F put) {
    const int64_t nx = tl.linear ? (int64_t)g.nx * g.ny : g.nx, ny = tl.linear ? 1 : g.ny;
    const int64_t X0 = (int64_t)(t % tl.ntx) << tl.tw, Y0 = (int64_t)(t / tl.ntx) << tl.th;
    for (int k = threadIdx.x; k < 1 << BITS; k += kSort) {
        const int64_t x = X0 + (k & ((1 << tl.tw) - 1)), y = Y0 + (k >> tl.tw);
        if (s[k] && x < nx && y < ny) put(hist + y * nx + x, s[k]);
    }
}

// A part of an over-full tile.
struct Item {
    int32_t tile, part, parts;
};

// 2. accumulate: block t owns tile t; the last block counts the drops
template <int BITS>
__global__ void __launch_bounds__(kSort) k_hist_accum(Segments sg, int64_t n, int64_t per, Geom g, Tiling tl,
                                                      uint32_t* hist, unsigned long long* dropped, bool accumulate,
                                                      Item* items, uint32_t* n_items) {
    __shared__ uint32_t s[1 << BITS];
    __shared__ uint64_t s_sum;
    const int nt = tl.ntiles, t = blockIdx.x;
    if (t == nt) {
        if (!dropped) return;
        // n less the kept of every segment: the starts' last column against 0
        unsigned long long kept = 0;
        if (threadIdx.x == 0) s_sum = 0ull;
        __syncthreads();
        for (int b = threadIdx.x; b < sg.nblk; b += kSort) kept += sg.starts[(int64_t)b * (nt + 1) + nt];
        if (kept) atomicAdd((unsigned long long*)&s_sum, kept);
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned long long drops = (unsigned long long)n - s_sum;
            if (accumulate) atomicAdd(dropped, drops);
            else *dropped = drops;
        }
        return;
    }
    const int64_t total = (int64_t)tile_total(sg, nt, t, 0, sg.nblk, &s_sum);
    if (total == 0) return;
    if (total > per) {
        const int parts = (int)((total + per - 1) / per);
        if (threadIdx.x == 0) {
            const uint32_t at = atomicAdd(n_items, (uint32_t)parts);
            for (int k = 0; k < parts; ++k) items[at + k] = {t, k, parts};
        }
        return;
    }
    gather_tile<BITS, 16>(s, sg, nt, t, 0, sg.nblk);
    // what is added to the caller's grid is added atomically: calls on several
    // streams may add to one grid
    if (accumulate) merge_tile<BITS>(s, g, tl, t, hist, [](uint32_t* d, uint32_t v) { atomicAdd(d, v); });
    else merge_tile<BITS>(s, g, tl, t, hist, [](uint32_t* d, uint32_t v) { *d = v; });
}

// 3. the listed parts of over-full tiles
template <int BITS>
__global__ void __launch_bounds__(kSort) k_hist_split(Segments sg, int64_t per, Geom g, Tiling tl, uint32_t* hist,
                                                      const Item* items, const uint32_t* n_items) {
    __shared__ uint32_t s[1 << BITS];
    const uint32_t m = *n_items;
    for (uint32_t k = blockIdx.x; k < m; k += gridDim.x) {  // uniform over the block
        const Item it = items[k];
        const int b0 = (int)((int64_t)sg.nblk * it.part / it.parts);
        const int b1 = (int)((int64_t)sg.nblk * (it.part + 1) / it.parts);
        // an ensemble in few tiles leaves few, long runs: the whole block
        // takes each (8M particles in one bin: 149 -> 45 us in all)
        if (it.parts * per > 2048ll * sg.nblk) gather_tile<BITS, kSort>(s, sg, tl.ntiles, it.tile, b0, b1);
        else gather_tile<BITS, 16>(s, sg, tl.ntiles, it.tile, b0, b1);
        merge_tile<BITS>(s, g, tl, it.tile, hist, [](uint32_t* d, uint32_t v) { atomicAdd(d, v); });
        __syncthreads();
    }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Scratch of the two-pass path: per block of C particles its sorted indices
// and the starts of its tiles, and the list of over-full tiles' parts.  C =
// 1024 K: one or two blocks for each of the 256 CUs while the ensemble is too
// small to fill them with 16 particles a thread (1.5M particles: K = 16 37 us,
// K = 4 30; 4M: K = 4 43, K = 16 38).
struct WsLayout {
    int K, nblk;
    size_t sorted, starts, items, n_items, total;
};

WsLayout layout(int64_t n, int nx, int ny) {
    WsLayout L{};
    const int64_t nbins = (int64_t)nx * ny;
    if (nbins <= (int64_t)kSmallBins) return L;
    const Tiling t = tiling(nx, ny);
    const int64_t full = 256 * (int64_t)kSort;
    L.K = t.ntiles > 1024 ? 16 : n <= full ? 1 : n <= 8 * full ? 4 : n <= 16 * full ? 8 : 16;
    const int64_t C = (int64_t)kSort * L.K;
    L.nblk = (int)((n + C - 1) / C);
    L.sorted = 0;
    L.starts = align256((size_t)n * 2);
    L.items = L.starts + align256((size_t)L.nblk * (t.ntiles + 1) * 2);
    L.n_items = L.items + (n > per_split(n, t) ? align256(kMaxItems * sizeof(Item)) : 0);
    // what the call asks for does not depend on the split above: 6 B per
    // particle, and 4 B per tile of 16384 bins and 4096 particles.  The buffers
    // above end at least a fifth before it wherever they are used (more than
    // kDirectMax particles), which leaves room to align them.
    const int64_t ntiles = (nbins + 16383) / 16384, nblk = (n + kChunk - 1) / kChunk;
    L.total = align256((size_t)n * 4) + align256((size_t)n * 2) + align256((size_t)ntiles * (size_t)nblk * 4) +
              align256((size_t)ntiles * 4) + 2 * align256((size_t)(ntiles + 1) * 4);
    return L;
}

template <typename R, int K>
void launch_partition(const R* ax, const R* ay, int64_t n, const Geom& g, const Tiling& t, const WsLayout& L,
                      char* ws, uint32_t* hist, int64_t clear, hipStream_t st) {
    // a block for every 64 KB to clear: 9,000 particles on a 4096 x 4096 grid
    // take 29 us, and 84 with the blocks that have particles
    const unsigned grid = (unsigned)std::max<int64_t>(L.nblk, std::min<int64_t>(1024, clear / (16 * kSort)));
    hipLaunchKernelGGL((k_hist_partition<R, K>), dim3(grid), dim3(kSort), 0, st, ax, ay, n, g, t,
                       (uint16_t*)(ws + L.sorted), (uint16_t*)(ws + L.starts), hist, clear,
                       (uint32_t*)(ws + L.n_items));
}

template <int BITS>
hipError_t launch_accumulate(int64_t n, const Geom& g, const Tiling& t, const WsLayout& L, char* ws, uint32_t* hist,
                             unsigned long long* dropped, bool accumulate, hipStream_t st) {
    const Segments sg{(const uint16_t*)(ws + L.sorted), (const uint16_t*)(ws + L.starts), L.nblk, L.K * kSort};
    Item* items = (Item*)(ws + L.items);
    uint32_t* n_items = (uint32_t*)(ws + L.n_items);
    const int64_t per = per_split(n, t);
    hipLaunchKernelGGL(k_hist_accum<BITS>, dim3(t.ntiles + 1), dim3(kSort), 0, st, sg, n, per, g, t, hist, dropped,
                       accumulate, items, n_items);
    if (hipError_t e = hipGetLastError()) return e;
    if (n <= per) return hipSuccess;  // no tile can be over-full
    const unsigned grid = (unsigned)std::min<int64_t>(512, 2 * n / per);
    hipLaunchKernelGGL(k_hist_split<BITS>, dim3(grid), dim3(kSort), 0, st, sg, per, g, t, hist, items, n_items);
    return hipGetLastError();
}

template <typename R>
hipError_t run_hist(const R* ax, const R* ay, int64_t n, const Geom& g, uint32_t* hist,
                    unsigned long long* dropped, bool accumulate, char* ws, hipStream_t st) {
    const int64_t nbins = (int64_t)g.nx * g.ny;
    const bool small = nbins <= (int64_t)kSmallBins;
    const bool two_pass = !small && n > kDirectMax;
    if (!accumulate && !two_pass) {
        const int64_t blocks = std::min<int64_t>((nbins + 1023) / 1024, 2048);
        hipLaunchKernelGGL(k_fill, dim3((unsigned)std::max<int64_t>(blocks, 1)), dim3(1024), 0, st, hist,
                           nbins, dropped);
        if (hipError_t e = hipGetLastError()) return e;
    }
    if (n == 0) return hipSuccess;
    if (small) {
        const int64_t blocks = std::min<int64_t>((n + kChunk - 1) / kChunk, 256);
        hipLaunchKernelGGL((k_hist_small<R>), dim3((unsigned)blocks), dim3(kSort), 0, st, ax, ay, n, g, hist,
                           dropped);
        return hipGetLastError();
    }
    if (!two_pass) {
        hipLaunchKernelGGL((k_hist_direct<R>), dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, st, ax,
                           ay, n, g, hist, dropped);
        return hipGetLastError();
    }
    const WsLayout L = layout(n, g.nx, g.ny);
    const Tiling t = tiling(g.nx, g.ny);
    ws += (16 - ((uintptr_t)ws & 15)) & 15;  // the 8-byte loads; a caller's workspace may have any alignment
    const int64_t clear = accumulate ? 0 : nbins;
    if (L.K == 1) launch_partition<R, 1>(ax, ay, n, g, t, L, ws, hist, clear, st);
    else if (L.K == 4) launch_partition<R, 4>(ax, ay, n, g, t, L, ws, hist, clear, st);
    else if (L.K == 8) launch_partition<R, 8>(ax, ay, n, g, t, L, ws, hist, clear, st);
    else launch_partition<R, 16>(ax, ay, n, g, t, L, ws, hist, clear, st);
    if (hipError_t e = hipGetLastError()) return e;
    switch (t.bits) {
        case 10: return launch_accumulate<10>(n, g, t, L, ws, hist, dropped, accumulate, st);
        case 12: return launch_accumulate<12>(n, g, t, L, ws, hist, dropped, accumulate, st);
        default: return launch_accumulate<14>(n, g, t, L, ws, hist, dropped, accumulate, st);
    }
}

}  // namespace

namespace {

// A validated projection request: the geometry and the two axis columns.
struct Projection {
    Geom g;
    const void* ax;
    const void* ay;
    int64_t n;
    bool f64;
};

ff_status check_projection(const ff_system_s* sys, const ff_batch* b, int32_t axis_x, int32_t axis_y,
                           double x_lo, double x_hi, double y_lo, double y_hi, int32_t nx, int32_t ny,
                           const uint32_t* hist, Projection* out) {
    if (ff_status s = check_system(sys)) return s;
    if (ff_status s = check_batch(sys, b, false)) return s;
    if (b->n > 0 && !b->state) return fail(FF_E_INVALID, "batch.state is NULL");
    auto axis_ok = [&](int a) { return (a >= 0 && a < sys->dim) || (a < 0 && -1 - a < b->n_pp); };
    if (!axis_ok(axis_x) || !axis_ok(axis_y))
        return fail(FF_E_INVALID, "axis must be a state component (>= 0) or -1 - k for a per-particle parameter k");
    if (nx <= 0 || ny <= 0) return fail(FF_E_INVALID, "nx and ny must be positive");
    if ((int64_t)nx * ny > kMaxBins) return fail(FF_E_UNSUPPORTED, "grid larger than 64M bins");
    if (!std::isfinite(x_lo) || !std::isfinite(x_hi) || !std::isfinite(y_lo) || !std::isfinite(y_hi) ||
        !(x_hi > x_lo) || !(y_hi > y_lo))
        return fail(FF_E_INVALID, "ranges must be finite with hi > lo");
    if (!hist) return fail(FF_E_INVALID, "hist is NULL");
    if (b->n > 0x7fffffffLL) return fail(FF_E_UNSUPPORTED, "more than 2^31 - 1 particles in one projection");
    Geom g;
    g.xlo = x_lo;
    g.ylo = y_lo;
    g.sx = (double)nx / (x_hi - x_lo);
    g.sy = (double)ny / (y_hi - y_lo);
    if (!std::isfinite(g.sx) || !std::isfinite(g.sy)) return fail(FF_E_INVALID, "range too small");
    g.nx = nx;
    g.ny = ny;
    const size_t esz = prec_size(b->prec);
    auto col = [&](int a) -> const void* {
        return a >= 0 ? (const char*)b->state + (size_t)a * b->ld * esz
                      : (const char*)b->pparams + (size_t)(-1 - a) * b->ld * esz;
    };
    out->g = g;
    out->ax = col(axis_x);
    out->ay = col(axis_y);
    out->n = b->n;
    out->f64 = b->prec == FF_FP64;
    return FF_OK;
}

hipError_t run_projection(const Projection& P, uint32_t* hist, unsigned long long* dropped, bool accumulate,
                          char* ws, hipStream_t st) {
    if (P.f64)
        return run_hist<double>((const double*)P.ax, (const double*)P.ay, P.n, P.g, hist, dropped, accumulate, ws,
                                st);
    return run_hist<float>((const float*)P.ax, (const float*)P.ay, P.n, P.g, hist, dropped, accumulate, ws, st);
}

}  // namespace

// Scratch of ff_project_histogram_noalloc: a file-scope device array, one
// copy per GPU (at its own address), held from the library's load on that
// GPU until the process ends.  Every buffer in it is written before it is
// read within one call, so nothing needs clearing between calls.  Host code
// never passes the array's name to a kernel (on the host it is only a
// stand-in): the per-device address comes from hipGetSymbolAddress.
constexpr size_t kNoAllocBytes = (size_t)FF_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) char scratch[kNoAllocBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mu;
void* g_noalloc_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up on the first
// call on that device (no allocation, now or later).
ff_status noalloc_scratch(void** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return device_fail(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return fail(FF_E_UNSUPPORTED, "device index beyond 63");
    std::lock_guard<std::mutex> lk(g_noalloc_mu);
    if (!g_noalloc_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return device_fail(e, "hipGetSymbolAddress of the histogram's static scratch");
        if (!p) return fail(FF_E_DEVICE, "hipGetSymbolAddress returned a null address for the static scratch");
        g_noalloc_ptr[dev] = p;
    }
    *out = g_noalloc_ptr[dev];
    return FF_OK;
}

}  // namespace

namespace {
// Library-owned scratch per device and use (grown on demand, kept for the
// process).
struct Scratch {
    void* ptr = nullptr;
    size_t bytes = 0;
};
std::mutex g_scratch_mu;
std::vector<Scratch> g_scratch[kScratchUses];
}  // namespace

ff_status library_scratch(int use, size_t need, hipStream_t stream, void** out) {
    static const char* const kWhat[kScratchUses] = {"histogram", "render"};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return device_fail(e, "hipGetDevice");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    std::vector<Scratch>& per_dev = g_scratch[use];
    if ((int)per_dev.size() <= dev) per_dev.resize(dev + 1);
    Scratch& s = per_dev[dev];
    if (s.bytes < need) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(stream, &cs) == hipSuccess && cs != hipStreamCaptureStatusNone)
            return fail(FF_E_NOMEM, std::string(kWhat[use]) + " scratch must be passed as `workspace` under stream capture");
        if (s.ptr) {
            e = hipStreamSynchronize(stream);
            if (e != hipSuccess) return device_fail(e, "hipStreamSynchronize");
            (void)hipFree(s.ptr);
            s.ptr = nullptr;
            s.bytes = 0;
        }
        e = hipMalloc(&s.ptr, need);
        if (e != hipSuccess) {
            s.ptr = nullptr;
            return fail(FF_E_NOMEM, std::string("hipMalloc of ") + kWhat[use] + " scratch: " + hipGetErrorString(e));
        }
        s.bytes = need;
    }
    *out = s.ptr;
    return FF_OK;
}

}  // namespace ff

using namespace ff;

extern "C" {

ff_status ff_histogram_workspace_size(int64_t n, int32_t nx, int32_t ny, size_t* bytes) {
    set_error("");
    if (!bytes) return fail(FF_E_INVALID, "bytes is NULL");
    if (n < 0 || nx <= 0 || ny <= 0) return fail(FF_E_INVALID, "n < 0 or grid size <= 0");
    const int64_t nbins = (int64_t)nx * ny;
    if (nbins > kMaxBins) return fail(FF_E_UNSUPPORTED, "grid larger than 64M bins");
    *bytes = layout(n, nx, ny).total;
    return FF_OK;
}

ff_status ff_project_histogram(ff_system_t sys, const ff_batch* b, int32_t axis_x, int32_t axis_y,
                               double x_lo, double x_hi, double y_lo, double y_hi, int32_t nx,
                               int32_t ny, uint32_t* hist, uint64_t* n_dropped, int32_t accumulate,
                               void* workspace, size_t workspace_bytes, void* stream) {
    set_error("");
    Projection P;
    if (ff_status s = check_projection(sys, b, axis_x, axis_y, x_lo, x_hi, y_lo, y_hi, nx, ny, hist, &P))
        return s;
    hipStream_t st = (hipStream_t)stream;
    const size_t need = layout(b->n, nx, ny).total;
    char* ws = nullptr;
    if (need > 0 && b->n > 0) {
        if (workspace) {
            if (workspace_bytes < need)
                return fail(FF_E_NOMEM, "histogram workspace too small: need " + std::to_string(need) + " bytes");
            ws = (char*)workspace;
        } else {
            void* p = nullptr;
            if (ff_status s = library_scratch(kScratchHistogram, need, st, &p)) return s;
            ws = (char*)p;
        }
    }
    const hipError_t e = run_projection(P, hist, (unsigned long long*)n_dropped, accumulate != 0, ws, st);
    if (e != hipSuccess) return device_fail(e, "ff_project_histogram launch");
    return FF_OK;
}

ff_status ff_project_histogram_noalloc(ff_system_t sys, const ff_batch* b, int32_t axis_x, int32_t axis_y,
                                       double x_lo, double x_hi, double y_lo, double y_hi, int32_t nx,
                                       int32_t ny, uint32_t* hist, uint64_t* n_dropped, int32_t accumulate,
                                       void* stream) {
    set_error("");
    Projection P;
    if (ff_status s = check_projection(sys, b, axis_x, axis_y, x_lo, x_hi, y_lo, y_hi, nx, ny, hist, &P))
        return s;
    const size_t need = layout(b->n, nx, ny).total;
    char* ws = nullptr;
    if (need > 0 && b->n > 0) {
        if (need > kNoAllocBytes)
            return fail(FF_E_NOMEM, "ff_project_histogram_noalloc: this projection needs " + std::to_string(need) +
                                        " bytes of scratch, more than the " + std::to_string(kNoAllocBytes) +
                                        " bytes its static buffer holds; use ff_project_histogram with a workspace");
        void* p = nullptr;
        if (ff_status s = noalloc_scratch(&p)) return s;
        ws = (char*)p;
    }
    const hipError_t e = run_projection(P, hist, (unsigned long long*)n_dropped, accumulate != 0, ws,
                                        (hipStream_t)stream);
    if (e != hipSuccess) return device_fail(e, "ff_project_histogram_noalloc launch");
    return FF_OK;
}

}  // extern "C"
