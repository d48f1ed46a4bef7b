// Mesh bounds, cell keys, counting sort into cell order, cell ranges.
//
// Cell-ordered numbering is the GPU form of the linked-list cells and the
// locality renumbering of sec. 4.2: a counting sort by cell key.  Keys are
// histogrammed with integer atomics (each particle also gets a provisional
// rank inside its cell), an exclusive scan of the histogram gives the cell
// ranges, a scatter places every particle in its cell's segment, and each
// particle's final place in the segment is the number of the segment's
// particles with a smaller input index, so the order is exactly the stable
// order by (key, input index) whatever order the atomics ran in.
#include "csph_internal.h"
#include "hostsync.h"
#include "wave.h"

namespace csph {

// Small sets (kSmallN particles at most; binning also fewer than kSmallKeys keys): one workgroup
// finds the bounds, and one bins, since at this size the chain of launches, ~4 us each, takes
// longer than the work.  A particle's place in its cell takes a look at each of the cell's others,
// n n / keys looks in an even set: the one workgroup bins up to kSmallLooks of them.  Ten
// binnings in a row, one workgroup against the launches: 8 192 particles at 24 a key 306 against
// 360 us, at 38 380 and 360; 12 000 at 9 304 and 380, at 23 415, at 35 516; 16 384 at 8 339 and 371,
// at 32 600; 4 096 at 64 292.
constexpr int kSmallBlock = 1024;
constexpr int kSmallPer = 16;  // particles and keys a thread
constexpr int kSmallN = kSmallPer * kSmallBlock;
constexpr int64_t kSmallLooks = 1 << 18;

// ---------------------------------------------------------------- reductions

// (a wave's reduction, every lane active: within rows of 16 lanes without LDS, whose six
// dependent exchanges a value were most of a reduction's time)
__device__ __forceinline__ double wave_min(double v) {
    v = fmin(v, row_ror<8>(v));
    v = fmin(v, row_ror<4>(v));
    v = fmin(v, row_ror<2>(v));
    v = fmin(v, row_ror<1>(v));
    v = fmin(v, __shfl_xor(v, 16, 64));
    return fmin(v, __shfl_xor(v, 32, 64));
}
__device__ __forceinline__ double wave_max(double v) { return -wave_min(-v); }

// The bounds of the thread's particles i0, i0 + stride, ... below n, U of them in flight.
template <int U>
__device__ __forceinline__ void thread_bounds(const double *__restrict__ x,
                                              const double *__restrict__ y,
                                              const double *__restrict__ z,
                                              const double *__restrict__ d, int64_t i0,
                                              int64_t stride, int64_t n, double (&v)[7]) {
    for (; i0 < n; i0 += U * stride) {
        double a[U], b[U], c[U], e[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {  // past the end: the thread's first particle again
            const int64_t i = i0 + q * stride < n ? i0 + q * stride : i0;
            a[q] = x[i];
            b[q] = y[i];
            c[q] = z[i];
            e[q] = d ? d[i] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            v[0] = fmin(v[0], a[q]); v[1] = fmin(v[1], b[q]); v[2] = fmin(v[2], c[q]);
            v[3] = fmax(v[3], a[q]); v[4] = fmax(v[4], b[q]); v[5] = fmax(v[5], c[q]);
            v[6] = fmax(v[6], e[q]);
        }
    }
}

// Workgroups of the bounds: four particles a thread, kReduceBlocks at most.
static int bounds_blocks(int64_t n) {
    const int64_t want = (n + 4 * kBlock - 1) / (4 * kBlock);
    return (int)(want < 1 ? 1 : (want > kReduceBlocks ? kReduceBlocks : want));
}

// part[b*8 + {0..6}] = min x, min y, min z, max x, max y, max z, max d.
__global__ __launch_bounds__(kBlock) void k_bounds(const double *__restrict__ x,
                                                   const double *__restrict__ y,
                                                   const double *__restrict__ z,
                                                   const double *__restrict__ d, int64_t n,
                                                   double *__restrict__ part) {
    double v[7] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY, 0.0};
    thread_bounds<4>(x, y, z, d, (int64_t)blockIdx.x * kBlock + threadIdx.x,
                     (int64_t)gridDim.x * kBlock, n, v);
    __shared__ double sh[kBlock / 64][7];
    int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int k = 0; k < 7; ++k) {
        double r = k < 3 ? wave_min(v[k]) : wave_max(v[k]);
        if (lane == 0) sh[wid][k] = r;
    }
    __syncthreads();
    if (threadIdx.x < 7) {
        int k = threadIdx.x;
        double r = sh[0][k];
        for (int q = 1; q < kBlock / 64; ++q) r = k < 3 ? fmin(r, sh[q][k]) : fmax(r, sh[q][k]);
        part[blockIdx.x * 8 + k] = r;
    }
}

__global__ __launch_bounds__(kBlock) void k_bounds_final(const double *__restrict__ part,
                                                         int nblocks, double *__restrict__ out) {
    double v[7] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY, 0.0};
#pragma unroll
    for (int q = 0; q < kReduceBlocks / kBlock; ++q) {  // past the end: the first block again
        const int b = (int)threadIdx.x + q * kBlock < nblocks ? (int)threadIdx.x + q * kBlock : 0;
#pragma unroll
        for (int k = 0; k < 7; ++k)
            v[k] = k < 3 ? fmin(v[k], part[b * 8 + k]) : fmax(v[k], part[b * 8 + k]);
    }
    __shared__ double sh[kBlock / 64][7];
    int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int k = 0; k < 7; ++k) {
        double r = k < 3 ? wave_min(v[k]) : wave_max(v[k]);
        if (lane == 0) sh[wid][k] = r;
    }
    __syncthreads();
    if (threadIdx.x < 7) {
        int k = threadIdx.x;
        double r = sh[0][k];
        for (int q = 1; q < kBlock / 64; ++q) r = k < 3 ? fmin(r, sh[q][k]) : fmax(r, sh[q][k]);
        out[k] = r;
    }
}

// The workgroup's minima and maxima of its threads' v (NW waves), also written to the host's
// pinned slot: each value with a system-scope fence, then (after the workgroup barrier) the
// sequence number with a system-scope release, which the host polls.
template <int NW>
__device__ __forceinline__ void bounds_to_host(const double (&v)[7], double *__restrict__ out,
                                               HostBounds *hb, unsigned long long seq) {
    __shared__ double sh[NW][7];
    int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    for (int k = 0; k < 7; ++k) {
        double r = k < 3 ? wave_min(v[k]) : wave_max(v[k]);
        if (lane == 0) sh[wid][k] = r;
    }
    __syncthreads();
    if (threadIdx.x < 7) {
        int k = threadIdx.x;
        double r = sh[0][k];
        for (int q = 1; q < NW; ++q) r = k < 3 ? fmin(r, sh[q][k]) : fmax(r, sh[q][k]);
        out[k] = r;
        hb->b[k] = r;
        __threadfence_system();
    }
    __syncthreads();
    if (threadIdx.x == 0)
        __hip_atomic_store(&hb->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(kBlock) void k_bounds_final_host(const double *__restrict__ part,
                                                              int nblocks,
                                                              double *__restrict__ out,
                                                              HostBounds *hb,
                                                              unsigned long long seq) {
    double v[7] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY, 0.0};
#pragma unroll
    for (int q = 0; q < kReduceBlocks / kBlock; ++q) {  // past the end: the first block again
        const int b = (int)threadIdx.x + q * kBlock < nblocks ? (int)threadIdx.x + q * kBlock : 0;
#pragma unroll
        for (int k = 0; k < 7; ++k)
            v[k] = k < 3 ? fmin(v[k], part[b * 8 + k]) : fmax(v[k], part[b * 8 + k]);
    }
    bounds_to_host<kBlock / 64>(v, out, hb, seq);
}

// A small set's bounds in one workgroup: one launch instead of two before the host's wait.
__global__ __launch_bounds__(kSmallBlock) void k_bounds_small(const double *__restrict__ x,
                                                              const double *__restrict__ y,
                                                              const double *__restrict__ z,
                                                              const double *__restrict__ d, int n,
                                                              double *__restrict__ out,
                                                              HostBounds *hb,
                                                              unsigned long long seq) {
    double v[7] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY, 0.0};
    thread_bounds<8>(x, y, z, d, threadIdx.x, kSmallBlock, n, v);
    bounds_to_host<kSmallBlock / 64>(v, out, hb, seq);
}

hipError_t launch_bounds_host(const double *x, const double *y, const double *z,
                              const double *d, int64_t n, double *part, double *out,
                              HostBounds *hb, unsigned long long seq, hipStream_t st) {
    if (n <= kSmallN) {
        k_bounds_small<<<1, kSmallBlock, 0, st>>>(x, y, z, d, (int)n, out, hb, seq);
        return hipGetLastError();
    }
    const int nb = bounds_blocks(n);
    k_bounds<<<nb, kBlock, 0, st>>>(x, y, z, d, n, part);
    k_bounds_final_host<<<1, kBlock, 0, st>>>(part, nb, out, hb, seq);
    return hipGetLastError();
}

__global__ void k_word_host(const unsigned long long *__restrict__ src, unsigned long long *sum,
                            HostBounds *hb, unsigned long long seq) {
    if (threadIdx.x != 0) return;
    const unsigned long long v = *src;
    if (sum) *sum += v;
    ((unsigned long long *)hb->b)[0] = v;
    __hip_atomic_store(&hb->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t launch_word_host(const unsigned long long *src, unsigned long long *sum,
                            HostBounds *hb, unsigned long long seq, hipStream_t st) {
    k_word_host<<<1, 64, 0, st>>>(src, sum, hb, seq);
    return hipGetLastError();
}

hipError_t launch_bounds(const double *x, const double *y, const double *z, const double *d,
                         int64_t n, double *part, double *out, hipStream_t st) {
    const int nb = bounds_blocks(n);
    k_bounds<<<nb, kBlock, 0, st>>>(x, y, z, d, n, part);
    k_bounds_final<<<1, kBlock, 0, st>>>(part, nb, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------- exclusive scan

template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T v, T *lds, T &total) {
    int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    T x = v;
    for (int o = 1; o < 64; o <<= 1) {
        T y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    if (lane == 63) lds[wid] = x;
    __syncthreads();
    if (threadIdx.x == 0) {
        T run = 0;
        for (int k = 0; k < kBlock / 64; ++k) {
            T t = lds[k];
            lds[k] = run;
            run += t;
        }
        lds[kBlock / 64] = run;
    }
    __syncthreads();
    T excl = (x - v) + lds[wid];
    total = lds[kBlock / 64];
    __syncthreads();
    return excl;
}

template <typename TI>
__global__ __launch_bounds__(kBlock) void k_scan_reduce(const TI *__restrict__ in, int64_t len,
                                                        int64_t *__restrict__ tile_sum, int vec) {
    int64_t base = (int64_t)blockIdx.x * kScanTile;
    int64_t s = 0;
    const int64_t own = base + (int64_t)threadIdx.x * kScanItems;  // the apply pass's layout
    if (sizeof(TI) == 4 && vec && own + kScanItems <= len) {
        const int4 a = ((const int4 *)(in + own))[0], b = ((const int4 *)(in + own))[1];
        s = (((int64_t)a.x + a.y) + ((int64_t)a.z + a.w)) + (((int64_t)b.x + b.y) + ((int64_t)b.z + b.w));
    } else {
        for (int k = 0; k < kScanItems; ++k) {
            int64_t i = own + k;
            if (i < len) s += (int64_t)in[i];
        }
    }
    __shared__ int64_t lds[kBlock / 64 + 1];
    int64_t total;
    block_exclusive_scan<int64_t>(s, lds, total);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
}

// Exclusive scan of the tile sums in one workgroup; out[len] = grand total.  Each thread
// takes a run of consecutive tiles, so one workgroup scan covers them all.
template <typename TO>
__global__ __launch_bounds__(kBlock) void k_scan_tops(int64_t *__restrict__ tile_sum,
                                                      int64_t ntiles, TO *__restrict__ out,
                                                      int64_t len) {
    __shared__ int64_t lds[kBlock / 64 + 1];
    const int64_t per = (ntiles + kBlock - 1) / kBlock;
    const int64_t a = (int64_t)threadIdx.x * per, b = a + per < ntiles ? a + per : ntiles;
    int64_t s = 0;
    for (int64_t i = a; i < b; ++i) s += tile_sum[i];
    int64_t total;
    int64_t run = block_exclusive_scan<int64_t>(s, lds, total);
    for (int64_t i = a; i < b; ++i) {
        const int64_t v = tile_sum[i];
        tile_sum[i] = run;
        run += v;
    }
    if (threadIdx.x == 0) out[len] = (TO)total;
}

constexpr int64_t kOwnTiles = 1024;

// sums: every workgroup adds up the sums of the tiles before its own (up to kOwnTiles of
// them), which leaves out the launch that scans them.  vec: in and out are 16-byte aligned 32-bit
// arrays; a thread's kScanItems = 8 values then move as two 16-byte loads and stores (the tail
// tile goes element by element).
template <typename TI, typename TO>
__global__ __launch_bounds__(kBlock) void k_scan_apply(const TI *in, TO *out, int64_t len,
                                                       const int64_t *__restrict__ tile_off,
                                                       int vec, int sums) {
    static_assert(kScanItems == 8, "two 16-byte vectors per thread");
    int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
    const bool wide = sizeof(TI) == 4 && sizeof(TO) == 4 && vec && base + kScanItems <= len;
    int64_t v[kScanItems];
    int64_t s = 0;
    if (wide) {
        const int4 a = ((const int4 *)(in + base))[0], b = ((const int4 *)(in + base))[1];
        const int w[kScanItems] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        for (int k = 0; k < kScanItems; ++k) v[k] = w[k];
    } else {
        for (int k = 0; k < kScanItems; ++k) {
            int64_t i = base + k;
            v[k] = i < len ? (int64_t)in[i] : 0;
        }
    }
    for (int k = 0; k < kScanItems; ++k) s += v[k];
    __shared__ int64_t lds[kBlock / 64 + 1];
    int64_t total;
    int64_t run = block_exclusive_scan<int64_t>(s, lds, total);
    if (sums) {  // tile_off holds the tiles' sums: add up those before this tile
        int64_t before = 0, all;
        for (int k = threadIdx.x; k < (int)blockIdx.x; k += kBlock) before += tile_off[k];
        block_exclusive_scan<int64_t>(before, lds, all);
        run += all;
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[len] = (TO)(all + total);
    } else {
        run += tile_off[blockIdx.x];
    }
    if (wide) {
        int o[kScanItems];
        for (int k = 0; k < kScanItems; ++k) {
            o[k] = (int)run;
            run += v[k];
        }
        ((int4 *)(out + base))[0] = make_int4(o[0], o[1], o[2], o[3]);
        ((int4 *)(out + base))[1] = make_int4(o[4], o[5], o[6], o[7]);
    } else {
        for (int k = 0; k < kScanItems; ++k) {
            int64_t i = base + k;
            if (i < len) out[i] = (TO)run;
            run += v[k];
        }
    }
}

// out[0..len) = exclusive prefix sums of in[0..len), out[len] = total.
// in may alias out when TI == TO.  tmp holds ceil(len / kScanTile) int64.
template <typename TI, typename TO>
hipError_t launch_scan_exclusive(const TI *in, TO *out, int64_t len, int64_t *tmp,
                                 hipStream_t st) {
    int64_t ntiles = (len + kScanTile - 1) / kScanTile;
    const int vec = ((uintptr_t)in % 16 == 0) && ((uintptr_t)out % 16 == 0);
    if (ntiles > 0) k_scan_reduce<TI><<<(unsigned)ntiles, kBlock, 0, st>>>(in, len, tmp, vec);
    const int own = ntiles > 0 && ntiles <= kOwnTiles;
    if (!own) k_scan_tops<TO><<<1, kBlock, 0, st>>>(tmp, ntiles, out, len);
    if (ntiles > 0)
        k_scan_apply<TI, TO><<<(unsigned)ntiles, kBlock, 0, st>>>(in, out, len, tmp, vec, own);
    return hipGetLastError();
}

template hipError_t launch_scan_exclusive<int32_t, int32_t>(const int32_t *, int32_t *, int64_t,
                                                            int64_t *, hipStream_t);
template hipError_t launch_scan_exclusive<int32_t, int64_t>(const int32_t *, int64_t *, int64_t,
                                                            int64_t *, hipStream_t);

// ---------------------------------------------------------------- counting sort by cell

// The histogram cleared, and the caller's words set.
__global__ __launch_bounds__(kBlock) void k_clear(int32_t *p, int64_t count, ClearWords w) {
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * kBlock)
        p[i] = 0;
    if (blockIdx.x == 0 && (int)threadIdx.x < w.n) *w.p[threadIdx.x] = w.v[threadIdx.x];
}

// Whether coordinate v lies on the mesh axis (origin o, 1/D inv, dim cells), in the cell
// arithmetic of cell_coord.
__device__ __forceinline__ bool on_axis(double v, double o, double inv, int dim) {
    const double f = floor((v - o) * inv);
    return f >= 0.0 && f < (double)dim;
}

__global__ __launch_bounds__(kBlock) void k_keys(const double *__restrict__ x,
                                                 const double *__restrict__ y,
                                                 const double *__restrict__ z, int64_t n,
                                                 GridDev g, uint32_t *__restrict__ key,
                                                 uint32_t *__restrict__ rank,
                                                 int32_t *__restrict__ count,
                                                 uint32_t *__restrict__ key_out, BinCheck chk) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const bool live = i < n;
    double xi = 0.0, yi = 0.0, zi = 0.0;
    if (live) {
        xi = x[i];
        yi = y[i];
        zi = z[i];
        int cx = cell_coord(xi, g.ox, g.inv, g.dx);
        int cy = cell_coord(yi, g.oy, g.inv, g.dy);
        int cz = cell_coord(zi, g.oz, g.inv, g.dz);
        uint32_t k = g.morton ? morton_key(cx, cy, cz) : cell_key(g, cx, cy, cz);
        key[i] = k;
        rank[i] = (uint32_t)atomicAdd(&count[k], 1);
        if (key_out) key_out[i] = k;
    }
    if (chk.yenc) {  // the wave's minimum y, one atomic per wave
        unsigned long long e = live ? order_enc(yi) : ~0ull;
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned long long f = __shfl_xor(e, o, 64);
            e = f < e ? f : e;
        }
        if ((threadIdx.x & 63) == 0 && e != ~0ull) atomicMin(chk.yenc, e);
    }
    if (chk.outside) {
        bool out = live && !(on_axis(xi, g.ox, g.inv, g.dx) && on_axis(yi, g.oy, g.inv, g.dy) &&
                             on_axis(zi, g.oz, g.inv, g.dz));
        const double p[3] = {xi, yi, zi};
        for (int a = 0; a < 3; ++a)
            if (live && ((chk.per >> a) & 1) && !(p[a] >= chk.lo[a] && p[a] <= chk.hi[a]))
                out = true;
        const unsigned long long c = __popcll(__ballot(out));
        if ((threadIdx.x & 63) == 0 && c) atomicAdd(chk.outside, c);
    }
}

__global__ __launch_bounds__(kBlock) void k_scatter(const uint32_t *__restrict__ key,
                                                    const uint32_t *__restrict__ rank,
                                                    const int32_t *__restrict__ cs, int64_t n,
                                                    int32_t *__restrict__ tmp) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    tmp[cs[key[i]] + (int32_t)rank[i]] = (int32_t)i;
}

// Final place of the particle in slot s of the scattered order: its cell segment's start plus
// the number of the segment's particles with a smaller input index.  O(k) per particle for a
// cell of k particles, all particles in parallel (an in-cell sort by one thread per cell would
// cost O(k^2) for a dense cell).
__global__ __launch_bounds__(kBlock) void k_cell_rank(const uint32_t *__restrict__ key,
                                                      const int32_t *__restrict__ cs, int64_t n,
                                                      const int32_t *__restrict__ tmp,
                                                      int32_t *__restrict__ perm) {
    int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (s >= n) return;
    const int p = tmp[s];
    const uint32_t k = key[p];
    const int a = cs[k], b = cs[k + 1];
    int r = 0;
    for (int t = a; t < b; ++t) r += tmp[t] < p ? 1 : 0;
    perm[a + r] = p;
}

// The whole binning of a small set in one workgroup: the histogram (16-bit counts, two to a
// word, whose atomics also rank the particles in their cells), its scan, the cell segments and
// the places in them, all in LDS.  Seven launches became one; a 13 824-particle binning took
// ~17 us of kernels in ~30 us of launches.
//
// A particle's place in its cell is the number of the cell's particles with a smaller index: a
// look at each of them.  Where a cell holds more than kSmallCell, the particles of such cells are
// first put in order of their rounds (index / kSmallBlock) by counts per cell and round, and look
// at those of their own round only, eight to a load where there are more than kSmallRow.  16 382
// particles over 8 000 cells: spread 0.037 ms; 120 cells of 130 0.060, 32 of 511 0.094, 16 000 in
// one 0.37; by looks at the whole cell 0.134, 0.71 and 12.0, by the launches above 0.055, 0.095
// and 1.52.  (Cells of 64: 0.068 by rounds, 0.063 by looks eight to a load, which every set's
// larger code pays for.)
constexpr int kSmallKeys = 16 * 1024;
constexpr int kSmallRow = 32;
constexpr int kSmallCellLog = 6;
constexpr int kSmallCell = 1 << kSmallCellLog;
__global__ __launch_bounds__(kSmallBlock) void k_bin_small(
    const double *__restrict__ x, const double *__restrict__ y, const double *__restrict__ z,
    int n, GridDev g, int nkey, int32_t *__restrict__ perm, uint32_t *__restrict__ key_out,
    int32_t *__restrict__ cs, ClearWords w) {
    // counts, then cell starts, as 16-bit halves
    __shared__ __align__(16) uint32_t hist[kSmallKeys / 2];
    __shared__ __align__(16) uint16_t seg[kSmallN];  // particles by cell, in atomic order
    __shared__ int lds[kSmallBlock / 64 + 1];
    // crowded cells' counts, then offsets, by round: those of number start / kSmallCell, which no two
    // of them share
    __shared__ int turn[kSmallN / kSmallCell][kSmallPer];
    __shared__ int crowded;
    uint16_t *const start = (uint16_t *)hist;
    const int tid = threadIdx.x;
    if (tid == 0) crowded = 0;
    for (int k = tid; k < kSmallKeys / 8; k += kSmallBlock)
        ((uint4 *)hist)[k] = make_uint4(0u, 0u, 0u, 0u);
    if (tid < w.n) *w.p[tid] = w.v[tid];
    __syncthreads();
    uint32_t key[kSmallPer];
    int rank[kSmallPer];
#pragma unroll
    for (int q0 = 0; q0 < kSmallPer; q0 += 8) {  // eight particles' positions in flight
        if (q0 * kSmallBlock >= n) break;
        double px[8], py[8], pz[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = (q0 + q) * kSmallBlock + tid, j = i < n ? i : 0;
            px[q] = x[j];
            py[q] = y[j];
            pz[q] = z[j];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = (q0 + q) * kSmallBlock + tid;
            const int cx = cell_coord(px[q], g.ox, g.inv, g.dx);
            const int cy = cell_coord(py[q], g.oy, g.inv, g.dy);
            const int cz = cell_coord(pz[q], g.oz, g.inv, g.dz);
            const uint32_t k = g.morton ? morton_key(cx, cy, cz) : cell_key(g, cx, cy, cz);
            key[q0 + q] = k;
            if (i < n) {
                if (key_out) key_out[i] = k;
                const int sh = (k & 1u) ? 16 : 0;
                rank[q0 + q] = (int)((atomicAdd(&hist[k >> 1], 1u << sh) >> sh) & 0xffffu);
            }
        }
    }
    __syncthreads();
    // exclusive scan: each thread's run of 16 keys, then the workgroup's
    static_assert(kSmallKeys == 16 * kSmallBlock, "16 keys a thread, eight to a vector");
    uint4 *const own = (uint4 *)hist + 2 * tid;
    const uint4 c0 = own[0], c1 = own[1];
    uint32_t c[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
    int sum = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) sum += (int)(c[k] & 0xffffu) + (int)(c[k] >> 16);
    int inc = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(inc, o, 64);
        if ((tid & 63) >= o) inc += v;
    }
    if ((tid & 63) == 63) lds[tid >> 6] = inc;
    __syncthreads();
    int run = inc - sum;
    int most = 0;
    for (int q = 0; q < (tid >> 6); ++q) run += lds[q];
#pragma unroll
    for (int k = 0; k < 8; ++k) {  // the thread's own keys; starts below n <= 16 384
        const int n0 = (int)(c[k] & 0xffffu), n1 = (int)(c[k] >> 16);
        most = max(most, max(n0, n1));
        const uint32_t first = (uint32_t)run;
        run += n0;
        const uint32_t second = (uint32_t)run;
        run += n1;
        c[k] = first | second << 16;
    }
    own[0] = make_uint4(c[0], c[1], c[2], c[3]);
    own[1] = make_uint4(c[4], c[5], c[6], c[7]);
    if (most > kSmallCell) crowded = 1;
    __syncthreads();
    for (int k = tid; k < nkey; k += kSmallBlock) cs[k] = start[k];
    if (tid == 0) cs[nkey] = n;
#pragma unroll
    for (int q = 0; q < kSmallPer; ++q) {
        const int i = q * kSmallBlock + tid;
        if (i >= n) break;
        seg[start[key[q]] + rank[q]] = (uint16_t)i;
    }
    const auto cell_of = [&](int q, int &a, int &b) {
        a = start[key[q]];
        b = (int)key[q] + 1 < kSmallKeys ? start[key[q] + 1] : n;
    };
    __syncthreads();
    if (!crowded) {
#pragma unroll
        for (int q = 0; q < kSmallPer; ++q) {
            const int i = q * kSmallBlock + tid;
            if (i >= n) break;
            int a, b;
            cell_of(q, a, b);
            int r = 0;
            for (int t = a; t < b; ++t) r += (int)seg[t] < i ? 1 : 0;
            perm[a + r] = i;
        }
        return;
    }
    // the particles of seg[a..b) with an index below i
    const auto smaller = [&](int a, int b, int i) {
        int r = 0, t = a;
        if (b - a > kSmallRow) {
            for (; t & 7; ++t) r += (int)seg[t] < i ? 1 : 0;
            for (; t + 8 <= b; t += 8) {
                const uint4 v = *(const uint4 *)(seg + t);
                const uint32_t h[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    r += ((int)(h[u] & 0xffffu) < i ? 1 : 0) + ((int)(h[u] >> 16) < i ? 1 : 0);
            }
        }
        for (; t < b; ++t) r += (int)seg[t] < i ? 1 : 0;
        return r;
    };
    constexpr int kTurns = kSmallN / kSmallCell * kSmallPer;
    int *const all = &turn[0][0];
    for (int k = tid; k < kTurns; k += kSmallBlock) all[k] = 0;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSmallPer; ++q) {
        int a, b;
        if (q * kSmallBlock + tid >= n) break;
        cell_of(q, a, b);
        if (b - a > kSmallCell) rank[q] = atomicAdd(&turn[a >> kSmallCellLog][q], 1);
    }
    __syncthreads();
    static_assert(kSmallPer == 16 && kSmallBlock % 16 == 0, "a cell's rounds in 16 lanes");
    for (int k = tid; k < kTurns; k += kSmallBlock) {
        const int count = all[k];
        int upto = count;
        for (int o = 1; o < 16; o <<= 1) {
            const int v = __shfl_up(upto, o, 16);
            if ((tid & 15) >= o) upto += v;
        }
        all[k] = upto - count;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSmallPer; ++q) {
        int a, b;
        const int i = q * kSmallBlock + tid;
        if (i >= n) break;
        cell_of(q, a, b);
        if (b - a > kSmallCell) seg[a + turn[a >> kSmallCellLog][q] + rank[q]] = (uint16_t)i;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kSmallPer; ++q) {
        const int i = q * kSmallBlock + tid;
        if (i >= n) break;
        int a, b;
        cell_of(q, a, b);
        if (b - a > kSmallCell) {  // those of its round
            const int *const off = turn[a >> kSmallCellLog];
            if (q + 1 < kSmallPer) b = a + off[q + 1];
            a += off[q];
        }
        perm[a + smaller(a, b, i)] = i;
    }
}

static unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

hipError_t launch_bin(const double *x, const double *y, const double *z, int64_t n,
                      const GridDev &g, const Ws &w, int32_t *perm, uint32_t *key_out,
                      int32_t *cell_start, hipStream_t st, const BinCheck *chk,
                      const ClearWords *words) {
    const BinCheck c = chk ? *chk : BinCheck{nullptr, nullptr, 0, {0, 0, 0}, {0, 0, 0}};
    const ClearWords cw = words ? *words : ClearWords{};
    const int64_t ncell = g.nkey;  // keys (cells, or the Morton key space)
    if (n > 0 && n <= kSmallN && ncell < kSmallKeys && n * n <= kSmallLooks * ncell && !chk) {
        k_bin_small<<<1, kSmallBlock, 0, st>>>(x, y, z, (int)n, g, (int)ncell, perm, key_out,
                                               cell_start, cw);
        return hipGetLastError();
    }
    unsigned fb = blocks_for(ncell + 1);
    k_clear<<<fb > 65535u ? 65535u : fb, kBlock, 0, st>>>(cell_start, ncell + 1, cw);
    if (n > 0)
        k_keys<<<blocks_for(n), kBlock, 0, st>>>(x, y, z, n, g, w.key, w.rank, cell_start,
                                                 key_out, c);
    hipError_t e = launch_scan_exclusive<int32_t, int32_t>(cell_start, cell_start, ncell,
                                                           w.scan_tmp, st);
    if (e != hipSuccess) return e;
    if (n > 0) {
        k_scatter<<<blocks_for(n), kBlock, 0, st>>>(w.key, w.rank, cell_start, n, w.bin_tmp);
        k_cell_rank<<<blocks_for(n), kBlock, 0, st>>>(w.key, cell_start, n, w.bin_tmp, perm);
    }
    return hipGetLastError();
}

}  // namespace csph
