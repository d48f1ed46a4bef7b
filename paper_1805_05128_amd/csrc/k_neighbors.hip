// Neighbour-set export N(i) = { j != i : |r_j - r_i|^2 < H_ij^2 } (sec. 4.1)
// as CSR over input indices, rows ascending.  Verification form only: the
// rate kernels gather partners on the fly and never materialise this list.
// The test is the FP64 expression ((dx*dx)+(dy*dy))+(dz*dz) < H*H without
// contraction, so membership is exact.  With periodic axes the partners
// include the periodic images, d = (r_j - r_i) - k L (each j appears once:
// the periods exceed twice the support).
#include "csph_internal.h"
#include "stencil.h"

namespace csph {

__global__ __launch_bounds__(kBlock) void k_gather_pos(int64_t n, const int32_t *__restrict__ perm,
                                                       const double *__restrict__ x,
                                                       const double *__restrict__ y,
                                                       const double *__restrict__ z,
                                                       const double *__restrict__ d,
                                                       double *__restrict__ xs,
                                                       double *__restrict__ ys,
                                                       double *__restrict__ zs,
                                                       double *__restrict__ ds) {
    int64_t s = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (s >= n) return;
    int i = perm[s];
    xs[s] = x[i];
    ys[s] = y[i];
    zs[s] = z[i];
    if (d) ds[s] = d[i];
}

hipError_t launch_gather_pos(int64_t n, const int32_t *perm, const double *x, const double *y,
                             const double *z, const double *d, const Ws &w, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    k_gather_pos<<<(unsigned)((n + kBlock - 1) / kBlock), kBlock, 0, st>>>(
        n, perm, x, y, z, d, w.srt[0], w.srt[1], w.srt[2], w.srt_d);
    return hipGetLastError();
}

// A wave's stores to memory seen by its own later loads, whichever lane made them.
__device__ __forceinline__ void wave_memory_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// a[0..c) sorted ascending in place by one wave, every lane taking part: runs of k/2 are merged
// into runs of k, k = 2, 4, .., by Batcher's bitonic network in the form whose first exchange
// pairs a run's entry with the mirrored one of its neighbour, so that every exchange puts the
// smaller value first and a pair that reaches past the end has nothing to exchange.
// O(c log^2 c / 64) with kInFlight pairs a lane at once.
__device__ void wave_sort(int32_t *a, int c, int lane) {
    constexpr int kInFlight = 4;
    auto exchange = [&](int sh, bool mirror) {  // pairs (lo, hi) in blocks of 2 << sh entries
        const int j = 1 << sh;
        for (int t0 = lane; (t0 >> sh) << (sh + 1) < c; t0 += 64 * kInFlight) {
            int lo[kInFlight], hi[kInFlight], x[kInFlight], y[kInFlight];
#pragma unroll
            for (int u = 0; u < kInFlight; ++u) {
                const int t = t0 + 64 * u, o = t & (j - 1), base = (t >> sh) << (sh + 1);
                lo[u] = base + o;
                hi[u] = mirror ? base + 2 * j - 1 - o : base + j + o;
                x[u] = hi[u] < c ? a[lo[u]] : 0;
                y[u] = hi[u] < c ? a[hi[u]] : 0;
            }
#pragma unroll
            for (int u = 0; u < kInFlight; ++u)
                if (x[u] > y[u]) {
                    a[lo[u]] = y[u];
                    a[hi[u]] = x[u];
                }
        }
        wave_memory_fence();
    };
    for (int sh = 0; (1 << sh) < c; ++sh) {
        exchange(sh, true);
        for (int q = sh - 1; q >= 0; --q) exchange(q, false);
    }
}

// One wave per particle: the lanes take the particle's stencil rows (64 at a time), clipped to
// the chord of the support, lay the rows' candidates end to end in LDS (row by row where they
// are too many) and test four of them each at once; the accepted ones are appended in candidate
// order, ranked among themselves in LDS and stored ascending.  A thread per particle walked
// ~570 candidates by itself, stored its row scattered and heap-sorted it in memory: for 83 143
// particles off the lattice (H = 3, ~92 neighbours) the count took 142 us and the fill 1 224 us;
// now 61 and 122 us (98 and 166 us on cells of the support's size, which the export cuts in
// three), bound by vector issue: ~350 instructions a particle for the search, ~370 for the ranks.
constexpr int kNbrWaves = kBlock / 64;
constexpr int kNbrList = 1024;     // candidates laid out at once
constexpr int kNbrShort = 32;      // longest row its own lane lays out
constexpr int kNbrBatch = 4;       // 64-candidate tests in flight
// Neighbours ranked in LDS, O(c^2 / 64); a longer row is sorted in memory by the wave, O(c log^2 c
// / 64).  83 248 particles: rows up to 322 ranked 0.70 ms, sorted 0.76; up to 431 1.08 and 0.93;
// up to 534 1.47 and 1.41; up to 721 sorted 2.9 ms, where a heap sort by one lane a row, 63
// waiting, took 29 ms.  A list of 1 024 costs occupancy: 3.5 ms.
constexpr int kNbrCap = 512;

// The export's inputs and outputs (cell order but for count_orig, offsets and idx).
struct NbrArgs {
    int64_t n;
    GridDev g;
    PairConst pc;
    const double *__restrict__ x, *__restrict__ y, *__restrict__ z, *__restrict__ d;
    const int32_t *__restrict__ cs, *__restrict__ perm;
    int32_t *__restrict__ count_orig;
    const int64_t *__restrict__ offsets;
    int32_t *__restrict__ idx;
};

// Particle s's count or row by the whole wave; list (kNbrList) and mine (kNbrCap) are the wave's.
template <bool PAIR, bool FILL, bool PER>
__device__ __forceinline__ void nbr_particle(const NbrArgs &A, int64_t s, int *list, int *mine,
                                             int lane) {
    const GridDev &g = A.g;
    const PairConst &pc = A.pc;
    const double *const x = A.x, *const y = A.y, *const z = A.z, *const d = A.d;
    const int32_t *const cs = A.cs, *const perm = A.perm;
    const int64_t *const offsets = A.offsets;
    int32_t *const idx = A.idx;
    const double xi = x[s], yi = y[s], zi = z[s];
    const double di = PAIR ? d[s] : 0.0;
    const int nf = PER ? image_faces(pc, xi, yi, zi) : 0;
    const int i = perm[s];
    const int64_t wpos = FILL ? offsets[i] : 0;
    const bool ranked = FILL && offsets[i + 1] - wpos <= kNbrCap;
    int cnt = 0;
    // image m = 0: i itself; m > 0: the periodic image of i across the faces of mask m
    for (int m = 0; m < (PER ? 8 : 1); ++m) {
        if ((nf & m) != m) continue;
        const double shx = image_shift(pc, nf, m, 0), shy = image_shift(pc, nf, m, 1),
                     shz = image_shift(pc, nf, m, 2);
        Stencil st = make_stencil(g, xi, yi, zi, pc.H);
        if (PER) st = shifted_stencil(g, st, m, xi + shx, yi + shy, zi + shz);
        // kNbrBatch candidates per lane (j < 0: none), their positions all asked for at once
        auto test = [&](const int (&j)[kNbrBatch]) {
            double dx[kNbrBatch], dy[kNbrBatch], dz[kNbrBatch], dd[kNbrBatch];
            int id[kNbrBatch];
#pragma unroll
            for (int u = 0; u < kNbrBatch; ++u) {
                const int k = j[u] >= 0 ? j[u] : 0;
                dx[u] = x[k];
                dy[u] = y[k];
                dz[u] = z[k];
                dd[u] = PAIR ? d[k] : 0.0;
                id[u] = FILL ? perm[k] : 0;
            }
#pragma unroll
            for (int u = 0; u < kNbrBatch; ++u) {
                double ex = dx[u] - xi, ey = dy[u] - yi, ez = dz[u] - zi;
                if (PER) {
                    ex = ex - shx;
                    ey = ey - shy;
                    ez = ez - shz;
                }
                const double r2 = ((ex * ex) + (ey * ey)) + (ez * ez);
                double H2 = pc.H2;
                if (PAIR) {
                    const double H = pc.kappa * (0.5 * (di + dd[u]));
                    H2 = H * H;
                }
                const bool in = j[u] >= 0 && !(m == 0 && j[u] == (int)s) && r2 < H2;
                const unsigned long long hit = __ballot(in);
                if (FILL && in) {
                    const int at = cnt + __popcll(hit & ((1ull << lane) - 1ull));
                    if (ranked)
                        mine[at] = id[u];
                    else
                        idx[wpos + at] = id[u];
                }
                cnt += __popcll(hit);
            }
        };
        const int W = 2 * st.R + 1;
        const float iw = 1.0f / (float)W;
        for (int q0 = 0; q0 < W * W; q0 += 64) {
            const int q = q0 + lane;
            const int iz = (int)(((float)q + 0.5f) * iw);  // q / W (as walk_rows_split)
            const int oz = iz - st.R, oy = q - iz * W - st.R;
            const int yy = st.cy + oy, zz = st.cz + oz;
            int j0, len;
            if (!row_range(cs, g, st, plane_rem(g, st, q < W * W, oz, zz), oy, yy,
                           cell_key(g, 0, yy, zz), j0, len))
                continue;
            int end = len;  // candidates of the rows up to the lane's
            for (int o = 1; o < 64; o <<= 1) {
                const int p = __shfl_up(end, o, 64);
                if (lane >= o) end += p;
            }
            const int total = __shfl(end, 63, 64);
            if (total <= kNbrList) {
                wave_fence();
                if (!__any(len > kNbrShort)) {
                    for (int k = 0; __any(k < len); ++k)
                        if (k < len) list[end - len + k] = j0 + k;
                } else {
                    for (unsigned long long rows = __ballot(len > 0); rows; rows &= rows - 1) {
                        const int r = __builtin_ctzll(rows);
                        const int a = __builtin_amdgcn_readlane(j0, r);
                        const int c = __builtin_amdgcn_readlane(len, r);
                        const int at = __builtin_amdgcn_readlane(end, r) - c;
                        for (int t = lane; t < c; t += 64) list[at + t] = a + t;
                    }
                }
                wave_fence();
                for (int t = 0; t < total; t += 64 * kNbrBatch) {
                    int j[kNbrBatch];
#pragma unroll
                    for (int u = 0; u < kNbrBatch; ++u) {
                        const int at = t + 64 * u + lane;
                        j[u] = at < total ? list[at] : -1;
                    }
                    test(j);
                }
            } else {
                for (unsigned long long rows = __ballot(len > 0); rows; rows &= rows - 1) {
                    const int r = __builtin_ctzll(rows);
                    const int a = __builtin_amdgcn_readlane(j0, r);
                    const int c = __builtin_amdgcn_readlane(len, r);
                    for (int t = 0; t < c; t += 64 * kNbrBatch) {
                        int j[kNbrBatch];
#pragma unroll
                        for (int u = 0; u < kNbrBatch; ++u) {
                            const int at = t + 64 * u + lane;
                            j[u] = at < c ? a + at : -1;
                        }
                        test(j);
                    }
                }
            }
        }
    }
    if (!FILL) {
        if (lane == 0) A.count_orig[i] = cnt;
        return;
    }
    if (ranked) {  // ascending: a neighbour's place is the number of smaller ones
        wave_fence();
        if (lane < 4 && cnt + lane < kNbrCap) mine[cnt + lane] = INT32_MAX;
        wave_fence();
        for (int t = lane; t < cnt; t += 64) {
            const int v = mine[t];
            int place = 0;
            for (int k = 0; k < cnt; k += 4) {
                const int4 w = *(const int4 *)(mine + k);
                place += (w.x < v) + (w.y < v) + (w.z < v) + (w.w < v);
            }
            idx[wpos + place] = v;
        }
    } else {
        wave_memory_fence();
        wave_sort(idx + wpos, cnt, lane);
    }
}

template <bool PAIR, bool FILL, bool PER>
__global__ __launch_bounds__(kBlock) void k_nbr(NbrArgs A) {
    __shared__ int lst[kNbrWaves][kNbrList];
    __shared__ __align__(16) int acc[FILL ? kNbrWaves : 1][FILL ? kNbrCap : 4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t s = xcd_block_upto(blockIdx.x, gridDim.x, 16384) * kNbrWaves + wave;
    if (s >= A.n) return;  // whole waves; no barrier follows
    nbr_particle<PAIR, FILL, PER>(A, s, lst[wave], acc[FILL ? wave : 0], lane);
}

// Large sparse sets, a handful of candidates a particle: a wave a particle would spend its ~700
// instructions on each, so a lane takes one, walks its candidates and inserts its neighbours into
// a list of its own.  A particle of more than kNbrThin candidates or kNbrOwn neighbours, or with
// periodic images, is left to the whole wave afterwards: dense spots cost what they cost above.
// The export of 1 M particles: 0.3 neighbours each 0.41 ms (a wave a particle 1.40), 9 each 0.68
// (1.47).
constexpr int kNbrThin = 96;
constexpr int kNbrOwn = kNbrList / 64;

template <bool PAIR, bool FILL, bool PER>
__global__ __launch_bounds__(kBlock) void k_nbr_sparse(NbrArgs A) {
    __shared__ int lst[kNbrWaves][kNbrList];
    __shared__ __align__(16) int acc[FILL ? kNbrWaves : 1][FILL ? kNbrCap : 4];
    const GridDev &g = A.g;
    const PairConst &pc = A.pc;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t s0 = (xcd_block_upto(blockIdx.x, gridDim.x, 256) * kNbrWaves + wave) * 64;
    const int64_t s = s0 + lane;
    if (s0 >= A.n) return;  // whole waves; no barrier follows
    const bool live = s < A.n;
    const double xi = live ? A.x[s] : 0.0, yi = live ? A.y[s] : 0.0, zi = live ? A.z[s] : 0.0;
    const double di = PAIR && live ? A.d[s] : 0.0;
    const int i = live ? A.perm[s] : 0;
    const int64_t wpos = FILL && live ? A.offsets[i] : 0;
    int *const own = lst[wave] + lane;  // entry t of the lane's list at 64 t
    bool left = live && PER && image_faces(pc, xi, yi, zi) != 0;
    if (FILL && live) left = left || A.offsets[i + 1] - wpos > kNbrOwn;
    const Stencil st = make_stencil(g, xi, yi, zi, pc.H);
    int cnt = 0, walked = 0;
    walk_rows(A.cs, g, st, live, [&](int, int, int, int j0, int len) {
        left = left || (len > 0 && walked + len > kNbrThin);
        len = left ? 0 : len;
        walked += len;
        for (int k = 0; __any(k < len); k += kNbrBatch) {
            double dx[kNbrBatch], dy[kNbrBatch], dz[kNbrBatch], dd[kNbrBatch];
            int id[kNbrBatch];
#pragma unroll
            for (int u = 0; u < kNbrBatch; ++u) {
                const int j = k + u < len ? j0 + k + u : 0;
                dx[u] = A.x[j];
                dy[u] = A.y[j];
                dz[u] = A.z[j];
                dd[u] = PAIR ? A.d[j] : 0.0;
                id[u] = FILL ? A.perm[j] : 0;
            }
#pragma unroll
            for (int u = 0; u < kNbrBatch; ++u) {
                const double ex = dx[u] - xi, ey = dy[u] - yi, ez = dz[u] - zi;
                const double r2 = ((ex * ex) + (ey * ey)) + (ez * ez);
                double H2 = pc.H2;
                if (PAIR) {
                    const double H = pc.kappa * (0.5 * (di + dd[u]));
                    H2 = H * H;
                }
                if (k + u < len && j0 + k + u != (int)s && r2 < H2) {
                    if (FILL) {  // (a row within kNbrOwn, so its list holds it)
                        int t = cnt;
                        for (; t > 0 && own[64 * (t - 1)] > id[u]; --t) own[64 * t] = own[64 * (t - 1)];
                        own[64 * t] = id[u];
                    }
                    ++cnt;
                }
            }
        }
    });
    if (live && !left) {
        if (FILL) {
            for (int t = 0; t < cnt; ++t) A.idx[wpos + t] = own[64 * t];
        } else {
            A.count_orig[i] = cnt;
        }
    }
    for (unsigned long long rest = __ballot(left); rest; rest &= rest - 1) {
        wave_fence();
        nbr_particle<PAIR, FILL, PER>(A, s0 + __builtin_ctzll(rest), lst[wave],
                                      acc[FILL ? wave : 0], lane);
    }
}

// A set is taken as sparse by its mean: candidates of a full stencil, n (2 R + 1)^3 / cells, up to
// 64 (beyond, more and more particles are left to the wave), and enough particles that a lane
// each still gives the chip two waves a SIMD (100 000 particles, 0.3 neighbours: a wave each 0.20 ms,
// 131 072 a lane each 0.12).
constexpr int64_t kNbrSparseN = 1 << 17;
static bool nbr_sparse(int64_t n, const GridDev &g) {
    const double W = 2.0 * g.reach + 1.0;
    return n >= kNbrSparseN && (double)n * W * W * W <= 64.0 * (double)g.nkey;
}

template <bool FILL>
static hipError_t launch_nbr(const NbrArgs &A, hipStream_t st) {
    if (A.n <= 0) return hipSuccess;
    const bool sparse = nbr_sparse(A.n, A.g);
    const int64_t per = sparse ? kBlock : kNbrWaves;  // particles a workgroup
    const unsigned nb = (unsigned)((A.n + per - 1) / per);
#define CSPH_NBR(P, X)                                            \
    if (!!A.pc.pair_mode == P && !!A.pc.per == X) {               \
        if (sparse)                                               \
            k_nbr_sparse<P, FILL, X><<<nb, kBlock, 0, st>>>(A);   \
        else                                                      \
            k_nbr<P, FILL, X><<<nb, kBlock, 0, st>>>(A);          \
    }
    CSPH_NBR(false, false)
    CSPH_NBR(true, false)
    CSPH_NBR(false, true)
    CSPH_NBR(true, true)
#undef CSPH_NBR
    return hipGetLastError();
}

hipError_t launch_nbr_count(int64_t n, const GridDev &g, const PairConst &pc, const double *x,
                            const double *y, const double *z, const double *d, const int32_t *cs,
                            const int32_t *perm, int32_t *count_orig, hipStream_t st) {
    return launch_nbr<false>(NbrArgs{n, g, pc, x, y, z, d, cs, perm, count_orig, nullptr, nullptr},
                             st);
}

hipError_t launch_nbr_fill(int64_t n, const GridDev &g, const PairConst &pc, const double *x,
                           const double *y, const double *z, const double *d, const int32_t *cs,
                           const int32_t *perm, const int64_t *offsets, int32_t *idx,
                           hipStream_t st) {
    return launch_nbr<true>(NbrArgs{n, g, pc, x, y, z, d, cs, perm, nullptr, offsets, idx}, st);
}

}  // namespace csph
