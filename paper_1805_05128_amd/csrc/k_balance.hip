// Voronoi load balancer (sec. 3): subdomain statistics and one generator move.
//
// Statistics (one pass over the particles, generators in LDS):
//   * particle and pair loads per subdomain (integers);
//   * geometric centres (eq. VoronoiGeomCenters) from fixed-point sums: each
//     particle adds round((x - g_k) * 2^32) (|x - g_k| < 2^24) to a 128-bit
//     integer per coordinate, so the sums are exact and do not depend on the
//     order in which the atomics run;
//   * which subdomains touch: a particle owned by k whose nearest other
//     generator l lies within D^sh of the k|l bisector plane marks (k, l) and
//     (l, k) in a K x K bit matrix (the same FP64 expressions as the CPU
//     reference, no contraction, so the bits are exact).
// Move (one wave per generator): two-body displacement
// (eq. BalancingOffset), three-body rotations about the circumcentre of each
// triplet of mutually touching subdomains (eqs. BalancingOffsetPlusRot,
// BalancingOffsetRot) with the shift capped at D^sh, and the cumulative
// movement (eq. TotalOffset); the sum of |g' - g| (eq. VDConvergence) is
// reduced in a fixed order.
#include "csph_internal.h"
#include "nearest.h"

namespace csph {

constexpr double kFix = 4294967296.0;  // 2^32: fixed-point scale of the centre sums
constexpr double kFixMax = 72057594037927936.0;  // 2^56: per-particle bound (|x - g| < 2^24)

// below this every wave's sum over 64 kNearPer particles fits 63 bits
constexpr double kFixWave = 9007199254740992.0;  // 2^53

// Words of the touching pairs a > b of K subdomains, one bit each.  A workgroup gathers them in
// LDS and adds them to the matrix at its end: set in memory by the lanes that find them, a few
// words (and the loads that look whether a bit is there already) took 0.45 ms of the 0.48 ms of
// 2.9 M particles.
__host__ __device__ constexpr int tri_words(int K) { return (K * (K - 1) / 2 + 31) / 32; }

__device__ __forceinline__ double norm2(double x, double y, double z) {
    return __dadd_rn(__dadd_rn(__dmul_rn(x, x), __dmul_rn(y, y)), __dmul_rn(z, z));
}

// 128-bit two's-complement accumulator {lo, hi}: add a signed 64-bit value.
__device__ __forceinline__ void add128(unsigned long long *lo, unsigned long long *hi, long long v) {
    const unsigned long long u = (unsigned long long)v;
    const unsigned long long old = atomicAdd(lo, u);
    const unsigned long long carry = (old + u < old) ? 1ull : 0ull;
    const unsigned long long ext = v < 0 ? ~0ull : 0ull;
    const unsigned long long h = ext + carry;
    if (h) atomicAdd(hi, h);
}

template <int NP>
__global__ __launch_bounds__(kBlock) void k_balance_stats(
    const double *__restrict__ x, const double *__restrict__ y, const double *__restrict__ z,
    int64_t n, const int32_t *__restrict__ owner, const int32_t *__restrict__ nbr_count,
    const double *__restrict__ sites, int K, int W, int bounds_from, double dsh,
    unsigned long long *__restrict__ g_part, unsigned long long *__restrict__ g_pairs,
    unsigned long long *__restrict__ g_sum, uint32_t *__restrict__ adj) {
    extern __shared__ double smem[];
    double *gs = smem;                                                   // 3K
    unsigned long long *s_lo = (unsigned long long *)(gs + 3 * K);       // 3K
    unsigned long long *s_hi = s_lo + 3 * K;                             // 3K
    unsigned long long *s_pairs = s_hi + 3 * K;                          // K
    unsigned int *s_part = (unsigned int *)(s_pairs + K);                // K
    uint32_t *s_tri = s_part + K;                                        // tri_words(K)
    for (int k = threadIdx.x; k < 3 * K; k += kBlock) {
        gs[k] = sites[k];
        s_lo[k] = 0ull;
        s_hi[k] = 0ull;
    }
    for (int k = threadIdx.x; k < K; k += kBlock) {
        s_pairs[k] = 0ull;
        s_part[k] = 0u;
    }
    for (int q = threadIdx.x; q < tri_words(K); q += kBlock) s_tri[q] = 0u;
    __syncthreads();
    const double lim = 4.0 * (dsh * dsh);
    const NearTiles run = near_tiles<NP>(n);
    for (int64_t tile = run.at; tile < run.end; ++tile) {
        const int64_t i0 = tile * (64 * NP) + (threadIdx.x & 63);
        LaneParticles<NP> w;
        int k[NP];
        long long v[NP][3];
        unsigned long long pc[NP];
        bool any = false, large = false;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int64_t i = i0 + 64 * q;
            const int kr = i < n ? owner[i] : -1;
            w.on[q] = kr >= 0 && kr < K;
            any = any || w.on[q];
            k[q] = w.on[q] ? kr : 0;
            w.p[q][0] = w.on[q] ? x[i] : 0.0;
            w.p[q][1] = w.on[q] ? y[i] : 0.0;
            w.p[q][2] = w.on[q] ? z[i] : 0.0;
            pc[q] = w.on[q] && nbr_count ? (unsigned long long)nbr_count[i] : 0ull;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const double f =
                    fmin(fmax((w.p[q][d] - gs[3 * k[q] + d]) * kFix, -kFixMax), kFixMax);
                v[q][d] = __double2ll_rn(f);
                large = large || (w.on[q] && fabs(f) >= kFixWave);
            }
        }
        if (!__any(any)) continue;
        bool on[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) on[q] = w.on[q];
        // the wave's sums per owner (exact integers), added by one lane
        if (!__any(large))
            for_owners<NP>(on, k, [&](int k0, const bool(&mine)[NP], int count) {
                unsigned long long sp = 0, sv[3] = {0, 0, 0};
#pragma unroll
                for (int q = 0; q < NP; ++q) {
                    sp += mine[q] ? pc[q] : 0ull;
#pragma unroll
                    for (int d = 0; d < 3; ++d)
                        sv[d] += mine[q] ? (unsigned long long)v[q][d] : 0ull;
                }
                if (nbr_count) sp = wave_all_sum(sp);
#pragma unroll
                for (int d = 0; d < 3; ++d) sv[d] = wave_all_sum(sv[d]);
                if ((threadIdx.x & 63) == 0) {
                    atomicAdd(&s_part[k0], (unsigned)count);
                    if (nbr_count) atomicAdd(&s_pairs[k0], sp);
#pragma unroll
                    for (int d = 0; d < 3; ++d)
                        add128(&s_lo[3 * k0 + d], &s_hi[3 * k0 + d], (long long)sv[d]);
                }
            });
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            if (!on[q]) continue;
            atomicAdd(&s_part[k[q]], 1u);
            if (nbr_count) atomicAdd(&s_pairs[k[q]], pc[q]);
#pragma unroll
            for (int d = 0; d < 3; ++d) add128(&s_lo[3 * k[q] + d], &s_hi[3 * k[q] + d], v[q][d]);
        }
        if (K > 1) {
            // nearest other generator (ties to the smaller index) and the owner's distance
            double bd[NP];
            int best[NP];
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                bd[q] = INFINITY;
                best[q] = -1;
            }
            near_sites<true, NP>(gs, K, bounds_from, w, [&](int l, double gx, double gy, double gz) {
#pragma unroll
                for (int q = 0; q < NP; ++q) {
                    const double d2 = norm2(w.p[q][0] - gx, w.p[q][1] - gy, w.p[q][2] - gz);
                    if (l != k[q] && d2 < bd[q]) {
                        bd[q] = d2;
                        best[q] = l;
                    }
                }
            });
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                // best < 0: no finite distance to another generator
                const int a = k[q], b = best[q] < 0 ? a : best[q];
                const double d2o = norm2(w.p[q][0] - gs[3 * a], w.p[q][1] - gs[3 * a + 1],
                                         w.p[q][2] - gs[3 * a + 2]);
                const double gg = norm2(gs[3 * b] - gs[3 * a], gs[3 * b + 1] - gs[3 * a + 1],
                                        gs[3 * b + 2] - gs[3 * a + 2]);
                const double u = __dsub_rn(bd[q], d2o);
                if (!w.on[q] || best[q] < 0 || !(__dmul_rn(u, u) < __dmul_rn(lim, gg))) continue;
                const int hi = max(a, b), bit = hi * (hi - 1) / 2 + min(a, b);
                const uint32_t m = 1u << (bit & 31);
                if (!(s_tri[bit >> 5] & m)) atomicOr(&s_tri[bit >> 5], m);
            }
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += kBlock) {
        if (s_part[k]) atomicAdd(&g_part[k], (unsigned long long)s_part[k]);
        if (s_pairs[k]) atomicAdd(&g_pairs[k], s_pairs[k]);
    }
    // the lower triangle, a word (a, w) of 32 pairs b < a at a time (bits a (a - 1) / 2 + 32 w on),
    // where the matrix lacks some: every workgroup of scattered particles meets every pair, and an
    // atomic a pair took most of 378 us for 1 M of them and 16 generators (47 us now)
    for (int q = threadIdx.x; q < K * W; q += kBlock) {
        const int a = q / W, b0 = 32 * (q - a * W), t = a * (a - 1) / 2 + b0;
        if (b0 >= a) continue;
        const int word = t >> 5, sh = t & 31;
        uint32_t m = s_tri[word] >> sh;
        if (sh && word + 1 < tri_words(K)) m |= s_tri[word + 1] << (32 - sh);
        if (a - b0 < 32) m &= (1u << (a - b0)) - 1u;
        if (m & ~__hip_atomic_load(&adj[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicOr(&adj[q], m);
    }
    for (int k = threadIdx.x; k < 3 * K; k += kBlock) {
        const unsigned long long lo = s_lo[k], hi = s_hi[k];
        if (lo == 0ull && hi == 0ull) continue;
        // add the block's 128-bit value {lo, hi}
        const unsigned long long old = atomicAdd(&g_sum[k], lo);
        const unsigned long long carry = (old + lo < old) ? 1ull : 0ull;
        if (hi + carry) atomicAdd(&g_sum[3 * K + k], hi + carry);
    }
}

// centre = g + sum / (2^32 N) (the generator itself for an empty subdomain);
// counts to int64 outputs.
__global__ __launch_bounds__(kBlock) void k_balance_finish(
    const double *__restrict__ sites, int K, const unsigned long long *__restrict__ g_part,
    const unsigned long long *__restrict__ g_pairs, const unsigned long long *__restrict__ g_sum,
    int64_t *__restrict__ site_particles, int64_t *__restrict__ site_pairs,
    double *__restrict__ centre, uint32_t *__restrict__ adj, int W) {
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k < K * W) {  // the touching pairs' upper triangle: word (a, w) holds b = 32 w on, b < a
        const int a = k / W, b0 = 32 * (k - a * W);
        uint32_t m = b0 < a ? __hip_atomic_load(&adj[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                            : 0u;
        if (a - b0 < 32) m &= b0 < a ? (1u << (a - b0)) - 1u : 0u;
        for (; m; m &= m - 1)
            atomicOr(&adj[(size_t)(b0 + __ffs(m) - 1) * W + (a >> 5)], 1u << (a & 31));
    }
    if (k >= K) return;
    const unsigned long long np = g_part[k];
    if (site_particles) site_particles[k] = (int64_t)np;
    if (site_pairs) site_pairs[k] = (int64_t)g_pairs[k];
    for (int d = 0; d < 3; ++d) {
        double c = sites[3 * k + d];
        if (np) {
            const unsigned long long lo = g_sum[3 * k + d];
            const long long hi = (long long)g_sum[3 * K + 3 * k + d];
            // hi 2^64 + lo with the first addition exact for |hi| < 2^20
            const double s = ((double)hi * 18446744073709551616.0 +
                              (double)(lo >> 32) * 4294967296.0) +
                             (double)(lo & 0xffffffffull);
            c += s / (kFix * (double)np);
        }
        centre[3 * k + d] = c;
    }
}

// ------------------------------------------------------------------ move

struct V3 {
    double x, y, z;
};
__device__ __forceinline__ V3 operator+(V3 a, V3 b) { return {a.x + b.x, a.y + b.y, a.z + b.z}; }
__device__ __forceinline__ V3 operator-(V3 a, V3 b) { return {a.x - b.x, a.y - b.y, a.z - b.z}; }
__device__ __forceinline__ V3 operator*(double s, V3 a) { return {s * a.x, s * a.y, s * a.z}; }
__device__ __forceinline__ double dot(V3 a, V3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ V3 cross(V3 a, V3 b) {
    return {a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x};
}

// Rotate v by angle a about the axis along u (right hand), Rodrigues' form.
__device__ V3 rotate(V3 v, V3 u, double a) {
    const double inv = 1.0 / sqrt(dot(u, u));
    u = inv * u;
    double s, c;
    sincos(a, &s, &c);
    return c * v + s * cross(u, v) + (dot(u, v) * (1.0 - c)) * u;
}

// One wave moves generator k = blockIdx.x.  A lane takes one neighbour l, then one triplet
// (l, m), at a time; the terms of up to 64 of them are then added in the order of (l, m), so the
// sums are those of a plain loop.  With a thread per generator the whole move was the chain of
// the longest generator's ~40 triplets, a few microseconds each (64 generators: 120 -> 13 us,
// and 5 us for the sum of the moves).
__global__ __launch_bounds__(64) void k_balance_move(
    const double *__restrict__ sites, int K, int W, const int64_t *__restrict__ loads,
    const double *__restrict__ centre, const uint32_t *__restrict__ adj, double sigma,
    double theta, double gamma, double dsh, double *__restrict__ out) {
    extern __shared__ double sm[];
    double *sg = sm;                         // 3K generators
    double *sL = sg + 3 * K;                 // K loads
    double *term = sL + K;                   // 64 terms of 3
    uint32_t *sa = (uint32_t *)(term + 192); // K x W adjacency words
    const int k = blockIdx.x, lane = threadIdx.x;
    for (int q = lane; q < 3 * K; q += 64) sg[q] = sites[q];
    for (int q = lane; q < K; q += 64) sL[q] = (double)loads[q];
#pragma unroll 8
    for (int q = lane; q < K * W; q += 64) sa[q] = adj[q];
    __syncthreads();
    const V3 gk{sg[3 * k], sg[3 * k + 1], sg[3 * k + 2]};
    const double Lk = sL[k];
    const uint32_t *rk = sa + (size_t)k * W;
    // adds the first `count` lanes' terms to sum in lane order (the same in every lane)
    auto add_terms = [&](V3 &sum, const V3 &t, bool counts, int count) {
        term[3 * lane] = t.x;
        term[3 * lane + 1] = t.y;
        term[3 * lane + 2] = t.z;
        const unsigned long long m = __ballot(counts);
        __syncthreads();
        for (int q = 0; q < count; ++q) {
            if (!((m >> q) & 1ull)) continue;
            sum = sum + V3{term[3 * q], term[3 * q + 1], term[3 * q + 2]};
        }
        __syncthreads();
    };
    V3 two{0.0, 0.0, 0.0}, three{0.0, 0.0, 0.0};
    int myl = 0, mym = 0, queued = 0;
    auto flush_two = [&]() {
        V3 t{0.0, 0.0, 0.0};
        bool counts = false;
        if (lane < queued) {
            const V3 gl{sg[3 * myl], sg[3 * myl + 1], sg[3 * myl + 2]};
            const double Ll = sL[myl];
            const V3 gkl = gk - gl;
            const double nd = sqrt(dot(gkl, gkl));
            counts = Lk + Ll != 0.0 && nd != 0.0;
            if (counts) t = (dsh * (Lk - Ll) / (Lk + Ll) / nd) * gkl;
        }
        add_terms(two, t, counts, queued);
        queued = 0;
    };
    auto flush_three = [&]() {
        V3 t{0.0, 0.0, 0.0};
        bool counts = false;
        if (lane < queued) {
            const V3 gl{sg[3 * myl], sg[3 * myl + 1], sg[3 * myl + 2]};
            const V3 gm{sg[3 * mym], sg[3 * mym + 1], sg[3 * mym + 2]};
            const double Ll = sL[myl], Lm = sL[mym];
            const double S = Lk + Ll + Lm;
            // circumcentre of the triangle (g_k, g_l, g_m)
            const V3 a = gl - gk, b = gm - gk;
            const V3 nrm = cross(a, b);
            const double n2 = dot(nrm, nrm);
            if (S != 0.0 && n2 > 1e-24 * dot(a, a) * dot(b, b)) {
                const V3 o = gk + (0.5 / n2) * cross(dot(a, a) * b - dot(b, b) * a, nrm);
                const V3 ck = gk - o, cl = gl - o, cm = gm - o;
                const V3 axl = cross(ck, cl), axm = cross(ck, cm);
                counts = dot(axl, axl) != 0.0 && dot(axm, axm) != 0.0;
                if (counts) {
                    const double al = (M_PI / 3.0) * (Ll - Lk) / S;
                    const double am = (M_PI / 3.0) * (Lm - Lk) / S;
                    t = rotate(rotate(ck, axl, al), axm, am) - ck;
                }
            }
        }
        add_terms(three, t, counts, queued);
        queued = 0;
    };
    // the wave hands out neighbours, then triplets, in order (wave-uniform loops)
    auto each_neighbour = [&](auto &&f) {
        for (int wl = 0; wl < W; ++wl)
            for (uint32_t bl = __builtin_amdgcn_readfirstlane(rk[wl]) &
                               ~(wl == (k >> 5) ? (1u << (k & 31)) : 0u);
                 bl; bl &= bl - 1)
                f(wl * 32 + __ffs(bl) - 1);
    };
    each_neighbour([&](int l) {
        if (lane == queued) myl = l;
        if (++queued == 64) flush_two();
    });
    if (queued) flush_two();
    each_neighbour([&](int l) {
        // m > l touching both k and l: the intersection of rows k and l
        const uint32_t *rl = sa + (size_t)l * W;
        for (int wm = l >> 5; wm < W; ++wm) {
            uint32_t bm = __builtin_amdgcn_readfirstlane(rk[wm] & rl[wm]);
            if (wm == (l >> 5)) bm &= ~((2u << (l & 31)) - 1u);  // m > l
            if (wm == (k >> 5)) bm &= ~(1u << (k & 31));         // m != k
            for (; bm; bm &= bm - 1) {
                if (lane == queued) {
                    myl = l;
                    mym = wm * 32 + __ffs(bm) - 1;
                }
                if (++queued == 64) flush_three();
            }
        }
    });
    if (queued) flush_three();
    const double nt = sqrt(dot(three, three));
    if (nt > dsh) three = (dsh / nt) * three;
    const V3 dg = (1.0 - sigma) * two + sigma * three;
    const V3 rc{centre[3 * k], centre[3 * k + 1], centre[3 * k + 2]};
    const V3 g2 = (1.0 - theta) * (gk + gamma * dg) + theta * rc;
    if (lane == 0) {
        out[3 * k] = g2.x;
        out[3 * k + 1] = g2.y;
        out[3 * k + 2] = g2.z;
    }
}

// sum_k |g'_k - g_k| in a fixed tree (one workgroup of a power of two >= K threads).
__global__ __launch_bounds__(1024) void k_balance_moved(const double *__restrict__ sites, int K,
                                                        const double *__restrict__ out,
                                                        double *__restrict__ move_sum) {
    __shared__ double red[1024];
    const int k = threadIdx.x;
    double mv = 0.0;
    if (k < K) {
        const V3 d = V3{out[3 * k], out[3 * k + 1], out[3 * k + 2]} -
                     V3{sites[3 * k], sites[3 * k + 1], sites[3 * k + 2]};
        mv = sqrt(dot(d, d));
    }
    red[threadIdx.x] = mv;
    __syncthreads();
    for (int st = blockDim.x / 2; st > 0; st >>= 1) {
        if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
        __syncthreads();
    }
    if (threadIdx.x == 0) *move_sum = red[0];
}

size_t balance_ws_bytes(int K) { return (size_t)K * 8 * sizeof(unsigned long long) + 256; }

hipError_t launch_balance_stats(const double *x, const double *y, const double *z, int64_t n,
                                const int32_t *owner, const int32_t *nbr_count,
                                const double *sites, int K, double dsh, int64_t *site_particles,
                                int64_t *site_pairs, double *centre, uint32_t *adj, void *ws,
                                hipStream_t st) {
    const int W = (K + 31) / 32;
    unsigned long long *g_part = (unsigned long long *)ws;   // K
    unsigned long long *g_pairs = g_part + K;                // K
    unsigned long long *g_sum = g_pairs + K;                 // 6K: lo[3K], hi[3K]
    launch_zero2(g_part, 16 * K, adj, K * W, st);
    if (n > 0) {
        const unsigned nb = near_blocks(n, near_per(n), kReduceBlocks);
        const size_t shm = (size_t)K * (3 * sizeof(double) + 7 * sizeof(unsigned long long) +
                                        sizeof(unsigned int)) +
                           sizeof(uint32_t) * tri_words(K);
        (near_per(n) == 1 ? k_balance_stats<1> : k_balance_stats<kNearPer>)<<<nb, kBlock, shm, st>>>(
            x, y, z, n, owner, nbr_count, sites, K, W, near_min(n), dsh, g_part, g_pairs, g_sum, adj);
    }
    k_balance_finish<<<(unsigned)((K * W + kBlock - 1) / kBlock), kBlock, 0, st>>>(
        sites, K, g_part, g_pairs, g_sum, site_particles, site_pairs, centre, adj, W);
    return hipGetLastError();
}

hipError_t launch_balance_move(const double *sites, int K, const int64_t *loads,
                               const double *centre, const uint32_t *adj, double sigma,
                               double theta, double gamma, double dsh, double *out,
                               double *move_sum, hipStream_t st) {
    const int W = (K + 31) / 32;
    // the sum's threads: one per generator, rounded up to whole waves
    int nt = 64;
    while (nt < K) nt *= 2;
    const size_t shm = sizeof(double) * (4 * (size_t)K + 192) + sizeof(uint32_t) * (size_t)K * W;
    k_balance_move<<<(unsigned)K, 64, shm, st>>>(sites, K, W, loads, centre, adj, sigma, theta,
                                                 gamma, dsh, out);
    k_balance_moved<<<1, nt, 0, st>>>(sites, K, out, move_sum);
    return hipGetLastError();
}

}  // namespace csph
