// Voronoi ownership (eq. VoronoiDefinition, sec. 3.1) and per-site load
// counts.  Generators sit in LDS; each particle takes the FP64 argmin of
// its squared distance in a fixed operation order without contraction,
// scanning k upwards with a strict comparison so a tie keeps the smaller k,
// over the generators that can be nearest to some particle of its wave
// (nearest.h).  Counts are integers (wave sums, LDS atomics per block, then one
// global atomic per site and block), hence exact and order independent.
#include "csph_internal.h"
#include "nearest.h"

namespace csph {

__global__ __launch_bounds__(kBlock) void k_zero2(uint32_t *a, int64_t na, uint32_t *b,
                                                  int64_t nb) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < na) a[i] = 0u;
    if (i < nb) b[i] = 0u;
}

hipError_t launch_zero2(void *a, int64_t na, void *b, int64_t nb, hipStream_t st) {
    if (!b) nb = 0;
    const int64_t len = na > nb ? na : nb;
    if (len <= 0) return hipSuccess;
    k_zero2<<<(unsigned)((len + kBlock - 1) / kBlock), kBlock, 0, st>>>((uint32_t *)a, na,
                                                                        (uint32_t *)b, nb);
    return hipGetLastError();
}

template <int NP>
__global__ __launch_bounds__(kBlock) void k_voronoi(const double *__restrict__ x,
                                                    const double *__restrict__ y,
                                                    const double *__restrict__ z, int64_t n,
                                                    const double *__restrict__ sites, int K,
                                                    int bounds_from,
                                                    const int32_t *__restrict__ nbr_count,
                                                    int32_t *__restrict__ owner,
                                                    unsigned long long *__restrict__ site_part,
                                                    unsigned long long *__restrict__ site_pairs) {
    extern __shared__ double smem[];
    double *gs = smem;                                                  // 3K
    unsigned long long *hq = (unsigned long long *)(smem + 3 * K);      // K
    unsigned int *hp = (unsigned int *)(hq + K);                        // K
    for (int k = threadIdx.x; k < 3 * K; k += kBlock) gs[k] = sites[k];
    for (int k = threadIdx.x; k < K; k += kBlock) {
        hp[k] = 0u;
        hq[k] = 0ull;
    }
    __syncthreads();
    const NearTiles mine = near_tiles<NP>(n);
    for (int64_t tile = mine.at; tile < mine.end; ++tile) {
        const int64_t i0 = tile * (64 * NP) + (threadIdx.x & 63);
        LaneParticles<NP> w;
        int32_t c[NP];
        int best[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int64_t i = i0 + 64 * q;
            w.on[q] = i < n;
            w.p[q][0] = w.on[q] ? x[i] : 0.0;
            w.p[q][1] = w.on[q] ? y[i] : 0.0;
            w.p[q][2] = w.on[q] ? z[i] : 0.0;
            c[q] = nbr_count && w.on[q] ? nbr_count[i] : 0;
        }
        nearest_site<NP>(gs, K, bounds_from, w, best);
#pragma unroll
        for (int q = 0; q < NP; ++q)
            if (w.on[q]) owner[i0 + 64 * q] = best[q];
        count_owners<NP>(w.on, best, nbr_count != nullptr, c, hp, hq);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += kBlock) {
        if (hp[k]) atomicAdd(&site_part[k], (unsigned long long)hp[k]);
        if (site_pairs && hq[k]) atomicAdd(&site_pairs[k], hq[k]);
    }
}

hipError_t launch_voronoi(const double *x, const double *y, const double *z, int64_t n,
                          const double *sites, int K, const int32_t *nbr_count, int32_t *owner,
                          int64_t *site_particles, int64_t *site_pairs, hipStream_t st) {
    launch_zero2(site_particles, 2 * K, site_pairs, 2 * K, st);
    if (n > 0) {
        const unsigned nb = near_blocks(n, near_per(n), kReduceBlocks);
        size_t shm = (size_t)K * (3 * sizeof(double) + sizeof(unsigned long long) + sizeof(unsigned));
        (near_per(n) == 1 ? k_voronoi<1> : k_voronoi<kNearPer>)<<<nb, kBlock, shm, st>>>(
            x, y, z, n, sites, K, near_min(n), site_pairs ? nbr_count : nullptr, owner,
            (unsigned long long *)site_particles, (unsigned long long *)site_pairs);
    }
    return hipGetLastError();
}

}  // namespace csph
