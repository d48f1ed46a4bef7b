// Voronoi generators near a wave's particles, and the wave sums of per-generator counts.
//
// The argmin over K generators costs ~10 FP64 operations and a selection per particle and
// generator, all of them for generators far outside the wave's reach: a wave's particles are
// neighbours in cell order.  The wave therefore bounds its particles by a box, a lane per
// generator bounds that generator's squared distance to the box from both sides, and only the
// generators whose lower bound does not exceed the smallest upper bound are scanned, in the
// same order and by the same expressions, so the argmin and its ties are the full scan's.
// 2.9 M particles and 64 generators: ownership with counts 82 -> 53 us (its 93 MB take 17 us at
// 5.5 TB/s; the rest is the wave's bounds and sums), the balancer's statistics 448 -> 85 us.
#pragma once

#include "csph_internal.h"
#include "wave.h"

#include <climits>
#include <type_traits>

namespace csph {

// Generators from which on a pass over n particles takes the bounds: below kNearMin they (about as
// much work as scanning 8 generators) are left out, and so they are where the chip has a wave a SIMD
// at most, whose time goes with the length of its chain (5 000 particles in cell order, 512
// generators: ownership 44 us with the bounds, 31 without).
constexpr int kNearMin = 12;
constexpr int64_t kNearFew = 1 << 16;
inline int near_min(int64_t n) { return n <= kNearFew ? INT_MAX : kNearMin; }

// Particles a lane holds in the passes over particles alone: the box, the bounds and the sums
// below are paid once per 256 consecutive particles, whose box is hardly larger than 64's (a
// cell row's worth and its neighbours).
// In smaller sets, a particle each: up to kNearOne that leaves the chip's 4 096 waves a tile each at
// most.  Ownership by 512 generators, one against four a lane: 100 000 particles 46 and 86 us,
// 260 000 75 (scattered) or 65 and 89 or 86, 500 000 161 or 116 and 123 or 105.
constexpr int kNearPer = 4;
constexpr int64_t kNearOne = 1 << 18;
inline int near_per(int64_t n) { return n <= kNearOne ? 1 : kNearPer; }

// Minimum of a wave's 64 integers (every lane active); the result is wave-uniform.
__device__ __forceinline__ int wave_all_min(int v) {
    v = min(v, row_ror<8>(v));
    v = min(v, row_ror<4>(v));
    v = min(v, row_ror<2>(v));
    v = min(v, row_ror<1>(v));
    return min(min(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
               min(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// The same of floats, as integers of the same order (exact; no NaN among them).
__device__ __forceinline__ int float_order(int b) { return b ^ ((b >> 31) & 0x7fffffff); }
__device__ __forceinline__ float wave_all_min(float v) {
    return __int_as_float(float_order(wave_all_min(float_order(__float_as_int(v)))));
}

// Sum of a wave's 64 integers (every lane active; wave-uniform).
__device__ __forceinline__ unsigned long long wave_all_sum(unsigned long long v) {
#define CSPH_ROR(N)                                                                      \
    v += (unsigned long long)(unsigned)row_ror<N>((int)(unsigned)v) |                    \
         (unsigned long long)(unsigned)row_ror<N>((int)(unsigned)(v >> 32)) << 32;
    CSPH_ROR(8) CSPH_ROR(4) CSPH_ROR(2) CSPH_ROR(1)
#undef CSPH_ROR
    unsigned long long s = 0;
#pragma unroll
    for (int r = 0; r < 64; r += 16)
        s += (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, r) |
             (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), r)
                 << 32;
    return s;
}

// The NP particles of a lane; on: it is there.
template <int NP>
struct LaneParticles {
    bool on[NP];
    double p[NP][3];
};

// Calls each(k, its x, y, z), k ascending and wave-uniform, for every generator that can be the nearest
// (SECOND: the nearest but for one that the particle leaves out) of some particle of the wave;
// now and then a k comes twice in a row.  gs: the generators (3 K doubles, LDS).  Every lane of
// the wave calls it, and each runs in every lane.  bounds_from: near_min of the pass.
//
// The bounds are FP32 with margins: a coordinate rounds by 2^-24 of itself and is widened by
// 2^-22, the squared bounds by 1e-5 (their few roundings are below 1e-6) and 1e-36 (underflow).
// Coordinates beyond FP32's squares give an infinite threshold, which admits every generator;
// a NaN coordinate is left out of the box (its particle has no nearest generator) and a NaN
// bound admits its generator.
template <bool SECOND, int NP, typename F>
__device__ __forceinline__ void near_sites(const double *gs, int K, int bounds_from,
                                           const LaneParticles<NP> &w, F &&each) {
    constexpr float kWide = 2.384185791015625e-7f;  // 2^-22
    const int lane = threadIdx.x & 63;
    float lo[3], hi[3], thr = 0.0f;
    // the generators l0 + lane that the bounds admit
    auto admitted = [&](int l0) {
        const int l = l0 + lane;
        bool in = l < K;
        if (in) {
            float d2 = 0.0f;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float g = (float)gs[3 * l + a], e = fabsf(g) * kWide;
                const float f = fmaxf(fmaxf(lo[a] - g, g - hi[a]) - e, 0.0f);
                d2 += f * f;
            }
            in = !(d2 * (1.0f - 1e-5f) > thr);
        }
        return (unsigned long long)__ballot(in);
    };
    bool all = K < bounds_from;
    if (!all) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float l = INFINITY, h = INFINITY;  // minima of x and of -x
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                const float p = (float)w.p[q][a], e = fabsf(p) * kWide;
                const float pl = p - e, ph = -p - e;  // NaN where p is NaN or an infinity of that side
                l = w.on[q] && pl < l ? pl : l;
                h = w.on[q] && ph < h ? ph : h;
            }
            lo[a] = wave_all_min(l);
            hi[a] = -wave_all_min(h);
        }
        float m1 = INFINITY, m2 = INFINITY;  // the lane's smallest (and second) upper bounds
        for (int l = lane; l < K; l += 64) {
            float d2 = 0.0f;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float g = (float)gs[3 * l + a];
                const float f = fmaxf(hi[a] - g, g - lo[a]) + fabsf(g) * kWide;
                d2 += f * f;
            }
            if (SECOND && d2 < m2) m2 = d2 < m1 ? m1 : d2;
            if (d2 < m1) m1 = d2;
        }
        thr = wave_all_min(m1);
        if (SECOND) {  // the smallest left when one lane gives up that minimum
            const int f = __ffsll((unsigned long long)__ballot(m1 == thr)) - 1;
            thr = wave_all_min(lane == f ? m2 : m1);
        }
        thr = thr * (1.0f + 1e-5f) + 1e-36f;
        // scattered particles admit nearly all generators (the first 64 tell): the plain loop, with
        // more LDS reads ahead, is the faster one (3 M such, 512 generators: 595 against 649 us)
        all = 8 * __popcll(admitted(0)) > 7 * min(K, 64);
    }
    // B generators at a time, their LDS reads ahead of the comparisons
    auto in_turn = [&](auto width, int k0) {
        constexpr int B = decltype(width)::value;
        double g[B][3];
#pragma unroll
        for (int u = 0; u < B; ++u)
#pragma unroll
            for (int a = 0; a < 3; ++a) g[u][a] = gs[3 * (k0 + u) + a];
#pragma unroll
        for (int u = 0; u < B; ++u) each(k0 + u, g[u][0], g[u][1], g[u][2]);
    };
    if (all) {
        constexpr int B = NP == 1 ? 8 : 4;
        int k = 0;
        for (; k + B <= K; k += B) in_turn(std::integral_constant<int, B>{}, k);
        for (; k < K; ++k) in_turn(std::integral_constant<int, 1>{}, k);
        return;
    }
    for (int l0 = 0; l0 < K; l0 += 64) {
        // two at a time, so that one's LDS reads pass while the other is compared
        for (unsigned long long m = admitted(l0); m;) {
            const int k0 = l0 + __ffsll(m) - 1;
            m &= m - 1;
            const int k1 = m ? l0 + __ffsll(m) - 1 : k0;
            m &= m - 1;
            const double x0 = gs[3 * k0], y0 = gs[3 * k0 + 1], z0 = gs[3 * k0 + 2];
            const double x1 = gs[3 * k1], y1 = gs[3 * k1 + 1], z1 = gs[3 * k1 + 2];
            each(k0, x0, y0, z0);
            each(k1, x1, y1, z1);
        }
    }
}

// The nearest generator of each particle (FP64 argmin, ties to the smaller index).
template <int NP>
__device__ __forceinline__ void nearest_site(const double *gs, int K, int bounds_from,
                                             const LaneParticles<NP> &w, int (&best)[NP]) {
    double bd[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        best[q] = 0;
        bd[q] = INFINITY;
    }
    near_sites<false, NP>(gs, K, bounds_from, w, [&](int k, double gx, double gy, double gz) {
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const double dx = w.p[q][0] - gx, dy = w.p[q][1] - gy, dz = w.p[q][2] - gz;
            const double d2 = ((dx * dx) + (dy * dy)) + (dz * dz);
            if (d2 < bd[q]) {
                bd[q] = d2;
                best[q] = k;
            }
        }
    });
}

// Calls one(k, mine, count) for up to kOwnersAtOnce of the values k[] that the particles with
// on[] hold (mine[q]: this one does; count: how many of the wave's do), every lane of the wave
// taking part; on[] is left set for the particles still to be counted.  A wave of neighbouring
// particles holds a few owners: their sums then cost one atomic per wave instead of one per
// particle to one address, which LDS takes in turn.
constexpr int kOwnersAtOnce = 6;

template <int NP, typename F>
__device__ __forceinline__ void for_owners(bool (&on)[NP], const int (&k)[NP], F &&one) {
    for (int t = 0; t < kOwnersAtOnce; ++t) {
        int k0 = -1;
#pragma unroll
        for (int q = NP - 1; q >= 0; --q) {
            const unsigned long long left = __ballot(on[q]);
            if (left) k0 = __builtin_amdgcn_readlane(k[q], __ffsll(left) - 1);
        }
        if (k0 < 0) return;
        bool mine[NP];
        int count = 0;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            mine[q] = on[q] && k[q] == k0;
            count += __popcll(__ballot(mine[q]));
            on[q] = on[q] && !mine[q];
        }
        one(k0, mine, count);
    }
}

// Particle and pair counts of the owners (LDS counters hp, hq).
template <int NP>
__device__ __forceinline__ void count_owners(const bool (&there)[NP], const int (&owner)[NP],
                                             bool pairs, const int32_t (&cnt)[NP],
                                             unsigned int *hp, unsigned long long *hq) {
    bool on[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) on[q] = there[q];
    for_owners<NP>(on, owner, [&](int k, const bool (&mine)[NP], int count) {
        unsigned long long s = 0;
        if (pairs) {
#pragma unroll
            for (int q = 0; q < NP; ++q) s += mine[q] ? (unsigned long long)(long long)cnt[q] : 0;
            s = wave_all_sum(s);
        }
        if ((threadIdx.x & 63) == 0) {
            atomicAdd(&hp[k], (unsigned)count);
            if (pairs) atomicAdd(&hq[k], s);
        }
    });
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        if (!on[q]) continue;
        atomicAdd(&hp[owner[q]], 1u);
        if (pairs) atomicAdd(&hq[owner[q]], (unsigned long long)(long long)cnt[q]);
    }
}

// The tiles of 64 NP particles a wave takes: consecutive ones, a workgroup's waves side by
// side, so that a workgroup meets few generators and adds few of them to the totals at its end.
struct NearTiles {
    int64_t at, end;
};
template <int NP>
__device__ __forceinline__ NearTiles near_tiles(int64_t n) {
    const int64_t tiles = (n + 64 * NP - 1) / (64 * NP);
    const int64_t waves = (int64_t)gridDim.x * (kBlock / 64);
    const int64_t w = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    return NearTiles{w * tiles / waves, (w + 1) * tiles / waves};
}
// Workgroups for them, `most` at most.
inline unsigned near_blocks(int64_t n, int np, int64_t most) {
    const int64_t tiles = (n + 64 * np - 1) / (64 * np);
    const int64_t want = (tiles + kBlock / 64 - 1) / (kBlock / 64);
    return (unsigned)(want > most ? most : want);
}

// Two arrays of 32-bit words set to 0 by one launch (k_voronoi.hip; b may be null).
hipError_t launch_zero2(void *a, int64_t na, void *b, int64_t nb, hipStream_t st);

}  // namespace csph
