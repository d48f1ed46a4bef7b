// Stencil walk shared by the pair kernels (rates and their adjoint): the
// rows of cells a particle's support sphere reaches, and the per-lane
// partner rings in LDS.
#pragma once

#include "csph_internal.h"

namespace csph {

// ---------------------------------------------------------------- partner queues
//
// A candidate test costs ~20 instructions, a pair interaction ~50.  Testing
// and interacting in the same loop would run the pair arithmetic whenever
// any lane of the wave accepts a candidate, with the other lanes idle (a
// particle accepts ~15-40 % of its candidates).  Instead each lane appends
// its accepted partners to a small ring in LDS while the wave walks the
// stencil in lock step, and as soon as some lane's ring is nearly full every
// lane pops one partner and the wave runs the pair arithmetic with (nearly)
// all lanes busy.  A lane's partners are summed in the order it popped them,
// which depends only on the input: results are reproducible.
//
// Each stencil row (cells cx-R..cx+R at fixed y, z) is clipped to the chord
// the support sphere of particle i cuts through it, with a safety margin,
// so that with cells smaller than the support the lanes test little more
// than the sphere.  The clipping only drops candidates that cannot be
// partners; membership is decided by the pair test itself.

constexpr int kQ = 8;  // ring slots per lane
constexpr int kU = 2;  // candidates tested per lock-step iteration

// Load base[idx] with a 32-bit byte offset from a wave-uniform base (records
// stay below 4 GiB), which keeps the address arithmetic in one VGPR.
template <typename T>
__device__ __forceinline__ T ld(const T *__restrict__ base, int idx) {
    return *(const T *)((const char *)base + (uint32_t)idx * (uint32_t)sizeof(T));
}

// Records of four doubles kept as two arrays of 16-byte halves (n records each): a wave
// gathering the records of neighbouring particles then reads whole lines in each of its two
// loads, where an array of 32-byte records gives it every other 16 bytes of twice the lines.
// off: the record's byte offset in either array (16 j).
struct Split4 {
    const double2 *__restrict__ lo;
    const double2 *__restrict__ hi;
    __device__ __forceinline__ double4 at(uint32_t off) const {
        const double2 a = *(const double2 *)((const char *)lo + off);
        const double2 b = *(const double2 *)((const char *)hi + off);
        return make_double4(a.x, a.y, b.x, b.y);
    }
    __device__ __forceinline__ double4 operator[](int64_t j) const {
        return make_double4(lo[j].x, lo[j].y, hi[j].x, hi[j].y);
    }
};
inline Split4 split4(const void *rec, int64_t n) {
    return Split4{(const double2 *)rec, (const double2 *)rec + n};
}

// The same records whole (off: 32 j), for Verlet-list steps: a list's partners are scattered, and
// a record in one place is one line to fetch.  FP64 list steps, whole against split: 1 M particles
// 1 397 against 1 465 us, 262 144 407 against 434; 8 000, whose records stay in the caches, 164
// against 155.
struct Whole4 {
    const double4 *__restrict__ rec;
    __device__ __forceinline__ double4 at(uint32_t off) const {
        return *(const double4 *)((const char *)rec + off);
    }
    __device__ __forceinline__ double4 operator[](int64_t j) const { return rec[j]; }
};

// The records of a stencil walk, or (LIST) of a Verlet-list step.
template <bool LIST>
struct Rec4 {
    using type = Split4;
    static type make(const void *rec, int64_t n) { return split4(rec, n); }
};
template <>
struct Rec4<true> {
    using type = Whole4;
    static type make(const void *rec, int64_t) { return Whole4{(const double4 *)rec}; }
};

// A wave-uniform float in a scalar register (it would otherwise hold a vector register, since
// the scalar unit has no floating point to form it in).
__device__ __forceinline__ float uniform_f(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// 1/sqrt(x) and 1/x for x > 0 in FP64: the hardware estimate y (v_rsq_f64, v_rcp_f64, relative
// error d of about 2^-23) refined by one step of third order.  With e = 1 - x y^2 = O(d),
// 1/sqrt(x) = y (1 - e)^(-1/2) = y (1 + e/2 + 3 e^2/8 + O(d^3)); with e = 1 - x y,
// 1/x = y / (1 - e) = y (1 + e + e^2 + O(d^3)): d^3 lies below FP64's last bit, so the result
// is within a few ulp (not correctly rounded: the rates are compared with a 1e-12 tolerance),
// in 5 and 3 operations where two Newton steps take 8 and 4.  They replace the compiler's
// correctly rounded FP64 square root and divisions, which take several times the instructions.
__device__ __forceinline__ double rsqrt64(double x) {
#pragma clang fp contract(fast)
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

__device__ __forceinline__ double rcp64(double x) {
#pragma clang fp contract(fast)
    const double y = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// Per-particle view of the stencil: cell, position within the cell in cell units (the
// difference formed in FP64, so it stays exact to ~1e-7 on a mesh of any length), reach.
struct Stencil {
    int cx, cy, cz;
    float fx, fy, fz;  // (x - origin) / D - cx; outside [0, 1) off the mesh
    float w2;          // (support/D)^2 with margin
    int R;
};

// Offset from cell c of coordinate v (in cell units), bounded for positions far off the mesh.
__device__ __forceinline__ float cell_offset(double v, double o, double inv, int c) {
    return (float)fmin(fmax((v - o) * inv - (double)c, -1048576.0), 1048576.0);
}

__device__ __forceinline__ Stencil make_stencil(const GridDev &g, double x, double y, double z,
                                                double H) {
    Stencil t;
    t.cx = cell_coord(x, g.ox, g.inv, g.dx);
    t.cy = cell_coord(y, g.oy, g.inv, g.dy);
    t.cz = cell_coord(z, g.oz, g.inv, g.dz);
    t.fx = cell_offset(x, g.ox, g.inv, t.cx);
    t.fy = cell_offset(y, g.oy, g.inv, t.cy);
    t.fz = cell_offset(z, g.oz, g.inv, t.cz);
    float hc = (float)(H * g.inv) * 1.0001f + 1e-3f;
    t.w2 = uniform_f(hc * hc);
    t.R = g.reach;
    return t;
}

// Stencil of the mirror image (x, y', z) of a particle across a wall plane
// normal to y (the kernels' y axis; see csph_internal.h): the image may lie
// off the mesh, so its y cell is not clamped (rows off the mesh are skipped);
// x, z, the chord centre and the reach are the particle's own.  Walking it
// visits every particle whose mirror image lies within the support of the
// particle, wherever the particles are relative to the wall.
__device__ __forceinline__ Stencil image_stencil(const GridDev &g, const Stencil &t,
                                                 double y_image) {
    Stencil s = t;
    const double f = floor((y_image - g.oy) * g.inv);
    s.cy = (int)fmin(fmax(f, -1048576.0), 1048576.0);
    s.fy = cell_offset(y_image, g.oy, g.inv, s.cy);
    return s;
}

// Periodic images (PairConst).  Faces of particle i: bit a set when axis a is periodic and i
// lies within the near-face band of one of its faces, bit 3 + a when that is the high face
// (shift k_a = -1) rather than the low one (k_a = +1).  An image is a non-empty mask m of
// such axes: the partners j at (x_j - k L) along the axes of m.
__device__ __forceinline__ int image_faces(const PairConst &pc, double x, double y, double z) {
    const double p[3] = {x, y, z};
    int f = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        if (!((pc.per >> a) & 1)) continue;
        if (p[a] - pc.lo[a] < pc.hb)
            f |= 1 << a;
        else if (pc.hi[a] - p[a] < pc.hb)
            f |= 9 << a;
    }
    return f;
}

// k_a L_a of image m along axis a (0 when m does not shift axis a): the displacement to the
// image of j is d_a = (x_j,a - x_i,a) - k_a L_a, formed in that order.
__device__ __forceinline__ double image_shift(const PairConst &pc, int f, int m, int a) {
    return ((m >> a) & 1) ? (((f >> (3 + a)) & 1) ? -pc.L[a] : pc.L[a]) : 0.0;
}

// Cell index of coordinate v, not clamped to the mesh (an image point lies off it; rows off
// the mesh are skipped), bounded to keep the integer arithmetic finite.
__device__ __forceinline__ int free_cell(double v, double o, double inv) {
    return (int)fmin(fmax(floor((v - o) * inv), -1048576.0), 1048576.0);
}

// Stencil around the image point p = (x_i, y_i, z_i) + k L of image m, starting from stencil s
// (of i, or of its mirror image, whose y it keeps): the shifted axes take the point's own
// unclamped cells and chord centres.
__device__ __forceinline__ Stencil shifted_stencil(const GridDev &g, Stencil s, int m, double px,
                                                   double py, double pz) {
    if (m & 1) {
        s.cx = free_cell(px, g.ox, g.inv);
        s.fx = cell_offset(px, g.ox, g.inv, s.cx);
    }
    if (m & 2) {
        s.cy = free_cell(py, g.oy, g.inv);
        s.fy = cell_offset(py, g.oy, g.inv, s.cy);
    }
    if (m & 4) {
        s.cz = free_cell(pz, g.oz, g.inv);
        s.fz = cell_offset(pz, g.oz, g.inv, s.cz);
    }
    return s;
}

// Whether a particle at y can have mirror partners within support H: some
// particle's image 2 yw - y_j lies within H of it.  The images lie at or below
// yw + (yw - min_j y_j), so particles behind the wall widen the band in front of it.
__device__ __forceinline__ bool mirror_band(const GridDev &g, double y, double yw, double H) {
    const double ymin = g.yenc ? order_dec(*g.yenc) : g.ymin;
    return y - yw < H + fmax(yw - ymin, 0.0);
}

// Gap in cell units between a point at offset f from its cell and the cell o places on
// (0 inside), shrunk by a margin of 1e-3: |o + 1/2 - f| is the distance to that cell's middle.
__device__ __forceinline__ float cell_gap(float o, float f) {
    return fmaxf(fabsf(o - (f - 0.5f)) - 0.501f, 0.0f);
}

// Orders a wave's LDS accesses for the compiler (the hardware carries them out in order).
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Squared support left for a row of plane zz after the z gap (cell units); -1 when no row of
// the plane counts (off the mesh, or a lane that does not walk).
__device__ __forceinline__ float plane_rem(const GridDev &g, const Stencil &t, bool on, int oz,
                                           int zz) {
    const float gz = cell_gap((float)oz, t.fz);
    return on && (unsigned)zz < (unsigned)g.dz ? t.w2 - gz * gz : -1.0f;
}

// floor(v) as an integer.  ONE (here and in row_range): as one instruction, and so the chord's
// half-width, for the FP32 kernel; the FP64 kernels, short of registers, spilled more with them
// (51 k particles' step VJP 157 -> 162 us).
template <bool ONE>
__device__ __forceinline__ int floor_i(float v) {
    if (!ONE) return (int)floorf(v);
    int r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}

// Candidate range [j0, j0+len) of row (yy, zz), `key` its first cell's: the cells of the row
// within the chord the support sphere cuts through it.  Branch-free per lane; a row off the
// mesh or missing the sphere gets len = 0, and when it does so for every lane of the wave the
// chord and the cell-range loads are skipped (and false returned).
template <bool ONE = false>
__device__ __forceinline__ bool row_range(const int32_t *__restrict__ cs, const GridDev &g,
                                          const Stencil &t, float rem_z, int oy, int yy,
                                          uint32_t key, int &j0, int &len) {
    const float gy = cell_gap((float)oy, t.fy);
    const float rem = rem_z - gy * gy;
    bool ok = rem > 0.0f && (unsigned)yy < (unsigned)g.dy;
    j0 = 0;
    len = 0;
    if (!__any(ok)) return false;
    // chord half-width; v_sqrt_f32 (1 ulp) is ample under the margins (a lane that is not ok may
    // take the root of a negative number: it is given an empty range below)
    const float root = __builtin_amdgcn_sqrtf(rem);
    const float hw = ONE ? fmaf(root, 1.0001f, 1e-3f) : root * 1.0001f + 1e-3f;
    const int xa = max(t.cx + floor_i<ONE>(t.fx - hw), 0);
    const int xb = min(t.cx + floor_i<ONE>(t.fx + hw), g.dx - 1);
    ok = ok && xb >= xa;
    // 64-bit addresses: a mesh may have 2e9 cells
    const uint32_t ia = ok ? key + (uint32_t)xa : 0u, ib = ok ? key + (uint32_t)xb + 1u : 0u;
    j0 = cs[ia];
    len = cs[ib] - j0;
    return __any(len > 0);
}

// Candidates whose FP32 squared distance lies within this relative band of the squared
// support are decided in FP64 from the FP64 positions (the FP32 error of r^2 is below 1e-6
// relative for offsets within a few cells), so every kernel accepts exactly the FP64
// neighbour set.
constexpr float kBand = 4e-5f;
// Pair-h mode: the FP32 test takes (kd d_i + kd d_j)^2 for H_ij^2 (1 + kBand), with room for
// the rounding of the sizes.
inline __device__ float pair_kd(double kappa) {
    return uniform_f((float)(0.5 * kappa) * (1.0f + 0.5f * kBand + 1e-6f));
}
// Zero records after the n FP32 stencil records (cell-relative offsets, read by the candidate
// tests): a walk reads up to kRecPad records past a row's last one.
constexpr int kRecPad = 2;

// Walks the rows (fixed y, z) of a lane's stencil in the order z, then y, calling
// row(oy, yy, oz, j0, len), some lane's len > 0, for every row that some lane of the wave has candidates in.  The
// offsets are wave-uniform; a row's key is carried from row to row (one addition) and formed
// anew where some lane enters another slab, since its three 32-bit products issue at a
// quarter of the rate; the z gap is squared once per plane, and a plane off every lane's mesh
// or sphere is left out.
template <bool ONE = false, typename F>
__device__ __forceinline__ void walk_rows(const int32_t *__restrict__ cs, const GridDev &g,
                                          const Stencil &t, bool on, F &&row) {
    for (int oz = -t.R; oz <= t.R; ++oz) {
        const int zz = t.cz + oz;
        const float rem_z = plane_rem(g, t, on, oz, zz);
        if (!__any(rem_z > 0.0f)) continue;
        int yy = t.cy - t.R;
        uint32_t key = cell_key(g, 0, yy, zz);
        for (int oy = -t.R;;) {
            int j0, len;
            if (row_range<ONE>(cs, g, t, rem_z, oy, yy, key, j0, len)) row(oy, yy, oz, j0, len);
            if (++oy > t.R) break;
            ++yy;
            key = __any((yy & g.ymask) == 0) ? cell_key(g, 0, yy, zz) : key + (uint32_t)g.dx;
        }
    }
}

// Calls part(j0, len) for a row's candidates, len <= 0 where a lane has none.  The row i itself
// lies in (CENTRE: one row of the walk is it; self16 = 16 i) is taken in two parts, before and
// after i, which spares every candidate of every row the comparison with i (3 of 51 vector
// instructions per three candidates; with the one-instruction floor, 589 824 particles with
// periodic sides 471 -> 466 us a step, 11.7 M 6 756 -> 6 732 us).
template <bool CENTRE, typename F>
__device__ __forceinline__ void around_self(int oy, int oz, uint32_t self16, int j0, int len,
                                            F &&part) {
    const bool centre = CENTRE && (oy | oz) == 0;
    int after = 0;  // candidates after i
    if (centre) {
        const int self = (int)(self16 >> 4);
        after = len > 0 ? j0 + len - self - 1 : 0;
        len = len > 0 ? self - j0 : 0;
        asm volatile("" : "+v"(after), "+v"(len));  // a branch, not selects in every row
    }
    for (bool again = centre;; again = false) {
        part(j0, len);
        if (!again) break;
        len = after;
        j0 = (int)(self16 >> 4) + 1;
    }
}

// ---------------------------------------------------------------- particles shared by lanes
//
// A small set leaves the chip idle with one lane per particle: 4 096 particles are 64 waves on
// 1 024 SIMDs, and the FP64 rates of such a set took the ~180 us one wave needs for its walk.
// The FP64 kernels then give each particle 2^ls neighbouring lanes, which deal its stencil rows
// out among themselves (or, where the stencil has only 3 x 3 long rows, each row's candidates)
// and add up their sums at the end in a fixed tree.  The results differ from the one-lane sums
// by the order of the additions only; the FP32 kernels keep one lane per particle, whose sums
// are taken in the walk's order.
constexpr int kSplitMax = 4;
constexpr int64_t kSplitLanes = 4096 * 64;  // lanes that fill the chip at four waves per SIMD

inline int split_log2(int64_t n) {
    int ls = 0;
    while (ls < kSplitMax && (n << (ls + 1)) <= kSplitLanes) ++ls;
    return ls;
}

// v summed over the 2^ls lanes of each particle (every lane gets the sum).
__device__ __forceinline__ double split_sum(double v, int ls) {
    for (int o = 1; o < (1 << ls); o <<= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// walk_rows for a lane that takes share `sub` of 2^ls of its particle's candidates.
template <typename F>
__device__ __forceinline__ void walk_rows_split(const int32_t *__restrict__ cs, const GridDev &g,
                                                const Stencil &t, bool on, int sub, int ls,
                                                F &&row) {
    const int W = 2 * t.R + 1;
    const bool deal = t.R > 1;  // rows dealt out, else each row's candidates cut into shares
    const float iw = 1.0f / (float)W;
    for (int q0 = 0; q0 < W * W; q0 += deal ? 1 << ls : 1) {
        const int q = q0 + (deal ? sub : 0);
        // q / W for q < 16 641 + 16, W <= 129: (q + 1/2) / W lies at least 1/258 from an integer
        const int z = (int)(((float)q + 0.5f) * iw);
        const int oz = z - t.R, oy = q - z * W - t.R;
        const int yy = t.cy + oy, zz = t.cz + oz;
        const float rem_z = plane_rem(g, t, on && q < W * W, oz, zz);
        int j0, len;
        if (!row_range(cs, g, t, rem_z, oy, yy, cell_key(g, 0, yy, zz), j0, len)) continue;
        if (!deal) {
            const int share = (len + (1 << ls) - 1) >> ls, a = share * sub;
            j0 = len > a ? j0 + a : 0;
            len = max(min(len - a, share), 0);
        }
        row(oy, yy, oz, j0, len);
    }
}

// ---------------------------------------------------------------- few lanes' images
//
// The walk around a periodic image that few of a wave's lanes have (kFew at most): a row of cells
// along a periodic axis holds a few particles near each end, and the ~45 stencil rows walked in
// lock step for those lanes alone took a quarter of the FP32 kernel's time.  For each of those
// particles the lanes take a row each, lay the rows' candidates end to end and test one each; the
// accepted ones are listed in the order of the rows, the one in which the lock-step walk queues
// them, and popped by the particle's own lane: the sums keep their bits.
constexpr int kFew = 8;       // particles whose images are walked by the whole wave
constexpr int kFewList = 64;  // partners each; the lists take the place of the wave's rings
constexpr int kLay = 128;     // candidates laid out, 8 bytes each

// One such particle (wave-uniform): the stencil around its image (ghost: around its mirror
// image's), its offsets and cell as the lock-step walk has them, the wall's distance, its part of
// the pair-h bound.
struct FewCentre {
    Stencil st;
    float ax, ay, az, cx, wl, kl;
    int cy0;
};

__device__ __forceinline__ int lane_of(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float lane_of(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
// Lane l's stencil.
__device__ __forceinline__ Stencil lane_of(Stencil st, int l) {
    st.cx = lane_of(st.cx, l);
    st.cy = lane_of(st.cy, l);
    st.cz = lane_of(st.cz, l);
    st.fx = lane_of(st.fx, l);
    st.fy = lane_of(st.fy, l);
    st.fz = lane_of(st.fz, l);
    return st;
}

// Calls emit(at, record offset, dx, dy, dz), at = 0, 1, .., for the candidates within the FP32
// bound, at most kFewList; returns their number, or -1 when there are more of them, or of the
// candidates, than fit.  Every lane of the wave calls it.
template <bool PAIR, bool GHOST, bool ONE, typename E>
__device__ __forceinline__ int few_candidates(const int32_t *__restrict__ cs, const GridDev &g,
                                              const float4 *__restrict__ rec,
                                              const float *__restrict__ d32, const FewCentre &c,
                                              float Df, float hi, float kd, int2 *lay, int lane,
                                              E &&emit) {
    const unsigned long long below = (1ull << lane) - 1ull;
    const int W = 2 * c.st.R + 1;
    const float iw = 1.0f / (float)W;
    int total = 0;
    wave_fence();  // the layout is read before it is written again
    for (int q0 = 0; q0 < W * W; q0 += 64) {
        const int q = q0 + lane;
        const int iz = (int)(((float)q + 0.5f) * iw);  // q / W (as walk_rows_split)
        const int oz = iz - c.st.R, oy = q - iz * W - c.st.R;
        const int yy = c.st.cy + oy, zz = c.st.cz + oz;
        int j0, len;
        if (!row_range<ONE>(cs, g, c.st, plane_rem(g, c.st, q < W * W, oz, zz), oy, yy,
                            cell_key(g, 0, yy, zz), j0, len))
            continue;
        len = max(len, 0);
        int end = len;  // candidates of the rows up to the lane's
        for (int o = 1; o < 64; o <<= 1) {
            const int p = __shfl_up(end, o, 64);
            if (lane >= o) end += p;
        }
        const int all = __builtin_amdgcn_readlane(end, 63);
        if (total + all > kLay) return -1;
        for (int k = 0; __any(k < len); ++k)
            if (k < len) lay[total + end - len + k] = make_int2(j0 + k, q);
        total += all;
    }
    wave_fence();
    int cnt = 0;
    for (int c0 = 0; c0 < total; c0 += 64) {
        const bool there = c0 + lane < total;
        const int2 e = lay[there ? c0 + lane : 0];
        const int iz = (int)(((float)e.y + 0.5f) * iw);
        const int oz = iz - c.st.R, oy = e.y - iz * W - c.st.R;
        const uint32_t jb = (uint32_t)e.x * (uint32_t)sizeof(float4);
        const float4 aj = *(const float4 *)((const char *)rec + jb);
        const float az = fmaf(-Df, (float)oz, c.az);
        const float ay = fmaf(-Df, (float)(c.st.cy + oy - c.cy0), c.ay);
        const float dx = fmaf(aj.w - c.cx, Df, aj.x) - c.ax;
        float dy = aj.y - ay;
        const float dz = aj.z - az;
        if (GHOST) dy = fmaf(2.0f, c.wl, -dy);
        const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
        float hj = hi;
        if (PAIR) {
            const float Hj = fmaf(kd, d32[e.x], c.kl);
            hj = Hj * Hj;
        }
        const bool acc = there & (r2 < hj);
        const unsigned long long hit = __ballot(acc);
        const int at = cnt + __popcll(hit & below);
        cnt += __popcll(hit);
        if (cnt > kFewList) return -1;
        if (acc) emit(at, jb, dx, dy, dz);
    }
    return cnt;
}

}  // namespace csph
