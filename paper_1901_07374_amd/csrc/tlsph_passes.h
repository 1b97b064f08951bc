// The two passes of a step (device code): the force pass's forms and the
// deformation pass, unstaged and staged.  Each kernel is compiled in one of the
// sources that include this.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "tlsph_internal.h"
#include "tlsph_math.h"

namespace tlsph {

// 1/sqrt(x): the hardware estimate refined by Newton-Raphson steps
// y <- y + y (1 - x y^2) / 2, two for double and one for float (each step
// doubles the number of correct bits).  Not correctly rounded: a few ulp.
// An estimate of 0 or infinity (x infinite or 0) is returned as it is.
__device__ __forceinline__ double rsqrt_nr(double x) {
    const double y0 = __builtin_amdgcn_rsq(x);
    double y = y0;
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const double e = fma(-x * y, y, 1.0);
        y = fma(0.5 * y, e, y);
    }
    return (y0 == 0.0 || __builtin_isinf(y0)) ? y0 : y;
}
__device__ __forceinline__ float rsqrt_nr(float x) {
    const float y0 = __builtin_amdgcn_rsqf(x);
    const float e = fmaf(-x * y0, y0, 1.0f);
    const float y = fmaf(0.5f * y0, e, y0);
    return (y0 == 0.0f || __builtin_isinf(y0)) ? y0 : y;
}

// Workgroups are dispatched round-robin over the 8 XCDs (each with its own
// L2).  Give XCD x a contiguous run of tiles instead, so the neighbour halos
// of adjacent tiles are shared through one L2.
// kBack: each XCD takes its run from the end.  The deformation pass does, so that
// it starts on what the force pass, which goes forward, has touched last, and
// the next force pass on what it has: the caches still hold that (steps of the
// 1M Taylor bar 1.4 % shorter, of 64 mixed bars 1.3 %, of the 4.1M plate 0.2 %,
// mixed 0.7 %).
template <bool kBack = false>
__device__ __forceinline__ int64_t xcd_tile(int64_t b, int64_t nblk) {
    constexpr int64_t kXcd = 8;
    const int64_t q = nblk / kXcd, r = nblk % kXcd;
    const int64_t x = b % kXcd, k = b / kXcd;
    const int64_t beg = x * q + (x < r ? x : r), len = q + (x < r ? 1 : 0);
    return beg + (kBack ? len - 1 - k : k);
}

// Tile `part` (of G per workgroup) of a staged pass's workgroup, -1 if none.
// Workgroups take groups of G consecutive tiles (XCD-contiguous: the groups
// an XCD runs are one range).  Under run control the grid still spans every
// tile, and the first workgroups take the listed tiles of running specimens,
// G at a time with the same mapping over the list; the others get -1 and
// return at once.
// (list: the pass's run-control list, null when off; count: its length)
template <bool kBack = false>
__device__ __forceinline__ int64_t work_tile(const int32_t* list, const int32_t* count, int G,
                                             int part, int64_t n_tiles) {
    if (list) {
        const int64_t nw = *count;
        const int64_t ng = (nw + G - 1) / G;
        if ((int64_t)blockIdx.x >= ng) return -1;
        const int64_t k = xcd_tile<kBack>(blockIdx.x, ng) * G + part;
        if (k >= nw) return -1;
        const int64_t t = list[k];
        return t < n_tiles ? t : -1;   // (a list of this tile size has none beyond)
    }
    const int64_t t = xcd_tile<kBack>(blockIdx.x, gridDim.x) * G + part;
    return t < n_tiles ? t : -1;
}

// The tiles of one workgroup of the staged force pass, whose workgroups each
// run several: XCD x takes one contiguous run of the tiles (of the running
// specimens' tiles, under run control), and its workgroups walk it side by
// side, so that the tiles in flight on an XCD are neighbours.  -1 past the end.
struct TileWalk {
    const int32_t* list;
    int32_t n_tiles;
    int64_t k, end, step;
    __device__ TileWalk(const int32_t* list_, const int32_t* count, int64_t n_tiles_)
        : list(list_), n_tiles((int32_t)n_tiles_) {
        constexpr int64_t kXcd = 8;
        const int64_t nw = list ? (int64_t)__builtin_amdgcn_readfirstlane(*count) : n_tiles_;
        const int64_t b = blockIdx.x, g = gridDim.x;
        const int64_t x = b % kXcd, nx = g < kXcd ? g : kXcd;   // XCDs with a workgroup
        const int64_t q = nw / nx, r = nw % nx;
        const int64_t beg = x * q + (x < r ? x : r);
        end = beg + q + (x < r ? 1 : 0);
        step = g / kXcd + (x < g % kXcd ? 1 : 0);   // workgroups on this XCD
        k = beg + b / kXcd;
    }
    // The next tile as it is loaded (a per-lane value, the same in every lane),
    // to be settled once the load has arrived.
    __device__ int32_t load() {
        int32_t t = -1;
        if (k < end) t = list ? list[k] : (int32_t)k;
        k += step;
        return t;
    }
    __device__ int32_t settle(int32_t t) const {
        const int32_t u = __builtin_amdgcn_readfirstlane(t);
        return u < n_tiles ? u : -1;   // (a list of this tile size has none beyond)
    }
};

// A specimen that run control has stopped keeps its state.
__device__ __forceinline__ bool frozen(const DevState& s, int sp) {
    return s.done != nullptr && s.done[sp] != kRunning;
}
// The same test in two parts, so that a kernel can load the flag early and
// wait for it only where it decides: the word is loaded whether run control
// is on or not (then from the specimen index array, a valid address: a
// specimen sp < n has a particle sp).
__device__ __forceinline__ int32_t run_word(const DevState& s, int sp) {
    return (s.done != nullptr ? s.done : s.spec)[sp];
}
__device__ __forceinline__ bool frozen_word(const DevState& s, int32_t w) {
    return s.done != nullptr && w != kRunning;
}

template <typename R>
__device__ __forceinline__ GQRec<R>* gq_of(const DevState& s);
template <>
__device__ __forceinline__ GQRec<double>* gq_of<double>(const DevState& s) { return s.GQ; }
template <>
__device__ __forceinline__ GQRec<float>* gq_of<float>(const DevState& s) { return s.GQ32; }
template <typename R>
__device__ __forceinline__ GHRec<R>* gh_of(const DevState& s);
template <>
__device__ __forceinline__ GHRec<double>* gh_of<double>(const DevState& s) { return s.GH; }
template <>
__device__ __forceinline__ GHRec<float>* gh_of<float>(const DevState& s) { return s.GH32; }

// Everything the force pass needs of a neighbour (and of the particle
// itself): reference position and volume, displacement, 1 - D, Q = P L^-T
// and H = F - I.  Also the LDS record of the staged kernel.
template <typename R>
struct LRecB;
template <>
struct alignas(16) LRecB<double> {
    double x, y, z, V0, ux, uy, uz, omd;
    double q[9], h[9];
    double hs;   // support radius (graded spacing only; not in the LDS image)
};
template <>
struct alignas(16) LRecB<float> {
    double x, y, z, ux, uy, uz;   // positions and displacements stay double
    float V0, omd;
    float q[9], h[9];
    double hs;   // support radius (graded spacing only; not in the LDS image)
};

template <typename R>
__device__ __forceinline__ LRecB<R> make_recb(const D4& xv, const GQRec<R>& g, const GHRec<R>& h,
                                               const D4& u) {
    LRecB<R> r;
    r.x = xv.x; r.y = xv.y; r.z = xv.z; r.V0 = R(xv.w);
    r.ux = u.x; r.uy = u.y; r.uz = u.z; r.omd = g.omd;
#pragma unroll
    for (int k = 0; k < 9; ++k) { r.q[k] = g.q[k]; r.h[k] = h.h[k]; }
    return r;
}

// Sums of the force pass over a particle's neighbours: the stress sums a and b
// and the hourglass sum g.
template <typename R>
struct StressAcc {
    R a0 = 0, a1 = 0, a2 = 0, b0 = 0, b1 = 0, b2 = 0;
};
template <typename R>
struct HgAcc {
    R g0 = 0, g1 = 0, g2 = 0;
};
template <typename R>
struct ForceAcc {
    StressAcc<R> st;
    HgAcc<R> hg;
};

// 1/sqrt(x) and 1/x for x > 0 finite (the refinement of rsqrt_nr and rcp_nr
// without their 0/infinity passthrough: callers select the zero cases).
__device__ __forceinline__ double rsqrt_pos(double x) {
    double y = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int it = 0; it < 2; ++it) y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
    return y;
}
__device__ __forceinline__ float rsqrt_pos(float x) {
    const float y = __builtin_amdgcn_rsqf(x);
    return fmaf(0.5f * y, fmaf(-x * y, y, 1.0f), y);
}
__device__ __forceinline__ double rcp_pos(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}
__device__ __forceinline__ float rcp_pos(float x) {
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(r, fmaf(-x, r, 1.0f), r);
}

// One pair of the force pass, with the kernel's constant factors left out
// (w = W / c and s = h dW/dr / c with c = 8 / (pi h^3); the finish applies
// c / h to a and b and c to the hourglass sum):
//   a += V_j (1 - D_j) s X_ij / r,  b += V_j Q_j s X_ij / r,
//   g += (1 - D_j) V_j w (e_ij . x_ij) / (|X_ij|^2 |x_ij|^2) x_ij
// with e_ij . x_ij = ((H_i + H_j) X_ij) . x_ij / 2 - (u_j - u_i) . x_ij
// (the error vector (F_i + F_j) X_ij / 2 - x_ij with F = I + H).  A pair
// whose current separation is zero adds no hourglass force.  With graded
// spacing (kVarH) each pair has its own support h_ij = (h_i + h_j) / 2, so
// the constant factors c / h_ij and c = 8 / (pi h_ij^3) enter per pair and the
// finish applies none.

// Geometry of a pair: X_ij, 1 / r, w, and gv = V_j s / r.
template <typename R>
struct PairGeom {
    R dx, dy, dz, ir, w, gv;
};
template <typename R, bool kVarH>
__device__ __forceinline__ PairGeom<R> pair_geom(double xi, double yi, double zi, double xj,
                                                 double yj, double zj, R Vj, double hsi,
                                                 double hsj, R inv_h, bool live) {
    // a padding slot (live = false) gets 1/r = 1/|x|^2 = 0: every term it
    // adds is an exact zero
    PairGeom<R> p;
    p.dx = R(xj - xi), p.dy = R(yj - yi), p.dz = R(zj - zi);
    const R r2 = fma(p.dx, p.dx, fma(p.dy, p.dy, p.dz * p.dz));
    const R ir = live ? rsqrt_pos(r2) : R(0);
    R kg = R(1), kw = R(1);
    if constexpr (kVarH) {
        inv_h = rcp_nr(R(0.5 * (hsi + hsj)));
        kw = R(8.0 / M_PI) * inv_h * inv_h * inv_h;
        kg = kw * inv_h;
    }
    const R q = r2 * ir * inv_h;
    // cubic spline: with a = 1 - q and b = max(1/2 - q, 0), W / c = 2 a^3 -
    // 8 b^3 and h dW/dr / c = -6 a^2 + 24 b^2 (b = 0 beyond q = 1/2, where
    // seven pairs in eight lie).  FP64 evaluates it without a branch; the
    // mixed form keeps the two-branch form, which fits its register budget
    // of four waves per SIMD without spilling.
    R w, sl;
    if constexpr (sizeof(R) == 8) {
        const R a = R(1) - q;
        const R b = fmax(R(0.5) - q, R(0));
        const R a2 = a * a, b2 = b * b;
        sl = fma(R(24), b2, R(-6) * a2);
        w = fma(R(-8) * b2, b, (a + a) * a2);
    } else if (q < R(0.5)) {
        w = fma(q * q, fma(R(6), q, R(-6)), R(1));
        sl = q * fma(R(18), q, R(-12));
    } else {
        const R a = R(1) - q;
        const R a2 = a * a;
        w = (a + a) * a2;
        sl = R(-6) * a2;
    }
    R gv = sl * ir * Vj;
    if constexpr (kVarH) {
        gv *= kg;
        w *= kw;
    }
    p.ir = ir;
    p.w = w;
    p.gv = gv;
    return p;
}

// Stress part of a pair: g = V_j s X_ij / r, omd and q the neighbour's 1 - D
// and Q.
template <typename R>
__device__ __forceinline__ void stress_pair(R gx, R gy, R gz, R omd, const R (&q)[9],
                                            StressAcc<R>& A) {
    A.a0 = fma(omd, gx, A.a0); A.a1 = fma(omd, gy, A.a1); A.a2 = fma(omd, gz, A.a2);
    A.b0 = fma(q[0], gx, fma(q[1], gy, fma(q[2], gz, A.b0)));
    A.b1 = fma(q[3], gx, fma(q[4], gy, fma(q[5], gz, A.b1)));
    A.b2 = fma(q[6], gx, fma(q[7], gy, fma(q[8], gz, A.b2)));
}

// Hourglass part of a pair: vw = V_j (1 - D_j), du = u_j - u_i.
template <typename R>
__device__ __forceinline__ void hg_pair(const PairGeom<R>& p, R vw, R du0, R du1, R du2,
                                        const R (&hi)[9], const R (&hj)[9], bool live,
                                        HgAcc<R>& A) {
    const R dx = p.dx, dy = p.dy, dz = p.dz;
    const R x0 = dx + du0, x1 = dy + du1, x2 = dz + du2;
    const R rc2 = fma(x0, x0, fma(x1, x1, x2 * x2));
    const R irc2 = (live && rc2 > R(0)) ? rcp_pos(rc2) : R(0);
    const R v0 = fma(hi[0] + hj[0], dx, fma(hi[1] + hj[1], dy, (hi[2] + hj[2]) * dz));
    const R v1 = fma(hi[3] + hj[3], dx, fma(hi[4] + hj[4], dy, (hi[5] + hj[5]) * dz));
    const R v2 = fma(hi[6] + hj[6], dx, fma(hi[7] + hj[7], dy, (hi[8] + hj[8]) * dz));
    const R hx = fma(v0, x0, fma(v1, x1, v2 * x2));
    const R ux = fma(du0, x0, fma(du1, x1, du2 * x2));
    const R ex = fma(R(0.5), hx, -ux);
    const R c = vw * p.w * ex * (p.ir * p.ir) * irc2;
    A.g0 = fma(c, x0, A.g0); A.g1 = fma(c, x1, A.g1); A.g2 = fma(c, x2, A.g2);
}

template <typename R, bool kVarH = false>
__device__ __forceinline__ void force_pair(const LRecB<R>& ni, const LRecB<R>& nj, R inv_h,
                                           ForceAcc<R>& A, bool live = true) {
    const PairGeom<R> p = pair_geom<R, kVarH>(ni.x, ni.y, ni.z, nj.x, nj.y, nj.z, nj.V0, ni.hs,
                                              nj.hs, inv_h, live);
    stress_pair<R>(p.gv * p.dx, p.gv * p.dy, p.gv * p.dz, nj.omd, nj.q, A.st);
    hg_pair<R>(p, nj.V0 * nj.omd, R(nj.ux - ni.ux), R(nj.uy - ni.uy), R(nj.uz - ni.uz), ni.h, nj.h,
               live, A.hg);
}

template <typename R>
__device__ __forceinline__ StressAcc<R> acc_sum(const StressAcc<R>& x, const StressAcc<R>& y) {
    StressAcc<R> r;
    r.a0 = x.a0 + y.a0; r.a1 = x.a1 + y.a1; r.a2 = x.a2 + y.a2;
    r.b0 = x.b0 + y.b0; r.b1 = x.b1 + y.b1; r.b2 = x.b2 + y.b2;
    return r;
}
template <typename R>
__device__ __forceinline__ HgAcc<R> acc_sum(const HgAcc<R>& x, const HgAcc<R>& y) {
    HgAcc<R> r;
    r.g0 = x.g0 + y.g0; r.g1 = x.g1 + y.g1; r.g2 = x.g2 + y.g2;
    return r;
}
template <typename R>
__device__ __forceinline__ ForceAcc<R> acc_sum(const ForceAcc<R>& x, const ForceAcc<R>& y) {
    return ForceAcc<R>{acc_sum(x.st, y.st), acc_sum(x.hg, y.hg)};
}

// The value of lane l ^ m (m = 1 or 2) within each group of four lanes, by a
// DPP quad permutation (a VALU operand modifier: no LDS traffic).
template <int M>
__device__ __forceinline__ float quad_xor(float v) {
    static_assert(M == 1 || M == 2, "quad permutations for xor 1 and 2");
    constexpr int ctrl = M == 1 ? 0xB1 : 0x4E;   // quad_perm [1,0,3,2] / [2,3,0,1]
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, 0xF, 0xF, false));
}
template <int M>
__device__ __forceinline__ double quad_xor(double v) {
    static_assert(M == 1 || M == 2, "quad permutations for xor 1 and 2");
    constexpr int ctrl = M == 1 ? 0xB1 : 0x4E;
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), ctrl, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), ctrl, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

template <int M, typename R>
__device__ __forceinline__ StressAcc<R> acc_xor(const StressAcc<R>& x) {
    StressAcc<R> r;
    r.a0 = quad_xor<M>(x.a0); r.a1 = quad_xor<M>(x.a1); r.a2 = quad_xor<M>(x.a2);
    r.b0 = quad_xor<M>(x.b0); r.b1 = quad_xor<M>(x.b1); r.b2 = quad_xor<M>(x.b2);
    return r;
}
template <int M, typename R>
__device__ __forceinline__ HgAcc<R> acc_xor(const HgAcc<R>& x) {
    HgAcc<R> r;
    r.g0 = quad_xor<M>(x.g0); r.g1 = quad_xor<M>(x.g1); r.g2 = quad_xor<M>(x.g2);
    return r;
}
template <int M, typename R>
__device__ __forceinline__ ForceAcc<R> acc_xor(const ForceAcc<R>& x) {
    return ForceAcc<R>{acc_xor<M>(x.st), acc_xor<M>(x.hg)};
}

// The partial sums of a particle's S lanes combined as (p0 + p1) + (p2 + p3)
// (A: the lane's kSub / S partials; every lane gets the result).
template <int S, typename Acc>
__device__ __forceinline__ Acc combine_partials(const Acc (&A)[kSub / S]) {
    if constexpr (S == 1) {
        return acc_sum(acc_sum(A[0], A[1]), acc_sum(A[2], A[3]));
    } else if constexpr (S == 2) {
        const Acc x = acc_sum(A[0], acc_xor<1>(A[0]));   // p0 + p1
        const Acc y = acc_sum(A[1], acc_xor<1>(A[1]));   // p2 + p3
        return acc_sum(x, y);
    } else {
        const Acc x = acc_sum(A[0], acc_xor<1>(A[0]));   // p0 + p1 | p2 + p3
        return acc_sum(x, acc_xor<2>(x));
    }
}

// A lane's share of a particle's first kPackGroups kSub neighbours as local
// slots, two to a word: list t of a lane (neighbours sub + S t, + kSub, ...) is
// kPackGroups consecutive entries of the particle's record, so a lane loads it
// with one instruction where the sliced list takes one per entry.
template <int S>
struct Slots {
    static constexpr int NP = kSub / S;
    static constexpr int W = kPackGroups / 2;
    uint32_t w[NP][W];
    __device__ int at(int g, int t) const {
        return (int)((g & 1) ? w[t][g >> 1] >> 16 : w[t][g >> 1] & 0xffffu);
    }
};
template <int S>
__device__ __forceinline__ Slots<S> load_slots(const uint32_t* __restrict__ pslot, int64_t i, int sub) {
    static_assert(kPackGroups == 6 && kPackWords == 12, "three words a list");
    struct alignas(4) W3 {
        uint32_t a, b, c;
    };
    Slots<S> f;
#pragma unroll
    for (int t = 0; t < Slots<S>::NP; ++t) {
        const W3 v = *reinterpret_cast<const W3*>(pslot + i * kPackWords + 3 * (sub + S * t));
        f.w[t][0] = v.a; f.w[t][1] = v.b; f.w[t][2] = v.c;
    }
    return f;
}

// Pair sums of one particle in the canonical order of the force pass:
// neighbour k feeds partial sum k mod kSub (each partial in increasing k) and
// the partials combine as (p0 + p1) + (p2 + p3).  S adjacent lanes share a
// particle (S = 1, 2 or 4), lane `sub` holding partials sub, sub + S, ...;
// every S rounds identically.  All lanes of the wave must call this (the
// partials are exchanged across lanes); lanes without a particle pass cnt = 0.
// Indices run one group of kSub ahead of the arithmetic.
template <typename R, int S, bool kVarH = false, typename IdxOf, typename RecOf>
__device__ __forceinline__ ForceAcc<R> pair_sums(const LRecB<R>& ni, int cnt, int sub, R inv_h,
                                                 IdxOf idx, RecOf rec) {
    static_assert(kSub == 4 && (S == 1 || S == 2 || S == 4), "canonical order has 4 partials");
    constexpr int NP = kSub / S;
    ForceAcc<R> A[NP];
    int first[NP], q[NP];
#pragma unroll
    for (int t = 0; t < NP; ++t) {
        const int k = sub + S * t;
        first[t] = idx(k < cnt ? k : 0);
        q[t] = idx(kSub + k < cnt ? kSub + k : 0);
    }
    if (0 < cnt) {
#pragma unroll
        for (int t = 0; t < NP; ++t)
            force_pair<R, kVarH>(ni, rec(first[t]), inv_h, A[t], sub + S * t < cnt);
    }
    for (int k0 = kSub; k0 < cnt; k0 += kSub) {
        int cur[NP];
#pragma unroll
        for (int t = 0; t < NP; ++t) {
            cur[t] = q[t];
            const int kn = k0 + kSub + sub + S * t;
            q[t] = idx(kn < cnt ? kn : 0);
        }
#pragma unroll
        for (int t = 0; t < NP; ++t) {
            const int k = k0 + sub + S * t;
            force_pair<R, kVarH>(ni, rec(cur[t]), inv_h, A[t], k < cnt);
        }
    }
    return combine_partials<S>(A);
}

// Penalty contact force on particle i at its position (xi, yi, zi) at t^n:
// the Hertz law of two spheres of radii a_i, a_j over every listed candidate
// closer than a_i + a_j, except reference neighbours of the same specimen
// that are both intact; F = k (4/3) E* sqrt(a_i a_j / (a_i + a_j)) delta^(3/2)
// along x_ij, k the mean of the two factors, 1/E* the sum of the shares.
// Also flags a particle that has left the list's skin.
__device__ __forceinline__ void contact_force(const DevState& s, int64_t i, int par, int sp,
                                              double xi, double yi, double zi, double Di,
                                              double f[3]) {
    const int64_t np = s.np;
    f[0] = f[1] = f[2] = 0.0;
    const DevSpec& Pi = s.specs[sp];
    const double ai = s.arad[i];
    const D4* __restrict__ Uc = s.U[par];
    const D4 ui = Uc[i];
    const double b0 = ui.x - s.ubuild[i], b1 = ui.y - s.ubuild[np + i],
                 b2 = ui.z - s.ubuild[2 * np + i];
    if (4.0 * (b0 * b0 + b1 * b1 + b2 * b2) > s.contact_skin * s.contact_skin)
        atomicOr(&s.err[2], kErrContact);
    const int cnt = s.ccnt[i];
    for (int k = 0; k < cnt; ++k) {
        const uint32_t e = (uint32_t)s.ccol[(int64_t)k * np + i];
        const int32_t q = (int32_t)(e & 0x7fffffffu);
        const bool ref = (e >> 31) != 0;
        if (ref && Di < 1.0 && s.D[q] < 1.0) continue;
        const DevSpec& Pq = s.specs[s.spec[q]];
        const double kc = 0.5 * (Pi.contact_k + Pq.contact_k);
        if (!(kc > 0.0)) continue;
        const D4 xq = s.XV[q], uq = Uc[q];
        const double d0 = (xq.x + uq.x) - xi, d1 = (xq.y + uq.y) - yi, d2 = (xq.z + uq.z) - zi;
        const double r2 = d0 * d0 + d1 * d1 + d2 * d2;
        const double aq = s.arad[q], rc = ai + aq;
        if (!(r2 < rc * rc) || !(r2 > 0.0)) continue;
        const double r = sqrt(r2), delta = rc - r;
        const double es = 1.0 / (Pi.contact_comp + Pq.contact_comp);
        const double F = kc * (4.0 / 3.0) * es * sqrt(ai * aq / rc) * delta * sqrt(delta);
        const double g = F / r;
        f[0] -= g * d0;
        f[1] -= g * d1;
        f[2] -= g * d2;
    }
}

// What the finish needs of a particle besides its record, loaded before the
// pair sums so that their latency is spent behind them.
struct FinishIn {
    double D, V, vx, vy, vz;
    int32_t bc;
};
// The velocity ramp 1 - exp(-t / tau) of the boundary group and specimen a wave
// met last (the same for every particle of a launch: the pipelined pass's waves
// finish many tiles, mostly of one group).  Scalars: set where the whole wave
// goes (meet_group), never in a turn of some of its lanes.
struct Ramp {
    int32_t group = -1, sp = -1;
    double value = 0.0;
};
__device__ __forceinline__ FinishIn finish_in(const DevState& s, int64_t i, double V) {
    const D4 v = s.VW[i];
    return FinishIn{s.D[i], V, v.x, v.y, v.z, s.bc[i]};
}

// A value that is the same in every active lane, as a scalar.
__device__ __forceinline__ double uniform(double x) {
    const long long b = __double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffll));
    const unsigned hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | lo);
}

// The specimen's constants that the finish needs (graded spacing: the pair
// sums carry the kernel's constant factors).
struct FinishSpec {
    double ck, hgk, dt, dt_rho0;
    int32_t wall;
};
template <bool kVarH>
__device__ __forceinline__ FinishSpec finish_spec(const DevSpec& P) {
    return FinishSpec{kVarH ? 1.0 : P.grad_k, kVarH ? -P.hg_alpha * P.E : P.hg_k, P.dt, P.dt_rho0,
                      P.has_wall};
}
__device__ __forceinline__ double ramp_value(const DevState& s, const DevBC& B, int sp, double dt) {
    const double th = s.t[sp] + 0.5 * dt;
    return B.tau > 0.0 ? 1.0 - exp(-th / B.tau) : 1.0;
}
__device__ __forceinline__ void prescribe(const DevBC& B, double ramp, double xi, double yi,
                                          double zi, double v[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c)
        if (B.mask & (1 << c))
            v[c] = B.v_max[c] * ramp +
                   (B.grad[3 * c] * xi + B.grad[3 * c + 1] * yi + B.grad[3 * c + 2] * zi);
}

// Nodal force, kick, prescribed velocities (the caller's: by lane, or by wave),
// failed particles at rest, drift, rigid wall; stores v, V0 (1 - D), u^{n+1} and
// (for groups) the force.  The force per unit volume f / V_i is formed first:
// the kick is dt / rho0 times it (m = rho0 V_i).
// kTwo: two adjacent lanes (sub 0, 1) hold the particle's sums and both come
// here; each stores half of every record, so that a wave's stores are contiguous.
template <typename R, bool kTwo, typename Prescribe>
__device__ __forceinline__ void finish_particle(const DevState& s, int64_t i, int par, int sp,
                                                const DevSpec& P, const FinishSpec& c,
                                                const LRecB<R>& ni, const ForceAcc<R>& A,
                                                const FinishIn& fin, int sub, Prescribe prescribed) {
    const int64_t np = s.np;
    const double Di = fin.D;
    const R omDi = R(1.0 - Di);
    const R ck = R(c.ck);
    const R hgk = R(c.hgk) * omDi;
    const double Vi = fin.V;
    const StressAcc<R>& a = A.st;
    const HgAcc<R>& g = A.hg;
    double fv0 = double(ck * (ni.q[0] * a.a0 + ni.q[1] * a.a1 + ni.q[2] * a.a2 + omDi * a.b0) + hgk * g.g0);
    double fv1 = double(ck * (ni.q[3] * a.a0 + ni.q[4] * a.a1 + ni.q[5] * a.a2 + omDi * a.b1) + hgk * g.g1);
    double fv2 = double(ck * (ni.q[6] * a.a0 + ni.q[7] * a.a1 + ni.q[8] * a.a2 + omDi * a.b2) + hgk * g.g2);
    if (s.av) {   // the artificial viscous force of the last deformation pass
        const double iv = rcp_nr(Vi);
        fv0 += s.fvisc[i] * iv;
        fv1 += s.fvisc[np + i] * iv;
        fv2 += s.fvisc[2 * np + i] * iv;
    }
    if (s.contact) {   // penalty contact with the listed candidates
        double fc[3];
        contact_force(s, i, par, sp, ni.x + ni.ux, ni.y + ni.uy, ni.z + ni.uz, Di, fc);
        const double iv = rcp_nr(Vi);
        fv0 += fc[0] * iv;
        fv1 += fc[1] * iv;
        fv2 += fc[2] * iv;
    }
    const double dt = c.dt;
    double v[3] = {fin.vx + c.dt_rho0 * fv0, fin.vy + c.dt_rho0 * fv1, fin.vz + c.dt_rho0 * fv2};
    const double xi = ni.x, yi = ni.y, zi = ni.z;
    if (fin.bc >= 0) prescribed(dt, xi, yi, zi, v);
    if (Di >= 1.0) v[0] = v[1] = v[2] = 0.0;
    double un[3] = {ni.ux + dt * v[0], ni.uy + dt * v[1], ni.uz + dt * v[2]};
    if (c.wall) {
        const double xw[3] = {xi + un[0], yi + un[1], zi + un[2]};
        const double dn = xw[0] * P.wall_n[0] + xw[1] * P.wall_n[1] + xw[2] * P.wall_n[2] - P.wall_d;
        if (dn < 0.0) {
            un[0] = (xw[0] - dn * P.wall_n[0]) - xi;
            un[1] = (xw[1] - dn * P.wall_n[1]) - yi;
            un[2] = (xw[2] - dn * P.wall_n[2]) - zi;
            const double vn = v[0] * P.wall_n[0] + v[1] * P.wall_n[1] + v[2] * P.wall_n[2];
            if (vn < 0.0) {
                v[0] -= vn * P.wall_n[0];
                v[1] -= vn * P.wall_n[1];
                v[2] -= vn * P.wall_n[2];
            }
        }
    }
    const double w = Vi * (1.0 - Di);
    const bool keep = (s.flags & kFlagStoreForce) || fin.bc >= 0;
    if constexpr (kTwo) {
        reinterpret_cast<double2*>(s.VW)[2 * i + sub] = sub ? double2{v[2], w} : double2{v[0], v[1]};
        reinterpret_cast<double2*>(s.U[par ^ 1])[2 * i + sub] =
            sub ? double2{un[2], 0.0} : double2{un[0], un[1]};
        if (keep) {
            s.force[sub * np + i] = Vi * (sub ? fv1 : fv0);
            if (!sub) s.force[2 * np + i] = Vi * fv2;
        }
    } else {
        s.VW[i] = D4{v[0], v[1], v[2], w};
        s.U[par ^ 1][i] = D4{un[0], un[1], un[2], 0.0};
        if (keep) {
            s.force[i] = Vi * fv0; s.force[np + i] = Vi * fv1; s.force[2 * np + i] = Vi * fv2;
        }
    }
}

// The ramp of the first lane of the wave that has a boundary group (-1: none),
// ahead of the lanes' turns in force_finish.  Every lane of the wave comes here.
__device__ __forceinline__ void meet_group(const DevState& s, int sp_lane, int bc_lane, Ramp& ramp) {
    const uint64_t with = __ballot(bc_lane >= 0);
    if (with == 0) return;
    const int l = __ffsll((unsigned long long)with) - 1;
    const int g = __builtin_amdgcn_readlane(bc_lane, l), sp = __builtin_amdgcn_readlane(sp_lane, l);
    if (g == ramp.group && sp == ramp.sp) return;
    ramp.group = g;
    ramp.sp = sp;
    ramp.value = uniform(ramp_value(s, s.bcs[g], sp, s.specs[sp].dt));
}

// The finish of the staged forms.  The lanes of a wave take turns by specimen,
// and within it by boundary group (one turn each unless the wave straddles two),
// so that both records arrive by scalar loads, which the CU's scalar cache
// keeps: per lane they would be two more dependent trips to memory at the end
// of a tile.  A turn leaves nothing behind but its stores: a scalar set in it
// and read after the turns could be another turn's.
template <typename R, bool kVarH = false, bool kTwo = false>
__device__ __forceinline__ void force_finish(const DevState& s, int64_t i, int par, int sp_lane,
                                             const LRecB<R>& ni, const ForceAcc<R>& A,
                                             const FinishIn& fin, const Ramp* ramp = nullptr,
                                             int sub = 0) {
    for (;;) {
        const int sp = __builtin_amdgcn_readfirstlane(sp_lane);
        if (sp != sp_lane) continue;
        if (frozen(s, sp)) return;
        const DevSpec& P = s.specs[sp];
        finish_particle<R, kTwo>(
            s, i, par, sp, P, finish_spec<kVarH>(P), ni, A, fin, sub,
            [&](double dt, double xi, double yi, double zi, double (&v)[3]) {
                for (;;) {
                    const int gw = __builtin_amdgcn_readfirstlane(fin.bc);
                    if (gw != fin.bc) continue;
                    const DevBC& B = s.bcs[gw];
                    const bool known = ramp && gw == ramp->group && sp == ramp->sp;
                    prescribe(B, known ? ramp->value : ramp_value(s, B, sp, dt), xi, yi, zi, v);
                    return;
                }
            });
        return;
    }
}

// Pass B (forces at t^n, kick, drift).  Nodal force of Sec. 3.1,
//   f_i = V_i sum_j V_j [(1 - D_j) Q_i + (1 - D_i) Q_j] gradW_ij,
// evaluated as V_i [Q_i a + (1 - D_i) b] with a = sum_j V_j (1 - D_j) gradW_ij
// and b = sum_j V_j Q_j gradW_ij, plus hourglass control: with the error
// vector e_ij = (F_i + F_j)/2 X_ij - x_ij and delta = e_ij . x_ij / |x_ij|,
//   f_i^HG = -alpha E (1 - D_i) V_i sum_j (1 - D_j) V_j W_ij delta / |X_ij|^2
//            x_ij / |x_ij|.
// Then v += dt f / m, prescribed velocities at t^{n+1/2}, D = 1 at rest,
// u^{n+1} = u^n + dt v (into the other displacement buffer), rigid wall, and
// the record (v, V0 (1 - D)) the deformation pass gathers.  This variant
// gathers neighbours straight from global memory.  It is chosen for problems of
// a few waves, which a chain of latencies bounds: what the finish needs of the
// specimen is loaded per lane ahead of the pair sums, and of its group where it
// has one (by wave, as the staged forms do, both ahead of the sums: 6k particles,
// four lanes, a step of 17.5 us FP64, 16.5 mixed; so 17.1 and 16.1).
template <typename R, int S, bool kVarH = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(S < 2 ? S : 2, 8)))
k_pass_b(DevState s, int par) {
    const int64_t t = xcd_tile(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    const int64_t i = t / S;
    const int sub = (int)(t % S);
    const bool in = i < s.n;
    const int64_t ii = in ? i : 0;
    const int sp = s.spec[ii];
    const DevSpec& P = s.specs[sp];
    const D4* __restrict__ XV = s.XV;
    const D4* __restrict__ Uc = s.U[par];
    const GQRec<R>* __restrict__ GQ = gq_of<R>(s);
    const GHRec<R>* __restrict__ GH = gh_of<R>(s);
    LRecB<R> ni = make_recb<R>(XV[ii], GQ[ii], GH[ii], Uc[ii]);
    if constexpr (kVarH) ni.hs = s.hs[ii];
    const R inv_h = R(P.inv_h);
    const bool live = in && !frozen(s, sp);
    const int cnt = live ? s.nnb[i] : 0;
    const FinishSpec fsp = finish_spec<kVarH>(P);
    const FinishIn fin = finish_in(s, ii, XV[ii].w);
    const int32_t* __restrict__ cp = s.col + s.slice_ptr[ii / kSlice] + (ii % kSlice);
    const auto idx = [&](int k) { return (int)cp[(int64_t)k * kSlice]; };
    const ForceAcc<R> A = pair_sums<R, S, kVarH>(
        ni, cnt, sub, inv_h, idx,
        [&](int j) {
            LRecB<R> r = make_recb<R>(XV[j], GQ[j], GH[j], Uc[j]);
            if constexpr (kVarH) r.hs = s.hs[j];
            return r;
        });
    // the particle's own Q is needed only now: reread it (the compiler barrier
    // keeps the load here) rather than keep it in registers through the loop
    asm volatile("" ::: "memory");
    if (live && sub == 0)
        finish_particle<R, false>(s, i, par, sp, P, fsp, make_recb<R>(XV[i], GQ[i], GH[i], Uc[i]), A,
                                  fin, 0,
                                  [&](double dt, double xi, double yi, double zi, double (&v)[3]) {
                                      const DevBC& B = s.bcs[fin.bc];
                                      prescribe(B, ramp_value(s, B, sp, dt), xi, yi, zi, v);
                                  });
}

// 16 bytes per lane from global memory straight into LDS: lane l of the wave
// lands at dst + 16 l (dst: an LDS address, the same for the wave's lanes); a lane
// that is switched off writes nothing.  Written as assembly because the
// compiler waits for every such load before the next LDS read, whichever part
// of LDS either touches.  The loads count as vector loads (lds_dma_wait), have
// no destination register, and take their address when they issue.
__device__ __forceinline__ void lds_dma16(const void* src, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :: "v"(src), "s"(__builtin_amdgcn_readfirstlane(dst)) : "memory", "m0");
}
// The 16 bytes after src (the instruction's offset moves both addresses).
__device__ __forceinline__ void lds_dma16_next(const void* src, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off offset:16"
                 :: "v"(src), "s"(__builtin_amdgcn_readfirstlane(dst - 16)) : "memory", "m0");
}
// Every vector memory access of the wave but the last N done (a builtin, so that
// the compiler knows its own loads have arrived too).
template <int N = 0>
__device__ __forceinline__ void lds_dma_wait() {
    static_assert(N < 16, "the counter's low bits");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0f70 | N);   // vmcnt(N), the other counters as they are
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// LDS image of one tile and its halo (M slots) in the staged force pass: four
// planes of 16 bytes a slot (X, Y | Z, V0 | u_x, u_y | u_z, -), then one
// region of records (GHRec, later GQRec, as they lie in memory: 5 units of 16
// bytes, 3 in the mixed form, an odd number, so that the slots the lanes of a
// 128-bit read address spread over the banks), with graded spacing the support
// radii, and the particle of each slot.
template <typename R>
struct alignas(16) LdsGQ : GQRec<R> {};
template <typename R>
struct alignas(16) LdsGH : GHRec<R> {};
template <typename R>
struct LdsB {
    static constexpr int kRec = (int)(sizeof(LdsGQ<R>) / 16);   // units of a record
    static constexpr int kBytes = 4 * 16 + kRec * 16 + 4;       // per slot
    static_assert(sizeof(LdsGQ<R>) == sizeof(LdsGH<R>) && kRec % 2 == 1,
                  "records of an odd number of 16-byte units");
    double2* xy;
    double2* zv;
    double2* uxy;
    double2* uz;
    unsigned char* rec;
    double* hs;
    int32_t* map;
    __device__ LdsB(unsigned char* raw, int M, bool var_h) {
        xy = reinterpret_cast<double2*>(raw);
        zv = xy + M;
        uxy = zv + M;
        uz = uxy + M;
        rec = reinterpret_cast<unsigned char*>(uz + M);
        hs = reinterpret_cast<double*>(rec + (size_t)M * kRec * 16);
        map = reinterpret_cast<int32_t*>(hs + (var_h ? M : 0));
    }
    __device__ LdsGH<R> gh(int m) const { return reinterpret_cast<const LdsGH<R>*>(rec)[m]; }
    __device__ LdsGQ<R> gq(int m) const { return reinterpret_cast<const LdsGQ<R>*>(rec)[m]; }
};

// Records of slots 0 .. tot - 1 (src: GQ or GH) to dst in LDS, by consecutive
// 16-byte units: a wave's load covers whole records, so it touches a fifth of the
// cache lines that a load of one unit per record does.  Full waves only.
template <int K, int kStride>
__device__ __forceinline__ void stage_records(const void* __restrict__ src, uint32_t dst,
                                              const int32_t* map, int tot, int wave, int n_waves,
                                              int lane) {
    constexpr int kU = 4;   // loads whose slots are looked up together
    const int units = tot * K;
    const int chunks = (units + 63) >> 6;
    const unsigned char* __restrict__ base = static_cast<const unsigned char*>(src);
    for (int c = wave; c < chunks; c += kU * n_waves) {
        int32_t g[kU];
        uint32_t f[kU];
#pragma unroll
        for (int q = 0; q < kU; ++q) {
            int e = (c + q * n_waves) * 64 + lane;
            e = e < units ? e : units - 1;
            const uint32_t m = (uint32_t)e / K;
            g[q] = map[m];
            f[q] = ((uint32_t)e - m * K) * 16;
        }
#pragma unroll
        for (int q = 0; q < kU; ++q) asm volatile("" : "+v"(g[q]), "+v"(f[q]));
#pragma unroll
        for (int q = 0; q < kU; ++q) {
            const int cq = c + q * n_waves;
            const unsigned char* p = base + ((uint64_t)(uint32_t)g[q] * kStride + f[q]);
            if (cq * 64 + 64 <= units)
                lds_dma16(p, dst + (uint32_t)cq * 1024);
            else if (cq * 64 + lane < units)
                lds_dma16(p, dst + (uint32_t)cq * 1024);
        }
    }
}

// Particle of slot m of a tile's LDS image: the tile's T particles from
// `start`, then its halo row hl (capacity cap); n for slots past the particle
// count.  The row entry is loaded unconditionally, at an index inside the row,
// and blended in with masks, so that the load needs neither the halo count nor
// a branch.
__device__ __forceinline__ int64_t slot_particle(int m, int T, int cap, int64_t start, int64_t n,
                                                 const int32_t* __restrict__ hl) {
    const int h = m - T;
    const int64_t hv = hl[h >= 0 && h < cap ? h : 0];
    const int64_t in_tile = -(int64_t)(h < 0), past = -(int64_t)(h >= cap);
    const int64_t g = ((start + m) & in_tile) | (hv & ~in_tile);
    return (n & past) | (g & ~past);
}

// Largest workgroup of the staged force pass with S lanes per particle: four
// lanes run tiles of at most 128 particles, so that the register budget
// stays at two waves per SIMD.
__host__ __device__ constexpr int staged_block_max(int S) { return S == 4 ? 512 : kTile * S; }

// Waves per SIMD the two-sweep form must leave room for.
template <int S>
__host__ __device__ constexpr int staged_waves_min() {
    return S >= 2 ? 3 : 1;
}

// The same pass with the tile's particles and its halo staged in LDS, in two
// sweeps over a particle's neighbours that share one LDS image: first the
// hourglass sums from (X, V0, u, H), then the stress sums from (X, Q, 1 - D),
// whose records replace H's.  S lanes per particle read the image through the
// 16-bit local neighbour slots; same arithmetic in the same order as the
// unstaged kernel, so results are bitwise identical.  Two sweeps need 148
// bytes of LDS per slot where one sweep's image takes 208, and fewer registers:
// three tiles share a CU instead of two (395k particles with contact, tiles of
// 97: 118 -> 100 us).  FP64 only: the mixed records save 12 bytes of 128.  The
// first sweep keeps each pair's V_j s / r in a register for the second.  Graded
// spacing (kVarH): the slots' support radii are in LDS too (one double per slot).
template <int S, bool kVarH>
__device__ __forceinline__ void pass_b_sweeps(const DevState& s, int par) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    using R = double;
    constexpr int K = LdsB<R>::kRec, NP = kSub / S, G = kPackGroups;
    const int M = s.lds_slots;
    const LdsB<R> L(lds_raw, M, kVarH);
    const int T = s.tile;
    const int tile = __builtin_amdgcn_readfirstlane(
        (int)work_tile(s.tile_list, s.run_count, 1, 0, gridDim.x));
    if (tile < 0) return;
    const int64_t start = (int64_t)tile * T;
    const int32_t* __restrict__ hl = s.halo + (int64_t)tile * s.halo_cap;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nw = (int)blockDim.x >> 6;   // full waves: they stage (a tile has at least one)
    // A full wave takes 64 consecutive slots at a time; the first two rounds'
    // row entries are loaded before the count is known.
    const auto particle_of = [&](int m) { return slot_particle(m, T, s.halo_cap, start, s.n, hl); };
    const int step = nw * 64;
    int m = wave * 64 + lane;
    int64_t g0 = particle_of(m), g1 = particle_of(m + step);
    const int tot = T + s.halo_cnt[tile];
    const int pl = threadIdx.x / S;
    const int sub = threadIdx.x % S;
    const int64_t i = start + pl;
    const bool in = i < s.n;
    const int64_t ii = in ? i : start;
    const int cnt = in ? s.nnb[ii] : 0;
    const int sp = s.spec[ii];
    const Slots<S> slots = load_slots<S>(s.pslot, ii, sub);
    if (wave < nw) {
        const uint32_t l_xy = lds_addr(L.xy), l_zv = lds_addr(L.zv), l_uxy = lds_addr(L.uxy),
                       l_uz = lds_addr(L.uz);
        for (int b = wave * 64; b < tot; b += step, m += step) {
            const int64_t g = g0 < s.n ? g0 : start;
            g0 = g1;
            if (b + 2 * step < tot) g1 = particle_of(m + 2 * step);
            if (m < tot) {
                L.map[m] = (int32_t)g;
                const double2* x = reinterpret_cast<const double2*>(s.XV + g);
                const double2* u = reinterpret_cast<const double2*>(s.U[par] + g);
                const uint32_t at = (uint32_t)b * 16;
                lds_dma16(x, l_xy + at);
                lds_dma16_next(x, l_zv + at);
                lds_dma16(u, l_uxy + at);
                lds_dma16_next(u, l_uz + at);
                if constexpr (kVarH) L.hs[m] = s.hs[g];
            }
        }
    }
    __syncthreads();   // the map
    if (wave < nw)
        stage_records<K, (int)sizeof(GQRec<R>)>(gh_of<R>(s), lds_addr(L.rec), L.map, tot, wave, nw, lane);
    const R inv_h = R(s.specs[sp].inv_h);
    // (neighbours past the packed slots)
    const uint16_t* __restrict__ lp = s.lcol + s.slice_ptr[ii / kSlice] + (ii % kSlice);
    const auto idx = [&](int k) { return (int)lp[(int64_t)(k < cnt ? k : 0) * kSlice]; };
    lds_dma_wait();
    __syncthreads();

    const int own = in ? pl : 0;
    const double2 xyi = L.xy[own], zvi = L.zv[own];
    const double hsi = kVarH ? L.hs[own] : 0.0;
    R gv[G][NP];   // V_j s / r of the packed slots' pairs
    const auto geom = [&](int j, bool live) {
        const double2 a = L.xy[j], b = L.zv[j];
        return pair_geom<R, kVarH>(xyi.x, xyi.y, zvi.x, a.x, a.y, b.x, R(b.y), hsi,
                                   kVarH ? L.hs[j] : 0.0, inv_h, live);
    };
    ForceAcc<R> A;
    {
        HgAcc<R> B[NP];
        const double2 uxyi = L.uxy[own];
        const double uzi = L.uz[own].x;
        const LdsGH<R> hi = L.gh(own);
        const auto pair = [&](int j, bool live, HgAcc<R>& acc) {
            const PairGeom<R> p = geom(j, live);
            const double2 a = L.uxy[j];
            const double uz = L.uz[j].x;
            const LdsGH<R> hj = L.gh(j);
            hg_pair<R>(p, hj.vw, R(a.x - uxyi.x), R(a.y - uxyi.y), R(uz - uzi), hi.h, hj.h, live, acc);
            return p.gv;
        };
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (g * kSub < cnt) {
#pragma unroll
                for (int t = 0; t < NP; ++t) {
                    const bool live = g * kSub + sub + S * t < cnt;
                    // (a bulk particle of a cubic lattice has 18 neighbours:
                    // its fifth group is half empty)
                    if (g < 4 || live) gv[g][t] = pair(slots.at(g, t), live, B[t]);
                }
            }
        for (int k0 = G * kSub; k0 < cnt; k0 += kSub) {
#pragma unroll
            for (int t = 0; t < NP; ++t) {
                const int k = k0 + sub + S * t;
                pair(idx(k), k < cnt, B[t]);
            }
        }
        A.hg = combine_partials<S>(B);
    }
    __syncthreads();   // every wave is done with H
    const FinishIn fin = finish_in(s, ii, zvi.y);
    if (wave < nw)
        stage_records<K, (int)sizeof(GQRec<R>)>(gq_of<R>(s), lds_addr(L.rec), L.map, tot, wave, nw, lane);
    lds_dma_wait();
    __syncthreads();
    {
        StressAcc<R> B[NP];
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (g * kSub < cnt) {
#pragma unroll
                for (int t = 0; t < NP; ++t)
                    if (g < 4 || g * kSub + sub + S * t < cnt) {
                        const int j = slots.at(g, t);
                        const double2 a = L.xy[j];
                        const double z = L.zv[j].x;
                        const LdsGQ<R> q = L.gq(j);
                        const R w = gv[g][t];
                        stress_pair<R>(w * R(a.x - xyi.x), w * R(a.y - xyi.y), w * R(z - zvi.x),
                                       q.omd, q.q, B[t]);
                    }
            }
        for (int k0 = G * kSub; k0 < cnt; k0 += kSub) {
#pragma unroll
            for (int t = 0; t < NP; ++t) {
                const int k = k0 + sub + S * t;
                const int j = idx(k);
                const PairGeom<R> p = geom(j, k < cnt);
                const LdsGQ<R> q = L.gq(j);
                stress_pair<R>(p.gv * p.dx, p.gv * p.dy, p.gv * p.dz, q.omd, q.q, B[t]);
            }
        }
        A.st = combine_partials<S>(B);
    }
    if (in && sub == 0) {
        LRecB<R> ni;
        const double2 a = L.uxy[pl];
        const LdsGQ<R> q = L.gq(pl);
        ni.x = xyi.x; ni.y = xyi.y; ni.z = zvi.x;
        ni.ux = a.x; ni.uy = a.y; ni.uz = L.uz[pl].x;
#pragma unroll
        for (int k = 0; k < 9; ++k) ni.q[k] = q.q[k];
        force_finish<R, kVarH>(s, i, par, sp, ni, A, fin);
    }
}

// LDS of the pipelined force pass for a tile and its halo (M slots): the planes
// and both regions of records of LdsB, and two maps (this tile's, the next's).
template <typename R>
struct LdsP {
    static constexpr int kRec = LdsB<R>::kRec;
    static constexpr int kBytes = 4 * 16 + 2 * kRec * 16 + 2 * 4;
    double2* xy;
    double2* zv;
    double2* uxy;
    double2* uz;
    LdsGH<R>* gh;
    LdsGQ<R>* gq;
    int32_t* map;
    __device__ LdsP(unsigned char* raw, int M) {
        xy = reinterpret_cast<double2*>(raw);
        zv = xy + M;
        uxy = zv + M;
        uz = uxy + M;
        gh = reinterpret_cast<LdsGH<R>*>(uz + M);
        gq = reinterpret_cast<LdsGQ<R>*>(gh + M);
        map = reinterpret_cast<int32_t*>(gq + M);
    }
};

// Workgroup barrier that publishes LDS stores and waits for no vector memory.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// stage_records a chunk (one load per lane) at a time, so that the loads can be
// issued between pieces of arithmetic: issuing them together stalls the wave
// for about twenty cycles each.
template <int K, int kStride>
struct RecordStager {
    const unsigned char* base;
    const int32_t* map;
    uint32_t dst;
    int c, n_waves, units, lane;
    int32_t m, f;   // slot and unit within its record of the lane's unit of chunk c
    int32_t g;      // the slot's particle
    __device__ void start(const void* src, uint32_t dst_, const int32_t* map_, int tot, int wave,
                          int n_waves_, int lane_) {
        base = static_cast<const unsigned char*>(src);
        map = map_;
        dst = dst_;
        units = wave < n_waves_ ? tot * K : 0;
        c = wave * 64;
        n_waves = n_waves_;
        lane = lane_;
        const uint32_t e = (uint32_t)(c + lane);
        m = (int32_t)(e / K);
        f = (int32_t)e - m * K;
        g = map[c + lane < units ? m : 0];
    }
    __device__ void issue() {
        if (c >= units) return;
        const unsigned char* p = base + ((uint64_t)(uint32_t)g * kStride + (uint32_t)(f << 4));
        if (c + 64 <= units)
            lds_dma16(p, dst + (uint32_t)c * 16);
        else if (c + lane < units)
            lds_dma16(p, dst + (uint32_t)c * 16);
        // the next chunk: 64 n_waves units on
        c += n_waves * 64;
        const int dm = n_waves * 64 / K, df = n_waves * 64 - dm * K;
        f += df;
        m += dm;
        const int over = f >= K ? 1 : 0;
        f -= over ? K : 0;
        m += over;
        if (c < units) g = map[c + lane < units ? m : 0];
    }
    __device__ void rest() {
        while (c < units) issue();
    }
};

// What a thread of the pipelined force pass holds of the next tile: loaded
// values as they are (nothing computes with them before they have arrived:
// vector loads return in order, so a wait for one of them would be a wait for
// the records travelling with it).
constexpr int kPipeRounds = 2;
struct TileIn {
    int32_t h[kPipeRounds];   // halo-row entries of the thread's first slots
    int32_t halo, nnb, sp;
};

// Values computed by here: not sunk past the loads issued between the pairs,
// which would keep every pair's inputs in registers instead.
template <typename R>
__device__ __forceinline__ void settle_here(R& a, R& b, R& c) {
    asm volatile("" : "+v"(a), "+v"(b), "+v"(c));
}

// The staged force pass pipelined over a workgroup's tiles (two lanes per
// particle, both records of the image in LDS).  One tile per workgroup spends a
// third of its time on the latencies of its first loads, of the staging and of
// the finish, and LDS holds too few workgroups to cover them.  Here the copies
// into LDS run behind the arithmetic: while the first sweep (H, u: the hourglass
// sums) runs, Q travels, and the next tile's first loads; while the second (Q:
// the stress sums) runs, the next tile's positions, displacements, H and
// neighbour slots, into what the first sweep is done with.  A wait is explicit,
// once per sweep (vmcnt counts the finish's two stores too, issued last).
// What bounds it: FP64 issue (1.89e8 VALU instructions at 4.1M particles, 307 us of
// them on every SIMD) and LDS (bank conflicts of records read at random alone hold
// it for 151 us).  4.1M-particle plate, FP64: one sweep, tiles of 96, 715 us, this,
// tiles of 253, 617; mixed 558 and 490.
template <typename R>
__device__ __forceinline__ void pass_b_pipe(const DevState& s, int par) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    constexpr int S = 2, K = LdsP<R>::kRec, G = kPipeGroups, NP = kSub / S;
    const int M = s.lds_slots;
    const LdsP<R> L(lds_raw, M);
    const int T = s.tile;
    const int32_t n = (int32_t)s.n;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nw = (int)blockDim.x >> 6;   // full waves: they stage (a tile has at least one)
    const int step = nw * 64;
    const int m0 = wave * 64 + lane;
    const int pl = threadIdx.x / S;
    const int sub = threadIdx.x % S;
    const uint32_t l_xy = lds_addr(L.xy), l_zv = lds_addr(L.zv), l_uxy = lds_addr(L.uxy),
                   l_uz = lds_addr(L.uz), l_gh = lds_addr(L.gh), l_gq = lds_addr(L.gq);
    TileWalk walk(s.tile_list, s.run_count, (s.n + T - 1) / T);
    int32_t tile = walk.settle(walk.load());
    if (tile < 0) return;
    int32_t next = walk.settle(walk.load());
    int32_t v0 = 0;   // a per-lane zero: loads through it stay vector loads, whose
    asm volatile("" : "+v"(v0));   // value nothing waits for until it is settled

    const auto row = [&](int32_t t, int m) {   // halo-row entry of slot m, an index inside the row
        const int h = m - T;
        return s.halo[(int64_t)t * s.halo_cap + (h >= 0 && h < s.halo_cap ? h : 0)];
    };
    const auto load_first = [&](int32_t t) {
        TileIn in;
#pragma unroll
        for (int q = 0; q < kPipeRounds; ++q) in.h[q] = row(t, m0 + q * step);
        const int32_t i = t * T + pl;
        const int32_t ii = i < n ? i : t * T;
        in.nnb = s.nnb[ii];
        in.sp = s.spec[ii];
        in.halo = s.halo_cnt[t + v0];
        return in;
    };
    // The particle of each slot of tile t into a map (the tile's own, then its
    // halo; a slot past the particle count, in the last tile, takes the tile's first).
    const auto put_map = [&](int32_t t, TileIn& in, int32_t* map) {
        const int tot = T + in.halo;
        const auto one = [&](int m, int32_t h) {
            const int32_t g = m < T ? t * T + m : h;
            return g < n ? g : t * T;
        };
#pragma unroll
        for (int q = 0; q < kPipeRounds; ++q) {
            const int m = m0 + q * step;
            in.h[q] = one(m, in.h[q]);
            if (wave < nw && m < tot) map[m] = in.h[q];
        }
        if (wave < nw)
            for (int m = m0 + kPipeRounds * step; m < tot; m += step) map[m] = one(m, row(t, m));
    };
    // positions and displacements of the thread's own slots, round q of 64 per wave
    const auto plane_round = [&](const TileIn& in, const int32_t* map, int q) {
        const int b = wave * 64 + q * step;
        if (wave >= nw || b + lane >= T + in.halo) return;
        const int32_t g = q < kPipeRounds ? in.h[q] : map[b + lane];
        const double2* x = reinterpret_cast<const double2*>(s.XV + g);
        const double2* u = reinterpret_cast<const double2*>(s.U[par] + g);
        const uint32_t at = (uint32_t)b * 16;
        lds_dma16(x, l_xy + at);
        lds_dma16_next(x, l_zv + at);
        lds_dma16(u, l_uxy + at);
        lds_dma16_next(u, l_uz + at);
    };
    const auto plane_rest = [&](const TileIn& in, const int32_t* map, int q) {
        for (; wave * 64 + q * step < T + in.halo; ++q) plane_round(in, map, q);
    };
    const auto settle = [&](TileIn& in) {   // the loads have arrived
#pragma unroll
        for (int q = 0; q < kPipeRounds; ++q) asm volatile("" : "+v"(in.h[q]));
        asm volatile("" : "+v"(in.nnb), "+v"(in.sp), "+v"(in.halo));
        in.halo = __builtin_amdgcn_readfirstlane(in.halo);
    };

    RecordStager<K, (int)sizeof(GQRec<R>)> rs;
    Ramp ramp;
    int32_t* map = L.map;
    TileIn cur = load_first(tile);
    Slots<S> slots;
    {
        const int32_t i = tile * T + pl;
        slots = load_slots<S>(s.pslot, i < n ? i : tile * T, sub);
    }
    settle(cur);
    R inv_h = R(s.specs[cur.sp].inv_h);
    put_map(tile, cur, map);
    plane_rest(cur, map, 0);
    lds_barrier();
    rs.start(gh_of<R>(s), l_gh, map, T + cur.halo, wave, nw, lane);
    rs.rest();
    lds_dma_wait();
    lds_barrier();
    for (;;) {
        // Sweep 1 (X, V0, u, H): hourglass sums, and V_j s X_ij / r of each pair
        // kept for sweep 2.  This tile's Q, what its finish needs and the next
        // tile's first loads travel meanwhile.
        const int32_t i = tile * T + pl;
        const bool in = i < n;
        const int32_t ii = in ? i : tile * T;
        const int own = in ? pl : 0;
        const int cnt = in ? cur.nnb : 0;
        TileIn nxt = cur;
        if (next >= 0) nxt = load_first(next);
        int32_t next2 = walk.load() | v0;
        const double2 xyi = L.xy[own], zvi = L.zv[own], uxyi = L.uxy[own];
        const double uzi = L.uz[own].x;
        const FinishIn fin = finish_in(s, ii, zvi.y);
        rs.start(gq_of<R>(s), l_gq, map, T + cur.halo, wave, nw, lane);
        R gx[G * NP], gy[G * NP], gz[G * NP];
        ForceAcc<R> A;
        // Pair e of a lane is its partial e % NP's pair e / NP.  A bulk particle of a
        // cubic lattice has 18 neighbours, so a lane has nine pairs: the first
        // eight are always run (a slot past the last neighbour adds zeros), each
        // pair's LDS reads going out ahead of the one before it; the last group's
        // where some lane of the wave has them.
        const auto live = [&](int e) { return (e / NP) * kSub + sub + S * (e % NP) < cnt; };
        const auto slot = [&](int e) { return slots.at(e / NP, e % NP); };
        constexpr int kFull = (G - 1) * NP;
        {
            HgAcc<R> B[NP];
            struct Nbr {
                double2 xy, zv, uxy;
                double uz;
            };
            const LdsGH<R> hi = L.gh[own];
            const auto load = [&](int e) {
                const int j = slot(e);
                return Nbr{L.xy[j], L.zv[j], L.uxy[j], L.uz[j].x};
            };
            const auto pair = [&](const Nbr& d, int e) {
                const LdsGH<R> hj = L.gh[slot(e)];
                const PairGeom<R> p = pair_geom<R, false>(xyi.x, xyi.y, zvi.x, d.xy.x, d.xy.y, d.zv.x,
                                                          R(d.zv.y), 0.0, 0.0, inv_h, live(e));
                gx[e] = p.gv * p.dx;
                gy[e] = p.gv * p.dy;
                gz[e] = p.gv * p.dz;
                hg_pair<R>(p, hj.vw, R(d.uxy.x - uxyi.x), R(d.uxy.y - uxyi.y), R(d.uz - uzi), hi.h,
                           hj.h, live(e), B[e % NP]);
                settle_here(gx[e], gy[e], gz[e]);
                settle_here(B[e % NP].g0, B[e % NP].g1, B[e % NP].g2);
            };
            Nbr d = load(0);
#pragma unroll
            for (int e = 0; e < kFull; ++e) {
                const Nbr ahead = load(e + 1);
                rs.issue();
                pair(d, e);
                d = ahead;
            }
            rs.rest();
#pragma unroll
            for (int e = kFull; e < G * NP; ++e)
                if (__any(live(e))) {
                    if (e > kFull) d = load(e);
                    pair(d, e);
                }
            A.hg = combine_partials<S>(B);
        }
        lds_dma_wait();
        int32_t* map_n = map == L.map ? L.map + M : L.map;
        settle(nxt);
        if (next >= 0) put_map(next, nxt, map_n);
        next2 = walk.settle(next2);
        lds_barrier();

        // Sweep 2 (Q, 1 - D): stress sums.  The next tile's X, u, H and neighbour
        // slots travel meanwhile (X, u and H of this one are no longer read).
        Slots<S> slots_n = slots;
        R inv_h_n = inv_h;
        rs.units = 0;
        if (next >= 0) {
            const int32_t j = next * T + pl;
            slots_n = load_slots<S>(s.pslot, j < n ? j : next * T, sub);
            inv_h_n = R(s.specs[nxt.sp].inv_h);
            rs.start(gh_of<R>(s), l_gh, map_n, T + nxt.halo, wave, nw, lane);
        }
        {
            StressAcc<R> B[NP];
            const auto load = [&](int e) { return L.gq[slot(e)]; };
            const auto pair = [&](const LdsGQ<R>& q, int e) {
                stress_pair<R>(gx[e], gy[e], gz[e], q.omd, q.q, B[e % NP]);
                settle_here(B[e % NP].a0, B[e % NP].a1, B[e % NP].a2);
                settle_here(B[e % NP].b0, B[e % NP].b1, B[e % NP].b2);
            };
            LdsGQ<R> q = load(0);
#pragma unroll
            for (int e = 0; e < kFull; ++e) {
                const LdsGQ<R> ahead = load(e + 1);
                if (next >= 0 && e < 2) plane_round(nxt, map_n, e);
                if (e >= 2) rs.issue();
                pair(q, e);
                q = ahead;
            }
            if (next >= 0) {
                plane_rest(nxt, map_n, 2);
                rs.rest();
            }
#pragma unroll
            for (int e = kFull; e < G * NP; ++e)
                if (__any(live(e))) pair(e == kFull ? q : load(e), e);
            A.st = combine_partials<S>(B);
        }
        const bool stores = in && !frozen(s, cur.sp);
        meet_group(s, cur.sp, stores ? fin.bc : -1, ramp);
        if (stores) {
            LRecB<R> ni;
            const LdsGQ<R> q = L.gq[pl];
            ni.x = xyi.x; ni.y = xyi.y; ni.z = zvi.x;
            ni.ux = uxyi.x; ni.uy = uxyi.y; ni.uz = uzi;
#pragma unroll
            for (int k = 0; k < 9; ++k) ni.q[k] = q.q[k];
            force_finish<R, false, true>(s, i, par, cur.sp, ni, A, fin, &ramp, sub);
        }
        if (next < 0) return;
        // the next tile's records have arrived (the finish's two stores, which
        // follow them, need not have)
        if (__any(stores))
            lds_dma_wait<2>();
        else
            lds_dma_wait();
#pragma unroll
        for (int t = 0; t < NP; ++t)
#pragma unroll
            for (int w = 0; w < Slots<S>::W; ++w) asm volatile("" : "+v"(slots_n.w[t][w]));
        asm volatile("" : "+v"(inv_h_n));
        lds_barrier();
        tile = next;
        next = next2;
        cur = nxt;
        slots = slots_n;
        inv_h = inv_h_n;
        map = map_n;
    }
}

// LDS image of the one-sweep form: a record of everything a pair needs per slot,
// 208 bytes (mixed: 128; M slots).  FP64: records of 13 units of 16 bytes (an
// odd number); mixed: a plane for each unit.
template <typename R>
struct LdsOne;
template <>
struct LdsOne<double> {
    static constexpr int kUnits = 13;   // 26 doubles
    __device__ static void put(double2* L, int, int m, const LRecB<double>& r) {
        double2* p = L + m * kUnits;
        p[0] = double2{r.x, r.y};
        p[1] = double2{r.z, r.V0};
        p[2] = double2{r.ux, r.uy};
        p[3] = double2{r.uz, r.omd};
        p[4] = double2{r.q[0], r.q[1]};
        p[5] = double2{r.q[2], r.q[3]};
        p[6] = double2{r.q[4], r.q[5]};
        p[7] = double2{r.q[6], r.q[7]};
        p[8] = double2{r.q[8], r.h[0]};
        p[9] = double2{r.h[1], r.h[2]};
        p[10] = double2{r.h[3], r.h[4]};
        p[11] = double2{r.h[5], r.h[6]};
        p[12] = double2{r.h[7], r.h[8]};
    }
    __device__ static LRecB<double> get(const double2* L, int, int m) {
        const double2* p = L + m * kUnits;
        LRecB<double> r;
        double2 t;
        t = p[0]; r.x = t.x; r.y = t.y;
        t = p[1]; r.z = t.x; r.V0 = t.y;
        t = p[2]; r.ux = t.x; r.uy = t.y;
        t = p[3]; r.uz = t.x; r.omd = t.y;
        t = p[4]; r.q[0] = t.x; r.q[1] = t.y;
        t = p[5]; r.q[2] = t.x; r.q[3] = t.y;
        t = p[6]; r.q[4] = t.x; r.q[5] = t.y;
        t = p[7]; r.q[6] = t.x; r.q[7] = t.y;
        t = p[8]; r.q[8] = t.x; r.h[0] = t.y;
        t = p[9]; r.h[1] = t.x; r.h[2] = t.y;
        t = p[10]; r.h[3] = t.x; r.h[4] = t.y;
        t = p[11]; r.h[5] = t.x; r.h[6] = t.y;
        t = p[12]; r.h[7] = t.x; r.h[8] = t.y;
        return r;
    }
};
template <>
struct LdsOne<float> {
    static constexpr int kUnits = 8;    // 6 doubles + 20 floats
    __device__ static void put(double2* L, int M, int m, const LRecB<float>& r) {
        L[0 * M + m] = double2{r.x, r.y};
        L[1 * M + m] = double2{r.z, r.ux};
        L[2 * M + m] = double2{r.uy, r.uz};
        float4* F = reinterpret_cast<float4*>(L + 3 * M);
        F[0 * M + m] = float4{r.V0, r.omd, r.q[0], r.q[1]};
        F[1 * M + m] = float4{r.q[2], r.q[3], r.q[4], r.q[5]};
        F[2 * M + m] = float4{r.q[6], r.q[7], r.q[8], r.h[0]};
        F[3 * M + m] = float4{r.h[1], r.h[2], r.h[3], r.h[4]};
        F[4 * M + m] = float4{r.h[5], r.h[6], r.h[7], r.h[8]};
    }
    __device__ static LRecB<float> get(const double2* L, int M, int m) {
        LRecB<float> r;
        double2 t;
        t = L[0 * M + m]; r.x = t.x; r.y = t.y;
        t = L[1 * M + m]; r.z = t.x; r.ux = t.y;
        t = L[2 * M + m]; r.uy = t.x; r.uz = t.y;
        const float4* F = reinterpret_cast<const float4*>(L + 3 * M);
        float4 f;
        f = F[0 * M + m]; r.V0 = f.x; r.omd = f.y; r.q[0] = f.z; r.q[1] = f.w;
        f = F[1 * M + m]; r.q[2] = f.x; r.q[3] = f.y; r.q[4] = f.z; r.q[5] = f.w;
        f = F[2 * M + m]; r.q[6] = f.x; r.q[7] = f.y; r.q[8] = f.z; r.h[0] = f.w;
        f = F[3 * M + m]; r.h[1] = f.x; r.h[2] = f.y; r.h[3] = f.z; r.h[4] = f.w;
        f = F[4 * M + m]; r.h[5] = f.x; r.h[6] = f.y; r.h[7] = f.z; r.h[8] = f.w;
        return r;
    }
};

// Waves per SIMD the one-sweep form must leave room for: two workgroups per
// CU need four (mixed form, two or four lanes per particle: tiles up to 196
// and 128 particles) or three (FP64, four lanes: tiles up to 96).  With graded
// spacing the mixed form needs more than 128 registers: three.
template <typename R, int S, bool kVarH = false>
__host__ __device__ constexpr int one_sweep_waves_min() {
    return sizeof(R) == 4 && S >= 2 ? (kVarH ? 3 : 4) : (S == 4 ? 3 : 1);
}
// Whether the finish's inputs are loaded before the staging (their registers
// then live through the pair sums; the mixed form with two lanes has none to
// spare within its 128).
template <typename R, int S>
__host__ __device__ constexpr bool one_sweep_finish_early() {
    return !(sizeof(R) == 4 && S == 2);
}

// The staged force pass in one sweep over an image of whole records, staged
// through registers, a workgroup per tile: a chain of few latencies, which is
// what bounds it where tiles are few (25k particles FP64, tiles of 98: 12.3 us,
// 12.8 with a load for each neighbour slot and the groups' records by lane).
// Graded spacing (kVarH): the slots' support radii follow the records in LDS (one
// double per slot).
template <typename R, int S, bool kVarH = false>
__global__ void __launch_bounds__(staged_block_max(S))
__attribute__((amdgpu_waves_per_eu(one_sweep_waves_min<R, S, kVarH>(), 8)))
k_pass_b_one(DevState s, int par) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    constexpr int NP = kSub / S, G = kPackGroups;
    double2* __restrict__ L = reinterpret_cast<double2*>(lds_raw);
    const int M = s.lds_slots;
    double* __restrict__ Lhs = reinterpret_cast<double*>(L + (size_t)M * LdsOne<R>::kUnits);
    const int T = s.tile;
    const int B = T * S;
    const int64_t tile = work_tile(s.tile_list, s.run_count, 1, 0, gridDim.x);
    if (tile < 0) return;
    const int64_t start = tile * T;
    const int32_t* __restrict__ hl = s.halo + tile * (int64_t)s.halo_cap;
    const D4* __restrict__ XV = s.XV;
    const D4* __restrict__ Uc = s.U[par];
    const GQRec<R>* __restrict__ GQ = gq_of<R>(s);
    const GHRec<R>* __restrict__ GH = gh_of<R>(s);
    // Two slots per thread per round, their index loads issued before their
    // record loads and those before the LDS stores.  The first round's halo
    // indices are loaded before anything else; the particle's own scalars, its
    // neighbour slots and what its finish needs follow, so that their
    // latencies overlap those of the staging.  The first round needs no halo
    // count (slots past the image hold n): FP64 reads the count after it (two
    // memory latencies before the barrier); the mixed form reads it first.
    // Slots past the image, and past the particle count (last tile), load the
    // tile's first record and store nothing.
    const auto particle_of = [&](int m) { return slot_particle(m, T, s.halo_cap, start, s.n, hl); };
    int m0 = threadIdx.x;
    int64_t g0 = particle_of(m0), g1 = particle_of(m0 + B);
    const int pl = threadIdx.x / S;
    const int sub = threadIdx.x % S;
    const int64_t i = start + pl;
    const bool in = i < s.n;
    const int64_t ii = in ? i : start;
    const int cnt = in ? s.nnb[i] : 0;
    const int sp = s.spec[ii];
    const Slots<S> slots = load_slots<S>(s.pslot, ii, sub);
    // (neighbours past the packed slots, which graded spacing often has: the first
    // of them too ahead of the staging)
    const uint16_t* __restrict__ lp = s.lcol + s.slice_ptr[ii / kSlice] + (ii % kSlice);
    int q[NP];
    const auto tail = [&](int k) { return (int)lp[(int64_t)(k < cnt ? k : 0) * kSlice]; };
    if constexpr (kVarH) {
#pragma unroll
        for (int t = 0; t < NP; ++t) q[t] = tail(G * kSub + sub + S * t);
    }
    const R inv_h = R(s.specs[sp].inv_h);
    constexpr bool kEarly = one_sweep_finish_early<R, S>();
    FinishIn fin_early;
    if constexpr (kEarly) fin_early = finish_in(s, ii, XV[ii].w);
    const auto stage = [&](int m0, int64_t g0, int64_t g1) {
        const int64_t l0 = g0 < s.n ? g0 : start, l1 = g1 < s.n ? g1 : start;
        const LRecB<R> r0 = make_recb<R>(XV[l0], GQ[l0], GH[l0], Uc[l0]);
        const LRecB<R> r1 = make_recb<R>(XV[l1], GQ[l1], GH[l1], Uc[l1]);
        double h0 = 0.0, h1 = 0.0;
        if constexpr (kVarH) {
            h0 = s.hs[l0];
            h1 = s.hs[l1];
        }
        if (g0 < s.n) {
            LdsOne<R>::put(L, M, m0, r0);
            if constexpr (kVarH) Lhs[m0] = h0;
        }
        if (g1 < s.n) {
            LdsOne<R>::put(L, M, m0 + B, r1);
            if constexpr (kVarH) Lhs[m0 + B] = h1;
        }
    };
    if constexpr (sizeof(R) == 8) {
        stage(m0, g0, g1);
        const int tot = T + s.halo_cnt[tile];
        for (m0 += 2 * B; m0 < tot; m0 += 2 * B) stage(m0, particle_of(m0), particle_of(m0 + B));
    } else {
        const int tot = T + s.halo_cnt[tile];
        for (; m0 < tot; m0 += 2 * B) {
            stage(m0, g0, g1);
            g0 = particle_of(m0 + 2 * B);
            g1 = particle_of(m0 + 3 * B);
        }
    }
    __syncthreads();
    const auto rec = [&](int m) {
        LRecB<R> r = LdsOne<R>::get(L, M, m);
        if constexpr (kVarH) r.hs = Lhs[m];
        return r;
    };
    ForceAcc<R> A;
    {
        const LRecB<R> ni = rec(in ? pl : 0);
        ForceAcc<R> P[NP];
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (g * kSub < cnt) {
#pragma unroll
                for (int t = 0; t < NP; ++t)
                    force_pair<R, kVarH>(ni, rec(slots.at(g, t)), inv_h, P[t],
                                         g * kSub + sub + S * t < cnt);
            }
        if (G * kSub < cnt) {   // neighbours past the packed slots, loaded one group ahead
            if constexpr (!kVarH) {
#pragma unroll
                for (int t = 0; t < NP; ++t) q[t] = tail(G * kSub + sub + S * t);
            }
            for (int k0 = G * kSub; k0 < cnt; k0 += kSub) {
                int cur[NP];
#pragma unroll
                for (int t = 0; t < NP; ++t) {
                    cur[t] = q[t];
                    q[t] = tail(k0 + kSub + sub + S * t);
                }
#pragma unroll
                for (int t = 0; t < NP; ++t)
                    force_pair<R, kVarH>(ni, rec(cur[t]), inv_h, P[t], k0 + sub + S * t < cnt);
            }
        }
        A = combine_partials<S>(P);
    }
    // the particle's own record is needed only now: reread it rather than keep
    // it in registers through the pair loop (the image is not written after the
    // barrier above, so a compiler barrier suffices: waves go on to their
    // finish as their own sums end)
    asm volatile("" ::: "memory");
    if (in && sub == 0)
        force_finish<R, kVarH>(s, i, par, sp, LdsOne<R>::get(L, M, pl), A,
                               kEarly ? fin_early : finish_in(s, ii, XV[ii].w));
}

// The same in the forms that stage by asynchronous copies: pipelined with two
// lanes per particle and one support for all, else (FP64) in two sweeps.
template <typename R, int S, bool kVarH = false>
__global__ void __launch_bounds__(staged_block_max(S))
__attribute__((amdgpu_waves_per_eu((!kVarH && S == 2) ? 2 : staged_waves_min<S>(), 8)))
k_pass_b_staged(DevState s, int par) {
    if constexpr (!kVarH && S == 2)
        pass_b_pipe<R>(s, par);
    else
        pass_b_sweeps<S, kVarH>(s, par);
}

// Pass A (deformation and constitutive update to t^{n+1}).
//   dF/dt_i = sum_j V_j (1 - D_j)(v_j - v_i) (x) gradW_ij L_i^-1
// (eq. Crack_approx_Fdot, D at level n), accumulated as
// M = sum_j V_j (1 - D_j)(v_j - v_i) (x) gradW_ij and dF/dt = M L_i^-1; then
// the constitutive update and Q_i = P_i L_i^-T (0 for failed particles).
// A neighbour as the deformation pass needs it: reference position,
// half-step velocity and V0 (1 - D).
struct NbrA {
    double x, y, z, vx, vy, vz, w;
    double hs;   // support radius (graded spacing only)
};

// Artificial viscosity of one specimen as the gather uses it: pair factor
// -Q1 c0 mu + Q2 mu^2 (Pi rho0) for approaching pairs, mu = h v_ij.X_ij /
// (|X_ij|^2 + 0.01 h^2).
template <typename R>
struct AvPar {
    R q1c0, q2, h, eh2;
    bool on;
};
template <typename R>
__device__ __forceinline__ AvPar<R> av_par(const DevSpec& P) {
    return AvPar<R>{R(P.av_q1 * P.c0), R(P.av_q2), R(P.h), R(0.01 * P.h * P.h),
                    P.av_q1 != 0.0 || P.av_q2 != 0.0};
}

// The first G groups of a particle's neighbour indices (neighbours below
// kGatherA G), loaded before the staging of the staged pass; its local slots
// are below 2^16, two to a register.
constexpr int kGatherA = 4;
template <int G>
struct PreIdxA {
    uint32_t w[G][kGatherA / 2];
    __device__ int at(int g, int t) const {
        return (int)((t & 1) ? w[g][t >> 1] >> 16 : w[g][t >> 1] & 0xffffu);
    }
};
template <int G, typename IdxOf>
__device__ __forceinline__ PreIdxA<G> pre_indices_a(int cnt, IdxOf idx) {
    PreIdxA<G> p;
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int t = 0; t < kGatherA; t += 2) {
            const int k = g * kGatherA + t;
            p.w[g][t >> 1] = (uint32_t)idx(k < cnt ? k : 0) |
                             ((uint32_t)idx(k + 1 < cnt ? k + 1 : 0) << 16);
        }
    return p;
}

// One group of kGatherA neighbours of the deformation pass's sums (group
// start k0): record loads first, then the arithmetic.
template <typename R, bool kExt, bool kVarH, typename RecOf>
__device__ __forceinline__ void gather_group(const D4& xi, const D4& vi, int cnt, int k0, R inv_h,
                                             const int (&j)[kGatherA], RecOf rec, R M[9],
                                             const AvPar<R>& av, R AV[3], double hi) {
    NbrA nb[kGatherA];
#pragma unroll
    for (int t = 0; t < kGatherA; ++t) nb[t] = rec(j[t]);
#pragma unroll
    for (int t = 0; t < kGatherA; ++t) {
        // past the last neighbour 1/r = 0 makes every term an exact zero
        const bool live = k0 + t < cnt;
        const R dx = R(nb[t].x - xi.x), dy = R(nb[t].y - xi.y), dz = R(nb[t].z - xi.z);
        const R r2 = fma(dx, dx, fma(dy, dy, dz * dz));
        const R ir = live ? rsqrt_pos(r2) : R(0);
        R ih = inv_h, hpair = av.h;
        if constexpr (kVarH) {
            hpair = R(0.5 * (hi + nb[t].hs));
            ih = rcp_nr(hpair);
        }
        const R q = r2 * ir * ih;
        // h dW/dr / c = -6 (1 - q)^2 + 24 max(1/2 - q, 0)^2, no branch
        const R a = R(1) - q;
        const R b = fmax(R(0.5) - q, R(0));
        const R sl = fma(R(24), b * b, R(-6) * (a * a));
        R gw = sl * ir * R(nb[t].w);
        if constexpr (kVarH) gw *= R(8.0 / M_PI) * ih * ih * ih * ih;
        const R gx = gw * dx, gy = gw * dy, gz = gw * dz;
        const R t0 = R(nb[t].vx - vi.x), t1 = R(nb[t].vy - vi.y), t2 = R(nb[t].vz - vi.z);
        M[0] = fma(t0, gx, M[0]); M[1] = fma(t0, gy, M[1]); M[2] = fma(t0, gz, M[2]);
        M[3] = fma(t1, gx, M[3]); M[4] = fma(t1, gy, M[4]); M[5] = fma(t1, gz, M[5]);
        M[6] = fma(t2, gx, M[6]); M[7] = fma(t2, gy, M[7]); M[8] = fma(t2, gz, M[8]);
        if constexpr (kExt) {
            // sum_j (-Q1 c0 mu + Q2 mu^2) V_j (1 - D_j) gradW_ij over approaching pairs
            if (av.on) {
                const R vx = fma(t0, dx, fma(t1, dy, t2 * dz));
                if (vx < R(0)) {
                    const R eh2 = kVarH ? R(0.01) * hpair * hpair : av.eh2;
                    const R mu = hpair * vx * rcp_nr(r2 + eh2);
                    const R pi = mu * fma(av.q2, mu, -av.q1c0);
                    AV[0] = fma(pi, gx, AV[0]);
                    AV[1] = fma(pi, gy, AV[1]);
                    AV[2] = fma(pi, gz, AV[2]);
                }
            }
        }
    }
}

// M = sum_j V_j (1 - D_j)(v_j - v_i) (x) gradW_ij over the neighbours in
// increasing order, in groups of kGatherA whose record loads are all issued
// before their arithmetic: the first G groups from preloaded indices, the
// rest with indices one group ahead.  The kernel slope enters without its
// constant factor c / h (c = 8 / (pi h^3)), applied to the sum.  Graded
// spacing (kVarH): each pair has its own support h_ij = (h_i + h_j)/2 (h_i =
// hi), and the kernel's constant factor enters per pair (grad_k = 1).
template <typename R, bool kExt, bool kVarH = false, int G = 0, typename IdxOf, typename RecOf>
__device__ __forceinline__ void gather_fdot(const D4& xi, const D4& vi, int cnt, R inv_h, R grad_k,
                                            IdxOf idx, RecOf rec, R M[9], const AvPar<R>& av,
                                            R AV[3], double hi = 0.0,
                                            const PreIdxA<(G > 0 ? G : 1)>* pre = nullptr) {
#pragma unroll
    for (int q = 0; q < 9; ++q) M[q] = R(0);
    AV[0] = AV[1] = AV[2] = R(0);
    // the first group past the preloaded ones goes out first
    int jn[kGatherA];
#pragma unroll
    for (int t = 0; t < kGatherA; ++t) {
        const int k = G * kGatherA + t;
        jn[t] = idx(k < cnt ? k : 0);
    }
    if constexpr (G > 0) {
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (g * kGatherA < cnt) {
                int j[kGatherA];
#pragma unroll
                for (int t = 0; t < kGatherA; ++t) j[t] = pre->at(g, t);
                gather_group<R, kExt, kVarH>(xi, vi, cnt, g * kGatherA, inv_h, j, rec, M, av, AV,
                                             hi);
            }
    }
    for (int k0 = G * kGatherA; k0 < cnt; k0 += kGatherA) {
        int j[kGatherA];
#pragma unroll
        for (int t = 0; t < kGatherA; ++t) {
            j[t] = jn[t];
            const int kn = k0 + kGatherA + t;
            jn[t] = idx(kn < cnt ? kn : 0);
        }
        gather_group<R, kExt, kVarH>(xi, vi, cnt, k0, inv_h, j, rec, M, av, AV, hi);
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) M[q] *= grad_k;
    if constexpr (kExt) {
        AV[0] *= grad_k; AV[1] *= grad_k; AV[2] *= grad_k;
    }
}

// The rest of the deformation pass for particle i (specimen sp) given M:
// dF/dt = M L_i^-1, the constitutive update, Q_i = P_i L_i^-T, stores.
// The first input of the particle's update, L^-1: the staged pass loads it
// before its neighbour sums, which then hide its latency (loading H^n and
// sigma^n there too would spill registers in the neighbour sums).
template <typename R>
struct UpdIn {
    R Li[9];
};
template <typename R>
__device__ __forceinline__ UpdIn<R> load_upd_in(const DevState& s, int64_t i) {
    const int64_t np = s.np;
    UpdIn<R> u;
    if constexpr (std::is_same<R, float>::value) {
#pragma unroll
        for (int k = 0; k < 9; ++k) u.Li[k] = s.Linv32[k * np + i];
    } else {
#pragma unroll
        for (int k = 0; k < 9; ++k) u.Li[k] = s.Linv[k * np + i];
    }
    return u;
}

template <typename R, int DM, bool kFlow>
__device__ __forceinline__ void pass_a_update(const DevState& s, int64_t i, int sp, const R M[9],
                                              double wi, const R AV[3], const UpdIn<R>& in) {
    const int64_t np = s.np;
    const DevSpec& P = s.specs[sp];
    R Li[9];
    R Fd[9];
    mm33(M, in.Li, Fd);
    GQRec<R>* __restrict__ GQ = gq_of<R>(s);
    GHRec<R>* __restrict__ GH = gh_of<R>(s);
    R Hn[9], sn[6], vw;
    {
        const GHRec<R> gi = GH[i];
#pragma unroll
        for (int k = 0; k < 9; ++k) Hn[k] = gi.h[k];
        vw = gi.vw;
    }
    if constexpr (std::is_same<R, float>::value) {
#pragma unroll
        for (int k = 0; k < 6; ++k) sn[k] = s.sig32[k * np + i];
    } else {
#pragma unroll
        for (int k = 0; k < 6; ++k) sn[k] = s.sig[k * np + i];
    }
    double eps = s.eps_p[i], rate = s.eps_rate[i], e = s.e[i];
    const double rate0 = rate;
    double dinit = 0.0, wp = 0.0, fv = 0.0;
    const int model = DM >= 0 ? DM : P.damage;
    if (model == 1 || model == 2) dinit = s.d_init[i];
    if (model == 1) wp = s.w_p[i];
    if (model == 3) fv = s.f_void[i];
    const double Di = s.D[i];
    PointOut<R> o;
    int32_t flags = 0;
    point_update<R, DM, kFlow>(P, Hn, Fd, sn, eps, rate, dinit, wp, fv, e, Di, o, flags);
    // stores: the index passes through an empty asm so that store addresses
    // are formed here rather than kept in registers from the loads above
    int64_t is = i;
    asm volatile("" : "+v"(is));
    if constexpr (std::is_same<R, float>::value) {
#pragma unroll
        for (int k = 0; k < 6; ++k) s.sig32[k * np + is] = o.sig[k];
    } else {
#pragma unroll
        for (int k = 0; k < 6; ++k) s.sig[k * np + is] = o.sig[k];
    }
    // L^-1 again (cached), rather than held in registers through the update
    if constexpr (std::is_same<R, float>::value) {
#pragma unroll
        for (int k = 0; k < 9; ++k) Li[k] = s.Linv32[k * np + is];
    } else {
#pragma unroll
        for (int k = 0; k < 9; ++k) Li[k] = s.Linv[k * np + is];
    }
    GQRec<R> go;
    GHRec<R> ho;
    const bool failed = o.D >= 1.0;
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b)
            go.q[3 * a + b] = failed ? R(0)
                                     : dot3(o.P[3 * a], Li[3 * b], o.P[3 * a + 1], Li[3 * b + 1],
                                            o.P[3 * a + 2], Li[3 * b + 2]);
#pragma unroll
    for (int k = 0; k < 9; ++k) ho.h[k] = o.H[k];
    go.omd = R(1.0 - o.D);
    // V0 (1 - D) for the force pass, kept with H: as it was unless D changed.  FP64:
    // formed anew from V0 (read again, as L^-1 is: cached), since the value held
    // through the update costs spills (1M particles 153 us, so 149; mixed 4.1M,
    // which has registers for it, 512 and 516)
    if constexpr (std::is_same<R, double>::value)
        ho.vw = s.XV[is].w * go.omd;
    else
        ho.vw = o.D != Di ? R(s.XV[is].w) * go.omd : vw;
    GQ[is] = go;
    GH[is] = ho;
    // The plastic strain and its accumulators change only where the particle
    // yields (rate = increment / dt is then nonzero; a zero increment leaves
    // every one of them as it was), the rate also where it stops yielding, D
    // only where it grows: the other particles (most, in an elastic body)
    // store none of them, and memory lines holding no changed value are not
    // written.
    if (Di < 1.0) {
        s.e[is] = e;
        if (rate != 0.0) {
            s.eps_p[is] = eps;
            if (model == 1 || model == 2) s.d_init[is] = dinit;
            if (model == 1) s.w_p[is] = wp;
            if (model == 3) s.f_void[is] = fv;
        }
        if (rate != rate0) s.eps_rate[is] = rate;
    }
    if (o.D != Di) s.D[is] = o.D;
    if constexpr (kFlow) {
        // artificial viscous force for the next kick: rho0 V_i (1 - D_i) times
        // the gathered sum (w_i = V_i (1 - D_i^n))
        if (s.av) {
            const double k = P.rho0 * wi;
            s.fvisc[is] = k * double(AV[0]);
            s.fvisc[np + is] = k * double(AV[1]);
            s.fvisc[2 * np + is] = k * double(AV[2]);
        }
    }
    if (i == P.first) s.t[sp] += P.dt;
    if (flags || (s.flags & kFlagCheckFinite)) {
        int32_t fl = flags;
        if (s.flags & kFlagCheckFinite) {
            bool ok = true;
#pragma unroll
            for (int k = 0; k < 6; ++k) ok = ok && isfinite(double(o.sig[k]));
            if (!ok) fl |= kErrNonFinite;
        }
        if (fl) atomicOr(&s.err[2], fl);
    }
}

// Waves per SIMD the deformation pass is compiled for: three (at most 168
// registers) for each single damage model with Johnson-Cook hardening and
// the explicit return, and for the mixed form with the other flow laws (JC
// or no damage).  The FP64 GTN variant then spills 76 bytes (outside its
// Newton loops) and still runs faster than at two waves; the mixed-model
// variant and the FP64 form with the other flow laws would spill more and
// keep their registers.
template <typename R, int DM, bool kFlow>
__host__ __device__ constexpr int pass_a_waves_min() {
    return DM >= 0 && DM <= 3 && (!kFlow || (sizeof(R) == 4 && DM != 1)) ? 3 : 1;
}

// Specimen parameters are read with scalar loads: the lanes of a wave take
// turns by specimen, one turn unless the wave straddles two specimens.
template <typename R, int DM, bool kFlow, bool kVarH = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(pass_a_waves_min<R, DM, kFlow>(), 8)))
k_pass_a(DevState s, int /* displacement buffer: unused here */) {
    const int64_t i = xcd_tile<true>(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    if (i >= s.n) return;
    const int sp_lane = s.spec[i];
    if (frozen(s, sp_lane)) return;
    for (;;) {
        const int sp = __builtin_amdgcn_readfirstlane(sp_lane);
        if (sp == sp_lane) {
            const DevSpec& P = s.specs[sp];
            const D4* __restrict__ XV = s.XV;
            const D4* __restrict__ VW = s.VW;
            const int32_t* __restrict__ cp = s.col + s.slice_ptr[i / kSlice] + (i % kSlice);
            R M[9], AV[3];
            const D4 vi = VW[i];
            gather_fdot<R, kFlow, kVarH>(XV[i], vi, s.nnb[i], R(P.inv_h),
                                         kVarH ? R(1) : R(P.grad_k),
                                         [&](int k) { return (int)cp[(int64_t)k * kSlice]; },
                                         [&](int j) {
                                             const D4 x = XV[j], v = VW[j];
                                             return NbrA{x.x, x.y, x.z, v.x, v.y, v.z, v.w,
                                                         kVarH ? s.hs[j] : 0.0};
                                         }, M, av_par<R>(P), AV, kVarH ? s.hs[i] : 0.0);
            pass_a_update<R, DM, kFlow>(s, i, sp, M, vi.w, AV, load_upd_in<R>(s, i));
            break;
        }
    }
}

// Neighbour-index groups the staged deformation pass loads before its
// staging.
template <typename R, bool kPacked>
__host__ __device__ constexpr int staged_a_pre_groups() {
    return sizeof(R) == 8 || kPacked ? kPackGroups : 3;
}
// The same from the packed slots (lists t, t + kSub, ... to groups of kGatherA).
__device__ __forceinline__ PreIdxA<kPackGroups> packed_indices_a(const uint32_t* __restrict__ pslot,
                                                                 int64_t i) {
    static_assert(kGatherA == kSub && kPackGroups == 6 && kPackWords == 12, "three words a list");
    uint32_t o[kPackWords];
    const uint4* __restrict__ q = reinterpret_cast<const uint4*>(pslot + i * kPackWords);
#pragma unroll
    for (int w = 0; w < kPackWords / 4; ++w) {
        const uint4 v = q[w];
        o[4 * w] = v.x; o[4 * w + 1] = v.y; o[4 * w + 2] = v.z; o[4 * w + 3] = v.w;
    }
    PreIdxA<kPackGroups> p;
#pragma unroll
    for (int g = 0; g < kPackGroups; ++g)
#pragma unroll
        for (int t = 0; t < kGatherA; t += 2) {   // halves g % 2 of two lists' words
            const uint32_t a = o[3 * t + g / 2], b = o[3 * (t + 1) + g / 2];
            p.w[g][t >> 1] = (g & 1) ? (a >> 16) | (b & 0xffff0000u) : (a & 0xffffu) | (b << 16);
        }
    return p;
}

// The same pass over the force pass's tiles: the records of the tile and its
// halo (position, velocity, V0 (1 - D): 56 bytes) are staged in LDS once and
// the neighbour sums read them through the 16-bit local slots.  Same
// arithmetic in the same order as k_pass_a.
// Graded spacing (kVarH): the support radius follows (64 bytes).
constexpr int kLdsABytes = 56;
// kPacked: the first neighbours from the force pass's packed slots, not from the
// sliced list, which is then hardly read: where both passes run over the same
// tiles.
template <typename R, int DM, bool kFlow, bool kVarH, bool kPacked>
__device__ __forceinline__ void pass_a_staged(const DevState& s) {
    extern __shared__ __align__(16) unsigned char lds_a[];
    // G tiles per workgroup (two where a tile is not a whole number of waves),
    // each with an image of M slots of its own; thread tx of part `part`
    // takes particle tx of that part's tile
    const int M = s.lds_slots_a;
    const int T = s.tile_a;
    const int G = s.a_group;
    const int part = G > 1 ? (int)threadIdx.x / T : 0;
    const int tx = (int)threadIdx.x - part * T;
    const int64_t n_tiles = (s.n + T - 1) / T;
    const int32_t* cnt_a = s.run_count ? s.run_count + 3 : nullptr;
    if (work_tile<true>(s.tile_list_a, cnt_a, G, 0, n_tiles) < 0) return;   // (then no part has a tile)
    const int64_t tile = work_tile<true>(s.tile_list_a, cnt_a, G, part, n_tiles);
    const int64_t tl = tile < 0 ? 0 : tile;
    const size_t base = (size_t)part * M;
    const size_t GM = (size_t)G * M;
    double2* __restrict__ Lxy = reinterpret_cast<double2*>(lds_a) + base;
    double2* __restrict__ Lzw = reinterpret_cast<double2*>(lds_a) + GM + base;
    double2* __restrict__ Lvxy = reinterpret_cast<double2*>(lds_a) + 2 * GM + base;
    double* __restrict__ Lvz = reinterpret_cast<double*>(reinterpret_cast<double2*>(lds_a) + 3 * GM) + base;
    double* __restrict__ Lhs = reinterpret_cast<double*>(reinterpret_cast<double2*>(lds_a) + 3 * GM) + GM + base;
    const int64_t start = tl * T;
    const int32_t* __restrict__ hl = s.halo_a + tl * (int64_t)s.halo_cap_a;
    const D4* __restrict__ XV = s.XV;
    const D4* __restrict__ VW = s.VW;
    // Up to four slots per thread per round: index loads, record loads, LDS
    // stores (two memory latencies a round).  The first round's index loads
    // go out before the particle's own scalars, whose latency then overlaps
    // them; it needs no halo count (slots past the image hold n), which is
    // read after it.  Slots past the image, and past the particle count (last
    // tile), load the tile's first record and store nothing.
    constexpr int kU = 4;
    int m0 = tx;
    int64_t g[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) g[u] = slot_particle(m0 + u * T, T, s.halo_cap_a, start, s.n, hl);
    const int64_t i = start + tx;
    const bool in = tile >= 0 && i < s.n;
    const int64_t ii = in ? i : start;
    const int cnt = s.nnb[ii];
    const int64_t slice0 = s.slice_ptr[ii / kSlice];
    const int sp_lane = s.spec[ii];
    const uint16_t* __restrict__ lp = s.lcol_a + slice0 + (ii % kSlice);
    const auto idx = [&](int k) { return (int)lp[(int64_t)k * kSlice]; };
    constexpr int kPre = staged_a_pre_groups<R, kPacked>();
    const PreIdxA<kPre> pre = [&] {
        if constexpr (kPacked)
            return packed_indices_a(s.pslot, ii);
        else
            return pre_indices_a<kPre>(cnt, idx);
    }();
    // whether the specimen runs and (FP64: the mixed form has no registers to
    // spare for them) what the neighbour sums need of it: also loaded before
    // the staging
    constexpr bool kEarlyP = sizeof(R) == 8;
    const DevSpec& Pl = s.specs[sp_lane];
    const R inv_h_l = R(Pl.inv_h), grad_k_l = kVarH ? R(1) : R(Pl.grad_k);
    const AvPar<R> av_l = av_par<R>(Pl);
    const int32_t run_w = run_word(s, sp_lane);
    const auto stage = [&](int m0, const int64_t (&g)[kU]) {
        D4 x[kU], v[kU];
        double hv[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int64_t l = g[u] < s.n ? g[u] : start;
            x[u] = XV[l];
            v[u] = VW[l];
            if constexpr (kVarH) hv[u] = s.hs[l];
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const int m = m0 + u * T;
            if (g[u] < s.n) {
                Lxy[m] = double2{x[u].x, x[u].y};
                Lzw[m] = double2{x[u].z, v[u].w};
                Lvxy[m] = double2{v[u].x, v[u].y};
                Lvz[m] = v[u].z;
                if constexpr (kVarH) Lhs[m] = hv[u];
            }
        }
    };
    // (a part without a tile stages the first round of tile 0 into its own
    // image, which nothing reads: no branch holds the first round's loads back)
    stage(m0, g);
    const int tot = tile < 0 ? 0 : T + s.halo_cnt_a[tl];
    for (m0 += kU * T; m0 < tot; m0 += kU * T) {
#pragma unroll
        for (int u = 0; u < kU; ++u) g[u] = slot_particle(m0 + u * T, T, s.halo_cap_a, start, s.n, hl);
        stage(m0, g);
    }
    __syncthreads();
    if (!in || frozen_word(s, run_w)) return;
    const UpdIn<R> upd = load_upd_in<R>(s, i);
    for (;;) {
        const int sp = __builtin_amdgcn_readfirstlane(sp_lane);
        if (sp == sp_lane) {
            const DevSpec& P = s.specs[sp];
            const R inv_h = kEarlyP ? inv_h_l : R(P.inv_h);
            const R grad_k = kEarlyP ? grad_k_l : kVarH ? R(1) : R(P.grad_k);
            const AvPar<R> av = kEarlyP ? av_l : av_par<R>(P);
            const int t = tx;
            const double2 a = Lxy[t], b = Lzw[t], c = Lvxy[t];
            R M9[9], AV[3];
            gather_fdot<R, kFlow, kVarH, kPre>(
                D4{a.x, a.y, b.x, 0.0}, D4{c.x, c.y, Lvz[t], b.y}, cnt, inv_h, grad_k, idx,
                [&](int m) {
                    const double2 a = Lxy[m], b = Lzw[m], c = Lvxy[m];
                    return NbrA{a.x, a.y, b.x, c.x, c.y, Lvz[m], b.y, kVarH ? Lhs[m] : 0.0};
                },
                M9, av, AV, kVarH ? Lhs[t] : 0.0, &pre);
            pass_a_update<R, DM, kFlow>(s, i, sp, M9, b.y, AV, upd);
            break;
        }
    }
}

template <typename R, int DM, bool kFlow, bool kVarH = false>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(pass_a_waves_min<R, DM, kFlow>(), 8)))
k_pass_a_staged(DevState s, int /* displacement buffer: unused here */) {
    pass_a_staged<R, DM, kFlow, kVarH, false>(s);
}

// Mixed, with the packed slots: 36 bytes a particle less to read beside the force
// pass's 48, for twelve registers more.  From about 450k particles on, where the
// two passes' data no longer fit the caches that they share, that pays (Taylor bar
// 599k, tiles of 128: 67.5 us, so 62.8; plate 567k, a step 142.1, so 137.7); below
// it does not (bar 200k, 112: 27.0 and 27.3).
constexpr int64_t kPackedFrom = 450000;
static inline bool update_packed(const DevState& s) {
    return s.n >= kPackedFrom && s.lcol_a == s.lcol;
}
template <int DM>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(pass_a_waves_min<float, DM, false>(), 8)))
k_pass_a_packed(DevState s, int /* displacement buffer: unused here */) {
    pass_a_staged<float, DM, false, false, true>(s);
}

// Launch of one deformation pass: `block` threads per workgroup, or 0 for the
// pass staged over its tiles, a_group of them per workgroup.
template <typename R, int DM, bool kFlow, bool kVarH = false>
static void launch_update(const DevState& s, int parity, int block, hipStream_t st) {
    if (block == 0) {
        const int64_t tiles = (s.n + s.tile_a - 1) / s.tile_a;
        const unsigned groups = (unsigned)((tiles + s.a_group - 1) / s.a_group);
        const size_t lds = (size_t)s.a_group * s.lds_slots_a * staged_a_record_bytes(kVarH);
        const int threads = s.tile_a * s.a_group;
        if constexpr (sizeof(R) == 4 && !kFlow)
            if (update_packed(s)) {
                k_pass_a_packed<DM><<<groups, threads, lds, st>>>(s, parity);
                return;
            }
        k_pass_a_staged<R, DM, kFlow, kVarH><<<groups, threads, lds, st>>>(s, parity);
    } else {
        const unsigned grid = (unsigned)((s.n + block - 1) / block);
        k_pass_a<R, DM, kFlow, kVarH><<<grid, block, 0, st>>>(s, parity);
    }
}

// Deformation passes whose registers are full (at three waves per SIMD, 168):
// FP64 with the GTN model's loops, mixed with every flow law; compiled, as the
// pipelined force pass FP64 is (252 registers), in a source of their own.
template <typename R, int DM, bool kFlow>
constexpr bool registers_full() {
    return sizeof(R) == 8 ? DM == 3 : kFlow;
}
hipError_t launch_pipe_fp64(const DevState& s, int parity, hipStream_t st, size_t lds_bytes);
const void* pipe_fp64();
void launch_update_full(const DevState& s, int parity, int block, int model, bool mixed,
                        hipStream_t st);

}  // namespace tlsph
