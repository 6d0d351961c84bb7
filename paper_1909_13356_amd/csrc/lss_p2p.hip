// Pair kernels of liblss (gfx950): the direct sum of the smoothed-indicator
// kernel over quadrature nodes (section 4.3, eq. discrete_int; kernel
// section 4.1, eq. kerpsi; exact gradient of the discrete sum).
//
// Per pair, with d = x - y, x = |d|^2 s2 (s2 = 1/(2 sigma^2)) and the folded
// dipole vector a' = c(sigma) w J:
//     Phi      -= (a'.d) S(x)
//     grad Phi += 2 s2 (a'.d) T(x) d - a' S(x)
// S(x) = gamma(3/2,x)/x^1.5, T(x) = gamma(5/2,x)/x^2.5 come from the rational
// fits of kfit_tables.h below the cut x = X (8 sigma in FP64, 6.32 sigma in
// FP32) and from the Laplace dipole S = (sqrt(pi)/2) x^-1.5, T = 1.5 S/x
// beyond it (section 4.4: the kernel equals the double-layer kernel there to
// the tail bound of the cut).
//
// Mixed path: the FP64 differences to a tile origin are carried as float-float
// (hi + lo) so that d keeps FP32 relative accuracy at any distance from it.
//
// Layout: one target per lane, TILE targets per workgroup (targets sorted by
// mesh, then Morton order); quadrature nodes are streamed through LDS in
// chunks of TILE packed records; each lane sums the nodes of its own mesh
// (per-lane node range, so a tile may straddle meshes of a ragged batch).
// Chunk partial sums are folded into compensated totals (two-sum).
#include <algorithm>
#include <cstring>
#include <hip/hip_runtime.h>

#include "fmm_math.h"
#include "kfit_tables.h"
#include "lss_internal.h"
#include "radial_exact.h"

namespace lss {

namespace {

// FP64 node record as staged in LDS: the far-form constants folded in as in
// SrcF (a' times sqrt(pi)/2, 2 s2 times 1.5)
__device__ __forceinline__ Src fold_src(Src f) {
    f.ax *= kFoldA;
    f.ay *= kFoldA;
    f.az *= kFoldA;
    f.fold = kFoldT * (2.0 * f.s2);
    return f;
}

// Padding records (chunks are filled to whole node groups): zero dipole
// vector, placed so far away that every target sees them beyond the cut
// (the dipole branch, whose terms underflow to zero), so they neither
// contribute nor pull a node group into the near-branch evaluation.
__device__ __forceinline__ Src pad_src() {
    Src f;
    f.yx = f.yy = f.yz = 1.0e150;
    f.ax = f.ay = f.az = f.fold = 0.0;
    f.s2 = 1.0;
    return f;
}

__device__ __forceinline__ SrcF pad_srcf() {
    SrcF f;
    f.yx = f.yy = f.yz = 1.0e18f;
    f.lx = f.ly = f.lz = 0.0f;
    f.ax = f.ay = f.az = f.s2x2 = 0.0f;
    f.s2 = 1.0f;
    f.pad = 0.0f;
    return f;
}

__device__ __forceinline__ void two_sum(double &s, double &e, double v) {
    double t = s + v;
    double bp = t - s;
    e += (s - (t - bp)) + (v - bp);
    s = t;
}

__device__ __forceinline__ void two_sum_f(float &s, float &e, float v) {
    float t = s + v;
    float bp = t - s;
    e += (s - (t - bp)) + (v - bp);
    s = t;
}

// S / (sqrt(pi)/2) and T / (1.5 sqrt(pi)/2) in FP64, for folded records (fold_src)
__device__ __forceinline__ void kfun64(double x, double &S, double &T) {
    if (x < KF64_X) {
        // power basis with shared powers t^k (t = x / X in [0, 1)): the
        // coefficients are the multiplicands, which the per-pair kernels keep
        // as scalar operands; Horner's addends are hoisted into vector
        // registers there, costing a wave per SIMD.  The coefficients are of
        // one sign but for a few small ones, so the sums stay well conditioned.
        const double t = x * KF64_INV_X;
        double ps = kf64_ps[0], pt = kf64_pt[0], q = kf64_q[0], tk = 1.0;
#pragma unroll
        for (int k = 1; k <= KF64_Q_DEG; ++k) {
            tk *= t;
            ps = fma(kf64_ps[k], tk, ps);
            pt = fma(kf64_pt[k], tk, pt);
            q = fma(kf64_q[k], tk, q);
        }
        double r = __builtin_amdgcn_rcp(q);
        const double er = fma(-q, r, 1.0);      // third-order correction of 1/q
        r = fma(r, fma(er, er, er), r);
        S = ps * r;
        T = pt * r;
    } else {
        const double r = rsq64(x);
        const double r2 = r * r;
        S = r2 * r;
        T = S * r2;
    }
}

// S / (sqrt(pi)/2) and T / (1.5 sqrt(pi)/2) in FP32, for SrcF records
__device__ __forceinline__ void kfun32(float x, float &S, float &T) {
    if (x < (float)KF32_X) {
        const float t = x * (float)KF32_INV_X;
        float ps = kf32_ps[KF32_PS_DEG], pt = kf32_pt[KF32_PT_DEG], q = kf32_q[KF32_Q_DEG];
#pragma unroll
        for (int k = KF32_Q_DEG - 1; k >= 0; --k) {
            ps = fmaf(ps, t, kf32_ps[k]);
            pt = fmaf(pt, t, kf32_pt[k]);
            q = fmaf(q, t, kf32_q[k]);
        }
        const float r = __builtin_amdgcn_rcpf(q);
        S = ps * r;
        T = pt * r;
    } else {
        const float r = __builtin_amdgcn_rsqf(x);
        const float r2 = r * r;
        S = r2 * r;
        T = S * r2;
    }
}

__device__ __forceinline__ void pair64(const Src &s, double x, double y, double z, double &p, double &gx,
                                       double &gy, double &gz) {
    const double dx = x - s.yx, dy = y - s.yy, dz = z - s.yz;
    const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
    const double ad = fma(s.ax, dx, fma(s.ay, dy, s.az * dz));
    double S, T;
    kfun64(r2 * s.s2, S, T);
    p = fma(-ad, S, p);
    const double g = ad * T * s.fold;
    gx = fma(g, dx, fma(-s.ax, S, gx));
    gy = fma(g, dy, fma(-s.ay, S, gy));
    gz = fma(g, dz, fma(-s.az, S, gz));
}

// K consecutive FP64 records against one target (see nodes32 below); with
// COUNT the pairs inside the cut are added to *cnt.  Neither form's argument
// is clamped to its side of the cut: the form of the other side is not
// selected, whatever it came out as (1 to 3 instructions of 33 to 75 a pair;
// 1.7e7 pairs of a small direct sum 466 -> 454 us).
template <int K, bool COUNT = false>
__device__ __forceinline__ void nodes64(const Src *sh, double x, double y, double z, double &p, double &gx,
                                        double &gy, double &gz, uint32_t *cnt = nullptr) {
    double dx[K], dy[K], dz[K], u[K], ad[K], S[K], T[K];
    double umin = 1.0e300;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const Src s = sh[k];
        dx[k] = x - s.yx;
        dy[k] = y - s.yy;
        dz[k] = z - s.yz;
        const double r2 = fma(dx[k], dx[k], fma(dy[k], dy[k], dz[k] * dz[k]));
        ad[k] = fma(s.ax, dx[k], fma(s.ay, dy[k], s.az * dz[k]));
        u[k] = r2 * s.s2;
        umin = fmin(umin, u[k]);
        const double r = rsq64(u[k]);       // inside the cut replaced below
        const double rr = r * r;
        S[k] = rr * r;                      // folded far form (see fold_src)
        T[k] = S[k] * rr;
    }
    if (umin < KF64_X) {                    // some pair of the group inside the cut
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double t = u[k] * KF64_INV_X;     // beyond the cut not selected
            double ps = kf64_ps[KF64_Q_DEG], pt = kf64_pt[KF64_Q_DEG], q = kf64_q[KF64_Q_DEG];
#pragma unroll
            for (int i = KF64_Q_DEG - 1; i >= 0; --i) {
                ps = fma(ps, t, kf64_ps[i]);
                pt = fma(pt, t, kf64_pt[i]);
                q = fma(q, t, kf64_q[i]);
            }
            double r = __builtin_amdgcn_rcp(q);
            const double er = fma(-q, r, 1.0);      // third-order correction of 1/q
            r = fma(r, fma(er, er, er), r);
            const bool nr = u[k] < KF64_X;
            S[k] = nr ? ps * r : S[k];
            T[k] = nr ? pt * r : T[k];
            if (COUNT) *cnt += nr ? 1u : 0u;
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const Src &s = sh[k];
        p = fma(-ad[k], S[k], p);
        const double g = ad[k] * T[k] * s.fold;
        gx = fma(g, dx[k], fma(-s.ax, S[k], gx));
        gy = fma(g, dy[k], fma(-s.ay, S[k], gy));
        gz = fma(g, dz[k], fma(-s.az, S[k], gz));
    }
}

constexpr int kNodeGroup64 = 4;

// FP64 record of a node beyond the cut of every target of a tile: position
// and a'' = (sqrt(pi)/2) a' s2^(-3/2)
struct alignas(16) FarD {
    double yx, yy, yz, ax, ay, az;
};

__device__ __forceinline__ FarD pad_fard() {
    FarD f;
    f.yx = f.yy = f.yz = 1.0e150;
    f.ax = f.ay = f.az = 0.0;
    return f;
}

// number of set bits of a wave mask below this lane
__device__ __forceinline__ int below(uint64_t m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// K consecutive FP64 far records against one target: the Laplace dipole with
// the width moved into a'' and the gradient summed in two parts, as
// nodes32_far; 1/sqrt refined to FP64 (rsq64)
template <int K>
__device__ __forceinline__ void nodes64_far(const FarD *sh, double x, double y, double z, double &p, double &gx,
                                            double &gy, double &gz, double &hx, double &hy, double &hz) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const FarD s = sh[k];
        const double dx = x - s.yx, dy = y - s.yy, dz = z - s.yz;
        const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
        const double r = rsq64(r2);
        const double rr = r * r, S = rr * r;
        const double ad = fma(s.ax, dx, fma(s.ay, dy, s.az * dz));
        p = fma(-ad, S, p);
        const double h = ad * S * rr;
        gx = fma(h, dx, gx);
        gy = fma(h, dy, gy);
        gz = fma(h, dz, gz);
        hx = fma(s.ax, S, hx);
        hy = fma(s.ay, S, hy);
        hz = fma(s.az, S, hz);
    }
}

// One FP64 far record against one target, the gradient accumulated whole
// (four accumulators instead of the seven of nodes64_far):
//   Phi -= (a''.d) S,  grad += 3 (a''.d) S |d|^-2 d - a'' S,  S = |d|^-3
__device__ __forceinline__ void pair_far64(const FarD &s, double x, double y, double z, double &p, double &gx,
                                           double &gy, double &gz) {
    const double dx = x - s.yx, dy = y - s.yy, dz = z - s.yz;
    const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
    const double r = rsq64(r2);
    const double rr = r * r, S = rr * r;
    const double ad = fma(s.ax, dx, fma(s.ay, dy, s.az * dz));
    p = fma(-ad, S, p);
    const double h = 3.0 * ad * S * rr;
    gx = fma(h, dx, fma(-s.ax, S, gx));
    gy = fma(h, dy, fma(-s.ay, S, gy));
    gz = fma(h, dz, fma(-s.az, S, gz));
}

constexpr int kNodeGroup = 4;

// The direct sum's records in LDS: groups of four nodes, component by
// component, so that every read is a full 16 bytes.  A 12-byte read
// (ds_read_b96) holds the LDS for 8.1 cycles, a 16-byte one for 4.4, and a
// SrcF read in three pieces has two of the former: 82 LDS cycles of a CU for
// four nodes and a wave, where the VALU needs 95; 48 as a group.  2.5e5
// targets x 242 000 nodes: 48.2 -> 46.6 ms, 1.3e12 pairs/s, now bound by VALU
// issue (1.5e12 at the clock it runs at).  (The octree
// kernels keep SrcF: there a node meets fewer targets, and writing eleven
// pieces costs what reading them saves.)
struct NearGroup {
    float __attribute__((ext_vector_type(4))) v[11];     // yx yy yz lx ly lz s2 ax ay az s2x2
};
__device__ __forceinline__ void put(NearGroup *sh, int i, const SrcF &f) {
    float *b = reinterpret_cast<float *>(sh + i / kNodeGroup) + i % kNodeGroup;
    const float c[11] = {f.yx, f.yy, f.yz, f.lx, f.ly, f.lz, f.s2, f.ax, f.ay, f.az, f.s2x2};
#pragma unroll
    for (int k = 0; k < 11; ++k) b[kNodeGroup * k] = c[k];
}
__device__ __forceinline__ SrcF record(const SrcF *sh, int k) { return sh[k]; }
__device__ __forceinline__ SrcF record(const NearGroup *sh, int k) {
    const NearGroup &g = sh[k / kNodeGroup];
    const int j = k % kNodeGroup;
    SrcF f;
    f.yx = g.v[0][j];
    f.yy = g.v[1][j];
    f.yz = g.v[2][j];
    f.lx = g.v[3][j];
    f.ly = g.v[4][j];
    f.lz = g.v[5][j];
    f.s2 = g.v[6][j];
    f.ax = g.v[7][j];
    f.ay = g.v[8][j];
    f.az = g.v[9][j];
    f.s2x2 = g.v[10][j];
    return f;
}

// K consecutive FP32 records against one target, as nodes64
template <int K, bool COUNT = false, class Rec>
__device__ __forceinline__ void nodes32(const Rec *sh, float x, float y, float z, float xl, float yl, float zl,
                                        float &p, float &gx, float &gy, float &gz, uint32_t *cnt = nullptr) {
    float dx[K], dy[K], dz[K], u[K], ad[K], S[K], T[K];
    float umin = 3.0e38f;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const SrcF s = record(sh, k);
        dx[k] = (x - s.yx) + (xl - s.lx);
        dy[k] = (y - s.yy) + (yl - s.ly);
        dz[k] = (z - s.yz) + (zl - s.lz);
        const float r2 = fmaf(dx[k], dx[k], fmaf(dy[k], dy[k], dz[k] * dz[k]));
        ad[k] = fmaf(s.ax, dx[k], fmaf(s.ay, dy[k], s.az * dz[k]));
        u[k] = r2 * s.s2;
        umin = fminf(umin, u[k]);
        const float r = __builtin_amdgcn_rsqf(u[k]);    // inside the cut replaced below
        const float rr = r * r;
        S[k] = rr * r;                      // folded far form (see SrcF)
        T[k] = S[k] * rr;
    }
    if (umin < (float)KF32_X) {             // some pair of the group inside the cut
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const float t = u[k] * (float)KF32_INV_X;       // beyond the cut not selected
            float ps = kf32_ps[KF32_PS_DEG], pt = kf32_pt[KF32_PT_DEG], q = kf32_q[KF32_Q_DEG];
#pragma unroll
            for (int i = KF32_Q_DEG - 1; i >= 0; --i) {
                ps = fmaf(ps, t, kf32_ps[i]);
                pt = fmaf(pt, t, kf32_pt[i]);
                q = fmaf(q, t, kf32_q[i]);
            }
            const float rq = __builtin_amdgcn_rcpf(q);
            const bool nr = u[k] < (float)KF32_X;
            S[k] = nr ? ps * rq : S[k];
            T[k] = nr ? pt * rq : T[k];
            if (COUNT) *cnt += nr ? 1u : 0u;
        }
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const SrcF s = record(sh, k);
        const float g = ad[k] * T[k] * s.s2x2;
        p = fmaf(-ad[k], S[k], p);
        gx = fmaf(g, dx[k], fmaf(-s.ax, S[k], gx));
        gy = fmaf(g, dy[k], fmaf(-s.ay, S[k], gy));
        gz = fmaf(g, dz[k], fmaf(-s.az, S[k], gz));
    }
}


// One (target, node) pair of a near list with the target's own width (see
// pair_ms), the node record's a' rescaled to a' s2^(-3/2) when staged (the
// caller multiplies the sums by s2x^(3/2) once): inside the cut and the FP64 fit's range the radial functions come
// from the fit (k1 = (sqrt(pi)/2) S, k2 = -(3 sqrt(pi)/2) s2x T) and exp(-t)
// from exp; inside the cut beyond that range from the exact forms (radial3);
// beyond the cut the kernel is the Laplace dipole, as in the far field
// (k1 = (sqrt(pi)/2) t^-3/2, k2 = -(3 sqrt(pi)/2) s2x t^-5/2, exp(-t) below
// the cut's truncation).
__device__ __forceinline__ void pair_ms_cut(const Src &s, double px, double py, double pz, double s2x, double tcut,
                                            MsAcc &A) {
    const double dx = px - s.yx, dy = py - s.yy, dz = pz - s.yz;
    const double t = (dx * dx + dy * dy + dz * dz) * s2x;
    double k1, k2, et = 0.0;
    if (t < tcut && t < KF64_X) {
        const double tt = t * KF64_INV_X;
        double ps = kf64_ps[0], pt = kf64_pt[0], q = kf64_q[0], tk = 1.0;     // power basis (see kfun64)
#pragma unroll
        for (int i = 1; i <= KF64_Q_DEG; ++i) {
            tk *= tt;
            ps = fma(kf64_ps[i], tk, ps);
            pt = fma(kf64_pt[i], tk, pt);
            q = fma(kf64_q[i], tk, q);
        }
        double r = __builtin_amdgcn_rcp(q);
        const double er = fma(-q, r, 1.0);      // third-order correction of 1/q
        r = fma(r, fma(er, er, er), r);
        k1 = (0.5 * kSqrtPi) * (ps * r);
        k2 = -(1.5 * kSqrtPi) * s2x * (pt * r);
        et = exp(-t);
    } else if (t < tcut) {
        double k3;
        radial3(t, s2x, k1, k2, k3, et);
    } else {
        const double iu = rsq64(t);
        const double iu3 = iu * iu * iu;
        k1 = (0.5 * kSqrtPi) * iu3;
        k2 = -(1.5 * kSqrtPi) * s2x * iu3 * iu * iu;
    }
    const double ad = s.ax * dx + s.ay * dy + s.az * dz;
    A.f += ad * k1;
    const double adk2 = ad * k2;
    A.gx += s.ax * k1 + adk2 * dx;
    A.gy += s.ay * k1 + adk2 * dy;
    A.gz += s.az * k1 + adk2 * dz;
    A.e += ad * et;
}

// pair_hess for the octree's near lists: inside the cut the three radial
// functions come from one rational fit (kf64h: fit error near FP64 rounding),
// beyond the cut (x >= tcut) they are those of the Laplace double layer, as in
// the far field: k1 = (sqrt(pi)/2) x^-3/2, k2 = -(3 sqrt(pi)/2) s2 x^-5/2,
// k3 = (15 sqrt(pi)/2) s2^2 x^-7/2.
static_assert(KF64H_PS_DEG == KF64H_Q_DEG && KF64H_PT_DEG == KF64H_Q_DEG && KF64H_PU_DEG == KF64H_Q_DEG,
              "pair_hess_cut evaluates the Hessian fit's numerators in one loop");
__device__ __forceinline__ void pair_hess_cut(const Src &s, double px, double py, double pz, double tcut,
                                              HessAcc &A) {
    const double dx = px - s.yx, dy = py - s.yy, dz = pz - s.yz;
    const double t = (dx * dx + dy * dy + dz * dz) * s.s2;
    double k1, k2, k3;
    if (t < tcut && t < KF64H_X) {
        // S, T, U from one rational fit (power basis, as kfun64):
        // k1 = S, k2 = -2 s2 T, k3 = 4 s2^2 U
        const double tt = t * KF64H_INV_X;
        double ps = kf64h_ps[0], pt = kf64h_pt[0], pu = kf64h_pu[0], q = kf64h_q[0], tk = 1.0;
#pragma unroll
        for (int i = 1; i <= KF64H_Q_DEG; ++i) {
            tk *= tt;
            ps = fma(kf64h_ps[i], tk, ps);
            pt = fma(kf64h_pt[i], tk, pt);
            pu = fma(kf64h_pu[i], tk, pu);
            q = fma(kf64h_q[i], tk, q);
        }
        double r = __builtin_amdgcn_rcp(q);
        const double er = fma(-q, r, 1.0);      // third-order correction of 1/q
        r = fma(r, fma(er, er, er), r);
        k1 = ps * r;
        k2 = -2.0 * s.s2 * (pt * r);
        k3 = 4.0 * s.s2 * s.s2 * (pu * r);
    } else if (t < tcut) {
        double et;
        radial3(t, s.s2, k1, k2, k3, et);
    } else {
        const double iu = rsq64(t);
        const double iu2 = iu * iu, iu3 = iu2 * iu, iu5 = iu3 * iu2;
        k1 = (0.5 * kSqrtPi) * iu3;
        k2 = -(1.5 * kSqrtPi) * s.s2 * iu5;
        k3 = (7.5 * kSqrtPi) * s.s2 * s.s2 * iu5 * iu2;
    }
    const double ad = s.ax * dx + s.ay * dy + s.az * dz;
    A.f -= ad * k1;
    const double adk2 = ad * k2, adk3 = ad * k3;
    A.gx -= s.ax * k1 + adk2 * dx;
    A.gy -= s.ay * k1 + adk2 * dy;
    A.gz -= s.az * k1 + adk2 * dz;
    const double ex = adk3 * dx, ey = adk3 * dy, ez = adk3 * dz;
    A.hxx -= 2.0 * k2 * s.ax * dx + adk2 + ex * dx;
    A.hyy -= 2.0 * k2 * s.ay * dy + adk2 + ey * dy;
    A.hzz -= 2.0 * k2 * s.az * dz + adk2 + ez * dz;
    A.hxy -= k2 * (s.ax * dy + s.ay * dx) + ex * dy;
    A.hxz -= k2 * (s.ax * dz + s.az * dx) + ex * dz;
    A.hyz -= k2 * (s.ay * dz + s.az * dy) + ey * dz;
}

// One (target, node) pair with the node beyond the cut of every target of the
// tile: pair_hess_cut's far form with the width folded into the record,
// a'' = (sqrt(pi)/2) a' s2^(-3/2) (FarD), S = |d|^-3, q = 3 S |d|^-2:
//   Phi -= (a''.d) S,  grad -= a'' S - q (a''.d) d,
//   Hess += q (a'' d^T + d a''^T) + q (a''.d) I - 5 q (a''.d) |d|^-2 d d^T
__device__ __forceinline__ void pair_hess_far(const FarD &s, double px, double py, double pz, HessAcc &A) {
    const double dx = px - s.yx, dy = py - s.yy, dz = pz - s.yz;
    const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
    const double ir = rsq64(r2);
    const double ir2 = ir * ir, S = ir2 * ir;
    const double ad = fma(s.ax, dx, fma(s.ay, dy, s.az * dz));
    A.f = fma(-ad, S, A.f);
    const double q = 3.0 * S * ir2;
    const double h = q * ad;
    A.gx = fma(h, dx, fma(-s.ax, S, A.gx));
    A.gy = fma(h, dy, fma(-s.ay, S, A.gy));
    A.gz = fma(h, dz, fma(-s.az, S, A.gz));
    const double e = 5.0 * h * ir2;
    const double ux = q * s.ax, uy = q * s.ay, uz = q * s.az;
    const double vx = e * dx, vy = e * dy, vz = e * dz;
    A.hxx = fma(fma(2.0, ux, -vx), dx, A.hxx + h);
    A.hyy = fma(fma(2.0, uy, -vy), dy, A.hyy + h);
    A.hzz = fma(fma(2.0, uz, -vz), dz, A.hzz + h);
    A.hxy = fma(ux - vx, dy, fma(uy, dx, A.hxy));
    A.hxz = fma(ux - vx, dz, fma(uz, dx, A.hxz));
    A.hyz = fma(uy - vy, dz, fma(uz, dy, A.hyz));
}

// FP32 record of a node that lies beyond the cut of every target of a tile:
// offset from the tile origin (no low part) and a'' = (sqrt(pi)/2) a' s2^(-3/2)
struct alignas(16) FarF {
    float yx, yy, yz, pad0;
    float ax, ay, az, pad1;
};

// Padding record of the far ring: zero vector, placed so far away that its
// terms underflow to zero.
__device__ __forceinline__ FarF pad_farf() {
    FarF f;
    f.yx = f.yy = f.yz = 1.0e18f;
    f.ax = f.ay = f.az = 0.0f;
    f.pad0 = f.pad1 = 0.0f;
    return f;
}

// K consecutive far records against one target: every node is beyond the cut
// of every target of the tile, so the kernel is the Laplace dipole.  With the
// width moved into a'' and r2 = |d|^2,
//   Phi -= (a''.d) r2^(-3/2),  grad Phi += 3 (a''.d) r2^(-5/2) d - a'' r2^(-3/2);
// the two gradient terms are summed apart (G += (a''.d) r2^(-5/2) d,
// H += a'' r2^(-3/2); the caller forms 3G - H once per run).  Positions are
// the FP32 offsets from the tile origin without the low parts: at |d| beyond
// the cut the rounding of the offsets is a relative error of a few units of
// FP32 rounding in d.
template <int K>
__device__ __forceinline__ void nodes32_far(const FarF *sh, float x, float y, float z, float &p, float &gx, float &gy,
                                            float &gz, float &hx, float &hy, float &hz) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const FarF s = sh[k];
        const float dx = x - s.yx, dy = y - s.yy, dz = z - s.yz;
        const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
        const float r = __builtin_amdgcn_rsqf(r2);
        const float rr = r * r, S = rr * r;
        const float ad = fmaf(s.ax, dx, fmaf(s.ay, dy, s.az * dz));
        p = fmaf(-ad, S, p);
        const float h = ad * S * rr;
        gx = fmaf(h, dx, gx);
        gy = fmaf(h, dy, gy);
        gz = fmaf(h, dz, gz);
        hx = fmaf(s.ax, S, hx);
        hy = fmaf(s.ay, S, hy);
        hz = fmaf(s.az, S, hz);
    }
}

__device__ __forceinline__ void pair32(const SrcF &s, float x, float y, float z, float xl, float yl, float zl,
                                       float &p, float &gx, float &gy, float &gz) {
    // d = (x_hi - y_hi) + (x_lo - y_lo): positions carried as float-float
    const float dx = (x - s.yx) + (xl - s.lx), dy = (y - s.yy) + (yl - s.ly), dz = (z - s.yz) + (zl - s.lz);
    const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
    const float ad = fmaf(s.ax, dx, fmaf(s.ay, dy, s.az * dz));
    float S, T;
    kfun32(r2 * s.s2, S, T);
    p = fmaf(-ad, S, p);
    const float g = ad * T * s.s2x2;
    gx = fmaf(g, dx, fmaf(-s.ax, S, gx));
    gy = fmaf(g, dy, fmaf(-s.ay, S, gy));
    gz = fmaf(g, dz, fmaf(-s.az, S, gz));
}

__device__ __forceinline__ double wave_sum(double v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// ------------------------------------------------- direct sum, split nodes
// A call with few targets has few tiles (16 for 4096 targets), so the tile's
// node range is cut into gridDim.y pieces of whole chunks of TILE nodes, one
// workgroup each.  A piece leaves its compensated sums (value and error term
// of Phi and the three gradient components) in part[piece][8][n], and
// k_direct_fold adds the pieces of a target in order by two-sum, so the sums
// do not depend on which workgroup ran first.  Chunks and runs are those of
// the unsplit loop: the pair arithmetic is the same bit for bit.  FP64, 4096
// targets on 36 864 nodes: 7.59 -> 0.45 ms a call (16 workgroups, each a
// serial chain of 144 chunks, before; 1152 of two chunks now).
template <int TILE>
__device__ __forceinline__ void split_range(int64_t &lo, int64_t &hi) {
    if (gridDim.y > 1) piece_range(TILE, blockIdx.y, gridDim.y, lo, hi);
}

template <class T>
__device__ __forceinline__ void store_part(T *part, int64_t n, int64_t i, T sp, T ep, T sx, T ex, T sy, T ey, T sz,
                                           T ez) {
    T *q = part + (int64_t)blockIdx.y * 8 * n + i;
    q[0] = sp;
    q[n] = ep;
    q[2 * n] = sx;
    q[3 * n] = ex;
    q[4 * n] = sy;
    q[5 * n] = ey;
    q[6 * n] = sz;
    q[7 * n] = ez;
}

// blockIdx.y: component (Phi, then the gradient), one target per lane
template <class T>
__global__ __launch_bounds__(64) void k_direct_fold(int64_t nmax, const int32_t *__restrict__ n_dev, int splits,
                                                    const T *__restrict__ part, const int32_t *__restrict__ out_idx,
                                                    double *__restrict__ phi, double *__restrict__ grad) {
    const int64_t n = n_dev ? (int64_t)*n_dev : nmax;
    const int64_t i = (int64_t)blockIdx.x * 64 + threadIdx.x;
    const int c = blockIdx.y;
    if (i >= n) return;
    const T *q = part + (int64_t)2 * c * nmax + i;
    double s = 0.0, e = 0.0;
#pragma unroll 4
    for (int k = 0; k < splits; ++k) {
        two_sum(s, e, (double)q[0]);
        e += (double)q[nmax];
        q += 8 * nmax;
    }
    const int64_t o = out_idx ? (int64_t)out_idx[i] : i;
    if (c == 0) phi[o] = s + e;
    else grad[3 * o + c - 1] = s + e;
}

// ---------------------------------------------------------------- FP64
template <int TILE>
__global__ __launch_bounds__(TILE) void k_p2p_direct_f64(
    int64_t nmax, const int32_t *__restrict__ n_dev, const double *__restrict__ tx,
    const double *__restrict__ ty, const double *__restrict__ tz, const int32_t *__restrict__ tmesh,
    const int64_t *__restrict__ node_off, const Src *__restrict__ src, const int32_t *__restrict__ out_idx,
    double *__restrict__ phi, double *__restrict__ grad, double *__restrict__ pairs, double *__restrict__ part) {
    __shared__ Src sh[TILE];
    const int64_t n = n_dev ? (int64_t)*n_dev : nmax;
    const int64_t t0 = (int64_t)blockIdx.x * TILE;
    if (t0 >= n) return;
    const int lane = threadIdx.x;
    const int64_t i = t0 + lane;
    const bool valid = i < n;
    const int64_t ii = valid ? i : n - 1;
    const double x = tx[ii], y = ty[ii], z = tz[ii];
    const int32_t m = tmesh[ii];
    const int64_t b = node_off[m], e = node_off[m + 1];
    // targets are sorted by mesh: the tile's node range runs from the first
    // target's mesh to the last target's mesh
    const int64_t tl = (t0 + TILE < n ? t0 + TILE : n) - 1;
    int64_t lo = node_off[tmesh[t0]], hi = node_off[tmesh[tl] + 1];
    split_range<TILE>(lo, hi);
    // a wave past the last target stages nodes and spends nothing on pairs
    const bool live = t0 + (lane & ~63) < n;

    double sp = 0, ep = 0, sx = 0, ex = 0, sy = 0, ey = 0, sz = 0, ez = 0;
    for (int64_t c0 = lo; c0 < hi; c0 += TILE) {
        const int cnt = (int)(hi - c0 < TILE ? hi - c0 : TILE);
        __syncthreads();
        if (lane < cnt) sh[lane] = fold_src(src[c0 + lane]);
        else sh[lane] = pad_src();              // pad the chunk to whole node groups
        __syncthreads();
        if (!live) continue;
        double p = 0, gx = 0, gy = 0, gz = 0;
        const bool full = c0 >= b && c0 + cnt <= e;
        if (__all(full)) {
            for (int j = 0; j < cnt; j += kNodeGroup64) nodes64<kNodeGroup64>(sh + j, x, y, z, p, gx, gy, gz);
        } else {
            const int jb = (int)(b - c0 > 0 ? (b - c0 < cnt ? b - c0 : cnt) : 0);
            const int je = (int)(e - c0 < cnt ? (e - c0 > 0 ? e - c0 : 0) : cnt);
            for (int j = jb; j < je; ++j) pair64(sh[j], x, y, z, p, gx, gy, gz);
        }
        two_sum(sp, ep, p);
        two_sum(sx, ex, gx);
        two_sum(sy, ey, gy);
        two_sum(sz, ez, gz);
    }
    if (part) {
        if (valid) store_part(part, nmax, i, sp, ep, sx, ex, sy, ey, sz, ez);
    } else if (valid) {
        const int64_t o = out_idx ? (int64_t)out_idx[i] : i;
        phi[o] = sp + ep;
        if (grad) {
            grad[3 * o] = sx + ex;
            grad[3 * o + 1] = sy + ey;
            grad[3 * o + 2] = sz + ez;
        }
    }
    if (pairs) {                            // [0] pairs of real targets, [1] lane slots spent
        const int64_t pb = b > lo ? b : lo, pe = e < hi ? e : hi;
        const double w = wave_sum(valid && pe > pb ? (double)(pe - pb) : 0.0);
        const double wl = wave_sum(live ? (double)(hi - lo) : 0.0);
        if ((lane & 63) == 0) { atomicAdd(pairs, w); atomicAdd(pairs + 1, wl); }
    }
}

// ---------------------------------------------------------------- mixed
template <int TILE>
__global__ __launch_bounds__(TILE) void k_p2p_direct_mixed(
    int64_t nmax, const int32_t *__restrict__ n_dev, const double *__restrict__ tx,
    const double *__restrict__ ty, const double *__restrict__ tz, const int32_t *__restrict__ tmesh,
    const int64_t *__restrict__ node_off, const Src *__restrict__ src, const int32_t *__restrict__ out_idx,
    double *__restrict__ phi, double *__restrict__ grad, double *__restrict__ pairs, float *__restrict__ part) {
    __shared__ NearGroup sh[TILE / kNodeGroup];
    const int64_t n = n_dev ? (int64_t)*n_dev : nmax;
    const int64_t t0 = (int64_t)blockIdx.x * TILE;
    if (t0 >= n) return;
    const int lane = threadIdx.x;
    const int64_t i = t0 + lane;
    const bool valid = i < n;
    const int64_t ii = valid ? i : n - 1;
    // tile origin: positions are differenced in FP64 against it, then rounded
    const double ox = tx[t0], oy = ty[t0], oz = tz[t0];
    const double dxo = tx[ii] - ox, dyo = ty[ii] - oy, dzo = tz[ii] - oz;
    const float x = (float)dxo, y = (float)dyo, z = (float)dzo;
    const float xl = (float)(dxo - (double)x), yl = (float)(dyo - (double)y), zl = (float)(dzo - (double)z);
    const int32_t m = tmesh[ii];
    const int64_t b = node_off[m], e = node_off[m + 1];
    const int64_t tl = (t0 + TILE < n ? t0 + TILE : n) - 1;
    int64_t lo = node_off[tmesh[t0]], hi = node_off[tmesh[tl] + 1];
    split_range<TILE>(lo, hi);
    // a wave past the last target stages nodes and spends nothing on pairs
    const bool live = t0 + (lane & ~63) < n;

    float sp = 0, ep = 0, sx = 0, ex = 0, sy = 0, ey = 0, sz = 0, ez = 0;
    for (int64_t c0 = lo; c0 < hi; c0 += TILE) {
        const int cnt = (int)(hi - c0 < TILE ? hi - c0 : TILE);
        __syncthreads();
        {
            SrcF f;
            if (lane < cnt) {
                const Src s = src[c0 + lane];
                const double qx = s.yx - ox, qy = s.yy - oy, qz = s.yz - oz;
                f.yx = (float)qx;
                f.yy = (float)qy;
                f.yz = (float)qz;
                f.lx = (float)(qx - (double)f.yx);
                f.ly = (float)(qy - (double)f.yy);
                f.lz = (float)(qz - (double)f.yz);
                f.s2 = (float)s.s2;
                f.ax = (float)(kFoldA * s.ax);
                f.ay = (float)(kFoldA * s.ay);
                f.az = (float)(kFoldA * s.az);
                f.s2x2 = (float)(kFoldT * (2.0 * s.s2));
            } else {
                f = pad_srcf();
            }
            put(sh, lane, f);
        }
        __syncthreads();
        if (!live) continue;
        const bool full = c0 >= b && c0 + cnt <= e;
        const int jb = full ? 0 : (int)(b - c0 > 0 ? (b - c0 < cnt ? b - c0 : cnt) : 0);
        const int je = full ? cnt : (int)(e - c0 < cnt ? (e - c0 > 0 ? e - c0 : 0) : cnt);
        const bool wave_full = __all(full);
        // FP32 partials over sub-chunks of 32 nodes, folded by two-sum
        for (int j0 = 0; j0 < cnt; j0 += 32) {
            float p = 0, gx = 0, gy = 0, gz = 0;
            const int j1 = j0 + 32 < cnt ? j0 + 32 : cnt;
            if (wave_full) {                // chunk padded with zero records to whole node groups
                for (int j = j0; j < j1; j += kNodeGroup) nodes32<kNodeGroup>(sh + j / kNodeGroup, x, y, z, xl, yl, zl, p, gx, gy, gz);
            } else {
                const int a0 = j0 > jb ? j0 : jb, a1 = j1 < je ? j1 : je;
                for (int j = a0; j < a1; ++j) pair32(record(sh, j), x, y, z, xl, yl, zl, p, gx, gy, gz);
            }
            two_sum_f(sp, ep, p);
            two_sum_f(sx, ex, gx);
            two_sum_f(sy, ey, gy);
            two_sum_f(sz, ez, gz);
        }
    }
    if (part) {
        if (valid) store_part(part, nmax, i, sp, ep, sx, ex, sy, ey, sz, ez);
    } else if (valid) {
        const int64_t o = out_idx ? (int64_t)out_idx[i] : i;
        phi[o] = (double)sp + (double)ep;
        if (grad) {
            grad[3 * o] = (double)sx + (double)ex;
            grad[3 * o + 1] = (double)sy + (double)ey;
            grad[3 * o + 2] = (double)sz + (double)ez;
        }
    }
    if (pairs) {                            // [0] pairs of real targets, [1] lane slots spent
        const int64_t pb = b > lo ? b : lo, pe = e < hi ? e : hi;
        const double w = wave_sum(valid && pe > pb ? (double)(pe - pb) : 0.0);
        const double wl = wave_sum(live ? (double)(hi - lo) : 0.0);
        if ((lane & 63) == 0) { atomicAdd(pairs, w); atomicAdd(pairs + 1, wl); }
    }
}


// ------------------------------------------------------------ FMM eval
// One tile = up to TILE targets of one octree leaf.  Near field: the full
// kernel over the node ranges of the leaf's direct list, streamed through
// LDS; far field: the leaf's local expansion (L2P with its gradient).  The
// grid is persistent: workgroups walk the tile list, whose length is read on
// the device.
struct FmmEvalArgs {
    const int32_t *ntiles_dev, *tile_start;
    int64_t n_max;
    const int32_t *n_dev;
    const int32_t *sleaf;       // leaf of each sorted target (nboxes + m: outside mesh m's root)
    // tiles [tile_start[k], tile_start[k+1]) (the last ends at the target count)
    // hold at most TILE targets of one leaf
    const int32_t *sidx;
    const double *tx, *ty, *tz;
    const int32_t *out_idx;
    double *phi, *grad;
    const int32_t *p2p_beg, *p2p_end, *p2p_src;
    const int64_t *nb, *ne;
    const int32_t *lev, *ijk;
    const Src *src;
    int64_t nnodes;
    int32_t nboxes;
    const double *L;
    const double *M;            // multipole expansions (for the M2P lists)
    const int32_t *m2p_beg, *m2p_end, *m2p_src;
    const int32_t *child, *parent;
    const double *rmax;         // largest cut radius of each box's nodes
    int K;                      // separation criterion of the M2P lists
    int p, ncp;
    double tcut;                // x = rho^2 s2 at the cut (beyond it the Hessian pairs take the dipole form)
    const double *root;         // per-mesh root cubes (corner xyz, side)
    const int32_t *bmesh;
    double *pairs;
    // tile queue: [0] next tile, [1] finished workgroups; for_tiles: [2] next
    // heavy tile, [3] finished workgroups; zero between launches (the last
    // workgroup to finish clears them)
    unsigned int *queue;
    const int32_t *order;       // queue position -> tile (most expensive first)
    // tiles at the front of the order that a whole workgroup takes (for_tiles),
    // and their part of the total cost in 1/1024
    const int32_t *nheavy;
};

// next tile for the workgroup (uniform); tiles are handed out in list order
__device__ __forceinline__ int next_tile(const FmmEvalArgs &a, int *slot) {
    __syncthreads();                    // everyone has read the previous slot value
    if (threadIdx.x == 0) *slot = (int)atomicAdd(a.queue, 1u);
    __syncthreads();
    return *slot;
}

__device__ __forceinline__ void queue_done(const FmmEvalArgs &a) {
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(a.queue + 1, 1u) == gridDim.x - 1) {
            atomicExch(a.queue, 0u);
            atomicExch(a.queue + 1, 0u);
        }
    }
}

// The near list of a tile (its leaf's source boxes) is streamed as one packed
// sequence: up to TILE ranges at a time are prefix-summed in LDS and each
// chunk of TILE nodes is filled across range boundaries, so no chunk is left
// partly empty at the end of a small box.
template <int TILE>
struct RangeBatch {
    int64_t beg[TILE];
    int64_t off[TILE + 1];
};

// load ranges [e, e + nr) of the leaf's direct list and prefix-sum their
// lengths; returns the packed length (uniform)
template <int TILE>
__device__ __forceinline__ int64_t load_ranges(const FmmEvalArgs &a, RangeBatch<TILE> &rb, int e, int nr) {
    const int t = threadIdx.x;
    int64_t len = 0;
    if (t < nr) {
        const int32_t S = a.p2p_src[e + t];
        rb.beg[t] = a.nb[S];
        len = a.ne[S] - a.nb[S];
    }
    rb.off[t + 1] = len;
    if (t == 0) rb.off[0] = 0;
    __syncthreads();
    for (int d = 1; d < TILE; d <<= 1) {      // inclusive scan of off[1..TILE]
        int64_t v = (t >= d) ? rb.off[t + 1 - d] : 0;
        __syncthreads();
        rb.off[t + 1] += v;
        __syncthreads();
    }
    return rb.off[nr];
}

// node index of packed position v (v < total)
template <int TILE>
__device__ __forceinline__ int64_t packed_node(const RangeBatch<TILE> &rb, int nr, int64_t v) {
    int lo = 0, hi = nr;                       // last r with off[r] <= v
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (rb.off[mid] <= v) lo = mid; else hi = mid;
    }
    return rb.beg[lo] + (v - rb.off[lo]);
}

// local expansion of leaf B staged in LDS by the whole workgroup (the caller
// synchronises before use)
__device__ __forceinline__ void stage_local(const FmmEvalArgs &a, int32_t B, double *Ls) {
    const double *src = a.L + (int64_t)B * a.ncp;
    for (int k = threadIdx.x; k < a.ncp; k += blockDim.x) Ls[k] = src[k];
}

// M2P and L2P by a wave, one target per lane: the sums of fmm::m2p and
// fmm::l2p before their scaling, term by term in their order (the same result bit for bit),
// with what is the same for every term of a column taken out of it.  The
// column's terms are split by the coefficients that they meet, so that a term
// has no branch (there were five to eight); T's and U's factors are counted up
// in FP64 (exact integers), or taken from a quotient per lane, instead of a
// conversion or a division per term; and a row's middle coefficient, which two
// terms meet, is read once.  An expansion of order 26 has 400 terms, and on a
// small tree a target meets as many terms as nodes: 24 ragged surfaces in mixed
// precision 44.5 -> 42.5 ms, charts of 3e4 triangles in FP64 46.1 -> 43.9, a step
// of 5e7 targets on 2e6 triangles 375 -> 368.
//   FUSED: every product goes straight into its column's sum (12 operations a
// term in the sums instead of 18, and the doubling of m > 0 taken out of them),
// and the columns' sums into the totals; for FP64 near fields.  A fused term
// rounds its sum twice: with one running sum over all columns the rms error of
// Phi was 4 to 10% above that of a rounding per term, with the columns apart it
// is 2 to 9% below (charts and steps of 1728 to 2e5 triangles, against the
// direct sum), at the same speed.  Mixed ones keep the order of roundings (see the top of
// lss_fmm.hip on M2L).  The coefficients are the wave's own, so they are read
// as scalars, where a read from LDS (8.7 cycles of it for two, three such a
// term) kept it as busy as the VALU: the two changes 2e6 targets on 2e5
// triangles 83.7 -> 81.9 ms, charts of 3e4 triangles 43.4 -> 43.1.
//   MM: 0, 1 or 2 for m = 0, m = 1, m >= 2
// coefficients of an expansion of one of the wave's boxes, read as scalars
using Coef = const double __attribute__((address_space(4))) *;
__device__ __forceinline__ Coef expansion(const double *all, int32_t box, int ncp) {
    return (Coef)(uint64_t)(all + (int64_t)__builtin_amdgcn_readfirstlane(box) * ncp);
}

struct ColumnSums {
    double s0, s1, are, aim;        // value, d/dz, and the two parts of dx + i dy
    fmm::cd t, t2;                  // T_j^m or U_j^m of this term and the one before
    double c, b;                    // 2 j - 1, (j - 1)^2 - m^2 of the next term
    double re, im;                  // middle coefficient of the row that the next term has met
};

// value += w Re(t m), and the pairs of the two parts: A += t m (sign +1), A -= conj(t m) (sign -1)
template <bool FUSED>
__device__ __forceinline__ void add_value(double &s, double w, const fmm::cd &t, double re, double im) {
    if (FUSED) {
        s = fma(t.re, re, s);
        s = fma(-t.im, im, s);
    } else {
        s += w * (t.re * re - t.im * im);
    }
}
template <bool FUSED, bool MINUS>
__device__ __forceinline__ void add_pair(ColumnSums &q, const fmm::cd &t, double re, double im) {
    if (FUSED) {
        q.are = fma(MINUS ? -t.re : t.re, re, q.are);
        q.are = fma(MINUS ? t.im : -t.im, im, q.are);
        q.aim = fma(t.re, im, q.aim);
        q.aim = fma(t.im, re, q.aim);
    } else {
        if (MINUS) q.are -= t.re * re - t.im * im;
        else q.are += t.re * re - t.im * im;
        q.aim += t.re * im + t.im * re;
    }
}

template <bool FUSED, int MM, bool REC, bool S0, bool S1, bool UP>
__device__ __forceinline__ void m2p_term(ColumnSums &q, Coef M, int j, int m, double w, double rz, double ir2) {
    if (REC) {
        const double a = q.c * rz;
        const fmm::cd tn = {(a * q.t.re - q.b * q.t2.re) * ir2, (a * q.t.im - q.b * q.t2.im) * ir2};
        q.t2 = q.t;
        q.t = tn;
        q.b += q.c;
        q.c += 2.0;
    }
    Coef rj = M + j * j, rn = M + (j - 1) * (j - 1);
    const fmm::cd t = q.t;
    double re = 0.0, im = 0.0;
    if (S0) {                                      // T_j^m M_j^m
        re = rj[MM ? 2 * m - 1 : 0];
        im = MM ? rj[2 * m] : 0.0;
        add_value<FUSED>(q.s0, w, t, re, im);
    }
    if (S1) add_value<FUSED>(q.s1, w, t, q.re, q.im);                                   // T_{n+1}^m M_n^m
    if (UP) add_pair<FUSED, false>(q, t, rn[2 * m + 1], rn[2 * m + 2]);                 // T_{n+1}^m M_n^{m+1}
    if (MM) add_pair<FUSED, true>(q, t, rn[MM == 1 ? 0 : 2 * m - 3], MM == 1 ? 0.0 : rn[2 * m - 2]);   // -conj(T_{n+1}^m M_n^{m-1})
    q.re = re;
    q.im = im;
}

template <bool FUSED, int MM>
__device__ __forceinline__ void m2p_column(ColumnSums &q, Coef M, int m, int p, double rz, double ir2) {
    const double w = MM == 0 ? 1.0 : 2.0;
    q.t2 = fmm::cd{0.0, 0.0};
    q.c = 2.0 * m + 1.0;
    q.b = 0.0;
    if (MM == 0) {                                 // j = 0 meets no row above
        q.re = M[0];
        q.im = 0.0;
        add_value<FUSED>(q.s0, w, q.t, q.re, q.im);
    } else if (m <= p) {
        m2p_term<FUSED, MM, false, true, false, false>(q, M, m, m, w, rz, ir2);
    } else {
        m2p_term<FUSED, MM, false, false, false, false>(q, M, m, m, w, rz, ir2);
        return;
    }
    if (m == p) {
        m2p_term<FUSED, MM, true, false, true, false>(q, M, p + 1, m, w, rz, ir2);
        return;
    }
    m2p_term<FUSED, MM, true, true, true, false>(q, M, m + 1, m, w, rz, ir2);
#pragma unroll 2
    for (int j = m + 2; j <= p; ++j) m2p_term<FUSED, MM, true, true, true, true>(q, M, j, m, w, rz, ir2);
    m2p_term<FUSED, MM, true, false, true, true>(q, M, p + 1, m, w, rz, ir2);
}

// FUSED: a column's sums into the totals (the values of m > 0 count twice), and cleared for the next
__device__ __forceinline__ void add_column(ColumnSums &q, int m, double s[4]) {
    const double w = m == 0 ? 1.0 : 2.0;
    s[0] = fma(w, q.s0, s[0]);
    s[1] += q.are;
    s[2] += q.aim;
    s[3] = fma(w, q.s1, s[3]);
    q.s0 = q.s1 = q.are = q.aim = 0.0;
}

template <bool FUSED>
__device__ __forceinline__ void wave_m2p_sums(Coef M, double rx, double ry, double rz, int p, double s[4]) {
    const double r2 = rx * rx + ry * ry + rz * rz, ir2 = 1.0 / r2;
    ColumnSums q;
    q.s0 = q.s1 = q.are = q.aim = 0.0;
    if (FUSED) s[0] = s[1] = s[2] = s[3] = 0.0;
    fmm::cd diag = {sqrt(ir2), 0.0};
    for (int m = 0; m <= p + 1; ++m) {
        if (m > 0) diag = fmm::cscale(fmm::cmul(diag, fmm::cd{rx, ry}), -(2.0 * m - 1.0) * ir2);
        q.t = diag;
        if (m == 0) m2p_column<FUSED, 0>(q, M, m, p, rz, ir2);
        else if (m == 1) m2p_column<FUSED, 1>(q, M, m, p, rz, ir2);
        else m2p_column<FUSED, 2>(q, M, m, p, rz, ir2);
        if (FUSED) add_column(q, m, s);
    }
    if (FUSED) return;
    s[0] = q.s0;
    s[1] = q.are;
    s[2] = q.aim;
    s[3] = q.s1;
}

template <bool FUSED, int MM, bool REC, bool LAST>
__device__ __forceinline__ void l2p_term(ColumnSums &q, Coef L, int j, int m, double w, double rz, double r2,
                                         double inv) {
    if (REC) {
        const double a = q.c * rz;
        const fmm::cd un = {(a * q.t.re - r2 * q.t2.re) * inv, (a * q.t.im - r2 * q.t2.im) * inv};
        q.t2 = q.t;
        q.t = un;
        q.c += 2.0;
    }
    const fmm::cd u = q.t;
    add_value<FUSED>(q.s0, w, u, q.re, q.im);
    if (LAST) return;
    Coef r = L + (j + 1) * (j + 1);
    q.re = r[MM ? 2 * m - 1 : 0];
    q.im = MM ? r[2 * m] : 0.0;
    add_value<FUSED>(q.s1, w, u, q.re, q.im);
    if (MM == 0) add_pair<FUSED, false>(q, u, -r[1], r[2]);                             // L_{j+1}^{-1} = -conj(L_{j+1}^1)
    else add_pair<FUSED, false>(q, u, r[MM == 1 ? 0 : 2 * m - 3], MM == 1 ? 0.0 : r[2 * m - 2]);   // L_{j+1}^{m-1}
    if (MM) add_pair<FUSED, true>(q, u, r[2 * m + 1], r[2 * m + 2]);                    // - conj(L_{j+1}^{m+1} U_j^m)
}

// lane i of v, the same for every lane
__device__ __forceinline__ double lane_value(double v, int i) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), i), __builtin_amdgcn_readlane(__double2loint(v), i));
}

template <bool FUSED, int MM>
__device__ __forceinline__ void l2p_column(ColumnSums &q, Coef L, int m, int p, double rz, double r2) {
    const double w = MM == 0 ? 1.0 : 2.0;
    const int jl = m + 1 + (threadIdx.x & 63);     // lane i: the quotient of term j = m + 1 + i
    const double invs = 1.0 / (double)((jl + m) * (jl - m));
    q.t2 = fmm::cd{0.0, 0.0};
    q.c = 2.0 * m + 1.0;
    q.re = L[MM ? m * m + 2 * m - 1 : 0];
    q.im = MM ? L[m * m + 2 * m] : 0.0;
    if (m == p) {
        l2p_term<FUSED, MM, false, true>(q, L, m, m, w, rz, r2, 0.0);
        return;
    }
    l2p_term<FUSED, MM, false, false>(q, L, m, m, w, rz, r2, 0.0);
#pragma unroll 2
    for (int j = m + 1; j < p; ++j) l2p_term<FUSED, MM, true, false>(q, L, j, m, w, rz, r2, lane_value(invs, j - m - 1));
    l2p_term<FUSED, MM, true, true>(q, L, p, m, w, rz, r2, lane_value(invs, p - m - 1));
}

template <bool FUSED>
__device__ __forceinline__ void wave_l2p_sums(Coef L, double rx, double ry, double rz, int p, double s[4]) {
    const double r2 = rx * rx + ry * ry + rz * rz;
    ColumnSums q;
    q.s0 = q.s1 = q.are = q.aim = 0.0;
    if (FUSED) s[0] = s[1] = s[2] = s[3] = 0.0;
    fmm::cd diag = {1.0, 0.0};
    for (int m = 0; m <= p; ++m) {
        if (m > 0) diag = fmm::cscale(fmm::cmul(diag, fmm::cd{rx, ry}), -0.5 / (double)m);
        q.t = diag;
        if (m == 0) l2p_column<FUSED, 0>(q, L, m, p, rz, r2);
        else if (m == 1) l2p_column<FUSED, 1>(q, L, m, p, rz, r2);
        else l2p_column<FUSED, 2>(q, L, m, p, rz, r2);
        if (FUSED) add_column(q, m, s);
    }
    if (FUSED) return;
    s[0] = q.s0;
    s[1] = q.are;
    s[2] = q.aim;
    s[3] = q.s1;
}

// as fmm::m2p and fmm::l2p
template <bool FUSED>
__device__ __forceinline__ void wave_m2p(Coef M, double rx, double ry, double rz, double inv_s, int p, double &phi,
                                         double g[3]) {
    double s[4];
    wave_m2p_sums<FUSED>(M, rx, ry, rz, p, s);
    const double is2 = inv_s * inv_s;
    phi = s[0] * inv_s;
    g[0] = -s[1] * is2;
    g[1] = s[2] * is2;
    g[2] = -s[3] * is2;
}
template <bool FUSED>
__device__ __forceinline__ void wave_l2p(Coef L, double rx, double ry, double rz, double inv_s, int p, double &phi,
                                         double g[3]) {
    double s[4];
    wave_l2p_sums<FUSED>(L, rx, ry, rz, p, s);
    phi = s[0];
    g[0] = s[1] * inv_s;
    g[1] = s[2] * inv_s;
    g[2] = s[3] * inv_s;
}

// WAVE: every lane of the wave takes part
template <bool WAVE = false>
__device__ __forceinline__ void fmm_l2p(const FmmEvalArgs &a, int32_t B, const double *Ls, double x, double y,
                                        double z, double &ph, double g[3]) {
    const double s = box_side(a.root, a.bmesh, B, a.lev[B]);
    const double *o = a.root + 4 * a.bmesh[B];
    const double cx = o[0] + (a.ijk[3 * B] + 0.5) * s, cy = o[1] + (a.ijk[3 * B + 1] + 0.5) * s,
                 cz = o[2] + (a.ijk[3 * B + 2] + 0.5) * s;
    const double inv = 1.0 / s;
    if (WAVE) wave_l2p<false>(expansion(a.L, B, a.ncp), (x - cx) * inv, (y - cy) * inv, (z - cz) * inv, inv, a.p, ph, g);
    else fmm::l2p(Ls, (x - cx) * inv, (y - cy) * inv, (z - cz) * inv, inv, a.p, ph, g);
}

// M2P list of leaf B at this lane's target: the multipole expansion of each
// listed box is staged in buf (ncp doubles) by the whole workgroup and
// evaluated at (x, y, z) (section 4.4: the far kernel is the Laplace double
// layer, so a box whose nodes are all beyond the cut of every target of B
// contributes through its expansion).  Uniform over the workgroup; buf is free
// again when it returns.
__device__ __forceinline__ void fmm_m2p_list(const FmmEvalArgs &a, int32_t B, double *buf, double x, double y,
                                             double z, double &ph, double g[3]) {
    const int e0 = a.m2p_beg[B], e1 = a.m2p_end[B];
    for (int e = e0; e < e1; ++e) {
        const int32_t S = a.m2p_src[e];
        __syncthreads();
        const double *src = a.M + (int64_t)S * a.ncp;
        for (int k = threadIdx.x; k < a.ncp; k += blockDim.x) buf[k] = src[k];
        __syncthreads();
        const double s = box_side(a.root, a.bmesh, S, a.lev[S]);
        const double *o = a.root + 4 * a.bmesh[S];
        const double cx = o[0] + (a.ijk[3 * S] + 0.5) * s, cy = o[1] + (a.ijk[3 * S + 1] + 0.5) * s,
                     cz = o[2] + (a.ijk[3 * S + 2] + 0.5) * s;
        const double inv = 1.0 / s;
        double p1, g1[3];
        fmm::m2p(buf, (x - cx) * inv, (y - cy) * inv, (z - cz) * inv, inv, a.p, p1, g1);
        ph += p1;
        g[0] += g1[0];
        g[1] += g1[1];
        g[2] += g1[2];
    }
    __syncthreads();
}

// Far field at a target outside its mesh's root cube (every node is then
// beyond the cut, the root cube being padded by twice the largest cut
// radius): one lane walks mesh m's tree depth first without a stack (the
// eight children of a box are consecutive, so the next box after a subtree is
// the next sibling of the first ancestor that is not an eighth child).  A box
// that passes the M2P test of the lists for this point is evaluated from its
// multipole expansion, a leaf that does not is summed directly, any other box
// is opened.  Returns the direct pairs spent.
__device__ __forceinline__ double fmm_outside(const FmmEvalArgs &a, int32_t m, double x, double y, double z, double &ph,
                              double g[3]) {
    double npair = 0.0, p = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
    int32_t b = m;                                  // level-0 box of mesh m
    while (b >= 0) {
        bool open = false;
        const int64_t n0 = a.nb[b], n1 = a.ne[b];
        if (n1 > n0) {
            const double s = box_side(a.root, a.bmesh, b, a.lev[b]);
            const double *o = a.root + 4 * a.bmesh[b];
            const double lo[3] = {o[0] + a.ijk[3 * b] * s, o[1] + a.ijk[3 * b + 1] * s, o[2] + a.ijk[3 * b + 2] * s};
            const double pt[3] = {x, y, z};
            double dc = 0.0, gap = 0.0;
            for (int d = 0; d < 3; ++d) {
                const double c = lo[d] + 0.5 * s, e = pt[d] - c;
                const double gd = fmax(fmax(lo[d] - pt[d], pt[d] - (lo[d] + s)), 0.0);
                dc += e * e;
                gap += gd * gd;
            }
            if (dc >= (double)a.K * s * s && gap >= a.rmax[b] * a.rmax[b]) {
                double p1, g1[3];
                const double inv = 1.0 / s;
                fmm::m2p(a.M + (int64_t)b * a.ncp, (x - lo[0]) * inv - 0.5, (y - lo[1]) * inv - 0.5,
                         (z - lo[2]) * inv - 0.5, inv, a.p, p1, g1);
                p += p1;
                gx += g1[0];
                gy += g1[1];
                gz += g1[2];
            } else if (a.child[b] < 0) {
                for (int64_t k = n0; k < n1; ++k) pair64(fold_src(a.src[k]), x, y, z, p, gx, gy, gz);
                npair += (double)(n1 - n0);
            } else {
                open = true;
            }
        }
        if (open) {
            b = a.child[b];
        } else {
            while (b != m && b == a.child[a.parent[b]] + 7) b = a.parent[b];
            b = b == m ? -1 : b + 1;
        }
    }
    ph = p;
    g[0] = gx;
    g[1] = gy;
    g[2] = gz;
    return npair;
}

// Targets outside their mesh's root cube (their tiles are skipped by the
// tile kernels): one thread per target over the sorted targets, both
// precisions in FP64.
__global__ __launch_bounds__(256) void k_eval_outside(FmmEvalArgs a) {
    const int64_t n = a.n_dev ? (int64_t)*a.n_dev : a.n_max;
    double npair = 0.0, lanes = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t B = a.sleaf[i];
        if (B < a.nboxes) continue;
        const int64_t ti = a.sidx ? (int64_t)a.sidx[i] : i;
        double ph, g[3];
        const double np = fmm_outside(a, B - a.nboxes, a.tx[ti], a.ty[ti], a.tz[ti], ph, g);
        npair += np;
        lanes += np;
        const int64_t o = a.out_idx ? (int64_t)a.out_idx[ti] : ti;
        a.phi[o] = ph;
        if (a.grad) {
            a.grad[3 * o] = g[0];
            a.grad[3 * o + 1] = g[1];
            a.grad[3 * o + 2] = g[2];
        }
    }
    if (a.pairs && npair > 0.0) {           // [0] pairs of real targets, [1] lane slots spent
        atomicAdd(a.pairs, npair);
        atomicAdd(a.pairs + 1, lanes);
    }
}

// ---------------------------------------------------------------- Hessian
// Phi, grad Phi and the Hessian through the same tree and lists (section
// 3.1 needs the Hessian for the charts' second derivatives): the near list
// with the full kernel and its third radial function inside the cut
// (pair_hess_cut: the double layer beyond it, as in the far field), the M2P
// list and the leaf's local expansion with their second derivatives
// (fmm::m2p_hess, fmm::l2p_hess).  Beyond the cut the kernel is the Laplace
// double layer to the truncation of the cut (8 sigma: P(7/2, 32) differs from
// 1 by 2e-11 relative, so the Hessian bar is looser than the field's).  FP64
// in either precision setting; the context's cut and order set the accuracy.
__device__ __forceinline__ void fmm_m2p_list_hess(const FmmEvalArgs &a, int32_t B, double *buf, double x, double y,
                                                  double z, double &ph, double g[3], double H[6]) {
    const int e0 = a.m2p_beg[B], e1 = a.m2p_end[B];
    for (int e = e0; e < e1; ++e) {
        const int32_t S = a.m2p_src[e];
        __syncthreads();
        const double *src = a.M + (int64_t)S * a.ncp;
        for (int k = threadIdx.x; k < a.ncp; k += blockDim.x) buf[k] = src[k];
        __syncthreads();
        const double s = box_side(a.root, a.bmesh, S, a.lev[S]);
        const double *o = a.root + 4 * a.bmesh[S];
        const double inv = 1.0 / s;
        const double rx = (x - (o[0] + (a.ijk[3 * S] + 0.5) * s)) * inv;
        const double ry = (y - (o[1] + (a.ijk[3 * S + 1] + 0.5) * s)) * inv;
        const double rz = (z - (o[2] + (a.ijk[3 * S + 2] + 0.5) * s)) * inv;
        double p1, g1[3], h1[6];
        fmm::m2p(buf, rx, ry, rz, inv, a.p, p1, g1);
        fmm::m2p_hess(buf, rx, ry, rz, inv, a.p, h1);
        ph += p1;
        for (int d = 0; d < 3; ++d) g[d] += g1[d];
        for (int d = 0; d < 6; ++d) H[d] += h1[d];
    }
    __syncthreads();
}

// one workgroup of TILE lanes per tile of more than 64 targets (the tiles of
// the evaluation, at most TILE targets of one leaf), tiles taken in a
// grid-stride loop (tiles of 64: k_hess_waves)
template <int TILE>
__global__ __launch_bounds__(TILE) __attribute__((amdgpu_waves_per_eu(3))) void k_hess_fmm(FmmEvalArgs a, double *hess) {
    __shared__ Src sh[TILE];
    __shared__ RangeBatch<TILE> rb;
    extern __shared__ double Ls[];      // local expansion of the tile's leaf (ncp doubles)
    const int ntiles = *a.ntiles_dev;
    const int64_t n = a.n_dev ? (int64_t)*a.n_dev : a.n_max;
    const int lane = threadIdx.x;
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int64_t s0 = a.tile_start[tile];
        const int32_t B = a.sleaf[s0];
        const int64_t s1 = tile + 1 < ntiles ? (int64_t)a.tile_start[tile + 1] : n;
        if (B >= a.nboxes) continue;        // outside the root cube: k_hess_outside
        const int64_t sp_ = s0 + lane;
        const bool valid = sp_ < s1;
        const int64_t ti = a.sidx ? (int64_t)a.sidx[valid ? sp_ : s0] : (valid ? sp_ : s0);
        const double x = a.tx[ti], y = a.ty[ti], z = a.tz[ti];
        const int e0 = a.p2p_beg[B], e1 = a.p2p_end[B];
        HessAcc A;
        for (int eb = e0; eb < e1; eb += TILE) {
            const int nr = e1 - eb < TILE ? e1 - eb : TILE;
            __syncthreads();
            const int64_t total = load_ranges<TILE>(a, rb, eb, nr);
            for (int64_t c0 = 0; c0 < total; c0 += TILE) {
                const int cnt = (int)(total - c0 < TILE ? total - c0 : TILE);
                __syncthreads();
                if (lane < cnt) sh[lane] = a.src[packed_node<TILE>(rb, nr, c0 + lane)];
                __syncthreads();
                for (int j = 0; j < cnt; ++j) pair_hess_cut(sh[j], x, y, z, a.tcut, A);
            }
        }
        double ph = 0.0, g[3] = {0.0, 0.0, 0.0}, H[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        fmm_m2p_list_hess(a, B, Ls, x, y, z, ph, g, H);
        stage_local(a, B, Ls);
        __syncthreads();
        {
            double lp, lg[3];                // fmm_l2p writes (does not add) its outputs
            fmm_l2p(a, B, Ls, x, y, z, lp, lg);
            ph += lp;
            for (int d = 0; d < 3; ++d) g[d] += lg[d];
        }
        {
            const double s = box_side(a.root, a.bmesh, B, a.lev[B]);
            const double *o = a.root + 4 * a.bmesh[B];
            const double inv = 1.0 / s;
            double h1[6];
            fmm::l2p_hess(Ls, (x - (o[0] + (a.ijk[3 * B] + 0.5) * s)) * inv,
                          (y - (o[1] + (a.ijk[3 * B + 1] + 0.5) * s)) * inv,
                          (z - (o[2] + (a.ijk[3 * B + 2] + 0.5) * s)) * inv, inv, a.p, h1);
            for (int d = 0; d < 6; ++d) H[d] += h1[d];
        }
        __syncthreads();                    // everyone is done with Ls before the next tile
        if (valid) {
            const int64_t o = a.out_idx ? (int64_t)a.out_idx[ti] : ti;
            if (a.phi) a.phi[o] = A.f + ph;
            if (a.grad) {
                a.grad[3 * o] = A.gx + g[0];
                a.grad[3 * o + 1] = A.gy + g[1];
                a.grad[3 * o + 2] = A.gz + g[2];
            }
            double *q = hess + 6 * o;
            q[0] = A.hxx + H[0];
            q[1] = A.hxy + H[1];
            q[2] = A.hxz + H[2];
            q[3] = A.hyy + H[3];
            q[4] = A.hyz + H[4];
            q[5] = A.hzz + H[5];
        }
    }
}

// targets outside their mesh's root cube: the direct sum over the mesh's
// nodes (the level-0 box m holds them all), one thread per target
__global__ __launch_bounds__(256) void k_hess_outside(FmmEvalArgs a, double *hess) {
    const int64_t n = a.n_dev ? (int64_t)*a.n_dev : a.n_max;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t B = a.sleaf[i];
        if (B < a.nboxes) continue;
        const int32_t m = B - a.nboxes;
        const int64_t ti = a.sidx ? (int64_t)a.sidx[i] : i;
        const double x = a.tx[ti], y = a.ty[ti], z = a.tz[ti];
        HessAcc A;
        for (int64_t k = a.nb[m]; k < a.ne[m]; ++k) pair_hess(a.src[k], x, y, z, A);
        const int64_t o = a.out_idx ? (int64_t)a.out_idx[ti] : ti;
        if (a.phi) a.phi[o] = A.f;
        if (a.grad) {
            a.grad[3 * o] = A.gx;
            a.grad[3 * o + 1] = A.gy;
            a.grad[3 * o + 2] = A.gz;
        }
        double *q = hess + 6 * o;
        q[0] = A.hxx;
        q[1] = A.hxy;
        q[2] = A.hxz;
        q[3] = A.hyy;
        q[4] = A.hyz;
        q[5] = A.hzz;
    }
}

// ------------------------------------------------ target-attached width
// Phi and grad Phi with sigma(x) (section 2, eq. basemodelk, sigma2) through
// a tree whose lists were built for these targets: a box is admissible when
// its gap clears cut * sigma(x) of every target in it, so every pair within
// the cut of sigma(x) is in a near list.  Near pairs use the target's width
// (pair_ms, which carries c(sigma(x)) a); the far field (Laplace double
// layer) does not depend on the width.  grad Phi gains (dPhi/dsigma) grad
// sigma, dPhi/dsigma = (2 c(x) / sigma(x)) sum (a.d) exp(-t) over the near
// pairs (beyond the cut exp(-t) is below the cut's truncation).  FP64.
__device__ __forceinline__ void ms_finish(double sx, const MsAcc &A, const double *gs, double &ph, double g[3]) {
    // Phi = -sum (c(x) a.d) k1, grad = -sum (c(x) a k1 + (c(x) a.d) k2 d),
    // dPhi/dsigma = (2 / sigma(x)) sum (c(x) a.d) e^-t
    const double dps = 2.0 * A.e / sx;
    ph -= A.f;
    g[0] += -A.gx + dps * gs[0];
    g[1] += -A.gy + dps * gs[1];
    g[2] += -A.gz + dps * gs[2];
}

template <int TILE>
__global__ __launch_bounds__(TILE) __attribute__((amdgpu_waves_per_eu(3))) void k_multiscale_fmm(FmmEvalArgs a, MsArgs ms) {
    __shared__ Src sh[TILE];
    __shared__ RangeBatch<TILE> rb;
    extern __shared__ double Ls[];
    const int ntiles = *a.ntiles_dev;
    const int64_t n = a.n_dev ? (int64_t)*a.n_dev : a.n_max;
    const int lane = threadIdx.x;
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int64_t s0 = a.tile_start[tile];
        const int32_t B = a.sleaf[s0];
        const int64_t s1 = tile + 1 < ntiles ? (int64_t)a.tile_start[tile + 1] : n;
        if (B >= a.nboxes) continue;        // outside the root cube: k_multiscale_outside
        const int64_t sp_ = s0 + lane;
        const bool valid = sp_ < s1;
        const int64_t ti = a.sidx ? (int64_t)a.sidx[valid ? sp_ : s0] : (valid ? sp_ : s0);
        const double x = a.tx[ti], y = a.ty[ti], z = a.tz[ti];
        const double sx = ms.sig[ti], s2x = 0.5 / (sx * sx);
        const int e0 = a.p2p_beg[B], e1 = a.p2p_end[B];
        MsAcc A;
        for (int eb = e0; eb < e1; eb += TILE) {
            const int nr = e1 - eb < TILE ? e1 - eb : TILE;
            __syncthreads();
            const int64_t total = load_ranges<TILE>(a, rb, eb, nr);
            for (int64_t c0 = 0; c0 < total; c0 += TILE) {
                const int cnt = (int)(total - c0 < TILE ? total - c0 : TILE);
                __syncthreads();
                if (lane < cnt) {           // a' s2^(-3/2): the width moves to the target (pair_ms_cut)
                    Src r = a.src[packed_node<TILE>(rb, nr, c0 + lane)];
                    const double f = 1.0 / (r.s2 * sqrt(r.s2));
                    r.ax *= f;
                    r.ay *= f;
                    r.az *= f;
                    sh[lane] = r;
                }
                __syncthreads();
                for (int j = 0; j < cnt; ++j) pair_ms_cut(sh[j], x, y, z, s2x, ms.tcut, A);
            }
        }
        {
            const double fx = s2x * sqrt(s2x);
            A.f *= fx;
            A.gx *= fx;
            A.gy *= fx;
            A.gz *= fx;
            A.e *= fx;
        }
        double ph = 0.0, g[3] = {0.0, 0.0, 0.0};
        if (a.m2p_end[B] > a.m2p_beg[B]) fmm_m2p_list(a, B, Ls, x, y, z, ph, g);
        stage_local(a, B, Ls);
        __syncthreads();
        {
            double lp, lg[3];
            fmm_l2p(a, B, Ls, x, y, z, lp, lg);
            ph += lp;
            for (int d = 0; d < 3; ++d) g[d] += lg[d];
        }
        __syncthreads();
        if (valid) {
            ms_finish(sx, A, ms.gsig + 3 * ti, ph, g);
            const int64_t o = a.out_idx ? (int64_t)a.out_idx[ti] : ti;
            a.phi[o] = ph;
            if (a.grad) {
                a.grad[3 * o] = g[0];
                a.grad[3 * o + 1] = g[1];
                a.grad[3 * o + 2] = g[2];
            }
        }
    }
}

// targets outside their mesh's root cube: every node of the mesh
__global__ __launch_bounds__(256) void k_multiscale_outside(FmmEvalArgs a, MsArgs ms) {
    const int64_t n = a.n_dev ? (int64_t)*a.n_dev : a.n_max;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t B = a.sleaf[i];
        if (B < a.nboxes) continue;
        const int32_t m = B - a.nboxes;
        const int64_t ti = a.sidx ? (int64_t)a.sidx[i] : i;
        const double x = a.tx[ti], y = a.ty[ti], z = a.tz[ti];
        const double sx = ms.sig[ti], s2x = 0.5 / (sx * sx);
        MsAcc A;
        for (int64_t k = a.nb[m]; k < a.ne[m]; ++k) pair_ms(a.src[k], x, y, z, s2x, A);
        double ph = 0.0, g[3] = {0.0, 0.0, 0.0};
        ms_finish(sx, A, ms.gsig + 3 * ti, ph, g);
        const int64_t o = a.out_idx ? (int64_t)a.out_idx[ti] : ti;
        a.phi[o] = ph;
        if (a.grad) {
            a.grad[3 * o] = g[0];
            a.grad[3 * o + 1] = g[1];
            a.grad[3 * o + 2] = g[2];
        }
    }
}

// Four waves per SIMD: the compiler fits the kernel in 128 VGPRs with a few
// spills outside the chunk loop (1% faster on C5 than three waves at 139).
// COUNT: also count the pairs inside the cut (pairs[2]), for the statistics
template <int TILE, bool COUNT>
__global__ __launch_bounds__(TILE) __attribute__((amdgpu_waves_per_eu(4))) void k_eval_fmm_f64(FmmEvalArgs a) {
    __shared__ Src sh[TILE];
    __shared__ RangeBatch<TILE> rb;
    extern __shared__ double Ls[];      // local expansion of the tile's leaf (ncp doubles)
    const int ntiles = *a.ntiles_dev;
    const int64_t n = a.n_dev ? (int64_t)*a.n_dev : a.n_max;
    const int lane = threadIdx.x;
    __shared__ int slot;
    // uniform over the grid: the queue is not touched (a launch without targets,
    // as the last iterations of a captured projection are, took 430 us)
    if (ntiles <= 0) return;
    for (int q = next_tile(a, &slot); q < ntiles; q = next_tile(a, &slot)) {
        const int tile = a.order[q];
        const int64_t s0 = a.tile_start[tile];
        const int32_t leafk = a.sleaf[s0];
        const int64_t s1 = tile + 1 < ntiles ? (int64_t)a.tile_start[tile + 1] : n;   // tile = [s0, s1)
        const int64_t sp_ = s0 + lane;
        const bool valid = sp_ < s1;
        const int64_t ti = a.sidx ? (int64_t)a.sidx[valid ? sp_ : s0] : (valid ? sp_ : s0);
        const double x = a.tx[ti], y = a.ty[ti], z = a.tz[ti];
        const int32_t B = leafk;
        if (B >= a.nboxes) continue;        // outside the root cube: k_eval_outside
        const int e0 = a.p2p_beg[B], e1 = a.p2p_end[B];
        __syncthreads();                    // previous tile is done with Ls
        stage_local(a, B, Ls);
        double sp = 0, ep = 0, sx = 0, ex = 0, sy = 0, ey = 0, sz = 0, ez = 0;
        double npair = 0.0;
        uint32_t nuse = 0;
        for (int eb = e0; eb < e1; eb += TILE) {
            const int nr = e1 - eb < TILE ? e1 - eb : TILE;
            __syncthreads();
            const int64_t total = load_ranges<TILE>(a, rb, eb, nr);
            npair += (double)total;
            for (int64_t c0 = 0; c0 < total; c0 += TILE) {
                const int cnt = (int)(total - c0 < TILE ? total - c0 : TILE);
                __syncthreads();
                if (lane < cnt) sh[lane] = fold_src(a.src[packed_node<TILE>(rb, nr, c0 + lane)]);
                else sh[lane] = pad_src();      // pad the chunk to whole node groups
                __syncthreads();
                double p = 0, gx = 0, gy = 0, gz = 0;
                for (int j = 0; j < cnt; j += kNodeGroup64)
                    nodes64<kNodeGroup64, COUNT>(sh + j, x, y, z, p, gx, gy, gz, &nuse);
                two_sum(sp, ep, p);
                two_sum(sx, ex, gx);
                two_sum(sy, ey, gy);
                two_sum(sz, ez, gz);
            }
        }
        double ph = 0.0, g[3] = {0.0, 0.0, 0.0}, mph = 0.0, mg[3] = {0.0, 0.0, 0.0};
        if (a.m2p_end[B] > a.m2p_beg[B]) {  // uniform: Ls is the M2P staging buffer, then L again
            fmm_m2p_list(a, B, Ls, x, y, z, mph, mg);
            stage_local(a, B, Ls);
        }
        __syncthreads();                    // Ls staged
        fmm_l2p(a, B, Ls, x, y, z, ph, g);
        ph += mph;
        g[0] += mg[0];
        g[1] += mg[1];
        g[2] += mg[2];
        if (valid) {
            const int64_t o = a.out_idx ? (int64_t)a.out_idx[ti] : ti;
            a.phi[o] = (sp + ph) + ep;
            if (a.grad) {
                a.grad[3 * o] = (sx + g[0]) + ex;
                a.grad[3 * o + 1] = (sy + g[1]) + ey;
                a.grad[3 * o + 2] = (sz + g[2]) + ez;
            }
        }
        if (a.pairs) {                      // [0] pairs of real targets, [1] lane slots spent, [2] inside the cut
            const double w = wave_sum(valid ? npair : 0.0), wl = wave_sum(npair);
            const double wu = COUNT ? wave_sum(valid ? (double)nuse : 0.0) : 0.0;
            if ((lane & 63) == 0) {
                atomicAdd(a.pairs, w);
                atomicAdd(a.pairs + 1, wl);
                if (COUNT) atomicAdd(a.pairs + 2, wu);
            }
        }
    }
    queue_done(a);
}


// ------------------------------------------------------- workgroups of waves
// The FP64 evaluation kernels run persistent workgroups of up to kWide waves.
// A workgroup takes heavy tiles (k_tile_bucket_scan) one by one: the waves
// share a tile's direct list chunk by chunk and its M2P boxes, each with
// staging and totals of its own, and add the totals in wave order at the end;
// there is no other barrier.  Light tiles go to single waves.  One wave alone on a SIMD issues about every fifth cycle that it
// could (FP64 latency), so a tile of many times the usual cost, on one wave,
// outlasts everything else: on 2e5 graded triangles a dozen of 40 000 tiles
// hold 1e5 to 4e5 nodes and hundreds of M2P boxes where a usual one has 1e4.
// FP64 evaluation, before with one wave per tile and after: 77 760 chart nodes
// 4.1 -> 1.8 ms, 4.7e5 chart nodes 26 -> 12.6, 2e6 targets on 2e5 triangles
// 117 -> 70; with what the records, ranges and expansions gained since, 1.6, 9.0
// and 61.

// LDS between lanes of one wave: orders the accesses, no barrier
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// up to 64 node ranges of a direct list, packed one after the other
struct RangeList {
    int64_t beg[64];
    int32_t off[65];
};

// ranges [e, e + nr), nr <= 64, of the direct list, by one wave; returns the
// packed length (64 boxes hold fewer than 2^31 nodes)
__device__ __forceinline__ int wave_ranges(const FmmEvalArgs &a, RangeList &rl, int e, int nr) {
    const int t = threadIdx.x & 63;
    int len = 0;
    wave_sync();                            // the previous batch is done with
    if (t < nr) {
        const int32_t S = a.p2p_src[e + t];
        rl.beg[t] = a.nb[S];
        len = (int)(a.ne[S] - a.nb[S]);
    }
    for (int d = 1; d < 64; d <<= 1) {
        const int v = __shfl_up(len, d);
        if (t >= d) len += v;
    }
    rl.off[t + 1] = len;
    if (t == 0) rl.off[0] = 0;
    wave_sync();
    return rl.off[nr];
}

// node index of packed position first + lane, for `width` positions from first on
// (uniform; all lanes take part, those past the list's end get no node).  The
// lanes look at one range each: the range of c0 is a count of the ranges that
// end before it, and the few ranges that begin among the positions are gone
// through one by one.  (A binary search per lane, six dependent LDS reads and
// thirty operations for 64 nodes, made octree evaluations 1% slower.)
__device__ __forceinline__ int64_t range_node(const RangeList &rl, int nr, int first, int width) {
    const int c0 = __builtin_amdgcn_readfirstlane(first);
    const int t = threadIdx.x & 63, v = c0 + t, bound = rl.off[t + 1];
    const int64_t base = rl.beg[t] - rl.off[t];
    auto base_of = [&](int q) {
        return (int64_t)((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(base >> 32), q) << 32 |
                         (uint32_t)__builtin_amdgcn_readlane((int)base, q));
    };
    int q = min(__popcll(__ballot(bound <= c0)), nr - 1);
    int64_t node = base_of(q) + v;
    for (int next = __builtin_amdgcn_readlane(bound, q); next < c0 + width && q + 1 < nr;
         next = __builtin_amdgcn_readlane(bound, q)) {
        ++q;
        if (v >= next) node = base_of(q) + v;
    }
    return node;
}

// bounding box of the wave's targets, lanes past the tile end holding its
// first (lo in box[0..2], hi in box[3..5])
__device__ __forceinline__ void wave_box(double x, double y, double z, double *box) {
    double lo[3] = {x, y, z}, hi[3] = {x, y, z};
    for (int off = 32; off > 0; off >>= 1)
        for (int c = 0; c < 3; ++c) {
            lo[c] = fmin(lo[c], __shfl_xor(lo[c], off));
            hi[c] = fmax(hi[c], __shfl_xor(hi[c], off));
        }
    wave_sync();
    if ((threadIdx.x & 63) == 0)
        for (int c = 0; c < 3; ++c) {
            box[c] = lo[c];
            box[3 + c] = hi[c];
        }
    wave_sync();
}

// squared distance of (x, y, z) from the box
__device__ __forceinline__ double box_gap2(const double *box, double x, double y, double z) {
    const double gx = fmax(fmax(box[0] - x, x - box[3]), 0.0);
    const double gy = fmax(fmax(box[1] - y, y - box[4]), 0.0);
    const double gz = fmax(fmax(box[2] - z, z - box[5]), 0.0);
    return gx * gx + gy * gy + gz * gz;
}

// scaled position of (x, y, z) in box S, and 1 / its side
__device__ __forceinline__ void box_position(const FmmEvalArgs &a, int32_t S, double x, double y, double z, double r[3],
                                             double &inv) {
    const double s = box_side(a.root, a.bmesh, S, a.lev[S]);
    const double *o = a.root + 4 * a.bmesh[S];
    inv = 1.0 / s;
    r[0] = (x - (o[0] + (a.ijk[3 * S] + 0.5) * s)) * inv;
    r[1] = (y - (o[1] + (a.ijk[3 * S + 1] + 0.5) * s)) * inv;
    r[2] = (z - (o[2] + (a.ijk[3 * S + 2] + 0.5) * s)) * inv;
}

// expansion of box S into the wave's buffer
__device__ __forceinline__ void wave_stage(const double *src, int ncp, double *buf) {
    wave_sync();
    for (int k = threadIdx.x & 63; k < ncp; k += 64) buf[k] = src[k];
    wave_sync();
}

// Tile loop of such a kernel: tile(t, W, w) for the heavy tiles with all the
// W waves of a workgroup (w: this wave), tile(t, 1, 0) wave by wave for the
// light ones.  The share of the workgroups that the heavy tiles' cost calls for
// starts with those, the others with the light tiles, which take a wave
// longest; each goes on with the other kind.  (Heavy tiles first everywhere:
// 2e5 targets on a uniform sphere, half of the tiles heavy, 7.8 ms against
// 5.0, mixed.)
// queue[2], queue[3]: next heavy tile, finished workgroups; queue[0]: next
// light tile; cleared by the last workgroup.  A launch without tiles returns
// at once (uniform over the grid).
template <class F>
__device__ __forceinline__ void for_tiles(const FmmEvalArgs &a, int *slot, F tile) {
    const int ntiles = *a.ntiles_dev, heavy = min(*a.nheavy, ntiles);
    if (ntiles <= 0) return;
    const int waves = (int)(blockDim.x >> 6), self = (int)(threadIdx.x >> 6);
    // one loop for both kinds: two copies of the tile code would compete for
    // the instruction cache while some workgroups are in either
    bool together = heavy > 0 && (int64_t)blockIdx.x * 1024 < (int64_t)a.nheavy[1] * gridDim.x;
    for (int left = heavy > 0 ? 2 : 1;;) {
        int q = 0;
        if (together) {
            __syncthreads();                // everyone has read the slot and left the totals
            if (threadIdx.x == 0) *slot = (int)atomicAdd(a.queue + 2, 1u);
            __syncthreads();
            q = *slot;
        } else {
            if ((threadIdx.x & 63) == 0) q = (int)atomicAdd(a.queue, 1u);
            q = heavy + __builtin_amdgcn_readfirstlane(q);
        }
        if (q >= (together ? heavy : ntiles)) {             // uniform: this kind is handed out
            if (--left == 0) break;
            together = !together;
            continue;
        }
        tile(a.order[q], together ? waves : 1, together ? self : 0);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(a.queue + 3, 1u) == gridDim.x - 1) {
            atomicExch(a.queue, 0u);
            atomicExch(a.queue + 2, 0u);
            atomicExch(a.queue + 3, 0u);
        }
    }
}

// Static LDS per wave of such a kernel, and the waves of a workgroup whose
// staging regions (rings, then an expansion where one is staged, then totals)
// fit 64 KiB
struct WaveLds {
    RangeList rl;
    double box[7];
};
inline int waves_for(size_t region) {
    const size_t n = (64 * 1024 - 64 - kWide * sizeof(WaveLds)) / region;
    return (int)(n < 1 ? 1 : (n > (size_t)kWide ? kWide : n));
}
inline size_t region_for(size_t rings, int ncp) {
    return (std::max(rings, sizeof(double) * (size_t)ncp) + 15) & ~(size_t)15;
}

// FP64 evaluation.  Every staged node is tested against the tile's target
// bounding box and goes to the near ring (the general loop: the far form for
// every pair, the rational fit for node groups with a pair inside the cut) or
// to the far ring (the dipole-only loop).  Nodes are staged 32 at a time, so
// that the two rings (7 KB) leave room for four waves per SIMD in a CU's LDS.
// Bound by FP64 VALU issue; four waves per SIMD (128 VGPRs, a few spills
// outside the pair loops).  COUNT: also count the pairs inside the cut
// (pairs[2]) and those of the dipole-only loop (pairs[3]), for the statistics.
constexpr int kNodeGroupSplit = 2;       // node group (fewer registers than 4)
constexpr int kRun64 = 32;               // records per partial sum
constexpr int kRing64 = 64;              // kRun64 - 1 left over + 32 staged

constexpr size_t kF64RingBytes = kRing64 * (sizeof(Src) + sizeof(FarD));

template <bool COUNT>
__global__ __launch_bounds__(64 * kWide) __attribute__((amdgpu_waves_per_eu(4))) void k_eval_fmm_f64_waves(FmmEvalArgs a,
                                                                                                      int region_doubles) {
    __shared__ WaveLds wl[kWide];
    __shared__ int slot;
    extern __shared__ __attribute__((aligned(16))) double Ls[];
    const int lane = threadIdx.x & 63, self = threadIdx.x >> 6;
    double *region = Ls + region_doubles * self, *box = wl[self].box;
    RangeList &rl = wl[self].rl;
    Src *ring_n = reinterpret_cast<Src *>(region);
    FarD *ring_f = reinterpret_cast<FarD *>(ring_n + kRing64);
    const int ntiles = *a.ntiles_dev;
    const int64_t n = a.n_dev ? (int64_t)*a.n_dev : a.n_max;
    const double far_u = KF64_X * (1.0 + 1e-6);
    for_tiles(a, &slot, [&](int tile, int W, int w) {
        const int64_t s0 = a.tile_start[tile];
        const int32_t B = a.sleaf[s0];
        if (B >= a.nboxes) return;          // outside the root cube: k_eval_outside
        const int64_t s1 = tile + 1 < ntiles ? (int64_t)a.tile_start[tile + 1] : n;   // tile = [s0, s1)
        const int64_t sp_ = s0 + lane;
        const bool valid = sp_ < s1;
        const int64_t ti = a.sidx ? (int64_t)a.sidx[valid ? sp_ : s0] : (valid ? sp_ : s0);
        const double x = a.tx[ti], y = a.ty[ti], z = a.tz[ti];
        wave_box(x, y, z, box);
        const int e1 = a.p2p_end[B];
        double sp = 0, ep = 0, sx = 0, ex = 0, sy = 0, ey = 0, sz = 0, ez = 0;
        double npair = 0.0, nfar = 0.0;
        uint32_t nuse = 0;
        int hn = 0, nn = 0, hf = 0, nf = 0;     // head and fill of the wave's rings (uniform)
        int eb = a.p2p_beg[B], nr = 0, total = 0, c0 = 0;
        for (bool last = false; !last;) {
            while (c0 >= total && eb < e1) {    // next batch of the leaf's direct list
                nr = e1 - eb < 64 ? e1 - eb : 64;
                total = wave_ranges(a, rl, eb, nr);
                npair += (double)total;
                c0 = w * kRun64;
                eb += nr;
            }
            last = c0 >= total;             // every node is staged: pad the remainders
            const int cnt = last ? 0 : (total - c0 < kRun64 ? total - c0 : kRun64);
            Src sr;
            bool isfar = false;
            const int64_t node = last ? 0 : range_node(rl, nr, c0, kRun64);
            if (lane < cnt) {
                sr = a.src[node];
                isfar = box_gap2(box, sr.yx, sr.yy, sr.yz) * sr.s2 >= far_u;
            }
            c0 += W * kRun64;
            const uint64_t fm = __ballot(isfar), nm = __ballot(lane < cnt && !isfar);
            wave_sync();                    // the runs taken last are read
            if (lane < cnt && !isfar) {
                int pos = hn + nn + below(nm);
                if (pos >= kRing64) pos -= kRing64;
                ring_n[pos] = fold_src(sr);
            } else if (isfar) {
                int pos = hf + nf + below(fm);
                if (pos >= kRing64) pos -= kRing64;
                const double fa = sr.fold;            // a'' (nodes64_far)
                FarD f;
                f.yx = sr.yx;
                f.yy = sr.yy;
                f.yz = sr.yz;
                f.ax = fa * sr.ax;
                f.ay = fa * sr.ay;
                f.az = fa * sr.az;
                ring_f[pos] = f;
            }
            nn += __popcll(nm);
            nf += __popcll(fm);
            if (COUNT) nfar += (double)__popcll(fm);
            // a full run of a ring, or at the end its remainder (< kRun64 records,
            // contiguous since the heads are multiples of kRun64) padded to whole
            // node groups
            const int ln = nn >= kRun64 ? kRun64 : (last ? (nn + kNodeGroupSplit - 1) / kNodeGroupSplit * kNodeGroupSplit : 0);
            const int lf = nf >= kRun64 ? kRun64 : (last ? (nf + kNodeGroupSplit - 1) / kNodeGroupSplit * kNodeGroupSplit : 0);
            if (last) {
                if (lane >= nn && lane < ln) ring_n[hn + lane] = pad_src();
                if (lane >= nf && lane < lf) ring_f[hf + lane] = pad_fard();
            }
            wave_sync();
            if (ln > 0) {
                double p = 0, gx = 0, gy = 0, gz = 0;
#pragma unroll 1
                for (int j = 0; j < ln; j += kNodeGroupSplit)
                    nodes64<kNodeGroupSplit, COUNT>(ring_n + hn + j, x, y, z, p, gx, gy, gz, &nuse);
                two_sum(sp, ep, p);
                two_sum(sx, ex, gx);
                two_sum(sy, ey, gy);
                two_sum(sz, ez, gz);
                hn = hn + kRun64 == kRing64 ? 0 : hn + kRun64;
                nn = nn > kRun64 ? nn - kRun64 : 0;
            }
            if (lf > 0) {
                double p = 0, gx = 0, gy = 0, gz = 0, hx = 0, hy = 0, hz = 0;
#pragma unroll 1
                for (int j = 0; j < lf; j += kNodeGroupSplit)
                    nodes64_far<kNodeGroupSplit>(ring_f + hf + j, x, y, z, p, gx, gy, gz, hx, hy, hz);
                gx = fma(3.0, gx, -hx);
                gy = fma(3.0, gy, -hy);
                gz = fma(3.0, gz, -hz);
                two_sum(sp, ep, p);
                two_sum(sx, ex, gx);
                two_sum(sy, ey, gy);
                two_sum(sz, ez, gz);
                hf = hf + kRun64 == kRing64 ? 0 : hf + kRun64;
                nf = nf > kRun64 ? nf - kRun64 : 0;
            }
        }
        // expansions: the wave's share of the M2P list, and for the last wave the
        // local expansion
        double ph = 0.0, g[3] = {0.0, 0.0, 0.0};
        const int m1 = a.m2p_end[B];
        for (int e = a.m2p_beg[B] + w; e < m1; e += W) {
            const int32_t S = a.m2p_src[e];
            double r[3], inv, p1, g1[3];
            box_position(a, S, x, y, z, r, inv);
            wave_m2p<true>(expansion(a.M, S, a.ncp), r[0], r[1], r[2], inv, a.p, p1, g1);
            ph += p1;
            for (int c = 0; c < 3; ++c) g[c] += g1[c];
        }
        if (w == W - 1) {
            double r[3], inv, p1, g1[3];
            box_position(a, B, x, y, z, r, inv);
            wave_l2p<true>(expansion(a.L, B, a.ncp), r[0], r[1], r[2], inv, a.p, p1, g1);
            ph += p1;
            for (int c = 0; c < 3; ++c) g[c] += g1[c];
        }
        if (W > 1) {                        // the waves' totals: sum, error term and far field of component c
            __syncthreads();                // every wave is done with its region
            const double ts[4] = {sp, sx, sy, sz}, te[4] = {ep, ex, ey, ez}, tf[4] = {ph, g[0], g[1], g[2]};
            for (int c = 0; c < 4; ++c) {
                double *t = Ls + (w * 4 + c) * 192 + lane;
                t[0] = ts[c];
                t[64] = te[c];
                t[128] = tf[c];
            }
            __syncthreads();
            for (int c = w; c < 4 && valid; c += W) {
                double s = 0.0, e = 0.0, f = 0.0;
                for (int v = 0; v < W; ++v) {
                    const double *t = Ls + (v * 4 + c) * 192 + lane;
                    two_sum(s, e, t[0]);
                    e += t[64];
                    f += t[128];
                }
                const int64_t o = a.out_idx ? (int64_t)a.out_idx[ti] : ti;
                const double v = (s + f) + e;
                if (c == 0) a.phi[o] = v;
                else if (a.grad) a.grad[3 * o + c - 1] = v;
            }
        } else if (valid) {
            const int64_t o = a.out_idx ? (int64_t)a.out_idx[ti] : ti;
            a.phi[o] = (sp + ph) + ep;
            if (a.grad) {
                a.grad[3 * o] = (sx + g[0]) + ex;
                a.grad[3 * o + 1] = (sy + g[1]) + ey;
                a.grad[3 * o + 2] = (sz + g[2]) + ez;
            }
        }
        if (a.pairs) {                      // [0] pairs of real targets, [1] lane slots spent, [2] inside the cut,
                                            // [3] taken by the dipole-only loop
            const double wu = COUNT ? wave_sum(valid ? (double)nuse : 0.0) : 0.0;
            const double wf = COUNT ? wave_sum(valid ? nfar : 0.0) : 0.0;
            if (lane == 0) {
                if (w == 0) {               // every wave counts the whole list
                    atomicAdd(a.pairs, (double)(s1 - s0) * npair);
                    atomicAdd(a.pairs + 1, 64.0 * npair);
                }
                if (COUNT) {
                    atomicAdd(a.pairs + 2, wu);
                    atomicAdd(a.pairs + 3, wf);
                }
            }
        }
    });
}

// The Hessian evaluation: as k_eval_fmm_f64_waves, heavy tiles by workgroups,
// light ones by waves; 64 nodes staged at a time, nodes beyond the cut of
// every target of the tile taking the folded far form (pair_hess_far), the
// others pair_hess_cut, which still chooses per pair.  Bound by FP64 VALU
// issue at three waves per SIMD (168 VGPRs).  2.9e5 chart nodes of 6348
// triangles: 30 -> 11 ms (one wave per tile in grid order before).
constexpr size_t kChunkBytes = 64 * (sizeof(Src) + sizeof(FarD));     // one staged chunk

__global__ __launch_bounds__(64 * kHessWaves) __attribute__((amdgpu_waves_per_eu(3))) void k_hess_waves(
    FmmEvalArgs a, double *hess, int region_doubles) {
    __shared__ WaveLds wl[kHessWaves];
    __shared__ int slot;
    extern __shared__ __attribute__((aligned(16))) double Ls[];
    const int lane = threadIdx.x & 63, self = threadIdx.x >> 6;
    double *region = Ls + region_doubles * self, *box = wl[self].box;
    RangeList &rl = wl[self].rl;
    Src *sh = reinterpret_cast<Src *>(region);
    FarD *shf = reinterpret_cast<FarD *>(sh + 64);
    const int ntiles = *a.ntiles_dev;
    const int64_t n = a.n_dev ? (int64_t)*a.n_dev : a.n_max;
    const double far_t = a.tcut * (1.0 + 1e-6);         // margin over the rounding of the box gap
    for_tiles(a, &slot, [&](int tile, int W, int w) {
        const int64_t s0 = a.tile_start[tile];
        const int32_t B = a.sleaf[s0];
        if (B >= a.nboxes) return;          // outside the root cube: k_hess_outside
        const int64_t s1 = tile + 1 < ntiles ? (int64_t)a.tile_start[tile + 1] : n;
        const int64_t sp_ = s0 + lane;
        const bool valid = sp_ < s1;
        const int64_t ti = a.sidx ? (int64_t)a.sidx[valid ? sp_ : s0] : (valid ? sp_ : s0);
        const double x = a.tx[ti], y = a.ty[ti], z = a.tz[ti];
        wave_box(x, y, z, box);
        HessAcc A;
        const int e1 = a.p2p_end[B];
        for (int eb = a.p2p_beg[B]; eb < e1; eb += 64) {
            const int nr = e1 - eb < 64 ? e1 - eb : 64;
            const int total = wave_ranges(a, rl, eb, nr);
            for (int c0 = 64 * w; c0 < total; c0 += 64 * W) {
                const int cnt = total - c0 < 64 ? total - c0 : 64;
                Src sr;
                bool isfar = false;
                const int64_t node = range_node(rl, nr, c0, 64);
                if (lane < cnt) {
                    sr = a.src[node];
                    isfar = box_gap2(box, sr.yx, sr.yy, sr.yz) * sr.s2 >= far_t;
                }
                const uint64_t fm = __ballot(isfar), nm = __ballot(lane < cnt && !isfar);
                wave_sync();                // the chunk taken last is read
                if (lane < cnt && !isfar) {
                    sh[below(nm)] = sr;
                } else if (isfar) {
                    const double fa = sr.fold;            // a''
                    FarD f;
                    f.yx = sr.yx;
                    f.yy = sr.yy;
                    f.yz = sr.yz;
                    f.ax = fa * sr.ax;
                    f.ay = fa * sr.ay;
                    f.az = fa * sr.az;
                    shf[below(fm)] = f;
                }
                wave_sync();
                const int nn = __popcll(nm), nf = __popcll(fm);
                for (int j = 0; j < nn; ++j) pair_hess_cut(sh[j], x, y, z, a.tcut, A);
                for (int j = 0; j < nf; ++j) pair_hess_far(shf[j], x, y, z, A);
            }
        }
        // expansions, one at a time in the wave's region
        const int m1 = a.m2p_end[B];
        for (int e = a.m2p_beg[B] + w; e < m1 + (w == W - 1 ? W : 0); e += W) {
            const bool local = e >= m1;     // once, for the last wave: the leaf's local expansion
            const int32_t S = local ? B : a.m2p_src[e];
            wave_stage((local ? a.L : a.M) + (int64_t)S * a.ncp, a.ncp, region);
            double r[3], inv, p1, g1[3], h1[6];
            box_position(a, S, x, y, z, r, inv);
            if (local) {
                wave_l2p<true>(expansion(a.L, B, a.ncp), r[0], r[1], r[2], inv, a.p, p1, g1);
                fmm::l2p_hess(region, r[0], r[1], r[2], inv, a.p, h1);
            } else {
                wave_m2p<true>(expansion(a.M, S, a.ncp), r[0], r[1], r[2], inv, a.p, p1, g1);
                fmm::m2p_hess(region, r[0], r[1], r[2], inv, a.p, h1);
            }
            A.f += p1;
            A.gx += g1[0];
            A.gy += g1[1];
            A.gz += g1[2];
            A.hxx += h1[0];
            A.hxy += h1[1];
            A.hxz += h1[2];
            A.hyy += h1[3];
            A.hyz += h1[4];
            A.hzz += h1[5];
            if (local) break;
        }
        double v[10] = {A.f, A.gx, A.gy, A.gz, A.hxx, A.hxy, A.hxz, A.hyy, A.hyz, A.hzz};
        if (W > 1) {                        // the waves' totals, added in wave order by wave 0
            __syncthreads();                // every wave is done with its region
            for (int c = 0; c < 10; ++c) Ls[(w * 10 + c) * 64 + lane] = v[c];
            __syncthreads();
            if (w > 0) return;
            for (int c = 0; c < 10; ++c)
                for (int u = 1; u < W; ++u) v[c] += Ls[(u * 10 + c) * 64 + lane];
        }
        if (valid) {
            const int64_t o = a.out_idx ? (int64_t)a.out_idx[ti] : ti;
            if (a.phi) a.phi[o] = v[0];
            if (a.grad)
                for (int c = 0; c < 3; ++c) a.grad[3 * o + c] = v[1 + c];
            for (int c = 0; c < 6; ++c) hess[6 * o + c] = v[4 + c];
        }
    });
}

// The evaluation with target-attached widths, in the same form: nodes beyond
// the cut of every target of the tile (the gap to the tile's bounding box
// against the tile's largest sigma(x)) take the Laplace double layer, the
// others pair_ms_cut, which still chooses per pair.  1e5 targets on 43 200
// triangles: 19 -> 3.4 ms.
__global__ __launch_bounds__(64 * kHessWaves) __attribute__((amdgpu_waves_per_eu(3))) void k_multiscale_waves(
    FmmEvalArgs a, MsArgs ms, int region_doubles) {
    __shared__ WaveLds wl[kHessWaves];
    __shared__ int slot;
    extern __shared__ __attribute__((aligned(16))) double Ls[];
    const int lane = threadIdx.x & 63, self = threadIdx.x >> 6;
    double *region = Ls + region_doubles * self, *box = wl[self].box;
    RangeList &rl = wl[self].rl;
    Src *sh = reinterpret_cast<Src *>(region);
    FarD *shf = reinterpret_cast<FarD *>(sh + 64);
    const int ntiles = *a.ntiles_dev;
    const int64_t n = a.n_dev ? (int64_t)*a.n_dev : a.n_max;
    const double far_t = ms.tcut * (1.0 + 1e-6);        // margin over the rounding of the box gap
    for_tiles(a, &slot, [&](int tile, int W, int w) {
        const int64_t s0 = a.tile_start[tile];
        const int32_t B = a.sleaf[s0];
        if (B >= a.nboxes) return;          // outside the root cube: k_multiscale_outside
        const int64_t s1 = tile + 1 < ntiles ? (int64_t)a.tile_start[tile + 1] : n;
        const int64_t sp_ = s0 + lane;
        const bool valid = sp_ < s1;
        const int64_t ti = a.sidx ? (int64_t)a.sidx[valid ? sp_ : s0] : (valid ? sp_ : s0);
        const double x = a.tx[ti], y = a.ty[ti], z = a.tz[ti];
        const double sx = ms.sig[ti], s2x = 0.5 / (sx * sx);
        wave_box(x, y, z, box);
        double s2min = s2x;                 // smallest s2(x): the tile's largest cut
        for (int off = 32; off > 0; off >>= 1) s2min = fmin(s2min, __shfl_xor(s2min, off));
        MsAcc A;
        double pf = 0.0, gfx = 0.0, gfy = 0.0, gfz = 0.0;  // the far nodes' double layer
        const int e1 = a.p2p_end[B];
        for (int eb = a.p2p_beg[B]; eb < e1; eb += 64) {
            const int nr = e1 - eb < 64 ? e1 - eb : 64;
            const int total = wave_ranges(a, rl, eb, nr);
            for (int c0 = 64 * w; c0 < total; c0 += 64 * W) {
                const int cnt = total - c0 < 64 ? total - c0 : 64;
                Src r;
                bool isfar = false;
                const int64_t node = range_node(rl, nr, c0, 64);
                if (lane < cnt) {
                    r = a.src[node];
                    isfar = box_gap2(box, r.yx, r.yy, r.yz) * s2min >= far_t;
                }
                const uint64_t fm = __ballot(isfar), nm = __ballot(lane < cnt && !isfar);
                wave_sync();                // the chunk taken last is read
                if (lane < cnt) {           // a' s2^(-3/2): the width moves to the target
                    const double f = 1.0 / (r.s2 * sqrt(r.s2));
                    if (!isfar) {
                        r.ax *= f;
                        r.ay *= f;
                        r.az *= f;
                        sh[below(nm)] = r;
                    } else {                // a'' = (sqrt(pi)/2) a' s2^(-3/2)
                        FarD q;
                        q.yx = r.yx;
                        q.yy = r.yy;
                        q.yz = r.yz;
                        q.ax = kFoldA * f * r.ax;
                        q.ay = kFoldA * f * r.ay;
                        q.az = kFoldA * f * r.az;
                        shf[below(fm)] = q;
                    }
                }
                wave_sync();
                const int nn = __popcll(nm), nf = __popcll(fm);
                for (int j = 0; j < nn; ++j) pair_ms_cut(sh[j], x, y, z, s2x, ms.tcut, A);
                for (int j = 0; j < nf; ++j) pair_far64(shf[j], x, y, z, pf, gfx, gfy, gfz);
            }
        }
        {
            const double fx = s2x * sqrt(s2x);
            A.f *= fx;
            A.gx *= fx;
            A.gy *= fx;
            A.gz *= fx;
            A.e *= fx;
        }
        double ph = 0.0, g[3] = {0.0, 0.0, 0.0};
        const int m1 = a.m2p_end[B];
        for (int e = a.m2p_beg[B] + w; e < m1 + (w == W - 1 ? W : 0); e += W) {
            const bool local = e >= m1;     // once, for the last wave: the leaf's local expansion
            const int32_t S = local ? B : a.m2p_src[e];
            double r[3], inv, p1, g1[3];
            box_position(a, S, x, y, z, r, inv);
            if (local) wave_l2p<true>(expansion(a.L, B, a.ncp), r[0], r[1], r[2], inv, a.p, p1, g1);
            else wave_m2p<true>(expansion(a.M, S, a.ncp), r[0], r[1], r[2], inv, a.p, p1, g1);
            ph += p1;
            for (int c = 0; c < 3; ++c) g[c] += g1[c];
            if (local) break;
        }
        // linear in the wave's sums: each wave finishes its own
        ms_finish(sx, A, ms.gsig + 3 * ti, ph, g);
        double v[4] = {ph + pf, g[0] + gfx, g[1] + gfy, g[2] + gfz};
        if (W > 1) {                        // the waves' totals, added in wave order by wave 0
            __syncthreads();                // every wave is done with its region
            for (int c = 0; c < 4; ++c) Ls[(w * 4 + c) * 64 + lane] = v[c];
            __syncthreads();
            if (w > 0) return;
            for (int c = 0; c < 4; ++c)
                for (int u = 1; u < W; ++u) v[c] += Ls[(u * 4 + c) * 64 + lane];
        }
        if (valid) {
            const int64_t o = a.out_idx ? (int64_t)a.out_idx[ti] : ti;
            a.phi[o] = v[0];
            if (a.grad)
                for (int c = 0; c < 3; ++c) a.grad[3 * o + c] = v[1 + c];
        }
    });
}

// Mixed path, in the tile loop of for_tiles.  Each staged node is tested
// against the tile's target bounding box: a node whose distance to the box is
// beyond its cut radius (u >= KF32_X for every target of the tile) goes to the
// far ring and the dipole-only loop, every other node to the near ring and the
// general loop (float-float offsets, the rational fit for node groups with a
// pair inside the cut).  Each ring is drained in runs of kRun records, one
// compensated partial sum per run; the remainders are padded to whole node
// groups at the end of the tile.  The expansions follow once the pairs
// are done.
//   One wave (light tiles): stages 64 nodes at a time into rings of its own.
//   A workgroup (heavy tiles): the same results bit for bit, whichever way a
// tile is taken.  The waves stage kWide chunks of 64 nodes at a time into
// shared rings in list order, so a run holds the same nodes; each run is
// summed by one wave, and wave 0 folds the runs' sums in the order in which one
// wave would have completed them (chunk by chunk, near runs before far ones).
// The expansions go to the waves in turn and are added in list order.
// Bound by FP32 VALU issue at four waves per SIMD.  One wave per tile before:
// 1000 targets on 242 000 nodes 3.4 -> 0.75 ms; a graded surface of 31 212
// triangles with 1e4 to 2e5 targets 18.8 -> 3.5 ms, 8e5 targets 20.5 -> 6.5 ms;
// 5e7 targets on 2e6 triangles as before (345, now 302: records, ranges, expansions).
constexpr int kRun = 32;                 // records per partial sum
constexpr int kRing = 96;                // a wave's ring: kRun - 1 left over + 64 staged
constexpr int kRingW = 64 * kWide + 32;  // a workgroup's: kRun - 1 left over + kWide * 64 staged
constexpr int kRunsW = (64 * kWide + 62) / kRun + 1;    // runs of both rings completed at once
static_assert(kRing % kRun == 0 && kRingW % kRun == 0, "a run is contiguous in its ring");
constexpr size_t kMixedRingBytes = kRing * (sizeof(SrcF) + sizeof(FarF));
constexpr size_t kMixedWideBytes = kRingW * (sizeof(SrcF) + sizeof(FarF)) + kRunsW * 4 * 64 * sizeof(float);

// record of a node at offset (qx, qy, qz) from the tile origin, near and far
__device__ __forceinline__ SrcF mixed_near(const Src &sr, double qx, double qy, double qz) {
    SrcF f;
    f.yx = (float)qx;
    f.yy = (float)qy;
    f.yz = (float)qz;
    f.lx = (float)(qx - (double)f.yx);
    f.ly = (float)(qy - (double)f.yy);
    f.lz = (float)(qz - (double)f.yz);
    f.s2 = (float)sr.s2;
    f.ax = (float)(kFoldA * sr.ax);
    f.ay = (float)(kFoldA * sr.ay);
    f.az = (float)(kFoldA * sr.az);
    f.s2x2 = (float)(kFoldT * (2.0 * sr.s2));
    f.pad = 0.0f;
    return f;
}
__device__ __forceinline__ FarF mixed_far(const Src &sr, double qx, double qy, double qz) {
    const double fa = sr.fold;            // a'' (nodes32_far)
    FarF f;
    f.yx = (float)qx;
    f.yy = (float)qy;
    f.yz = (float)qz;
    f.ax = (float)(fa * sr.ax);
    f.ay = (float)(fa * sr.ay);
    f.az = (float)(fa * sr.az);
    f.pad0 = f.pad1 = 0.0f;
    return f;
}

template <bool COUNT>
__global__ __launch_bounds__(64 * kWide) __attribute__((amdgpu_waves_per_eu(4))) void k_eval_fmm_mixed_waves(FmmEvalArgs a,
                                                                                                        int region_doubles,
                                                                                                        int nexp) {
    __shared__ WaveLds wl[kWide];
    __shared__ int cnts[2][2][kWide], slot;         // heavy tiles: near and far nodes per chunk, of this step and the last
    __shared__ double scale[kWide];                 // and 1 / side of the boxes of the expansions
    extern __shared__ __attribute__((aligned(16))) double Ls[];
    const int lane = threadIdx.x & 63, self = threadIdx.x >> 6;
    const int ntiles = *a.ntiles_dev;
    const int64_t n = a.n_dev ? (int64_t)*a.n_dev : a.n_max;
    const double far_u = (double)KF32_X * (1.0 + 1e-4);     // margin over the FP32 rounding of u
    for_tiles(a, &slot, [&](int tile, int W, int w) {
        const int64_t s0 = a.tile_start[tile];
        const int32_t B = a.sleaf[s0];
        if (B >= a.nboxes) return;          // outside the root cube: k_eval_outside
        const int64_t s1 = tile + 1 < ntiles ? (int64_t)a.tile_start[tile + 1] : n;   // tile = [s0, s1)
        const int nt = (int)(s1 - s0);
        const int64_t sp_ = s0 + lane;
        const bool valid = sp_ < s1;
        const int64_t ti = a.sidx ? (int64_t)a.sidx[valid ? sp_ : s0] : (valid ? sp_ : s0);
        const int64_t t0 = a.sidx ? (int64_t)a.sidx[s0] : s0;
        const double ox = a.tx[t0], oy = a.ty[t0], oz = a.tz[t0];     // tile origin
        const double dxo = a.tx[ti] - ox, dyo = a.ty[ti] - oy, dzo = a.tz[ti] - oz;
        const float x = (float)dxo, y = (float)dyo, z = (float)dzo;
        const float xl = (float)(dxo - (double)x), yl = (float)(dyo - (double)y), zl = (float)(dzo - (double)z);
        const int e0 = a.p2p_beg[B], e1 = a.p2p_end[B];
        // bounding box of the tile's targets (offsets from the origin), one
        // copy per wave; heavy tiles share wave 0's range list
        double *box = wl[self].box;
        wave_box(dxo, dyo, dzo, box);
        RangeList &rl = wl[W > 1 ? 0 : self].rl;
        SrcF *ring_n = reinterpret_cast<SrcF *>(W > 1 ? Ls : Ls + region_doubles * self);
        FarF *ring_f = reinterpret_cast<FarF *>(ring_n + (W > 1 ? kRingW : kRing));
        if (W == 1) {
            float sp = 0, ep = 0, sx = 0, ex = 0, sy = 0, ey = 0, sz = 0, ez = 0;
            double npair = 0.0, nfar = 0.0;
            uint32_t nuse = 0;
            int hn = 0, nn = 0, hf = 0, nf = 0;     // head and fill of each ring (uniform)
            for (int eb = e0; eb < e1; eb += 64) {
                const int nr = e1 - eb < 64 ? e1 - eb : 64;
                const int total = wave_ranges(a, rl, eb, nr);
                npair += (double)total;
                for (int c0 = 0; c0 < total; c0 += 64) {
                    const int cnt = total - c0 < 64 ? total - c0 : 64;
                    Src sr;
                    double qx = 0.0, qy = 0.0, qz = 0.0;
                    bool isfar = false;
                    const int64_t node = range_node(rl, nr, c0, 64);
                    if (lane < cnt) {
                        sr = a.src[node];
                        qx = sr.yx - ox;
                        qy = sr.yy - oy;
                        qz = sr.yz - oz;
                        isfar = box_gap2(box, qx, qy, qz) * sr.s2 >= far_u;
                    }
                    const uint64_t fm = __ballot(isfar), nm = __ballot(lane < cnt && !isfar);
                    wave_sync();                // the runs taken last are read
                    if (lane < cnt && !isfar) {
                        int pos = hn + nn + below(nm);
                        if (pos >= kRing) pos -= kRing;
                        ring_n[pos] = mixed_near(sr, qx, qy, qz);
                    } else if (isfar) {
                        int pos = hf + nf + below(fm);
                        if (pos >= kRing) pos -= kRing;
                        ring_f[pos] = mixed_far(sr, qx, qy, qz);
                    }
                    nn += __popcll(nm);
                    nf += __popcll(fm);
                    if (COUNT) nfar += (double)__popcll(fm);
                    wave_sync();
                    for (; nn >= kRun; nn -= kRun) {
                        float p = 0, gx = 0, gy = 0, gz = 0;
#pragma unroll 1
                        for (int j = 0; j < kRun; j += kNodeGroup)
                            nodes32<kNodeGroup, COUNT>(ring_n + hn + j, x, y, z, xl, yl, zl, p, gx, gy, gz, &nuse);
                        two_sum_f(sp, ep, p);
                        two_sum_f(sx, ex, gx);
                        two_sum_f(sy, ey, gy);
                        two_sum_f(sz, ez, gz);
                        hn = hn + kRun == kRing ? 0 : hn + kRun;
                    }
                    for (; nf >= kRun; nf -= kRun) {
                        float p = 0, gx = 0, gy = 0, gz = 0, hx = 0, hy = 0, hz = 0;
#pragma unroll 1
                        for (int j = 0; j < kRun; j += kNodeGroup)
                            nodes32_far<kNodeGroup>(ring_f + hf + j, x, y, z, p, gx, gy, gz, hx, hy, hz);
                        gx = fmaf(3.0f, gx, -hx);
                        gy = fmaf(3.0f, gy, -hy);
                        gz = fmaf(3.0f, gz, -hz);
                        two_sum_f(sp, ep, p);
                        two_sum_f(sx, ex, gx);
                        two_sum_f(sy, ey, gy);
                        two_sum_f(sz, ez, gz);
                        hf = hf + kRun == kRing ? 0 : hf + kRun;
                    }
                }
            }
            if (nn > 0 || nf > 0) {             // remainders (< kRun each), padded to whole node groups
                const int pn = (nn + kNodeGroup - 1) / kNodeGroup * kNodeGroup;
                const int pf = (nf + kNodeGroup - 1) / kNodeGroup * kNodeGroup;
                wave_sync();
                if (lane >= nn && lane < pn) ring_n[hn + lane] = pad_srcf();    // hn + kRun <= kRing
                if (lane >= nf && lane < pf) ring_f[hf + lane] = pad_farf();
                wave_sync();
                if (nn > 0) {
                    float p = 0, gx = 0, gy = 0, gz = 0;
                    for (int j = 0; j < pn; j += kNodeGroup)
                        nodes32<kNodeGroup, COUNT>(ring_n + hn + j, x, y, z, xl, yl, zl, p, gx, gy, gz, &nuse);
                    two_sum_f(sp, ep, p);
                    two_sum_f(sx, ex, gx);
                    two_sum_f(sy, ey, gy);
                    two_sum_f(sz, ez, gz);
                }
                if (nf > 0) {
                    float p = 0, gx = 0, gy = 0, gz = 0, hx = 0, hy = 0, hz = 0;
                    for (int j = 0; j < pf; j += kNodeGroup)
                        nodes32_far<kNodeGroup>(ring_f + hf + j, x, y, z, p, gx, gy, gz, hx, hy, hz);
                    gx = fmaf(3.0f, gx, -hx);
                    gy = fmaf(3.0f, gy, -hy);
                    gz = fmaf(3.0f, gz, -hz);
                    two_sum_f(sp, ep, p);
                    two_sum_f(sx, ex, gx);
                    two_sum_f(sy, ey, gy);
                    two_sum_f(sz, ez, gz);
                }
            }
            const double X = a.tx[ti], Y = a.ty[ti], Z = a.tz[ti];
            double ph = 0.0, g[3] = {0.0, 0.0, 0.0}, mph = 0.0, mg[3] = {0.0, 0.0, 0.0};
            for (int e = a.m2p_beg[B]; e < a.m2p_end[B]; ++e) {
                const int32_t S = a.m2p_src[e];
                double r[3], inv, p1, g1[3];
                box_position(a, S, X, Y, Z, r, inv);
                wave_m2p<false>(expansion(a.M, S, a.ncp), r[0], r[1], r[2], inv, a.p, p1, g1);
                mph += p1;
                for (int c = 0; c < 3; ++c) mg[c] += g1[c];
            }
            fmm_l2p<true>(a, B, nullptr, X, Y, Z, ph, g);
            ph += mph;
            g[0] += mg[0];
            g[1] += mg[1];
            g[2] += mg[2];
            if (valid) {
                const int64_t o = a.out_idx ? (int64_t)a.out_idx[ti] : ti;
                a.phi[o] = ((double)sp + (double)ep) + ph;
                if (a.grad) {
                    a.grad[3 * o] = ((double)sx + (double)ex) + g[0];
                    a.grad[3 * o + 1] = ((double)sy + (double)ey) + g[1];
                    a.grad[3 * o + 2] = ((double)sz + (double)ez) + g[2];
                }
            }
            if (a.pairs) {                      // [0] pairs of real targets, [1] lane slots spent, [2] inside the cut,
                                                // [3] taken by the dipole-only loop
                const double wu = COUNT ? wave_sum(valid ? (double)nuse : 0.0) : 0.0;
                if (lane == 0) {
                    atomicAdd(a.pairs, (double)nt * npair);
                    atomicAdd(a.pairs + 1, 64.0 * npair);
                    if (COUNT) {
                        atomicAdd(a.pairs + 2, wu);
                        atomicAdd(a.pairs + 3, (double)nt * nfar);
                    }
                }
            }
            return;
        }
        float *part = reinterpret_cast<float *>(ring_f + kRingW);       // [run][component][lane]
        float sp = 0, ep = 0, sx = 0, ex = 0, sy = 0, ey = 0, sz = 0, ez = 0;      // wave 0's totals
        double npair = 0.0, nfar = 0.0;
        uint32_t nuse = 0;
        int hn = 0, nn = 0, hf = 0, nf = 0;     // head and fill of each ring (uniform)
        int par = 0;
        // sums of a run of a ring into slot u
        auto run = [&](bool near, int at, int len, int u) {
            float p = 0, gx = 0, gy = 0, gz = 0;
            if (near) {
#pragma unroll 1
                for (int j = 0; j < len; j += kNodeGroup)
                    nodes32<kNodeGroup, COUNT>(ring_n + at + j, x, y, z, xl, yl, zl, p, gx, gy, gz, &nuse);
            } else {
                float hx = 0, hy = 0, hz = 0;
#pragma unroll 1
                for (int j = 0; j < len; j += kNodeGroup)
                    nodes32_far<kNodeGroup>(ring_f + at + j, x, y, z, p, gx, gy, gz, hx, hy, hz);
                gx = fmaf(3.0f, gx, -hx);
                gy = fmaf(3.0f, gy, -hy);
                gz = fmaf(3.0f, gz, -hz);
            }
            float *o = part + u * 256 + lane;
            o[0] = p;
            o[64] = gx;
            o[128] = gy;
            o[192] = gz;
        };
        auto fold = [&](int u) {
            const float *o = part + u * 256 + lane;
            two_sum_f(sp, ep, o[0]);
            two_sum_f(sx, ex, o[64]);
            two_sum_f(sy, ey, o[128]);
            two_sum_f(sz, ez, o[192]);
        };
        for (int eb = e0; eb < e1; eb += 64) {
            const int nr = e1 - eb < 64 ? e1 - eb : 64;
            __syncthreads();                // the previous batch is done with
            if (w == 0) wave_ranges(a, rl, eb, nr);
            __syncthreads();
            const int total = rl.off[nr];
            npair += (double)total;
            for (int c0 = 0; c0 < total; c0 += 64 * kWide) {
                const int c1 = c0 + 64 * w, cnt = min(max(total - c1, 0), 64);
                Src sr;
                double qx = 0.0, qy = 0.0, qz = 0.0;
                bool isfar = false;
                const int64_t node = range_node(rl, nr, c1, 64);
                if (lane < cnt) {
                    sr = a.src[node];
                    qx = sr.yx - ox;
                    qy = sr.yy - oy;
                    qz = sr.yz - oz;
                    isfar = box_gap2(box, qx, qy, qz) * sr.s2 >= far_u;
                }
                const uint64_t fm = __ballot(isfar), nm = __ballot(lane < cnt && !isfar);
                par ^= 1;                   // wave 0 may still fold with the last step's counts
                int *cntn = cnts[par][0], *cntf = cnts[par][1];
                if (lane == 0) {
                    cntn[w] = __popcll(nm);
                    cntf[w] = __popcll(fm);
                }
                __syncthreads();            // counts; the runs taken last are read and folded
                int bn = nn, bf = nf, tn = nn, tf = nf;
                for (int v = 0; v < kWide; ++v) {
                    if (v < w) {
                        bn += cntn[v];
                        bf += cntf[v];
                    }
                    tn += cntn[v];
                    tf += cntf[v];
                }
                if (lane < cnt && !isfar) {
                    int pos = hn + bn + below(nm);
                    if (pos >= kRingW) pos -= kRingW;
                    ring_n[pos] = mixed_near(sr, qx, qy, qz);
                } else if (isfar) {
                    int pos = hf + bf + below(fm);
                    if (pos >= kRingW) pos -= kRingW;
                    ring_f[pos] = mixed_far(sr, qx, qy, qz);
                }
                if (COUNT) nfar += (double)(tf - nf);
                __syncthreads();
                const int rn = tn / kRun, rf = tf / kRun;
                for (int u = w; u < rn + rf; u += kWide) {
                    int at = u < rn ? hn + u * kRun : hf + (u - rn) * kRun;
                    if (at >= kRingW) at -= kRingW;
                    run(u < rn, at, kRun, u);
                }
                __syncthreads();
                if (w == 0) {               // fold chunk by chunk
                    int kn = nn, kf = nf, dn = 0, df = 0;
                    for (int v = 0; v < kWide; ++v) {
                        kn += cntn[v];
                        kf += cntf[v];
                        for (; dn < kn / kRun; ++dn) fold(dn);
                        for (; df < kf / kRun; ++df) fold(rn + df);
                    }
                }
                hn += rn * kRun;
                if (hn >= kRingW) hn -= kRingW;
                hf += rf * kRun;
                if (hf >= kRingW) hf -= kRingW;
                nn = tn - rn * kRun;
                nf = tf - rf * kRun;
            }
        }
        if (nn > 0 || nf > 0) {             // remainders (< kRun each), padded to whole node groups
            const int pn = (nn + kNodeGroup - 1) / kNodeGroup * kNodeGroup;
            const int pf = (nf + kNodeGroup - 1) / kNodeGroup * kNodeGroup;
            __syncthreads();
            if (w == 0 && lane >= nn && lane < pn) ring_n[hn + lane] = pad_srcf();
            if (w == 1 && lane >= nf && lane < pf) ring_f[hf + lane] = pad_farf();
            __syncthreads();
            if (w == 0 && nn > 0) run(true, hn, pn, 0);
            if (w == 1 && nf > 0) run(false, hf, pf, 1);
            __syncthreads();
            if (w == 0) {
                if (nn > 0) fold(0);
                if (nf > 0) fold(1);
            }
        }
        // expansions: entry 0 the leaf's local one, then the M2P list, nexp at a
        // time, one per wave; wave 0 scales and adds them in list order, each
        // product and sum in one rounding as where one wave takes the tile (the
        // compiler contracts them there)
        const double X = a.tx[ti], Y = a.ty[ti], Z = a.tz[ti];
        double *res = Ls;                   // [wave][sum][lane]
        double lv[4] = {0.0, 0.0, 0.0, 0.0}, mv[4] = {0.0, 0.0, 0.0, 0.0}, linv = 0.0;
        const int m0 = a.m2p_beg[B], entries = 1 + a.m2p_end[B] - m0;
        for (int k0 = 0; k0 < entries; k0 += nexp) {
            const int k = k0 + w;
            __syncthreads();                // the rings, or the results folded last, are done with
            if (w < nexp && k < entries) {
                const int32_t S = k == 0 ? B : a.m2p_src[m0 + k - 1];
                double r[3], inv, sums[4];
                box_position(a, S, X, Y, Z, r, inv);
                if (k == 0) wave_l2p_sums<false>(expansion(a.L, B, a.ncp), r[0], r[1], r[2], a.p, sums);
                else wave_m2p_sums<false>(expansion(a.M, S, a.ncp), r[0], r[1], r[2], a.p, sums);
                for (int c = 0; c < 4; ++c) res[w * 256 + 64 * c + lane] = sums[c];
                if (lane == 0) scale[w] = inv;
            }
            __syncthreads();
            if (w == 0)
                for (int v = 0; v < nexp && k0 + v < entries; ++v) {
                    const double *e = res + v * 256 + lane;
                    const double inv = scale[v], is2 = inv * inv;
                    if (k0 + v == 0) {
                        for (int c = 0; c < 4; ++c) lv[c] = e[64 * c];
                        linv = inv;
                    } else {
                        mv[0] = fma(e[0], inv, mv[0]);
                        mv[1] = fma(-e[64], is2, mv[1]);
                        mv[2] = fma(e[128], is2, mv[2]);
                        mv[3] = fma(-e[192], is2, mv[3]);
                    }
                }
        }
        if (w == 0 && valid) {
            const int64_t o = a.out_idx ? (int64_t)a.out_idx[ti] : ti;
            a.phi[o] = ((double)sp + (double)ep) + (lv[0] + mv[0]);
            if (a.grad) {
                a.grad[3 * o] = ((double)sx + (double)ex) + fma(lv[1], linv, mv[1]);
                a.grad[3 * o + 1] = ((double)sy + (double)ey) + fma(lv[2], linv, mv[2]);
                a.grad[3 * o + 2] = ((double)sz + (double)ez) + fma(lv[3], linv, mv[3]);
            }
        }
        if (a.pairs) {                      // as above; the list counts once per tile
            const double wu = COUNT ? wave_sum(valid ? (double)nuse : 0.0) : 0.0;
            if (lane == 0) {
                if (w == 0) {
                    atomicAdd(a.pairs, (double)nt * npair);
                    atomicAdd(a.pairs + 1, 64.0 * npair);
                    if (COUNT) atomicAdd(a.pairs + 3, (double)nt * nfar);
                }
                if (COUNT) atomicAdd(a.pairs + 2, wu);
            }
        }
    });
}

// targets per workgroup of the direct sum
int direct_tile(const Ctx &c) { return c.opt.tile == 64 || c.opt.tile == 128 ? c.opt.tile : 256; }

template <int TILE>
void launch_tile(Ctx &c, int64_t n, const int32_t *n_dev, const double *tx, const double *ty, const double *tz,
                 const int32_t *tmesh, const int32_t *out_idx, double *phi, double *grad, double *pairs, void *part) {
    const int splits = part ? direct_splits(c, n) : 1;
    dim3 grid((unsigned)ceil_div(n, TILE), (unsigned)splits), block(TILE);
    if (splits == 1) part = nullptr;
    const dim3 fold((unsigned)ceil_div(n, 64), grad ? 4u : 1u);
    if (c.opt.precision == LSS_MIXED) {
        hipLaunchKernelGGL(k_p2p_direct_mixed<TILE>, grid, block, 0, c.stream, n, n_dev, tx, ty, tz, tmesh,
                           c.node_off.as<int64_t>(), c.src.as<Src>(), out_idx, phi, grad, pairs, (float *)part);
        if (part)
            hipLaunchKernelGGL(k_direct_fold<float>, fold, dim3(64), 0, c.stream, n, n_dev, splits, (float *)part,
                               out_idx, phi, grad);
    } else {
        hipLaunchKernelGGL(k_p2p_direct_f64<TILE>, grid, block, 0, c.stream, n, n_dev, tx, ty, tz, tmesh,
                           c.node_off.as<int64_t>(), c.src.as<Src>(), out_idx, phi, grad, pairs, (double *)part);
        if (part)
            hipLaunchKernelGGL(k_direct_fold<double>, fold, dim3(64), 0, c.stream, n, n_dev, splits, (double *)part,
                               out_idx, phi, grad);
    }
    LSS_CHECK_LAUNCH("k_p2p_direct");
}

// persistent workgroups of the Hessian and sigma(x) kernels: three of
// kHessWaves waves fill a CU (168 VGPRs)
unsigned hess_grid(int64_t max_tiles, int W) {
    return (unsigned)std::min<int64_t>(max_tiles > 0 ? max_tiles : 1, kHessResident / W);
}

template <int TILE>
void launch_hess_tile(Ctx &c, unsigned grid, const FmmEvalArgs &a, double *hess) {
    const size_t shm = sizeof(double) * (size_t)a.ncp;
    hipLaunchKernelGGL(k_hess_fmm<TILE>, dim3(grid), dim3(TILE), shm, c.stream, a, hess);
    LSS_CHECK_LAUNCH("k_hess_fmm");
}

// nexp: expansions of a heavy tile evaluated at once (their results fit the
// rings' LDS)
void launch_mixed_waves(Ctx &c, int64_t max_tiles, const FmmEvalArgs &a) {
    const size_t region = region_for(std::max(kMixedRingBytes, (kMixedWideBytes + kWide - 1) / kWide), 0);
    const int nexp = (int)std::min<size_t>(kWide, region * kWide / (sizeof(double) * 256));
    const unsigned grid = (unsigned)std::min<int64_t>(max_tiles > 0 ? max_tiles : 1, kWideWaves / kWide);
    auto k = c.opt.count_useful ? k_eval_fmm_mixed_waves<true> : k_eval_fmm_mixed_waves<false>;
    hipLaunchKernelGGL(k, dim3(grid), dim3(64 * kWide), region * kWide, c.stream, a, (int)(region / sizeof(double)), nexp);
    LSS_CHECK_LAUNCH("k_eval_fmm_mixed_waves");
}

// persistent workgroups of waves: two of kWide waves fill a CU at 128 VGPRs
void launch_f64_waves(Ctx &c, int64_t max_tiles, const FmmEvalArgs &a) {
    const size_t region = region_for(kF64RingBytes, 0);
    const int W = waves_for(region);
    const unsigned grid = (unsigned)std::min<int64_t>(max_tiles > 0 ? max_tiles : 1, kWideWaves / W);
    auto k = c.opt.count_useful ? k_eval_fmm_f64_waves<true> : k_eval_fmm_f64_waves<false>;
    hipLaunchKernelGGL(k, dim3(grid), dim3(64 * W), region * W, c.stream, a, (int)(region / sizeof(double)));
    LSS_CHECK_LAUNCH("k_eval_fmm_f64_waves");
}

template <int TILE>
void launch_fmm_tile(Ctx &c, unsigned grid, const FmmEvalArgs &a) {
    const size_t shm = sizeof(double) * (size_t)a.ncp;
    if (c.opt.count_useful)
        hipLaunchKernelGGL((k_eval_fmm_f64<TILE, true>), dim3(grid), dim3(TILE), shm, c.stream, a);
    else
        hipLaunchKernelGGL((k_eval_fmm_f64<TILE, false>), dim3(grid), dim3(TILE), shm, c.stream, a);
    LSS_CHECK_LAUNCH("k_eval_fmm");
}

}  // namespace

// FMM tiles: 0 = default 64 (narrow tiles keep the lanes of small leaves
// busy); the mixed kernel always takes 64-target tiles
int fmm_tile(const Ctx &c) {
    if (c.opt.precision == LSS_MIXED) return 64;
    if (c.opt.tile == 64 || c.opt.tile == 128 || c.opt.tile == 256) return c.opt.tile;
    return 64;
}

void launch_eval_fmm(Ctx &c, int64_t max_tiles, const int32_t *ntiles_dev, const int32_t *tile_start,
                     const int32_t *n_dev, int64_t n_max, const int32_t *sorted_leaf, const int32_t *sorted_idx,
                     const double *tx, const double *ty, const double *tz, const int32_t *out_idx, double *phi,
                     double *grad, const int32_t *order, double *pairs, double *hess, const MsArgs *ms) {
    const Tree &t = c.tree;
    FmmEvalArgs a;
    a.ntiles_dev = ntiles_dev;
    a.tile_start = tile_start;
    a.n_max = n_max;
    a.n_dev = n_dev;
    a.sleaf = sorted_leaf;
    a.sidx = sorted_idx;
    a.tx = tx; a.ty = ty; a.tz = tz;
    a.out_idx = out_idx;
    a.phi = phi;
    a.grad = grad;
    a.p2p_beg = t.p2p_beg.as<int32_t>();
    a.p2p_end = t.p2p_end.as<int32_t>();
    a.p2p_src = t.p2p_val2.as<int32_t>();
    a.nb = t.nb.as<int64_t>();
    a.ne = t.ne.as<int64_t>();
    a.lev = t.level.as<int32_t>();
    a.ijk = t.ijk.as<int32_t>();
    a.src = t.src.as<Src>();
    a.nnodes = c.nnodes;
    a.nboxes = (int32_t)t.nboxes;
    a.L = t.L.as<double>();
    a.M = t.M.as<double>();
    a.m2p_beg = t.m2p_beg.as<int32_t>();
    a.m2p_end = t.m2p_end.as<int32_t>();
    a.m2p_src = t.m2p_val2.as<int32_t>();
    a.p = t.p;
    a.ncp = t.ncp;
    a.root = t.root.as<double>();
    a.bmesh = t.bmesh.as<int32_t>();
    a.pairs = pairs;
    a.queue = c.tile_queue.as<unsigned int>();
    a.order = order;
    a.nheavy = c.tile_bucket.as<int32_t>() + 2 * kCostBuckets;
    a.child = t.child.as<int32_t>();
    a.parent = t.parent.as<int32_t>();
    a.rmax = t.rmax.as<double>();
    a.K = t.K;
    {
        const double cut = c.opt.cut_factor > 0 ? c.opt.cut_factor
                                                 : (c.opt.precision == LSS_MIXED ? kCutMixed : kCutFP64);
        a.tcut = 0.5 * cut * cut;
    }
    int64_t g = max_tiles < 16384 ? max_tiles : 16384;
    unsigned grid = (unsigned)(g > 0 ? g : 1);
    if (ms) {                               // target-attached width (FP64)
        const size_t shm = sizeof(double) * (size_t)a.ncp;
        switch (fmm_tile(c)) {
            case 64: {
                const size_t region = region_for(kChunkBytes, 0);   // it stages no expansion
                const int W = std::min(kHessWaves, waves_for(region));
                hipLaunchKernelGGL(k_multiscale_waves, dim3(hess_grid(max_tiles, W)), dim3(64 * W), region * W, c.stream,
                                   a, *ms, (int)(region / sizeof(double)));
                break;
            }
            case 128: hipLaunchKernelGGL(k_multiscale_fmm<128>, dim3(grid), dim3(128), shm, c.stream, a, *ms); break;
            default: hipLaunchKernelGGL(k_multiscale_fmm<256>, dim3(grid), dim3(256), shm, c.stream, a, *ms); break;
        }
        LSS_CHECK_LAUNCH("k_multiscale_fmm");
        const int64_t go = ceil_div(n_max > 0 ? n_max : 1, 256);
        hipLaunchKernelGGL(k_multiscale_outside, dim3((unsigned)(go < 1024 ? go : 1024)), dim3(256), 0, c.stream, a,
                           *ms);
        LSS_CHECK_LAUNCH("k_multiscale_outside");
        return;
    }
    if (hess) {                             // Phi, grad Phi and the Hessian (FP64)
        switch (fmm_tile(c)) {
            case 64: {
                const size_t region = region_for(kChunkBytes, a.ncp);
                const int W = std::min(kHessWaves, waves_for(region));
                hipLaunchKernelGGL(k_hess_waves, dim3(hess_grid(max_tiles, W)), dim3(64 * W), region * W, c.stream, a,
                                   hess, (int)(region / sizeof(double)));
                LSS_CHECK_LAUNCH("k_hess_waves");
                break;
            }
            case 128: launch_hess_tile<128>(c, grid, a, hess); break;
            default: launch_hess_tile<256>(c, grid, a, hess); break;
        }
        const int64_t go = ceil_div(n_max > 0 ? n_max : 1, 256);
        hipLaunchKernelGGL(k_hess_outside, dim3((unsigned)(go < 1024 ? go : 1024)), dim3(256), 0, c.stream, a, hess);
        LSS_CHECK_LAUNCH("k_hess_outside");
        return;
    }
    if (c.opt.precision == LSS_MIXED) {
        launch_mixed_waves(c, max_tiles, a);
    } else {
        switch (fmm_tile(c)) {
            case 64: launch_f64_waves(c, max_tiles, a); break;
            case 128: launch_fmm_tile<128>(c, grid, a); break;
            default: launch_fmm_tile<256>(c, grid, a); break;
        }
    }
    const int64_t go = ceil_div(n_max > 0 ? n_max : 1, 256);
    hipLaunchKernelGGL(k_eval_outside, dim3((unsigned)(go < 1024 ? go : 1024)), dim3(256), 0, c.stream, a);
    LSS_CHECK_LAUNCH("k_eval_outside");
}

int direct_splits(const Ctx &c, int64_t n) {
    const int tile = direct_tile(c);
    return direct_pieces(ceil_div(n > 0 ? n : 1, tile), ceil_div(c.nnodes > 0 ? c.nnodes : 1, tile), tile,
                         c.nmesh == 1);
}

// bytes of partial sums of one target and piece
size_t direct_part_size(const Ctx &c) { return 8 * (c.opt.precision == LSS_MIXED ? sizeof(float) : sizeof(double)); }

size_t direct_part_bytes(const Ctx &c, int64_t n) {
    const int s = direct_splits(c, n);
    return s > 1 ? (size_t)n * (size_t)s * direct_part_size(c) : 0;
}

void ensure_direct_part(Ctx &c, int64_t n) {
    const int tile = direct_tile(c);
    c.part.ensure((size_t)direct_partials_kept(n, ceil_div(c.nnodes > 0 ? c.nnodes : 1, tile), tile) * direct_part_size(c));
}

void launch_p2p_direct(Ctx &c, int64_t n, const int32_t *n_dev, const double *tx, const double *ty,
                       const double *tz, const int32_t *tmesh, const int32_t *out_idx, double *phi,
                       double *grad, int /*grad_stride*/, double *pairs, void *part) {
    if (n <= 0) return;
    switch (direct_tile(c)) {
        case 64: launch_tile<64>(c, n, n_dev, tx, ty, tz, tmesh, out_idx, phi, grad, pairs, part); break;
        case 128: launch_tile<128>(c, n, n_dev, tx, ty, tz, tmesh, out_idx, phi, grad, pairs, part); break;
        default: launch_tile<256>(c, n, n_dev, tx, ty, tz, tmesh, out_idx, phi, grad, pairs, part); break;
    }
}

}  // namespace lss
