// Laplace-dipole fast multipole far field (section 4.4, eq. kerdecomp: beyond
// the cut the kernel is the double-layer kernel, summed here by an FMM):
// translation operators as dense real matrices, dipole P2M at the leaves, and
// every translation (M2M, M2L, L2L) as a gathered matrix product
//     Y[dst_j] += scale_j * Op * X[src_j]
// on the FP64 matrix cores (v_mfma_f64_16x16x4f64).  M2M and L2L run one
// launch per level.  M2L has two forms, both race free and deterministic:
//   FP64 near fields (m2l_plan, m2l_pass; FP64 contexts and the
//     target-attached width, whose 1e5 points on 43 200 triangles take 4 ms
//     less of some 20 than with the other form): all pairs sorted by operator, rotated
//     so that the operators split in two halves; one product launch and one
//     sum launch per block of target boxes, each pair's product in a slot of
//     its own and the sums in a fixed order.
//   mixed contexts, and lists of 2^31 pairs and more: one launch per
//     displacement class (one dense operator per class); inside a launch every
//     destination box appears once.  The rotated form would change the far field by 1e-16, and a Newton iterate
//     moved by that makes a few FP32 pair sums of a million nodes round the
//     other way (up to 7e-9 sigma in a node's h); the mixed projection is
//     kept the same bit for bit.  What it gained there when it was tried is
//     small: 1 to 3 ms of a batch of 24 surfaces (43 ms), nothing at 2e6
//     triangles.
#include <cstring>
#include <algorithm>
#include <hip/hip_runtime.h>

#include <cmath>
#include <map>
#include <vector>

#include "fmm_math.h"
#include "lss_internal.h"

namespace lss {

namespace {

using fmm::cd;
constexpr int kBlk = 256;
constexpr int kR = 7;
constexpr int kNClass = (2 * kR + 1) * (2 * kR + 1) * (2 * kR + 1);
constexpr double kPi = 3.14159265358979323846;

inline unsigned grid_for(int64_t n, int blk = kBlk) { return (unsigned)ceil_div(n > 0 ? n : 1, blk); }

// ------------------------------------------------------------- operators
// one table per operator: irregular (M2L, order 2p) or regular (M2M/L2L, order p)
__global__ void k_op_tables(int nops, const double *__restrict__ vecs, int order, int irregular, int stride, cd *tabs) {
    int o = blockIdx.x * blockDim.x + threadIdx.x;
    if (o >= nops) return;
    const double *v = vecs + 3 * o;
    if (irregular) fmm::irregular_table(v[0], v[1], v[2], order, tabs + (int64_t)o * stride);
    else fmm::regular_table(v[0], v[1], v[2], order, tabs + (int64_t)o * stride);
}

// entry (row, k) of operator o stored k-major: opT[o][k * ncp + row]
__global__ void k_fill_op(int kind, int p, int ncp, int nops, const cd *__restrict__ tabs, int stride, double *ops) {
    const int64_t per = (int64_t)ncp * ncp;
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int o = blockIdx.y;
    if (e >= per || o >= nops) return;
    const int k = (int)(e / ncp), row = (int)(e - (int64_t)k * ncp);
    const int nc = fmm::ncoef(p);
    double v = 0.0;
    if (row < nc && k < nc) {
        int kk, l, n, m;
        bool oi, ii;
        fmm::decode(row, kk, l, oi);
        fmm::decode(k, n, m, ii);
        const cd *tab = tabs + (int64_t)o * stride;
        if (kind == 0) v = fmm::folded_entry(fmm::M2LMap{tab}, kk, l, oi, n, m, ii);
        else if (kind == 1) v = fmm::folded_entry(fmm::M2MMap{tab}, kk, l, oi, n, m, ii);
        else v = fmm::folded_entry(fmm::L2LMap{tab}, kk, l, oi, n, m, ii);
    }
    ops[(int64_t)o * per + e] = v;
}

// Irregular tables (order 2p) of the M2L operators: thread (operator, m) runs
// column m of fmm::irregular_table, the same recurrences
__global__ void k_m2l_tables(int nops, const double *__restrict__ vecs, int order, int stride, cd *tabs) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const int o = i / (order + 1), m = i % (order + 1);
    if (o >= nops) return;
    const double x = vecs[3 * o], y = vecs[3 * o + 1], z = vecs[3 * o + 2];
    cd *T = tabs + (int64_t)o * stride;
    const double r2 = x * x + y * y + z * z, ir2 = 1.0 / r2;
    cd tm1 = {sqrt(ir2), 0.0}, tm2 = {0.0, 0.0};
    for (int k = 1; k <= m; ++k) tm1 = fmm::cscale(fmm::cmul(tm1, cd{x, y}), -(2.0 * k - 1.0) * ir2);
    T[fmm::tri(m, m)] = tm1;
    for (int n = m + 1; n <= order; ++n) {
        const double a = (2 * n - 1) * z, b = (double)(n - 1 + m) * (double)(n - 1 - m);
        const cd tn = {(a * tm1.re - b * tm2.re) * ir2, (a * tm1.im - b * tm2.im) * ir2};
        T[fmm::tri(n, m)] = tn;
        tm2 = tm1;
        tm1 = tn;
    }
}

// M2L operator o of a displacement with y = 0 as its two halves: entry (row,
// col) of the product of the Re parts at ops[2 o], of the Im parts at
// ops[2 o + 1], k-major (col * ldr + row), rows and columns q = (n, m >= 0) in
// the order of fmm::tri, zero beyond order p
__global__ void k_fill_m2l(int p, int ldk, int ldr, int nops, const cd *__restrict__ tabs, int stride,
                           const int32_t *__restrict__ qtab, double *ops) {
    const int64_t per = (int64_t)ldk * ldr;
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int o = blockIdx.y >> 1, im = blockIdx.y & 1;
    if (e >= per || o >= nops) return;
    const int col = (int)(e / ldr), row = (int)(e % ldr), nq = (p + 1) * (p + 2) / 2;
    double v = 0.0;
    if (row < nq && col < nq) {
        const int tr = qtab[row], tc = qtab[col];
        const int k = tr >> 24, l = (tr >> 16) & 0xff, n = tc >> 24, m = (tc >> 16) & 0xff;
        if (!im || (l > 0 && m > 0))
            v = fmm::folded_entry(fmm::M2LMap{tabs + (int64_t)o * stride}, k, l, im, n, m, im);
    }
    ops[(2 * (int64_t)o + im) * per + e] = v;
}

// ------------------------------------------------------------------ P2M
// Neighbour lanes through DPP wave shifts (one VALU move per 32-bit half, no
// LDS round trip): the value of lane + 1 and of lane - 1; the lanes without a
// neighbour (63 and 0) receive 0.
__device__ __forceinline__ double dpp_f64(double v, int ctrl_is_next) {
    const long long b = __double_as_longlong(v);
    int lo = (int)b, hi = (int)(b >> 32);
    if (ctrl_is_next) {
        lo = __builtin_amdgcn_mov_dpp(lo, 0x130, 0xf, 0xf, true);     // wave_shl:1
        hi = __builtin_amdgcn_mov_dpp(hi, 0x130, 0xf, 0xf, true);
    } else {
        lo = __builtin_amdgcn_mov_dpp(lo, 0x138, 0xf, 0xf, true);     // wave_shr:1
        hi = __builtin_amdgcn_mov_dpp(hi, 0x138, 0xf, 0xf, true);
    }
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double from_next_lane(double v) { return dpp_f64(v, 1); }
__device__ __forceinline__ double from_prev_lane(double v) { return dpp_f64(v, 0); }

struct Geo {
    const double *root;         // per-mesh root cubes (corner xyz, side)
    const int32_t *bmesh;
};

// P2M by columns: one wavefront per non-empty leaf; lane (g, m) owns column
// m = 0..p of the regular solid harmonics of node g of a group of G = 64/(p+1)
// nodes.  At step s every lane holds U_s^m (zero for m > s; the diagonal is
// built up meanwhile), takes U_s^{m-1} and U_s^{m+1} from its neighbours and
// adds the dipole term of M_{s+1}^m into an LDS accumulator of its node slot.
// No division and no barrier inside the node loop.
__global__ __launch_bounds__(64) void k_p2m_cols(const int32_t *__restrict__ nleaf_dev,
                                                 const int32_t *__restrict__ leaves, int p, int ncp, Geo g,
                                                 const int32_t *__restrict__ lev, const int32_t *__restrict__ ijk,
                                                 const int64_t *__restrict__ nb, const int64_t *__restrict__ ne,
                                                 const Src *__restrict__ src, double *M) {
    extern __shared__ double smem[];
    const int C = p + 1, G = 64 / C;
    const int ntri = (p + 1) * (p + 2) / 2;
    cd *acc = reinterpret_cast<cd *>(smem);               // G x ntri, at tri(n, m)
    double *rinv = smem + 2 * G * ntri;                   // 1/((n+m)(n-m)) at tri(n, m), n > m
    double *dfac = rinv + ntri;                           // -1/(2t), t = 1..p
    if ((int)blockIdx.x >= *nleaf_dev) return;
    const int lane = threadIdx.x;
    for (int i = lane; i < ntri; i += 64) {
        int n = 0;
        while ((n + 1) * (n + 2) / 2 <= i) ++n;
        const int m = i - n * (n + 1) / 2;
        rinv[i] = n > m ? 1.0 / ((double)(n + m) * (double)(n - m)) : 0.0;
    }
    for (int t = lane; t <= p; t += 64) dfac[t] = t > 0 ? -0.5 / (double)t : 0.0;
    for (int i = lane; i < G * ntri; i += 64) acc[i] = cd{0.0, 0.0};
    __syncthreads();
    const int32_t b = leaves[blockIdx.x];
    const double s = box_side(g.root, g.bmesh, b, lev[b]);
    const double *o = g.root + 4 * g.bmesh[b];
    const double c0 = o[0] + (ijk[3 * b] + 0.5) * s, c1 = o[1] + (ijk[3 * b + 1] + 0.5) * s,
                 c2 = o[2] + (ijk[3 * b + 2] + 0.5) * s;
    const double inv4pis = 1.0 / (4.0 * kPi * s);
    const double invs = 1.0 / s;
    const int gi = lane / C, m = lane % C;
    const bool slot = gi < G;                             // lane holds a (node, column) slot
    cd *accg = acc + (slot ? gi : 0) * ntri;
    const int64_t b0 = nb[b], b1 = ne[b];
    for (int64_t k0 = b0; k0 < b1; k0 += G) {
        const int64_t k = k0 + gi;
        const bool live = slot && k < b1;
        double x = 0, y = 0, z = 0, ax = 0, ay = 0, az = 0;
        if (live) {
            const Src sr = src[k];
            // unfold the dipole: a = a' / c(sigma), 1/c = 4 sqrt2 pi^1.5 sigma^3, sigma^2 = 1/(2 s2)
            const double sg2 = 0.5 / sr.s2;
            const double f = 4.0 * 1.4142135623730951 * 5.568327996831708 * sg2 * sqrt(sg2);
            x = (sr.yx - c0) * invs;
            y = (sr.yy - c1) * invs;
            z = (sr.yz - c2) * invs;
            ax = sr.ax * f;
            ay = sr.ay * f;
            az = sr.az * f;
        }
        const double r2 = x * x + y * y + z * z;
        cd d = {1.0, 0.0}, u1 = {0.0, 0.0}, u2 = {0.0, 0.0};
        for (int st = 0; st < p; ++st) {
            cd u = {0.0, 0.0};
            if (st == m) {
                u = d;
            } else if (st > m) {
                const double w = rinv[fmm::tri(st, m)];
                const double a2 = (double)(2 * st - 1) * z;
                u = cd{(a2 * u1.re - r2 * u2.re) * w, (a2 * u1.im - r2 * u2.im) * w};
            } else {
                d = fmm::cscale(fmm::cmul(d, cd{x, y}), dfac[st + 1]);
            }
            if (st >= m) { u2 = u1; u1 = u; }
            // neighbours' columns at order st (same node slot; U^{-1} = -conj(U^1))
            const double upre = from_next_lane(u.re), upim = from_next_lane(u.im);
            const double dnre = from_prev_lane(u.re), dnim = from_prev_lane(u.im);
            cd up = m + 1 < C ? cd{upre, upim} : cd{0.0, 0.0};
            cd dn = m >= 1 ? cd{dnre, dnim} : cd{-upre, upim};
            if (live && m <= st + 1) {
                const cd t = fmm::cadd(fmm::cadd(fmm::cmul(cd{0.5 * ax, -0.5 * ay}, up),
                                                 fmm::cmul(cd{-0.5 * ax, -0.5 * ay}, dn)),
                                       fmm::cscale(u, az));
                cd &A = accg[fmm::tri(st + 1, m)];
                A.re -= inv4pis * t.re;         // conj, times -1/(4 pi s)
                A.im += inv4pis * t.im;
            }
        }
    }
    __syncthreads();
    double *Mb = M + (int64_t)b * ncp;
    for (int i = lane; i < ntri; i += 64) {
        int n = 0;
        while ((n + 1) * (n + 2) / 2 <= i) ++n;
        const int mm = i - n * (n + 1) / 2;
        if (n == 0) continue;
        double re = 0.0, im = 0.0;
        for (int q = 0; q < G; ++q) { re += acc[q * ntri + i].re; im += acc[q * ntri + i].im; }
        Mb[fmm::ire(n, mm)] = re;
        if (mm > 0) Mb[fmm::iim(n, mm)] = im;
    }
}


// The same P2M for the default orders (P known at compile time): lane (g, m)
// keeps its column's contributions to M_n^m, n = 1..P, in registers across
// all the leaf's nodes (the step loop is unrolled), instead of a read-modify-
// write in LDS per step; the G node slots are summed by shuffles at the end,
// in the order the LDS version sums them.
template <int P>
__global__ __launch_bounds__(64) void k_p2m_reg(const int32_t *__restrict__ nleaf_dev,
                                                const int32_t *__restrict__ leaves, int ncp, Geo g,
                                                const int32_t *__restrict__ lev, const int32_t *__restrict__ ijk,
                                                const int64_t *__restrict__ nb, const int64_t *__restrict__ ne,
                                                const Src *__restrict__ src, double *M) {
    constexpr int C = P + 1, G = 64 / C, ntri = (P + 1) * (P + 2) / 2;
    __shared__ double rinv[ntri];                         // 1/((n+m)(n-m)) at tri(n, m), n > m
    __shared__ double dfac[P + 1];                        // -1/(2t), t = 1..P
    if ((int)blockIdx.x >= *nleaf_dev) return;
    const int lane = threadIdx.x;
    for (int i = lane; i < ntri; i += 64) {
        int n = 0;
        while ((n + 1) * (n + 2) / 2 <= i) ++n;
        const int m = i - n * (n + 1) / 2;
        rinv[i] = n > m ? 1.0 / ((double)(n + m) * (double)(n - m)) : 0.0;
    }
    for (int t = lane; t <= P; t += 64) dfac[t] = t > 0 ? -0.5 / (double)t : 0.0;
    __syncthreads();
    const int32_t b = leaves[blockIdx.x];
    const double s = box_side(g.root, g.bmesh, b, lev[b]);
    const double *o = g.root + 4 * g.bmesh[b];
    const double c0 = o[0] + (ijk[3 * b] + 0.5) * s, c1 = o[1] + (ijk[3 * b + 1] + 0.5) * s,
                 c2 = o[2] + (ijk[3 * b + 2] + 0.5) * s;
    const double inv4pis = 1.0 / (4.0 * kPi * s);
    const double invs = 1.0 / s;
    const int gi = lane / C, m = lane % C;
    const bool slot = gi < G;
    double are[P], aim[P];                                // contributions to M_{st+1}^m
#pragma unroll
    for (int st = 0; st < P; ++st) are[st] = aim[st] = 0.0;
    double w[P];                                          // recurrence weights of column m
#pragma unroll
    for (int st = 0; st < P; ++st) w[st] = rinv[fmm::tri(st, m)];     // in range for every m <= P
    const int64_t b0 = nb[b], b1 = ne[b];
    for (int64_t k0 = b0; k0 < b1; k0 += G) {
        const int64_t k = k0 + gi;
        const bool live = slot && k < b1;
        double x = 0, y = 0, z = 0, ax = 0, ay = 0, az = 0;
        if (live) {
            const Src sr = src[k];
            // unfold the dipole: a = a' / c(sigma), 1/c = 4 sqrt2 pi^1.5 sigma^3, sigma^2 = 1/(2 s2)
            const double sg2 = 0.5 / sr.s2;
            const double f = 4.0 * 1.4142135623730951 * 5.568327996831708 * sg2 * sqrt(sg2);
            x = (sr.yx - c0) * invs;
            y = (sr.yy - c1) * invs;
            z = (sr.yz - c2) * invs;
            ax = sr.ax * f;
            ay = sr.ay * f;
            az = sr.az * f;
        }
        const double r2 = x * x + y * y + z * z;
        // The dipole term of M_{st+1}^m is t = hp U^{m+1} + hm U^{m-1} + az U^m
        // (hp = (ax - i ay) / 2, hm = (-ax - i ay) / 2, U at order st), taken
        // conjugated and times -1/(4 pi s).  Written out as real coefficients
        // of (Re, Im) of U^{m+1}, U^{m-1} and U^m, with the two edge columns
        // folded in: U^{-1} = -conj(U^1) for m = 0, and no U^{P+1} for m = P;
        // a dead slot has all coefficients 0.
        const double hpr = 0.5 * ax, hpi = -0.5 * ay, hmr = -0.5 * ax, hmi = -0.5 * ay;
        double qr[4] = {hpr, -hpi, hmr, -hmi}, qi[4] = {hpi, hpr, hmi, hmr};
        if (m == 0) {
            qr[0] = hpr - hmr; qr[1] = -hpi - hmi; qr[2] = 0.0; qr[3] = 0.0;
            qi[0] = hpi - hmi; qi[1] = hpr + hmr; qi[2] = 0.0; qi[3] = 0.0;
        } else if (m == P) {
            qr[0] = qr[1] = 0.0;
            qi[0] = qi[1] = 0.0;
        }
        const double sr_ = -inv4pis, si_ = inv4pis;
        const double cr0 = sr_ * qr[0], cr1 = sr_ * qr[1], cr2 = sr_ * qr[2], cr3 = sr_ * qr[3], cr4 = sr_ * az;
        const double ci0 = si_ * qi[0], ci1 = si_ * qi[1], ci2 = si_ * qi[2], ci3 = si_ * qi[3], ci4 = si_ * az;
        // U^m at order st, for every lane and step without branches: the
        // diagonal d = U^m_m is carried up (multiplied by (x + i y) / (-2 t)
        // at every step, read at st = m), the column recurrence starts from
        // zeros (so it is 0 for st <= m)
        double dr = 1.0, di = 0.0, u1r = 0.0, u1i = 0.0, u2r = 0.0, u2i = 0.0;
#pragma unroll
        for (int st = 0; st < P; ++st) {
            const double a2 = (double)(2 * st - 1) * z;
            double ur = (a2 * u1r - r2 * u2r) * w[st], ui = (a2 * u1i - r2 * u2i) * w[st];
            const bool diag = st == m;
            ur = diag ? dr : ur;
            ui = diag ? di : ui;
            const double sc = -0.5 / (double)(st + 1);
            const double ndr = (dr * x - di * y) * sc, ndi = (dr * y + di * x) * sc;
            dr = ndr;
            di = ndi;
            u2r = u1r; u2i = u1i;
            u1r = ur; u1i = ui;
            const double upr = from_next_lane(ur), upi = from_next_lane(ui);
            const double dnr = from_prev_lane(ur), dni = from_prev_lane(ui);
            are[st] = fma(cr0, upr, fma(cr1, upi, fma(cr2, dnr, fma(cr3, dni, fma(cr4, ur, are[st])))));
            aim[st] = fma(ci0, upr, fma(ci1, upi, fma(ci2, dnr, fma(ci3, dni, fma(ci4, ui, aim[st])))));
        }
    }
    // sum the node slots into lanes (0, m) and write M~_n^m, n = 1..P
    double *Mb = M + (int64_t)b * ncp;
#pragma unroll
    for (int st = 0; st < P; ++st) {
        double re = 0.0 + are[st], im = 0.0 + aim[st];
#pragma unroll
        for (int q = 1; q < G; ++q) {
            re += __shfl(are[st], lane + q * C);
            im += __shfl(aim[st], lane + q * C);
        }
        const int n = st + 1;
        if (gi == 0 && m <= n) {
            Mb[fmm::ire(n, m)] = re;
            if (m > 0) Mb[fmm::iim(n, m)] = im;
        }
    }
}

__global__ void k_leaf_flags(int64_t n, const int32_t *__restrict__ child, const int64_t *__restrict__ nb,
                             const int64_t *__restrict__ ne, int32_t *flag, int32_t *ids) {
    int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n) return;
    flag[b] = (child[b] < 0 && ne[b] > nb[b]) ? 1 : 0;
    ids[b] = (int32_t)b;
}

// --------------------------------------------------------- gathered GEMM
typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int kKB = 16;

enum { G_LIST = 0, G_M2M = 1, G_L2L = 2 };

// One launch of translations Y[dst] += scale * Op X[src] over a list of pairs.
//   G_LIST: M2L pairs of one displacement class (dst = low 32 bits of mkey, src = mval).
//   G_M2M:  pair j = the j-th parent of a level; its 8 children (consecutive boxes
//           base + 8j ..) are one input column of 8 ncp coefficients and the 8 octant
//           operators, stored one after the other in k-major order, are one
//           ncp x 8 ncp operator, so each parent is written once per launch.
//   G_L2L:  grid.z = octant o; pair j writes child base + 8j + o from its parent with
//           operator o.  Children are distinct, so the 8 octants share the launch.
struct GemmArgs {
    int mode, ncp, nk;          // nk: length of the contraction (ncp, or 8 ncp for G_M2M)
    int64_t npairs;
    const double *opT;          // ncp rows, k-major (G_L2L: 8 such matrices)
    const double *X;
    double *Y;
    const uint64_t *mkey;       // G_LIST
    const int32_t *mval;        // G_LIST
    int64_t base;               // G_M2M / G_L2L: first child box of the level
    const int32_t *parent, *lev;
    const double *root;
    const int32_t *bmesh;
    int rows = 0;               // output rows (leading coefficients written); 0 = ncp
};

// destination box, first element of the input column and output scale of pair j
__device__ inline void pair_of(const GemmArgs &a, int64_t j, int oct, int64_t &dst, int64_t &col, double &scale) {
    scale = 1.0;
    if (a.mode == G_LIST) {
        dst = (int64_t)(uint32_t)(a.mkey[j] & 0xffffffffu);
        col = (int64_t)a.mval[j] * a.ncp;
        scale = 1.0 / box_side(a.root, a.bmesh, (int32_t)dst, a.lev[dst]);   // 1 / side of the target box
    } else if (a.mode == G_M2M) {
        const int64_t ch = a.base + 8 * j;
        dst = a.parent[ch];
        col = ch * a.ncp;
    } else {
        dst = a.base + 8 * j + oct;
        col = (int64_t)a.parent[dst] * a.ncp;
    }
}

// 64 output rows x 128 pairs per workgroup; wave w owns pairs 32w..32w+31 of
// the tile and eight 16x16 accumulator tiles (4 row groups x 2 pair groups).
// The operator (k-major) and the gathered input columns go through LDS in
// blocks of kKB coefficients; the next block is fetched into registers while
// the MFMAs of the current one run.  Asking for four waves per SIMD makes the
// compiler keep the accumulators in ordinary VGPRs (126 in all, no AGPRs):
// four workgroups share a CU instead of two, which hides the barrier and load
// latency of one workgroup behind the MFMAs of the others.
// TP = 128 pairs per workgroup for long pair lists, 64 for short ones (twice
// the workgroups for the same work where one launch would not fill the chip).
constexpr int kTR = 64;
template <int TP>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_gemm(GemmArgs a) {
    constexpr int kTP = TP, NT = TP / 64, TPC = 256 / TP;   // 16-pair groups per wave, threads per column
    __shared__ double As[kKB][kTR + 1];
    __shared__ double Bs[kKB][kTP + 1];
    __shared__ int64_t scol[kTP];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r0 = blockIdx.x * kTR;
    const int64_t j0 = (int64_t)blockIdx.y * kTP;
    const int oct = blockIdx.z;
    const double *__restrict__ op = a.opT + (int64_t)oct * a.ncp * a.ncp;
    if (threadIdx.x < kTP) {
        int64_t j = j0 + threadIdx.x, d, col;
        double sc;
        if (j < a.npairs) { pair_of(a, j, oct, d, col, sc); scol[threadIdx.x] = col; }
        else scol[threadIdx.x] = -1;
    }
    __syncthreads();
    // per thread: A elements (k, r) = (e / kTR, e % kTR) for e = tid + 256 i, i < 4;
    // B elements (k, c) with c = tid / TPC, k = kNB (tid % TPC) + i, i < kNB (TPC threads per column)
    constexpr int kNA = kKB * kTR / 256, kNB = kKB * kTP / 256;
    const int bc = threadIdx.x / TPC, bk = (threadIdx.x % TPC) * kNB;
    const int64_t bcol = scol[bc];
    double ra[kNA], rb[kNB];
    auto fetch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < kNA; ++i) {
            const int e = threadIdx.x + 256 * i, kk = e / kTR, rr = e % kTR;
            ra[i] = (r0 + rr < a.rows) ? op[(int64_t)(k0 + kk) * a.ncp + r0 + rr] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < kNB; ++i) rb[i] = bcol >= 0 ? a.X[bcol + k0 + bk + i] : 0.0;
    };
    d4 acc[4][NT];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        for (int t = 0; t < NT; ++t) acc[i][t] = d4{0.0, 0.0, 0.0, 0.0};
    fetch(0);
    for (int k0 = 0; k0 < a.nk; k0 += kKB) {
        __syncthreads();                                   // previous block's MFMAs are done with LDS
#pragma unroll
        for (int i = 0; i < kNA; ++i) {
            const int e = threadIdx.x + 256 * i;
            As[e / kTR][e % kTR] = ra[i];
        }
#pragma unroll
        for (int i = 0; i < kNB; ++i) Bs[bk + i][bc] = rb[i];
        __syncthreads();
        if (k0 + kKB < a.nk) fetch(k0 + kKB);
#pragma unroll
        for (int kk = 0; kk < kKB; kk += 4) {
            double bv[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) bv[t] = Bs[kk + (lane >> 4)][16 * NT * w + 16 * t + (lane & 15)];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const double av = As[kk + (lane >> 4)][16 * i + (lane & 15)];
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[i][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv[t], acc[i][t], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int64_t j = j0 + 16 * NT * w + 16 * t + (lane & 15);
        if (j >= a.npairs) continue;
        int64_t d, col;
        double sc;
        pair_of(a, j, oct, d, col, sc);
        double *y = a.Y + d * a.ncp;
        // v_mfma_f64_16x16x4f64 accumulator: register q of lane l holds row (l/16) + 4q, column l%16
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int row = r0 + 16 * i + (lane >> 4) + 4 * q;
                if (row < a.rows) y[row] += sc * acc[i][t][q];
            }
    }
}

// The same translations for launches that do not fill the chip, whose time is
// the chain of one workgroup's steps: 16 rows x 64 pairs (one accumulator tile
// per wave, a quarter of the chain's products, four times the workgroups) and
// kKS coefficients per step, so that fewer and longer fetches stand in the
// chain.  The products of an output are added in the same order: the result is
// that of k_gemm bit for bit.  Two steps' fetches are on their way.  M2M of a
// small tree at p = 26 (5832 coefficients a parent) 280 -> 131 us a level, L2L
// 40 -> 26, M2L of a class of 500 to 2000 pairs 26 -> 11 to 28.
constexpr int kKS = 32;
// 64 x 64 workgroups of a launch below which it is short: at 300 to 400 both
// forms take 35 to 45 us a launch (p = 20), at 150 to 200 this one 23 and
// k_gemm 33 to 44
constexpr int64_t kShortLaunch = 256;
__global__ __launch_bounds__(256) void k_gemm_short(GemmArgs a) {
    __shared__ double As[kKS][17];
    __shared__ double Bs[kKS][65];
    __shared__ int64_t scol[64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int r0 = blockIdx.x * 16;
    const int64_t j0 = (int64_t)blockIdx.y * 64;
    const int oct = blockIdx.z;
    const double *__restrict__ op = a.opT + (int64_t)oct * a.ncp * a.ncp;
    if (threadIdx.x < 64) {
        int64_t j = j0 + threadIdx.x, d, col;
        double sc;
        if (j < a.npairs) { pair_of(a, j, oct, d, col, sc); scol[threadIdx.x] = col; }
        else scol[threadIdx.x] = -1;
    }
    __syncthreads();
    // per thread: A elements (k, r) = (tid / 16 + 16 i, tid % 16), B elements of the columns
    // tid / kKS + (256 / kKS) i at k = tid % kKS (a wave reads along a column)
    constexpr int kNA = kKS / 16, kNB = kKS / 4, kStep = 256 / kKS;
    const int ar = threadIdx.x & 15, ak = threadIdx.x >> 4, bk = threadIdx.x % kKS, bc = threadIdx.x / kKS;
    const bool arow = r0 + ar < a.rows;
    double ra[2][kNA], rb[2][kNB];
    int64_t cols[kNB];
#pragma unroll
    for (int i = 0; i < kNB; ++i) cols[i] = scol[bc + kStep * i];
    auto fetch = [&](int k0, double (&fa)[kNA], double (&fb)[kNB]) {
#pragma unroll
        for (int i = 0; i < kNA; ++i) {
            const int k = k0 + ak + 16 * i;
            fa[i] = arow && k < a.nk ? op[(int64_t)k * a.ncp + r0 + ar] : 0.0;
        }
#pragma unroll
        for (int i = 0; i < kNB; ++i) fb[i] = cols[i] >= 0 && k0 + bk < a.nk ? a.X[cols[i] + k0 + bk] : 0.0;
    };
    d4 acc = {0.0, 0.0, 0.0, 0.0};
    auto step = [&](int k0, double (&fa)[kNA], double (&fb)[kNB]) {
        __syncthreads();                                   // previous block's MFMAs are done with LDS
#pragma unroll
        for (int i = 0; i < kNA; ++i) As[ak + 16 * i][ar] = fa[i];
#pragma unroll
        for (int i = 0; i < kNB; ++i) Bs[bk][bc + kStep * i] = fb[i];
        __syncthreads();
        fetch(k0 + 2 * kKS, fa, fb);                       // zeros past the end
#pragma unroll
        for (int kk = 0; kk < kKS; kk += 4)
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(As[kk + (lane >> 4)][lane & 15], Bs[kk + (lane >> 4)][16 * w + (lane & 15)],
                                                       acc, 0, 0, 0);
    };
    fetch(0, ra[0], rb[0]);
    fetch(kKS, ra[1], rb[1]);
    for (int k0 = 0; k0 < a.nk; k0 += 2 * kKS) {
        step(k0, ra[0], rb[0]);
        if (k0 + kKS < a.nk) step(k0 + kKS, ra[1], rb[1]);
    }
    const int64_t j = j0 + 16 * w + (lane & 15);
    if (j >= a.npairs) return;
    int64_t d, col;
    double sc;
    pair_of(a, j, oct, d, col, sc);
    double *y = a.Y + d * a.ncp;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int row = r0 + (lane >> 4) + 4 * q;
        if (row < a.rows) y[row] += sc * acc[q];
    }
}

void gemm(Ctx &c, GemmArgs a) {
    if (a.rows <= 0) a.rows = a.ncp;
    if (a.npairs > 0 && ceil_div(a.rows, kTR) * ceil_div(a.npairs, 64) * (a.mode == G_L2L ? 8 : 1) < kShortLaunch) {
        const dim3 grid((unsigned)ceil_div(a.rows, 16), (unsigned)ceil_div(a.npairs, 64), a.mode == G_L2L ? 8u : 1u);
        hipLaunchKernelGGL(k_gemm_short, grid, dim3(256), 0, c.stream, a);
        LSS_CHECK_LAUNCH("k_gemm_short");
        return;
    }
    // short lists (fewer than four 128-pair workgroups per CU) take 64-pair workgroups
    const bool small = a.npairs * (a.mode == G_L2L ? 8 : 1) * ceil_div(a.rows, kTR) < 4 * 256 * 128;
    const int tp = small ? 64 : 128;
    // split long pair lists so that grid.y stays within the launch limit
    const int64_t chunk = (int64_t)32768 * tp;
    for (int64_t j0 = 0; j0 < a.npairs; j0 += chunk) {
        GemmArgs b = a;
        b.npairs = a.npairs - j0 < chunk ? a.npairs - j0 : chunk;
        if (a.mode == G_LIST) { b.mkey = a.mkey + j0; b.mval = a.mval + j0; }
        else b.base = a.base + 8 * j0;
        dim3 grid((unsigned)ceil_div(b.rows, kTR), (unsigned)ceil_div(b.npairs, tp), a.mode == G_L2L ? 8u : 1u);
        if (small) hipLaunchKernelGGL(k_gemm<64>, grid, dim3(256), 0, c.stream, b);
        else hipLaunchKernelGGL(k_gemm<128>, grid, dim3(256), 0, c.stream, b);
        LSS_CHECK_LAUNCH("k_gemm");
    }
}

__global__ void k_fill_zero(int64_t n, double *y) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] = 0.0;
}

__global__ void k_add(int64_t n, double *y, const double *x) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        y[i] += x[i];
}

void launch_fill_zero(Ctx &c, double *y, int64_t n) {
    if (n <= 0) return;
    const int64_t g = ceil_div(n, kBlk);
    hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)(g < 65536 ? g : 65536)), dim3(kBlk), 0, c.stream, n, y);
    LSS_CHECK_LAUNCH("k_fill_zero");
}

void launch_add(Ctx &c, double *y, const double *x, int64_t n) {
    if (n <= 0) return;
    const int64_t g = ceil_div(n, kBlk);
    hipLaunchKernelGGL(k_add, dim3((unsigned)(g < 65536 ? g : 65536)), dim3(kBlk), 0, c.stream, n, y, x);
    LSS_CHECK_LAUNCH("k_add");
}

// M2L of the small displacement classes, target-major.  The pairs of all
// small classes are sorted by (target box, class) (key = T << 12 | class);
// the workgroup that meets the first pair of a target box applies every pair
// of that box in key order, each a matrix-vector product with the class
// operator (k-major, leading nkv coefficients in and out), and adds the sum,
// times 1 / side of the box, once.  A box is written by one workgroup only.
constexpr int kSmallClassPairs = 512;        // classes with at most this many pairs
constexpr int kSmallMaxCoeffs = 512;         // target-major only for ncp up to this
constexpr int kSmallRows = 2;                // rows per thread (256 threads)
static_assert(256 * kSmallRows >= kSmallMaxCoeffs, "k_m2l_small: every coefficient needs a thread");
static_assert(kNClass <= 4096, "k_m2l_small: the class index takes the low 12 bits of the key");
__global__ __launch_bounds__(256) void k_m2l_small(int64_t npairs, const uint64_t *__restrict__ key,
                                                   const int32_t *__restrict__ src, const int32_t *__restrict__ cls_slot,
                                                   const int32_t *__restrict__ cls_nkv, const double *__restrict__ ops,
                                                   const double *__restrict__ M, double *L, int ncp, Geo g,
                                                   const int32_t *__restrict__ lev) {
    extern __shared__ double xs[];           // the source box's leading coefficients
    const int tid = threadIdx.x;
    for (int64_t i = blockIdx.x; i < npairs; i += gridDim.x) {
        const uint32_t T = (uint32_t)(key[i] >> 12);
        if (i > 0 && (uint32_t)(key[i - 1] >> 12) == T) continue;      // uniform: not the box's first pair
        double acc[kSmallRows];
#pragma unroll
        for (int q = 0; q < kSmallRows; ++q) acc[q] = 0.0;
        for (int64_t j = i; j < npairs && (uint32_t)(key[j] >> 12) == T; ++j) {
            const int cls = (int)(key[j] & 0xfffu);
            const int nkv = cls_nkv[cls];
            const double *__restrict__ op = ops + (int64_t)cls_slot[cls] * ncp * ncp;
            const double *__restrict__ x = M + (int64_t)src[j] * ncp;
            __syncthreads();                 // the previous pair is done with xs
            for (int k = tid; k < nkv; k += 256) xs[k] = x[k];
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kSmallRows; ++q) {
                const int r = tid + 256 * q;
                if (r < nkv) {
                    double sum = 0.0;
                    for (int k = 0; k < nkv; ++k) sum = fma(op[(int64_t)k * ncp + r], xs[k], sum);
                    acc[q] += sum;
                }
            }
        }
        const double sc = 1.0 / box_side(g.root, g.bmesh, (int32_t)T, lev[T]);
        double *y = L + (int64_t)T * ncp;
#pragma unroll
        for (int q = 0; q < kSmallRows; ++q) {
            const int r = tid + 256 * q;
            if (r < ncp) y[r] += sc * acc[q];
        }
    }
}

// keys (T << 12 | class) and sources of the pairs of the small classes:
// block b copies class b's segment [beg[b], beg[b] + n[b]) of the class-sorted
// M2L list to out + off[b]
__global__ void k_small_pairs(const int64_t *__restrict__ beg, const int64_t *__restrict__ off,
                              const int32_t *__restrict__ cls, const uint64_t *__restrict__ mkey,
                              const int32_t *__restrict__ mval, uint64_t *okey, int32_t *oval) {
    const int b = blockIdx.x;
    const int64_t b0 = beg[b], o0 = off[b], n = off[b + 1] - off[b];
    for (int64_t j = threadIdx.x; j < n; j += blockDim.x) {
        const uint32_t T = (uint32_t)(mkey[b0 + j] & 0xffffffffu);
        okey[o0 + j] = ((uint64_t)T << 12) | (uint64_t)cls[b];
        oval[o0 + j] = mval[b0 + j];
    }
}

// ------------------------------------------------------------------- M2L
// A translation over v = (x, y, z) is a rotation about z by the angle of
// (x, y), the translation over (rho, 0, |z|), rho = |(x, y)|, and the rotation
// back; a negative z adds the signs (-1)^(n+m) on both sides:
//     L_k^l = e^{-i l phi} s_kl sum_{n,m} A(k,l,n,m) s_nm e^{i m phi} M_n^m.
// With y = 0 the operator A is real, so it acts on the Re and on the Im parts
// apart: two products of half the rows and columns, i.e. half the operations
// of the full matrix, and one operator serves every class of equal x^2 + y^2
// and |z| (a "group": up to 16 classes, 60 to 70 groups where there were 850
// classes at order 26).  The rotations are applied where the columns are
// staged and where the products are stored.
//
// Pairs are sorted by (block of target boxes, group, class, box).  k_m2l takes
// 64 pairs of one group x 64 rows (both halves) per workgroup and leaves each
// pair's product in its own slot of Y; k_m2l_sum adds the products of a box in
// rank order.  One launch of each per block, where one launch per class left
// the chip idle between (and inside) thousands of short launches: 850 of them
// took 14 ms of two streams for the 17 428 pairs of a 1728-triangle skeleton,
// which are 0.3 ms of work.
struct M2LArgs {
    const uint64_t *key;        // sorted: (block << (kRankBits + shift)) | (rank << shift) | low bits of T
    const int32_t *src;         // source box
    const int32_t *ts;          // tile t holds the pairs ts[t] .. ts[t + 1) (at most kPairs, one group)
    int tile0, ntiles;          // tiles of the block
    int64_t p0;                 // first pair of the block
    int shift, rowtiles;
    const int32_t *info;        // per rank: group | angle << 10 | reflected << 18
    const int32_t *grp;         // per group: slot, rows (q) and coefficients (real layout) of its order
    const double *ops;          // slot: Re and Im halves, each ldk x ldr, k-major
    int ldk, ldr;
    const double2 *trig;        // (cos, sin) of m times the angle, m = 0 .. p, per angle
    int p1;                     // p + 1
    const int32_t *qtab;        // q -> index of Im (Re at m = 0) | m << 16 | n << 24; 0xffff past the order
    const double *M;
    int ncp;
    double2 *Y;                 // products, ystride (Re, Im) pairs per pair of boxes
    int ystride;
};

constexpr int kRankBits = 12;
constexpr int kPairs = 64;      // pairs per tile
constexpr int kQ = 64;          // rows (both halves) per workgroup
constexpr int kKQ = 8;          // columns per staged block
constexpr int kLd = kQ + 1;     // LDS row length
static_assert(kNClass <= (1 << kRankBits), "the rank takes kRankBits bits of the key");

__device__ __forceinline__ int rank_of(uint64_t key, int shift) { return (int)(key >> shift) & ((1 << kRankBits) - 1); }

// Bound by the FP64 matrix cores.  64 rows x 64 pairs of both halves: wave w
// owns 16 pairs and NS + NS accumulator tiles of 16 x 16 (NS = 4 but for the
// last rows of a group).  The next block of kKQ columns is loaded into
// registers while the MFMAs of the current one run.
template <int NS>
__device__ __forceinline__ void m2l_tile(const M2LArgs &a, int i0, int i1, int r0, int nq, int nkv, int slot,
                                         double (&AR)[kKQ][kLd], double (&AI)[kKQ][kLd],
                                         double (&BR)[kKQ][kLd], double (&BI)[kKQ][kLd]) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t per_op = (int64_t)a.ldk * a.ldr;
    // staging of the operator: column ak, ak + 4, rows ar
    const int ak = threadIdx.x / kQ, ar = threadIdx.x % kQ;
    const double *__restrict__ opr = a.ops + 2 * (int64_t)slot * per_op + (int64_t)ak * a.ldr + r0 + ar;
    const double *__restrict__ opi = opr + per_op;
    // staging of the columns: pair bc, rows bq, bq + 1 of the block
    const int bc = threadIdx.x >> 2, bq = (threadIdx.x & 3) * 2;
    const bool live = i0 + bc < i1;
    const int jb = live ? i0 + bc : i0;
    const int binfo = a.info[rank_of(a.key[jb], a.shift)];
    const double *__restrict__ x = a.M + (int64_t)a.src[jb] * a.ncp;
    const double2 *__restrict__ bt = a.trig + (int64_t)((binfo >> 10) & 255) * a.p1;
    const int bflip = binfo >> 18;
    double va[4], vb[4];
    int fn[2], fm[2];                                      // (n, m) of the q that is fetched next
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        fn[i] = 0;
        fm[i] = bq + i;
        while (fm[i] > fn[i]) fm[i] -= ++fn[i];
    }
    auto fetch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            va[2 * i] = opr[(int64_t)(k0 + 4 * i) * a.ldr];
            va[2 * i + 1] = opi[(int64_t)(k0 + 4 * i) * a.ldr];
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int n = fn[i], m = fm[i], off = fmm::iim(n, m), ore = m ? off - 1 : off;
            // the order's leading nkv coefficients
            const double vr = live && ore < nkv ? x[ore] : 0.0, vi = live && m && off < nkv ? x[off] : 0.0;
            double2 cs = bt[m < a.p1 ? m : 0];
            if (bflip & (n + m)) cs = double2{-cs.x, -cs.y};
            fm[i] += kKQ;
            while (fm[i] > fn[i]) fm[i] -= ++fn[i];
            vb[2 * i] = cs.x * vr - cs.y * vi;
            vb[2 * i + 1] = cs.y * vr + cs.x * vi;
        }
    };
    d4 cr[NS], ci[NS];
#pragma unroll
    for (int i = 0; i < NS; ++i) cr[i] = ci[i] = d4{0.0, 0.0, 0.0, 0.0};
    fetch(0);
    for (int k0 = 0; k0 < nq; k0 += kKQ) {
        __syncthreads();                                   // previous block's MFMAs are done with LDS
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            AR[ak + 4 * i][ar] = va[2 * i];
            AI[ak + 4 * i][ar] = va[2 * i + 1];
            BR[bq + i][bc] = vb[2 * i];
            BI[bq + i][bc] = vb[2 * i + 1];
        }
        __syncthreads();
        if (k0 + kKQ < nq) fetch(k0 + kKQ);
#pragma unroll
        for (int kk = 0; kk < kKQ; kk += 4) {
            const double vr = BR[kk + (lane >> 4)][16 * w + (lane & 15)], vi = BI[kk + (lane >> 4)][16 * w + (lane & 15)];
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                cr[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(AR[kk + (lane >> 4)][16 * i + (lane & 15)], vr, cr[i], 0, 0, 0);
                ci[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(AI[kk + (lane >> 4)][16 * i + (lane & 15)], vi, ci[i], 0, 0, 0);
            }
        }
    }
    const int j = i0 + 16 * w + (lane & 15);
    if (j >= i1) return;
    const int info = a.info[rank_of(a.key[j], a.shift)];
    const double2 *__restrict__ tr = a.trig + (int64_t)((info >> 10) & 255) * a.p1;
    const int flip = info >> 18;
    double2 *__restrict__ y = a.Y + (j - a.p0) * a.ystride;
    // v_mfma_f64_16x16x4f64 accumulator: register q of lane l holds row (l/16) + 4q, column l%16
#pragma unroll
    for (int i = 0; i < NS; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row = r0 + 16 * i + (lane >> 4) + 4 * q;
            if (row >= nq) continue;
            const int t = a.qtab[row], off = t & 0xffff, m = (t >> 16) & 0xff;
            double2 cs = tr[m];
            if (flip & ((t >> 24) + m)) cs = double2{-cs.x, -cs.y};
            const double re = cs.x * cr[i][q] + cs.y * ci[i][q], im = cs.x * ci[i][q] - cs.y * cr[i][q];
            y[row] = double2{(m ? off - 1 : off) < nkv ? re : 0.0, off < nkv ? im : 0.0};
        }
}

// Workgroups go to the 8 XCDs in turn; the work is dealt in runs of kXcdTiles
// tiles per XCD, so that the row tiles of one tile and its neighbours (same
// operator) share an L2.  Longer runs would leave XCDs idle: the far groups
// have a fifth of the near groups' work (2e5 graded triangles, order 26: 24 ms
// with one run per XCD, 14.6 ms with these).
constexpr int kXcdTiles = 8;
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_m2l(M2LArgs a) {
    __shared__ double AR[kKQ][kLd], AI[kKQ][kLd], BR[kKQ][kLd], BI[kKQ][kLd];
    const int run = kXcdTiles * a.rowtiles, i = (int)(blockIdx.x >> 3);
    const int rt = i % run, tl = (i / run * 8 + (int)(blockIdx.x & 7)) * kXcdTiles + rt / a.rowtiles;
    if (tl >= a.ntiles) return;
    const int tile = a.tile0 + tl, r0 = (rt % a.rowtiles) * kQ;
    const int i0 = a.ts[tile], i1 = a.ts[tile + 1];
    const int grp = a.info[rank_of(a.key[i0], a.shift)] & 1023;
    const int slot = a.grp[3 * grp], nq = a.grp[3 * grp + 1], nkv = a.grp[3 * grp + 2];
    if (r0 >= nq) return;
    switch ((nq - r0 + 15) / 16) {                         // uniform
        case 1: m2l_tile<1>(a, i0, i1, r0, nq, nkv, slot, AR, AI, BR, BI); break;
        case 2: m2l_tile<2>(a, i0, i1, r0, nq, nkv, slot, AR, AI, BR, BI); break;
        case 3: m2l_tile<3>(a, i0, i1, r0, nq, nkv, slot, AR, AI, BR, BI); break;
        default: m2l_tile<4>(a, i0, i1, r0, nq, nkv, slot, AR, AI, BR, BI); break;
    }
}

// Local expansion of box b0 + blockIdx.x: its pairs' products added in rank
// order, times 1 / side; boxes without pairs and the padding get zeros.
// Bound by reading Y (16 bytes per row and pair, coalesced).
__global__ __launch_bounds__(256) void k_m2l_sum(M2LArgs a, int64_t b0, const int32_t *__restrict__ beg,
                                                 const int32_t *__restrict__ end, const int32_t *__restrict__ list,
                                                 int nqmax, Geo g, const int32_t *__restrict__ lev, double *L) {
    __shared__ int spair[256], snq[256];
    const int64_t T = b0 + blockIdx.x;
    const int e0 = beg[T], e1 = end[T], tid = threadIdx.x;
    const double sc = 1.0 / box_side(g.root, g.bmesh, (int32_t)T, lev[T]);
    double *__restrict__ l = L + T * a.ncp;
    for (int q0 = 0; q0 < nqmax; q0 += 256) {
        const int q = q0 + tid;
        double re = 0.0, im = 0.0;
        for (int e = e0; e < e1; e += 256) {
            const int n = min(256, e1 - e);
            __syncthreads();
            if (tid < n) {
                const int j = list[e + tid];
                spair[tid] = (int)(j - a.p0);
                snq[tid] = a.grp[3 * (a.info[rank_of(a.key[j], a.shift)] & 1023) + 1];
            }
            __syncthreads();
#pragma unroll 4
            for (int k = 0; k < n; ++k)
                if (q < snq[k]) {
                    const double2 v = a.Y[(int64_t)spair[k] * a.ystride + q];
                    re += v.x;
                    im += v.y;
                }
        }
        if (q < nqmax) {
            const int t = a.qtab[q], off = t & 0xffff, m = (t >> 16) & 0xff;
            l[m ? off - 1 : off] = sc * re;
            if (m) l[off] = sc * im;
        }
    }
    const int nc = a.p1 * a.p1;
    if (nc + tid < a.ncp) l[nc + tid] = 0.0;               // ncp - nc < 16
}

// plan: keys by (block, rank, box) from the emitted (class << 32 | T); word 0: the count
__global__ void k_m2l_rekey(int64_t n, const int32_t *__restrict__ rank, int shift, uint64_t *key, int32_t *word) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *word = (int32_t)n;
    if (i >= n) return;
    const uint32_t cls = (uint32_t)(key[i] >> 32), T = (uint32_t)key[i];
    key[i] = ((uint64_t)(T >> shift) << (kRankBits + shift)) | ((uint64_t)rank[cls] << shift) |
             (T & ((1u << shift) - 1u));
}

// the same keys for blocks of 2^to boxes instead of 2^from, to < from
__global__ void k_m2l_reshift(int64_t n, int from, int to, uint64_t *key, int32_t *word) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *word = (int32_t)n;
    if (i >= n) return;
    const uint64_t k = key[i], rank = (k >> from) & ((1u << kRankBits) - 1u);
    const uint64_t T = (k >> (kRankBits + from) << from) | (k & ((1ull << from) - 1ull));
    key[i] = ((T >> to) << (kRankBits + to)) | (rank << to) | (T & ((1ull << to) - 1ull));
}

// Sorted pairs: tile heads (every kPairs-th pair of a (block, group) segment,
// the segment starting at the first key with its block and its group's lowest
// rank), the groups in use, the first pair of every block, and the pairs
// keyed by target box for the sums
__global__ void k_m2l_mark(int64_t n, const uint64_t *__restrict__ key, int shift, int nblk,
                           const int32_t *__restrict__ info, const int32_t *__restrict__ grp_rank, int32_t *flag,
                           int32_t *pos, int32_t *used, int32_t *blk, uint64_t *tkey, int32_t *tval) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t k = key[i];
    const int64_t b = (int64_t)(k >> (kRankBits + shift)), bp = i > 0 ? (int64_t)(key[i - 1] >> (kRankBits + shift)) : -1;
    for (int64_t q = bp + 1; q <= b; ++q) blk[q] = (int32_t)i;
    if (i == n - 1)
        for (int64_t q = b + 1; q <= nblk; ++q) blk[q] = (int32_t)n;
    const int g = info[rank_of(k, shift)] & 1023;
    const uint64_t first = ((uint64_t)b << (kRankBits + shift)) | ((uint64_t)grp_rank[g] << shift);
    int64_t lo = 0, hi = i;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (key[mid] < first) lo = mid + 1; else hi = mid;
    }
    if (lo == i) used[g] = 1;
    flag[i] = (i - lo) % kPairs == 0 ? 1 : 0;
    pos[i] = (int32_t)i;
    tkey[i] = ((uint64_t)b << shift) | (k & ((1ull << shift) - 1ull));
    tval[i] = (int32_t)i;
}

// first tile of every block, and the end of the tile list
__global__ void k_m2l_blk_tiles(int nblk, const int32_t *__restrict__ blk, const int32_t *__restrict__ ntiles,
                                int32_t n, int32_t *ts, int32_t *blk_tile) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b > nblk) return;
    const int nt = *ntiles;
    if (b == 0) ts[nt] = n;
    int lo = 0, hi = nt;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ts[mid] < blk[b]) lo = mid + 1; else hi = mid;
    }
    blk_tile[b] = lo;
}

__global__ void k_m2l_ranges(int64_t n, const uint64_t *__restrict__ key, int32_t *beg, int32_t *end) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t T = key[i];
    if (i == 0 || key[i - 1] != T) beg[T] = (int32_t)i;
    if (i == n - 1 || key[i + 1] != T) end[T] = (int32_t)(i + 1);
}

// class index -> offset vector
void class_vec(int cls, double v[3]) {
    const int W = 2 * kR + 1;
    v[0] = cls / (W * W) - kR;
    v[1] = (cls / W) % W - kR;
    v[2] = cls % W - kR;
}

// Order of the M2L of displacement class v (in box sides, |v|^2 >= K): the
// truncation error of the translation of a box's multipole to a same-size box
// at centre distance |v| falls like r^(p+1), r = a / |v|, a = sqrt(3)/2 the
// half-diagonal (on the octree workloads the error at the closest class
// follows this rate: p = 18 mixed loses 1.5e-7 at |v| = 2).  A class farther
// than the closest admissible one (|v| = sqrt(K)) reaches the same error at a
// lower order; kM2lMargin orders are kept on top.
constexpr int kM2lMargin = 2;

int m2l_order(int p, int K, const double v[3]) {
    const double a = 0.8660254037844386;
    const double d = std::sqrt(v[0] * v[0] + v[1] * v[1] + v[2] * v[2]);
    const double r0 = a / std::sqrt((double)K), r = a / d;
    if (!(r < r0)) return p;
    const int pv = (int)std::ceil((p + 1) * std::log(r0) / std::log(r)) - 1 + kM2lMargin;
    return std::min(p, std::max(pv, 4));
}

void build_ops(Ctx &c, int kind, int nops, const std::vector<double> &vecs, int p, int ncp, double *dst) {
    const int order = kind == 0 ? 2 * p : p;
    const int stride = fmm::tri(order, order) + 1;
    DBuf dv, tabs;
    dv.ensure(sizeof(double) * 3 * nops);
    tabs.ensure(sizeof(cd) * (size_t)stride * nops);
    LSS_HIP(hipMemcpyAsync(dv.p, vecs.data(), sizeof(double) * 3 * nops, hipMemcpyHostToDevice, c.stream));
    hipLaunchKernelGGL(k_op_tables, dim3(grid_for(nops, 64)), dim3(64), 0, c.stream, nops, dv.as<double>(), order,
                       kind == 0 ? 1 : 0, stride, tabs.as<cd>());
    LSS_CHECK_LAUNCH("k_op_tables");
    const int64_t per = (int64_t)ncp * ncp;
    hipLaunchKernelGGL(k_fill_op, dim3(grid_for(per), nops), dim3(kBlk), 0, c.stream, kind, p, ncp, nops,
                       tabs.as<cd>(), stride, dst);
    LSS_CHECK_LAUNCH("k_fill_op");
    LSS_HIP(hipStreamSynchronize(c.stream));
}

// The displacement classes ordered by group (equal x^2 + y^2 and |z|): rank of
// each class, and per rank its group, angle index and reflection.
struct M2LClasses {
    int ngroups = 0;
    std::vector<int32_t> rank, info, grp_rank;     // per class; per rank; lowest rank of each group
    std::vector<double> vec;                       // per group: (rho, 0, |z|)
    M2LClasses() {
        const int W = 2 * kR + 1;
        std::map<std::pair<int, int>, std::vector<int>> by;
        for (int cls = 0; cls < kNClass; ++cls) {
            double v[3];
            class_vec(cls, v);
            by[{(int)(v[0] * v[0] + v[1] * v[1]), (int)std::fabs(v[2])}].push_back(cls);
        }
        ngroups = (int)by.size();
        rank.assign(kNClass, 0);
        info.assign(kNClass, 0);
        int r = 0, g = 0;
        for (const auto &e : by) {
            grp_rank.push_back(r);
            vec.insert(vec.end(), {std::sqrt((double)e.first.first), 0.0, (double)e.first.second});
            for (int cls : e.second) {
                double v[3];
                class_vec(cls, v);
                rank[cls] = r;
                info[r] = g | (((int)v[0] + kR) * W + (int)v[1] + kR) << 10 | (v[2] < 0.0 ? 1 << 18 : 0);
                ++r;
            }
            ++g;
        }
    }
};
const M2LClasses &m2l_classes() {
    static const M2LClasses k;
    return k;
}
static_assert((2 * kR + 1) * (2 * kR + 1) <= 256, "the angle index takes 8 bits of a rank's info");

// The M2L plan of the emitted list: pairs sorted by (block, rank, box), tiles,
// and each box's pairs.  A block holds 2^shift target boxes, as many as keep
// the products of an average block near kM2LBytes: large enough to fill the
// chip several times over (about 1e5 pairs), small enough that the expansions
// of a block's sources stay in the caches between its groups.  Blocks of a
// surface's tree differ little (the fullest holds at most 1.2 times the mean's
// pairs on the graded surfaces measured), but boxes without pairs pull the mean
// down: where the fullest block would take more than twice kM2LBytes the
// blocks are halved and the pairs sorted again, until it does not or a block
// is one box.  (4096 boxes of a volume's triangles beside 36 000 boxes of small
// meshes, order 26: 8.2 GiB before.)
constexpr double kM2LBytes = 1024.0 * 1024.0 * 1024.0;

void m2l_plan(Ctx &c) {
    Tree &t = c.tree;
    const int64_t n = t.n_m2l;
    if (n == 0) return;
    const M2LClasses &cl = m2l_classes();
    const int p = t.p;
    const double pair_bytes = 8.0 * (p + 1) * (p + 2);     // at most: the highest order's rows
    const double per_box = (double)n / (double)t.nboxes * pair_bytes;
    int shift = 0;
    while ((int64_t(1) << shift) < t.nboxes && 2.0 * per_box * (double)(int64_t(1) << shift) <= kM2LBytes) ++shift;
    if (!t.m2l_tab.p) {
        t.m2l_tab.ensure(4 * (2 * kNClass + cl.ngroups));
        LSS_HIP(hipMemcpyAsync(t.m2l_tab.p, cl.rank.data(), 4 * kNClass, hipMemcpyHostToDevice, c.stream));
        LSS_HIP(hipMemcpyAsync(t.m2l_tab.as<int32_t>() + kNClass, cl.info.data(), 4 * kNClass, hipMemcpyHostToDevice,
                               c.stream));
        LSS_HIP(hipMemcpyAsync(t.m2l_tab.as<int32_t>() + 2 * kNClass, cl.grp_rank.data(), 4 * cl.ngroups,
                               hipMemcpyHostToDevice, c.stream));
    }
    const int32_t *rank = t.m2l_tab.as<int32_t>(), *info = rank + kNClass, *grp_rank = info + kNClass;
    t.m2l_key2.ensure(8 * n);
    t.m2l_val2.ensure(4 * n);
    // own sort workspace (the near lists are sorted on the other stream meanwhile)
    const size_t stb = sort_pairs_u64_tmp_bytes(n);
    t.m2l_tmp.ensure(stb);
    t.m2l_flag.ensure(4 * n);
    t.m2l_pos.ensure(4 * n);
    t.m2l_ts.ensure(4 * (n + 1));
    t.m2l_csr_key.ensure(8 * n);
    t.m2l_csr_key2.ensure(8 * n);
    t.m2l_csr.ensure(4 * n);
    t.m2l_csr2.ensure(4 * n);
    t.m2l_bsum.ensure(4 * ((size_t)compact_blocks(n) + 2));
    for (int from = -1;;) {
        const int nblk = (int)((t.nboxes - 1) >> shift) + 1;
        // meta: used flag per group, first pair per block (+ end), first tile per block (+ end), count, tiles
        const int64_t nmeta = cl.ngroups + 2 * ((int64_t)nblk + 1) + 2;
        t.m2l_meta.ensure(4 * nmeta);
        int32_t *used = t.m2l_meta.as<int32_t>(), *blk = used + cl.ngroups, *blk_tile = blk + nblk + 1,
                *count = blk_tile + nblk + 1, *ntiles = count + 1;
        LSS_HIP(hipMemsetAsync(used, 0, 4 * cl.ngroups, c.stream));
        if (from < 0)
            hipLaunchKernelGGL(k_m2l_rekey, dim3(grid_for(n)), dim3(kBlk), 0, c.stream, n, rank, shift,
                               t.m2l_key.as<uint64_t>(), count);
        else
            hipLaunchKernelGGL(k_m2l_reshift, dim3(grid_for(n)), dim3(kBlk), 0, c.stream, n, from, shift,
                               t.m2l_key.as<uint64_t>(), count);
        int bb = 1;
        while ((int64_t(1) << bb) < nblk) ++bb;
        sort_pairs_u64(t.m2l_tmp.p, stb, t.m2l_key.as<uint64_t>(), t.m2l_key2.as<uint64_t>(), t.m2l_val.as<int32_t>(),
                       t.m2l_val2.as<int32_t>(), n, 0, kRankBits + shift + bb, c.stream);
        hipLaunchKernelGGL(k_m2l_mark, dim3(grid_for(n)), dim3(kBlk), 0, c.stream, n, t.m2l_key2.as<uint64_t>(), shift,
                           nblk, info, grp_rank, t.m2l_flag.as<int32_t>(), t.m2l_pos.as<int32_t>(), used, blk,
                           t.m2l_csr_key.as<uint64_t>(), t.m2l_csr.as<int32_t>());
        LSS_CHECK_LAUNCH("k_m2l_mark");
        compact_flags(c, n, count, t.m2l_flag.as<int32_t>(), t.m2l_pos.as<int32_t>(), t.m2l_ts.as<int32_t>(), ntiles,
                      t.m2l_bsum.as<int32_t>());
        hipLaunchKernelGGL(k_m2l_blk_tiles, dim3(grid_for(nblk + 1)), dim3(kBlk), 0, c.stream, nblk, blk, ntiles,
                           (int32_t)n, t.m2l_ts.as<int32_t>(), blk_tile);
        LSS_CHECK_LAUNCH("k_m2l_blk_tiles");
        std::vector<int32_t> h(cl.ngroups + 2 * ((size_t)nblk + 1));
        LSS_HIP(hipMemcpyAsync(h.data(), used, 4 * h.size(), hipMemcpyDeviceToHost, c.stream));
        // the pairs of every box, in rank order (the sort is stable)
        int tb = 1;
        while ((int64_t(1) << tb) < t.nboxes) ++tb;
        sort_pairs_u64(t.m2l_tmp.p, stb, t.m2l_csr_key.as<uint64_t>(), t.m2l_csr_key2.as<uint64_t>(),
                       t.m2l_csr.as<int32_t>(), t.m2l_csr2.as<int32_t>(), n, 0, tb, c.stream);
        t.m2l_beg.ensure(4 * t.nboxes);
        t.m2l_end.ensure(4 * t.nboxes);
        LSS_HIP(hipMemsetAsync(t.m2l_beg.p, 0, 4 * t.nboxes, c.stream));
        LSS_HIP(hipMemsetAsync(t.m2l_end.p, 0, 4 * t.nboxes, c.stream));
        hipLaunchKernelGGL(k_m2l_ranges, dim3(grid_for(n)), dim3(kBlk), 0, c.stream, n, t.m2l_csr_key2.as<uint64_t>(),
                           t.m2l_beg.as<int32_t>(), t.m2l_end.as<int32_t>());
        LSS_CHECK_LAUNCH("k_m2l_ranges");
        LSS_HIP(hipStreamSynchronize(c.stream));
        t.m2l_shift = shift;
        t.m2l_used.clear();
        for (int g = 0; g < cl.ngroups; ++g)
            if (h[g]) t.m2l_used.push_back(g);
        t.m2l_blk.assign(h.begin() + cl.ngroups, h.begin() + cl.ngroups + nblk + 1);
        t.m2l_blk_tile.assign(h.begin() + cl.ngroups + nblk + 1, h.end());
        int64_t most = 0;
        for (int b = 0; b < nblk; ++b) most = std::max(most, t.m2l_blk[b + 1] - t.m2l_blk[b]);
        double over = (double)most * pair_bytes / (2.0 * kM2LBytes);
        if (over <= 1.0 || shift == 0) return;
        for (from = shift; over > 1.0 && shift > 0; over *= 0.5) --shift;
    }
}

// M2L of every pair: t.L from t.M (written whole), operators of the groups in
// use built first where they are missing.  Each group runs at the order that
// its distance needs (m2l_order): the leading rows and columns of its operator.
void m2l_pass(Ctx &c, int p, int ncp) {
    Tree &t = c.tree;
    if (t.n_m2l == 0) {
        launch_fill_zero(c, t.L.as<double>(), t.nboxes * (int64_t)ncp);
        return;
    }
    const M2LClasses &cl = m2l_classes();
    const int nqmax = (p + 1) * (p + 2) / 2;
    const int ldk = (int)ceil_div(nqmax, kKQ) * kKQ, ldr = (int)ceil_div(nqmax, kQ) * kQ;
    const int64_t per = 2 * (int64_t)ldk * ldr;            // both halves
    if (t.m2l_p != p) {     // index table, rotations by every angle: ((x + i y) / rho)^m in extended precision
        std::vector<int32_t> qtab(ldk, 0xffff);            // padding: past every order
        for (int n = 0; n <= p; ++n)
            for (int m = 0; m <= n; ++m)
                qtab[fmm::tri(n, m)] = (m ? fmm::iim(n, m) : fmm::ire(n, 0)) | m << 16 | n << 24;
        const int W = 2 * kR + 1;
        std::vector<double> trig((size_t)2 * W * W * (p + 1));
        for (int k = 0; k < W * W; ++k) {
            const long double x = k / W - kR, y = k % W - kR, rho = std::sqrt(x * x + y * y);
            const long double cx = rho > 0 ? x / rho : 1.0L, sx = rho > 0 ? y / rho : 0.0L;
            long double cm = 1.0L, sm = 0.0L;
            for (int m = 0; m <= p; ++m) {
                trig[2 * ((size_t)k * (p + 1) + m)] = (double)cm;
                trig[2 * ((size_t)k * (p + 1) + m) + 1] = (double)sm;
                const long double q = cm * cx - sm * sx;
                sm = sm * cx + cm * sx;
                cm = q;
            }
        }
        t.m2l_qtab.ensure(4 * qtab.size());
        t.m2l_trig.ensure(8 * trig.size());
        LSS_HIP(hipMemcpyAsync(t.m2l_qtab.p, qtab.data(), 4 * qtab.size(), hipMemcpyHostToDevice, c.stream));
        LSS_HIP(hipMemcpyAsync(t.m2l_trig.p, trig.data(), 8 * trig.size(), hipMemcpyHostToDevice, c.stream));
        LSS_HIP(hipStreamSynchronize(c.stream));           // the host tables end here
        t.op_group_slot.assign(cl.ngroups, -1);
        t.m2l_p = p;
    }
    std::vector<int> need;
    int have = 0;
    for (int s : t.op_group_slot) have += s >= 0;
    for (int g : t.m2l_used)
        if (t.op_group_slot[g] < 0) need.push_back(g);
    if (!need.empty()) {
        t.opM2G.grow_copy(sizeof(double) * (size_t)(have + (int64_t)need.size()) * per,
                          sizeof(double) * (size_t)have * per, c.stream);
        const int nops = (int)need.size(), order = 2 * p, stride = fmm::tri(order, order) + 1;
        std::vector<double> v;
        for (int g : need) v.insert(v.end(), cl.vec.begin() + 3 * g, cl.vec.begin() + 3 * g + 3);
        DBuf dv, tabs;
        dv.ensure(8 * v.size());
        tabs.ensure(sizeof(cd) * (size_t)stride * nops);
        LSS_HIP(hipMemcpyAsync(dv.p, v.data(), 8 * v.size(), hipMemcpyHostToDevice, c.stream));
        hipLaunchKernelGGL(k_m2l_tables, dim3(grid_for((int64_t)nops * (order + 1), 64)), dim3(64), 0, c.stream, nops,
                           dv.as<double>(), order, stride, tabs.as<cd>());
        hipLaunchKernelGGL(k_fill_m2l, dim3(grid_for((int64_t)ldk * ldr), 2 * nops), dim3(kBlk), 0, c.stream, p, ldk,
                           ldr, nops, tabs.as<cd>(), stride, t.m2l_qtab.as<int32_t>(),
                           t.opM2G.as<double>() + (int64_t)have * per);
        LSS_CHECK_LAUNCH("k_fill_m2l");
        LSS_HIP(hipStreamSynchronize(c.stream));
        for (int g : need) t.op_group_slot[g] = have++;
    }
    // slot, rows and coefficients of every group in use (K may change between
    // builds): the leading coefficients in and out, (p_v + 1)^2 rounded up to
    // 16 in the real layout, and the q whose Re is among them
    t.h_m2l_grp.assign(3 * cl.ngroups, 0);
    int rowmax = 0;
    for (int g : t.m2l_used) {
        const int pv = m2l_order(p, t.K, &cl.vec[3 * g]);
        const int nkv = std::min((p + 1) * (p + 1), (int)ceil_div((int64_t)(pv + 1) * (pv + 1), kKB) * kKB);
        int nq = 0;
        for (int n = 0; n <= p; ++n)
            for (int m = 0; m <= n; ++m)
                if (fmm::ire(n, m) < nkv) nq = fmm::tri(n, m) + 1;
        t.h_m2l_grp[3 * g] = t.op_group_slot[g];
        t.h_m2l_grp[3 * g + 1] = nq;
        t.h_m2l_grp[3 * g + 2] = nkv;
        rowmax = std::max(rowmax, nq);
    }
    t.m2l_grp.ensure(4 * t.h_m2l_grp.size());
    LSS_HIP(hipMemcpyAsync(t.m2l_grp.p, t.h_m2l_grp.data(), 4 * t.h_m2l_grp.size(), hipMemcpyHostToDevice, c.stream));
    // a launch takes as many blocks as the products of the fullest one hold
    const int nblk = (int)t.m2l_blk.size() - 1;
    int64_t most = 0;
    for (int b = 0; b < nblk; ++b) most = std::max(most, t.m2l_blk[b + 1] - t.m2l_blk[b]);
    std::vector<int> cut{0};
    for (int b = 1; b <= nblk; ++b)
        if (b == nblk || t.m2l_blk[b + 1] - t.m2l_blk[cut.back()] > most) cut.push_back(b);
    t.m2l_y.ensure(sizeof(double2) * (size_t)most * rowmax);
    M2LArgs a;
    a.key = t.m2l_key2.as<uint64_t>();
    a.src = t.m2l_val2.as<int32_t>();
    a.ts = t.m2l_ts.as<int32_t>();
    a.shift = t.m2l_shift;
    a.rowtiles = (int)ceil_div(rowmax, kQ);
    a.info = t.m2l_tab.as<int32_t>() + kNClass;
    a.grp = t.m2l_grp.as<int32_t>();
    a.ops = t.opM2G.as<double>();
    a.ldk = ldk;
    a.ldr = ldr;
    a.trig = t.m2l_trig.as<double2>();
    a.p1 = p + 1;
    a.qtab = t.m2l_qtab.as<int32_t>();
    a.M = t.M.as<double>();
    a.ncp = ncp;
    a.Y = t.m2l_y.as<double2>();
    a.ystride = rowmax;
    const Geo g{t.root.as<double>(), t.bmesh.as<int32_t>()};
    for (size_t k = 0; k + 1 < cut.size(); ++k) {
        a.tile0 = t.m2l_blk_tile[cut[k]];
        a.ntiles = t.m2l_blk_tile[cut[k + 1]] - a.tile0;
        a.p0 = t.m2l_blk[cut[k]];
        if (a.ntiles > 0) {
            const int64_t wg = ceil_div(a.ntiles, 8 * kXcdTiles) * 8 * kXcdTiles * a.rowtiles;
            hipLaunchKernelGGL(k_m2l, dim3((unsigned)wg), dim3(256), 0, c.stream, a);
        }
        const int64_t b0 = (int64_t)cut[k] << t.m2l_shift,
                      nb = std::min<int64_t>((int64_t)cut[k + 1] << t.m2l_shift, t.nboxes) - b0;
        hipLaunchKernelGGL(k_m2l_sum, dim3((unsigned)nb), dim3(256), 0, c.stream, a, b0, t.m2l_beg.as<int32_t>(),
                           t.m2l_end.as<int32_t>(), t.m2l_csr2.as<int32_t>(), nqmax, g, t.level.as<int32_t>(),
                           t.L.as<double>());
        LSS_CHECK_LAUNCH("k_m2l");
    }
}

}  // namespace

// Expansions at the leaves (P2M) and up the tree (M2M) on c.stream; the
// workspace buffers belong to the caller and must outlive the kernels.
void upward_pass(Ctx &c, int p, int ncp, DBuf &flag, DBuf &ids, DBuf &leaves, DBuf &nleaf) {
    Tree &t = c.tree;
    // expansions
    LSS_HIP(hipMemsetAsync(t.M.p, 0, sizeof(double) * t.nboxes * ncp, c.stream));
    if (!m2l_rotated(c))                                    // m2l_pass writes all of L
        LSS_HIP(hipMemsetAsync(t.L.p, 0, sizeof(double) * t.nboxes * ncp, c.stream));
    Geo g{t.root.as<double>(), t.bmesh.as<int32_t>()};
    // P2M on the non-empty leaves
    flag.ensure(4 * t.nboxes); ids.ensure(4 * t.nboxes); leaves.ensure(4 * t.nboxes); nleaf.ensure(16);
    hipLaunchKernelGGL(k_leaf_flags, dim3(grid_for(t.nboxes)), dim3(kBlk), 0, c.stream, t.nboxes, t.child.as<int32_t>(),
                       t.nb.as<int64_t>(), t.ne.as<int64_t>(), flag.as<int32_t>(), ids.as<int32_t>());
    LSS_CHECK_LAUNCH("k_leaf_flags");
    compact_flags(c, t.nboxes, nullptr, flag.as<int32_t>(), ids.as<int32_t>(), leaves.as<int32_t>(), nleaf.as<int32_t>());
    int32_t nl = 0;
    LSS_HIP(hipMemcpyAsync(&nl, nleaf.p, 4, hipMemcpyDeviceToHost, c.stream));
    LSS_HIP(hipStreamSynchronize(c.stream));
    c.stats.n_leaves = nl;
    if (nl > 0) {
        if (p == 20 || p == 26) {
            auto k = p == 20 ? k_p2m_reg<20> : k_p2m_reg<26>;
            hipLaunchKernelGGL(k, dim3(nl), dim3(64), 0, c.stream, nleaf.as<int32_t>(), leaves.as<int32_t>(), ncp, g,
                               t.level.as<int32_t>(), t.ijk.as<int32_t>(), t.nb.as<int64_t>(), t.ne.as<int64_t>(),
                               t.src.as<Src>(), t.M.as<double>());
            LSS_CHECK_LAUNCH("k_p2m_reg");
        } else {
            const int ntri = (p + 1) * (p + 2) / 2, G = 64 / (p + 1);
            size_t shm = sizeof(double) * (2 * G * ntri + ntri + p + 1);
            hipLaunchKernelGGL(k_p2m_cols, dim3(nl), dim3(64), shm, c.stream, nleaf.as<int32_t>(), leaves.as<int32_t>(),
                               p, ncp, g, t.level.as<int32_t>(), t.ijk.as<int32_t>(), t.nb.as<int64_t>(),
                               t.ne.as<int64_t>(), t.src.as<Src>(), t.M.as<double>());
            LSS_CHECK_LAUNCH("k_p2m_cols");
        }
    }
    // upward pass: M2M from level depth to 1 into their parents
    for (int lvl = t.depth; lvl >= 1; --lvl) {
        const int64_t base = t.level_begin[lvl], npar = (t.level_begin[lvl + 1] - base) / 8;
        GemmArgs a{G_M2M, ncp, 8 * ncp, npar, t.opM2M.as<double>(), t.M.as<double>(), t.M.as<double>(), nullptr,
                   nullptr, base, t.parent.as<int32_t>(), t.level.as<int32_t>(), t.root.as<double>(),
                   t.bmesh.as<int32_t>()};
        gemm(c, a);
    }
}

// M2L class by class, into t.L (cleared before): mixed contexts, and lists
// longer than the plan holds
void m2l_classwise(Ctx &c, int p, int ncp) {
    Tree &t = c.tree;
    const int64_t per = (int64_t)ncp * ncp;
    struct StreamSwap {
        Ctx &c;
        hipStream_t saved;
        ~StreamSwap() { c.stream = saved; }
    };
    {   // M2L operators of the classes in use not built yet
        std::vector<int> need;
        for (int cls : t.class_used)
            if (t.op_class_slot[cls] < 0) need.push_back(cls);
        if (!need.empty()) {
            int have = 0;
            for (int s : t.op_class_slot) have += s >= 0;
            t.opM2L.grow_copy(sizeof(double) * (size_t)(have + need.size()) * per, sizeof(double) * (size_t)have * per,
                              c.stream);
            std::vector<double> v(3 * need.size());
            for (size_t i = 0; i < need.size(); ++i) class_vec(need[i], &v[3 * i]);
            build_ops(c, 0, (int)need.size(), v, p, ncp, t.opM2L.as<double>() + (int64_t)have * per);
            for (size_t i = 0; i < need.size(); ++i) t.op_class_slot[need[i]] = have + (int)i;
        }
    }
    // M2L, one launch per displacement class, each at its own order: the
    // leading (p_v + 1)^2 coefficients in and out (the real layout orders them
    // by degree), p_v = m2l_order(p, K, v).  Within a class every target box
    // occurs once, so a launch has no write conflicts; the classes run in two
    // sets, one on each stream, into two accumulators (L, and L2 on the
    // auxiliary stream), so that each stream's launches fill the other's gaps;
    // L += L2 once both are done.  The sets depend only on the class sizes, so
    // every box sums its classes in a fixed order.
    struct M2LJob { int cls; int nkv; int64_t b0, n; };
    std::vector<M2LJob> jobs;
    for (int cls : t.class_used) {
        double v[3];
        class_vec(cls, v);
        const int pv = m2l_order(p, t.K, v);
        const int nkv = std::min(ncp, (int)ceil_div((int64_t)(pv + 1) * (pv + 1), kKB) * kKB);
        jobs.push_back({cls, nkv, t.class_beg[cls], t.class_end[cls] - t.class_beg[cls]});
    }
    // classes with few pairs would be one short launch each (graded meshes use
    // thousands of classes): they go to one target-major launch instead.  That
    // launch reads a class operator once per pair rather than once per tile of
    // pairs, so it pays only while the operators are small (measured: faster
    // at order 20, 441 coefficients; slower at order 26, 729)
    std::vector<M2LJob> small;
    {
        std::vector<M2LJob> big;
        const bool use_small = ncp <= kSmallMaxCoeffs;
        for (const M2LJob &j : jobs) (use_small && j.n <= kSmallClassPairs ? small : big).push_back(j);
        jobs.swap(big);
    }
    std::vector<char> on_aux(jobs.size(), 0);
    {   // largest work first to the less loaded set (ties: the class index)
        std::vector<size_t> ord(jobs.size());
        for (size_t i = 0; i < ord.size(); ++i) ord[i] = i;
        auto work = [&](size_t i) { return (double)jobs[i].n * jobs[i].nkv * jobs[i].nkv; };
        std::stable_sort(ord.begin(), ord.end(), [&](size_t a, size_t b) { return work(a) > work(b); });
        double load[2] = {0.0, 0.0};
        for (size_t i : ord) {
            const int side = load[1] < load[0] ? 1 : 0;
            on_aux[i] = (char)side;
            load[side] += work(i);
        }
    }
    t.L2.ensure(sizeof(double) * t.nboxes * ncp);
    LSS_HIP(hipEventRecord(c.aux_ev[4], c.stream));         // operators built
    auto m2l = [&](const M2LJob &j, double *L) {
        GemmArgs a{G_LIST, ncp, j.nkv, j.n, t.opM2L.as<double>() + (int64_t)t.op_class_slot[j.cls] * per, t.M.as<double>(),
                   L, t.m2l_key2.as<uint64_t>() + j.b0, t.m2l_val2.as<int32_t>() + j.b0, 0,
                   t.parent.as<int32_t>(), t.level.as<int32_t>(), t.root.as<double>(), t.bmesh.as<int32_t>(), j.nkv};
        gemm(c, a);
    };
    {
        StreamSwap swap{c, c.stream};
        c.stream = c.aux_stream;
        LSS_HIP(hipStreamWaitEvent(c.aux_stream, c.aux_ev[4], 0));
        launch_fill_zero(c, t.L2.as<double>(), t.nboxes * (int64_t)ncp);
        for (size_t i = 0; i < jobs.size(); ++i)
            if (on_aux[i]) m2l(jobs[i], t.L2.as<double>());
        LSS_HIP(hipEventRecord(c.aux_ev[5], c.aux_stream));
    }
    if (!small.empty()) {
        // host arrays kept in the tree until the next build: the copies below
        // are asynchronous
        std::vector<int64_t> &hb = t.sm_hb, &ho = t.sm_ho;
        std::vector<int32_t> &hc = t.sm_hc, &hslot = t.sm_hslot, &hnkv = t.sm_hnkv;
        hb.assign(small.size(), 0);
        ho.assign(small.size() + 1, 0);
        hc.assign(small.size(), 0);
        hslot.assign(kNClass, 0);
        hnkv.assign(kNClass, 0);
        for (size_t i = 0; i < small.size(); ++i) {
            hb[i] = small[i].b0;
            hc[i] = small[i].cls;
            ho[i + 1] = ho[i] + small[i].n;
            hslot[small[i].cls] = t.op_class_slot[small[i].cls];
            hnkv[small[i].cls] = small[i].nkv;
        }
        const int64_t nsp = ho.back();
        const size_t ns = small.size();
        t.sm_meta.ensure(sizeof(int64_t) * (2 * ns + 1) + sizeof(int32_t) * (ns + 2 * kNClass));
        char *mp = t.sm_meta.as<char>();
        int64_t *db = reinterpret_cast<int64_t *>(mp), *dofs = db + ns;
        int32_t *dc = reinterpret_cast<int32_t *>(dofs + ns + 1), *dslot = dc + ns, *dnkv = dslot + kNClass;
        LSS_HIP(hipMemcpyAsync(db, hb.data(), sizeof(int64_t) * ns, hipMemcpyHostToDevice, c.stream));
        LSS_HIP(hipMemcpyAsync(dofs, ho.data(), sizeof(int64_t) * (ns + 1), hipMemcpyHostToDevice, c.stream));
        LSS_HIP(hipMemcpyAsync(dc, hc.data(), sizeof(int32_t) * ns, hipMemcpyHostToDevice, c.stream));
        LSS_HIP(hipMemcpyAsync(dslot, hslot.data(), sizeof(int32_t) * kNClass, hipMemcpyHostToDevice, c.stream));
        LSS_HIP(hipMemcpyAsync(dnkv, hnkv.data(), sizeof(int32_t) * kNClass, hipMemcpyHostToDevice, c.stream));
        t.sm_key.ensure(8 * nsp); t.sm_key2.ensure(8 * nsp); t.sm_val.ensure(4 * nsp); t.sm_val2.ensure(4 * nsp);
        hipLaunchKernelGGL(k_small_pairs, dim3((unsigned)ns), dim3(kBlk), 0, c.stream, db, dofs, dc,
                           t.m2l_key2.as<uint64_t>(), t.m2l_val2.as<int32_t>(), t.sm_key.as<uint64_t>(),
                           t.sm_val.as<int32_t>());
        LSS_CHECK_LAUNCH("k_small_pairs");
        int tb = 1;
        while ((int64_t(1) << tb) < t.nboxes) ++tb;
        // own sort workspace: the near lists may be sorted on the other stream meanwhile
        const size_t stb = sort_pairs_u64_tmp_bytes(nsp);
        t.sm_tmp.ensure(stb);
        sort_pairs_u64(t.sm_tmp.p, stb, t.sm_key.as<uint64_t>(), t.sm_key2.as<uint64_t>(), t.sm_val.as<int32_t>(),
                       t.sm_val2.as<int32_t>(), nsp, 0, 12 + tb, c.stream);
        const int64_t gs = std::min<int64_t>(nsp, 65535);
        hipLaunchKernelGGL(k_m2l_small, dim3((unsigned)gs), dim3(256), sizeof(double) * (size_t)ncp, c.stream, nsp,
                           t.sm_key2.as<uint64_t>(), t.sm_val2.as<int32_t>(), dslot, dnkv, t.opM2L.as<double>(),
                           t.M.as<double>(), t.L.as<double>(), ncp, Geo{t.root.as<double>(), t.bmesh.as<int32_t>()},
                           t.level.as<int32_t>());
        LSS_CHECK_LAUNCH("k_m2l_small");
    }
    for (size_t i = 0; i < jobs.size(); ++i)
        if (!on_aux[i]) m2l(jobs[i], t.L.as<double>());
    LSS_HIP(hipStreamWaitEvent(c.stream, c.aux_ev[5], 0));
    launch_add(c, t.L.as<double>(), t.L2.as<double>(), t.nboxes * (int64_t)ncp);
}

void build_fmm(Ctx &c) {
    build_tree_boxes(c);
    Tree &t = c.tree;
    const int p = fmm_order_for(c);
    const int ncp = (int)ceil_div(fmm::ncoef(p), kKB) * kKB;
    const int64_t per = (int64_t)ncp * ncp;
    // operators: M2M / L2L for the 8 octants, M2L for the classes in use
    if (t.ops_p != p) {
        std::vector<double> w(24);
        for (int o = 0; o < 8; ++o) {
            w[3 * o] = (o & 1) ? 0.5 : -0.5;
            w[3 * o + 1] = ((o >> 1) & 1) ? 0.5 : -0.5;
            w[3 * o + 2] = ((o >> 2) & 1) ? 0.5 : -0.5;
        }
        t.opM2M.ensure(sizeof(double) * 8 * per);
        t.opL2L.ensure(sizeof(double) * 8 * per);
        build_ops(c, 1, 8, w, p, ncp, t.opM2M.as<double>());
        build_ops(c, 2, 8, w, p, ncp, t.opL2L.as<double>());
        t.op_class_slot.assign(kNClass, -1);
        t.opM2L.release();
        t.ops_p = p;
    }
    t.p = p;
    t.ncp = ncp;
    t.M.ensure(sizeof(double) * t.nboxes * ncp);
    t.L.ensure(sizeof(double) * t.nboxes * ncp);
    // The upward pass (P2M, M2M) needs only the boxes: it runs on the
    // auxiliary stream while the interaction lists are built on the context
    // stream; the M2L waits for both.  The direct and M2P lists are sorted
    // on the auxiliary stream after the upward pass, beside the
    // translations; the context stream waits for them before returning.
    // Same kernels, same order per buffer, so the results do not depend on
    // the overlap.
    if (!c.aux_stream) {
        LSS_HIP(hipStreamCreateWithFlags(&c.aux_stream, hipStreamNonBlocking));
        for (hipEvent_t &e : c.aux_ev) LSS_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    }
    struct StreamSwap {
        Ctx &c;
        hipStream_t saved;
        ~StreamSwap() { c.stream = saved; }
    };
    LSS_HIP(hipEventRecord(c.aux_ev[0], c.stream));
    LSS_HIP(hipStreamWaitEvent(c.aux_stream, c.aux_ev[0], 0));
    DBuf flag, ids, leaves, nleaf;
    {
        StreamSwap swap{c, c.stream};
        c.stream = c.aux_stream;
        upward_pass(c, p, ncp, flag, ids, leaves, nleaf);
        LSS_HIP(hipEventRecord(c.aux_ev[1], c.aux_stream));
    }
    build_tree_lists(c);
    LSS_HIP(hipEventRecord(c.aux_ev[2], c.stream));        // lists emitted, M2L list sorted
    {
        StreamSwap swap{c, c.stream};
        c.stream = c.aux_stream;
        LSS_HIP(hipStreamWaitEvent(c.aux_stream, c.aux_ev[2], 0));
        sort_near_lists(c);
        LSS_HIP(hipEventRecord(c.aux_ev[3], c.aux_stream));
    }
    if (!m2l_planned(c)) {
        LSS_HIP(hipStreamWaitEvent(c.stream, c.aux_ev[1], 0));
        if (m2l_rotated(c)) launch_fill_zero(c, t.L.as<double>(), t.nboxes * (int64_t)ncp);   // upward_pass did not
        m2l_classwise(c, p, ncp);
    } else {
        m2l_plan(c);
        LSS_HIP(hipStreamWaitEvent(c.stream, c.aux_ev[1], 0));
        m2l_pass(c, p, ncp);
    }
    // downward pass: L2L from level 0 to depth-1 into their children
    for (int lvl = 1; lvl <= t.depth; ++lvl) {
        const int64_t base = t.level_begin[lvl], npar = (t.level_begin[lvl + 1] - base) / 8;
        GemmArgs a{G_L2L, ncp, ncp, npar, t.opL2L.as<double>(), t.L.as<double>(), t.L.as<double>(), nullptr, nullptr,
                   base, t.parent.as<int32_t>(), t.level.as<int32_t>(), t.root.as<double>(), t.bmesh.as<int32_t>()};
        gemm(c, a);
    }
    LSS_HIP(hipStreamWaitEvent(c.stream, c.aux_ev[3], 0));   // the direct and M2P lists
    c.stats.fmm_order = p;
}

}  // namespace lss
