// Polynomial interpolation of chart data between the chart nodes (section
// 3.3: each chart is approximated on the standard simplex T0 by a polynomial
// of total degree p, through an orthogonal basis of Koornwinder polynomials
// sampled at the p-th order nodes).  The interpolation matrix from the np
// nodes to the ne evaluation points is the same for every triangle: one kernel
// forms it (the host for degrees above 14), I = E V^-1 with V_ik = K_k(node i),
// E_ek = K_k(point e), and another applies it to every triangle's node values.
#include <hip/hip_runtime.h>

#include <cmath>
#include <vector>

#include "lss_internal.h"

namespace lss {

namespace {

// Koornwinder (Dubiner) basis on T0 = {u, v >= 0, u + v <= 1}, ordered by
// (m, n) with m + n <= p:  K_mn = L_m(s, t) P_n^(2m+1,0)(2v - 1), where
// s = 2u + v - 1, t = 1 - v and L_m(s, t) = t^m P_m(s / t) is the Legendre
// polynomial made homogeneous (a polynomial in u, v also at v = 1).
// The functions of one m, by Put(index, value).
template <class Put>
__host__ __device__ inline void koornwinder(double u, double v, int p, int m, Put put) {
    const double s = 2.0 * u + v - 1.0, t = 1.0 - v, x = 2.0 * v - 1.0;
    double lm1 = 0.0, lm = 1.0;                       // L_{m-1}, L_m
    for (int j = 0; j < m; ++j) {
        const double next = j == 0 ? s : ((2.0 * j + 1.0) * s * lm - j * t * t * lm1) / (j + 1.0);
        lm1 = lm;
        lm = next;
    }
    int k = m * (p + 1) - m * (m - 1) / 2;
    const double a = 2.0 * m + 1.0;                   // Jacobi P_n^(a, 0)
    double pm2 = 0.0, pm1 = 1.0;
    for (int n = 0; m + n <= p; ++n) {
        double pn;
        if (n == 0) pn = 1.0;
        else if (n == 1) pn = 0.5 * ((a + 2.0) * x + a);
        else {
            const double c = 2.0 * n + a;
            pn = ((c - 1.0) * (c * (c - 2.0) * x + a * a) * pm1 - 2.0 * (n + a - 1.0) * (n - 1.0) * c * pm2) /
                 (2.0 * n * (n + a) * (c - 2.0));
        }
        if (n >= 1) { pm2 = pm1; pm1 = pn; }
        put(k++, lm * pn);
    }
}

// Where entry (node i, point e) of the matrix lies: node-major for
// k_chart_interp (G = 0), as MFMA fragments for k_chart_interp_mfma:
// [group of G row tiles][k step][row tile of the group][lane].
__host__ __device__ inline int64_t matrix_slot(int64_t i, int64_t e, int64_t np, int64_t ne, int64_t G) {
    if (!G) return i * ne + e;
    const int64_t ks = (np + 3) / 4, t = e >> 4;
    return 64 * ((t - t % G) * ks + (i >> 2) * G + t % G) + 16 * (i & 3) + (e & 15);
}

constexpr int kMatrixNp = 120;                       // degree 14: V and 16 right-hand sides fit LDS
constexpr int kMatrixThreads = 512;

// maximum over the wave, in all its lanes
__device__ __forceinline__ unsigned wave_max(unsigned v) {
#define LSS_DPP_MAX(ctrl, rows)                                                                             \
    {                                                                                                       \
        const unsigned o = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xf, false);        \
        v = o > v ? o : v;                                                                                  \
    }
    LSS_DPP_MAX(0x111, 0xf)      // lane - 1 of the row of 16
    LSS_DPP_MAX(0x112, 0xf)      // lane - 2
    LSS_DPP_MAX(0x114, 0xf)      // lane - 4
    LSS_DPP_MAX(0x118, 0xf)      // lane - 8
    LSS_DPP_MAX(0x142, 0xa)      // last lane of the row before, rows 1 and 3
    LSS_DPP_MAX(0x143, 0xc)      // lane 31, rows 2 and 3
#undef LSS_DPP_MAX
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// The interpolation matrix by Gauss-Jordan elimination with partial pivoting
// of V^T I^T = E^T; a workgroup takes 16 points and eliminates V for itself.
// The matrix is held in registers, eight lanes to a row (rows tid/8 + 64 r,
// columns tid%8 + 8 u); LDS carries the leading column and the pivot row of
// a step.  Every wave finds the pivot for itself, and rows are marked instead
// of swapped.  bad is set where V is singular to 1e-13 of its largest entry.
// Bound by the latency of np steps, one after the other, each by its
// instructions: 37 us for 45 nodes (82 on the host, and the copies there and
// back; 45 to 50 with the matrix in LDS).
template <int R, int NU>
__global__ __launch_bounds__(kMatrixThreads) void k_interp_matrix(int32_t p, int32_t np, int32_t ne, int32_t G,
                                                                  const double *__restrict__ nodes,
                                                                  const double *__restrict__ points, double *mat,
                                                                  int32_t *bad) {
    extern __shared__ double sm[];
    __shared__ double lead[2][64 * R], prow[8 * NU], wmax[kMatrixThreads / 64], pivots[64 * R];
    __shared__ int unknown[64 * R];                   // of a row
    const int e0 = 16 * blockIdx.x, width = np + 16, lane = threadIdx.x & 63, q0 = threadIdx.x >> 3, l8 = threadIdx.x & 7;
    // column i < np: node i; column np + e: point e0 + e; row: basis function
    for (int k = threadIdx.x; k < width * (p + 1); k += kMatrixThreads) {
        const int i = k % width, m = k / width;
        const double *q = i < np ? nodes + 2 * i : points + 2 * (int64_t)(e0 + i - np < ne ? e0 + i - np : ne - 1);
        koornwinder(q[0], q[1], p, m, [&](int f, double val) { sm[f * width + i] = val; });
    }
    __syncthreads();
    double a[R][NU], amax = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int q = q0 + 64 * r, c = l8 + 8 * u;
            a[r][u] = q < np && c < width ? sm[q * width + c] : 0.0;
            if (c < np) amax = fmax(amax, fabs(a[r][u]));
        }
#pragma unroll
    for (int o = 32; o; o >>= 1) amax = fmax(amax, __shfl_xor(amax, o));
    if (lane == 0) wmax[threadIdx.x >> 6] = amax;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kMatrixThreads / 64; ++w) amax = fmax(amax, wmax[w]);
    bool used[R];
#pragma unroll
    for (int r = 0; r < R; ++r) used[r] = lane + 64 * r >= np;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
        for (int l = 0; l < 8 && 8 * u + l < np; ++l) {
            const int col = 8 * u + l;
            double *head = lead[l & 1];
            if (l8 == l) {
#pragma unroll
                for (int r = 0; r < R; ++r) head[q0 + 64 * r] = a[r][u];
            }
            __syncthreads();
            // largest |entry| to its first 13 bits and the row in one word; NaN comes out on top and fails
            unsigned key = 0;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const unsigned hi = (unsigned)__double2hiint(head[lane + 64 * r]) & 0x7fffff80u;
                const unsigned k = used[r] ? 0u : hi | (unsigned)(127 - lane - 64 * r);
                key = k > key ? k : key;
            }
            const int row = 127 - (int)(wave_max(key) & 127u);
            const double pivot = head[row], scale = 1.0 / pivot;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                used[r] = used[r] || lane + 64 * r == row;
                if (q0 + 64 * r == row) {
#pragma unroll
                    for (int k = u; k < NU; ++k) prow[l8 + 8 * k] = a[r][k];
                }
            }
            if (!(fabs(pivot) > 1e-13 * amax)) {      // the same for all waves of all workgroups
                if (blockIdx.x == 0 && threadIdx.x == 0) *bad = 1;
                return;
            }
            if (threadIdx.x == 0) {
                unknown[row] = col;
                pivots[row] = pivot;
            }
            __syncthreads();
            double x[NU];
#pragma unroll
            for (int k = u; k < NU; ++k) x[k] = prow[l8 + 8 * k];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const double m = q0 + 64 * r == row ? 0.0 : head[q0 + 64 * r] * scale;
#pragma unroll
                for (int k = u; k < NU; ++k) a[r][k] -= m * x[k];
            }
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *bad = 0;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int q = q0 + 64 * r, e = l8 + 8 * u - np;
            if (q >= np || e < 0 || e >= 16 || (!G && e0 + e >= ne)) continue;
            mat[matrix_slot(unknown[q], e0 + e, np, ne, G)] = e0 + e < ne ? a[r][u] / pivots[q] : 0.0;
        }
    if (G)                                            // the nodes that fill the last k step
        for (int k = threadIdx.x; k < 16 * (3 & -np); k += kMatrixThreads)
            mat[matrix_slot(np + (k >> 4), e0 + (k & 15), np, ne, G)] = 0.0;
}

// one thread per (triangle j, point e); IT is the interpolation matrix
// stored node-major (IT[i * ne + e]), so the threads of a wave, which hold
// consecutive points, read consecutive entries
__global__ void k_chart_interp(int64_t ntris, int32_t np, int32_t ne, int32_t ncomp, const double *__restrict__ IT,
                               const int32_t *__restrict__ bad, const double *__restrict__ f, double *out) {
    if (*bad) return;
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= ntris * ne) return;
    const int64_t j = q / ne;
    const int32_t e = (int32_t)(q - j * ne);
    const double *fj = f + j * np * ncomp;
    for (int32_t c = 0; c < ncomp; ++c) {
        double acc = 0.0;
        for (int32_t i = 0; i < np; ++i) acc = fma(IT[(int64_t)i * ne + e], fj[(int64_t)i * ncomp + c], acc);
        out[q * ncomp + c] = acc;
    }
}

using f64x4 = double __attribute__((ext_vector_type(4)));

// LDS between lanes of one wave: orders the accesses, no barrier
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

constexpr int kInterpTiles = 5;                      // row tiles of 16 points that a wave accumulates at once
constexpr int kInterpWaves = 16;                     // waves of a workgroup, at most
constexpr int64_t kInterpRegion = 24 * 1024;         // node values that a wave stages, bytes, at most
constexpr int kInterpLoads = 12;                     // of them on their way at once
constexpr int64_t kInterpLds = 160 * 1024;
constexpr size_t kMatrixKept = (size_t)64 << 20;     // matrix buffer that the context keeps between calls, at most

// Same product on the FP64 matrix cores: rows are the points, columns the
// (triangle, component) pairs, the nodes are contracted.  A wave takes T
// triangles and G row tiles at a time: it stages their node values, which lie together, in
// its part of LDS, and multiplies them by the matrix (held as the fragments
// of v_mfma_f64_16x16x4f64, zero where it is padded; in LDS when IL, else it
// comes from L2).  No barrier after the matrix is staged, so the waves of a
// CU load, multiply and store at different times.  A lane of the accumulator
// holds one column, and a store instruction four consecutive points of every
// component: runs of 4 * ncomp values, which L2 joins to full lines.
// Bound by HBM: 45 nodes to 66 points of 3 components for 2e5 triangles are
// 0.53 GB, 111 us at the rate of a copy; 142 here (341 with a thread per point
// and the matrix in LDS, bound by its LDS reads).  Two other forms measured:
// 16 triangles a wave, staged one batch ahead in registers, 163 (7 waves per
// CU, whose matrix products collide); nontemporal stores 168.
template <int G, bool IL>
__global__ __launch_bounds__(64 * kInterpWaves) void k_chart_interp_mfma(int64_t ntris, int32_t np, int32_t ne,
                                                                         int32_t ncomp, int32_t T, int32_t et,
                                                                         const double *__restrict__ frag,
                                                                         const int32_t *__restrict__ bad,
                                                                         const double *__restrict__ f, double *out) {
    extern __shared__ double sm[];
    if (*bad) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int ks = (np + 3) / 4, per = np * ncomp;
    const int nfrag = IL ? 64 * ks * et : 0;
    if (IL) {
        for (int k = threadIdx.x; k < nfrag; k += blockDim.x) sm[k] = frag[k];
        __syncthreads();
    }
    const double *A = IL ? sm : frag;
    double *F = sm + nfrag + (int64_t)w * T * per;
    const int64_t batches = (ntris + T - 1) / T;
    for (int64_t b = (int64_t)blockIdx.x * nw + w; b < batches; b += (int64_t)gridDim.x * nw) {
        const int64_t j0 = b * T;
        const int ncol = (int)(ntris - j0 < T ? ntris - j0 : T) * ncomp, cnt = ncol * np;
        const double *src = f + j0 * per;
        for (int k0 = lane; k0 < cnt; k0 += 64 * kInterpLoads) {
            double v[kInterpLoads];
#pragma unroll
            for (int u = 0; u < kInterpLoads; ++u) v[u] = k0 + 64 * u < cnt ? src[k0 + 64 * u] : 0.0;
#pragma unroll
            for (int u = 0; u < kInterpLoads; ++u)
                if (k0 + 64 * u < cnt) F[k0 + 64 * u] = v[u];
        }
        wave_sync();
        for (int c0 = 0; c0 < ncol; c0 += 16) {
            const int col = c0 + (lane & 15), cc = col < ncol ? col : 0, j = cc / ncomp, comp = cc - j * ncomp;
            const double *B = F + j * per + comp;
            double *o = out + (j0 + j) * (int64_t)ne * ncomp + comp;
            for (int t0 = G * blockIdx.y; t0 < et; t0 += G * gridDim.y) {
                const double *At = A + 64 * (int64_t)t0 * ks + lane;
                f64x4 acc[G];
#pragma unroll
                for (int i = 0; i < G; ++i) acc[i] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
                for (int s = 0; s < ks; ++s) {
                    const int k = 4 * s + (lane >> 4);
                    const double bv = k < np ? B[k * ncomp] : 0.0;       // never 0 * what lies behind
#pragma unroll
                    for (int i = 0; i < G; ++i)
                        acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(At[64 * (s * G + i)], bv, acc[i], 0, 0, 0);
                }
                // register q of lane l holds row (l/16) + 4q, column l%16
                if (col < ncol) {
#pragma unroll
                    for (int i = 0; i < G; ++i)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const unsigned e = 16u * (unsigned)(t0 + i) + (unsigned)(lane >> 4) + 4u * q;
                            if (e < (unsigned)ne) o[(int64_t)e * ncomp] = acc[i][q];
                        }
                }
            }
        }
        wave_sync();
    }
}

constexpr const char *kNotUnisolvent = "lss_chart_interp: the chart nodes are not unisolvent for degree p";

// The matrix for the degrees whose V does not fit LDS, node-major
std::vector<double> matrix_on_host(const double *chart_uv, int32_t np, const double *eval_uv, int32_t ne, int p, bool dev) {
    std::vector<double> nuv(2 * (size_t)np), euv(2 * (size_t)ne);
    LSS_HIP(hipMemcpy(nuv.data(), chart_uv, sizeof(double) * nuv.size(), dev ? hipMemcpyDeviceToHost : hipMemcpyHostToHost));
    LSS_HIP(hipMemcpy(euv.data(), eval_uv, sizeof(double) * euv.size(), dev ? hipMemcpyDeviceToHost : hipMemcpyHostToHost));
    // V^T I^T = E^T: LU with partial pivoting of V^T (np x np), ne right-hand sides
    std::vector<double> A((size_t)np * np), B((size_t)np * ne);
    for (int i = 0; i < np; ++i)
        for (int m = 0; m <= p; ++m) koornwinder(nuv[2 * i], nuv[2 * i + 1], p, m, [&](int k, double v) { A[(size_t)k * np + i] = v; });     // A = V^T
    for (int e = 0; e < ne; ++e)
        for (int m = 0; m <= p; ++m) koornwinder(euv[2 * e], euv[2 * e + 1], p, m, [&](int k, double v) { B[(size_t)k * ne + e] = v; });     // B = E^T
    double amax = 0.0;
    for (double a : A) amax = std::fmax(amax, std::fabs(a));
    for (int col = 0; col < np; ++col) {
        int piv = col;
        for (int r = col + 1; r < np; ++r)
            if (std::fabs(A[(size_t)r * np + col]) > std::fabs(A[(size_t)piv * np + col])) piv = r;
        if (!(std::fabs(A[(size_t)piv * np + col]) > 1e-13 * amax))
            throw Error{LSS_EINVAL, kNotUnisolvent};
        if (piv != col) {
            for (int k = 0; k < np; ++k) std::swap(A[(size_t)col * np + k], A[(size_t)piv * np + k]);
            for (int e = 0; e < ne; ++e) std::swap(B[(size_t)col * ne + e], B[(size_t)piv * ne + e]);
        }
        for (int r = col + 1; r < np; ++r) {
            const double m = A[(size_t)r * np + col] / A[(size_t)col * np + col];
            if (m == 0.0) continue;
            for (int k = col; k < np; ++k) A[(size_t)r * np + k] -= m * A[(size_t)col * np + k];
            for (int e = 0; e < ne; ++e) B[(size_t)r * ne + e] -= m * B[(size_t)col * ne + e];
        }
    }
    for (int r = np - 1; r >= 0; --r)                                          // B becomes I^T, node-major: [i][e]
        for (int e = 0; e < ne; ++e) {
            double s = B[(size_t)r * ne + e];
            for (int k = r + 1; k < np; ++k) s -= A[(size_t)r * np + k] * B[(size_t)k * ne + e];
            B[(size_t)r * ne + e] = s / A[(size_t)r * np + r];
        }
    return B;
}

}  // namespace

void chart_interp(Ctx &c, const double *chart_uv, int32_t np, const double *f, int32_t ncomp, const double *eval_uv,
                  int32_t ne, double *out, unsigned flags) {
    if (!c.have_sources) throw Error{LSS_ESTATE, "lss_chart_interp: no sources set"};
    if (np <= 0 || ne <= 0 || ncomp <= 0) throw Error{LSS_EINVAL, "lss_chart_interp: np, ne and ncomp must be >= 1"};
    if (!chart_uv || !f || !eval_uv || !out) throw Error{LSS_EINVAL, "lss_chart_interp: null argument"};
    int p = 0;
    while ((p + 1) * (p + 2) / 2 < np) ++p;
    if ((p + 1) * (p + 2) / 2 != np) throw Error{LSS_EINVAL, "lss_chart_interp: np is not (p+1)(p+2)/2"};
    if ((int64_t)c.ntris * ne > (int64_t)INT32_MAX * 64) throw Error{LSS_EINVAL, "lss_chart_interp: too many outputs"};
    const bool dev = flags & LSS_PTR_DEVICE;
    // The matrix cores take every size whose one triangle fits a wave's part
    // of LDS (k_chart_interp, which reads everything from memory, the rest).
    // A batch is the fewest triangles that fill their tiles of 16 columns to
    // nine tenths: 16 waves then share a CU (2e5 triangles, 45 nodes, 66
    // points: 5 triangles 142 us, 16 triangles 163).  The matrix is staged
    // when four waves fit beside it.
    const int64_t per = (int64_t)np * ncomp, ks = ceil_div(np, 4);
    int64_t T = 0;
    double least = 16.0;
    for (int64_t t = 1, cols = ncomp; t <= 16 && t * per * (int64_t)sizeof(double) <= kInterpRegion; ++t, cols += ncomp) {
        const double waste = (double)(16 * ceil_div(cols, 16)) / (double)cols;
        if (T && waste >= least) continue;
        T = t;
        least = waste;
        if (waste <= 1.1) break;
    }
    const bool mfma = T > 0;
    // Row tiles that a wave accumulates at once, G: the groups of G are as
    // full as they can be, and smaller where few triangles would leave the
    // chip empty unless the points are shared as well.
    int64_t et = ceil_div(ne, 16), G = 1, batches = 0;
    if (mfma) {
        batches = ceil_div(c.ntris, T);
        G = et * batches / 2048;
        G = G < 1 ? 1 : G > kInterpTiles ? kInterpTiles : G;
        const int64_t groups = ceil_div(et, G);
        G = ceil_div(et, groups);
        et = G * groups;
    }
    const int64_t mat = 64 * ks * et * (int64_t)sizeof(double), region = T * per * (int64_t)sizeof(double);
    const bool staged = mfma && mat + 4 * region <= kInterpLds;
    const int64_t nmat = mfma ? 64 * ks * et : (int64_t)np * ne;
    c.interp_mat.ensure(sizeof(double) * (nmat + 1));
    double *dI = c.interp_mat.as<double>();
    int32_t *dbad = reinterpret_cast<int32_t *>(dI + nmat);
    const bool on_device = np <= kMatrixNp && ne <= 1 << 26;     // a workgroup per 16 points: the launch's limit
    DBuf duv;
    const double *pn = chart_uv, *pe = eval_uv;
    if (dev) {
        // inputs queued on the null stream are waited for, whatever the context's stream
        if (c.stream) LSS_HIP(hipStreamSynchronize(nullptr));
    } else if (on_device) {
        duv.ensure(sizeof(double) * 2 * ((size_t)np + ne));
        LSS_HIP(hipMemcpyAsync(duv.p, chart_uv, sizeof(double) * 2 * np, hipMemcpyHostToDevice, c.stream));
        LSS_HIP(hipMemcpyAsync(duv.as<double>() + 2 * np, eval_uv, sizeof(double) * 2 * ne, hipMemcpyHostToDevice, c.stream));
        pn = duv.as<double>();
        pe = pn + 2 * np;
    }
    if (on_device) {
        const size_t lds = sizeof(double) * np * (np + 16);
        hipLaunchKernelGGL((np <= 48 ? k_interp_matrix<1, 8> : k_interp_matrix<2, 17>), dim3((unsigned)(mfma ? et : ceil_div(ne, 16))), dim3(kMatrixThreads), lds, c.stream,
                           p, np, ne, (int32_t)(mfma ? G : 0), pn, pe, dI, dbad);
        LSS_CHECK_LAUNCH("k_interp_matrix");
    } else {
        std::vector<double> I = matrix_on_host(chart_uv, np, eval_uv, ne, p, dev);
        std::vector<double> packed(nmat, 0.0);
        for (int64_t i = 0; i < np; ++i)
            for (int64_t e = 0; e < ne; ++e) packed[matrix_slot(i, e, np, ne, mfma ? G : 0)] = I[(size_t)i * ne + e];
        LSS_HIP(hipMemcpyAsync(dI, packed.data(), sizeof(double) * nmat, hipMemcpyHostToDevice, c.stream));
        LSS_HIP(hipMemsetAsync(dbad, 0, sizeof(int32_t), c.stream));
        LSS_HIP(hipStreamSynchronize(c.stream));      // packed goes away
    }
    const int64_t nin = c.ntris * (int64_t)np * ncomp, nout = c.ntris * (int64_t)ne * ncomp;
    DBuf df, dout;
    const double *pf = f;
    double *po = out;
    if (!dev) {
        df.ensure(sizeof(double) * nin);
        LSS_HIP(hipMemcpyAsync(df.p, f, sizeof(double) * nin, hipMemcpyHostToDevice, c.stream));
        pf = df.as<double>();
        dout.ensure(sizeof(double) * nout);
        po = dout.as<double>();
    }
    const int64_t nthr = c.ntris * (int64_t)ne;
    if (nthr > 0 && mfma) {
        int64_t nw = (kInterpLds - (staged ? mat : 0)) / region;
        if (nw > kInterpWaves) nw = kInterpWaves;
        const int64_t blocks = ceil_div(batches, nw), groups = et / G;
        const int64_t shares = batches >= 2048 ? 1 : groups < 4096 ? groups : 4096;
        const size_t lds = (size_t)((staged ? mat : 0) + nw * region);
        using Kernel = void (*)(int64_t, int32_t, int32_t, int32_t, int32_t, int32_t, const double *, const int32_t *, const double *, double *);
        static const Kernel kernels[2][kInterpTiles] = {
            {k_chart_interp_mfma<1, false>, k_chart_interp_mfma<2, false>, k_chart_interp_mfma<3, false>,
             k_chart_interp_mfma<4, false>, k_chart_interp_mfma<5, false>},
            {k_chart_interp_mfma<1, true>, k_chart_interp_mfma<2, true>, k_chart_interp_mfma<3, true>,
             k_chart_interp_mfma<4, true>, k_chart_interp_mfma<5, true>}};
        hipLaunchKernelGGL(kernels[staged][G - 1],
                           dim3((unsigned)(blocks < 256 ? blocks : 256), (unsigned)shares), dim3((unsigned)(64 * nw)), lds, c.stream,
                           c.ntris, np, ne, ncomp, (int32_t)T, (int32_t)et, dI, dbad, pf, po);
        LSS_CHECK_LAUNCH("k_chart_interp_mfma");
    } else if (nthr > 0) {
        hipLaunchKernelGGL(k_chart_interp, dim3((unsigned)ceil_div(nthr, 256)), dim3(256), 0, c.stream, c.ntris, np, ne,
                           ncomp, dI, dbad, pf, po);
        LSS_CHECK_LAUNCH("k_chart_interp");
    }
    int32_t bad = 0;
    LSS_HIP(hipMemcpyAsync(&bad, dbad, sizeof(bad), hipMemcpyDeviceToHost, c.stream));
    LSS_HIP(hipStreamSynchronize(c.stream));                // the temporaries are freed on return
    if (c.interp_mat.bytes > kMatrixKept) c.interp_mat.release();
    if (bad) throw Error{LSS_EINVAL, kNotUnisolvent};
    if (!dev) LSS_HIP(hipMemcpy(out, po, sizeof(double) * nout, hipMemcpyDeviceToHost));
}

}  // namespace lss
