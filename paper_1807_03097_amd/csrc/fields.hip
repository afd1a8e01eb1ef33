// Incident and scattered fields: right-hand sides of plane waves and point sources for
// several columns at once (Sec. 3.2 eq. (eq:linsys); scalar: Sec. 2.2), and the scattered
// field (scalar: the single layer potential) at points off the surface (Sec. 2 eq. (eq:ESLP)).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "device_math.hpp"
#include "op.hpp"

namespace ige {

namespace {

using dm::cadd;
using dm::cscale;
typedef double dx4 __attribute__((ext_vector_type(4)));

// the columns of one launch: direction or source point, and the polarisation (EFIE)
struct RhsCols {
    double a[kRhsCols][3];
    double2 pol[kRhsCols][3];
};

// Element moments of the incident fields,
//   EFIE   loc[e][l][c] = -sum_q e^{i kappa d_c.x_q} (Psi_l(q) . pol_c)
//   scalar loc[e][l][c] =  sum_q g_c(x_q) psi_l(q),  g_c a plane wave or G(x - a_c)
// with the quadrature weights inside Psi.  A workgroup takes 16 (element, column) pairs:
// its threads first evaluate the fields at the Gauss points into shared memory, then
// sum them against the local functions, one (element, function, column) each, the
// columns innermost, so that each value of Psi is read once for the columns of a wave.
// Bound by the sines and cosines (one per element point and column) and by the
// products; one thread per unknown and column evaluated each of them for all of its
// (up to nine, p = 2) elements again and read Psi across unknowns: 64 waves on 24,576
// elements (p = 2, 5 x 5 points) 24.2 ms then, 0.67 ms in this form alone.
template <bool SC>
__global__ __launch_bounds__(256) void k_rhs_elem(DevOp o, int64_t E, int rw, int nc, int kind, RhsCols cols, double2 *loc)
{
    extern __shared__ double2 sex[];   // [16 pairs][G2]
    const int G2 = o.G2, NL = o.nl, ne = 16 / rw;
    const int64_t e0 = (int64_t)blockIdx.x * ne;
    for (int i = threadIdx.x; i < 16 * G2; i += blockDim.x) {
        const int pr = i / G2, q = i % G2, c = pr % rw;
        const int64_t e = e0 + pr / rw;
        double2 g = make_double2(0.0, 0.0);
        if (e < E && c < nc) {
            const double *X = o.eX + e * 3 * G2;
            const double x0 = X[q], x1 = X[G2 + q], x2 = X[2 * G2 + q];
            const double *a = cols.a[c];
            double sn, cs;
            if (!SC || kind == 0) {
                sincos(o.kappa * (a[0] * x0 + a[1] * x1 + a[2] * x2), &sn, &cs);
                g = make_double2(cs, sn);
            } else {
                const double d0 = x0 - a[0], d1 = x1 - a[1], d2 = x2 - a[2];
                const double r = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
                sincos(o.kappa * r, &sn, &cs);
                const double f = 0.07957747154594767 / r;   // 1 / (4 pi r)
                g = make_double2(cs * f, sn * f);
            }
        }
        sex[i] = g;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 16 * NL; i += blockDim.x) {
        const int c = i % rw, l = (i / rw) % NL, el = i / (rw * NL);
        const int64_t e = e0 + el;
        if (e >= E || c >= nc) continue;
        const double2 *ex = sex + (el * rw + c) * G2;
        const double *Ps = o.ePsi + (e * 4 * NL + l) * G2;
        double2 v;
        if (SC) {
            const double *P3 = Ps + (size_t)3 * NL * G2;
            v = make_double2(0.0, 0.0);
            for (int q = 0; q < G2; ++q) v = cadd(v, cscale(P3[q], ex[q]));
        } else {
            double2 t[3] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
            for (int q = 0; q < G2; ++q) {
                const double2 g = ex[q];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    const double w = Ps[(size_t)d * NL * G2 + q];
                    t[d].x = fma(w, g.x, t[d].x);
                    t[d].y = fma(w, g.y, t[d].y);
                }
            }
            v = make_double2(0.0, 0.0);
#pragma unroll
            for (int d = 0; d < 3; ++d) v = cadd(v, dm::cmul(cols.pol[c][d], t[d]));
            v = make_double2(-v.x, -v.y);
        }
        loc[((size_t)e * NL + l) * nc + c] = v;
    }
}

// The same for more than eight columns and up to 16 local functions, on the FP64 matrix instruction: a
// wave takes one element.  Per step of four Gauss points lane (hi, n) evaluates point 4 t + hi of column
// n, which is operand B as it stands; the stored operand of the 16 local functions at the four
// points is operand A, one product per component of the tested field and for the real and the
// imaginary parts.
// Bound by the sines and cosines (seven per lane at 5 x 5 points), FP64 issue and the 11 KB of
// operands per element, which are read in whole lines (from the row layout, 16 rows of 200 bytes
// at a time, 16 columns took 135 us).  24,576 elements of 12 functions, with the sum: 16 columns 171 us
// in the form above, 102 here; 12 columns 154 and 98; 64 columns 674 and 393.
template <bool SC>
__global__ __launch_bounds__(256) void k_rhs_mx(DevOp o, int64_t E, int nc, int kind, RhsCols cols, double2 *loc)
{
    constexpr int ND = SC ? 1 : 3;
    const int G2 = o.G2, NL = o.nl, lane = threadIdx.x & 63, n = lane & 15, hi = lane >> 4;
    const int64_t e = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (e >= E) return;   // the whole wave
    const int c = min(n, nc - 1), T = 4 * ((G2 + 15) / 16);
    const double a0 = cols.a[c][0], a1 = cols.a[c][1], a2 = cols.a[c][2];
    const double *X = o.eX + e * 3 * G2, *F = o.ePsiF + (e * 4 + (SC ? 3 : 0)) * T * 64 + lane;
    dx4 re[ND], im[ND];
#pragma unroll
    for (int d = 0; d < ND; ++d) re[d] = im[d] = dx4{0.0, 0.0, 0.0, 0.0};
    for (int t = 0; 4 * t < G2; ++t) {
        const int q = 4 * t + hi, qc = min(q, G2 - 1);
        double A[ND];
#pragma unroll
        for (int d = 0; d < ND; ++d) A[d] = F[(d * T + t) * 64];
        const double x0 = X[qc], x1 = X[G2 + qc], x2 = X[2 * G2 + qc];
        double2 g;
        double sn, cs;
        if (!SC || kind == 0) {
            sincos(o.kappa * (a0 * x0 + a1 * x1 + a2 * x2), &sn, &cs);
            g = make_double2(cs, sn);
        } else {
            const double d0 = x0 - a0, d1 = x1 - a1, d2 = x2 - a2;
            const double r = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
            sincos(o.kappa * r, &sn, &cs);
            const double f = 0.07957747154594767 / r;   // 1 / (4 pi r)
            g = make_double2(cs * f, sn * f);
        }
        if (q >= G2) g = make_double2(0.0, 0.0);
#pragma unroll
        for (int d = 0; d < ND; ++d) {
            re[d] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[d], g.x, re[d], 0, 0, 0);
            im[d] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[d], g.y, im[d], 0, 0, 0);
        }
    }
    if (n >= nc) return;
    // lane: column n, functions hi + 4 j
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int l = hi + 4 * j;
        if (l >= NL) continue;
        double2 v;
        if constexpr (SC) {
            v = make_double2(re[0][j], im[0][j]);
        } else {
            v = make_double2(0.0, 0.0);
#pragma unroll
            for (int d = 0; d < 3; ++d) v = cadd(v, dm::cmul(cols.pol[c][d], make_double2(re[d][j], im[d][j])));
            v = make_double2(-v.x, -v.y);
        }
        loc[((size_t)e * NL + l) * nc + n] = v;
    }
}

// f[c][i] = sum of the element moments of unknown i (incarnations, then elements row by
// row), with the gluing sign; columns innermost over the threads
__global__ __launch_bounds__(256) void k_rhs_sum(DevOp o, int nc, const double2 *loc, double2 *f)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int i = (int)(t / nc), c = (int)(t % nc);
    if (i >= o.N) return;
    const int p = o.p, n = o.n, NL = o.nl;
    double2 acc = make_double2(0.0, 0.0);
    for (int k = 0; k < 2; ++k) {
        const int32_t *in = o.inc + ((size_t)i * 2 + k) * 5;
        const int j = in[0];
        if (j < 0) continue;
        const int a = in[1], i1 = in[2], i2 = in[3];
        const double sg = (double)in[4];
        const int du = (a == 0) ? p : p - 1, dv = (a == 0 && !o.scalar) ? p - 1 : p;
        for (int e2 = max(0, i2 - dv); e2 <= min(n - 1, i2); ++e2)
            for (int e1 = max(0, i1 - du); e1 <= min(n - 1, i1); ++e1) {
                const int t1 = i1 - e1, t2 = i2 - e2;
                const int l = (a == 0) ? t2 * (p + 1) + t1 : p * (p + 1) + t2 * p + t1;
                const int64_t e = ((int64_t)j * n + e2) * n + e1;
                acc = cadd(acc, cscale(sg, loc[((size_t)e * NL + l) * nc + c]));
            }
    }
    f[(size_t)c * o.N + i] = acc;
}

}  // namespace

size_t rhs_scratch_values(const DevOp &o, int nc) { return (size_t)o.P * o.n * o.n * o.nl * nc; }

// What the operator keeps from its assembly on, so that a captured launch finds it: element moments of
// one column, or of as many as a launch takes within 1 MiB
size_t rhs_base_values(size_t one)
{
    const size_t most = ((size_t)1 << 20) / sizeof(double2);
    return std::max(one, std::min(most, kRhsCols * one));
}

void launch_rhs(ige_op op, int kind, int nc, const double *a, const double2 *pol, double2 *f, double2 *scr, size_t nscr)
{
    const DevOp &o = op->view;
    IGE_REQUIRE(nc >= 1 && nc <= kRhsCols && nscr >= rhs_scratch_values(o, nc), "right-hand side scratch too small");
    RhsCols cols{};
    for (int c = 0; c < nc; ++c)
        for (int d = 0; d < 3; ++d) {
            cols.a[c][d] = a[3 * c + d];
            cols.pol[c][d] = pol ? pol[3 * c + d] : make_double2(0.0, 0.0);
        }
    int rw = 1;   // columns per workgroup: the smallest power of two that holds them
    while (rw < nc) rw *= 2;
    const int64_t E = (int64_t)o.P * o.n * o.n;
    const int ne = 16 / rw;
    const dim3 grid((unsigned)((E + ne - 1) / ne));
    const size_t shm = sizeof(double2) * 16 * o.G2;
    hipStream_t s = lstream(op);
    // The matrix form always works on 16 columns and 16 functions: from nine columns on, where the other
    // pads to 16 as well (8 columns: 87 us there, 91 here; 12: 154 and 98); 24 functions in two
    // tiles leave two waves per SIMD (16 columns: 53 and 58)
    const bool mx = nc > 8 && o.nl <= kRhsMxFns;
    const dim3 gm((unsigned)((E + 3) / 4));
    if (mx && o.scalar) hipLaunchKernelGGL(k_rhs_mx<true>, gm, dim3(256), 0, s, o, E, nc, kind, cols, scr);
    else if (mx) hipLaunchKernelGGL(k_rhs_mx<false>, gm, dim3(256), 0, s, o, E, nc, kind, cols, scr);
    else if (o.scalar) hipLaunchKernelGGL(k_rhs_elem<true>, grid, dim3(256), shm, s, o, E, rw, nc, kind, cols, scr);
    else hipLaunchKernelGGL(k_rhs_elem<false>, grid, dim3(256), shm, s, o, E, rw, nc, kind, cols, scr);
    IGE_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_rhs_sum, dim3((unsigned)(((int64_t)o.N * nc + 255) / 256)), dim3(256), 0, s, o, nc, scr, f);
    IGE_HIP(hipGetLastError());
}

}  // namespace ige

// ---------------------------------------------------------------------------
// Scattered field e_s = V~ w at points off the surface:
//   e_s(x) = sum_e sum_q [G(x - y_q) W_q + kappa^-2 grad_x G(x - y_q) D_q],
// W_q = sum_l w_l Psi_l(q) (weighted phi_hat^a d_aF), D_q = sum_l w_l div_l(q), on the
// regular g x g Gauss points of every element; grad_x G = (x - y) G (i kappa r - 1) / r^2.
// Scalar: u(x) = sum_e sum_q G(x - y_q) D_q in component 0.
// ---------------------------------------------------------------------------
namespace ige {
namespace {

// per Gauss point of every element: y (3), W (3 complex), kappa^-2 D (scalar: D) as
// [kPotStride][nsrc]
constexpr int kPotStride = 11;
constexpr int kPotPts = 4;   // points per workgroup

template <int NL>
__global__ __launch_bounds__(64) void k_pot_sources(DevOp o, const double2 *w, double *src)
{
    __shared__ double2 cf[NL];
    const int64_t e = blockIdx.x;
    const int G2 = o.G2, nn = o.n * o.n;
    const int j = (int)(e / nn), e2 = (int)(e % nn) / o.n, e1 = (int)(e % nn) % o.n;
    if (threadIdx.x < NL) {
        const int l = threadIdx.x, p = o.p;
        int a = 0, t1 = l % (p + 1), t2 = l / (p + 1);
        if (!o.scalar && l >= p * (p + 1)) {
            a = 1;
            t2 = (l - p * (p + 1)) / p;
            t1 = (l - p * (p + 1)) % p;
        }
        const size_t off = (((size_t)j * 2 + a) * o.nb + (e2 + t2)) * o.nb + (e1 + t1);
        const int idx = o.dof[off];
        cf[l] = idx >= 0 ? cscale((double)o.sgn[off], w[idx]) : make_double2(0.0, 0.0);
    }
    __syncthreads();
    const int64_t nsrc = (int64_t)gridDim.x * G2;
    const double fd = o.scalar ? 1.0 : 1.0 / (o.kappa * o.kappa);
    for (int q = threadIdx.x; q < G2; q += blockDim.x) {
        double *s = src + e * G2 + q;
        for (int d = 0; d < 3; ++d) s[d * nsrc] = o.eX[((size_t)e * 3 + d) * G2 + q];
        for (int c = 0; c < 4; ++c) {
            double2 W = make_double2(0.0, 0.0);
#pragma unroll
            for (int l = 0; l < NL; ++l) W = cadd(W, cscale(o.ePsi[(((size_t)e * 4 + c) * NL + l) * G2 + q], cf[l]));
            if (c == 3) W = cscale(fd, W);
            s[(3 + 2 * c) * nsrc] = W.x;
            s[(4 + 2 * c) * nsrc] = W.y;
        }
    }
}

// kPotPts target points per workgroup, its threads over the source points of the part
// blockIdx.y; a fixed butterfly over each wave, then the waves in order.  Bound by the
// FP64 arithmetic, about 60 operations per point and source: the sources are read once
// for kPotPts points (coalesced), 1/r comes from the hardware estimate with one
// third-order step instead of a root and two divisions, and sine and cosine from the
// table.  With few points the sources are split over workgroups until the device is
// full.  3,000 points, 153,600 sources (level 5, p = 2): 3.03 ms with one point per
// workgroup, sqrt and divisions, 1.09 ms now (both with the copies to and from the host).
template <bool SC>
__global__ __launch_bounds__(256) void k_potential(int64_t nsrc, int64_t per, double kappa, const double *src, int npts,
                                                   const double *pts, const double2 *sctab, double2 *out)
{
    constexpr int V = SC ? 2 : 6;
    __shared__ double2 sTab[256];
    __shared__ double red[4][kPotPts][V];
    for (int i = threadIdx.x; i < 256; i += blockDim.x) sTab[i] = sctab[i];
    double X[kPotPts][3], acc[kPotPts][V];
#pragma unroll
    for (int k = 0; k < kPotPts; ++k) {
        const int t = min(npts - 1, (int)blockIdx.x * kPotPts + k);
#pragma unroll
        for (int d = 0; d < 3; ++d) X[k][d] = pts[3 * (size_t)t + d];
#pragma unroll
        for (int v = 0; v < V; ++v) acc[k][v] = 0.0;
    }
    __syncthreads();
    const int64_t b = blockIdx.y * per, e = min(nsrc, b + per);
    for (int64_t i = b + threadIdx.x; i < e; i += blockDim.x) {
        const double *s = src + i;
        const double y0 = s[0], y1 = s[nsrc], y2 = s[2 * nsrc];
        double2 W[3];
        if constexpr (!SC)
#pragma unroll
            for (int d = 0; d < 3; ++d) W[d] = make_double2(s[(3 + 2 * d) * nsrc], s[(4 + 2 * d) * nsrc]);
        const double2 D = make_double2(s[9 * nsrc], s[10 * nsrc]);
#pragma unroll
        for (int k = 0; k < kPotPts; ++k) {
            const double rv[3] = {X[k][0] - y0, X[k][1] - y1, X[k][2] - y2};
            double ir, kr;
            const double2 G = dm::helmholtz_r2_tab(kappa, fma(rv[0], rv[0], fma(rv[1], rv[1], rv[2] * rv[2])), sTab, ir, kr);
            const double2 GD = dm::cmul(G, D);
            if constexpr (SC) {
                acc[k][0] += GD.x;
                acc[k][1] += GD.y;
            } else {
                // grad_x G D / kappa^2 = (x - y) (G D / kappa^2) (i kappa r - 1) / r^2
                const double i2 = ir * ir;
                const double gx = i2 * fma(-kr, GD.y, -GD.x), gy = i2 * fma(kr, GD.x, -GD.y);
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    acc[k][2 * d] = fma(G.x, W[d].x, fma(-G.y, W[d].y, fma(rv[d], gx, acc[k][2 * d])));
                    acc[k][2 * d + 1] = fma(G.x, W[d].y, fma(G.y, W[d].x, fma(rv[d], gy, acc[k][2 * d + 1])));
                }
            }
        }
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < kPotPts; ++k)
#pragma unroll
        for (int v = 0; v < V; ++v) {
            double a = acc[k][v];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) a += __shfl_xor(a, off, 64);
            if (lane == 0) red[wv][k][v] = a;
        }
    __syncthreads();
    const int k = threadIdx.x / 3, d = threadIdx.x % 3, t = blockIdx.x * kPotPts + k;
    if (k >= kPotPts || t >= npts) return;
    double2 z = make_double2(0.0, 0.0);
    if (2 * d < V)
        for (int w = 0; w < 4; ++w) z = cadd(z, make_double2(red[w][k][2 * d], red[w][k][2 * d + 1]));
    out[((size_t)blockIdx.y * npts + t) * 3 + d] = z;
}

// out[i] = sum of the parts of the sources, in order
__global__ __launch_bounds__(256) void k_pot_sum(int64_t n, int parts, const double2 *part, double2 *out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double2 z = make_double2(0.0, 0.0);
    for (int p = 0; p < parts; ++p) z = cadd(z, part[p * n + i]);
    out[i] = z;
}

}  // namespace

// ---------------------------------------------------------------------------
// Fixed device scratch of ige_potential_noalloc: the per-element source data of the
// potential (kPotStride doubles per Gauss point of every element), at most
// kPotScratchDoubles doubles (64 MiB).  Every device the library runs on holds its
// own copy until the process ends.  Host code never passes the symbol itself: its
// device address is looked up once per device (potential_scratch_init, with that
// device current) and kept per device ordinal.
// ---------------------------------------------------------------------------
constexpr size_t kPotScratchDoubles = (size_t)8 << 20;
static __device__ __align__(256) double scratch[kPotScratchDoubles];

namespace {
std::mutex g_scratch_mu;
std::vector<double *> g_scratch_ptr;   // device address of scratch per device ordinal
}  // namespace

void potential_scratch_init(int device)
{
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if ((int)g_scratch_ptr.size() <= device) g_scratch_ptr.resize((size_t)device + 1, nullptr);
    if (g_scratch_ptr[device]) return;
    void *ptr = nullptr;
    IGE_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    g_scratch_ptr[device] = static_cast<double *>(ptr);
}

double *potential_scratch(int device)
{
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    return device >= 0 && device < (int)g_scratch_ptr.size() ? g_scratch_ptr[device] : nullptr;
}

size_t potential_scratch_doubles() { return kPotScratchDoubles; }

size_t potential_source_doubles(ige_op op) { return (size_t)op->view.P * op->view.n * op->view.n * op->view.G2 * kPotStride; }

// parts of the sources for npts points: enough workgroups for every CU to hold eight (256 of
// them), at least 2048 sources (eight per thread) each; for an operator that fits the fixed
// scratch no more than that has room for behind its sources, with either entry point, so that
// both give the same bits
int potential_parts(ige_op op, int npts)
{
    const size_t need = (potential_source_doubles(op) + 1) / 2 * 2;
    const int64_t nsrc = (int64_t)(need / kPotStride), groups = (npts + kPotPts - 1) / kPotPts;
    int64_t parts = std::max<int64_t>(1, std::min((2048 + groups - 1) / std::max<int64_t>(1, groups), nsrc / 2048));
    if (need <= kPotScratchDoubles && npts > 0) {
        const int64_t room = (int64_t)((kPotScratchDoubles - need) / ((size_t)6 * npts));
        parts = std::min(parts, std::max<int64_t>(1, room));
    }
    return (int)parts;
}

void launch_potential(ige_op op, const double2 *w, int npts, const double *pts, double2 *out, double *src, int parts,
                      double2 *part)
{
    const DevOp &o = op->view;
    const int64_t E = (int64_t)o.P * o.n * o.n;
    hipStream_t s = lstream(op);
#define IGE_PS(NLV) hipLaunchKernelGGL(k_pot_sources<NLV>, dim3((unsigned)E), dim3(64), 0, s, o, w, src)
    switch (o.nl) {
        case 4: IGE_PS(4); break;
        case 9: IGE_PS(9); break;
        case 12: IGE_PS(12); break;
        case 16: IGE_PS(16); break;
        case 24: IGE_PS(24); break;
        case 25: IGE_PS(25); break;
        default: IGE_PS(40); break;
    }
#undef IGE_PS
    IGE_HIP(hipGetLastError());
    if (npts <= 0) return;
    const int64_t nsrc = E * o.G2, per = (nsrc + parts - 1) / parts;
    const dim3 grid((unsigned)((npts + kPotPts - 1) / kPotPts), (unsigned)parts);
    double2 *to = parts > 1 ? part : out;
    if (o.scalar)
        hipLaunchKernelGGL(k_potential<true>, grid, dim3(256), 0, s, nsrc, per, o.kappa, src, npts, pts, o.sctab, to);
    else
        hipLaunchKernelGGL(k_potential<false>, grid, dim3(256), 0, s, nsrc, per, o.kappa, src, npts, pts, o.sctab, to);
    IGE_HIP(hipGetLastError());
    if (parts > 1) {
        const int64_t n = (int64_t)3 * npts;
        hipLaunchKernelGGL(k_pot_sum, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, parts, part, out);
        IGE_HIP(hipGetLastError());
    }
}

}  // namespace ige
