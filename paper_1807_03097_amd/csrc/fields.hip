// Incident fields: right-hand sides of plane waves and point sources for several
// columns at once (Sec. 3.2 eq. (eq:linsys); scalar: Sec. 2.2).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_math.hpp"
#include "op.hpp"

namespace ige {

namespace {

using dm::cadd;
using dm::cscale;

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
// elements (p = 2, 5 x 5 points) 24.2 ms before, 0.69 ms now.
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

void launch_rhs(ige_op op, int kind, int nc, const double *a, const double2 *pol, double2 *f)
{
    const DevOp &o = op->view;
    IGE_REQUIRE(nc >= 1 && nc <= kRhsCols && op->d_rhs.n >= rhs_scratch_values(o, nc), "right-hand side scratch too small");
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
    if (o.scalar) hipLaunchKernelGGL(k_rhs_elem<true>, grid, dim3(256), shm, s, o, E, rw, nc, kind, cols, op->d_rhs.p);
    else hipLaunchKernelGGL(k_rhs_elem<false>, grid, dim3(256), shm, s, o, E, rw, nc, kind, cols, op->d_rhs.p);
    IGE_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_rhs_sum, dim3((unsigned)(((int64_t)o.N * nc + 255) / 256)), dim3(256), 0, s, o, nc, op->d_rhs.p, f);
    IGE_HIP(hipGetLastError());
}

}  // namespace ige
