// Element-local evaluation shared by the assembly kernels: patch geometry from the rational
// Bezier form, B-spline pieces, the local functions of an element.
#pragma once

#include <hip/hip_runtime.h>

#include "device_math.hpp"
#include "op.hpp"

namespace ige {
namespace {

typedef double dx4 __attribute__((ext_vector_type(4)));   // FP64 matrix-core accumulator

// Bernstein values and derivatives of degree deg <= kMaxP at x
__device__ inline void bernstein(int deg, double x, double *B, double *D)
{
    double T[kMaxP + 1];
    T[0] = 1.0;
    for (int k = 1; k < deg; ++k) {
        T[k] = x * T[k - 1];
        for (int i = k - 1; i >= 1; --i) T[i] = (1.0 - x) * T[i] + x * T[i - 1];
        T[0] = (1.0 - x) * T[0];
    }
    if (deg == 0) {
        B[0] = 1.0;
        D[0] = 0.0;
        return;
    }
    for (int i = 0; i <= deg; ++i) {
        const double lo = (i >= 1) ? T[i - 1] : 0.0;
        const double hi = (i <= deg - 1) ? T[i] : 0.0;
        D[i] = deg * (lo - hi);
        B[i] = (1.0 - x) * hi + x * lo;
    }
}

// 1-D spline pieces on element e at element-local x: degree p values/derivatives
// (derivatives w.r.t. the patch parameter) and degree p-1 values
__device__ inline void spline_pieces(const DevOp &o, int e, double x, double *Pv, double *Pd, double *Qv)
{
    const int p = o.p;
    double B[kMaxP + 1], D[kMaxP + 1];
    bernstein(p, x, B, D);
    for (int t = 0; t <= p; ++t) {
        double v = 0.0, d = 0.0;
        const double *c = o.ext_p + ((size_t)e * (p + 1) + t) * (p + 1);
        for (int a = 0; a <= p; ++a) {
            v += c[a] * B[a];
            d += c[a] * D[a];
        }
        Pv[t] = v;
        Pd[t] = d / o.h;
    }
    double Bq[kMaxP + 1], Dq[kMaxP + 1];
    bernstein(p - 1, x, Bq, Dq);
    for (int t = 0; t < p; ++t) {
        double v = 0.0;
        const double *c = o.ext_q + ((size_t)e * p + t) * p;
        for (int a = 0; a < p; ++a) v += c[a] * Bq[a];
        Qv[t] = v;
    }
}

// Fixed-degree variants (fully unrolled, no scratch): Bernstein values and
// derivatives, spline pieces and rational Bezier patch evaluation.
template <int DEG>
__device__ inline void bernstein_t(double x, double *B, double *D)
{
    if constexpr (DEG == 0) {
        B[0] = 1.0;
        D[0] = 0.0;
    } else {
        double T[DEG];
        T[0] = 1.0;
#pragma unroll
        for (int k = 1; k < DEG; ++k) {
            T[k] = x * T[k - 1];
#pragma unroll
            for (int i = k - 1; i >= 1; --i) T[i] = (1.0 - x) * T[i] + x * T[i - 1];
            T[0] = (1.0 - x) * T[0];
        }
#pragma unroll
        for (int i = 0; i <= DEG; ++i) {
            const double lo = (i >= 1) ? T[i >= 1 ? i - 1 : 0] : 0.0;
            const double hi = (i <= DEG - 1) ? T[i <= DEG - 1 ? i : 0] : 0.0;
            D[i] = DEG * (lo - hi);
            B[i] = (1.0 - x) * hi + x * lo;
        }
    }
}

// 1-D spline pieces of degree P and P - 1 at element-local x from the element's coefficients
// (degree P row by row, then degree P - 1); ih: 1 / element length
template <int P>
__device__ inline void spline_pieces_lds(const double *c, double ih, double x, double *Pv, double *Pd, double *Qv)
{
    double B[P + 1], D[P + 1];
    bernstein_t<P>(x, B, D);
#pragma unroll
    for (int t = 0; t <= P; ++t) {
        double v = 0.0, d = 0.0;
#pragma unroll
        for (int a = 0; a <= P; ++a) {
            v += c[t * (P + 1) + a] * B[a];
            d += c[t * (P + 1) + a] * D[a];
        }
        Pv[t] = v;
        Pd[t] = d * ih;
    }
    double Bq[P], Dq[P];
    bernstein_t<P - 1>(x, Bq, Dq);
#pragma unroll
    for (int t = 0; t < P; ++t) {
        double v = 0.0;
#pragma unroll
        for (int a = 0; a < P; ++a) v += c[(P + 1) * (P + 1) + t * P + a] * Bq[a];
        Qv[t] = v;
    }
}

// other degrees: out of line, so that its stack arrays do not enlarge the callers
__device__ __noinline__ void geom_eval_generic(const GeomView &g, int j, double u, double v, double X[3], double Xu[3],
                                               double Xv[3])
{
    bezier_eval(g, j, u, v, X, Xu, Xv);
}

// local function l of an element: (component, t1, t2); the scalar operator has the
// (p+1)^2 tensor B-splines, t2 major, in component 0
__device__ inline void local_index(const DevOp &o, int l, int &a, int &t1, int &t2)
{
    const int p = o.p;
    if (o.scalar) {
        a = 0;
        t2 = l / (p + 1);
        t1 = l % (p + 1);
        return;
    }
    const int n0 = p * (p + 1);
    if (l < n0) {
        a = 0;
        t2 = l / (p + 1);
        t1 = l % (p + 1);
    } else {
        a = 1;
        const int r = l - n0;
        t2 = r / p;
        t1 = r % p;
    }
}

// values of the local functions at element-local (x, y): Phi (3) and div, unsigned
// (scalar operator: Phi = 0 and the value times the surface element in place of div)
template <int NL>
__device__ inline void local_values(const DevOp &o, int e1, int e2, double x, double y, const double Fu[3],
                                    const double Fv[3], double Phi[NL][3], double Dv[NL])
{
    double Pu[kMaxP + 1], dPu[kMaxP + 1], Qu[kMaxP + 1], Pv[kMaxP + 1], dPv[kMaxP + 1], Qv[kMaxP + 1];
    spline_pieces(o, e1, x, Pu, dPu, Qu);
    spline_pieces(o, e2, y, Pv, dPv, Qv);
    if (o.scalar) {   // value times the surface element, no field part
        const double J = dm::surf_elem(Fu, Fv);
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            int a, t1, t2;
            local_index(o, l, a, t1, t2);
            Phi[l][0] = Phi[l][1] = Phi[l][2] = 0.0;
            Dv[l] = Pu[t1] * Pv[t2] * J;
        }
        return;
    }
#pragma unroll
    for (int l = 0; l < NL; ++l) {
        int a, t1, t2;
        local_index(o, l, a, t1, t2);
        double val, div;
        if (a == 0) {
            val = Pu[t1] * Qv[t2];
            div = dPu[t1] * Qv[t2];
        } else {
            val = Qu[t1] * Pv[t2];
            div = Qu[t1] * dPv[t2];
        }
        const double *F = (a == 0) ? Fu : Fv;
        Phi[l][0] = val * F[0];
        Phi[l][1] = val * F[1];
        Phi[l][2] = val * F[2];
        Dv[l] = div;
    }
}

__device__ inline void elem_of(const DevOp &o, int64_t e, int &j, int &e1, int &e2)
{
    const int nn = o.n * o.n;
    j = (int)(e / nn);
    const int r = (int)(e % nn);
    e2 = r / o.n;
    e1 = r % o.n;
}

__device__ inline void local_dof(const DevOp &o, int j, int e1, int e2, int l, int &idx, double &sg)
{
    int a, t1, t2;
    local_index(o, l, a, t1, t2);
    const size_t off = (((size_t)j * 2 + a) * o.nb + (e2 + t2)) * o.nb + (e1 + t1);
    idx = o.dof[off];
    sg = (double)o.sgn[off];
}

// FP64 matrix-core instruction 16x16x4: lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16]; accumulator register j of lane l holds D[l / 16 + 4 j][l % 16].
// Operand order: for step t a lane supplies the entry with quadrature index
// q = frag_q(t, lane) in reduction slot lane / 16, so that accumulator register j of
// a first product over tile qt is the operand of step t = 4 qt + j of a second.
__device__ inline int frag_q(int t, int lane) { return 16 * (t >> 2) + 4 * (t & 3) + (lane >> 4); }

}  // namespace
}  // namespace ige
