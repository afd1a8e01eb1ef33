// HIP kernels of the igaefie library (gfx950, wave64), by step of the path:
//
//   geometry   element_data / node_geometry : geometry from the rational Bezier form at
//              the regular Gauss points of every element and at the Chebyshev nodes of
//              every cluster
//   near field near_regular / near_singular : element-pair Galerkin quadrature,
//              accumulated into dense blocks over leaf function slots (regular pairs on
//              the FP64 matrix cores)
//   P2M        leaf moments, fused with the gather x_super = T x (1-D factors of T)
//   M2M        upward transfer of the moments (nested cluster bases)
//   M2L        coupling of admissible cluster pairs with the interpolated kernel
//   L2L        downward transfer
//   L2P        test-side moments, fused with the scatter T^T
//   near product near_blk + near_gather: product with the stored blocks and their
//              transposes, then a fixed-order sum per unknown
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "device_math.hpp"
#include "element.hpp"
#include "op.hpp"

namespace ige {

namespace {

constexpr int kWave = 64;

__device__ inline double2 cmul(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 cscale(double s, double2 a) { return make_double2(s * a.x, s * a.y); }
using dm::surf_elem;

// ---------------------------------------------------------------------------
// a0: element data at the regular Gauss points
// ---------------------------------------------------------------------------
// ePsiF[e][c][lt][t][lane] = ePsi[e][c][16 lt + lane % 16][frag_q(t, lane)] (zero padded
// to 16-row tiles in l and to 4*QT steps in q, QT = ceil(G2 / 16))
template <int NL>
__global__ void k_element_data(DevOp o, double *eX, double *ePsi, double *ePsiF, double *eC)
{
    const int64_t e = blockIdx.x;
    int j, e1, e2;
    elem_of(o, e, j, e1, e2);
    const int G2 = o.G2;
    for (int q = threadIdx.x; q < G2; q += blockDim.x) {
        const int a = q % o.g, b = q / o.g;
        const double x = o.gx[a], y = o.gx[b];
        const double u = (e1 + x) * o.h, v = (e2 + y) * o.h;
        double X[3], Fu[3], Fv[3];
        bezier_eval(o.geo, j, u, v, X, Fu, Fv);
        const double w = o.gw[a] * o.gw[b] * o.h * o.h;
        double Phi[NL][3], Dv[NL];
        local_values<NL>(o, e1, e2, x, y, Fu, Fv, Phi, Dv);
        for (int d = 0; d < 3; ++d) eX[((size_t)e * 3 + d) * G2 + q] = X[d];
        constexpr int LT = (NL + 15) / 16;
        const int T = 4 * ((G2 + 15) / 16);
        const int t = 4 * (q / 16) + (q % 16) / 4, lq = 16 * (q % 4);
        double *F = ePsiF + (size_t)e * 4 * LT * T * 64;
        for (int l = 0; l < NL; ++l) {
            for (int d = 0; d < 3; ++d) ePsi[(((size_t)e * 4 + d) * NL + l) * G2 + q] = w * Phi[l][d];
            ePsi[(((size_t)e * 4 + 3) * NL + l) * G2 + q] = w * Dv[l];
            const int lt = l / 16, lane = l % 16 + lq;
            for (int d = 0; d < 3; ++d) F[((d * LT + lt) * T + t) * 64 + lane] = w * Phi[l][d];
            F[((3 * LT + lt) * T + t) * 64 + lane] = w * Dv[l];
        }
    }
    if (threadIdx.x < 4) {
        const int k = threadIdx.x;
        const int cu = (k == 1 || k == 2) ? 1 : 0, cv = (k >= 2) ? 1 : 0;
        double X[3], Fu[3], Fv[3];
        bezier_eval(o.geo, j, (e1 + cu) * o.h, (e2 + cv) * o.h, X, Fu, Fv);
        for (int d = 0; d < 3; ++d) eC[(size_t)e * 12 + k * 3 + d] = X[d];
    }
}

// a0: geometry at the Chebyshev nodes of every cluster
__global__ void k_node_geometry(DevOp o, int NC, double *nodeX, double *nodeT)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)NC * o.Q) return;
    const int gc = (int)(t / o.Q), mm = (int)(t % o.Q);
    int lvl = 0;
    while (lvl < o.L && gc >= o.lvl_off[lvl + 1]) ++lvl;
    const int id = gc - (int)o.lvl_off[lvl];
    const int S = 1 << lvl;
    const int j = id / (S * S), r = id % (S * S), k2 = r / S, k1 = r % S;
    // the nodes of the level's degree (stored with the stride of the largest degree)
    const int Q1l = o.ql[lvl] + 1;
    if (mm >= Q1l * Q1l) return;
    const int m1 = mm % Q1l, m2 = mm / Q1l;
    const double *xn = o.xnl + (size_t)lvl * kMaxQ1;
    const double H = 1.0 / S;
    double X[3], Fu[3], Fv[3];
    bezier_eval(o.geo, j, (k1 + xn[m1]) * H, (k2 + xn[m2]) * H, X, Fu, Fv);
    for (int d = 0; d < 3; ++d) {
        nodeX[((size_t)gc * 3 + d) * o.Q + mm] = X[d];
        nodeT[((size_t)gc * 6 + d) * o.Q + mm] = Fu[d];
        nodeT[((size_t)gc * 6 + 3 + d) * o.Q + mm] = Fv[d];
    }
}

// ---------------------------------------------------------------------------
// a3: P2M on the leaf clusters, fused with the gather of the glued coefficients
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_p2m(DevOp o, const double2 *x, double2 *mom, double2 *src)
{
    extern __shared__ double2 sm2[];
    const int id = blockIdx.x;            // leaf id
    const int SL = o.SL, s = o.s, p = o.p, Q1 = o.Q1, Q = o.Q, RL = o.rowlen;
    const int j = id / (SL * SL), r = id % (SL * SL), k2 = r / SL, k1 = r % SL;
    const int gc = (int)o.lvl_off[o.L] + id;
    const int w1a = s + p, w2a = s + p - 1;   // component 0 block: [w2a][w1a]
    const int w1b = s + p - 1, w2b = s + p;   // component 1 block: [w2b][w1b]
    double2 *X1 = sm2;                        // [w2a][w1a]
    double2 *X2 = X1 + w2a * w1a;             // [w2b][w1b]
    double2 *Z1 = X2 + w2b * w1b;             // [w2a][Q1]
    double2 *Zd = Z1 + w2a * Q1;              // [w2a][Q1]
    double2 *Z2 = Zd + w2a * Q1;              // [w2b][Q1]
    // Mp, Mq, Mdp of k1, then of k2, read with the coefficients
    const int QR = Q1 * RL;
    double *Mt = reinterpret_cast<double *>(Z2 + w2b * Q1);
    for (int i = threadIdx.x; i < 6 * QR; i += blockDim.x) {
        const int a = i / QR, m = i - a * QR, k = a < 3 ? k1 : k2, b = a % 3;
        Mt[i] = (b == 0 ? o.Mp : (b == 1 ? o.Mq : o.Mdp))[(size_t)k * QR + m];
    }
    for (int i = threadIdx.x; i < w2a * w1a; i += blockDim.x) {
        const int i2 = i / w1a, i1 = i % w1a;
        const size_t off = (((size_t)j * 2 + 0) * o.nb + (k2 * s + i2)) * o.nb + (k1 * s + i1);
        const double2 v = x[o.dof[off]];
        X1[i] = cscale((double)o.sgn[off], v);
    }
    for (int i = threadIdx.x; i < w2b * w1b; i += blockDim.x) {
        const int i2 = i / w1b, i1 = i % w1b;
        const size_t off = (((size_t)j * 2 + 1) * o.nb + (k2 * s + i2)) * o.nb + (k1 * s + i1);
        const double2 v = x[o.dof[off]];
        X2[i] = cscale((double)o.sgn[off], v);
    }
    __syncthreads();
    const double *Mpu = Mt, *Mqu = Mt + QR, *Mdu = Mt + 2 * QR, *Mpv = Mt + 3 * QR, *Mqv = Mt + 4 * QR, *Mdv = Mt + 5 * QR;
    // contract along u
    for (int i = threadIdx.x; i < w2a * Q1; i += blockDim.x) {
        const int i2 = i / Q1, m1 = i % Q1;
        double2 z = make_double2(0, 0), zd = make_double2(0, 0);
        for (int i1 = 0; i1 < w1a; ++i1) {
            const double2 v = X1[i2 * w1a + i1];
            z = cadd(z, cscale(Mpu[m1 * RL + i1], v));
            zd = cadd(zd, cscale(Mdu[m1 * RL + i1], v));
        }
        Z1[i] = z;
        Zd[i] = zd;
    }
    for (int i = threadIdx.x; i < w2b * Q1; i += blockDim.x) {
        const int i2 = i / Q1, m1 = i % Q1;
        double2 z = make_double2(0, 0);
        for (int i1 = 0; i1 < w1b; ++i1) z = cadd(z, cscale(Mqu[m1 * RL + i1], X2[i2 * w1b + i1]));
        Z2[i] = z;
    }
    __syncthreads();
    // contract along v; cartesian source vectors
    for (int mm = threadIdx.x; mm < Q; mm += blockDim.x) {
        const int m2 = mm / Q1, m1 = mm % Q1;
        double2 s1 = make_double2(0, 0), s2v = make_double2(0, 0), d = make_double2(0, 0);
        for (int i2 = 0; i2 < w2a; ++i2) {
            s1 = cadd(s1, cscale(Mqv[m2 * RL + i2], Z1[i2 * Q1 + m1]));
            d = cadd(d, cscale(Mqv[m2 * RL + i2], Zd[i2 * Q1 + m1]));
        }
        for (int i2 = 0; i2 < w2b; ++i2) {
            s2v = cadd(s2v, cscale(Mpv[m2 * RL + i2], Z2[i2 * Q1 + m1]));
            d = cadd(d, cscale(Mdv[m2 * RL + i2], Z2[i2 * Q1 + m1]));
        }
        double2 *M = mom + (size_t)gc * 3 * Q;
        M[mm] = s1;
        M[Q + mm] = s2v;
        M[2 * Q + mm] = d;
        const double *T = o.nodeT + (size_t)gc * 6 * Q;
        double2 *S = src + (size_t)gc * 4 * Q;
        for (int k = 0; k < 3; ++k) S[k * Q + mm] = cadd(cscale(T[k * Q + mm], s1), cscale(T[(3 + k) * Q + mm], s2v));
        S[3 * Q + mm] = d;
    }
}

// scalar single layer: leaf moments d = (M_p (x) M_p) c of the tensor B-spline
// coefficients over the leaf's W x W window (fields 0 and 1 stay zero), and the source
// values |J(x_m)| d at the nodes
__global__ __launch_bounds__(256) void k_p2m_sc(DevOp o, const double2 *x, double2 *mom, double2 *src)
{
    extern __shared__ double2 sm2[];
    const int id = blockIdx.x;
    const int SL = o.SL, s = o.s, p = o.p, Q1 = o.Q1, Q = o.Q, RL = o.rowlen, W = s + p;
    const int j = id / (SL * SL), r = id % (SL * SL), k2 = r / SL, k1 = r % SL;
    const int gc = (int)o.lvl_off[o.L] + id;
    double2 *X = sm2;           // [W (i2)][W (i1)]
    double2 *Z = X + W * W;     // [W (i2)][Q1 (m1)]
    for (int i = threadIdx.x; i < W * W; i += blockDim.x) {
        const int i2 = i / W, i1 = i % W;
        X[i] = x[o.dof[((size_t)j * 2 * o.nb + (k2 * s + i2)) * o.nb + (k1 * s + i1)]];
    }
    __syncthreads();
    const double *Mpu = o.Mp + (size_t)k1 * Q1 * RL, *Mpv = o.Mp + (size_t)k2 * Q1 * RL;
    for (int i = threadIdx.x; i < W * Q1; i += blockDim.x) {
        const int i2 = i / Q1, m1 = i % Q1;
        double2 z = make_double2(0, 0);
        for (int i1 = 0; i1 < W; ++i1) z = cadd(z, cscale(Mpu[m1 * RL + i1], X[i2 * W + i1]));
        Z[i] = z;
    }
    __syncthreads();
    for (int mm = threadIdx.x; mm < Q; mm += blockDim.x) {
        const int m2 = mm / Q1, m1 = mm % Q1;
        double2 d = make_double2(0, 0);
        for (int i2 = 0; i2 < W; ++i2) d = cadd(d, cscale(Mpv[m2 * RL + i2], Z[i2 * Q1 + m1]));
        double2 *M = mom + (size_t)gc * 3 * Q;
        M[mm] = make_double2(0, 0);
        M[Q + mm] = make_double2(0, 0);
        M[2 * Q + mm] = d;
        const double *T = o.nodeT + (size_t)gc * 6 * Q;
        const double Fu[3] = {T[mm], T[Q + mm], T[2 * Q + mm]}, Fv[3] = {T[3 * Q + mm], T[4 * Q + mm], T[5 * Q + mm]};
        double2 *S = src + (size_t)gc * 4 * Q;
        for (int k = 0; k < 3; ++k) S[k * Q + mm] = make_double2(0, 0);
        S[3 * Q + mm] = cscale(surf_elem(Fu, Fv), d);
    }
}

// ---------------------------------------------------------------------------
// a4: M2M, parents on level lvl from children on lvl+1
// parent[m2][m1] = sum_c sum_{n1,n2} T_c1[n1][m1] T_c2[n2][m2] child_c[n2][n1]
// ---------------------------------------------------------------------------
// Bound by latency (a few dozen to a few hundred workgroups, two short sums): the transfer
// matrices come to shared memory with the children's moments, the node tangents to registers,
// a workgroup has a thread per value and the sums over the four children are taken apart.
// 96 parents of 225 nodes: 27.9 us with 256 threads and the matrices from
// global memory, 11.5 now; 24 of 64 nodes: 7.8 and 6.4.
__global__ __launch_bounds__(1024) void k_m2m(DevOp o, int lvl, double2 *mom, double2 *src)
{
    extern __shared__ double2 sm2[];
    const int id = blockIdx.x;
    const int S = 1 << lvl, Q1 = o.Q1, Q = o.Q;
    const int j = id / (S * S), r = id % (S * S), k2 = r / S, k1 = r % S;
    const int gc = (int)o.lvl_off[lvl] + id;
    double2 *ch = sm2;            // [4 children][3 fields][Q]
    double2 *W = ch + 12 * Q;     // [4][3][Q1 (n2)][Q1 (m1)]
    double *T = reinterpret_cast<double *>(W + 12 * Q);   // [2][Q1 (n)][Q1 (m)]
    // one read phase: the moments of the four children, the transfer matrices, this thread's tangents
    for (int i = threadIdx.x; i < 12 * Q; i += blockDim.x) {
        const int c = i / (3 * Q), rem = i % (3 * Q);
        const int c1 = c & 1, c2 = c >> 1;
        const int cgc = (int)o.lvl_off[lvl + 1] + (j * 2 * S + 2 * k2 + c2) * 2 * S + 2 * k1 + c1;
        ch[i] = mom[(size_t)cgc * 3 * Q + rem];
    }
    for (int i = threadIdx.x; i < 2 * Q; i += blockDim.x) T[i] = i < Q ? o.T0[i] : o.T1[i - Q];
    double F[6];   // a workgroup has at least Q threads
#pragma unroll
    for (int k = 0; k < 6; ++k) F[k] = threadIdx.x < Q ? o.nodeT[((size_t)gc * 6 + k) * Q + threadIdx.x] : 0.0;
    __syncthreads();
    // contract along u: W[c][f][n2][m1] = sum_n1 T_c1[n1][m1] child_c[f][n2][n1]
    for (int i = threadIdx.x; i < 12 * Q; i += blockDim.x) {
        const int cf = i / Q, nm = i - cf * Q, n2 = nm / Q1, m1 = nm - n2 * Q1;
        const double *Tu = T + (cf / 3 & 1) * Q + m1;
        const double2 *v = ch + cf * Q + n2 * Q1;
        double2 z = make_double2(0, 0);
        for (int n1 = 0; n1 < Q1; ++n1) z = cadd(z, cscale(Tu[n1 * Q1], v[n1]));
        W[i] = z;
    }
    __syncthreads();
    // contract along v (into the place of the children, no longer needed)
    for (int i = threadIdx.x; i < 12 * Q; i += blockDim.x) {
        const int cf = i / Q, mm = i - cf * Q, m2 = mm / Q1, m1 = mm - m2 * Q1;
        const double *Tv = T + (cf / 6) * Q + m2;
        const double2 *v = W + cf * Q + m1;
        double2 z = make_double2(0, 0);
        for (int n2 = 0; n2 < Q1; ++n2) z = cadd(z, cscale(Tv[n2 * Q1], v[n2 * Q1]));
        ch[i] = z;
    }
    __syncthreads();
    const int mm = threadIdx.x;
    if (mm >= Q) return;
    double2 f[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {   // sum of the children
        f[k] = ch[k * Q + mm];
        for (int c = 1; c < 4; ++c) f[k] = cadd(f[k], ch[(c * 3 + k) * Q + mm]);
    }
    double2 *M = mom + (size_t)gc * 3 * Q, *Sv = src + (size_t)gc * 4 * Q;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        M[k * Q + mm] = f[k];
        Sv[k * Q + mm] = cadd(cscale(F[k], f[0]), cscale(F[3 + k], f[1]));
    }
    // scalar: the moments times the surface element at the node
    Sv[3 * Q + mm] = o.scalar ? cscale(surf_elem(F, F + 3), f[2]) : f[2];
}

// Levels of a smaller interpolation degree q_l (variable order): their moments are the
// exact restriction of the degree-q moments, m_l = (R_l (x) R_l)^T m with
// R_l[n][m] = L^{q_l}_m(x^q_n), turned into the source fields at the level's own nodes;
// the coupling's local expansions go back through R_l (x) R_l before L2L.
__global__ __launch_bounds__(256) void k_restrict(DevOp o, int lvl, const double2 *mom, double2 *src)
{
    extern __shared__ double2 sm2[];
    const int gc = (int)o.lvl_off[lvl] + blockIdx.x;
    const int Q1h = o.Q1, Qs = o.Q, Q1l = o.ql[lvl] + 1, Ql = Q1l * Q1l;
    const double *R = o.Rl + (size_t)lvl * Q1h * Q1h;   // [n][m], m < Q1l
    double2 *M = sm2;               // [3][Qs]
    double2 *Z = M + 3 * Qs;        // [3][Q1h (n2)][Q1l (m1)]
    for (int i = threadIdx.x; i < 3 * Qs; i += blockDim.x) M[i] = mom[(size_t)gc * 3 * Qs + i];
    __syncthreads();
    for (int i = threadIdx.x; i < 3 * Q1h * Q1l; i += blockDim.x) {
        const int f = i / (Q1h * Q1l), r = i % (Q1h * Q1l), n2 = r / Q1l, m1 = r % Q1l;
        double2 z = make_double2(0, 0);
        for (int n1 = 0; n1 < Q1h; ++n1) z = cadd(z, cscale(R[n1 * Q1h + m1], M[f * Qs + n2 * Q1h + n1]));
        Z[i] = z;
    }
    __syncthreads();
    const double *T = o.nodeT + (size_t)gc * 6 * Qs;
    double2 *Sv = src + (size_t)gc * 4 * Qs;
    for (int mm = threadIdx.x; mm < Ql; mm += blockDim.x) {
        const int m2 = mm / Q1l, m1 = mm % Q1l;
        double2 sf[3];
        for (int f = 0; f < 3; ++f) {
            double2 v = make_double2(0, 0);
            for (int n2 = 0; n2 < Q1h; ++n2) v = cadd(v, cscale(R[n2 * Q1h + m2], Z[(f * Q1h + n2) * Q1l + m1]));
            sf[f] = v;
        }
        const double Fu[3] = {T[mm], T[Qs + mm], T[2 * Qs + mm]}, Fv[3] = {T[3 * Qs + mm], T[4 * Qs + mm], T[5 * Qs + mm]};
        if (o.scalar) {
            for (int k = 0; k < 3; ++k) Sv[k * Qs + mm] = make_double2(0, 0);
            Sv[3 * Qs + mm] = cscale(surf_elem(Fu, Fv), sf[2]);
        } else {
            for (int k = 0; k < 3; ++k) Sv[k * Qs + mm] = cadd(cscale(Fu[k], sf[0]), cscale(Fv[k], sf[1]));
            Sv[3 * Qs + mm] = sf[2];
        }
    }
}

__global__ __launch_bounds__(256) void k_lift(DevOp o, int lvl, double2 *loc)
{
    extern __shared__ double2 sm2[];
    const int gc = (int)o.lvl_off[lvl] + blockIdx.x;
    const int Q1h = o.Q1, Qs = o.Q, Q1l = o.ql[lvl] + 1, Ql = Q1l * Q1l;
    const double *R = o.Rl + (size_t)lvl * Q1h * Q1h;
    double2 *A = sm2;               // [3][Ql]
    double2 *Y = A + 3 * Ql;        // [3][Q1l (m2)][Q1h (n1)]
    double2 *Lc = loc + (size_t)gc * 3 * Qs;
    for (int i = threadIdx.x; i < 3 * Ql; i += blockDim.x) A[i] = Lc[(i / Ql) * Qs + i % Ql];
    __syncthreads();
    for (int i = threadIdx.x; i < 3 * Q1l * Q1h; i += blockDim.x) {
        const int f = i / (Q1l * Q1h), r = i % (Q1l * Q1h), m2 = r / Q1h, n1 = r % Q1h;
        double2 y = make_double2(0, 0);
        for (int m1 = 0; m1 < Q1l; ++m1) y = cadd(y, cscale(R[n1 * Q1h + m1], A[f * Ql + m2 * Q1l + m1]));
        Y[i] = y;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 3 * Qs; i += blockDim.x) {
        const int f = i / Qs, nn = i % Qs, n2 = nn / Q1h, n1 = nn % Q1h;
        double2 v = make_double2(0, 0);
        for (int m2 = 0; m2 < Q1l; ++m2) v = cadd(v, cscale(R[n2 * Q1h + m2], Y[(f * Q1l + m2) * Q1h + n1]));
        Lc[i] = v;
    }
}

// ---------------------------------------------------------------------------
// a5: M2L of one column with FP32 kernel values (FP64: coupling_sym.hip). Work item = (target cluster, range of far partners).  The localized
// kernel is interpolated in both parameter squares:
//   u[m] += sum_m' G(|x_m - x'_m'|) (v_x, v_y, v_z, d)'[m']
// Threads: kM2LNT target nodes each (register blocking: every source value read
// from LDS serves kM2LNT targets) x a part of the source nodes; the parts are
// summed once per work item through LDS.
// ---------------------------------------------------------------------------
constexpr int kM2LThreads = 256;
constexpr int kM2LNT = 3;

__global__ __launch_bounds__(kM2LThreads) void k_m2l(DevOp o, int nwork, const M2LWork *work, const int32_t *partner,
                                                      const double2 *src, double2 *part)
{
    using T = float;
    using C = float2;
    extern __shared__ double smd[];
    // one work item per workgroup, or (a grid smaller than the work) items blockIdx.x,
    // blockIdx.x + gridDim.x, ...
    for (int wi = blockIdx.x; wi < nwork; wi += gridDim.x) {
    const M2LWork wk = work[wi];
    // nodes of the target's level (the partners are on the same level); per-cluster
    // arrays keep the stride Qs of the largest degree
    const int Qs = o.Q;
    int lvw = 0;
    while (lvw < o.L && wk.tgt >= o.lvl_off[lvw + 1]) ++lvw;
    const int Q = (o.ql[lvw] + 1) * (o.ql[lvw] + 1);
    const int TPG = (Q + kM2LNT - 1) / kM2LNT;
    const int S = min(kM2LThreads / TPG, Q);
    const int SP = (Q + S - 1) / S;
    const int tid = threadIdx.x;
    const int mt = tid % TPG, sp = tid / TPG;
    const bool active = sp < S;
    // node-major staging, so one address (and immediate offsets) reaches a node's data
    T *sX = reinterpret_cast<T *>(smd);                        // [Q][4]: x, y, z, unused
    C *sV = reinterpret_cast<C *>(smd + (4 * Q * (int)sizeof(T) + 15) / 16 * 2);   // [Q][4], 16-B aligned after sX
    double2 *red = reinterpret_cast<double2 *>(smd);           // [S][Q][2] after the partner loop
    const T kap = (T)o.kappa;
    T xt[kM2LNT][3];
    bool val[kM2LNT];
    C acc[kM2LNT][4];
    const double *Xt = o.nodeX + (size_t)wk.tgt * 3 * Qs;
#pragma unroll
    for (int k = 0; k < kM2LNT; ++k) {
        const int mm = mt + k * TPG;
        val[k] = active && mm < Q;
        const int mc = val[k] ? mm : 0;
        xt[k][0] = (T)Xt[mc];
        xt[k][1] = (T)Xt[Qs + mc];
        xt[k][2] = (T)Xt[2 * Qs + mc];
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[k][j] = C{0, 0};
    }
    const int mb = min(Q, sp * SP), me = min(Q, mb + SP);
    for (int kp = wk.beg; kp < wk.end; ++kp) {
        const int sc = partner[kp];
        __syncthreads();
        const double *Xs = o.nodeX + (size_t)sc * 3 * Qs;
        const double2 *Vs = src + (size_t)sc * 4 * Qs;
        for (int i = tid; i < 3 * Q; i += kM2LThreads) sX[(i % Q) * 4 + i / Q] = (T)Xs[(i / Q) * Qs + i % Q];
        for (int i = tid; i < 4 * Q; i += kM2LThreads) sV[(i % Q) * 4 + i / Q] = dm::to_f(Vs[(i / Q) * Qs + i % Q]);
        __syncthreads();
        if (active) {
            for (int ms = mb; ms < me; ++ms) {
                const T x0 = sX[4 * ms], x1 = sX[4 * ms + 1], x2 = sX[4 * ms + 2];
                const C v0 = sV[4 * ms], v1 = sV[4 * ms + 1], v2 = sV[4 * ms + 2], v3 = sV[4 * ms + 3];
#pragma unroll
                for (int k = 0; k < kM2LNT; ++k) {
                    const T d0 = xt[k][0] - x0, d1 = xt[k][1] - x1, d2 = xt[k][2] - x2;
                    const C G = dm::helmholtz_r2(kap, fma(d0, d0, fma(d1, d1, d2 * d2)));
                    acc[k][0] = dm::cmac(acc[k][0], G, v0);
                    acc[k][1] = dm::cmac(acc[k][1], G, v1);
                    acc[k][2] = dm::cmac(acc[k][2], G, v2);
                    acc[k][3] = dm::cmac(acc[k][3], G, v3);
                }
            }
        }
    }
    // the source parts summed in a fixed order, two fields at a time (half the
    // shared memory of all four: one more workgroup per CU)
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kM2LNT; ++k)
            if (val[k]) {
                const int mm = mt + k * TPG;
#pragma unroll
                for (int j = 0; j < 2; ++j) red[((size_t)sp * Q + mm) * 2 + j] = dm::to_d(acc[k][2 * hf + j]);
            }
        __syncthreads();
        for (int i = tid; i < 2 * Q; i += kM2LThreads) {
            const int j = i / Q, mm = i % Q;
            double2 v = make_double2(0, 0);
            for (int q2 = 0; q2 < S; ++q2) v = cadd(v, red[((size_t)q2 * Q + mm) * 2 + j]);
            part[((size_t)wi * 4 + 2 * hf + j) * Qs + mm] = v;
        }
    }
    __syncthreads();   // the next item's staging reuses the shared memory
    }
}

// sum the partial couplings of every cluster (fixed order) and convert to the
// test-side fields t^a = d_aF . u_xyz, t^d = -kappa^-2 u_d
__global__ void k_m2l_reduce(DevOp o, const int32_t *wrk_of_tgt, const double2 *part, double2 *loc)
{
    const int gc = blockIdx.x, Qs = o.Q;
    int lvl = 0;
    while (lvl < o.L && gc >= o.lvl_off[lvl + 1]) ++lvl;
    const int Q = (o.ql[lvl] + 1) * (o.ql[lvl] + 1);   // nodes of the level (stride Qs)
    const int b = wrk_of_tgt[gc], e = wrk_of_tgt[gc + 1];
    const double ik2 = 1.0 / (o.kappa * o.kappa);
    for (int mm = threadIdx.x; mm < Q; mm += blockDim.x) {
        double2 u[4] = {make_double2(0, 0), make_double2(0, 0), make_double2(0, 0), make_double2(0, 0)};
        for (int w = b; w < e; ++w)
            for (int k = 0; k < 4; ++k) u[k] = cadd(u[k], part[((size_t)w * 4 + k) * Qs + mm]);
        const double *T = o.nodeT + (size_t)gc * 6 * Qs;
        double2 t1 = make_double2(0, 0), t2 = make_double2(0, 0);
        for (int k = 0; k < 3; ++k) {
            t1 = cadd(t1, cscale(T[k * Qs + mm], u[k]));
            t2 = cadd(t2, cscale(T[(3 + k) * Qs + mm], u[k]));
        }
        double2 *L = loc + (size_t)gc * 3 * Qs;
        if (o.scalar) {   // scalar: t = |J(x_m)| u (the localized kernel's target surface element)
            const double Fu[3] = {T[mm], T[Qs + mm], T[2 * Qs + mm]}, Fv[3] = {T[3 * Qs + mm], T[4 * Qs + mm], T[5 * Qs + mm]};
            L[mm] = make_double2(0, 0);
            L[Qs + mm] = make_double2(0, 0);
            L[2 * Qs + mm] = cscale(surf_elem(Fu, Fv), u[3]);
            continue;
        }
        L[mm] = t1;
        L[Qs + mm] = t2;
        L[2 * Qs + mm] = cscale(-ik2, u[3]);
    }
}

// ---------------------------------------------------------------------------
// a6: L2L, children on level lvl from parents on lvl-1
// child[n2][n1] += sum_{m1,m2} T_c1[n1][m1] T_c2[n2][m2] parent[m2][m1]
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_l2l(DevOp o, int lvl, double2 *loc)
{
    extern __shared__ double2 sm2[];
    const int id = blockIdx.x;
    const int S = 1 << lvl, Q1 = o.Q1, Q = o.Q;
    const int j = id / (S * S), r = id % (S * S), k2 = r / S, k1 = r % S;
    const int gc = (int)o.lvl_off[lvl] + id;
    const int Sp = S / 2;
    const int pgc = (int)o.lvl_off[lvl - 1] + (j * Sp + k2 / 2) * Sp + k1 / 2;
    const int c1 = k1 & 1, c2 = k2 & 1;
    const double *Tu = c1 ? o.T1 : o.T0, *Tv = c2 ? o.T1 : o.T0;
    const double2 *par = loc + (size_t)pgc * 3 * Q;
    double2 *W = sm2;   // [3][Q1 (m2)][Q1 (n1)]
    for (int i = threadIdx.x; i < 3 * Q; i += blockDim.x) {
        const int f = i / Q, rem = i % Q, m2 = rem / Q1, n1 = rem % Q1;
        double2 z = make_double2(0, 0);
        for (int m1 = 0; m1 < Q1; ++m1) z = cadd(z, cscale(Tu[n1 * Q1 + m1], par[f * Q + m2 * Q1 + m1]));
        W[i] = z;
    }
    __syncthreads();
    double2 *ch = loc + (size_t)gc * 3 * Q;
    for (int i = threadIdx.x; i < 3 * Q; i += blockDim.x) {
        const int f = i / Q, rem = i % Q, n2 = rem / Q1, n1 = rem % Q1;
        double2 z = ch[i];
        for (int m2 = 0; m2 < Q1; ++m2) z = cadd(z, cscale(Tv[n2 * Q1 + m2], W[f * Q + m2 * Q1 + n1]));
        ch[i] = z;
    }
}

// ---------------------------------------------------------------------------
// a8: near-field product.  A workgroup streams rc rows of one stored block B
// (target leaf t, source leaf s) once: every row gives the row partial
// (B x_s)[k] and, for t != s, the same loads give the column partials of B^T x_t
// over the chunk.  Lanes own columns (coalesced 16-byte loads, bypassing the
// caches); the four waves take every fourth row and combine their column
// partials in a fixed order.
// ---------------------------------------------------------------------------
typedef double d2v __attribute__((ext_vector_type(2)));

__device__ inline double wave_sum(double v)
{
#pragma unroll
    for (int off = kWave / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

__device__ inline d2v ld_blk(const double2 *B, size_t i)
{
    return __builtin_nontemporal_load(reinterpret_cast<const d2v *>(B) + i);
}

template <int U>
__global__ __launch_bounds__(256) void k_near_blk(DevOp o, const double2 *x, double2 *part)
{
    __shared__ double2 sxr[64 * U];
    __shared__ double2 syc[3][64 * U];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t b = blockIdx.x / o.nch;
    const int ch = blockIdx.x % o.nch;
    const int lt = o.bpair[2 * b], ls = o.bpair[2 * b + 1];
    const int nF = o.nF, r0 = ch * o.rc, r1 = min(nF, r0 + o.rc);
    d2v xc[U], yc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int c = lane + 64 * u;
        const int d = c < nF ? o.leafdof[(size_t)ls * nF + c] : -1;
        const double2 v = d >= 0 ? x[d] : make_double2(0.0, 0.0);
        xc[u] = d2v{v.x, v.y};
        yc[u] = d2v{0.0, 0.0};
    }
    for (int k = threadIdx.x; k < r1 - r0; k += blockDim.x) {
        const int d = o.leafdof[(size_t)lt * nF + r0 + k];
        sxr[k] = d >= 0 ? x[d] : make_double2(0.0, 0.0);
    }
    __syncthreads();
    const double2 *B = o.bval + (size_t)b * nF * nF;
    int r = r0 + wv;
    // RS rows per step (r, r + 4, ...): RS U independent streaming loads in flight per
    // lane; the last step of a wave may hold fewer rows (the others load and add zeros)
    constexpr int RS = 2;
    for (; r < r1; r += 4 * RS) {
        d2v al[RS][U];
#pragma unroll
        for (int q = 0; q < RS; ++q)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = lane + 64 * u;
                al[q][u] = (c < nF && r + 4 * q < r1) ? ld_blk(B, (size_t)(r + 4 * q) * nF + c) : d2v{0.0, 0.0};
            }
        double2 xq[RS];
        double re[RS], im[RS];
#pragma unroll
        for (int q = 0; q < RS; ++q) {
            xq[q] = r + 4 * q < r1 ? sxr[r + 4 * q - r0] : make_double2(0.0, 0.0);
            re[q] = 0.0;
            im[q] = 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            d2v a[RS];
#pragma unroll
            for (int q = 0; q < RS; ++q) a[q] = al[q][u];
#pragma unroll
            for (int q = 0; q < RS; ++q) {
                re[q] = fma(a[q].x, xc[u].x, fma(-a[q].y, xc[u].y, re[q]));
                im[q] = fma(a[q].x, xc[u].y, fma(a[q].y, xc[u].x, im[q]));
            }
#pragma unroll
            for (int q = 0; q < RS; ++q) {
                yc[u].x = fma(a[q].x, xq[q].x, fma(-a[q].y, xq[q].y, yc[u].x));
                yc[u].y = fma(a[q].x, xq[q].y, fma(a[q].y, xq[q].x, yc[u].y));
            }
        }
        // the 2 RS row sums over the wave by recursive halving (one value per lane group)
        double v[2 * RS];
#pragma unroll
        for (int q = 0; q < RS; ++q) {
            v[2 * q] = re[q];
            v[2 * q + 1] = im[q];
        }
        const double tot = dm::Halve<2 * RS>::run(v, lane, 32);
        constexpr int SH = 6 - dm::log2c<2 * RS>();
        if ((lane & ((1 << SH) - 1)) == 0) {
            const int k = lane >> SH;   // value 2 q + (0: real, 1: imaginary part)
            if (r + 4 * (k >> 1) < r1)
                reinterpret_cast<double *>(part)[2 * ((size_t)b * nF + r + 4 * (k >> 1)) + (k & 1)] = tot;
        }
    }
    if (lt == ls) return;   // diagonal block: no transposed product (uniform branch)
    if (wv > 0)
#pragma unroll
        for (int u = 0; u < U; ++u) syc[wv - 1][lane + 64 * u] = make_double2(yc[u].x, yc[u].y);
    __syncthreads();
    if (wv == 0) {
        double2 *cp = part + (size_t)o.nblk * nF + ((size_t)b * o.nch + ch) * nF;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = lane + 64 * u;
            if (c < nF) {
                const double2 s1 = syc[0][c], s2 = syc[1][c], s3 = syc[2][c];
                cp[c] = make_double2(((yc[u].x + s1.x) + s2.x) + s3.x, ((yc[u].y + s1.y) + s2.y) + s3.y);
            }
        }
    }
}

// y[i] = sum of the partial results of unknown i: 16 lanes take every 16th entry of
// its list, then a fixed butterfly (the order does not depend on the launch)
__global__ __launch_bounds__(256) void k_near_gather(int N, const int64_t *ptr, const int32_t *idx,
                                                     const double2 *part, double2 *y)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int i = (int)(t >> 4), sub = (int)(t & 15);
    double re = 0.0, im = 0.0;
    if (i < N)
        for (int64_t k = ptr[i] + sub; k < ptr[i + 1]; k += 16) {
            const double2 v = part[idx[k]];
            re += v.x;
            im += v.y;
        }
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) {
        re += __shfl_xor(re, off, 16);
        im += __shfl_xor(im, off, 16);
    }
    if (i < N && sub == 0) y[i] = make_double2(re, im);
}

// ---------------------------------------------------------------------------
// a7: L2P.  Per leaf cluster, the test-side moments of the local spline pieces
// against the local fields (tensor contraction, u then v):
//   Y0[i2][i1] = sum Mp(k1)[m1][i1] Mq(k2)[m2][i2] t^1[m2][m1] + Mdp(k1) Mq(k2) t^d
//   Y1[i2][i1] = sum Mq(k1)[m1][i1] Mp(k2)[m2][i2] t^2[m2][m1] + Mq(k1) Mdp(k2) t^d
// then one thread per unknown gathers (with the gluing sign) the entries of the
// leaf clusters that its incarnations touch: the scatter T^T without atomics.
// ---------------------------------------------------------------------------
// With the expansions of the parents (down): the leaf's own L2L comes first, in the same
// workgroup.  Bound by latency: fields and tables come to shared memory in one read phase.
__device__ __forceinline__ void leaf_l2l(const DevOp &o, int k1, int k2, int Q1, int Q, double2 *t, const double2 *par, double2 *W,
                                         const double *T, int f0, int nf)
{
    // t[f][n2][n1] += sum T_c2[n2][m2] sum T_c1[n1][m1] par[f][m2][m1] (fields f0 .. f0 + nf - 1)
    const double *Tu = T + (k1 & 1) * Q, *Tv = T + (k2 & 1) * Q;
    for (int i = threadIdx.x; i < nf * Q; i += blockDim.x) {
        const int f = i / Q, rem = i - f * Q, m2 = rem / Q1, n1 = rem - m2 * Q1;
        double2 z = make_double2(0, 0);
        for (int m1 = 0; m1 < Q1; ++m1) z = cadd(z, cscale(Tu[n1 * Q1 + m1], par[(f0 + f) * Q + m2 * Q1 + m1]));
        W[i] = z;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nf * Q; i += blockDim.x) {
        const int f = i / Q, rem = i - f * Q, n2 = rem / Q1, n1 = rem - n2 * Q1;
        double2 z = t[(f0 + f) * Q + rem];
        for (int m2 = 0; m2 < Q1; ++m2) z = cadd(z, cscale(Tv[n2 * Q1 + m2], W[f * Q + m2 * Q1 + n1]));
        t[(f0 + f) * Q + rem] = z;
    }
    __syncthreads();
}

// the leaf's fields (and its parent's) and the transfer matrices to shared memory
__device__ __forceinline__ void leaf_read(const DevOp &o, bool down, int id, int k1, int k2, int Q, const double2 *loc, double2 *t,
                                          double2 *par, double *T)
{
    const int SL = o.SL, gc = (int)o.lvl_off[o.L] + id;
    for (int i = threadIdx.x; i < 3 * Q; i += blockDim.x) t[i] = loc[(size_t)gc * 3 * Q + i];
    if (!down) return;
    const int Sp = SL / 2, pgc = (int)o.lvl_off[o.L - 1] + (id / (SL * SL) * Sp + k2 / 2) * Sp + k1 / 2;
    for (int i = threadIdx.x; i < 3 * Q; i += blockDim.x) par[i] = loc[(size_t)pgc * 3 * Q + i];
    for (int i = threadIdx.x; i < 2 * Q; i += blockDim.x) T[i] = i < Q ? o.T0[i] : o.T1[i - Q];
}

__global__ __launch_bounds__(512) void k_l2p_leaf(DevOp o, int down, const double2 *loc, double2 *ybuf)
{
    extern __shared__ double2 sm2[];
    const int id = blockIdx.x;
    const int SL = o.SL, s = o.s, p = o.p, Q1 = o.Q1, Q = o.Q, RL = o.rowlen, QR = Q1 * RL;
    const int r = id % (SL * SL), k2 = r / SL, k1 = r % SL;
    double2 *W0 = sm2;                 // [Q1 (m2)][RL (i1)]  component 0 field + divergence
    double2 *W1 = W0 + QR;             // component 1 field
    double2 *W1d = W1 + QR;            // component 1 divergence
    double2 *t = W1d + QR;             // [3][Q] the leaf's fields
    double *M = reinterpret_cast<double *>(t + 3 * Q);   // Mp, Mq, Mdp of k1, then of k2
    double2 *par = reinterpret_cast<double2 *>(M + 6 * QR + (6 * QR & 1)), *W = par + 3 * Q;   // with down only
    double *T = reinterpret_cast<double *>(W + 3 * Q);
    for (int i = threadIdx.x; i < 6 * QR; i += blockDim.x) {
        const int a = i / QR, m = i - a * QR, k = a < 3 ? k1 : k2, b = a % 3;
        M[i] = (b == 0 ? o.Mp : (b == 1 ? o.Mq : o.Mdp))[(size_t)k * QR + m];
    }
    leaf_read(o, down != 0, id, k1, k2, Q, loc, t, par, T);
    __syncthreads();
    if (down) leaf_l2l(o, k1, k2, Q1, Q, t, par, W, T, 0, 3);
    const double *Mpu = M, *Mqu = M + QR, *Mdu = M + 2 * QR, *Mpv = M + 3 * QR, *Mqv = M + 4 * QR, *Mdv = M + 5 * QR;
    const int w1a = s + p, w1b = s + p - 1;
    for (int i = threadIdx.x; i < 3 * QR; i += blockDim.x) {
        const int g = i / QR, e = i - g * QR, m2 = e / RL, i1 = e - m2 * RL;
        double2 a = make_double2(0, 0);
        if (g == 0) {
            if (i1 < w1a)
                for (int m1 = 0; m1 < Q1; ++m1)
                    a = cadd(a, cadd(cscale(Mpu[m1 * RL + i1], t[m2 * Q1 + m1]), cscale(Mdu[m1 * RL + i1], t[2 * Q + m2 * Q1 + m1])));
        } else if (i1 < w1b) {
            const double2 *f = t + g * Q + m2 * Q1;   // field 2, then the divergence
            for (int m1 = 0; m1 < Q1; ++m1) a = cadd(a, cscale(Mqu[m1 * RL + i1], f[m1]));
        }
        W0[i] = a;
    }
    __syncthreads();
    double2 *Y = ybuf + (size_t)id * 2 * RL * RL;
    for (int i = threadIdx.x; i < 2 * RL * RL; i += blockDim.x) {
        const int c = i / (RL * RL), rem = i % (RL * RL), i2 = rem / RL, i1 = rem % RL;
        double2 v = make_double2(0, 0);
        if (c == 0 && i2 < s + p - 1 && i1 < w1a) {
            for (int m2 = 0; m2 < Q1; ++m2) v = cadd(v, cscale(Mqv[m2 * RL + i2], W0[m2 * RL + i1]));
        } else if (c == 1 && i2 < s + p && i1 < w1b) {
            for (int m2 = 0; m2 < Q1; ++m2)
                v = cadd(v, cadd(cscale(Mpv[m2 * RL + i2], W1[m2 * RL + i1]), cscale(Mdv[m2 * RL + i2], W1d[m2 * RL + i1])));
        }
        Y[i] = v;
    }
}

// scalar single layer: Y[i2][i1] = sum (M_p (x) M_p)^T t^d over the leaf's W x W window
// (component 0 of the leaf's result rows)
__global__ __launch_bounds__(512) void k_l2p_leaf_sc(DevOp o, int down, const double2 *loc, double2 *ybuf)
{
    extern __shared__ double2 sm2[];
    const int id = blockIdx.x;
    const int SL = o.SL, s = o.s, p = o.p, Q1 = o.Q1, Q = o.Q, RL = o.rowlen, W = s + p, QR = Q1 * RL;
    const int r = id % (SL * SL), k2 = r / SL, k1 = r % SL;
    double2 *Wm = sm2;       // [Q1 (m2)][W (i1)]
    double2 *t = Wm + QR;    // [3][Q] the leaf's fields (the third one counts)
    double *M = reinterpret_cast<double *>(t + 3 * Q);   // Mp of k1, then of k2
    double2 *par = reinterpret_cast<double2 *>(M + 2 * QR), *Wd = par + 3 * Q;   // with down only
    double *T = reinterpret_cast<double *>(Wd + Q);
    for (int i = threadIdx.x; i < 2 * QR; i += blockDim.x) M[i] = o.Mp[(size_t)(i < QR ? k1 : k2) * QR + i % QR];
    leaf_read(o, down != 0, id, k1, k2, Q, loc, t, par, T);
    __syncthreads();
    if (down) leaf_l2l(o, k1, k2, Q1, Q, t, par, Wd, T, 2, 1);
    const double *Mpu = M, *Mpv = M + QR;
    for (int i = threadIdx.x; i < Q1 * W; i += blockDim.x) {
        const int m2 = i / W, i1 = i % W;
        double2 a = make_double2(0, 0);
        for (int m1 = 0; m1 < Q1; ++m1) a = cadd(a, cscale(Mpu[m1 * RL + i1], t[2 * Q + m2 * Q1 + m1]));
        Wm[i] = a;
    }
    __syncthreads();
    double2 *Y = ybuf + (size_t)id * 2 * RL * RL;
    for (int i = threadIdx.x; i < RL * RL; i += blockDim.x) {
        const int i2 = i / RL, i1 = i % RL;
        double2 v = make_double2(0, 0);
        if (i2 < W && i1 < W)
            for (int m2 = 0; m2 < Q1; ++m2) v = cadd(v, cscale(Mpv[m2 * RL + i2], Wm[m2 * W + i1]));
        Y[i] = v;
    }
}

// contributions of the leaf clusters that the incarnations of unknown i touch
__device__ __forceinline__ double2 l2p_sum(const DevOp &o, int i, const double2 *ybuf)
{
    const int s = o.s, p = o.p, SL = o.SL, n = o.n, RL = o.rowlen;
    double2 acc = make_double2(0, 0);
    for (int c = 0; c < 2; ++c) {
        const int32_t *in = o.inc + ((size_t)i * 2 + c) * 5;
        const int j = in[0];
        if (j < 0) continue;
        const int a = in[1], i1 = in[2], i2 = in[3];
        const double sg = (double)in[4];
        const int du = (a == 0) ? p : p - 1, dv = (a == 0 && !o.scalar) ? p - 1 : p;
        const int k1b = max(0, i1 - du) / s, k1e = min(n - 1, i1) / s;
        const int k2b = max(0, i2 - dv) / s, k2e = min(n - 1, i2) / s;
        for (int k2 = k2b; k2 <= k2e; ++k2)
            for (int k1 = k1b; k1 <= k1e; ++k1) {
                const int leaf = (j * SL + k2) * SL + k1;
                const double2 v = ybuf[(((size_t)leaf * 2 + a) * RL + (i2 - k2 * s)) * RL + (i1 - k1 * s)];
                acc = cadd(acc, cscale(sg, v));
            }
    }
    return acc;
}

__global__ void k_l2p_gather(DevOp o, const double2 *ybuf, double2 *y)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= o.N) return;
    y[i] = cadd(y[i], l2p_sum(o, i, ybuf));
}

// k_near_gather and k_l2p_gather in one launch, the same sums in the same order
__global__ __launch_bounds__(256) void k_gather(DevOp o, const int64_t *ptr, const int32_t *idx, const double2 *part,
                                                const double2 *ybuf, double2 *y)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int i = (int)(t >> 4), sub = (int)(t & 15);
    double re = 0.0, im = 0.0;
    double2 far = make_double2(0.0, 0.0);
    if (i < o.N) {
        for (int64_t k = ptr[i] + sub; k < ptr[i + 1]; k += 16) {
            const double2 v = part[idx[k]];
            re += v.x;
            im += v.y;
        }
        if (sub == 0) far = l2p_sum(o, i, ybuf);
    }
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) {
        re += __shfl_xor(re, off, 16);
        im += __shfl_xor(im, off, 16);
    }
    if (i < o.N && sub == 0) y[i] = cadd(make_double2(re, im), far);
}

__global__ void k_helmholtz_eval(int64_t n, double kappa, const double *r2, double2 *out, int prec,
                                 const double2 *sctab)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (prec == IGE_F32) out[i] = dm::to_d(dm::helmholtz_r2((float)kappa, (float)r2[i]));
    else out[i] = dm::helmholtz_r2_tab(kappa, r2[i], sctab);
}

}  // namespace

void launch_helmholtz_eval(hipStream_t s, int64_t n, double kappa, const double *r2, double2 *out, int prec,
                           const double2 *sctab)
{
    hipLaunchKernelGGL(k_helmholtz_eval, dim3((n + 255) / 256), dim3(256), 0, s, n, kappa, r2, out, prec, sctab);
    IGE_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
#define IGE_LAUNCH_CHECK() IGE_HIP(hipGetLastError())

void launch_element_data(ige_op op)
{
    const DevOp &o = op->view;
    const int64_t E = (int64_t)o.P * o.n * o.n;
    const int threads = 64;
    hipStream_t s = lstream(op);
#define IGE_ED(NLV) hipLaunchKernelGGL(k_element_data<NLV>, dim3(E), dim3(threads), 0, s, o, op->d_eX.p, op->d_ePsi.p, op->d_ePsiF.p, op->d_eC.p)
    switch (o.nl) {
        case 4: IGE_ED(4); break;
        case 9: IGE_ED(9); break;
        case 12: IGE_ED(12); break;
        case 16: IGE_ED(16); break;
        case 24: IGE_ED(24); break;
        case 25: IGE_ED(25); break;
        default: IGE_ED(40); break;
    }
#undef IGE_ED
    IGE_LAUNCH_CHECK();
}

void launch_node_geometry(ige_op op)
{
    const DevOp &o = op->view;
    const int64_t tot = (int64_t)op->NC * o.Q;
    hipLaunchKernelGGL(k_node_geometry, dim3((tot + 255) / 256), dim3(256), 0, lstream(op), o, op->NC,
                       op->d_nodeX.p, op->d_nodeT.p);
    IGE_LAUNCH_CHECK();
}

size_t psi_fragment_doubles(int nl, int G2)
{
    const int LT = (nl + 15) / 16, QT = (G2 + 15) / 16;
    return (size_t)4 * LT * 4 * QT * 64;
}

void launch_p2m(ige_op op, const double2 *x)
{
    const DevOp &o = op->view;
    const int nleaf = o.P * o.SL * o.SL;
    if (o.scalar) {
        const size_t W = o.s + o.p;
        const size_t shm = sizeof(double2) * (W * W + W * o.Q1);
        hipLaunchKernelGGL(k_p2m_sc, dim3(nleaf), dim3(256), shm, lstream(op), o, x, op->d_mom.p, op->d_src.p);
        IGE_LAUNCH_CHECK();
        return;
    }
    const int w1a = o.s + o.p, w2a = o.s + o.p - 1;
    const size_t shm = sizeof(double2) * (2 * w1a * w2a + 3 * (size_t)(w1a) * o.Q1) + sizeof(double) * 6 * o.Q1 * o.rowlen;
    lds_attr_once(reinterpret_cast<const void *>(&k_p2m), shm);
    hipLaunchKernelGGL(k_p2m, dim3(nleaf), dim3(256), shm, lstream(op), o, x, op->d_mom.p, op->d_src.p);
    IGE_LAUNCH_CHECK();
}

void launch_m2m(ige_op op)
{
    const DevOp &o = op->view;
    const size_t shm = sizeof(double2) * 25 * o.Q;
    const int nth = std::min(1024, std::max((o.Q + 63) / 64 * 64, (12 * o.Q / 2 + 63) / 64 * 64));   // two values a thread
    lds_attr_once(reinterpret_cast<const void *>(&k_m2m), shm);
    // parents down to the coarsest level with far pairs (coarser moments are unused)
    for (int lvl = o.L - 1; lvl >= std::max(0, op->lfar); --lvl) {
        const int ncl = o.P << (2 * lvl);
        hipLaunchKernelGGL(k_m2m, dim3(ncl), dim3(nth), shm, lstream(op), o, lvl, op->d_mom.p, op->d_src.p);
        IGE_LAUNCH_CHECK();
    }
    if (!o.varq) return;
    // levels of a smaller degree: source fields from the restricted moments
    for (int lvl = std::max(0, op->lfar); lvl <= o.L; ++lvl) {
        const int Q1l = o.ql[lvl] + 1;
        if (Q1l == o.Q1) continue;
        const size_t sh = sizeof(double2) * (3 * (size_t)o.Q + 3 * (size_t)o.Q1 * Q1l);
        hipLaunchKernelGGL(k_restrict, dim3(o.P << (2 * lvl)), dim3(256), sh, lstream(op), o, lvl, op->d_mom.p,
                           op->d_src.p);
        IGE_LAUNCH_CHECK();
    }
}

// dynamic shared memory above the 64 KB granted without asking (degrees 12..15 of the
// transfer kernels): the kernel's limit is raised once, before any graph capture
void lds_attr_once(const void *kern, size_t shm)
{
    if (shm <= (size_t)64 * 1024) return;
    static std::mutex mu;
    static std::map<const void *, size_t> done;
    std::lock_guard<std::mutex> lk(mu);
    size_t &have = done[kern];
    if (have >= shm) return;
    IGE_HIP(hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm));
    have = shm;
}

size_t m2l_shared_bytes(int Q)
{
    const int TPG = (Q + kM2LNT - 1) / kM2LNT;
    const int S = std::min(kM2LThreads / TPG, Q);
    // [Q][4] positions + [Q][4] complex, or the reduction of two fields
    return std::max(sizeof(double) * 4 * Q + sizeof(double2) * 4 * Q, sizeof(double2) * 2 * (size_t)Q * S);
}

void launch_m2l(ige_op op, int prec)
{
    const DevOp &o = op->view;
    if (op->work.empty()) return;
    if (op->stored && !op->m2l_generate_one) {
        m2l_stored_one(op, prec);
        return;
    }
    if (prec == IGE_F64) {
        launch_m2l_sym(op);
        return;
    }
    size_t shm = m2l_shared_bytes(o.Q);   // the largest over the levels' node counts
    for (int lvl = 0; lvl <= o.L; ++lvl) shm = std::max(shm, m2l_shared_bytes((o.ql[lvl] + 1) * (o.ql[lvl] + 1)));
    shm = std::max(shm, op->m2l_lds);
    // k = IGE_M2L_PERSIST workgroups per CU loop over the work items (room for the near
    // field's workgroups beside them); 0 (default): one workgroup per item
    const int nwork = (int)op->work1.size();
    int grid = nwork;
    if (op->m2l_persist > 0) {
        int ncu = 0;
        IGE_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, op->ctx->device));
        grid = std::max(1, std::min(nwork, ncu * op->m2l_persist));
    }
    lds_attr_once(reinterpret_cast<const void *>(&k_m2l), shm);
    hipLaunchKernelGGL(k_m2l, dim3(grid), dim3(kM2LThreads), shm, lstream(op), o, nwork, op->d_work1.p, op->d_partner.p,
                       op->d_src.p, op->d_spart.p);
    IGE_LAUNCH_CHECK();
}

void launch_m2l_reduce(ige_op op, int prec)
{
    const DevOp &o = op->view;
    if (op->stored && !op->m2l_generate_one) {
        m2l_stored_reduce_one(op);
        return;
    }
    if (prec == IGE_F64)
        launch_m2l_reduce_sym(op);
    else
        hipLaunchKernelGGL(k_m2l_reduce, dim3(op->NC), dim3(128), 0, lstream(op), o, op->d_wrk_of_tgt1.p, op->d_spart.p,
                           op->d_loc.p);
    IGE_LAUNCH_CHECK();
    if (!o.varq) return;
    // levels of a smaller degree: local expansions back to the degree-q nodes
    for (int lvl = std::max(0, op->lfar); lvl <= o.L; ++lvl) {
        const int Q1l = o.ql[lvl] + 1;
        if (Q1l == o.Q1) continue;
        const size_t sh = sizeof(double2) * (3 * (size_t)Q1l * Q1l + 3 * (size_t)Q1l * o.Q1);
        hipLaunchKernelGGL(k_lift, dim3(o.P << (2 * lvl)), dim3(256), sh, lstream(op), o, lvl, op->d_loc.p);
        IGE_LAUNCH_CHECK();
    }
}

// children from level first to level last
static void l2l_levels(ige_op op, int last)
{
    const DevOp &o = op->view;
    const size_t shm = sizeof(double2) * 3 * o.Q;
    // children below the coarsest level with far pairs (the expansions above it are zero)
    for (int lvl = std::max(1, op->lfar + 1); lvl <= last; ++lvl) {
        const int ncl = o.P << (2 * lvl);
        hipLaunchKernelGGL(k_l2l, dim3(ncl), dim3(256), shm, lstream(op), o, lvl, op->d_loc.p);
        IGE_LAUNCH_CHECK();
    }
}

// the leaves' own level is left to launch_l2p_leaf
void launch_l2l(ige_op op) { l2l_levels(op, op->view.L - 1); }

int near_blk_u(int nF)
{
    const int u = (nF + 63) / 64;
    for (int c : {1, 2, 3, 4, 6, 8, 12, 16})
        if (u <= c) return c;
    return 16;
}

void launch_spmv(ige_op op, const double2 *x, double2 *y, hipStream_t st, hipEvent_t mid)
{
    const DevOp &o = op->view;
    if (o.nblk == 0) {
        IGE_HIP(hipMemsetAsync(y, 0, sizeof(double2) * o.N, st));
        if (mid) IGE_HIP(hipEventRecord(mid, st));
        return;
    }
    if (op->cmp_on) {
        double2 *part = op->d_cpart.p;
        launch_near_once(op, x, part, st);
        if (mid) IGE_HIP(hipEventRecord(mid, st));
        hipLaunchKernelGGL(k_near_gather, dim3((unsigned)(((int64_t)o.N * 16 + 255) / 256)), dim3(256), 0, st, o.N,
                           op->d_cred_ptr.p, op->d_cred_idx.p, part, y);
        IGE_LAUNCH_CHECK();
        return;
    }
    const dim3 grid((unsigned)(o.nblk * o.nch)), blk(256);
    double2 *part = op->d_npart.p;
    switch (near_blk_u(o.nF)) {
        case 1: hipLaunchKernelGGL(k_near_blk<1>, grid, blk, 0, st, o, x, part); break;
        case 2: hipLaunchKernelGGL(k_near_blk<2>, grid, blk, 0, st, o, x, part); break;
        case 3: hipLaunchKernelGGL(k_near_blk<3>, grid, blk, 0, st, o, x, part); break;
        case 4: hipLaunchKernelGGL(k_near_blk<4>, grid, blk, 0, st, o, x, part); break;
        case 6: hipLaunchKernelGGL(k_near_blk<6>, grid, blk, 0, st, o, x, part); break;
        case 8: hipLaunchKernelGGL(k_near_blk<8>, grid, blk, 0, st, o, x, part); break;
        case 12: hipLaunchKernelGGL(k_near_blk<12>, grid, blk, 0, st, o, x, part); break;
        default: hipLaunchKernelGGL(k_near_blk<16>, grid, blk, 0, st, o, x, part); break;
    }
    IGE_LAUNCH_CHECK();
    if (mid) IGE_HIP(hipEventRecord(mid, st));
    hipLaunchKernelGGL(k_near_gather, dim3((unsigned)(((int64_t)o.N * 16 + 255) / 256)), dim3(256), 0, st, o.N, o.red_ptr, o.red_idx, part, y);
    IGE_LAUNCH_CHECK();
}

void launch_l2p_leaf(ige_op op)
{
    const DevOp &o = op->view;
    const int nleaf = o.P * o.SL * o.SL, down = o.L >= std::max(1, op->lfar + 1) ? 1 : 0;
    const size_t Q = o.Q, QR = (size_t)o.Q1 * o.rowlen;
    if (o.scalar) {
        const size_t shm = sizeof(double2) * (QR + 3 * Q + (down ? 4 * Q : 0)) + sizeof(double) * (2 * QR + (down ? 2 * Q : 0));
        lds_attr_once(reinterpret_cast<const void *>(&k_l2p_leaf_sc), shm);
        hipLaunchKernelGGL(k_l2p_leaf_sc, dim3(nleaf), dim3(256), shm, lstream(op), o, down, op->d_loc.p, op->d_ybuf.p);
        IGE_LAUNCH_CHECK();
        return;
    }
    const size_t shm = sizeof(double2) * (3 * QR + 3 * Q + (down ? 6 * Q : 0)) + sizeof(double) * (6 * QR + 1 + (down ? 2 * Q : 0));
    lds_attr_once(reinterpret_cast<const void *>(&k_l2p_leaf), shm);
    const int nth = std::min<int>(512, (int)(3 * std::max(Q, QR) + 63) / 64 * 64);
    hipLaunchKernelGGL(k_l2p_leaf, dim3(nleaf), dim3(nth), shm, lstream(op), o, down, op->d_loc.p, op->d_ybuf.p);
    IGE_LAUNCH_CHECK();
}

// sums of a fused one-column apply: near-field partial results and leaf rows
void launch_gather(ige_op op, double2 *y)
{
    const DevOp &o = op->view;
    hipLaunchKernelGGL(k_gather, dim3((unsigned)(((int64_t)o.N * 16 + 255) / 256)), dim3(256), 0, lstream(op), o,
                       op->d_cred_ptr.p, op->d_cred_idx.p, op->d_cpart.p, op->d_ybuf.p, y);
    IGE_LAUNCH_CHECK();
}

void launch_l2p_gather(ige_op op, double2 *y)
{
    const DevOp &o = op->view;
    hipLaunchKernelGGL(k_l2p_gather, dim3((o.N + 255) / 256), dim3(256), 0, lstream(op), o, op->d_ybuf.p, y);
    IGE_LAUNCH_CHECK();
}

}  // namespace ige
