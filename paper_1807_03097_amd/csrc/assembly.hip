// a1: element-pair Galerkin quadrature of the near field, accumulated into dense blocks over
// leaf function slots (Sec. 4.1).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_math.hpp"
#include "element.hpp"
#include "op.hpp"

namespace ige {

namespace {

__device__ inline double2 cscale(double s, double2 a) { return make_double2(s * a.x, s * a.y); }

// row tiles of test functions per workgroup of k_near_regular: all up to 24 local
// functions, one 16-row tile for more (p = 4: 40 functions, three workgroups)
constexpr int near_regular_lr(int nl) { return nl <= 24 ? (nl + 15) / 16 : 1; }

// ---------------------------------------------------------------------------
// a1: regular element pairs (no shared corner).  With S = (1, 1, 1, -kappa^-2) and
// the weights folded into Psi,
//   B[l][l'] = sum_c S_c sum_q Psi_e^c[l][q] sum_q' K(q, q') Psi_f^c[l'][q'],
// computed as two products on the FP64 matrix cores per trial element f:
//   Y_c(q', l) = sum_q K(q, q') Psi_e^c[l][q]      (K as operand A, Psi_e as B)
//   B(l, l') += sum_q' Y_c(q', l) Psi_f^c[l'][q']  (Y from the accumulators as A)
// The accumulator layout of the first product (row lane/16 + 4 j) is the operand
// layout of the second when its reduction slots are ordered by frag_q.
// A workgroup takes one block, one test element e of the target leaf and a square
// of sb x sb trial elements of the source leaf; wave w takes the trial elements of the
// quadrant (w mod 2, w / 2) of the square, row by row, and adds their element-pair blocks
// to its own copy of the block rows of e over that quadrant in shared memory, so the
// waves share nothing and never wait for one another.  Then the element pairs of e that
// share a corner with a trial element of the square (computed before by k_near_singular)
// are added to the quadrant that holds the trial element, in list order, and the
// quadrants are summed in order where they overlap.  Every sum therefore has a fixed order.
// Launched once per colour: the test elements of a launch are p + 1 apart in both
// directions (no glued function in common, so no block row in common), and with
// several trial squares per leaf the squares of a launch are two apart (sb >= p: no
// column in common).  Each block entry thus has at most one writer per launch, and
// the launches run in a fixed order on one stream: the assembled blocks are the same
// bits on every run.
// Bound by FP64 issue: for p = 2 and 25 points 168 instructions of 64 cycles and some 450
// vector FP64 operations (14 kernel values per lane) per element pair.  The waves once staged
// their blocks and added them in turn (five barriers per four pairs), compared the corners one
// pair after the other, and rounded the points up to 32 in both products.  Sphere level 5, p = 2,
// 996 blocks of 64 x 64 element pairs: 61.0 ms then, 31.9 now (51 TFLOP/s of matrix instructions).
// ---------------------------------------------------------------------------
// NL local functions, TS = ceil(G2 / 4) steps of four quadrature points, LR row tiles
template <int NL, int TS, int LR>
__device__ __forceinline__ void near_regular_body(const DevOp &o, int sb, int ce1, int ce2, int cs1, int cs2, int sstep)
{
    // LR of the LT 16-row tiles of test functions per workgroup (LR = LT: all rows;
    // otherwise the rows are split over LT / LR workgroups, for the larger degrees)
    constexpr int LT = (NL + 15) / 16, QT = (TS + 3) / 4, T = 4 * QT, NRT = LT / LR;
    constexpr int NR = LR == LT ? NL : 16 * LR;       // test-function rows of this workgroup
    extern __shared__ double2 sacc[];                 // [4 quadrants][NR][components][Wq^2]
    __shared__ double sXe[3][4 * TS];                 // test element points (the last one repeated)
    __shared__ double2 sTab[256];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int s = o.s, nsb = s / sb, Wsb = sb + o.p, P1 = o.p + 1, ncomp = o.scalar ? 1 : 2;
    const int hs = (sb + 1) / 2, Wq = hs + o.p, nq = ncomp * Wq * Wq;
    // test elements and trial squares of this colour
    const int n1 = (s - ce1 + P1 - 1) / P1, n2 = (s - ce2 + P1 - 1) / P1;
    const int m1 = (nsb - cs1 + sstep - 1) / sstep, m2 = (nsb - cs2 + sstep - 1) / sstep;
    int64_t blk = blockIdx.x;
    const int u0 = LR * (int)(blk % NRT);             // first row tile
    blk /= NRT;
    const int l0 = 16 * u0;                           // first test function
    const int sub = (int)(blk % (m1 * m2));
    blk /= m1 * m2;
    const int tc = (int)(blk % (n1 * n2));
    const int64_t b = blk / (n1 * n2);
    const int lt = o.bpair[2 * b], ls = o.bpair[2 * b + 1];
    const int SL = o.SL;
    const int jt = lt / (SL * SL), jr = lt % (SL * SL), js = ls / (SL * SL), jsr = ls % (SL * SL);
    const int tl1 = ce1 + P1 * (tc % n1), tl2 = ce2 + P1 * (tc / n1);   // e inside its leaf
    const int ti = tl2 * s + tl1;
    const int te1 = (jr % SL) * s + tl1, te2 = (jr / SL) * s + tl2;
    const int sl1 = (cs1 + sstep * (sub % m1)) * sb, sl2 = (cs2 + sstep * (sub / m1)) * sb;   // trial square
    const int fx0 = (jsr % SL) * s + sl1, fy0 = (jsr / SL) * s + sl2;
    const int64_t e = ((int64_t)jt * o.n + te2) * o.n + te1;
    const int G2 = o.G2;
    for (int i = threadIdx.x; i < 4 * NR * nq; i += blockDim.x) sacc[i] = make_double2(0.0, 0.0);
    for (int i = threadIdx.x; i < 256; i += blockDim.x) sTab[i] = o.sctab[i];
    for (int i = threadIdx.x; i < 3 * 4 * TS; i += blockDim.x) {
        const int d = i / (4 * TS), q = i % (4 * TS);
        sXe[d][q] = o.eX[(e * 3 + d) * G2 + min(q, G2 - 1)];
    }
    constexpr size_t FE = (size_t)4 * LT * T * 64;
    double pa[4][LR][TS];
    {
        const double *Fe = o.ePsiF + (size_t)e * FE;
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int u = 0; u < LR; ++u)
#pragma unroll
                for (int t = 0; t < TS; ++t)
                    pa[c][u][t] = Fe[((c * LT + u0 + u) * T + t) * 64 + lane] * (c == 3 ? o.cdiv : 1.0);
    }
    // corner lane / 4 mod 4 of e, for the comparison with corner lane mod 4 of a trial element
    const double *ec = o.eC + e * 12 + 3 * ((lane >> 2) & 3);
    const double c0 = ec[0], c1 = ec[1], c2 = ec[2];
    // this lane's columns in the copy (component and offsets of local function 16 v + lane % 16)
    int col[LT];
#pragma unroll
    for (int v = 0; v < LT; ++v) {
        int a, t1, t2;
        local_index(o, min(16 * v + (lane & 15), NL - 1), a, t1, t2);
        col[v] = (a * Wq + t2) * Wq + t1;
    }
    __syncthreads();
    const int qx = (wv & 1) * hs, qy = (wv >> 1) * hs;   // the wave's quadrant
    const int nx = max(0, min(hs, sb - qx)), ny = max(0, min(hs, sb - qy)), nf = nx * ny;
    double2 *acc = sacc + (size_t)wv * NR * nq;
    unsigned long long near = 0;   // of the next four trial elements: pairs of equal corners
    for (int k = 0; k < nf; ++k) {
        if ((k & 3) == 0) {
            const int kk = min(k + (lane >> 4), nf - 1);
            const int64_t fk = ((int64_t)js * o.n + fy0 + qy + kk / nx) * o.n + fx0 + qx + kk % nx;
            const double *fc = o.eC + fk * 12 + 3 * (lane & 3);
            const double d0 = c0 - fc[0], d1 = c1 - fc[1], d2 = c2 - fc[2];
            near = __ballot(sqrt(d0 * d0 + d1 * d1 + d2 * d2) <= o.scale_tol);
        }
        // pairs with a shared corner come from the singular kernel (uniform over the wave)
        if ((near >> (16 * (k & 3)) & 0xffffull) != 0) continue;
        const int r1 = k % nx, r2 = k / nx;
        const int64_t f = ((int64_t)js * o.n + fy0 + qy + r2) * o.n + fx0 + qx + r1;
        dx4 br[LR][LT], bi[LR][LT];
#pragma unroll
        for (int u = 0; u < LR; ++u)
#pragma unroll
            for (int v = 0; v < LT; ++v) {
                br[u][v] = dx4{0.0, 0.0, 0.0, 0.0};
                bi[u][v] = dx4{0.0, 0.0, 0.0, 0.0};
            }
        // kernel values as operand A: row q' = 16 qt + lane % 16, slot q = frag_q(t, lane)
        // (points beyond G2 repeat the last one; Psi is zero there)
        double kre[QT][TS], kim[QT][TS];
#pragma unroll
        for (int qt = 0; qt < QT; ++qt) {
            const int qb = min(16 * qt + (lane & 15), G2 - 1);
            const double xb0 = o.eX[(f * 3 + 0) * G2 + qb], xb1 = o.eX[(f * 3 + 1) * G2 + qb], xb2 = o.eX[(f * 3 + 2) * G2 + qb];
#pragma unroll
            for (int t = 0; t < TS; ++t) {
                const int qa = frag_q(t, lane);
                const double d0 = sXe[0][qa] - xb0, d1 = sXe[1][qa] - xb1, d2 = sXe[2][qa] - xb2;
                const double2 K = dm::helmholtz_r2_tab(o.kappa, fma(d0, d0, fma(d1, d1, d2 * d2)), sTab);
                kre[qt][t] = K.x;
                kim[qt][t] = K.y;
            }
        }
        const double *Ff = o.ePsiF + (size_t)f * FE;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            dx4 yr[QT][LR], yi[QT][LR];
#pragma unroll
            for (int qt = 0; qt < QT; ++qt)
#pragma unroll
                for (int u = 0; u < LR; ++u) {
                    yr[qt][u] = dx4{0.0, 0.0, 0.0, 0.0};
                    yi[qt][u] = dx4{0.0, 0.0, 0.0, 0.0};
                }
#pragma unroll
            for (int t = 0; t < TS; ++t)
#pragma unroll
                for (int qt = 0; qt < QT; ++qt)
#pragma unroll
                    for (int u = 0; u < LR; ++u) {
                        yr[qt][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(kre[qt][t], pa[c][u][t], yr[qt][u], 0, 0, 0);
                        yi[qt][u] = __builtin_amdgcn_mfma_f64_16x16x4f64(kim[qt][t], pa[c][u][t], yi[qt][u], 0, 0, 0);
                    }
#pragma unroll
            for (int v = 0; v < LT; ++v)
#pragma unroll
                for (int t = 0; t < TS; ++t) {
                    const double pb = Ff[((c * LT + v) * T + t) * 64 + lane];
#pragma unroll
                    for (int u = 0; u < LR; ++u) {
                        br[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(yr[t / 4][u][t % 4], pb, br[u][v], 0, 0, 0);
                        bi[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(yi[t / 4][u][t % 4], pb, bi[u][v], 0, 0, 0);
                    }
                }
        }
        // rows l = 16 u + lane / 16 + 4 j, columns l' = 16 v + lane % 16 of the pair's block
#pragma unroll
        for (int v = 0; v < LT; ++v)
#pragma unroll
            for (int u = 0; u < LR; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int lr = 16 * u + (lane >> 4) + 4 * j;   // row of this workgroup
                    if (l0 + lr < NL && 16 * v + (lane & 15) < NL) {
                        double2 &d = acc[lr * nq + col[v] + r2 * Wq + r1];
                        d = make_double2(d.x + br[u][v][j], d.y + bi[u][v][j]);
                    }
                }
        // the next element's lanes read entries that other lanes of this wave wrote
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    // element pairs of e with a shared corner whose trial element lies in the square
    const int kb = o.sing_ptr[b * (int64_t)(s * s) + ti], ke = o.sing_ptr[b * (int64_t)(s * s) + ti + 1];
    for (int k = kb; k < ke; ++k) {
        const int64_t f = o.sing[k].f;
        int jf, f1, f2;
        elem_of(o, f, jf, f1, f2);
        const int q1 = f1 - fx0, q2 = f2 - fy0;
        if (q1 < 0 || q1 >= sb || q2 < 0 || q2 >= sb) continue;   // uniform over the workgroup
        const int x = q1 / hs, y = q2 / hs;
        double2 *aq = sacc + (size_t)(x + 2 * y) * NR * nq + (q2 - y * hs) * Wq + q1 - x * hs;
        const double2 *P = o.sblk + (size_t)k * NL * NL + (size_t)l0 * NL;
        for (int i = threadIdx.x; i < NR * NL; i += blockDim.x) {
            const int l = i / NL, lb = i % NL;
            if (l0 + l >= NL) continue;
            int a, t1, t2;
            local_index(o, lb, a, t1, t2);
            const double2 v = P[i];
            double2 &d = aq[l * nq + (a * Wq + t2) * Wq + t1];
            d = make_double2(d.x + v.x, d.y + v.y);
        }
        __syncthreads();
    }
    const int W = o.W, nF = o.nF, nslot = ncomp * Wsb * Wsb;
    for (int i = threadIdx.x; i < NR * nslot; i += blockDim.x) {
        const int lr = i / nslot, l = l0 + lr, sl = i % nslot;
        if (l >= NL) continue;
        const int a = sl / (Wsb * Wsb), r = sl % (Wsb * Wsb), r1 = r % Wsb, r2 = r / Wsb;
        double2 v = make_double2(0.0, 0.0);
        for (int w = 0; w < 4; ++w) {
            const int x = r1 - (w & 1) * hs, y = r2 - (w >> 1) * hs;
            if (x < 0 || x >= Wq || y < 0 || y >= Wq) continue;
            const double2 d = sacc[(w * NR + lr) * nq + (a * Wq + y) * Wq + x];
            v = make_double2(v.x + d.x, v.y + d.y);
        }
        if (v.x == 0.0 && v.y == 0.0) continue;
        const int i1 = sl1 + r1, i2 = sl2 + r2;
        if (i1 >= (a == 0 ? W : W - 1) || i2 >= ((a == 0 && !o.scalar) ? W - 1 : W)) {
            atomicAdd(o.err, 1);
            continue;
        }
        const int kc = leaf_slot(W, a, i1, i2);
        int ar, t1, t2;
        local_index(o, l, ar, t1, t2);
        const int kr = leaf_slot(W, ar, tl1 + t1, tl2 + t2);
        // signs of the glued unknowns folded in; slots without an unknown are skipped
        const double sg = (double)o.leafsgn[(size_t)lt * nF + kr] * (double)o.leafsgn[(size_t)ls * nF + kc];
        if (sg == 0.0) continue;
        double2 *dst = o.bval + ((size_t)b * nF + kr) * nF + kc;   // the only writer in this launch
        double2 cur = *dst;
        cur.x += sg * v.x;
        cur.y += sg * v.y;
        *dst = cur;
    }
}

// the small rules (up to 28 points, up to 12 local functions) fit two
// workgroups per CU without spilling; the others take all registers of one
template <int NL, int TS>
__global__ __launch_bounds__(256) void k_near_regular(DevOp o, int sb, int ce1, int ce2, int cs1, int cs2, int sstep)
{
    near_regular_body<NL, TS, near_regular_lr(NL)>(o, sb, ce1, ce2, cs1, cs2, sstep);
}
template <int NL, int TS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_near_regular_o2(DevOp o, int sb, int ce1,
                                                                                                   int ce2, int cs1, int cs2,
                                                                                                   int sstep)
{
    near_regular_body<NL, TS, near_regular_lr(NL)>(o, sb, ce1, ce2, cs1, cs2, sstep);
}

// ---------------------------------------------------------------------------
// a1: element pairs sharing a corner (relative-coordinate / Duffy sub-rules),
// one wavefront per pair; each pair's NL x NL block is written to its own slot of a
// scratch array (no accumulation here).
// ---------------------------------------------------------------------------
// canonical point (s1, s2) on the test element, (t1, t2) on the trial element and
// weight of sub-rule point idx
__device__ inline void singular_point(const DevOp &o, int kind, int idx, double &s1, double &s2, double &t1,
                                      double &t2, double &wt)
{
    const int gs = o.gs, g4 = gs * gs * gs * gs;
    const int sub = idx / g4;
    int r = idx % g4;
    const int id = r % gs; r /= gs;
    const int ic = r % gs; r /= gs;
    const int ib = r % gs; r /= gs;
    const int ia = r;
    const double xi = o.sx[ia], y1 = o.sx[ib], y2 = o.sx[ic], y3 = o.sx[id];
    const double w4 = o.sw[ia] * o.sw[ib] * o.sw[ic] * o.sw[id];
    if (kind == 1) {
        // identical: per direction |x_k - y_k| = w_k with both orders; (w1, w2) triangle split
        const int tri = sub >> 2, sg1 = (sub >> 1) & 1, sg2 = sub & 1;
        const double w1 = tri == 0 ? xi : xi * y1;
        const double w2 = tri == 0 ? xi * y1 : xi;
        if (!sg1) { s1 = (1.0 - w1) * y2; t1 = s1 + w1; } else { t1 = (1.0 - w1) * y2; s1 = t1 + w1; }
        if (!sg2) { s2 = (1.0 - w2) * y3; t2 = s2 + w2; } else { t2 = (1.0 - w2) * y3; s2 = t2 + w2; }
        wt = w4 * xi * (1.0 - w1) * (1.0 - w2);
    } else if (kind == 2) {
        // common edge at s1 = t1 = 0: distances A, B to the edge and W = |s2 - t2|
        const int pyr = sub >> 1, sg = sub & 1;
        double A, B, W;
        if (pyr == 0) { A = xi; B = xi * y1; W = xi * y2; }
        else if (pyr == 1) { B = xi; A = xi * y1; W = xi * y2; }
        else { W = xi; A = xi * y1; B = xi * y2; }
        double a2, b2;
        if (!sg) { a2 = (1.0 - W) * y3; b2 = a2 + W; } else { b2 = (1.0 - W) * y3; a2 = b2 + W; }
        s1 = A; s2 = a2; t1 = B; t2 = b2;
        wt = w4 * xi * xi * (1.0 - W);
    } else {
        // common vertex at the origin of both: the largest of the four coordinates is xi
        double z[4];
        const double rest[3] = {xi * y1, xi * y2, xi * y3};
        int k = 0;
        for (int i = 0; i < 4; ++i) z[i] = (i == sub) ? xi : rest[k++];
        s1 = z[0]; s2 = z[1]; t1 = z[2]; t2 = z[3];
        wt = w4 * xi * xi * xi;
    }
}

// The rule of each kind as a table: rule[kind - 1] holds s1, s2, t1, t2 and the weight of its
// points, one array after the other (kinds of 8, 6 and 4 sub-rules of gs^4 points).
__host__ __device__ inline int singular_subrules(int kind) { return kind == 1 ? 8 : (kind == 2 ? 6 : 4); }
__host__ __device__ inline int singular_rule_offset(int kind, int g4) { return 5 * g4 * (kind == 1 ? 0 : (kind == 2 ? 8 : 14)); }
size_t singular_rule_doubles(int gs) { return (size_t)5 * 18 * gs * gs * gs * gs; }

__global__ __launch_bounds__(256) void k_singular_rule(DevOp o, double *rule)
{
    const int g4 = o.gs * o.gs * o.gs * o.gs;
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 18 * g4) return;
    const int kind = i < 8 * g4 ? 1 : (i < 14 * g4 ? 2 : 3);
    i -= kind == 1 ? 0 : (kind == 2 ? 8 * g4 : 14 * g4);
    const int n = singular_subrules(kind) * g4;
    double *r = rule + singular_rule_offset(kind, g4), v[5];
    singular_point(o, kind, i, v[0], v[1], v[2], v[3], v[4]);
    for (int k = 0; k < 5; ++k) r[(size_t)k * n + i] = v[k];
}

// Singular pairs: one wave per pair.  The points of the sub-rules are processed in
// batches of 32: the lower half-wave evaluates geometry and local values on the
// test element, the upper half on the trial element, into shared memory; then
//   B[l][l'] += sum_q K_q sum_c Psi_a[q][l][c] Psi_b[q][l'][c]
// runs on the FP64 matrix cores (K_q = weight * kernel folded into the test side) with
// the four components c as the reduction slots of one instruction per point, or four
// points as its slots where only one component is not zero (the scalar operator).  A
// point's row of shared memory holds the scalar values and divergences of the local functions
// and the two tangents; the products Psi_l^c are formed as they are read, so a row is half
// as long and twice the waves fit.  Control points and spline coefficients of the two elements
// are kept in shared memory, the points come from the rule's table.
// The form and the rules are symmetric: of two pairs that differ in the order of their elements
// (both are listed where they lie in one leaf) one is computed, the other its transpose.
// GD: degree in both directions of all patches of the surface (1 or 2; 0: any, out of line)
// Bound by FP64 issue: two instructions of 64 cycles per point and 400 vector FP64 operations
// per batch (two of the longest at a time on a SIMD).  Before, a point's rule came from five
// integer divisions, every coefficient and control point from global memory, eleven FP64
// divisions, and its rows (48 values per side) left room for six waves per CU: sphere level 5,
// p = 2, 5 Gauss points (160 million points): 45.5 ms, 19.2 then, 13.1 with one of each two pairs.
template <int P, bool SC, int GD>
__global__ __launch_bounds__(64) void k_near_singular(DevOp o, const SingularPair *list, const int2 *work, const double *rule)
{
    // points per batch: 32 (16 for p = 4, whose 40 local functions would not fit);
    // SC: the scalar operator's (p+1)^2 local functions
    constexpr int NL = SC ? (P + 1) * (P + 1) : 2 * P * (P + 1), LT = (NL + 15) / 16;
    constexpr int NB = 2 * P * (P + 1) > 24 ? 16 : 32;
    // a point's row: values, divergences, (Fu, 1), (Fv, 1), 0; scalar: values, 0 (odd lengths)
    constexpr int ROW = SC ? (NL + 1) | 1 : 2 * NL + 9, ZERO = ROW - 1, FU = 2 * NL;
    constexpr int NP = (P + 1) * (P + 1), NQ = P * P, NE = NP + NQ, NC = GD > 0 ? 4 * (GD + 1) * (GD + 1) : 1;
    __shared__ double sV[2][NB][ROW];
    __shared__ double2 sK[NB];
    __shared__ double sX[NB][3];
    __shared__ double sExt[2][2][NE];   // spline coefficients by side and direction: degree p, degree p - 1
    __shared__ double sCp[2][NC];       // control points of the element's span, by side
    const int2 wk = work[blockIdx.x];   // the pair and the one with the elements exchanged (-1: none listed)
    const SingularPair sp = list[wk.x];
    const int lane = threadIdx.x, half = lane >> 5, qi = lane & 31;
    int ja, a1, a2, jb, b1, b2;
    elem_of(o, sp.e, ja, a1, a2);
    elem_of(o, sp.f, jb, b1, b2);
    const int g4 = o.gs * o.gs * o.gs * o.gs, npts = singular_subrules(sp.kind) * g4;
    const double h = o.h, h4 = h * h * h * h;
    // this half's element, its frame and the span that holds it
    const int j = half ? jb : ja, e1 = half ? b1 : a1, e2 = half ? b2 : a2;
    const int code = sp.kind == 1 ? 0 : (half ? sp.fb : sp.fa);
    const double ox = code & 1, oy = (code >> 1) & 1, dx = 1.0 - 2.0 * ox, dy = 1.0 - 2.0 * oy;
    const bool swap = (code & 4) != 0;
    double ua = 0.0, va = 0.0, du = 1.0, dv = 1.0;
    bool inside = false;   // the element lies in one span
    if constexpr (GD > 0) {
        const PatchHdr hd = o.geo.hdr[j];
        const double *bu = o.geo.brk + hd.brk_u, *bv = o.geo.brk + hd.brk_v;
        int su = 0, sv = 0;
        while (su < hd.su - 1 && (e1 + 0.5) * h >= bu[su + 1]) ++su;
        while (sv < hd.sv - 1 && (e2 + 0.5) * h >= bv[sv + 1]) ++sv;
        ua = bu[su];
        va = bv[sv];
        inside = (su == 0 || e1 * h >= ua) && (su == hd.su - 1 || (e1 + 1) * h <= bu[su + 1]) &&
                 (sv == 0 || e2 * h >= va) && (sv == hd.sv - 1 || (e2 + 1) * h <= bv[sv + 1]);
        du = 1.0 / (bu[su + 1] - ua);
        dv = 1.0 / (bv[sv + 1] - va);
        const double *c = o.geo.cp + hd.cp + (size_t)(sv * hd.su + su) * NC;
        for (int i = qi; i < NC; i += 32) sCp[half][i] = c[i];
    }
    for (int i = qi; i < 2 * NE; i += 32) {
        const int d = i / NE, k = i % NE, e = d ? e2 : e1;
        sExt[half][d][k] = k < NP ? o.ext_p[(size_t)e * NP + k] : o.ext_q[(size_t)e * NQ + k - NP];
    }
    for (int i = qi; i < NB; i += 32) sV[half][i][ZERO] = 0.0;
    const double ih = 1.0 / h, cdiv = half ? 1.0 : o.cdiv;
    const double *r1 = rule + singular_rule_offset(sp.kind, g4) + (size_t)(half ? 2 : 0) * npts, *r2 = r1 + npts;
    const double *rw = rule + singular_rule_offset(sp.kind, g4) + (size_t)4 * npts;
    dx4 br[LT][LT], bi[LT][LT];
#pragma unroll
    for (int u = 0; u < LT; ++u)
#pragma unroll
        for (int v = 0; v < LT; ++v) {
            br[u][v] = dx4{0.0, 0.0, 0.0, 0.0};
            bi[u][v] = dx4{0.0, 0.0, 0.0, 0.0};
        }
    const int c = lane >> 4, m = lane & 15;
    // where this lane reads its operands in a point's row: value (or divergence) and tangent component
    int vo[LT], fo[LT];
#pragma unroll
    for (int u = 0; u < LT; ++u) {
        const int l = 16 * u + m;
        vo[u] = l >= NL ? ZERO : (SC || c < 3 ? l : NL + l);
        fo[u] = SC ? ZERO : FU + (l < P * (P + 1) ? 0 : 4) + c;
    }
    for (int p0 = 0; p0 < npts; p0 += NB) {
        const int pt = min(p0 + qi, npts - 1);   // beyond the end: the last point with the weight 0
        const double p1 = r1[pt], p2 = r2[pt], wt = p0 + qi < npts ? rw[pt] : 0.0;
        __syncthreads();   // the previous batch has been consumed
        double X[3] = {0.0, 0.0, 0.0};
        if (qi < NB) {
            const double x = ox + dx * (swap ? p2 : p1), y = oy + dy * (swap ? p1 : p2);
            double Fu[3], Fv[3];
            if (GD > 0 && inside) {
                constexpr int D = GD > 0 ? GD : 1;
                double Bu[D + 1], Du[D + 1], Bv[D + 1], Dv[D + 1];
                bernstein_t<D>(((e1 + x) * h - ua) * du, Bu, Du);
                bernstein_t<D>(((e2 + y) * h - va) * dv, Bv, Dv);
                double A[4] = {0, 0, 0, 0}, Au[4] = {0, 0, 0, 0}, Av[4] = {0, 0, 0, 0};
#pragma unroll
                for (int j2 = 0; j2 <= D; ++j2)
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        double w = 0.0, wu = 0.0;
#pragma unroll
                        for (int j1 = 0; j1 <= D; ++j1) {
                            const double q = sCp[half][(j2 * (D + 1) + j1) * 4 + k];
                            w = fma(Bu[j1], q, w);
                            wu = fma(Du[j1], q, wu);
                        }
                        A[k] = fma(Bv[j2], w, A[k]);
                        Au[k] = fma(Bv[j2], wu, Au[k]);
                        Av[k] = fma(Dv[j2], w, Av[k]);
                    }
                const double iw = 1.0 / A[3];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    X[k] = A[k] * iw;
                    Fu[k] = (Au[k] - X[k] * Au[3]) * iw * du;
                    Fv[k] = (Av[k] - X[k] * Av[3]) * iw * dv;
                }
            } else {
                double Y[3], Yu[3], Yv[3];
                geom_eval_generic(o.geo, j, (e1 + x) * h, (e2 + y) * h, Y, Yu, Yv);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    X[k] = Y[k];
                    Fu[k] = Yu[k];
                    Fv[k] = Yv[k];
                }
            }
            double Pu[P + 1], dPu[P + 1], Qu[P], Pv[P + 1], dPv[P + 1], Qv[P];
            spline_pieces_lds<P>(sExt[half][0], ih, x, Pu, dPu, Qu);
            spline_pieces_lds<P>(sExt[half][1], ih, y, Pv, dPv, Qv);
            double *row = sV[half][qi];
            if constexpr (SC) {
                const double J = cdiv * dm::surf_elem(Fu, Fv);
#pragma unroll
                for (int l = 0; l < NL; ++l) row[l] = Pu[l % (P + 1)] * Pv[l / (P + 1)] * J;
            } else {
#pragma unroll
                for (int l = 0; l < NL; ++l) {
                    const bool a0 = l < P * (P + 1);
                    const int r = a0 ? l : l - P * (P + 1);
                    const int t2 = a0 ? r / (P + 1) : r / P, t1 = a0 ? r % (P + 1) : r % P;
                    row[l] = a0 ? Pu[t1] * Qv[t2] : Qu[t1] * Pv[t2];
                    row[NL + l] = cdiv * (a0 ? dPu[t1] * Qv[t2] : Qu[t1] * dPv[t2]);
                }
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    row[FU + k] = Fu[k];
                    row[FU + 4 + k] = Fv[k];
                }
                row[FU + 3] = 1.0;
                row[FU + 7] = 1.0;
            }
            if (half == 1) {
                sX[qi][0] = X[0];
                sX[qi][1] = X[1];
                sX[qi][2] = X[2];
            }
        }
        __syncthreads();
        if (half == 0 && qi < NB) {
            const double d0 = X[0] - sX[qi][0], d1 = X[1] - sX[qi][1], d2 = X[2] - sX[qi][2];
            const double2 K = dm::helmholtz_r2(o.kappa, fma(d0, d0, fma(d1, d1, d2 * d2)));
            sK[qi] = p0 + qi < npts ? cscale(wt * h4, K) : make_double2(0.0, 0.0);
        }
        __syncthreads();
#pragma unroll 8
        for (int q0 = 0; q0 < NB; q0 += SC ? 4 : 1) {
            const int q = SC ? q0 + c : q0;
            const double2 K = sK[q];
            double av[LT], bv[LT];
#pragma unroll
            for (int u = 0; u < LT; ++u) {
                av[u] = SC ? sV[0][q][vo[u]] : sV[0][q][vo[u]] * sV[0][q][fo[u]];
                bv[u] = SC ? sV[1][q][vo[u]] : sV[1][q][vo[u]] * sV[1][q][fo[u]];
            }
#pragma unroll
            for (int u = 0; u < LT; ++u)
#pragma unroll
                for (int v = 0; v < LT; ++v) {
                    br[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(K.x * av[u], bv[v], br[u][v], 0, 0, 0);
                    bi[u][v] = __builtin_amdgcn_mfma_f64_16x16x4f64(K.y * av[u], bv[v], bi[u][v], 0, 0, 0);
                }
        }
    }
    // lane holds B[16 u + lane/16 + 4 j][16 v + lane % 16]; the element-pair block goes
    // to its own slot, added to the near-field block by k_near_regular in list order
    double2 *dst = o.sblk + (size_t)wk.x * NL * NL, *tr = o.sblk + (size_t)max(wk.y, 0) * NL * NL;
#pragma unroll
    for (int u = 0; u < LT; ++u)
#pragma unroll
        for (int v = 0; v < LT; ++v)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int l = 16 * u + (lane >> 4) + 4 * j, lb = 16 * v + (lane & 15);
                if (l >= NL || lb >= NL) continue;
                const double2 b = make_double2(br[u][v][j], bi[u][v][j]);
                dst[l * NL + lb] = b;
                if (wk.y >= 0) tr[lb * NL + l] = b;
            }
}

}  // namespace

namespace {
template <int NL>
void launch_near_regular_nl(ige_op op, dim3 grid, size_t shm, int sb, int ce1, int ce2, int cs1, int cs2, int sstep)
{
    const DevOp &o = op->view;
    hipStream_t s = lstream(op);
    auto run = [&](auto kern) {
        if (shm > 48 * 1024)
            IGE_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm));
        hipLaunchKernelGGL(kern, grid, dim3(256), shm, s, o, sb, ce1, ce2, cs1, cs2, sstep);
    };
    // steps of four points: the rules have g^2 points, g <= 8
    const int ts = (o.G2 + 3) / 4;
    if (ts <= 4) {
        if constexpr (NL <= 12) run(k_near_regular_o2<NL, 4>);
        else run(k_near_regular<NL, 4>);
    } else if (ts <= 7) {
        if constexpr (NL <= 12) run(k_near_regular_o2<NL, 7>);
        else run(k_near_regular<NL, 7>);
    } else if (ts <= 9) run(k_near_regular<NL, 9>);
    else if (ts <= 13) run(k_near_regular<NL, 13>);
    else run(k_near_regular<NL, 16>);
}

// shared memory of k_near_regular: the block rows of the test element over each
// quadrant of a trial square of sb x sb elements
size_t near_regular_shm(int sb, int p, int nl, bool scalar)
{
    const size_t nr = nl <= 24 ? nl : 16 * near_regular_lr(nl), wq = (sb + 1) / 2 + p;   // rows per workgroup
    return sizeof(double2) * 4 * nr * (scalar ? 1 : 2) * wq * wq;
}

// trial squares of sb x sb elements: the largest power of two <= s of which two
// workgroups fit on a CU (with their 5 KB of tables)
int near_regular_sb(int s, int p, int nl, bool scalar)
{
    int sb = s;
    while (sb > 1 && near_regular_shm(sb, p, nl, scalar) > 75 * 1024) sb /= 2;
    return sb;
}
}  // namespace

void launch_near_regular(ige_op op)
{
    const DevOp &o = op->view;
    if (o.nblk == 0) return;
    IGE_REQUIRE(o.G2 <= 64, "regular near-field rule limited to 8 x 8 points");
    const int sb = near_regular_sb(o.s, o.p, o.nl, o.scalar);
    const int nsb = o.s / sb;
    // colours: test elements p + 1 apart (a glued function spans at most p + 1
    // elements per direction); with several trial squares per leaf, squares whose gap
    // of (sstep - 1) sb elements is at least p
    const int P1 = o.p + 1, sstep = nsb > 1 ? 1 + (o.p + sb - 1) / sb : 1;
    const size_t shm = near_regular_shm(sb, o.p, o.nl, o.scalar);
    for (int ce2 = 0; ce2 < std::min(P1, o.s); ++ce2)
        for (int ce1 = 0; ce1 < std::min(P1, o.s); ++ce1)
            for (int cs2 = 0; cs2 < std::min(sstep, nsb); ++cs2)
                for (int cs1 = 0; cs1 < std::min(sstep, nsb); ++cs1) {
                    const int64_t n1 = (o.s - ce1 + P1 - 1) / P1, n2 = (o.s - ce2 + P1 - 1) / P1;
                    const int64_t m1 = (nsb - cs1 + sstep - 1) / sstep, m2 = (nsb - cs2 + sstep - 1) / sstep;
                    const int LT = (o.nl + 15) / 16;
                    const int64_t nrt = LT / near_regular_lr(o.nl);   // row-tile workgroups per element
                    const int64_t nwg = o.nblk * n1 * n2 * m1 * m2 * nrt;
                    if (nwg == 0) continue;
                    const dim3 grid((unsigned)nwg);
                    switch (o.nl) {
                        case 4: launch_near_regular_nl<4>(op, grid, shm, sb, ce1, ce2, cs1, cs2, sstep); break;
                        case 9: launch_near_regular_nl<9>(op, grid, shm, sb, ce1, ce2, cs1, cs2, sstep); break;
                        case 12: launch_near_regular_nl<12>(op, grid, shm, sb, ce1, ce2, cs1, cs2, sstep); break;
                        case 16: launch_near_regular_nl<16>(op, grid, shm, sb, ce1, ce2, cs1, cs2, sstep); break;
                        case 24: launch_near_regular_nl<24>(op, grid, shm, sb, ce1, ce2, cs1, cs2, sstep); break;
                        case 25: launch_near_regular_nl<25>(op, grid, shm, sb, ce1, ce2, cs1, cs2, sstep); break;
                        default: launch_near_regular_nl<40>(op, grid, shm, sb, ce1, ce2, cs1, cs2, sstep); break;
                    }
                    IGE_HIP(hipGetLastError());
                }
}

namespace {
template <int P, bool SC>
void launch_near_singular_p(ige_op op, int gd, const double *rule)
{
    const DevOp &o = op->view;
    const dim3 grid((unsigned)op->d_sing_work.n), blk(64);
    hipStream_t s = lstream(op);
    if (gd == 1) hipLaunchKernelGGL((k_near_singular<P, SC, 1>), grid, blk, 0, s, o, op->d_sing.p, op->d_sing_work.p, rule);
    else if (gd == 2) hipLaunchKernelGGL((k_near_singular<P, SC, 2>), grid, blk, 0, s, o, op->d_sing.p, op->d_sing_work.p, rule);
    else hipLaunchKernelGGL((k_near_singular<P, SC, 0>), grid, blk, 0, s, o, op->d_sing.p, op->d_sing_work.p, rule);
    IGE_HIP(hipGetLastError());
}
}  // namespace

// scratch of launch_near_singular: the pairs' blocks, then the rule's table
size_t near_singular_scratch(ige_op op)
{
    const DevOp &o = op->view;
    return std::max<size_t>(1, (size_t)op->nsing * o.nl * o.nl) + singular_rule_doubles(o.gs) / 2;
}

void launch_near_singular(ige_op op, const Geometry &G)
{
    const DevOp &o = op->view;
    if (op->nsing == 0) return;
    // unrolled geometry where all patches are bilinear or all biquadratic
    int gd = G.hdr.empty() ? 0 : G.hdr[0].pu;
    for (const auto &h : G.hdr)
        if (h.pu != gd || h.pv != gd) gd = 0;
    double *rule = reinterpret_cast<double *>(op->d_sblk.p + (size_t)op->nsing * o.nl * o.nl);
    const int n = 18 * o.gs * o.gs * o.gs * o.gs;
    hipLaunchKernelGGL(k_singular_rule, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, lstream(op), o, rule);
    IGE_HIP(hipGetLastError());
#define IGE_SP(P) \
    if (o.scalar) launch_near_singular_p<P, true>(op, gd, rule); \
    else launch_near_singular_p<P, false>(op, gd, rule); \
    break
    switch (o.p) {
        case 1: IGE_SP(1);
        case 2: IGE_SP(2);
        case 3: IGE_SP(3);
        default: IGE_SP(4);
    }
#undef IGE_SP
}

}  // namespace ige
