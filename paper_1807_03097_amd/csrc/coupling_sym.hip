// a5 for one FP64 column: the coupling over unordered far pairs on the 4x4x4 FP64 matrix
// instruction.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <string>

#include "device_math.hpp"
#include "near_item.hpp"
#include "op.hpp"

namespace ige {

namespace {

using dm::cadd;
using dm::cscale;
using dm::row_ror;
using dm::surf_elem;

__device__ inline double perm_lane(int addr, double v)
{
    const int lo = __builtin_amdgcn_ds_bpermute(addr, __double2loint(v)), hi = __builtin_amdgcn_ds_bpermute(addr, __double2hiint(v));
    return __hiloint2double(hi, lo);
}
// The kernel is symmetric and both clusters of a far pair have the same reference nodes, so
// the block of (s, t) is the transpose of the block of (t, s): every kernel value serves
//   u_t[m]  += sum_m' G(|x_m - x'_m'|) v_s[m']   (row side, summed over the item's partners)
//   u_s[m'] += sum_m  G(|x_m - x'_m'|) v_t[m]    (column side, per pair)
// Work item = cluster t (a chunk of its rows) with a few partners s > t.  In a step a wave evaluates 16 rows x
// 4 columns of G, one value per lane (row 16 t + lane % 16, column 4 g + lane / 16): the A
// operand of v_mfma_f64_4x4x4 (four blocks of 4 rows) whose 4 output columns are the four
// source fields, so real and imaginary parts take four instructions with nothing idle; a
// transposition inside the wave (four ds_bpermute) gives the operand of the column side.
// All sums stay in registers: the rows of the item over all partners, a group's 4 columns
// over the row tiles.
// Bound by FP64 issue: about 36 operations of the kernel value, eight 4x4x4 products (18
// cycles each) and the transposition per 64 values that stand for 128 ordered node pairs;
// the ordered form (one value per ordered pair, 16 complex multiply-adds of a lane, partner
// nodes and fields through shared memory) issued 61 instructions per 64.  Level 5, 5,520
// ordered pairs of 81 nodes: 92 us before, 69 now (73 between events), the apply beside
// the near-field product 164 and 138 us (with that product's own step).
//
// The waves are two row halves (RT tiles each) x two column halves of the same partner.  The
// next partner's nodes and fields are on their way into registers during the whole of the
// current one and then go to the other half of a double buffer in shared memory: beside the
// near-field product, which keeps the memory system full, a load takes several microseconds,
// and loading them group by group stalled the kernel (the pair of them took as long as one
// after the other).
constexpr int kSymGroup = 3;   // row tiles in one phase
template <int RT>
struct SymShared {
    double2 tab[256];                 // (cos, sin)(j pi/128) / (4 pi)
    // per buffer: fields [node][4], then nodes [3][node]; after the last partner the rows' sums
    double2 v[2][4 * 16 * 2 * RT];
    double x[2][3 * 16 * 2 * RT];
    double2 col[2][4 * 16 * 2 * RT];  // column side of the pair, per row half
    // the last row of clusters of 16 k + 1 nodes: its node and fields, its sums per column
    double left[12];
    double lacc[8][16 * 2 * RT];
};

// one group of 4 columns against NT row tiles: phase by phase over a few tiles, so that the
// table reads and the transpositions of one tile return behind the arithmetic of the others
template <int NT, int RT>
__device__ __forceinline__ void sym_group(double kap, const double2 *tab, int tr, const double (&x)[RT][3],
                                          const double (&vr)[RT], const double (&vi)[RT], double (&yr)[RT], double (&yi)[RT],
                                          double y0, double y1, double y2, double2 vs, double2 &col)
{
    double cr = 0.0, ci = 0.0, dr = 0.0, di = 0.0;
#pragma unroll
    for (int t0 = 0; t0 < NT; t0 += kSymGroup) {
        constexpr int TG = kSymGroup;
        double ir[TG], c0[TG], s0[TG];
        double2 cs2[TG], G[TG], H[TG];
#pragma unroll
        for (int k = 0; k < TG; ++k) {
            const int t = t0 + k;
            if (t >= NT) break;
            const double d0 = x[t][0] - y0, d1 = x[t][1] - y1, d2 = x[t][2] - y2;
            dm::helmholtz_tab_begin(kap, fma(d0, d0, fma(d1, d1, d2 * d2)), tab, ir[k], c0[k], s0[k], cs2[k]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < TG; ++k) {
            if (t0 + k >= NT) break;
            G[k] = dm::helmholtz_tab_end(ir[k], c0[k], s0[k], cs2[k]);
            H[k] = make_double2(perm_lane(tr, G[k].x), perm_lane(tr, G[k].y));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int k = 0; k < TG; ++k) {
                const int t = t0 + k;
                if (t >= NT) break;
                if (h == 0) {
                    yr[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(G[k].x, vs.x, yr[t], 0, 0, 0);
                    yi[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(G[k].x, vs.y, yi[t], 0, 0, 0);
                } else {
                    yr[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(G[k].y, vs.y, yr[t], 0, 0, 1);   // - A B + C
                    yi[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(G[k].y, vs.x, yi[t], 0, 0, 0);
                }
            }
#pragma unroll
        for (int k = 0; k < TG; ++k) {
            const int t = t0 + k;
            if (t >= NT) break;
            cr = __builtin_amdgcn_mfma_f64_4x4x4f64(H[k].x, vr[t], cr, 0, 0, 0);
            ci = __builtin_amdgcn_mfma_f64_4x4x4f64(H[k].x, vi[t], ci, 0, 0, 0);
            dr = __builtin_amdgcn_mfma_f64_4x4x4f64(H[k].y, vi[t], dr, 0, 0, 1);
            di = __builtin_amdgcn_mfma_f64_4x4x4f64(H[k].y, vr[t], di, 0, 0, 0);
        }
    }
    col.x += cr + dr;
    col.y += ci + di;
}

template <int RT>
__device__ __forceinline__ void m2l_sym_body(const DevOp &o, int w, int nwork, const SymWork &wk, const int32_t *partner,
                                             const double2 *src, double2 *part, int Q, SymShared<RT> &sh)
{
    constexpr int NP = 16 * 2 * RT;                  // padded nodes
    constexpr int LV = (4 * NP + 255) / 256, LX = (3 * NP + 255) / 256;
    const int Qs = o.Q, tid = threadIdx.x, lane = tid & 63;
    const int th = __builtin_amdgcn_readfirstlane((tid >> 6) & 1), ch = __builtin_amdgcn_readfirstlane(tid >> 7);
    const int fi = lane & 3, blk = (lane >> 2) & 3, hi = lane >> 4;
    const int tr = 4 * (hi + 4 * blk + 16 * fi);     // lane that holds the transposed entry, in bytes
    // one row beyond the last full tile is not worth a tile of its own: the waves of the second
    // row half take it with a column per lane
    const bool left = Q % 16 == 1 && Q > 16 && Q <= NP;
    const int ntile = left ? Q / 16 : (min(Q - wk.r0, NP) + 15) / 16, na = (ntile + 1) / 2;
    const int r0 = wk.r0 + 16 * na * th, nt = __builtin_amdgcn_readfirstlane(th ? ntile - na : na);
    const int rows = max(0, min((left ? Q - 1 : Q) - r0, 16 * nt));
    // the partners in column chunks of NP nodes (one chunk up to degree 10)
    const int nc = (Q + NP - 1) / NP, nstep = (wk.end - wk.beg) * nc;
    const double kap = o.kappa;
    double2 lv[LV];
    double lx[LX];
    auto fetch = [&](int st) {
        const int sc = partner[wk.beg + st / nc], c0 = (st % nc) * NP;
        const double *Xs = o.nodeX + (size_t)sc * 3 * Qs;
        const double2 *Vs = src + (size_t)sc * 4 * Qs;
#pragma unroll
        for (int i = 0; i < LV; ++i) {   // [field][node] in memory
            const int j = tid + 256 * i, f = j / NP, m = j % NP;
            lv[i] = (f < 4 && c0 + m < Q) ? Vs[(size_t)f * Qs + c0 + m] : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int i = 0; i < LX; ++i) {
            const int j = tid + 256 * i, d = j / NP, m = j % NP;
            lx[i] = d < 3 ? Xs[(size_t)d * Qs + min(c0 + m, Q - 1)] : 0.0;
        }
    };
    auto stage = [&](int b) {
#pragma unroll
        for (int i = 0; i < LV; ++i) {
            const int j = tid + 256 * i;
            if (j < 4 * NP) sh.v[b][(j % NP) * 4 + j / NP] = lv[i];
        }
#pragma unroll
        for (int i = 0; i < LX; ++i)
            if (tid + 256 * i < 3 * NP) sh.x[b][tid + 256 * i] = lx[i];
    };
    fetch(0);
    const double *Xt = o.nodeX + (size_t)wk.tgt * 3 * Qs;
    const double2 *Vt = src + ((size_t)wk.tgt * 4 + fi) * Qs;
    double x[RT][3], vr[RT], vi[RT], yr[RT], yi[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int r = min(Q - 1, r0 + 16 * t + (lane & 15)), rv = 16 * t + 4 * blk + hi;
        x[t][0] = Xt[r];
        x[t][1] = Xt[Qs + r];
        x[t][2] = Xt[2 * Qs + r];
        const double2 v = rv < rows ? Vt[r0 + rv] : make_double2(0.0, 0.0);
        vr[t] = v.x;
        vi[t] = v.y;
        yr[t] = yi[t] = 0.0;
    }
    stage(0);
    if (left) {
        if (tid < 3) sh.left[tid] = Xt[tid * Qs + Q - 1];
        else if (tid < 7) {
            const double2 v = src[((size_t)wk.tgt * 4 + tid - 3) * Qs + Q - 1];
            sh.left[4 + 2 * (tid - 3)] = v.x;
            sh.left[5 + 2 * (tid - 3)] = v.y;
        }
        for (int i = tid; i < 8 * NP; i += 256) (&sh.lacc[0][0])[i] = 0.0;
    }
    __syncthreads();
    for (int st = 0; st < nstep; ++st) {
        const int b = st & 1, c0 = (st % nc) * NP;
        if (st + 1 < nstep) fetch(st + 1);
        const int ng = (min(Q - c0, NP) + 3) / 4, gm = (ng + 1) / 2, g0 = ch == 0 ? 0 : gm, g1 = ch == 0 ? gm : ng;
        for (int g = g0; g < g1; ++g) {
            const int m = 4 * g + hi;
            const double y0 = sh.x[b][m], y1 = sh.x[b][NP + m], y2 = sh.x[b][2 * NP + m];
            const double2 vs = sh.v[b][4 * m + fi];
            double2 col = make_double2(0.0, 0.0);
            if (nt == RT) {
                sym_group<RT, RT>(kap, sh.tab, tr, x, vr, vi, yr, yi, y0, y1, y2, vs, col);
            } else if (RT > 1 && nt == RT - 1) {
                sym_group<(RT > 1 ? RT - 1 : 1), RT>(kap, sh.tab, tr, x, vr, vi, yr, yi, y0, y1, y2, vs, col);
            } else {   // levels of a smaller degree
                if (RT > 2 && nt == 2) sym_group<(RT > 2 ? 2 : 1), RT>(kap, sh.tab, tr, x, vr, vi, yr, yi, y0, y1, y2, vs, col);
                else if (nt == 1) sym_group<1, RT>(kap, sh.tab, tr, x, vr, vi, yr, yi, y0, y1, y2, vs, col);
            }
            // column 4 g + lane / 16, field lane % 4: sum over the four row blocks
            col.x += row_ror<8>(col.x);
            col.y += row_ror<8>(col.y);
            col.x += row_ror<4>(col.x);
            col.y += row_ror<4>(col.y);
            if (blk == 0) sh.col[th][fi * NP + m] = col;
        }
        if (left && th == 1 && lane < 4 * (g1 - g0)) {
            // the last row against this wave's own columns, one per lane (which other lanes of the
            // wave have just written)
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const int m = 4 * g0 + lane, sl = ch * (NP / 2) + lane;
            const double d0 = sh.left[0] - sh.x[b][m], d1 = sh.left[1] - sh.x[b][NP + m], d2 = sh.left[2] - sh.x[b][2 * NP + m];
            double ir, kr;
            const double2 G = dm::helmholtz_r2_tab(kap, fma(d0, d0, fma(d1, d1, d2 * d2)), sh.tab, ir, kr);
#pragma unroll
            for (int f = 0; f < 4; ++f) {
                const double2 a = dm::cmac(make_double2(sh.lacc[2 * f][sl], sh.lacc[2 * f + 1][sl]), G, sh.v[b][4 * m + f]);
                sh.lacc[2 * f][sl] = a.x;
                sh.lacc[2 * f + 1][sl] = a.y;
                double2 &cm = sh.col[1][f * NP + m];
                cm = dm::cmac(cm, G, make_double2(sh.left[4 + 2 * f], sh.left[5 + 2 * f]));
            }
        }
        __syncthreads();
        // the pair's column side out, the next partner in
        double2 *out = part + (size_t)(nwork + wk.beg + st / nc) * 4 * Qs + c0;
        for (int i = tid; i < 4 * NP; i += 256) {
            const int f = i / NP, m = i % NP;
            if (c0 + m < Q) out[(size_t)f * Qs + m] = cadd(sh.col[0][i], sh.col[1][i]);
        }
        if (st + 1 < nstep) stage(b ^ 1);
        __syncthreads();
    }
    // row side: the two column halves in order.  A lane holds row 16 t + 4 blk + lane / 16 of its half
    double *red = reinterpret_cast<double *>(&sh.v[0][0]);   // [column half][tile][2][64]
#pragma unroll
    for (int t = 0; t < RT; ++t)
        if (t < nt) {
            double *d = red + ((size_t)(ch * 2 * RT + th * na + t) * 2) * 64 + lane;
            d[0] = yr[t];
            d[64] = yi[t];
        }
    __syncthreads();
    const int rtop = wk.r0 + 16 * ntile;
    for (int i = tid; i < 4 * Q; i += 256) {
        const int f = i / Q, mm = i % Q, r = mm - wk.r0;
        if (left && mm == Q - 1) continue;
        double2 v = make_double2(0.0, 0.0);
        if (r >= 0 && mm < rtop) {
            const int t = r / 16, l = f + 4 * ((r % 16) / 4) + 16 * (r % 4);
            const double *p0 = red + (size_t)t * 128 + l, *p1 = p0 + (size_t)2 * RT * 128;
            v = make_double2(p0[0] + p1[0], p0[64] + p1[64]);
        }
        part[((size_t)w * 4 + f) * Qs + mm] = v;
    }
    if (left) {   // 32 threads per value, a fixed butterfly
        const int k = tid >> 5;
        double a = 0.0;
        for (int i = tid & 31; i < NP; i += 32) a += sh.lacc[k][i];
#pragma unroll
        for (int off = 16; off >= 1; off >>= 1) a += __shfl_xor(a, off, 32);
        if ((tid & 31) == 0) reinterpret_cast<double *>(part + ((size_t)w * 4 + k / 2) * Qs + Q - 1)[k & 1] = a;
    }
}

template <int RT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(RT <= 3 ? 4 : 3))) void k_m2l_sym(
    DevOp o, int nwork, const SymWork *work, const int32_t *partner, const double2 *src, double2 *part)
{
    __shared__ SymShared<RT> sh;
    sh.tab[threadIdx.x] = o.sctab[threadIdx.x];
    const SymWork wk = work[blockIdx.x];
    int lvl = 0;
    while (lvl < o.L && wk.tgt >= o.lvl_off[lvl + 1]) ++lvl;
    const int Q = (o.ql[lvl] + 1) * (o.ql[lvl] + 1);
    m2l_sym_body<RT>(o, blockIdx.x, nwork, wk, partner, src, part, Q, sh);
}

// The same with the near-field product's items in the same launch, behind the coupling's: where that
// product is short, a second stream's fork and join cost more than the two hide (level 4, 64 nodes
// per cluster: 40.4 and 17.0 us one after the other, 49.9 together)
template <int RT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(RT <= 3 ? 4 : 3))) void k_m2l_sym_near(
    DevOp o, int nwork, const SymWork *work, const int32_t *partner, const double2 *src, double2 *part, NearCmpView v,
    int64_t na, int64_t nw, const double2 *x, double2 *npart)
{
    struct NearShared {
        double2 xr[kCmpRows], yc[3][256];
    };
    constexpr size_t kBytes = sizeof(SymShared<RT>) > sizeof(NearShared) ? sizeof(SymShared<RT>) : sizeof(NearShared);
    __shared__ __attribute__((aligned(16))) char smem[kBytes];
    if ((int)blockIdx.x < nwork) {
        SymShared<RT> &sh = *reinterpret_cast<SymShared<RT> *>(smem);
        sh.tab[threadIdx.x] = o.sctab[threadIdx.x];
        const SymWork wk = work[blockIdx.x];
        int lvl = 0;
        while (lvl < o.L && wk.tgt >= o.lvl_off[lvl + 1]) ++lvl;
        const int Q = (o.ql[lvl] + 1) * (o.ql[lvl] + 1);
        m2l_sym_body<RT>(o, blockIdx.x, nwork, wk, partner, src, part, Q, sh);
        return;
    }
    NearShared &ns = *reinterpret_cast<NearShared *>(smem);
    const int64_t b = (int64_t)blockIdx.x - nwork;
    if (b < nw) near_cmp_item<3, 2, 0>(v, v.order[na + b], x, npart, ns.xr, ns.yc);
    else near_cmp_item<2, 2, 0>(v, v.order[b - nw], x, npart, ns.xr, ns.yc);
}

// Per cluster, the sum of its slots (row sides of its items, then the column sides of its pairs),
// converted to the test-side fields.  S threads per value take every S-th slot, eight loads at a
// time, and are added in order: one thread per value waited for six rounds of loads (level 4,
// 64 nodes, about 40 slots: 10.2 us, 7 now).
__global__ __launch_bounds__(1024) void k_m2l_reduce_sym(DevOp o, int S, const int32_t *ptr, const int32_t *idx,
                                                         const double2 *part, double2 *loc)
{
    extern __shared__ double2 su[];   // [S][4][Q]
    const int gc = blockIdx.x, Qs = o.Q;
    int lvl = 0;
    while (lvl < o.L && gc >= o.lvl_off[lvl + 1]) ++lvl;
    const int Q = (o.ql[lvl] + 1) * (o.ql[lvl] + 1);
    const int b = ptr[gc], e = ptr[gc + 1];
    const int G = blockDim.x / S, q = __builtin_amdgcn_readfirstlane(threadIdx.x / G);   // uniform: scalar list reads
    for (int r = threadIdx.x - q * G; r < 4 * Q; r += G) {
        const int f = r / Q, mm = r - f * Q;
        double2 v = make_double2(0, 0);
        for (int w0 = b + q; w0 < e; w0 += 8 * S) {
            double2 t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                t[u] = w0 + u * S < e ? part[((size_t)idx[w0 + u * S] * 4 + f) * Qs + mm] : make_double2(0, 0);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (w0 + u * S < e) v = cadd(v, t[u]);
        }
        su[q * 4 * Q + r] = v;
    }
    __syncthreads();
    if (S > 1) {
        for (int i = threadIdx.x; i < 4 * Q; i += blockDim.x) {
            double2 v = su[i];
            for (int q = 1; q < S; ++q) v = cadd(v, su[q * 4 * Q + i]);
            su[i] = v;
        }
        __syncthreads();
    }
    const double ik2 = 1.0 / (o.kappa * o.kappa);
    for (int mm = threadIdx.x; mm < Q; mm += blockDim.x) {
        const double *T = o.nodeT + (size_t)gc * 6 * Qs;
        double2 *L = loc + (size_t)gc * 3 * Qs;
        if (o.scalar) {   // scalar: t = |J(x_m)| u (the target's surface element)
            const double Fu[3] = {T[mm], T[Qs + mm], T[2 * Qs + mm]}, Fv[3] = {T[3 * Qs + mm], T[4 * Qs + mm], T[5 * Qs + mm]};
            L[mm] = make_double2(0, 0);
            L[Qs + mm] = make_double2(0, 0);
            L[2 * Qs + mm] = cscale(surf_elem(Fu, Fv), su[3 * Q + mm]);
            continue;
        }
        double2 t1 = make_double2(0, 0), t2 = make_double2(0, 0);
        for (int k = 0; k < 3; ++k) {
            t1 = cadd(t1, cscale(T[k * Qs + mm], su[k * Q + mm]));
            t2 = cadd(t2, cscale(T[(3 + k) * Qs + mm], su[k * Q + mm]));
        }
        L[mm] = t1;
        L[Qs + mm] = t2;
        L[2 * Qs + mm] = cscale(-ik2, su[3 * Q + mm]);
    }
}

}  // namespace

SymRule sym_rule(const ige_op_s *op)
{
    const auto &T = op->T;
    const auto &F = op->F;
    SymRule R;
    // IGE_M2L_SYM=1 takes IGE_M2L_SYM_CHUNK (default 4) partners per item instead of the rule's
    if (const char *e = std::getenv("IGE_M2L_SYM"))
        R.asked = std::atoi(e) != 0 && !F.varq && (F.q + 1) * (F.q + 1) <= 81 && !T.far.empty();
    if (R.asked) {
        R.chunk = 4;
        if (const char *e = std::getenv("IGE_M2L_SYM_CHUNK")) R.chunk = std::max(1, std::min(64, std::atoi(e)));
    }
    // Partners per item when not asked for.  Two: the shorter items hide the kernel's own
    // latencies and end together (level 4 solve, 829 iterations, 107 ms against 113 with three and
    // 118 with four).  Four beside a near-field product that takes at least half as long: fewer
    // items start and load their rows beside it (level 5, one column, 141 us against 150 with two
    // or three, 153 with six; torus level 5, degree 5, near field four times the coupling: 616
    // against 663; a tie at level 6, degrees up to 14: 725 against 719).  The times compared are near bytes
    // at 4.7 TB/s and steps of 16 rows x 4 columns at 340 cycles on 1,024 SIMDs, all of them
    // busy: a scale for the coupling, not its time (level 5: 40 us by it, 69 measured).
    double steps = 0.0;
    int64_t items = 0;
    int rt = 1;
    for (const auto &f : T.far) {
        const int Q = (F.ql[f[0]] + 1) * (F.ql[f[0]] + 1);
        steps += 0.5 * ((Q + 12) / 16) * ((Q + 3) / 4);
        rt = std::max(rt, (Q + 15) / 16);   // node tiles of a cluster
    }
    R.near_us = (double)op->cmp.nval * 16.0 / 4.7e6;
    R.far_us = steps * 340.0 / (1024.0 * 2400.0);
    rt = 2 * ((std::min(rt, kSymTiles) + 1) / 2);
    // Few pairs: one partner per item where that makes no more than four items per CU, and with less
    // than one per CU 64 rows per item.  A wave is then bound by its own latencies (level 4, 60
    // pairs of 81 nodes: 39 us with two partners and all rows, 14 now; torus level 3, 72 pairs of 225
    // nodes, 128 rows per item: 70 and 47).
    for (const auto &f : T.far) items += ((F.ql[f[0]] + 1) * (F.ql[f[0]] + 1) + 16 * rt - 1) / (16 * rt);
    if (R.chunk <= 0) R.chunk = items / 2 < 1024 ? 1 : (R.near_us > 0.5 * R.far_us ? 4 : 2);
    if (items / 2 < 256) rt = std::min(rt, 4);
    R.rows = 16 * rt;
    // partial results: one per item and one per pair, for each chunk of rows
    for (size_t i = 0, k; i < T.far.size(); i = k) {   // sorted by level, cluster, partner
        const int lvl = T.far[i][0], tg = T.far[i][1], Q = (F.ql[lvl] + 1) * (F.ql[lvl] + 1);
        size_t up = 0;
        for (k = i; k < T.far.size() && T.far[k][0] == lvl && T.far[k][1] == tg; ++k) up += T.far[k][2] > tg;
        R.parts += (up + (up + R.chunk - 1) / R.chunk) * ((Q + R.rows - 1) / R.rows);
    }
    return R;
}

void plan_m2l_sym(ige_op op, hipStream_t s)
{
    const auto &T = op->T;
    const auto &F = op->F;
    const SymRule rule = sym_rule(op);
    const int chunk = rule.chunk, rt = rule.rows / 16;
    std::vector<int32_t> spart;
    op->swork.clear();
    // each pair is visited from the cluster of smaller index alone
    const auto upper = std::count_if(T.far.begin(), T.far.end(), [](const auto &f) { return f[2] > f[1]; });
    IGE_REQUIRE(2 * (size_t)upper == T.far.size(), "far pairs are not symmetric");
    op->m2l_sym = rule.asked;
    op->near_us = rule.near_us;
    op->far_us = rule.far_us;
    op->sym_rt = rt / 2;
    size_t i = 0;
    while (i < T.far.size()) {   // sorted by level, cluster, partner
        const int lvl = T.far[i][0], tg = T.far[i][1], Q = (F.ql[lvl] + 1) * (F.ql[lvl] + 1);
        size_t k = i;
        while (k < T.far.size() && T.far[k][0] == lvl && T.far[k][1] == tg) ++k;
        for (int r0 = 0; r0 < Q; r0 += 16 * rt) {
            const int beg = (int)spart.size();
            for (size_t j = i; j < k; ++j)
                if (T.far[j][2] > tg) spart.push_back((int32_t)(op->lvl_off[lvl] + T.far[j][2]));
            for (int b = beg; b < (int)spart.size(); b += chunk)
                op->swork.push_back({(int32_t)(op->lvl_off[lvl] + tg), b, std::min((int)spart.size(), b + chunk), r0});
        }
        i = k;
    }
    // the longest items launch first
    std::stable_sort(op->swork.begin(), op->swork.end(),
                     [](const SymWork &a, const SymWork &b) { return a.end - a.beg > b.end - b.beg; });
    // per cluster its slots: the row sides of its items, then the column sides of its pairs,
    // in that fixed order
    const int nw = (int)op->swork.size();
    std::vector<int32_t> sptr((size_t)op->NC + 1, 0);
    for (const auto &w : op->swork) sptr[w.tgt + 1]++;
    for (int32_t c : spart) sptr[c + 1]++;
    for (int c = 0; c < op->NC; ++c) sptr[c + 1] += sptr[c];
    std::vector<int32_t> sidx(sptr[op->NC]), fill(sptr.begin(), sptr.end() - 1);
    for (int w = 0; w < nw; ++w) sidx[fill[op->swork[w].tgt]++] = w;
    for (size_t k = 0; k < spart.size(); ++k) sidx[fill[spart[k]]++] = nw + (int32_t)k;
    op->d_swork.upload(op->swork, s);
    op->d_spartner.upload(spart, s);
    op->d_sred_ptr.upload(sptr, s);
    op->d_sred_idx.upload(sidx, s);
    IGE_REQUIRE((size_t)nw + spart.size() == rule.parts, "coupling partials miscounted");
    op->nspart = rule.parts * 4 * op->view.Q;   // d_spart, allocated at the end of the assembly
}

void launch_m2l_sym(ige_op op)
{
    const DevOp &o = op->view;
    const int nw = (int)op->swork.size();
    if (nw == 0) return;
    hipStream_t s = lstream(op);
#define IGE_MS(RT) \
    hipLaunchKernelGGL(k_m2l_sym<RT>, dim3(nw), dim3(256), 0, s, o, nw, op->d_swork.p, op->d_spartner.p, op->d_src.p, \
                       op->d_spart.p)
    switch (op->sym_rt) {
        case 1: IGE_MS(1); break;
        case 2: IGE_MS(2); break;
        case 3: IGE_MS(3); break;
        default: IGE_MS(4); break;
    }
#undef IGE_MS
    IGE_HIP(hipGetLastError());
}

// whether the near-field product of one column can go into the coupling's launch
bool m2l_sym_near_ok(const ige_op_s *op)
{
    return op->cmp_on && op->near_one && op->cmp_rs == 2 && op->cmp.maxn <= 192 && !op->swork.empty();
}

void launch_m2l_sym_near(ige_op op, const double2 *x)
{
    const DevOp &o = op->view;
    const NearCmpView &v = op->cview;
    const int nw = (int)op->swork.size();
    const int64_t na = op->cmp.nnarrow, nn = v.nwork;
    hipStream_t s = lstream(op);
#define IGE_MSN(RT) \
    hipLaunchKernelGGL(k_m2l_sym_near<RT>, dim3((unsigned)(nw + nn)), dim3(256), 0, s, o, nw, op->d_swork.p, op->d_spartner.p, \
                       op->d_src.p, op->d_spart.p, v, na, nn - na, x, op->d_cpart.p)
    switch (op->sym_rt) {
        case 1: IGE_MSN(1); break;
        case 2: IGE_MSN(2); break;
        case 3: IGE_MSN(3); break;
        default: IGE_MSN(4); break;
    }
#undef IGE_MSN
    IGE_HIP(hipGetLastError());
}

void launch_m2l_reduce_sym(ige_op op)
{
    const DevOp &o = op->view;
    // up to four threads per value where a list is long
    const int64_t len = ((int64_t)op->swork.size() + (int64_t)op->d_spartner.n) / std::max(1, op->NC);
    int S = 1;
    const int G = std::min(512, (4 * o.Q + 63) / 64 * 64);
    while (S < 4 && len > 8 * S && 2 * S * G <= 1024) S *= 2;
    const int nt = S * G;
    const size_t shm = sizeof(double2) * 4 * o.Q * S;
    hipLaunchKernelGGL(k_m2l_reduce_sym, dim3(op->NC), dim3(nt), shm, lstream(op), o, S, op->d_sred_ptr.p, op->d_sred_idx.p,
                       op->d_spart.p, op->d_loc.p);
    IGE_HIP(hipGetLastError());
}

}  // namespace ige
