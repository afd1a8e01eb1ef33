// a5 for several FP64 columns: the coupling with kernel values evaluated in place as the
// operand of the 16x16x4 FP64 matrix instruction.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_math.hpp"
#include "op.hpp"

namespace ige {

namespace {

typedef double dx4 __attribute__((ext_vector_type(4)));

// One workgroup per work item (cluster t, up to 8 or 32 partners) and column chunk; wave w takes the
// rows 16 w .. 16 w + 15 of t.  In a step a wave evaluates 16 rows x 4 nodes of G, one value per
// lane, which is the A operand as it stands; a tile of the B operand holds 8 complex columns as
// [Re V | Im V] against Re G and [-Im V | Re V] against Im G, so the accumulators are [Re U | Im U].
// The complex columns of a chunk are the fields (EFIE 4; scalar: only the fourth, the others are
// zero) times its right-hand sides.  Nodes and fields of KC source nodes at a time are staged
// in shared memory (Re, Im and -Im planes, so a lane reads its operand without arithmetic),
// double-buffered through registers.
// Bound by FP64 issue (matrix instructions and vector FP64 do not overlap here): 150 cycles for
// the value, 64 per instruction, two per 8 columns.  The form with one (row, node range) per
// lane took its fields from shared memory for 3 rows at a time and spent 4 fields on the
// scalar operator; the one with stored blocks padded 2 Q to multiples of 32 on both sides and
// the columns to 64 or 128.
// Level 6, 27,912 ordered pairs of 81 nodes, 64 columns: 10.7 ms from stored blocks, 9.2 now (50
// TFLOP/s of matrix instructions); torus level 4, 26,848 pairs of 49 nodes, 23 columns: 2.66 and
// 1.40 ms beside the near field; scalar, sphere level 4, 64 nodes, 5 columns: 504 us evaluated before, 88 now.
template <int NT, int KC, int KS>
__global__ __launch_bounds__(KS > 1 ? 768 : 1024) void k_m2l_gen(DevOp o, int r, int rc, int nf, const M2LWork *work, const int32_t *partner,
                                                  const double2 *src, double2 *part)
{
    constexpr int NC = 8 * NT;               // complex columns of the chunk
    constexpr int PS = NC + 8, NS = 3 * PS + (NT == 8 ? 0 : 8);   // doubles from plane to plane, from node to node (bank spread)
    constexpr int G = 2;                     // steps in one phase
    __shared__ double2 sTab[256];
    __shared__ double sV[2][KC * NS];
    __shared__ double sX[2][3 * KC];
    const M2LWork wk = work[blockIdx.x];
    const int Qs = o.Q, tid = threadIdx.x, nth = blockDim.x, lane = tid & 63;
    // the waves of the first half of the steps, then those of the second: every SIMD gets both
    const int nrow = nth / (64 * KS), wv = __builtin_amdgcn_readfirstlane((tid >> 6) % nrow);
    const int ks = __builtin_amdgcn_readfirstlane((tid >> 6) / nrow);
    const int c0 = blockIdx.y * rc, nc = min(rc, r - c0), f0 = 4 - nf, ncol = nf * rc;
    int lvl = 0;
    while (lvl < o.L && wk.tgt >= o.lvl_off[lvl + 1]) ++lvl;
    const int Q = (o.ql[lvl] + 1) * (o.ql[lvl] + 1), nck = (Q + KC - 1) / KC, nst = (wk.end - wk.beg) * nck;
    for (int i = tid; i < 256; i += nth) sTab[i] = o.sctab[i];
    const double kap = o.kappa;
    const int n = lane & 15, hi = lane >> 4, row = min(Q - 1, 16 * wv + n);
    const bool rows = 16 * wv < Q;   // wave-uniform: levels of a smaller degree leave waves without rows
    const double *Xt = o.nodeX + (size_t)wk.tgt * 3 * Qs;
    const double x0 = Xt[row], x1 = Xt[Qs + row], x2 = Xt[2 * Qs + row];
    // operand offsets of this lane: Re | Im against Re G, -Im | Re against Im G
    const int ob1 = (n < 8 ? 0 : PS) + (n & 7), ob2 = (n < 8 ? 2 * PS : 0) + (n & 7);
    dx4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = dx4{0.0, 0.0, 0.0, 0.0};
    // stage st: nodes [k0, k0 + KC) of a partner (values beyond the cluster zero, nodes clamped).
    // fetch puts a thread's first PF values under way into registers, commit writes them and
    // whatever a small workgroup has beyond them; where a value comes from and goes to does not
    // change from stage to stage
    constexpr int PF = KS > 1 ? 3 : 4, BIG = 1 << 28;
    auto origin = [&](int i, int &go, int &m) {   // offset in the cluster's fields, node in the stage
        const int j = i % NC, f = j / rc, c = j - f * rc;
        m = i / NC;
        go = ((f0 + f) * Qs + m) * r + c0 + c;
        if (i >= KC * NC || j >= ncol || c >= nc) m = BIG;
    };
    int go[PF], mo[PF];
#pragma unroll
    for (int k = 0; k < PF; ++k) origin(tid + k * nth, go[k], mo[k]);
    double2 pv[PF];
    double px = 0.0;
    const double *xsrc = o.nodeX + (size_t)(tid / KC) * Qs;
    auto put = [&](int b, int i, double2 v) {
        double *d = &sV[b][i / NC * NS + i % NC];
        d[0] = v.x;
        d[PS] = v.y;
        d[2 * PS] = -v.y;
    };
    auto fetch = [&](int sc, int k0) {
        const double2 *Vs = src + ((size_t)sc * 4 * Qs + k0) * r;
#pragma unroll
        for (int k = 0; k < PF; ++k) pv[k] = k0 + mo[k] < Q ? Vs[go[k]] : make_double2(0.0, 0.0);
        if (tid < 3 * KC) px = xsrc[(size_t)sc * 3 * Qs + min(Q - 1, k0 + tid % KC)];
    };
    auto commit = [&](int sc, int k0, int b) {
#pragma unroll
        for (int k = 0; k < PF; ++k)
            if (tid + k * nth < KC * NC) put(b, tid + k * nth, pv[k]);
        if (tid < 3 * KC) sX[b][tid] = px;
        if (PF * nth < KC * NC) {
            const double2 *Vs = src + ((size_t)sc * 4 * Qs + k0) * r;
            for (int i = tid + PF * nth; i < KC * NC; i += nth) {
                int g, m;
                origin(i, g, m);
                put(b, i, k0 + m < Q ? Vs[g] : make_double2(0.0, 0.0));
            }
        }
        for (int i = tid + nth; i < 3 * KC; i += nth) sX[b][i] = o.nodeX[((size_t)sc * 3 + i / KC) * Qs + min(Q - 1, k0 + i % KC)];
    };
    int kp = wk.beg, k0 = 0;   // partner and first node of the stage
    fetch(partner[kp], 0);
    commit(partner[kp], 0, 0);
    __syncthreads();
    for (int st = 0; st < nst; ++st) {
        const int b = st & 1, ng = (min(KC, Q - k0) + 3) / 4;
        k0 += KC;
        if (k0 >= Q) {
            k0 = 0;
            ++kp;
        }
        if (st + 1 < nst) fetch(partner[kp], k0);
        if (rows)
            for (int g0 = ks; g0 < ng; g0 += G * KS) {
                const bool two = g0 + KS < ng;   // uniform
                double ir[G], cc[G], ss[G];
                double2 cs[G];
#pragma unroll
                for (int k = 0; k < G; ++k) {
                    if (k == 1 && !two) break;
                    const int m = 4 * (g0 + KS * k) + hi;
                    const double d0 = x0 - sX[b][m], d1 = x1 - sX[b][KC + m], d2 = x2 - sX[b][2 * KC + m];
                    dm::helmholtz_tab_begin(kap, fma(d0, d0, fma(d1, d1, d2 * d2)), sTab, ir[k], cc[k], ss[k], cs[k]);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < G; ++k) {
                    if (k == 1 && !two) break;
                    const double2 Gv = dm::helmholtz_tab_end(ir[k], cc[k], ss[k], cs[k]);
                    const double *Vm = &sV[b][(4 * (g0 + KS * k) + hi) * NS];
#pragma unroll
                    for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(Gv.x, Vm[ob1 + 8 * t], acc[t], 0, 0, 0);
#pragma unroll
                    for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(Gv.y, Vm[ob2 + 8 * t], acc[t], 0, 0, 0);
                }
            }
        if (st + 1 < nst) commit(partner[kp], k0, b ^ 1);   // that buffer was last read before the previous barrier
        __syncthreads();
    }
    if constexpr (KS > 1) {   // the waves that share rows, as many column tiles at a time as fit
        double *red = &sV[0][0];
        const int tr = min(NT, (int)(2 * KC * NS / (nrow * 256)));
        for (int t0 = 0; t0 < NT; t0 += tr) {
            if (ks == 1)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    if (t >= t0 && t < t0 + tr)
#pragma unroll
                        for (int j = 0; j < 4; ++j) red[((wv * tr + t - t0) * 4 + j) * 64 + lane] = acc[t][j];
            __syncthreads();
            if (ks == 0)
#pragma unroll
                for (int t = 0; t < NT; ++t)
                    if (t >= t0 && t < t0 + tr)
#pragma unroll
                        for (int j = 0; j < 4; ++j) acc[t][j] += red[((wv * tr + t - t0) * 4 + j) * 64 + lane];
            __syncthreads();
        }
        if (ks != 0) return;
    }
    // lane: column n, rows lane / 16 + 4 j; the imaginary parts come over to the lanes of the real ones
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double re = acc[t][j], im = dm::row_ror<8>(re);
            const int mm = 16 * wv + hi + 4 * j, cj = 8 * t + n, f = cj / rc, c = cj - f * rc;
            if (n < 8 && mm < Q && cj < ncol && c < nc)
                part[(((size_t)blockIdx.x * 4 + f0 + f) * Qs + mm) * r + c0 + c] = make_double2(re, im);
        }
}

}  // namespace

// Items of up to 32 partners instead of 8 where they still give each CU eight workgroups: a
// quarter of the starts, ends and partial results (level 6, 64 columns: the sum of the partials
// 412 us with 8, 137 with 32)
bool m2l_gen_long(const ige_op_s *op, int r)
{
    const int nf = op->view.scalar ? 1 : 4;
    return op->mwork.size() * (size_t)((nf * r + 63) / 64) >= 8 * 256;
}

// partials of r columns per work item into d_bpart (scalar: field 3 only; the others are not read)
void m2l_generate(ige_op op, int r, const double2 *src, hipStream_t s)
{
    const DevOp &o = op->view;
    const int nf = o.scalar ? 1 : 4;
    // chunks of at most 64 complex columns, of equal numbers of right-hand sides
    const int nchunk = (nf * r + 63) / 64, rc = (r + nchunk - 1) / nchunk, nt = (nf * rc + 7) / 8;
    int Q = 1;
    for (int lvl = std::max(0, op->lfar); lvl <= o.L; ++lvl) Q = std::max(Q, (o.ql[lvl] + 1) * (o.ql[lvl] + 1));
    // two waves per row tile where that makes the waves a multiple of the four SIMDs (degrees 4 and
    // 8): the workgroups' waves then load every SIMD alike
    const int nrow = (Q + 15) / 16, ks = nrow == 2 || nrow == 6 ? 2 : 1;
    const bool lng = m2l_gen_long(op, r);
    const size_t items = lng ? op->mwork.size() : op->work.size();
    IGE_REQUIRE(op->d_bpart.n >= items * 4 * (size_t)o.Q * r, "coupling partials too small");
    const auto *work = lng ? op->d_mwork.p : op->d_work.p;
    const int32_t *partner = lng ? op->d_mpartner.p : op->d_partner.p;
    const dim3 grid((unsigned)items, (unsigned)((r + rc - 1) / rc)), blk(64 * nrow * ks);
#define IGE_MG(NT, KC, KS) \
    hipLaunchKernelGGL((k_m2l_gen<NT, KC, KS>), grid, blk, 0, s, o, r, rc, nf, work, partner, src, op->d_bpart.p)
#define IGE_MGK(NT) \
    if (ks == 2) IGE_MG(NT, 32, 2); \
    else IGE_MG(NT, (NT <= 2 ? 32 : 16), 1)
    switch (nt) {
        case 1: IGE_MGK(1); break;
        case 2: IGE_MGK(2); break;
        case 3: IGE_MGK(3); break;
        case 4: IGE_MGK(4); break;
        case 5: IGE_MGK(5); break;
        case 6: IGE_MGK(6); break;
        case 7: IGE_MGK(7); break;
        default: IGE_MGK(8); break;
    }
#undef IGE_MGK
#undef IGE_MG
    IGE_HIP(hipGetLastError());
}

}  // namespace ige
