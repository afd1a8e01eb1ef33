// Near-field product of several FP64 columns over ordered leaf pairs on the FP64 matrix
// cores, from the stored unordered blocks.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_math.hpp"
#include "op.hpp"

namespace ige {

namespace {

typedef double dx4 __attribute__((ext_vector_type(4)));

// A workgroup takes a target leaf t with some of its near leaves (work item) and a chunk of
// columns; the sums over the partners stay in registers, so only the items' sums are written and
// added per unknown.  Wave w takes the rows 16 w .. 16 w + 15 of t.  A block is read as it is stored, one complex value per lane, which
// is the A operand of the 16x16x4 instruction for both parts: B[row][k] where t is its row leaf,
// B[k][row] where it is its column leaf (the operator is symmetric), loaded a few steps ahead.  A
// B operand tile holds 8 complex columns as [Re X | Im X] against Re B and [-Im X | Re X] against
// Im B; the partner's columns are gathered 32 slots at a time into shared memory (Re, Im and -Im
// planes), double-buffered through registers.
// Up to about 16 columns bound by reading each block twice (level 5, 516 MB of unordered blocks,
// 180 slots, 8 columns: 192 us = 5.4 TB/s; with one partial result per block, row and column, two
// products per block and 16 columns' worth of matrix instructions 349 us), beyond by the matrix
// instructions (level 6, 64 columns, 132 GFLOP: 2.70 ms = 49 TFLOP/s; from blocks padded to 32
// slots, split into parts and stored per ordered pair 4.5 ms, 2.1 GB more).  Scalar level 4, 36
// slots, 5 columns: 22 us (54 in an earlier form), 138 with the unordered blocks in passes of 4 columns.
// Contiguous items per XCD measured slower (level 6, 64 columns 2.90 ms against 2.70), 4x4x4
// instructions for up to 6 columns no faster.
// UG: steps of four slots loaded ahead
template <int NT, int UG, int WPE>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(WPE))) void k_near_cols(int nF, int r, int rc, const int32_t *order, const M2LWork *work,
                                                    const int32_t *partner, const int32_t *aslot, const int32_t *leafdof,
                                                    const double2 *bval, const double2 *xt, double2 *part)
{
    constexpr int KC = NT >= 4 ? 16 : 32, NC = 8 * NT;
    constexpr int PS = NC + 8, NS = 3 * PS + (NT == 8 ? 0 : 8);   // doubles from plane to plane, from slot to slot (bank spread)
    constexpr int PF = 4;
    __shared__ double sV[2][KC * NS];
    const int wi = order[blockIdx.x];
    const M2LWork wk = work[wi];
    const int tid = threadIdx.x, nth = blockDim.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int c0 = blockIdx.y * rc, nc = min(rc, r - c0), n = lane & 15, hi = lane >> 4;
    const int rt = 16 * (blockIdx.z * 16 + wv), row = min(nF - 1, rt + n);
    const int ob1 = (n < 8 ? 0 : PS) + (n & 7), ob2 = (n < 8 ? 2 * PS : 0) + (n & 7);
    dx4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = dx4{0.0, 0.0, 0.0, 0.0};
    double2 a[UG], an[UG], pv[PF];
    // the entries of the wave's steps j0 .. j0 + UG - 1 of a stage (slots from k0 of partner kp)
    auto entries = [&](int kp, int k0, int j0, double2 (&d)[UG]) {
        const int sl = aslot[kp];
        const double2 *B = bval + (size_t)(sl >> 1) * nF * nF;
        const int sr = (sl & 1) ? 1 : nF, sc = (sl & 1) ? nF : 1;
        const double2 *Br = B + (size_t)row * sr;
#pragma unroll
        for (int u = 0; u < UG; ++u) d[u] = Br[(size_t)min(nF - 1, k0 + 4 * (j0 + u) + hi) * sc];
    };
    auto value = [&](int sc, int k0, int i) {
        const int j = i % NC, k = k0 + i / NC;
        const int d = (j < nc && k < nF) ? leafdof[(size_t)sc * nF + k] : -1;
        return d >= 0 ? xt[(size_t)d * r + c0 + j] : make_double2(0.0, 0.0);
    };
    auto put = [&](int b, int i, double2 v) {
        double *d = &sV[b][i / NC * NS + i % NC];
        d[0] = v.x;
        d[PS] = v.y;
        d[2 * PS] = -v.y;
    };
    auto fetch = [&](int sc, int k0) {
#pragma unroll
        for (int k = 0; k < PF; ++k)
            if (tid + k * nth < KC * NC) pv[k] = value(sc, k0, tid + k * nth);
    };
    auto commit = [&](int sc, int k0, int b) {
#pragma unroll
        for (int k = 0; k < PF; ++k)
            if (tid + k * nth < KC * NC) put(b, tid + k * nth, pv[k]);
        for (int i = tid + PF * nth; i < KC * NC; i += nth) put(b, i, value(sc, k0, i));
    };
    int kp = wk.beg, k0 = 0;
    entries(kp, 0, 0, an);
    fetch(partner[kp], 0);
    commit(partner[kp], 0, 0);
    __syncthreads();
    const int nst = (wk.end - wk.beg) * ((nF + KC - 1) / KC);
    for (int st = 0; st < nst; ++st) {
        const int b = st & 1, ng = (min(KC, nF - k0) + 3) / 4;
        int kn = k0 + KC, kpn = kp;   // the next stage
        if (kn >= nF) {
            kn = 0;
            ++kpn;
        }
        const bool more = st + 1 < nst;
        if (more) fetch(partner[kpn], kn);
        for (int j0 = 0; j0 < ng; j0 += UG) {
#pragma unroll
            for (int u = 0; u < UG; ++u) a[u] = an[u];
            if (j0 + UG < ng) entries(kp, k0, j0 + UG, an);
            else if (more) entries(kpn, kn, 0, an);
#pragma unroll
            for (int u = 0; u < UG; ++u) {
                if (j0 + u >= ng) break;   // uniform
                const double *Vm = &sV[b][(4 * (j0 + u) + hi) * NS];
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].x, Vm[ob1 + 8 * t], acc[t], 0, 0, 0);
#pragma unroll
                for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u].y, Vm[ob2 + 8 * t], acc[t], 0, 0, 0);
            }
        }
        if (more) commit(partner[kpn], kn, b ^ 1);   // that buffer was last read before the previous barrier
        kp = kpn;
        k0 = kn;
        __syncthreads();
    }
    // lane: column lane % 16, rows lane / 16 + 4 j; the imaginary parts come over to the lanes of the real ones
    double2 *out = part + (size_t)wi * nF * r + c0;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const double re = acc[t][j], im = dm::row_ror<8>(re);
            const int m = rt + hi + 4 * j, c = 8 * t + n;
            if (n < 8 && m < nF && c < nc) out[(size_t)m * r + c] = make_double2(re, im);
        }
}

// yt[i][c] = sum of the item sums of unknown i: S threads per (unknown, column) take every S-th
// one, eight loads at a time, and are added in order
__global__ __launch_bounds__(256) void k_near_cols_sum(int64_t N, int r, int S, const int64_t *ptr, const int32_t *idx,
                                                       const double2 *part, double2 *yt)
{
    __shared__ double2 sh[256];
    const int per = blockDim.x / S, j = threadIdx.x % per, q = threadIdx.x / per;
    const int64_t t = (int64_t)blockIdx.x * per + j;
    double re = 0.0, im = 0.0;
    if (t < N * r) {
        const int64_t i = t / r, e = ptr[i + 1];
        const int c = (int)(t % r);
        for (int64_t k0 = ptr[i] + q; k0 < e; k0 += 8 * S) {
            double2 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = k0 + u * S < e ? part[(size_t)idx[k0 + u * S] * r + c] : make_double2(0.0, 0.0);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (k0 + u * S < e) {
                    re += v[u].x;
                    im += v[u].y;
                }
        }
    }
    if (S > 1) {
        sh[threadIdx.x] = make_double2(re, im);
        __syncthreads();
        for (int s = 1; s < S && q == 0; ++s) {
            re += sh[s * per + j].x;
            im += sh[s * per + j].y;
        }
    }
    if (q == 0 && t < N * r) yt[t] = make_double2(re, im);
}

}  // namespace

// Several columns, except where the unordered-block kernel takes all of them in one pass over
// large leaves: it reads half the bytes and uses the vector units beside the coupling's matrix
// instructions (level 6, 180 slots per leaf, 4 columns: 1,650 us per apply with it, 1,735 here; 6
// columns: 3,144 and 2,009; level 4, 4 columns: 101 and 107, 8 columns: 157 and 131; 84 slots, 4
// columns: 351 and 314).  The line lies where the blocks of level 6 put it; with the same 180
// slots at level 5, 3 columns, it is 3 % off (437 with the unordered blocks, 422 here).
bool near_cols_use(const ige_op_s *op, int r)
{
    const int nF = op->view.nF;
    if (r < 2 || op->nb_nwork == 0 || op->near_blocks) return false;
    return nF <= 128 || r > (nF <= 256 ? 4 : 2);
}

void near_cols(ige_op op, int r, const double2 *xt, double2 *yt, hipStream_t s)
{
    const DevOp &o = op->view;
    const int ntile = (o.nF + 15) / 16, nrow = std::min(16, ntile);
    // the list of short items where there is one
    const bool fine = op->d_nfwork.n > 0;
    const int64_t nw = fine ? (int64_t)op->d_nfwork.n : op->nb_nwork;
    // Up to 64 columns per workgroup (level 6, 64 columns: 2.7 ms); fewer where that leaves under two
    // waves per SIMD (level 3, 64 columns: 86 us with 64, 61 with 32, 53 with 16).
    int cols = 64;
    while (cols > 16 && nw * nrow * ((r + cols - 1) / cols) < 2048) cols /= 2;
    const int nchunk = (r + cols - 1) / cols, rc = (r + nchunk - 1) / nchunk, nt = (rc + 7) / 8;
    const size_t pn = (size_t)nw * o.nF * r;
    if (op->d_ndpart.n < pn) op->d_ndpart.alloc(pn);
    const int32_t *order = fine ? op->d_nforder.p : op->d_nborder.p;
    const M2LWork *work = fine ? op->d_nfwork.p : op->d_nbwork.p;
    const dim3 grid((unsigned)nw, (unsigned)((r + rc - 1) / rc), (unsigned)((ntile + 15) / 16)), blk(64 * nrow);
#define IGE_NC(NT, UU, WW) \
    hipLaunchKernelGGL((k_near_cols<NT, UU, WW>), grid, blk, 0, s, o.nF, r, rc, order, work, op->d_nbpartner.p, op->d_nbslot.p, \
                       o.leafdof, o.bval, xt, op->d_ndpart.p)
    // Two steps loaded ahead in 79 registers, or four in 103: alone the first is as fast or faster
    // (level 4, 84 slots, 4 columns: 70 us against 78), but with the large leaves of many waves it
    // leaves no room on a CU for the coupling's (level 6, 180 slots, 6 columns: 2,089 us against 2,009).
    if (nt == 1 && nrow <= 8) { IGE_NC(1, 2, 5); }
    else switch (nt) {
        case 1: IGE_NC(1, 4, 4); break;
        case 2: IGE_NC(2, 4, 4); break;
        case 3: IGE_NC(3, 4, 4); break;
        case 4: IGE_NC(4, 2, 4); break;
        case 5: IGE_NC(5, 2, 4); break;
        case 6: IGE_NC(6, 2, 4); break;
        case 7: IGE_NC(7, 2, 4); break;
        default: IGE_NC(8, 2, 4); break;
    }
#undef IGE_NC
    IGE_HIP(hipGetLastError());
    // one thread per four item sums of an unknown, up to eight
    const int64_t tot = (int64_t)o.N * r;
    const DBuf<int32_t> &ridx = fine ? op->d_nfred_idx : op->d_nbred_idx;
    int S = 1;
    while (S < 8 && (int64_t)ridx.n > 8 * S * (int64_t)o.N) S *= 2;
    const int per = 256 / S;
    hipLaunchKernelGGL(k_near_cols_sum, dim3((unsigned)((tot + per - 1) / per)), dim3(256), 0, s, (int64_t)o.N, r, S,
                       fine ? op->d_nfred_ptr.p : op->d_nbred_ptr.p, ridx.p, op->d_ndpart.p, yt);
    IGE_HIP(hipGetLastError());
}

}  // namespace ige
