// Near-field product of one column over the distinct entries of the symmetric
// near-field matrix (Sec. 4.2: the non-admissible blocks carry the exact Galerkin
// entries of Sec. 4.1, and the matrix is complex symmetric).  The entries are stored
// once, in dense rectangles of owner blocks (see NearCompact in setup.hpp); the
// values are summed at assembly from the leaf-pair blocks (k_near_merge).  The
// product writes per-rectangle row and column sums, which the fixed-order gather of
// kernels.hip adds per unknown, so the result does not depend on timing.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "near_item.hpp"
#include "op.hpp"

namespace ige {

namespace {

// Work items of at most 128 columns take two column groups of 64 per lane; the wider
// ones U of them, in a second launch (obase: first item of the launch in the order).
template <int U, int RS, int PRIO>
__global__ __launch_bounds__(256) void k_near_cmp(NearCmpView v, int64_t obase, const double2 *x, double2 *part)
{
    __shared__ double2 sxr[kCmpRows];
    __shared__ double2 syc[3][256];
    // issue priority of these waves over others resident on the same SIMD (the
    // coupling kernel runs beside this one); a compile-time choice, so the kernel's
    // registers are those of the plain form
    near_cmp_item<U, RS, PRIO>(v, v.order[obase + blockIdx.x], x, part, sxr, syc);
}

// Both kinds of work items in one launch: the nw wide ones first (launch order
// positions na .. na + nw - 1, UW column groups per lane), then the na narrow ones
// (two column groups); one launch tail instead of two
// (at most 96 registers, five waves per SIMD: alone 73 against 76 us at 102)
template <int UW, int PRIO>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void k_near_cmp1(
    NearCmpView v, int64_t na, int64_t nw, const double2 *x, double2 *part)
{
    __shared__ double2 sxr[kCmpRows];
    __shared__ double2 syc[3][256];
    const int64_t b = blockIdx.x;
    if (b < nw) near_cmp_item<UW, 2, PRIO>(v, v.order[na + b], x, part, sxr, syc);
    else near_cmp_item<2, 2, PRIO>(v, v.order[b - nw], x, part, sxr, syc);
}

// Values of the once-per-entry near field: entry (i, j) is the sum over the leaf
// slots holding i and those holding j (ascending) of the leaf-pair block entries,
// (B_ts)[slot_t(i)][slot_s(j)] for t <= s and (B_st)[slot_s(j)][slot_t(i)] for t > s,
// for the near leaf pairs only.
__global__ __launch_bounds__(256) void k_near_merge(NearCmpView v, const double2 *bval, int nF)
{
    const int64_t k = blockIdx.x;
    const int nr = v.nr[k], nc = v.nc[k], ld = v.ld[k];
    const int32_t *rows = v.idx + v.lst[k], *cols = rows + nr;
    double2 *out = v.val + v.val_off[k];
    for (int64_t e = threadIdx.x; e < (int64_t)nr * ld; e += blockDim.x) {
        const int kr = (int)(e / ld), kc = (int)(e % ld);
        if (kc >= nc) {   // row padding
            out[e] = make_double2(0.0, 0.0);
            continue;
        }
        const int32_t i = rows[kr], j = cols[kc];
        double re = 0.0, im = 0.0;
        for (int a = v.occ_ptr[i]; a < v.occ_ptr[i + 1]; ++a) {
            const int32_t qa = v.occ[a];
            const int t = qa / nF, st = qa % nF;
            const int p0 = v.np_ptr[t], p1 = v.np_ptr[t + 1];
            for (int b = v.occ_ptr[j]; b < v.occ_ptr[j + 1]; ++b) {
                const int32_t qb = v.occ[b];
                const int sl = qb / nF, ss = qb % nF;
                int lo = p0, hi = p1;
                while (lo < hi) {
                    const int mid = (lo + hi) >> 1;
                    if (v.np_leaf[mid] < sl) lo = mid + 1;
                    else hi = mid;
                }
                if (lo < p1 && v.np_leaf[lo] == sl) {
                    const int code = v.np_code[lo];
                    const int64_t blk = code >> 1;
                    const double2 val = (code & 1) ? bval[((size_t)blk * nF + ss) * nF + st]
                                                   : bval[((size_t)blk * nF + st) * nF + ss];
                    re += val.x;
                    im += val.y;
                }
            }
        }
        out[e] = make_double2(re, im);
    }
}

}  // namespace

int near_cmp_max() { return 256; }

void launch_near_merge(ige_op op)
{
    const NearCmpView &v = op->cview;
    if (!op->cmp_on || v.nsub == 0) return;
    hipLaunchKernelGGL(k_near_merge, dim3((unsigned)v.nsub), dim3(256), 0, lstream(op), v, op->view.bval, op->view.nF);
    IGE_HIP(hipGetLastError());
}

void launch_near_once(ige_op op, const double2 *x, double2 *part, hipStream_t st)
{
    const NearCmpView &v = op->cview;
    const dim3 blk(256);
    const int64_t na = op->cmp.nnarrow, nw = v.nwork - na;
    const bool pr = op->near_prio > 0;
    if (op->near_one && op->cmp_rs == 2 && (op->cmp.maxn + 63) / 64 <= 3 && na + nw > 0) {
        const dim3 grid((unsigned)(na + nw));
        if (pr) hipLaunchKernelGGL((k_near_cmp1<3, 1>), grid, blk, 0, st, v, na, nw, x, part);
        else hipLaunchKernelGGL((k_near_cmp1<3, 0>), grid, blk, 0, st, v, na, nw, x, part);
        IGE_HIP(hipGetLastError());
        return;
    }
    if (na > 0) {
        const dim3 grid((unsigned)na);
        if (op->cmp_rs == 4) {
            if (pr) hipLaunchKernelGGL((k_near_cmp<2, 4, 1>), grid, blk, 0, st, v, (int64_t)0, x, part);
            else hipLaunchKernelGGL((k_near_cmp<2, 4, 0>), grid, blk, 0, st, v, (int64_t)0, x, part);
        } else {
            if (pr) hipLaunchKernelGGL((k_near_cmp<2, 2, 1>), grid, blk, 0, st, v, (int64_t)0, x, part);
            else hipLaunchKernelGGL((k_near_cmp<2, 2, 0>), grid, blk, 0, st, v, (int64_t)0, x, part);
        }
        IGE_HIP(hipGetLastError());
    }
    if (nw > 0) {
        const dim3 grid((unsigned)nw);
        if ((op->cmp.maxn + 63) / 64 <= 3) {
            if (pr) hipLaunchKernelGGL((k_near_cmp<3, 2, 1>), grid, blk, 0, st, v, na, x, part);
            else hipLaunchKernelGGL((k_near_cmp<3, 2, 0>), grid, blk, 0, st, v, na, x, part);
        } else {
            if (pr) hipLaunchKernelGGL((k_near_cmp<4, 2, 1>), grid, blk, 0, st, v, na, x, part);
            else hipLaunchKernelGGL((k_near_cmp<4, 2, 0>), grid, blk, 0, st, v, na, x, part);
        }
        IGE_HIP(hipGetLastError());
    }
}

}  // namespace ige
