// One work item of the near-field product over the distinct entries.  Bound by HBM alone, but
// its waves share the SIMDs with the coupling, so what it issues counts: whole rows are loaded
// without a test per lane (only a diagonal square needs one), row addresses are scalar, and the
// row sums take two half-wave and row exchanges and four rotations instead of shuffles through
// shared memory: 122 instructions per two rows of 192 columns, 238 before.  Level 5, 318 MB: 72.5
// us alone before, 67 now (4.75 TB/s).
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "device_math.hpp"
#include "op.hpp"

namespace ige {
namespace {

typedef double d2v __attribute__((ext_vector_type(2)));

// streaming load of one complex entry (not kept in the caches)
__device__ inline d2v ld_once(const double2 *B, size_t i)
{
    return __builtin_nontemporal_load(reinterpret_cast<const d2v *>(B) + i);
}

// ---------------------------------------------------------------------------
// a8, once per distinct entry: a workgroup streams rows [r0, r1) of one dense
// rectangle of the symmetric near-field matrix (rows and columns are lists of glued
// unknowns); each row gives its row sum (B x_cols)[r] and the same loads give the
// column sums of B^T x_rows.  A diagonal square is read in its upper triangle only:
// row r takes the columns c >= r for its row sum and c > r for the column sums.
// ---------------------------------------------------------------------------
constexpr int kCmpRows = 128;   // largest rows per work item (host: rows_per_item)

template <int U, int RS, int PRIO>
__device__ __forceinline__ void near_cmp_item(const NearCmpView &v, int w, const double2 *x, double2 *part,
                                              double2 *sxr, double2 (*syc)[256])
{
    // wave-uniform indices in scalar registers: the entry loads are then a scalar row address
    // plus the lane's column
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int4 it = v.work[w];
    const int k = it.x, r0 = it.y, r1 = it.z;
    const int nr = v.nr[k], nc = v.nc[k], ld = v.ld[k];
    const bool sym = v.sym[k] != 0;
    const int32_t *rows = v.idx + v.lst[k], *cols = rows + nr;
    const double2 *B = v.val + v.val_off[k];
    double *rout = reinterpret_cast<double *>(part + v.wpart[w]);
    d2v xc[U], yc[U];
    int cl[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int c = lane + 64 * u;
        cl[u] = min(c, nc - 1);   // lanes without a column read the last one against x = 0
        const double2 xv = c < nc ? x[cols[c]] : make_double2(0.0, 0.0);
        xc[u] = d2v{xv.x, xv.y};
        yc[u] = d2v{0.0, 0.0};
    }
    for (int q = threadIdx.x; q < r1 - r0; q += blockDim.x) sxr[q] = x[rows[r0 + q]];
    __syncthreads();
    if constexpr (PRIO > 0) __builtin_amdgcn_s_setprio(PRIO);
    auto step = [&](auto symc, int r) {
        constexpr bool SYM = decltype(symc)::value;
        d2v al[RS][U];
        double2 xq[RS];
        double re[RS], im[RS];
#pragma unroll
        for (int q = 0; q < RS; ++q) {
            const int rq = r + 4 * q, rc = min(rq, r1 - 1);   // beyond the last row: that row against x = 0
            const double2 *Br = B + (size_t)rc * ld;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if constexpr (SYM) al[q][u] = cl[u] >= rc ? ld_once(Br, cl[u]) : d2v{0.0, 0.0};
                else al[q][u] = ld_once(Br, cl[u]);
            }
            xq[q] = rq < r1 ? sxr[rc - r0] : make_double2(0.0, 0.0);
            re[q] = 0.0;
            im[q] = 0.0;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int q = 0; q < RS; ++q) {
                const d2v a = al[q][u];
                re[q] = fma(a.x, xc[u].x, fma(-a.y, xc[u].y, re[q]));
                im[q] = fma(a.x, xc[u].y, fma(a.y, xc[u].x, im[q]));
            }
#pragma unroll
            for (int q = 0; q < RS; ++q) {
                // the diagonal entry of a square counts once (row sum only)
                d2v a = al[q][u];
                if constexpr (SYM)
                    if (lane + 64 * u == r + 4 * q) a = d2v{0.0, 0.0};
                yc[u].x = fma(a.x, xq[q].x, fma(-a.y, xq[q].y, yc[u].x));
                yc[u].y = fma(a.x, xq[q].y, fma(a.y, xq[q].x, yc[u].y));
            }
        }
        // row sums over the lanes, two rows (four values) at a time: halves and 16-lane rows
        // exchanged between two values (each then holds half the lanes' sums of both), then
        // rotations inside the 16 lanes.  Lane row 0: re, 1: re of the second row, 2: im, 3: its im
#pragma unroll
        for (int q = 0; q < RS; q += 2) {
            double t = dm::swap16_add(dm::swap32_add(re[q], im[q]), dm::swap32_add(re[q + 1], im[q + 1]));
            t += dm::row_ror<8>(t);
            t += dm::row_ror<4>(t);
            t += dm::row_ror<2>(t);
            t += dm::row_ror<1>(t);
            const int rq = r + 4 * (q + ((lane >> 4) & 1));
            if ((lane & 15) == 0 && rq < r1) rout[2 * (rq - r0) + (lane >> 5)] = t;
        }
    };
    if (sym)
        for (int r = r0 + wv; r < r1; r += 4 * RS) step(std::true_type{}, r);
    else
        for (int r = r0 + wv; r < r1; r += 4 * RS) step(std::false_type{}, r);
    if (wv > 0)
#pragma unroll
        for (int u = 0; u < U; ++u) syc[wv - 1][lane + 64 * u] = make_double2(yc[u].x, yc[u].y);
    __syncthreads();
    if (wv == 0) {
        double2 *cp = part + v.wpart[w] + (r1 - r0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int c = lane + 64 * u;
            if (c < nc) {
                const double2 s1 = syc[0][c], s2 = syc[1][c], s3 = syc[2][c];
                cp[c] = make_double2(((yc[u].x + s1.x) + s2.x) + s3.x, ((yc[u].y + s1.y) + s2.y) + s3.y);
            }
        }
    }
}

}  // namespace
}  // namespace ige
