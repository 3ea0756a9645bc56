// fdirw_balance.h -- Eq. 7's far-field balance from per-workgroup partial sums
// (arXiv 2408.11376), run by one workgroup of BALANCE_NT threads: as a launch of
// its own (fdirw_mp.hip) or beside the next step's mapping (fdirw_coarse.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "fdirw_launch.h"

namespace fdirw {

constexpr int BALANCE_NT = 256;

// Block-wide fixed-order tree sum of two values (every thread gets them), in
// the caller's LDS scratch (2 x BALANCE_NT doubles).
__device__ inline void mp_block_sum2_in(double &a, double &b, double *sa, double *sb)
{
    __syncthreads();
    sa[threadIdx.x] = a;
    sb[threadIdx.x] = b;
    __syncthreads();
    for (int w = BALANCE_NT / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            sa[threadIdx.x] += sa[threadIdx.x + w];
            sb[threadIdx.x] += sb[threadIdx.x + w];
        }
        __syncthreads();
    }
    a = sa[0];
    b = sb[0];
}

// Q_L in part[0 .. nblk), Q_S in part[nblk .. 2 nblk): the partials in workgroup
// order, then c_ff = (M_total - Q_L - Q_S) / V_ff into *cff and the history row.
// sa, sb: BALANCE_NT doubles of LDS each.
__device__ __forceinline__ void balance_finish(const BalanceArgs &b, double *sa, double *sb)
{
    double ql = 0.0, qs = 0.0;
    for (int k = threadIdx.x; k < b.nblk; k += BALANCE_NT) {
        ql += b.part[k];
        qs += b.part[b.nblk + k];
    }
    mp_block_sum2_in(ql, qs, sa, sb);
    if (threadIdx.x == 0) {
        const double v = (b.m_total - ql - qs) / b.v_ff;
        b.cff[0] = v;
        if (b.hist_row) {
            b.hist_row[0] = ql;
            b.hist_row[1] = qs;
            b.hist_row[2] = v;
        }
    }
}

}  // namespace fdirw
