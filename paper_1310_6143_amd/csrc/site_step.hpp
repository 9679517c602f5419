// What the steps on declared or found lattices (fused.hip, brick.hip,
// longrange.hip) share: the record of a replica from its work items' sums.
#pragma once

#include "device_common.hpp"

namespace sllg {
namespace dev {

// Sum of four values over the first 256 threads (fixed order: per wave, then
// the four waves in turn); result valid in thread 0.  Every thread of the
// block calls it.
template <int BT>
__device__ __forceinline__ void sum4_256(const double v[4], double out[4], double (*red)[BT / 64])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const double s = wave_sum(threadIdx.x < 256 ? v[c] : 0.0);
        if (lane == 0 && wave < 4)
            red[c][wave] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int c = 0; c < 4; ++c)
            out[c] = ((red[c][0] + red[c][1]) + red[c][2]) + red[c][3];
    __syncthreads();
}

// Record `slot` of replica r from its items' sums of parity `par`: thread t
// < 256 adds items t, t + 256, ... in order, then the fixed 256-lane sum.
// The same order whichever kernel runs it.  ZEEMAN: the items' energies leave
// the applied field out (record_terms in fused.hip), and it is added here.
template <typename R, int BT, bool ZEEMAN>
__device__ void item_record(const ReplicaDev<R>& r, int par, int64_t slot, double (*red)[BT / 64])
{
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    const double* p = r.f_partials + 4 * (int64_t)par * r.f_items;
    if (threadIdx.x < 256)
        for (int q = (int)threadIdx.x; q < r.f_items; q += 256) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                v[c] += p[4 * (int64_t)q + c];
        }
    double tot[4];
    sum4_256<BT>(v, tot, red);
    if (threadIdx.x == 0) {
        double* out = r.records + 4 * (r.rec_pos + slot);
        const double f = r.mu_ref * r.inv_mu_total;
        out[0] = tot[0] * f;
        out[1] = tot[1] * f;
        out[2] = tot[2] * f;
        // the Zeeman part from the summed spins: S.H_app summed over the
        // sites is H_app.(sum of S)
        const double zee = (double)r.H[0] * tot[0] + (double)r.H[1] * tot[1] + (double)r.H[2] * tot[2];
        out[3] = -r.mu_ref * (ZEEMAN ? tot[3] + zee : tot[3]);
    }
}

}  // namespace dev
}  // namespace sllg
