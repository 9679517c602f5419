// Pieces that the steps on declared or found lattices (fused.hip, brick.hip,
// longrange.hip) share: the record of a replica from its work items' sums,
// and, for the plane march, the record terms, predictor and corrector of one
// site of a uniform material with scalar exchange.
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
// the applied field out (record_terms), and it is added here.
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

// m and E terms of one site: S and S.H_ex/2 + (k_u/mu_s)(S.e)^2, with se =
// S.e as the predictor forms it (-E_i/mu_s is that plus S.H_app, which the
// record adds from the summed spins).  A replica takes these steps only
// with one material, so mu_s is the reference moment and every site weighs
// 1.  Written with explicit fmas so that the step and the measuring launch
// round alike.
template <typename R>
__device__ __forceinline__ void record_terms(const MaterialDev<R>& m, const V3<R>& s, R se, const V3<R>& hex, R t[4])
{
    const R sh = fma(s.z, hex.z, fma(s.y, hex.y, s.x * hex.x));
    t[0] = s.x;
    t[1] = s.y;
    t[2] = s.z;
    t[3] = fma((R)0.5, sh, m.ku_mu * se * se);
}

// Predictor of one site from its exchange field hex and normals gn: the
// thermal plus applied field th (held for the corrector), S' = sp and
// base = S + dS dt / 2.
template <typename R>
__device__ __forceinline__ void predict_site(const ReplicaDev<R>& r, const MaterialDev<R>& m, const V3<R>& e,
                                             const V3<R>& s, const V3<R>& hex, R se, const R gn[3], V3<R>& th,
                                             V3<R>& sp, V3<R>& base)
{
    const V3<R> Happ{r.H[0], r.H[1], r.H[2]};
    th = V3<R>{fma(m.sigma, gn[0], Happ.x), fma(m.sigma, gn[1], Happ.y), fma(m.sigma, gn[2], Happ.z)};
    const R as = m.ani * se;
    const V3<R> h{fma(as, e.x, hex.x) + th.x, fma(as, e.y, hex.y) + th.y, fma(as, e.z, hex.z) + th.z};
    const V3<R> ds = llg_step(s, h, r.gdt, r.alpha);
    sp = normalised(V3<R>{s.x + ds.x, s.y + ds.y, s.z + ds.z});
    base = V3<R>{s.x + (R)0.5 * ds.x, s.y + (R)0.5 * ds.y, s.z + (R)0.5 * ds.z};
}

// Corrector of one site: its S' = sp, the exchange field hc at S' and what
// the predictor held.
template <typename R>
__device__ __forceinline__ V3<R> correct_site(const ReplicaDev<R>& r, const MaterialDev<R>& m, const V3<R>& e,
                                              const V3<R>& sp, const V3<R>& hc, const V3<R>& th, const V3<R>& base)
{
    const R as = m.ani * dot(sp, e);
    const V3<R> h{fma(as, e.x, hc.x) + th.x, fma(as, e.y, hc.y) + th.y, fma(as, e.z, hc.z) + th.z};
    // half the step's dS' dt (a step of dt / 2: the halving is exact)
    const V3<R> dsh = llg_step(sp, h, (R)0.5 * r.gdt, r.alpha);
    return normalised(V3<R>{base.x + dsh.x, base.y + dsh.y, base.z + dsh.z});
}

}  // namespace dev
}  // namespace sllg
