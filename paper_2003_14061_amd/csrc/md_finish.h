// md_finish.h -- the per-system finish of an integration pass (reductions of
// section 2.3 F2, step count and history, rebuild decision), shared by the
// finish kernel and the kernels that take it over: the binning of list steps
// (k_bin_finish) and the one-workgroup cell builds.
#pragma once
#include "md_device.h"

namespace md {

// Sum partials [nb][stride] (component k) over workgroups in a fixed order,
// by one workgroup (the step's finish, or the last workgroup of k_observe,
// see last_block), reading the partials with coherent loads.  The first kT
// threads of the workgroup take the partials (strided by kT); any further
// threads add zeros, so a larger workgroup sums in the same order.
template <int kT>
__device__ __forceinline__ double finish_sum(const double* part, int nb, int stride, int k,
                                             double* red)
{
    double v[1] = {0.0};
    if ((int)threadIdx.x < kT)
        for (int b = threadIdx.x; b < nb; b += kT) v[0] += load_coherent(part + b * stride + k);
    block_sum<1>(v, red);
    return v[0];
}

template <int kT>
__device__ __forceinline__ double finish_max(const double* part, int nb, int stride, int k,
                                             double* red)
{
    double m = 0.0;
    if ((int)threadIdx.x < kT)
        for (int b = threadIdx.x; b < nb; b += kT) {
            double t = load_coherent(part + b * stride + k);
            m = t > m ? t : m;
        }
    m = wave_max(m);
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave;
    __syncthreads();
    if (lane == 0) red[wid] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < (int)blockDim.x / kWave; ++w) t = red[w] > t ? red[w] : t;
        m = t;
    }
    __syncthreads();
    return m;
}

// Whether the history asks for step (record_every > 0: every multiple of it).
__device__ __forceinline__ bool recorded(int64_t step, int record_every)
{
    if (record_every <= 1) return record_every == 1;
    if (step < 0x7fffffff) return (uint32_t)step % (uint32_t)record_every == 0;
    return step % record_every == 0;
}

// Finish a completed step: count it, and on steps the history asks for, sum
// U, W (last force pass) and K, P (the partials of the integration pass, or
// with fused those of the fused force pass, step_part) and append them.
__device__ __forceinline__ void record_step(const KParams& p, int n_wg, int record_every,
                                            bool fused, double* red)
{
    DevState* dd = p.dev;
    const int64_t step = dd->step + 1;
    __syncthreads();
    if (threadIdx.x == 0) dd->step = step;
    if (!recorded(step, record_every)) return;
    double U = finish_sum<kFinishThreads>(p.fpart, p.nblk_force, 2, 0, red);
    double W = finish_sum<kFinishThreads>(p.fpart, p.nblk_force, 2, 1, red);
    if (p.bonded_on) {
        U += finish_sum<kFinishThreads>(p.bpart, p.nblk_bonded, 2, 0, red);
        W += finish_sum<kFinishThreads>(p.bpart, p.nblk_bonded, 2, 1, red);
    }
    double kp[4];
    for (int c = 0; c < 4; ++c)
        kp[c] = fused ? finish_sum<kFinishThreads>(step_part(p) + c * (int64_t)p.nblk_force,
                                                   p.nblk_force, 1, 0, red)
                      : finish_sum<kFinishThreads>(p.ipart, n_wg, 8, c, red);
    if (threadIdx.x == 0) {
        md_record* r = p.hist + (dd->hist_count % kHistCap);
        r->step = step;
        r->U = U;
        r->K = 0.5 * p.mass * kp[0];
        r->W = W;
        r->P[0] = p.mass * kp[1];
        r->P[1] = p.mass * kp[2];
        r->P[2] = p.mass * kp[3];
        r->dmax = sqrt(dd->dmax2);
        r->rebuilt = dd->rebuild;
        r->pad = 0;
        dd->hist_count += 1;
    }
}

// The largest of the displacement maxima in dev->dmax_slot (in every lane; a whole
// wave calls it).
__device__ __forceinline__ double step_dmax2(const KParams& p)
{
    const int lane = threadIdx.x & (kWave - 1);
    double v = 0.0;
    if (lane < kDmaxSlots) v = __longlong_as_double((long long)p.dev->dmax_slot[lane]);
    return wave_max(v);
}

// The end of an integration pass: count the step and record it (phase >= 1),
// and from the largest displacement decide whether the cells and list are
// rebuilt before the next force pass (phase <= 1; returned in every thread).  By one
// workgroup of at least kFinishThreads threads (red: LDS, (blockDim / 64) * 5
// doubles).  fused: the pass was a fused force pass (launch_forces_step).
// kSlots: its displacement maxima are in dev->dmax_slot in any case, and a later
// kernel clears them (k_bin_finish); else a fused pass's are cleared here.
template <bool kSlots = false>
__device__ __forceinline__ bool finish_step(const KParams& p, int phase, int record_every,
                                            bool fused, double* red)
{
    bool rebuild = false;
    const int n_wg = grid_of(p, G_INTEGRATE);
    if (phase >= 1) record_step(p, n_wg, record_every, fused, red);
    if (phase <= 1) {
        __shared__ int rb_all;
        double m = 0.0;
        if (kSlots || fused) {
            if (threadIdx.x < kWave) {
                m = step_dmax2(p);
                if (!kSlots && threadIdx.x < kDmaxSlots) p.dev->dmax_slot[threadIdx.x] = 0;
            }
        } else {
            m = finish_max<kFinishThreads>(p.ipart, n_wg, 8, 4, red);
        }
        if (threadIdx.x == 0) {
            DevState* d = p.dev;
            d->dmax2 = m;
            // whether the step that the next fused force pass ends is recorded
            d->record = recorded(d->step + 1, record_every) ? 1 : 0;
            const int rb = p.mode == MD_CELLS_ONLY ? 1 : (m > p.disp_thr2 ? 1 : 0);
            d->rebuild = rb;
            if (rb) d->n_rebuilds += 1;
            rb_all = rb;
        }
        __syncthreads();
        rebuild = rb_all != 0;
        if (p.gate_tab[0]) {  // a batch replica: its gate bits in the workgroup table
            const uint16_t v = (uint16_t)(p.rep | (rebuild ? kGateBit : 0));
            for (int j = 0; j < 3; ++j)
                for (int i = threadIdx.x; i < p.gate_n[j]; i += blockDim.x) p.gate_tab[j][i] = v;
        }
    }
    return rebuild;
}

}  // namespace md
