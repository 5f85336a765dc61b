// ladder.hip -- what follows the updates of a sweep, in one launch, a work-group per
// (sample, copy) ladder or for several: the energies from their partial sums, the
// tempering walk of Eq. (4), the run statistics, and the step of the sweep counter.
//
// What bounds it: latency alone (a ladder is at most 256 energies). As launches of
// their own the four steps took 4.6 + 7 .. 16 + 6 + 4 us per sweep (reduction,
// tempering, statistics, counter; 16 us for 32 rungs), since one thread walked each
// ladder with a dependent load, a Philox block and an exponential per rung. Here
// everything but the walk itself is done for all rungs at once, and the walk
// compares exponents from LDS.
#include "device.h"
#include "kernels.h"

namespace hsg {

__global__ __launch_bounds__(256) void k_sweep_end(MultiLadderArgs m)
{
    __shared__ double sE[256], s_db[256], s_lu[256], s_u[256];
    __shared__ int32_t s_slot[256];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = (int)blockIdx.x;
    int k = 0;
    while (k + 1 < m.n_groups && b >= m.block_start[k + 1]) ++k;
    const LadderArgs &a = m.g[k];
    // A ladder takes `seg` threads: 2^n >= T within a wave up to 64 rungs, else all.
    // Its values stand at `base` in the arrays above.
    const int T = a.T, sg = tid >> a.seg_log2, l = tid - (sg << a.seg_log2), base = tid - l;
    const int64_t lad0 = (int64_t)(b - m.block_start[k]) * a.per_block, lad = lad0 + sg;
    const bool mine = sg < a.per_block && lad < a.n_lad;
    const int d = (int)(lad / a.O), o = (int)(lad - (int64_t)d * a.O);
    int32_t *sat = a.slot_at_temp + lad * T;
    int32_t *tos = a.temp_of_slot + lad * T;
    double *E = a.E + lad * T;
    const uint32_t t = m.tptr ? *m.tptr : m.ctr1;
    uint32_t one = 1;
    asm volatile("" : "+v"(one) : "s"(t));  // the ticket below is drawn after the counter has been read

    // Energies by slot. Several partials per replica: one wave per replica, lane l
    // adds partials l, l + 64, ... in order, then a fixed butterfly.
    if (a.n_pb > 1) {
        const double *p = a.partials + lad0 * T * a.n_pb;
        const int n = (int)min((int64_t)a.per_block, a.n_lad - lad0) * T;
#pragma unroll 4
        for (int r = wave; r < n; r += 4) {
            double v = 0.0;
            for (int i = lane; i < a.n_pb; i += 64) v += p[(int64_t)r * a.n_pb + i];
            v = wave_sum(v);
            if (lane == 0) {
                const int q = r / T;
                sE[(q << a.seg_log2) + r - q * T] = v;
                a.E[lad0 * T + r] = v;
            }
        }
    } else if (mine && l < T) {
        const double v = a.n_pb == 1 ? a.partials[lad * T + l] : E[l];
        sE[tid] = v;
        if (a.n_pb == 1) E[l] = v;
    }
    if (mine && l < T) s_slot[tid] = sat[l];
    const bool pt = m.pt && T > 1;
    if (pt && mine && l + 1 < T) {
        const u32x4 r = philox4x32_10(
            u32x4{(uint32_t)l, t, ((uint32_t)o << 8) | (m.purpose << 20), a.uid_base + (uint32_t)d}, m.key0, m.key1);
        const double u = u53(r.x, r.y);
        s_u[tid] = u;
        s_lu[tid] = log(u);
        s_db[tid] = a.beta64[l + 1] - a.beta64[l];
    }
    __syncthreads();

    // The walk k = 0 .. T-2 from the lowest temperature (float64 acceptance exponent;
    // temperatures move, spins stay): the replica that stands at rung k after the
    // steps below it is carried up while it is accepted. u <= exp(delta) is decided
    // by delta against ln u; within 1e-10 of each other (far above the rounding of
    // either) by the exponential itself, so that the decisions are those of the
    // direct comparison. Every lane of the ladder walks; lane k keeps what becomes of
    // rung k.
    if (pt && mine && l < 64) {
        int32_t car = s_slot[base];
        double ecar = sE[base + car];
        for (int c = 0; c + 1 < T; c += 64) {
            int32_t slot = 0;
            bool accepted = false;
            const int n = min(64, T - 1 - c);
#pragma unroll 4
            for (int i = 0; i < n; ++i) {
                const int32_t sb = s_slot[base + c + i + 1];
                const double eb = sE[base + sb], lu = s_lu[base + c + i];
                const double delta = s_db[base + c + i] * (eb - ecar);
                bool acc = delta >= 0.0 || delta > lu + 1e-10;
                if (__builtin_expect(!acc && !(delta < lu - 1e-10), 0)) acc = s_u[base + c + i] <= exp(delta);
                if (l == i) {
                    slot = acc ? sb : car;
                    accepted = acc;
                }
                if (!acc) {
                    car = sb;
                    ecar = eb;
                }
            }
            if (l < n) {
                sat[c + l] = slot;
                tos[slot] = c + l;
                if (accepted) a.accepts[lad * (T - 1) + c + l] += 1ull;
                if (m.stats) s_slot[base + c + l] = slot;  // rungs below the next chunk's
            }
        }
        if (l == 0) {
            sat[T - 1] = car;
            tos[car] = T - 1;
            if (m.stats) s_slot[base + T - 1] = car;
        }
    }

    // The energy of the configuration now at each rung is added to float64 sums of E
    // and E^2 (for U_L and C_L), and a replica that reaches the lowest rung after
    // visiting the highest since its last visit to the lowest completes a round
    // trip. flag per slot: 0 none yet, 1 at the lowest rung since, 2 reached the
    // highest rung after that.
    if (m.stats) {
        __syncthreads();
        if (mine && l < T) {
            const double e = sE[base + s_slot[tid]];
            double *sum = a.stat_sum + (lad * T + l) * 2;
            sum[0] += e;
            sum[1] += e * e;
        }
        if (mine && l == 0 && T > 1) {
            int32_t *flag = a.stat_flag + lad * T;
            uint32_t *trips = a.stat_trips + lad * T;
            const int32_t lo = s_slot[base], hi = s_slot[base + T - 1];
            if (flag[lo] == 2) trips[lo] += 1u;
            flag[lo] = 1;
            if (flag[hi] == 1) flag[hi] = 2;
        }
    }

    // The last work-group to get here (all have read the counter) advances it and
    // leaves the ticket at zero for the next launch.
    if (m.advance && tid == 0) {
        if (atomicAdd(m.ticket, one) + 1u == gridDim.x) {
            *m.ticket = 0u;
            *m.advance = t + 1u;
        }
    }
}

hipError_t launch_sweep_end(const MultiLadderArgs &m, hipStream_t s)
{
    if (m.n_groups < 1 || m.n_groups > kMaxStreamGroups || m.n_blocks < 1 || (m.advance && !m.ticket))
        return hipErrorInvalidValue;
    for (int k = 0; k < m.n_groups; ++k) {
        const LadderArgs &a = m.g[k];
        // a ladder's threads within a wave, or the whole work-group
        if (a.T < 1 || a.T > 256 || a.seg_log2 < 0 || a.seg_log2 > 8 || a.T > 1 << a.seg_log2 ||
            (a.T > 64 ? a.seg_log2 != 8 : a.seg_log2 > 6) || a.per_block < 1 || a.per_block << a.seg_log2 > 256 ||
            (int64_t)a.per_block * (m.block_start[k + 1] - m.block_start[k]) < a.n_lad)
            return hipErrorInvalidValue;
    }
    hipLaunchKernelGGL(k_sweep_end, dim3((unsigned)m.n_blocks), dim3(256), 0, s, m);
    return hipGetLastError();
}

}  // namespace hsg
