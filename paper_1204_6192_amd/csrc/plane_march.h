// plane_march.h -- a pair of half-sweeps, or two over-relaxation pairs, in one walk of
// whole planes along z (one replica per work-group; any even L whose planes fit).
//
// Stage s (a half-sweep of parity s & 1) takes the positions s .. L - 1 + s; position
// L + w is plane w again. A group of threads, one per site pair of a plane and
// parity, runs two stages: at step z group 0 runs stage 0 on position z, then stage 1
// on position z - 1; group 1 (four half-sweeps) stage 2 on position z - 3 and stage 3
// on z - 4, from what group 0 made in earlier steps. The z neighbours at a thread's
// own sites roll through registers; a plane is staged in LDS, decoded, for the
// in-plane neighbours and for the other group:
//   IN[2]  old parity-1 spins     R0[2 or 4]  stage 0's output
//   R1[3]  stage 1's output       R2[2]       stage 2's output
// One barrier per step.
//
// The periodic direction: plane w < s is not ready for stage s when it first passes.
// Its spins go home to HBM as they are, encoded, and come back at position L + w,
// where the stages that have done their part pass them through unchanged (decoding
// the codes gives the staged values).
//
// So every spin is read and written once per launch (and K - 1 planes twice), and
// the two groups of a four-half-sweep launch run side by side. Whole planes, so that
// a launch reads no halo, and a thread per pair, so that the rolled values stay in
// registers; one walk per replica, so that planes of any even L stage alike. Bound by
// the chain of steps where a CU has one work-group (a step's LDS reads, its sums and
// one barrier), by VALU in the heat bath and by HBM in bulk over-relaxation: a pair of
// 768 replicas of L = 64 in float32 moves 4.8 GB in 1.49 ms (3.2 TB/s; as two single
// passes 1.99 ms), the heat bath 1.57 -> 1.32 ms; two pairs of 1024 replicas of L = 32 in
// bfloat16 260 -> 226 us; L = 30, 512 replicas, float32, a sweep 1020 -> 389 us
// (gather passes). Which calls come here: use_plane.
#pragma once
#include <type_traits>

#include "device.h"
#include "kernels.h"
#include "lds_sites.h"

namespace hsg {

template <int STORE, int KIND, int G, int GRP, bool ENERGY, bool FIELD, bool JB, bool PAIRED>
__device__ __forceinline__ void march_group(const PlaneArgs &a, const int64_t r, float *lds, double *red)
{
    using C = Codec<STORE>;
    using T = typename C::T;
    constexpr bool HW = KIND == 2;
    constexpr bool LASTG = GRP == G - 1;
    constexpr bool EN = ENERGY && LASTG;  // the second stage of the last group sums the energy
    constexpr int NR0 = G == 1 ? 2 : 4;
    const int pq = (int)threadIdx.x - GRP * a.tpg;
    const bool active = pq < a.pp;
    const int64_t d = r / a.slots_per_sample;
    const int L = a.L, Lh = a.Lh;
    const uint32_t Nh = (uint32_t)a.Nh;
    const int cst = L * Lh;  // sites of a parity per plane
    T *sp0 = (T *)a.spins + r * 2 * C::kPlanes * (int64_t)Nh;
    T *sp1 = sp0 + (int64_t)C::kPlanes * Nh;
    const bool jbits = JB && a.Jbits != nullptr;
    const bool field = FIELD && a.Hp != nullptr;
    const float *J0 = a.J6 + d * 12 * (int64_t)Nh;
    const uint8_t *Jb0 = jbits ? a.Jbits + d * 2 * (int64_t)Nh : nullptr, *Jb1 = jbits ? Jb0 + Nh : nullptr;
    const float *H0 = field ? a.Hp + d * 6 * (int64_t)Nh : nullptr, *H1 = field ? H0 + 3 * (int64_t)Nh : nullptr;
    const float *J1 = J0 + 6 * (int64_t)Nh;  // one uniform base per coupling plane
    const float *const Jp0[3] = {J0, J0 + 2 * (int64_t)Nh, J0 + 4 * (int64_t)Nh};
    const float *const Jp1[3] = {J1, J1 + 2 * (int64_t)Nh, J1 + 4 * (int64_t)Nh};
    float beta = 0.0f;
    uint32_t c2 = 0, tsweep = 0;
    const uint32_t uid = a.uid_base + (uint32_t)d;
    if (KIND != 1) {
        const int sis = (int)(r - d * a.slots_per_sample);
        beta = a.beta32[a.temp_of_slot[r]];
        const int oc = sis / a.T, ts = sis - oc * a.T;
        c2 = (uint32_t)ts | ((uint32_t)oc << 8) | (a.rep << 12);
        tsweep = *a.tptr;
    }
    const int c = active ? 2 * pq : 0;  // idle lanes address the first pair
    PairPos<PAIRED> q = pair_pos<PAIRED>(c, L, Lh);
    const int psz = 3 * cst;  // floats per staged plane
    float *IN = lds, *R0 = lds + 2 * psz, *R1 = lds + (2 + NR0) * psz, *R2 = lds + (5 + NR0) * psz;

    auto next_plane = [&](int j) { return j + cst == (int)Nh ? 0 : j + cst; };
    auto slot_after = [&](int o, int n) { return o + psz == n * psz ? 0 : o + psz; };
    float2 jA[6], jB[6];
    v3 fA0, fA1, fB0, fB1;
    auto load_A = [&](int j) __attribute__((always_inline)) {
        load_couplings_planes<JB, FIELD>(Jp0, Jb0, H0, jbits, field, Nh, (uint32_t)(j + c), jA, fA0, fA1);
    };
    auto load_B = [&](int j) __attribute__((always_inline)) {
        load_couplings_planes<JB, FIELD>(Jp1, Jb1, H1, jbits, field, Nh, (uint32_t)(j + c), jB, fB0, fB1);
    };
    const int n_steps = G == 1 ? L + 2 : L + 7;
    double e = 0.0;

    // Values at my sites. Group 0: p, c, n = old parity 1 of positions z - 1, z, z + 1.
    // Group 1: stage 1's output of z - 4, z - 3, z - 2. a1, a2: the first stage's
    // output one and two positions before.
    v3 p0{}, p1{}, k0{}, k1{}, a10{}, a11{}, a20{}, a21{};
    // Group 0: old parity 1 of z + 1 and old parity 0 of z, one step in flight (two
    // steps measured the same).
    typename C::R raw1, raw0;
    if constexpr (GRP == 0) {
        C::template load_pair<true>(sp1, Nh, (uint32_t)((L - 1) * cst + c), p0, p1);
        C::template load_pair<true>(sp1, Nh, (uint32_t)c, k0, k1);
        if (active) pair_put(IN + q.c, k0, k1);
        C::template load_raw_pair<true>(sp1, Nh, (uint32_t)(cst + c), raw1);
        C::template load_raw_pair<true>(sp0, Nh, (uint32_t)c, raw0);
    }
    // plane of the first stage's position (z, or z - 3), of the second stage's, of
    // the spins to load
    int jw = GRP == 0 ? 0 : (L - 3) * cst;
    int jv = GRP == 0 ? (L - 1) * cst : (L - 4) * cst;
    int jl = cst;                     // group 0: plane of z + 1
    int oin = 0;                      // IN slot of z
    int or0 = 0;                      // R0 slot of z
    int or1 = (GRP == 0 ? 2 : 0) * psz;  // R1 slot of z - 1 (group 0), of z - 3 (group 1)
    int or2 = (GRP == 0 ? 0 : 1) * psz;  // R2 slot of z - 3
    load_A(jw);
    load_B(jv);
    __syncthreads();

    // The phases of a step are kept apart (sched_barrier): each one's LDS reads and
    // loads go out as registers of the one before become free, which keeps the
    // kernel at 128 registers, four waves per SIMD.
    // F: the steps 8 <= z < L, where every stage is active and only final spins go
    // home, compiled without the tests of the others.
    auto step = [&](auto zc, auto fc, const int z) __attribute__((always_inline)) {
        constexpr int t = decltype(zc)::value;  // z mod 2
        constexpr bool F = decltype(fc)::value;
        PlaneNb nb;
        v3 n0, n1;  // the plane above
        hide_pos(q);
        const int w = GRP == 0 ? z : z - 3;
        if constexpr (GRP == 0) {
            plane_neighbours<PAIRED>(q, t, IN + oin, nb);
            C::decode_pair(raw1, n0, n1);
            if (active) pair_put(IN + (psz - oin) + q.c, n0, n1);
        } else {
            const int r1n = slot_after(or1, 3);
            plane_neighbours<PAIRED>(q, 1 - t, R1 + or1, nb);
            pair_get(R1 + r1n + q.c, n0, n1);  // z - 2
            or1 = r1n;
        }
        // first stage
        u32x4 rr{0u, 0u, 0u, 0u};
        if (KIND != 1) rr = philox4x32_10(u32x4{(uint32_t)(jw + c) >> 1, tsweep, c2, uid}, a.key0, a.key1);
        PairField<false> fA = pair_field<false>(nb, n0, n1, p0, p1, jA, fA0, fA1);
        pin_field(fA);
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t jA0 = (uint32_t)(jw + c);
        jw = next_plane(jw);
        if constexpr (!EN) load_A(jw);
        v3 o0, o1;  // the first stage's old spins
        if constexpr (GRP == 0) {
            C::decode_pair(raw0, o0, o1);
            plane_neighbours<PAIRED>(q, t, R0 + (or0 == 0 ? (NR0 - 1) * psz : or0 - psz), nb);
        } else {
            const int r0o = or0 + psz;
            pair_get(R0 + (r0o >= 4 * psz ? r0o - 4 * psz : r0o) + q.c, o0, o1);  // z - 3
            plane_neighbours<PAIRED>(q, 1 - t, R2 + (psz - or2), nb);
        }
        v3 s0, s1;
        if (F || (w < L + 2 * GRP && w >= 2 * GRP)) {
            double none = 0.0;
            const typename C::R code = pair_update<STORE, KIND, false, HW>(fA, o0, o1, rr, beta, s0, s1, none);
            if ((LASTG || (!F && w <= 1)) && active) C::template store_raw_pair<true>(sp0, Nh, jA0, code);
        } else {
            s0 = o0;
            s1 = o1;
        }
        if (active) pair_put((GRP == 0 ? R0 + or0 : R2 + or2) + q.c, s0, s1);
        __builtin_amdgcn_sched_barrier(0);
        auto load_ahead = [&]() __attribute__((always_inline)) {
            if constexpr (GRP == 0) {
                // The spins of the next step. The heat bath needs old parity-0 spins only
                // where planes pass through; before, the load repeats plane 0 (a cache hit).
                const int jn = next_plane(jl);
                C::template load_raw_pair<true>(sp1, Nh, (uint32_t)(jn + c), raw1);
                C::template load_raw_pair<true>(sp0, Nh, (uint32_t)((KIND == 1 || z + 1 >= L ? jl : 0) + c),
                                                raw0);
                jl = jn;
            }
        };
        if constexpr (!EN) load_ahead();
        // second stage, a position behind
        if (KIND != 1)
            rr = philox4x32_10(u32x4{(uint32_t)(jv + c) >> 1, tsweep, c2 | (1u << 16), uid}, a.key0, a.key1);
        PairField<EN> fB = pair_field<EN>(nb, s0, s1, a20, a21, jB, fB0, fB1);
        pin_field(fB);
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t jB0 = (uint32_t)(jv + c);
        jv = next_plane(jv);
        // with the float64 sums, the loads wait until their registers are free again
        if constexpr (EN) {
            load_A(jw);
            load_ahead();
        }
        load_B(jv);
        v3 u0, u1;
        if (F || (w - 1 < L + 2 * GRP + 1 && w - 1 >= 2 * GRP + 1)) {
            const typename C::R code = pair_update<STORE, KIND, EN, HW>(fB, p0, p1, rr, beta, u0, u1, e);
            if (EN && field) field_energy<true>(a10, a11, H0, Nh, jB0, e);
            if ((LASTG || (!F && w - 1 <= 2)) && active) C::template store_raw_pair<true>(sp1, Nh, jB0, code);
        } else {
            u0 = p0;
            u1 = p1;
        }
        if constexpr (!LASTG) {
            if (active) pair_put(R1 + or1 + q.c, u0, u1);
        }
        a20 = a10; a21 = a11;
        a10 = s0; a11 = s1;
        p0 = k0; p1 = k1;
        k0 = n0; k1 = n1;
        oin = psz - oin;
        or0 = slot_after(or0, NR0);
        if constexpr (GRP == 0) or1 = slot_after(or1, 3);
        or2 = psz - or2;
        __syncthreads();
    };
    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, 1>;
    using Any = std::false_type;
    using Steady = std::true_type;
    // The numbers of steps are the same for both groups: every thread meets the same
    // barriers. L is even.
    int z = 0;
#pragma unroll 1
    for (; z < 8; z += 2) {
        step(Even{}, Any{}, z);
        step(Odd{}, Any{}, z + 1);
    }
#pragma unroll 1
    for (; z < L; z += 2) {
        step(Even{}, Steady{}, z);
        step(Odd{}, Steady{}, z + 1);
    }
#pragma unroll 1
    for (; z < n_steps; z += 2) {
        step(Even{}, Any{}, z);
        if (z + 1 >= n_steps) break;
        step(Odd{}, Any{}, z + 1);
    }
    if constexpr (EN) {
        if (!active) e = 0.0;
        e = wave_sum(e);
        if ((threadIdx.x & 63) == 0) red[pq >> 6] = e;
    }
}

template <int STORE, int KIND, int G, bool ENERGY, bool FIELD, bool JB, bool PAIRED>
__global__ __launch_bounds__(G == 1 ? 1024 : 512, 4) void k_plane_march(MultiPlaneArgs m)
{
    extern __shared__ __align__(16) float lds[];
    __shared__ double red[16];
    const int b = xcd_remap((int)blockIdx.x, m.n_blocks);
    int k = 0;
    while (k + 1 < m.n_groups && b >= m.block_start[k + 1]) ++k;
    const PlaneArgs &a = m.g[k];
    const int64_t r = a.r_base + (b - m.block_start[k]);
    const int g = __builtin_amdgcn_readfirstlane((int)threadIdx.x / a.tpg);
    if (g == 0) march_group<STORE, KIND, G, 0, ENERGY, FIELD, JB, PAIRED>(a, r, lds, red);
    if constexpr (G == 2) {
        if (g == 1) march_group<STORE, KIND, G, 1, ENERGY, FIELD, JB, PAIRED>(a, r, lds, red);
    }
    if (ENERGY) {  // the last group's waves, in order
        __syncthreads();
        if (threadIdx.x == 0) {
            double sum = 0.0;
            for (int w = 0; w < a.tpg / 64; ++w) sum += red[w];
            a.E[r] = sum;
        }
    }
}

template <int STORE, int KIND, int G>
static hipError_t launch_plane_g(const MultiPlaneArgs &m, bool energy, bool field, bool jb, bool paired,
                                 unsigned threads, size_t lds, hipStream_t s)
{
    const dim3 grid((unsigned)m.n_blocks), block(threads);
#define HSG_M(E, F, J, P) hipLaunchKernelGGL((k_plane_march<STORE, KIND, G, E, F, J, P>), grid, block, lds, s, m)
#define HSG_MP(E, F, J) \
    do { if (paired) HSG_M(E, F, J, true); else HSG_M(E, F, J, false); } while (0)
#define HSG_ME(F, J) \
    do { if (energy) HSG_MP(true, F, J); else HSG_MP(false, F, J); } while (0)
    if (field) {
        if (jb) HSG_ME(true, true); else HSG_ME(true, false);
    } else {
        if (jb) HSG_ME(false, true); else HSG_ME(false, false);
    }
#undef HSG_ME
#undef HSG_MP
#undef HSG_M
    return hipGetLastError();
}

template <int STORE>
hipError_t launch_plane_s(const MultiPlaneArgs &m, int kind, int groups, bool energy, bool field, bool jb, bool paired,
                          unsigned threads, size_t lds, hipStream_t s)
{
    if (groups == 2 && kind == 1)
        return launch_plane_g<STORE, 1, 2>(m, energy, field, jb, paired, threads, lds, s);
    if (groups != 1) return hipErrorInvalidValue;
    if (kind == 0) return launch_plane_g<STORE, 0, 1>(m, energy, field, jb, paired, threads, lds, s);
    if (kind == 2) return launch_plane_g<STORE, 2, 1>(m, energy, field, jb, paired, threads, lds, s);
    return launch_plane_g<STORE, 1, 1>(m, energy, field, jb, paired, threads, lds, s);
}

}  // namespace hsg
