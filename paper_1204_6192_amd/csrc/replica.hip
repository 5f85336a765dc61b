// replica.hip -- whole sweeps of small lattices, a replica per group of waves,
// its spins held in LDS from the first half-sweep to the last.
//
// Both parities of a replica, decoded, take 12 L^3 bytes of LDS (6 KiB at
// L = 8, 48 KiB at L = 16, 125 KiB at L = 22). One launch runs every half-sweep
// of one sweep (Eqs. (2), (3)) and the float64 energy of Eq. (1); tempering needs
// the other replicas' energies and is a launch of its own.
//
// What bounds it: instruction issue and, with few replicas, the latency of one
// half-sweep (a load of the couplings, the LDS reads of the neighbours, a chain
// of dependent multiply-adds, one barrier). A z-march instead walks the planes
// one by one, with a barrier each: L + 6 dependent steps for four half-sweeps.
// Here a half-sweep of L = 8 is a single step, and one of L = 16 one or two.
//
// Thread (z, pair of the plane) of a replica owns the site pair (2q, 2q + 1) of
// either parity in the planes z, z + ZB, z + 2 ZB, ... The same per-site functions, neighbour order, counter map and codec as
// the other kernels: the same spins bit for bit; the energies to rounding
// (another summation order). The couplings are read from the cache once per
// half-sweep, the same for all replicas of the sample.
#include <type_traits>

#include "device.h"
#include "kernels.h"
#include "lds_sites.h"

namespace hsg {

// SUB: four replicas of L = 4 per wave, 16 threads each (rows of 4 need PAIRED).
template <int STORE, bool FIELD, bool JB, bool HW, bool PAIRED, bool SUB>
__device__ __forceinline__ void replica_body(const ReplicaArgs &a, const int lb, float *lds, double *red)
{
    using C = Codec<STORE>;
    using T = typename C::T;
    const int tid = (int)threadIdx.x;
    // whole waves per replica, so everything that depends on it alone is uniform
    const int rb = SUB ? tid / a.tpr : __builtin_amdgcn_readfirstlane(tid / a.tpr);
    const int rem = tid - rb * a.tpr;
    const int zz = rem / a.pp, pq = rem - zz * a.pp;
    const int64_t r_lane = a.r_base + (int64_t)lb * a.RB + rb;
    const bool mine = rb < a.RB && r_lane < a.r_end;      // the wave has a replica
    const bool active = mine && zz < a.ZB;
    const int64_t r = mine ? r_lane : a.r_base;
    const int64_t d = r / a.slots_per_sample;
    const int sis = (int)(r - d * a.slots_per_sample);
    const int L = a.L, Lh = a.Lh;
    const uint32_t Nh = (uint32_t)a.Nh;
    const int cst = L * Lh;  // sites of a parity per plane
    T *sp0 = (T *)a.spins + r * 2 * C::kPlanes * (int64_t)Nh;
    T *sp1 = sp0 + (int64_t)C::kPlanes * Nh;
    float *mem = lds + (size_t)(mine ? rb : 0) * 6 * Nh;  // [parity][site][3]
    const bool jbits = JB && a.Jbits != nullptr;
    const bool field = FIELD && a.Hp != nullptr;
    const float beta = a.beta32[a.temp_of_slot[r]];
    const int oc = sis / a.T, ts = sis - oc * a.T;
    const uint32_t c2r = (uint32_t)ts | ((uint32_t)oc << 8);
    const uint32_t uid = a.uid_base + (uint32_t)d;
    const uint32_t tsweep = *a.tptr;

    const int c = 2 * pq;
    const PairPos<PAIRED> q = pair_pos<PAIRED>(c, L, Lh);

    // spins into LDS
    if (active)
        for (int z = zz; z < L; z += a.ZB) {
            const uint32_t j0 = (uint32_t)(z * cst + c);
            v3 s0, s1, u0, u1;
            C::template load_pair<true>(sp0, Nh, j0, s0, s1);
            C::template load_pair<true>(sp1, Nh, j0, u0, u1);
            pair_put(mem + 3 * j0, s0, s1);
            pair_put(mem + 3 * (Nh + j0), u0, u1);
        }
    __syncthreads();

    double e = 0.0;
    auto half = [&](auto kc, auto ec, const int p, const uint32_t rep, const bool store)
                    __attribute__((always_inline)) {
        constexpr int KIND = decltype(kc)::value;
        constexpr bool ENERGY = decltype(ec)::value;
        if (!active) return;
        const float *Jb = a.J6 + (d * 2 + p) * 6 * (int64_t)Nh;
        const uint8_t *Jbb = jbits ? a.Jbits + (d * 2 + p) * (int64_t)Nh : nullptr;
        const float *Hb = field ? a.Hp + (d * 2 + p) * 3 * (int64_t)Nh : nullptr;
        const float *const Jp[3] = {Jb, Jb + 2 * (int64_t)Nh, Jb + 4 * (int64_t)Nh};
        float *own = mem + (p ? 3 * Nh : 0u);
        const float *oth = mem + (p ? 0u : 3 * Nh);
#pragma unroll 1
        for (int z = zz; z < L; z += a.ZB) {
            const int zb = z * cst;
            const uint32_t j0 = (uint32_t)(zb + c);
            float2 jc[6];
            v3 h0, h1;
            load_couplings_planes<JB, FIELD>(Jp, Jbb, Hb, jbits, field, Nh, j0, jc, h0, h1);
            u32x4 rr{0u, 0u, 0u, 0u};
            if (KIND != 1)
                rr = philox4x32_10(u32x4{j0 >> 1, tsweep, c2r | (rep << 12) | ((uint32_t)p << 16), uid}, a.key0,
                                   a.key1);
            const float *pl = oth + 3 * zb;
            const float *pu = oth + 3 * (z + 1 == L ? 0 : zb + cst);
            const float *pd = oth + 3 * (z == 0 ? (L - 1) * cst : zb - cst);
            PlaneNb nb;
            plane_neighbours<PAIRED>(q, (z + p) & 1, pl, nb);
            v3 u0, u1, d0, d1, o0{}, o1{}, s0, s1;
            pair_get(pu + q.c, u0, u1);
            pair_get(pd + q.c, d0, d1);
            if (KIND == 1) pair_get(own + 3 * j0, o0, o1);
            const PairField<ENERGY> f = pair_field<ENERGY>(nb, u0, u1, d0, d1, jc, h0, h1);
            const typename C::R code = pair_update<STORE, KIND, ENERGY, HW>(f, o0, o1, rr, beta, s0, s1, e);
            pair_put(own + 3 * j0, s0, s1);
            if (store) C::template store_raw_pair<true>(p ? sp1 : sp0, Nh, j0, code);
            if (ENERGY && field) {
                pair_get(oth + 3 * j0, o0, o1);
                field_energy<true>(o0, o1, a.Hp + d * 2 * 3 * (int64_t)Nh, Nh, j0, e);
            }
        }
    };
    using K0 = std::integral_constant<int, 0>;
    using K1 = std::integral_constant<int, 1>;
    using NoE = std::false_type;
    using WithE = std::true_type;
    const int n_half = 2 * (a.n_hb + a.n_or);
#pragma unroll 1
    for (int it = 0; it < n_half; ++it) {
        const bool last = it + 1 == n_half;
        if (it < 2 * a.n_hb) {
            if (last) half(K0{}, WithE{}, it & 1, (uint32_t)(it >> 1), true);
            else half(K0{}, NoE{}, it & 1, (uint32_t)(it >> 1), it + 2 >= n_half);
        } else {
            if (last) half(K1{}, WithE{}, it & 1, 0u, true);
            else half(K1{}, NoE{}, it & 1, 0u, it + 2 >= n_half);
        }
        __syncthreads();
    }
    if constexpr (SUB) {  // the replica's energy: its quarter of the wave
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) e += __shfl_xor(e, off, 64);
        if (mine && rem == 0) a.E[r] = e;
        return;
    }
    // the replica's energy: waves, then its waves in order
    e = wave_sum(e);
    if ((tid & 63) == 0) red[tid >> 6] = e;
    __syncthreads();
    if (mine && rem == 0) {
        double s = 0.0;
        for (int w = 0; w < a.tpr / 64; ++w) s += red[(tid >> 6) + w];
        a.E[r] = s;
    }
}

template <int STORE, bool FIELD, bool JB, bool HW, bool PAIRED, bool SUB>
__global__ __launch_bounds__(SUB ? 64 : 1024) void k_replica_sweep(MultiReplicaArgs m)
{
    extern __shared__ __align__(16) float lds[];
    __shared__ double red[16];
    const int b = xcd_remap((int)blockIdx.x, m.n_blocks);
    int k = 0;
    while (k + 1 < m.n_groups && b >= m.block_start[k + 1]) ++k;
    replica_body<STORE, FIELD, JB, HW, PAIRED, SUB>(m.g[k], b - m.block_start[k], lds, red);
}

template <int STORE>
static hipError_t launch_replica_s(const MultiReplicaArgs &m, bool field, bool jb, bool hw, bool paired, bool sub,
                                   unsigned threads, size_t lds, hipStream_t s)
{
    const dim3 grid((unsigned)m.n_blocks), block(threads);
#define HSG_P(F, J, H, P, S) hipLaunchKernelGGL((k_replica_sweep<STORE, F, J, H, P, S>), grid, block, lds, s, m)
#define HSG_PP(F, J, H) \
    do { \
        if (sub) HSG_P(F, J, H, true, true); \
        else if (paired) HSG_P(F, J, H, true, false); \
        else HSG_P(F, J, H, false, false); \
    } while (0)
#define HSG_PH(F, J) \
    do { if (hw) HSG_PP(F, J, true); else HSG_PP(F, J, false); } while (0)
    if (field) {
        if (jb) HSG_PH(true, true); else HSG_PH(true, false);
    } else {
        if (jb) HSG_PH(false, true); else HSG_PH(false, false);
    }
#undef HSG_PH
#undef HSG_PP
#undef HSG_P
    return hipGetLastError();
}

hipError_t launch_replica(const MultiReplicaArgs &m, int storage, bool hw, unsigned threads, size_t lds,
                          hipStream_t s)
{
    if (m.n_groups < 1 || m.n_groups > kMaxStreamGroups || threads == 0 || threads > 1024 || threads % 64 != 0)
        return hipErrorInvalidValue;
    bool field = false, jb = false, paired = true;
    const bool sub = m.g[0].tpr == 16;
    for (int k = 0; k < m.n_groups; ++k) {
        const ReplicaArgs &a = m.g[k];
        if ((sub ? a.tpr != 16 || a.L != 4 || threads != 64 : a.tpr % 64 != 0) || a.ZB * a.pp > a.tpr || (unsigned)(a.RB * a.tpr) > threads ||
            (size_t)a.RB * 6 * a.Nh * sizeof(float) > lds)
            return hipErrorInvalidValue;
        field = field || a.Hp != nullptr;
        jb = jb || a.Jbits != nullptr;
        paired = paired && a.L % 4 == 0;
    }
    switch (storage) {
    case 0: return launch_replica_s<0>(m, field, jb, hw, paired, sub, threads, lds, s);
    case 1: return launch_replica_s<1>(m, field, jb, hw, paired, sub, threads, lds, s);
    case 2: return launch_replica_s<2>(m, field, jb, hw, paired, sub, threads, lds, s);
    case 3: return launch_replica_s<3>(m, field, jb, hw, paired, sub, threads, lds, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace hsg
