// lds_sites.h -- updates of site pairs whose spins, decoded, are held in LDS as
// three consecutive floats per site (replica.hip, plane_march.h).
//
// A pair of sites is three 8-byte LDS accesses from one address, and consecutive
// lanes (24 bytes apart) fall into distinct banks. A plane holds (L/2)^2 pairs
// of a parity for every even L; only rows of L % 4 = 2 are straddled by a pair.
#pragma once
#include "device.h"

namespace hsg {

__device__ __forceinline__ v3 site_get(const float *s) { return v3{s[0], s[1], s[2]}; }

__device__ __forceinline__ void pair_get(const float *s, v3 &a, v3 &b)
{
    const float2 u = *reinterpret_cast<const float2 *>(s);
    const float2 v = *reinterpret_cast<const float2 *>(s + 2);
    const float2 w = *reinterpret_cast<const float2 *>(s + 4);
    a = v3{u.x, u.y, v.x};
    b = v3{v.y, w.x, w.y};
}

__device__ __forceinline__ void pair_put(float *s, v3 a, v3 b)
{
    *reinterpret_cast<float2 *>(s) = make_float2(a.x, a.y);
    *reinterpret_cast<float2 *>(s + 2) = make_float2(a.z, b.x);
    *reinterpret_cast<float2 *>(s + 4) = make_float2(b.y, b.z);
}

// Where a pair's sites and in-plane neighbours stand, in floats from the start of
// a plane of one parity, with periodic wrap: the pair itself (c), the rows above
// and below (up, dn), and the x neighbours for either parity t = (z + parity) & 1
// of the plane. x = 2 xh + o on a row with o = (y + t) & 1, so +x -> xh + 1 and
// -x -> xh for o = 1, +x -> xh and -x -> xh - 1 for o = 0: the address depends on
// o, not the value (a select per site instead of six per pair). PAIRED
// (L % 4 = 0): both sites are in one row, and the first one's +x is the second
// one's -x.
template <bool PAIRED>
struct PairPos {
    int c, up0, dn0, up1, dn1;
    int xp0[2], xm0[2], xp1[2], xm1[2];
};

template <bool PAIRED>
__device__ __forceinline__ PairPos<PAIRED> pair_pos(int j, int L, int Lh)
{
    PairPos<PAIRED> q;
    const int cst = L * Lh;
    const int y0 = j / Lh, xh0 = j - y0 * Lh;
    const int y1 = PAIRED ? y0 : (j + 1) / Lh, xh1 = PAIRED ? xh0 + 1 : j + 1 - y1 * Lh;
    q.c = 3 * j;
    q.up0 = 3 * (j + (y0 + 1 == L ? Lh - cst : Lh));
    q.dn0 = 3 * (j + (y0 == 0 ? cst - Lh : -Lh));
    q.up1 = 3 * (j + 1 + (y1 + 1 == L ? Lh - cst : Lh));
    q.dn1 = 3 * (j + 1 + (y1 == 0 ? cst - Lh : -Lh));
    const int le0 = xh0 == 0 ? j + Lh - 1 : j - 1, ri0 = xh0 + 1 == Lh ? j + 1 - Lh : j + 1;
    const int le1 = xh1 == 0 ? j + Lh : j, ri1 = xh1 + 1 == Lh ? j + 2 - Lh : j + 2;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int o0 = (y0 + t) & 1, o1 = (y1 + t) & 1;
        q.xp0[t] = 3 * (o0 ? ri0 : j);
        q.xm0[t] = 3 * (o0 ? j : le0);
        q.xp1[t] = 3 * (o1 ? ri1 : j + 1);
        q.xm1[t] = PAIRED ? q.xp0[t] : 3 * (o1 ? j + 1 : le1);
    }
    return q;
}

// Hides that the offsets never change, so that the compiler adds them to a plane's
// base where they are used, and does not hold every sum across a loop.
template <bool PAIRED>
__device__ __forceinline__ void hide_pos(PairPos<PAIRED> &q)
{
    asm volatile("" : "+v"(q.c), "+v"(q.up0), "+v"(q.dn0));
    asm volatile("" : "+v"(q.xp0[0]), "+v"(q.xm0[0]), "+v"(q.xp1[0]), "+v"(q.xp0[1]), "+v"(q.xm0[1]), "+v"(q.xp1[1]));
    if constexpr (!PAIRED) asm volatile("" : "+v"(q.up1), "+v"(q.dn1), "+v"(q.xm1[0]), "+v"(q.xm1[1]));
}

// The in-plane neighbours (+x, -x, +y, -y) of a pair in the other parity's plane at
// pl; t as above.
struct PlaneNb {
    v3 a[4], b[4];
};

template <bool PAIRED>
__device__ __forceinline__ void plane_neighbours(const PairPos<PAIRED> &q, int t, const float *pl, PlaneNb &n)
{
    n.a[0] = site_get(pl + (t ? q.xp0[1] : q.xp0[0]));
    n.a[1] = site_get(pl + (t ? q.xm0[1] : q.xm0[0]));
    n.b[0] = site_get(pl + (t ? q.xp1[1] : q.xp1[0]));
    if constexpr (PAIRED) {
        n.b[1] = n.a[0];
        pair_get(pl + q.up0, n.a[2], n.b[2]);
        pair_get(pl + q.dn0, n.a[3], n.b[3]);
    } else {
        n.b[1] = site_get(pl + (t ? q.xm1[1] : q.xm1[0]));
        n.a[2] = site_get(pl + q.up0);
        n.b[2] = site_get(pl + q.up1);
        n.a[3] = site_get(pl + q.dn0);
        n.b[3] = site_get(pl + q.dn1);
    }
}

// The local fields (Eq. (2)) of a pair from its neighbours in the plane, above
// (u0, u1) and below (d0, d1), in the neighbour order of the other kernels; with
// ENERGY also in float64.
template <bool ENERGY>
struct PairField {
    v3 h0, h1;
    double x0, y0, z0, x1, y1, z1;
};

template <bool ENERGY>
__device__ __forceinline__ PairField<ENERGY> pair_field(const PlaneNb &n, v3 u0, v3 u1, v3 d0, v3 d1,
                                                        const float2 (&jc)[6], v3 hs0, v3 hs1)
{
    const v3 nb0[6] = {n.a[0], n.a[1], n.a[2], n.a[3], u0, d0}, nb1[6] = {n.b[0], n.b[1], n.b[2], n.b[3], u1, d1};
    PairField<ENERGY> f;
    f.h0 = hs0;
    f.h1 = hs1;
    f.x0 = hs0.x; f.y0 = hs0.y; f.z0 = hs0.z;
    f.x1 = hs1.x; f.y1 = hs1.y; f.z1 = hs1.z;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        acc3(f.h0, jc[k].x, nb0[k]);
        acc3(f.h1, jc[k].y, nb1[k]);
        if (ENERGY) {
            f.x0 = fma((double)jc[k].x, (double)nb0[k].x, f.x0);
            f.y0 = fma((double)jc[k].x, (double)nb0[k].y, f.y0);
            f.z0 = fma((double)jc[k].x, (double)nb0[k].z, f.z0);
            f.x1 = fma((double)jc[k].y, (double)nb1[k].x, f.x1);
            f.y1 = fma((double)jc[k].y, (double)nb1[k].y, f.y1);
            f.z1 = fma((double)jc[k].y, (double)nb1[k].z, f.z1);
        }
    }
    return f;
}

// Makes the compiler form the fields here: it would otherwise move the sums into the
// branch that uses them, and hold neighbours and couplings until then.
template <bool ENERGY>
__device__ __forceinline__ void pin_field(PairField<ENERGY> &f)
{
    asm volatile("" : "+v"(f.h0.x), "+v"(f.h0.y), "+v"(f.h0.z), "+v"(f.h1.x), "+v"(f.h1.y), "+v"(f.h1.z));
    if constexpr (ENERGY)
        asm volatile("" : "+v"(f.x0), "+v"(f.y0), "+v"(f.z0), "+v"(f.x1), "+v"(f.y1), "+v"(f.z1));
}

// The new spins of a pair from its fields and (over-relaxation) its old spins o0,
// o1: their codes, and in s0, s1 what reading the codes back gives. With ENERGY the
// bond energy of the two sites is added to e (each bond has one endpoint on a
// parity).
template <int STORE, int KIND, bool ENERGY, bool HW>
__device__ __forceinline__ typename Codec<STORE>::R pair_update(const PairField<ENERGY> &f, v3 o0, v3 o1, u32x4 rr,
                                                                float beta, v3 &s0, v3 &s1, double &e)
{
    using C = Codec<STORE>;
    v3 n0, n1;
    if (KIND != 1) {
        n0 = heat_bath<HW, STORE == 0>(f.h0, beta, rr.x, rr.y);
        n1 = heat_bath<HW, STORE == 0>(f.h1, beta, rr.z, rr.w);
    } else {
        over_relax_pair<STORE == 0>(o0, f.h0, o1, f.h1, n0, n1);
    }
    const typename C::R code = C::encode_pair(n0, n1);
    C::decode_pair(code, s0, s1);
    if (ENERGY) {
        e -= (double)s0.x * f.x0 + (double)s0.y * f.y0 + (double)s0.z * f.z0;
        e -= (double)s1.x * f.x1 + (double)s1.y * f.y1 + (double)s1.z * f.z1;
    }
    return code;
}

}  // namespace hsg
