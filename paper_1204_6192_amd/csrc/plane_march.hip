// plane_march.hip -- dispatch of the plane march by spin storage codec.
#include "kernels.h"

namespace hsg {

template <int STORE>
hipError_t launch_plane_s(const MultiPlaneArgs &m, int kind, int groups, bool energy, bool field, bool jb, bool paired,
                          unsigned threads, size_t lds, hipStream_t s);

hipError_t launch_plane_march(const MultiPlaneArgs &m, int storage, int kind, int groups, bool energy,
                              unsigned threads, size_t lds, hipStream_t s)
{
    if (m.n_groups < 1 || m.n_groups > kMaxStreamGroups || m.n_blocks < 1 || threads == 0 || threads % 64 != 0 ||
        threads > (groups == 1 ? 1024u : 512u) || groups < 1 || groups > 2)
        return hipErrorInvalidValue;
    bool field = false, jb = false, paired = true;
    for (int k = 0; k < m.n_groups; ++k) {
        const PlaneArgs &a = m.g[k];
        // L >= 8: a plane that goes home in the first steps is back there before it
        // is read again; 32-bit byte offsets within a replica and a sample
        if (a.L < 8 || a.L > 512 || a.tpg % 64 != 0 || a.pp > a.tpg || (unsigned)(groups * a.tpg) != threads ||
            plane_march_lds(a.L, groups) > lds)
            return hipErrorInvalidValue;
        field = field || a.Hp != nullptr;
        jb = jb || a.Jbits != nullptr;
        paired = paired && a.L % 4 == 0;
    }
    switch (storage) {
    case 0: return launch_plane_s<0>(m, kind, groups, energy, field, jb, paired, threads, lds, s);
    case 1: return launch_plane_s<1>(m, kind, groups, energy, field, jb, paired, threads, lds, s);
    case 2: return launch_plane_s<2>(m, kind, groups, energy, field, jb, paired, threads, lds, s);
    case 3: return launch_plane_s<3>(m, kind, groups, energy, field, jb, paired, threads, lds, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace hsg
