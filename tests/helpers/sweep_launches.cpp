// The host side of a sweep (api.hip) on the CPU, its kernels replaced by stand-ins that
// record what each launch does: which half-sweeps every replica gets, with which
// counter, and where the energies are left. The energy pass leaves the true value in E
// or as partial sums in scratch, and the end of the sweep reads E as the library tells
// it to; what has not been written since the last sweep holds NaN.
//
// Reads one case per line from standard input,
//   storage n_hb n_or variant batch overlap sweeps  n_groups  (L samples copies rungs field)...
// (field: 1 with a field, + 2 with couplings of one sign bit)
// and prints "ok" or what is wrong for each; overlap = 2: and the halves have to be in effect.
#include <hip/hip_runtime.h>
#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) static_cast<const void *>(x)
#include "../../paper_1204_6192_amd/csrc/api.hip"

#include <sys/mman.h>

#include <iostream>
#include <sstream>

namespace {

struct Rep {
    uint64_t seq = 0;  // hash of the half-sweeps of this sweep
    int32_t n = 0;
};
hsg_lattice *g_h = nullptr;
std::vector<std::vector<Rep>> g_reps;  // [group][replica]
std::string g_bad;
uint32_t g_t = 0;  // the counter that every launch of the sweep has to read
int g_ended = 0;   // work of the sweeps' ends: replicas whose ladders have been walked
int g_steps = 0;   // counters that the sweep's ends stepped

void bad(const std::string &s)
{
    if (g_bad.empty()) g_bad = s;
}

uint64_t code(int kind, uint32_t rep, int parity) { return 1 + (kind == 1 ? 100u : 2 * rep) + (uint64_t)parity; }
uint64_t join(uint64_t h, uint64_t c) { return h * 1000003u + c; }

size_t group_of(const void *spins)
{
    for (size_t k = 0; k < g_h->lay.g.size(); ++k)
        if (spins == g_h->state + g_h->lay.g[k].o_spins) return k;
    bad("spins of no group");
    return 0;
}

void half_sweep(size_t k, int64_t r, int kind, uint32_t rep, int parity, const uint32_t *tptr)
{
    if (*tptr != g_t) bad("a launch reads another sweep's counter");
    Rep &x = g_reps[k].at(r);
    x.seq = join(x.seq, code(kind, rep, parity));
    x.n += 1;
}

double true_energy(size_t k, int64_t r) { return 1e6 * (double)(g_t + 1) + 1e4 * (double)k + (double)r; }

double *energies(size_t k) { return reinterpret_cast<double *>(g_h->state + g_h->lay.g[k].o_E); }

void leave_partials(double *p, size_t k, int64_t r, int n_pb)
{
    for (int i = 1; i < n_pb; ++i) p[r * n_pb + i] = 0.0;
    p[r * n_pb] = true_energy(k, r);
}

}  // namespace

namespace hsg {

hipError_t launch_half_sweep(const SweepArgs &a, int, int kind, bool, bool energy, hipStream_t)
{
    const size_t k = group_of(a.spins);
    if (a.n_blocks < 1 || a.n_blocks % a.n_pb != 0) bad("a gather pass with part of an item");
    for (int64_t i = a.item0; i < a.item0 + a.n_blocks / a.n_pb; ++i) {
        const int64_t d = i / a.n_chunks, ch = i - d * a.n_chunks;
        bool any = false;
        for (int64_t s = ch * a.chunk; s < std::min((ch + 1) * a.chunk, (int64_t)a.slots_per_sample); ++s) {
            const int64_t r = d * a.slots_per_sample + s;
            if (r < a.r_begin || r >= a.r_end) continue;
            any = true;
            half_sweep(k, r, kind, a.rep, (int)a.parity, a.tptr);
            if (energy) leave_partials(a.e_partials, k, r, a.n_pb);
        }
        if (!any) bad("a gather pass with an item of no replica");
    }
    return hipSuccess;
}

hipError_t launch_half_sweep_stream(const MultiStreamArgs &m, int, int kind, bool energy, int fuse, unsigned, size_t,
                                    hipStream_t)
{
    for (int i = 0; i < m.n_groups; ++i) {
        const StreamArgs &a = m.g[i];
        const size_t k = group_of(a.spins);
        for (int64_t r = a.r_base; r < a.n_rep; ++r) {
            if (fuse == 0) half_sweep(k, r, kind, a.rep, (int)a.parity, a.tptr);
            for (int p = 0; p < 2 * fuse; ++p) half_sweep(k, r, kind, a.rep, p & 1, a.tptr);
            if (energy) leave_partials(a.e_partials, k, r, a.n_ytiles * a.n_zslabs);
        }
    }
    return hipSuccess;
}

hipError_t launch_plane_march(const MultiPlaneArgs &m, int, int kind, int groups, bool energy, unsigned threads, size_t,
                              hipStream_t)
{
    for (int i = 0; i < m.n_groups; ++i) {
        const PlaneArgs &a = m.g[i];
        const size_t k = group_of(a.spins);
        if ((unsigned)(groups * a.tpg) != threads) bad("a plane march with idle waves");
        const int64_t n = m.block_start[i + 1] - m.block_start[i];
        for (int64_t r = a.r_base; r < a.r_base + n; ++r) {
            for (int p = 0; p < 2 * groups; ++p) half_sweep(k, r, kind, a.rep, p & 1, a.tptr);
            if (energy) energies(k)[r] = true_energy(k, r);
        }
    }
    return hipSuccess;
}

hipError_t launch_replica(const MultiReplicaArgs &m, int, bool, unsigned, size_t, hipStream_t)
{
    for (int i = 0; i < m.n_groups; ++i) {
        const ReplicaArgs &a = m.g[i];
        const size_t k = group_of(a.spins);
        const int64_t blocks = (i + 1 < m.n_groups ? m.block_start[i + 1] : m.n_blocks) - m.block_start[i];
        if (blocks != a.n_blocks || blocks * a.RB < a.r_end - a.r_base) bad("a replica launch of too few work-groups");
        for (int64_t r = a.r_base; r < a.r_end; ++r) {
            for (int j = 0; j < 2 * a.n_hb; ++j) half_sweep(k, r, 0, (uint32_t)(j / 2), j & 1, a.tptr);
            for (int j = 0; j < 2 * a.n_or; ++j) half_sweep(k, r, 1, 0, j & 1, a.tptr);
            energies(k)[r] = true_energy(k, r);
        }
    }
    return hipSuccess;
}

hipError_t launch_sweep_end(const MultiLadderArgs &m, hipStream_t)
{
    for (int i = 0; i < m.n_groups; ++i) {
        const LadderArgs &a = m.g[i];
        size_t k = 0;
        while (k < g_h->lay.g.size() &&
               !(a.E >= energies(k) && a.E < energies(k) + g_h->lay.g[k].n_rep))
            ++k;
        const int64_t r0 = a.E - energies(k), n = a.n_lad * a.T;
        const int64_t blocks = m.block_start[i + 1] - m.block_start[i];
        if (blocks * a.per_block < a.n_lad || (blocks - 1) * a.per_block >= a.n_lad || (a.per_block << a.seg_log2) > 256 ||
            a.T > 1 << a.seg_log2)
            bad("the ladders do not fit their work-groups");
        for (int64_t j = 0; j < n; ++j) {
            if (a.n_pb > 0) {
                double e = 0.0;
                for (int p = 0; p < a.n_pb; ++p) e += a.partials[j * a.n_pb + p];
                a.E[j] = e;
            }
            if (!(a.E[j] == true_energy(k, r0 + j))) {
                std::ostringstream s;
                s << "group " << k << " replica " << r0 + j << ": the end of sweep " << g_t << " reads an energy of "
                  << a.E[j] << ", the last pass left " << true_energy(k, r0 + j);
                bad(s.str());
            }
        }
        g_ended += (int)n;
    }
    if (m.advance) {
        *m.advance = *m.tptr + 1;
        if (m.ticket != reinterpret_cast<uint32_t *>(g_h->state) + 2 + (m.advance - reinterpret_cast<uint32_t *>(g_h->state)))
            bad("the halves share a ticket");
        g_steps += 1;
    }
    return hipSuccess;
}

hipError_t launch_copy_u32(const uint32_t *src, uint32_t *dst, hipStream_t)
{
    *dst = *src;
    return hipSuccess;
}
hipError_t launch_advance(uint32_t *p, hipStream_t)
{
    *p += 1;
    g_steps += 1;
    return hipSuccess;
}

// not part of a sweep of the full-lattice chain
hipError_t launch_set_u32(uint32_t *, uint32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_energy(const EnergyArgs &, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_kmodes(const KmodeArgs &, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_philox(const uint32_t *, const uint32_t *, uint32_t *, int64_t, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_series(const SeriesArgs &, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_hw_math(const float *, float *, int64_t, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_overlap(const OverlapArgs &, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_pair_overlaps(const PairOvArgs &, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_reduce_partials(const double *, int, int64_t, double *, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_tile_visit(const TileArgs &, int, bool, bool, bool, unsigned, size_t, hipStream_t)
{
    return hipErrorUnknown;
}
hipError_t launch_invert_maps(const int32_t *, int32_t *, int64_t, int32_t, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_unpack_spins(const PackArgs &, int, hipStream_t) { return hipErrorUnknown; }
hipError_t launch_check_pm1(const float *, int64_t, int32_t *, hipStream_t) { return hipSuccess; }
hipError_t launch_pack_jbits(const float *, uint8_t *, int64_t, int32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_pack_field(const PackArgs &, hipStream_t) { return hipSuccess; }
hipError_t launch_pack_spins(const PackArgs &, int, hipStream_t) { return hipSuccess; }
hipError_t launch_pack_couplings(const PackArgs &, hipStream_t) { return hipSuccess; }
hipError_t launch_stats_clear(double *, int32_t *, uint32_t *, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_fill_identity_maps(int32_t *, int32_t *, int64_t, int32_t, hipStream_t) { return hipSuccess; }
int64_t energy_partials(int, int64_t, int64_t n_pb_site) { return n_pb_site; }
int64_t march_partials(int, int64_t, int64_t q_pb) { return q_pb; }
int64_t kmode_partials(int, int64_t q_pb) { return q_pb; }

}  // namespace hsg

extern "C" {
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    *v = 160 * 1024;
    return hipSuccess;
}
hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "a stand-in's error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s)
{
    *p = const_cast<void *>(s);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t)
{
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *, unsigned) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipErrorUnknown; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    return hipErrorUnknown;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorUnknown; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorUnknown; }
hipError_t hipStreamCreateWithFlags(hipStream_t *, unsigned) { return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorUnknown; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}

namespace {

void *reserve(size_t n)  // pages of spins and couplings are never touched
{
    return mmap(nullptr, n + 1, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
}

std::string run(std::istringstream &in)
{
    int storage, n_hb, n_or, variant, overlap, sweeps, n_groups;
    long long batch;
    in >> storage >> n_hb >> n_or >> variant >> batch >> overlap >> sweeps >> n_groups;
    std::vector<double> temps(256);
    for (int k = 0; k < 256; ++k) temps[k] = 0.1 + 0.01 * k;
    std::vector<hsg_group_desc> gd(n_groups);
    uint32_t uid = 0;
    for (auto &g : gd) {
        g = hsg_group_desc{};
        in >> g.L >> g.n_samples >> g.n_copies >> g.n_temps >> g.has_field;
        g.coupling_kind = g.has_field >> 1;
        g.has_field &= 1;
        g.temps = temps.data();
        g.sample_uid_base = uid;
        uid += (uint32_t)g.n_samples;
    }
    if (!in) return "unreadable case";
    hsg_desc d{};
    d.groups = gd.data();
    d.n_groups = n_groups;
    d.storage = storage;
    d.n_hb = n_hb;
    d.n_or = n_or;
    d.pt_every = 1;
    hsg_sizes sz{};
    if (hsg_query_sizes(&d, &sz) != HSG_OK) return hsg_last_error();
    const size_t bytes[4] = {sz.state_bytes, sz.coupling_bytes, sz.field_bytes, sz.scratch_bytes};
    void *buf[4];
    for (int k = 0; k < 4; ++k) buf[k] = reserve(bytes[k]);
    float one = 0.0f;  // the canonical inputs are not read
    g_h = nullptr;
    std::string out;
    hsg_lattice *h = nullptr;
    if (hsg_init_lattice(&d, &one, &one, &one, buf[0], buf[1], buf[2], buf[3], nullptr, &h) != HSG_OK) {
        out = hsg_last_error();
    } else {
        g_h = h;
        g_bad.clear();
        if (hsg_set_kernel(h, variant) != HSG_OK || hsg_set_batch(h, batch) != HSG_OK ||
            hsg_set_overlap(h, overlap != 0) != HSG_OK)
            bad(hsg_last_error());
        uint64_t want = 0;
        for (int j = 0; j < 2 * n_hb; ++j) want = join(want, code(0, (uint32_t)(j / 2), j & 1));
        for (int j = 0; j < 2 * n_or; ++j) want = join(want, code(1, 0, j & 1));
        for (int s = 0; s < sweeps; ++s) {
            g_t = (uint32_t)s;
            g_ended = g_steps = 0;
            g_reps.assign(h->lay.g.size(), {});
            for (size_t k = 0; k < h->lay.g.size(); ++k) {
                const Group &g = h->lay.g[k];
                g_reps[k].resize(g.n_rep);
                for (int64_t r = 0; r < g.n_rep; ++r) energies(k)[r] = NAN;
                double *scr = reinterpret_cast<double *>(h->scratch + g.o_scr);
                for (int64_t r = 0; r < g.n_rep * std::max(g.n_pb_sweep, 1); ++r) scr[r] = NAN;
            }
            if (hsg_sweep(h, 1, nullptr) != HSG_OK) bad(hsg_last_error());
            for (size_t k = 0; k < g_reps.size(); ++k)
                for (const Rep &x : g_reps[k])
                    if (x.seq != want || x.n != 2 * (n_hb + n_or)) bad("a replica got other half-sweeps");
            if (overlap == 2 && g_steps != 2) bad("no halves");
            if (g_ended != (int)sz.n_replicas) bad("ladders left out, or walked twice");
            if (*reinterpret_cast<uint32_t *>(h->state) != (uint32_t)s + 1) bad("the counter was not advanced");
        }
        out = g_bad.empty() ? "ok" : g_bad;
        hsg_destroy(h);
    }
    for (int k = 0; k < 4; ++k) munmap(buf[k], bytes[k] + 1);
    return out;
}

}  // namespace

int main()
{
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        std::cout << run(in) << "\n";
    }
    return 0;
}
