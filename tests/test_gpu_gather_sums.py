"""The measurements that gather (L % 4 = 2, where a pair of sites may straddle rows)
against the oracle on the GPU's own configurations: sizes whose site pairs leave the
last work-group of 128 or 256 partly idle, one and several work-groups, every storage.
Float64 sums of at most 3 L^3 exact or once-rounded terms of order 1 in two orders: an
overlap or wave-vector sum, divided by L^3, differs by less than 3 L^3 2^-53 < 2e-11 at
L = 38 at the very worst and by 1e-14 at random; energies by as much of |E|."""

import numpy as np
import pytest

from paper_1204_6192_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hsg():
    from paper_1204_6192_amd import hsg as mod
    return mod


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16", "qangle"])
@pytest.mark.parametrize("field", [None, ("gaussian", 0.2)])
def test_gathering_measurements(hsg, oracle_lib, storage, field):
    rng = np.random.Generator(np.random.Philox(inputs.INSTANCE_SEED_BASE + 94))
    groups, uid = [], 0
    for L, D in ((6, 2), (10, 1), (14, 2), (18, 1), (22, 1), (30, 1), (38, 1)):
        groups.append(inputs.make_group(rng, L, D, 4, inputs.geometric_ladder(0.1, 0.5, 2), field=field,
                                        sample_uid_base=uid))
        uid += D
    seed = inputs.PHILOX_KEY_BASE + 94
    lat = hsg.Lattice(groups, seed=seed, storage=storage)
    lat.sweep(3)
    E, q, km, po = (t.cpu().numpy() for t in (lat.measure_energy(), lat.measure_overlap(), lat.measure_kmodes(),
                                              lat.measure_pair_overlaps()))
    spins, maps = lat.get_spins().cpu().numpy(), lat.get_temp_map().cpu().numpy()
    at = dict.fromkeys(("s", "m", "E", "q", "km", "po"), 0)

    def part(key, a, n):
        at[key] += n
        return a[at[key] - n:at[key]]

    for g in groups:
        o = oracle_lib.Oracle.from_group(g, seed=seed)
        o.spins = part("s", spins, g.n_slots * 3 * g.N).astype(np.float64).reshape(o.spins.shape)
        o.slot_at_temp = np.ascontiguousarray(part("m", maps, g.n_slots).reshape(o.slot_at_temp.shape), dtype=np.int32)
        assert np.allclose(part("E", E, g.n_slots), o.measure_energy().reshape(-1), rtol=1e-12, atol=1e-10), g.L
        for key, got, want in (("q", q, o.measure_overlap()), ("km", km, o.measure_kmodes()),
                               ("po", po, o.measure_pair_overlaps())):
            want = want.reshape(-1)
            assert np.abs(part(key, got, want.size) - want).max() < 1e-12, (g.L, key)
    lat.close()
