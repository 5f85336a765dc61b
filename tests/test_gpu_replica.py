"""Sweeps of small lattices with a replica's spins in LDS (the automatic choice up
to L = 22) against single half-sweep launches (kernel variant 1, the gather kernel):
the same spins, temperature maps and acceptances bit for bit, the energies to
rounding. Sums of at most 3 L^3 float64 terms of order 1 in two orders differ by
less than 3 L^3 2^-53 of their absolute sum, a few 1e-12 of |E|."""

import numpy as np
import pytest
import torch

from paper_1204_6192_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hsg():
    from paper_1204_6192_amd import hsg as mod
    return mod


def _run(hsg, groups, variant, storage, n_hb, n_or, math, sweeps):
    lat = hsg.Lattice(groups, storage=storage, n_hb=n_hb, n_or=n_or, seed=inputs.PHILOX_KEY_BASE + 90)
    lat.set_kernel(variant)
    lat.set_math(math)
    lat.sweep(sweeps)
    out = [t.cpu() for t in (lat.get_spins(), lat.get_temp_map(), lat.get_pt_accepts(), lat.get_energies())]
    E = lat.measure_energy().cpu()
    lat.close()
    return out, E


def _check(a, b, E):
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])
    assert torch.allclose(a[3], b[3], rtol=1e-11, atol=1e-9)
    assert torch.allclose(a[3], E, rtol=1e-11, atol=1e-9)


# (L, samples, copies, rungs): one wave per replica (4), rows that a pair straddles
# (6, 10, 14, 18, 22), planes that do not divide the threads' share (12, 14, 18, 22),
# 1024 threads per replica (few replicas), 512 (512 replicas) and 256 (more), the
# largest that fits LDS (22)
@pytest.mark.parametrize("L,D,O,T", [(4, 3, 2, 5), (6, 1, 1, 1), (8, 2, 2, 3), (10, 130, 2, 4), (12, 70, 2, 4),
                                     (14, 70, 2, 4), (14, 1, 2, 2), (16, 2, 2, 2), (16, 64, 2, 4), (18, 1, 2, 3),
                                     (18, 64, 2, 4), (20, 1, 1, 2), (22, 1, 2, 2)])
@pytest.mark.parametrize("storage,field,couplings,n_hb,n_or,math",
                         [("f32", None, "gaussian", 1, 4, 0), ("f32", ("gaussian", 0.2), "bimodal", 2, 1, 0),
                          ("bf16", ("gaussian", 0.1), "gaussian", 1, 0, 1), ("f16", None, "bimodal", 1, 3, 0),
                          ("qangle", None, "gaussian", 0, 2, 0)])
def test_replica_sweeps_bit_identical(hsg, L, D, O, T, storage, field, couplings, n_hb, n_or, math):
    rng = np.random.Generator(np.random.Philox(inputs.INSTANCE_SEED_BASE + 90))
    g = inputs.make_group(rng, L, D, O, inputs.geometric_ladder(0.1, 0.6, T), couplings=couplings, field=field)
    a, E = _run(hsg, [g], 0, storage, n_hb, n_or, math, 2)
    b, _ = _run(hsg, [g], 1, storage, n_hb, n_or, math, 2)
    _check(a, b, E)


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_replica_sweeps_of_several_sizes(hsg, storage):
    """Eleven lattice sizes in one handle: more than one launch takes, several
    replicas per work-group for the smallest, sizes on both sides of the limit, with
    and without a field and +-1 couplings."""
    rng = np.random.Generator(np.random.Philox(inputs.INSTANCE_SEED_BASE + 91))
    groups, uid = [], 0
    for k, L in enumerate((4, 6, 8, 10, 12, 14, 16, 20, 22, 24, 26)):
        groups.append(inputs.make_group(rng, L, 1 + k % 3, 2, inputs.geometric_ladder(0.1, 0.5, 3),
                                        couplings=("gaussian", "bimodal")[k % 2],
                                        field=("gaussian", 0.1) if k % 3 == 1 else None, sample_uid_base=uid))
        uid += 3
    a, E = _run(hsg, groups, 0, storage, 1, 4, 0, 3)
    b, _ = _run(hsg, groups, 1, storage, 1, 4, 0, 3)
    _check(a, b, E)


# L = 4, four replicas per wave: one replica, remainders, several groups, a launch of its
# own beside other sizes (4100 replicas) and one with them (3)
@pytest.mark.parametrize("sizes", [((4, 1, 1, 1),), ((4, 4097, 1, 1),), ((4, 5, 1, 1), (4, 2, 2, 3)),
                                   ((4, 1025, 2, 2), (8, 2, 2, 3)), ((4, 3, 1, 1), (6, 2, 1, 3))])
@pytest.mark.parametrize("storage,field,couplings,n_hb,n_or,math",
                         [("f32", None, "gaussian", 1, 4, 0), ("f16", ("gaussian", 0.2), "bimodal", 2, 1, 1),
                          ("qangle", None, "gaussian", 1, 0, 0)])
def test_smallest_lattices(hsg, sizes, storage, field, couplings, n_hb, n_or, math):
    rng = np.random.Generator(np.random.Philox(inputs.INSTANCE_SEED_BASE + 98))
    groups, uid = [], 0
    for L, D, O, T in sizes:
        groups.append(inputs.make_group(rng, L, D, O, inputs.geometric_ladder(0.1, 0.6 if T > 1 else 0.1, T),
                                        couplings=couplings, field=field, sample_uid_base=uid))
        uid += D
    a, E = _run(hsg, groups, 0, storage, n_hb, n_or, math, 2)
    b, _ = _run(hsg, groups, 1, storage, n_hb, n_or, math, 2)
    _check(a, b, E)
