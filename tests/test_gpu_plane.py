"""Pairs of half-sweeps, and two over-relaxation pairs, in one walk of whole planes
against single half-sweep launches (kernel variant 1, the gather kernel): the same
spins, temperature maps and acceptances bit for bit, the energies to rounding. Sums
of at most 3 L^3 float64 terms of order 1 in two orders differ by less than
3 L^3 2^-53 of their absolute sum, a few 1e-11 of |E| at L = 64 at worst."""

import numpy as np
import pytest
import torch

from paper_1204_6192_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hsg():
    from paper_1204_6192_amd import hsg as mod
    return mod


def _group(L, D, O, T, field, couplings, uid=0):
    rng = np.random.Generator(np.random.Philox(inputs.INSTANCE_SEED_BASE + 97))
    one = inputs.make_group(rng, L, D, 1, inputs.geometric_ladder(0.1, 0.6, 1), couplings=couplings, field=field)
    return inputs.Group(L=L, n_samples=D, n_copies=O, temps=inputs.geometric_ladder(0.1, 0.6, T), J=one.J, H=one.H,
                        spins0=np.broadcast_to(one.spins0, (D, O, T, 3, L ** 3)).copy(),
                        coupling_kind=one.coupling_kind, sample_uid_base=uid)


def _run(hsg, groups, variant, storage, n_hb, n_or, math, batch=None, overlap=False):
    lat = hsg.Lattice(groups, storage=storage, n_hb=n_hb, n_or=n_or, seed=inputs.PHILOX_KEY_BASE + 97)
    lat.set_kernel(variant)
    lat.set_math(math)
    if batch is not None:
        lat.set_batch(batch)
    if overlap:
        lat.set_overlap(True)
    lat.sweep(2)
    out = [lat.get_spins(), lat.get_temp_map(), lat.get_pt_accepts(), lat.get_energies()]
    E = lat.measure_energy()
    torch.cuda.synchronize()
    lat.close()
    return out, E


# (L, samples, copies, rungs): every plane size class -- idle lanes (26, 30, 34, 36, 46,
# 62), whole waves (24, 32, 64), rows that a pair straddles (L % 4 = 2) -- at replica
# counts on both sides of the lines that the choice of the walk draws
@pytest.mark.parametrize("L,D,O,T", [(24, 1, 2, 3), (24, 2, 1, 100), (28, 1, 2, 97), (26, 1, 2, 48), (26, 2, 2, 64), (28, 1, 1, 1), (30, 1, 2, 128),
                                     (32, 2, 2, 3), (32, 3, 2, 86), (32, 5, 2, 110), (34, 1, 2, 64), (36, 1, 2, 95),
                                     (36, 1, 2, 96), (44, 2, 2, 64), (46, 2, 1, 128), (48, 1, 2, 96), (62, 1, 1, 97),
                                     (62, 1, 2, 129), (64, 2, 1, 97), (64, 2, 1, 128)])
@pytest.mark.parametrize("storage,field,couplings,n_hb,n_or,math",
                         [("f32", None, "gaussian", 1, 4, 0), ("f32", ("gaussian", 0.2), "bimodal", 2, 1, 0),
                          ("bf16", ("gaussian", 0.1), "gaussian", 1, 0, 1), ("f16", None, "bimodal", 1, 3, 0),
                          ("qangle", None, "gaussian", 1, 2, 0), ("bf16", None, "gaussian", 1, 0, 0)])
def test_plane_march_bit_identical(hsg, L, D, O, T, storage, field, couplings, n_hb, n_or, math):
    g = _group(L, D, O, T, field, couplings)
    a, E = _run(hsg, [g], 0, storage, n_hb, n_or, math)
    b, _ = _run(hsg, [g], 1, storage, n_hb, n_or, math)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])
    assert torch.allclose(a[3], b[3], rtol=1e-10, atol=1e-9)
    assert torch.allclose(a[3], E, rtol=1e-10, atol=1e-9)


@pytest.mark.parametrize("storage,n_or", [("f32", 4), ("bf16", 3), ("f16", 0)])
def test_plane_march_of_several_sizes(hsg, storage, n_or):
    """Several sizes in one handle, in batches that leave a remainder and as two
    halves on two streams: the same result, energies included."""
    groups, uid = [], 0
    for L, D, O, T in ((24, 2, 2, 7), (32, 2, 2, 5), (36, 2, 2, 64), (40, 2, 2, 48)):
        groups.append(_group(L, D, O, T, None, "gaussian", uid))
        uid += D
    ref, _ = _run(hsg, groups, 0, storage, 1, n_or, 0)
    for kw in ({"batch": 50}, {"batch": 200}, {"overlap": True}):
        got, _ = _run(hsg, groups, 0, storage, 1, n_or, 0, **kw)
        for x, y in zip(got, ref):
            assert torch.equal(x, y)


# few replicas: gather passes, with one and several slots per work item, and with one
# kind of pass on each side of its line (24 of 100, 32 of 60, 40 of 60 replicas)
@pytest.mark.parametrize("L,D,O,T", [(24, 1, 1, 1), (24, 2, 2, 25), (28, 1, 2, 12), (32, 2, 2, 15), (36, 2, 2, 3),
                                     (40, 3, 2, 10), (64, 1, 2, 2), (64, 2, 1, 8), (128, 1, 1, 2)])
@pytest.mark.parametrize("storage,field,couplings,n_hb,n_or,math",
                         [("f32", None, "gaussian", 1, 4, 0), ("f32", ("gaussian", 0.2), "bimodal", 2, 1, 0),
                          ("bf16", None, "gaussian", 1, 3, 1), ("qangle", None, "bimodal", 1, 0, 0)])
def test_few_replicas_bit_identical(hsg, L, D, O, T, storage, field, couplings, n_hb, n_or, math):
    g = _group(L, D, O, T, field, couplings)
    a, E = _run(hsg, [g], 0, storage, n_hb, n_or, math)
    b, _ = _run(hsg, [g], 2, storage, n_hb, n_or, math)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])
    assert torch.allclose(a[3], b[3], rtol=1e-10, atol=1e-9)
    assert torch.allclose(a[3], E, rtol=1e-10, atol=1e-9)
    for kw in ({"batch": 3}, {"overlap": True}):
        c, _ = _run(hsg, [g], 0, storage, n_hb, n_or, math, **kw)
        for x, y in zip(c, a):
            assert torch.equal(x, y)


# quantised angles, where two pairs go in one launch only in the walk of whole planes:
# batches, a remainder and halves of so few replicas that their passes take another
# route than the group's, which decides where the energies are left
@pytest.mark.parametrize("L,D,O,T,field,kw",
                         [(32, 8, 1, 65, None, {"batch": 64}), (32, 5, 1, 107, None, {"batch": 500}),
                          (24, 8, 2, 33, None, {"batch": 50}), (28, 3, 2, 64, ("gaussian", 0.1), {"batch": 72}),
                          (32, 2, 2, 32, ("gaussian", 0.1), {"overlap": True}),
                          (24, 3, 1, 66, ("gaussian", 0.1), {"overlap": True})])
@pytest.mark.parametrize("n_or", [2, 4])
def test_energies_of_parts_of_a_size(hsg, L, D, O, T, field, kw, n_or):
    g = _group(L, D, O, T, field, "gaussian")
    a, E = _run(hsg, [g], 0, "qangle", 1, n_or, 0, **kw)
    b, _ = _run(hsg, [g], 1, "qangle", 1, n_or, 0)
    whole, _ = _run(hsg, [g], 0, "qangle", 1, n_or, 0)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])
    assert torch.allclose(a[3], E, rtol=1e-10, atol=1e-9)
    assert torch.equal(a[3], whole[3])


# many sites of L >= 128: bands of two rows by default, several replicas per work-group
# (L = 144: three, of 216 threads)
@pytest.mark.parametrize("L,D,T,storage,field", [(128, 3, 4, "f32", None), (128, 1, 12, "f16", ("gaussian", 0.1)),
                                                 (144, 2, 4, "qangle", None), (144, 1, 10, "bf16", None)])
def test_flat_bands_bit_identical(hsg, L, D, T, storage, field):
    g = _group(L, D, 1, T, field, "gaussian")
    lat = hsg.Lattice([g], storage=storage)
    assert lat.get_geometry(0)[0] == 2
    lat.close()
    a, E = _run(hsg, [g], 2, storage, 1, 1, 0)
    b, _ = _run(hsg, [g], 1, storage, 1, 1, 0)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])
    assert torch.allclose(a[3], b[3], rtol=1e-10, atol=1e-9)
    assert torch.allclose(a[3], E, rtol=1e-10, atol=1e-9)


# sign-bit couplings are too few bytes to be worth the halo rows of flat bands
@pytest.mark.parametrize("L,rows", [(128, 8), (144, 6)])
def test_sign_bits_keep_tall_bands(hsg, L, rows):
    lat = hsg.Lattice([_group(L, 1, 1, 12, None, "bimodal")], storage="qangle")
    assert lat.get_geometry(0)[0] == rows
    lat.close()


# both sides of the walk's lines with sign bits (the walk: the second of each pair)
@pytest.mark.parametrize("L,n,storage,field", [(36, 384, "f16", None), (36, 385, "f16", None), (40, 257, "qangle", None),
                                               (40, 256, "qangle", None), (44, 287, "f32", ("gaussian", 0.2)),
                                               (44, 288, "f32", ("gaussian", 0.2)), (52, 223, "bf16", None),
                                               (52, 224, "bf16", None)])
def test_sign_bits_bit_identical(hsg, L, n, storage, field):
    g = _group(L, n, 1, 1, field, "bimodal")
    a, E = _run(hsg, [g], 0, storage, 1, 1, 0)
    b, _ = _run(hsg, [g], 1, storage, 1, 1, 0)
    assert torch.equal(a[0], b[0])
    assert torch.allclose(a[3], b[3], rtol=1e-10, atol=1e-9)
    assert torch.allclose(a[3], E, rtol=1e-10, atol=1e-9)
