"""Halves of the samples on two streams, and batches of replicas, on the routes that they
are for: the marches of every kind (kernel variant 4), and lattice sizes with the spins
in LDS beside them. Every replica gets the same updates in the same order and every
energy the same sum, so all results agree bit for bit with one stream and no batches."""

import numpy as np
import pytest
import torch

from paper_1204_6192_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hsg():
    from paper_1204_6192_amd import hsg as mod
    return mod


def _groups(sizes):
    rng = np.random.Generator(np.random.Philox(inputs.INSTANCE_SEED_BASE + 95))
    out, uid = [], 0
    for L, D, T in sizes:
        out.append(inputs.make_group(rng, L, D, 2, inputs.geometric_ladder(0.1, 0.3, T), sample_uid_base=uid))
        uid += D
    return out


def _results(lat):
    sums, trips, n = lat.get_stats()
    return [t.cpu() for t in (lat.get_spins(), lat.get_temp_map(), lat.get_energies(), lat.get_pt_accepts(), sums,
                              trips)] + [n, lat.get_state()]


def _same(a, b):
    return all(torch.equal(x, y) if isinstance(x, torch.Tensor) else x == y for x, y in zip(a, b))


@pytest.mark.parametrize("variant,sizes", [(4, ((8, 3, 4), (16, 2, 3), (36, 2, 2))),
                                           (0, ((8, 3, 4), (18, 2, 3), (24, 3, 5), (36, 2, 12))),
                                           (0, ((16, 2, 40), (32, 2, 128)))])
@pytest.mark.parametrize("storage,n_hb,n_or,pt_every", [("f32", 1, 4, 1), ("qangle", 2, 3, 2), ("bf16", 1, 0, 1)])
def test_halves_bit_identical(hsg, variant, sizes, storage, n_hb, n_or, pt_every):
    groups = _groups(sizes)
    res = []
    for overlap in (False, True):
        lat = hsg.Lattice(groups, storage=storage, n_hb=n_hb, n_or=n_or, pt_every=pt_every,
                          seed=inputs.PHILOX_KEY_BASE + 95)
        lat.set_kernel(variant)
        lat.set_stats(True)
        lat.set_overlap(overlap)
        lat.sweep(3)
        lat.set_overlap(False)  # one stream in between: only the first counter is stepped
        lat.sweep(2)
        lat.set_overlap(overlap)
        lat.sweep(1)
        res.append(_results(lat))
        lat.pt_exchange()
        res[-1].append(lat.get_temp_map().cpu())
        lat.close()
    assert _same(*res)


@pytest.mark.parametrize("storage", ["f32", "f16"])
def test_batches_bit_identical(hsg, storage):
    groups = _groups(((8, 3, 5), (16, 2, 3), (36, 1, 2), (6, 2, 2), (48, 2, 2)))
    res = []
    for batch in (-1, 1, 3, 7, 0):
        lat = hsg.Lattice(groups, storage=storage, seed=inputs.PHILOX_KEY_BASE + 96)
        lat.set_kernel(4 if batch != 7 else 3)
        lat.set_stats(True)
        lat.set_batch(batch)
        lat.sweep(4)
        res.append(_results(lat))
        lat.close()
    for k, r in enumerate(res[1:]):
        if k == 2:  # another kernel: the energies to rounding, and so the sums over them
            assert _same(r[:2] + r[3:4], res[0][:2] + res[0][3:4])
            assert torch.allclose(r[2], res[0][2], rtol=1e-11, atol=1e-9)
        else:
            assert _same(r, res[0]), k
