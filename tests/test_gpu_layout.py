"""The canonical arrays to the stored layout and back: spins at addresses that are
only 4-byte aligned take single accesses in place of 16-byte ones, and give the same
values; rows that a pair of half-indices straddles (L % 4 = 2) and the smallest
lattice; every codec. What comes back is the codec's rounding of what went in:
exactly for float32, to half a step of the code otherwise (2^-11 and 2^-8 of a
component of magnitude at most 1, renormalised; 10^-4 for quantised angles)."""

import numpy as np
import pytest
import torch

from paper_1204_6192_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,tol", [("f32", 0.0), ("f16", 2.0 ** -10), ("bf16", 2.0 ** -7), ("qangle", 1.5e-4)])
def test_spins_at_any_alignment(storage, tol):
    from paper_1204_6192_amd import hsg
    rng = np.random.Generator(np.random.Philox(inputs.INSTANCE_SEED_BASE + 93))
    groups, uid = [], 0
    for L in (4, 6, 10, 12, 18, 34):
        groups.append(inputs.make_group(rng, L, 2, 2, inputs.geometric_ladder(0.1, 0.3, 3), sample_uid_base=uid))
        uid += 2
    lat = hsg.Lattice(groups, storage=storage, seed=1)
    want = torch.cat([torch.from_numpy(g.spins0.reshape(-1)) for g in groups]).cuda()
    buf = torch.empty(want.numel() + 4, dtype=torch.float32, device="cuda")
    ref = None
    for off in (0, 1, 2, 3):
        lat.set_spins(torch.zeros_like(want))
        src = buf[off:off + want.numel()]
        src.copy_(want)
        lat.set_spins(src)
        torch.cuda.synchronize()
        dst = torch.full_like(buf, float("nan"))
        out = dst[off:off + want.numel()]
        hsg.check(hsg.lib.hsg_get_spins(lat.h, out.data_ptr(), torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        assert float((out - want).abs().max()) <= tol
        assert int(torch.isnan(dst).sum()) == 4  # nothing beside the array is written
        if ref is None:
            ref = out.clone()
        assert torch.equal(out, ref)
    lat.close()
