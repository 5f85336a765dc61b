"""The tile-local chain at the edges of what its launch choices depend on, against the
oracle's chain of the same tiles (bounds as in test_gpu_parity._trajectory): planes
padded against bank conflicts (8^3, 4^3 with several replicas in half a wave, 16 x 4 x 4
with few), left as they are where padding would pass 64 KiB (16 x 4 x 4 with nine
replicas per work-group and a remainder), one tile without a halo, and codecs whose
own sites are kept in two forms."""

import numpy as np
import pytest

from paper_1204_6192_amd import inputs
from test_gpu_parity import _trajectory, hsg  # noqa: F401 (the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,tiles,O,T,storage,field", [
    (16, (8, 8, 8, 1), 2, 2, "f32", True), (16, (8, 8, 8, 1), 1, 7, "bf16", False), (8, (4, 4, 4, 1), 2, 4, "f32", True),
    (16, (16, 4, 4, 1), 2, 1, "f32", False), (16, (16, 4, 4, 2), 2, 5, "f32", True), (16, (16, 4, 4, 1), 1, 10, "f16", False),
    (8, (8, 8, 8, 1), 1, 3, "f32", True), (8, (8, 4, 2, 1), 1, 3, "qangle", False)])
def test_tile_launch_choices(hsg, oracle_lib, L, tiles, O, T, storage, field):  # noqa: F811
    rng = np.random.Generator(np.random.Philox(inputs.INSTANCE_SEED_BASE + 98))
    g = inputs.make_group(rng, L, 2, O, inputs.geometric_ladder(0.1, 0.3, T),
                          field=("gaussian", 0.2) if field else None)
    inst = inputs.Instance(groups=[g], seed=inputs.PHILOX_KEY_BASE + 98, n_hb=1, n_or=2)
    kw = {} if storage == "f32" else dict(storage=storage, spin_tol=None)
    _trajectory(hsg, oracle_lib, inst, 3, tiles=tiles, **kw)
