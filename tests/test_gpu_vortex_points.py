"""Vortex points against 64-bit arithmetic on the exact cofactors: weights and coordinates are not negative, so nothing
cancels, and a binary32 point lies within one unit of its last place of the 64-bit value (half a unit of rounding, and
room for a 64-bit value next to a tie)."""
import numpy as np
import pytest

from oracle import vortex as OV
from paper_2011_08697_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2011_08697_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)


@pytest.mark.parametrize("kind", ["noise", "ties", "waves", "large", "uneven"])
def test_points_to_the_last_place(kind):
    nt, nz, ny, nx = 3, 4, 5, 67
    rng = np.random.default_rng(11)
    full = (nt, 2, nz, ny, nx)
    if kind == "noise":
        f = rng.normal(size=full)
    elif kind == "ties":
        f = rng.integers(-1, 2, size=full)
    elif kind == "waves":
        f = synth.random_waves_3d(nx, ny, nz, nt, K=4, seed=nx)
    elif kind == "large":  # up to the 31 bits allowed
        f = 2047.9 * rng.uniform(-1, 1, size=full)
    else:  # cofactors of very different size
        f = rng.choice([-1.0, 1.0], size=full) * 2.0 ** rng.uniform(-19, 10.9, size=full)
    f = np.ascontiguousarray(f, np.float32)
    r = F.track_vortex3d(torch.from_numpy(f).to(DEV))
    torch.cuda.synchronize()
    o = OV.track_vortex(f)
    assert r["n_hits"] == o.n_hits > 100
    assert np.array_equal(r["tri_id"].cpu().numpy(), o.tri_id)
    pos = r["pos"].cpu().numpy()
    unit = np.spacing(np.abs(o.pos).astype(np.float32)).astype(np.float64)
    assert np.all(np.abs(pos.astype(np.float64) - o.pos) <= unit)
