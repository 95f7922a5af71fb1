"""2D detection at the edges of its tiles (a wavefront's 64 x 8 anchors, slabs of steps, workgroups of 8 to 32 rows) and
of its number ranges, against the oracle: bit-exact faces, types and labels."""
import numpy as np
import pytest

from oracle import oracle as O
from tests.parity import assert_full_parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2011_08697_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)


def run(field, kind, **kw):
    r = F.track_cp2d(torch.from_numpy(np.ascontiguousarray(field)).to(DEV), kind=kind, **kw)
    torch.cuda.synchronize()
    return r


@pytest.mark.parametrize("nx", [2, 63, 64, 65, 66, 128, 130])
@pytest.mark.parametrize("ny,nt,slab", [(2, 2, 0), (7, 3, 1), (8, 4, 3), (9, 2, 2), (17, 5, 4), (33, 3, 16)])
def test_tile_edges(nx, ny, nt, slab):
    """Smooth noise (few exact zeros) and small integers (mostly exact zeros), scalar and vector."""
    rng = np.random.default_rng(nx * 1000 + ny * 10 + nt)
    for kind, shape in ((0, (nt, ny, nx)), (1, (nt, 2, ny, nx))):
        for f in (rng.normal(size=shape), rng.integers(-1, 2, size=shape)):
            f = f.astype(np.float32)
            assert_full_parity(run(f, kind, slab_depth=slab), O.track(f, n=2, kind=kind))


@pytest.mark.parametrize("scale", [15.9, 16.1, 2047.0, 2.0 ** 30, 2.0 ** 41 * 0.99])
def test_sign_facts_and_magnitudes(scale):
    """Components around and beyond 2^24 (up to just below 2^62), with regions of one strict sign, of zeros, and sign
    changes on tile borders; pairs of equal and opposite vectors give exactly zero determinants at every magnitude."""
    rng = np.random.default_rng(5)
    nt, ny, nx = 4, 27, 140
    u = rng.normal(size=(nt, 2, ny, nx))
    u[:, 0, :, 64:] = np.abs(u[:, 0, :, 64:])
    u[:, :, 8:16, :64] = 0.0
    u[:, 0, 16:, :64] = -np.abs(u[:, 0, 16:, :64])
    u[:, 0, 16, 63] *= -1.0
    u[:, :, 3, 5:9] = u[:, :, 4, 5:9]
    u[1:, :, 5, 20:30] = -u[:-1, :, 5, 20:30]
    u *= scale / np.abs(u).max()
    u = u.astype(np.float32)
    assert_full_parity(run(u, 1), O.track(u, n=2, kind=1))


def test_range_and_nonfinite_reported_wherever_they_are():
    for y, x in ((0, 0), (7, 63), (8, 64), (16, 65), (26, 139)):
        for t in (0, 3):
            for bad, status in ((np.nan, 2), (np.inf, 2), (2.0 ** 43, 3)):
                u = np.ones((4, 2, 27, 140), np.float32)
                u[t, 1, y, x] = bad
                with pytest.raises(F.FtkError) as e:
                    run(u, 1)
                assert e.value.status == status, (y, x, t, bad)
