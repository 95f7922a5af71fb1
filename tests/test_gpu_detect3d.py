"""3D detection and emission at the edges of their tiles (16 x 8 x 4 anchors, wavefronts of 64 along x, runs of steps),
on fields that the sign facts decide wholly, partly and not at all, one-shot and streamed, against the oracle."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2011_08697_amd import synth
from tests.parity import assert_full_parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2011_08697_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)


def fields(shape, seed):
    nt, nz, ny, nx = shape
    rng = np.random.default_rng(seed)
    yield "noise", 1e-2 * rng.normal(size=shape)
    yield "integers", rng.integers(-1, 2, size=shape)
    yield "zero", np.zeros(shape)
    g = np.zeros(shape)  # flat but for a few vertices, at the grid's corners and inside
    for p in ((0, 0, 0, 0), (-1, -1, -1, -1), (0, nz // 2, ny // 2, nx // 2), (-1, 0, -1, nx // 2)):
        g[p] = 2.0 ** -19
    yield "spots", g
    yield "wide", 40.0 * rng.normal(size=shape)
    x = np.arange(nx)[None, None, None, :] + np.zeros(shape)
    yield "ramp", x + 0.3 * rng.normal(size=shape) * (np.arange(ny)[None, None, :, None] == ny - 1)


@pytest.mark.parametrize("shape", [(2, 2, 2, 2), (3, 4, 8, 16), (3, 5, 9, 17), (2, 6, 10, 63), (2, 3, 7, 65),
                                   (4, 4, 9, 33), (9, 2, 3, 5)])
def test_tile_edges(shape):
    for name, f in fields(shape, sum(shape)):
        f = f.astype(np.float32)
        ref = O.track(f, n=3, kind=0)
        for slab in (0, 1, 3, 64):
            r = F.track_cp3d(torch.from_numpy(f).to(DEV), slab_depth=slab)
            torch.cuda.synchronize()
            assert_full_parity(r, ref)
        tr = F.Tracker(3, (shape[3], shape[2], shape[1]))
        for t in range(shape[0]):
            tr.push(torch.from_numpy(f[t].copy()).to(DEV))
        r = tr.finish()
        torch.cuda.synchronize()
        if ref.n_hits:
            assert_full_parity(r, ref)
        else:  # a stream without hits never allocates its output arrays
            assert r["n_hits"] == 0 and r["n_trajectories"] == 0
        tr.close()


def test_mixed_tiles():
    """Blobs on a grid of several tiles: empty, partly and wholly tested tile-steps side by side."""
    f = synth.moving_gaussians_3d(70, 41, 23, 6, 5, sigma=(2.0, 4.0), seed=8)
    assert_full_parity(F.track_cp3d(torch.from_numpy(f).to(DEV)), O.track(f, n=3, kind=0))


def test_errors_wherever_they_are():
    for p in ((0, 0, 0, 0), (2, 4, 9, 69), (1, 3, 8, 64), (2, 0, 7, 15)):
        for bad, status in ((np.nan, 2), (np.inf, 2), (2.0 ** 23, 3)):
            f = np.zeros((3, 5, 10, 70), np.float32)
            f[p] = bad
            with pytest.raises(F.FtkError) as e:
                F.track_cp3d(torch.from_numpy(f).to(DEV))
            assert e.value.status == status, (p, bad)
