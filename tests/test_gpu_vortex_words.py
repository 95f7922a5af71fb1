"""Vortex surfaces at the edges of their 64-vertex words and with many positive triangles per vertex, against the oracle:
ids, labels and component count bit-exact."""
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


@pytest.mark.parametrize("shape", [(2, 2, 2, 2), (2, 2, 3, 63), (2, 3, 2, 64), (3, 2, 2, 65), (2, 2, 2, 66),
                                   (2, 2, 2, 129), (3, 4, 5, 6)])
@pytest.mark.parametrize("kind", ["noise", "ties", "zeros", "waves", "large"])
def test_words(shape, kind):
    nt, nz, ny, nx = shape
    rng = np.random.default_rng(nx + ny)
    full = (nt, 2, nz, ny, nx)
    if kind == "noise":
        f = rng.normal(size=full)
    elif kind == "ties":
        f = rng.integers(-1, 2, size=full)
    elif kind == "zeros":
        f = np.zeros(full)
        f[:, :, :, :, nx // 2:] = rng.integers(-2, 3, size=f[:, :, :, :, nx // 2:].shape)
    elif kind == "waves":
        f = synth.random_waves_3d(nx, ny, nz, nt, K=4, seed=nx)
    else:
        f = 2047.0 * rng.uniform(-1, 1, size=full)
    f = np.ascontiguousarray(f, np.float32)
    r = F.track_vortex3d(torch.from_numpy(f).to(DEV))
    torch.cuda.synchronize()
    o = OV.track_vortex(f)
    assert r["n_hits"] == o.n_hits and r["n_components"] == o.n_components
    assert np.array_equal(r["tri_id"].cpu().numpy(), o.tri_id)
    assert np.array_equal(r["label"].cpu().numpy(), o.label)
    pos = r["pos"].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(pos - o.pos) <= 1e-5 * np.maximum(1.0, np.abs(o.pos)))
