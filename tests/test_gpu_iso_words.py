"""Isovolume tracking at the edges of its 64-vertex words and on fields with many components, against the oracle:
crossings, labels (from vertex components), component count and tetrahedra bit-exact."""
import numpy as np
import pytest

from oracle import iso as OI

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2011_08697_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)


@pytest.mark.parametrize("shape", [(2, 2, 2, 2), (2, 2, 3, 63), (2, 3, 2, 64), (3, 2, 2, 65), (2, 2, 2, 66),
                                   (2, 2, 2, 129), (4, 5, 6, 7)])
@pytest.mark.parametrize("kind", ["noise", "two_levels", "checker", "shells", "one_vertex", "plane_x"])
def test_components_and_words(shape, kind):
    nt, nz, ny, nx = shape
    rng = np.random.default_rng(nx * 7 + ny)
    t, z, y, x = np.meshgrid(*[np.arange(n) for n in shape], indexing="ij")
    if kind == "noise":
        f = rng.normal(size=shape)
    elif kind == "two_levels":  # every value on the level or below it
        f = rng.integers(0, 2, size=shape) - 1.0
    elif kind == "checker":  # the most runs and crossings
        f = ((x + y + z + t) & 1) - 0.5
    elif kind == "shells":  # nested components, some split by the grid's end
        f = np.cos(0.9 * (x % 64)) + 0.3 * y - 0.2 * z
    elif kind == "one_vertex":
        f = -np.ones(shape)
        f[-1, 0, -1, nx // 2] = 1.0
        f[0, 0, 0, nx - 1] = 1.0
    else:
        f = x - (nx - 1.5)
    f = f.astype(np.float32)
    r = F.track_iso3d(torch.from_numpy(f).to(DEV), 0.0)
    torch.cuda.synchronize()
    o = OI.track_iso(f, 0.0)
    assert r["n_hits"] == o.n_hits and r["n_components"] == o.n_components
    assert np.array_equal(r["edge_id"].cpu().numpy(), o.edge_id)
    assert np.array_equal(r["label"].cpu().numpy(), o.label)
    assert np.array_equal(r["tets"].cpu().numpy().reshape(-1, 4), np.asarray(o.tets).reshape(-1, 4))
    pos = r["pos"].cpu().numpy().astype(np.float64)
    assert np.all(np.abs(pos - o.pos) <= 1e-5 * np.maximum(1.0, np.abs(o.pos)))
