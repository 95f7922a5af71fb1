"""The 2D emission of listed hits (a lane per hit) where its parts end: segments of one vertex and of full width, few and
many hits of a segment (the search for a partner's index), hits in no multiple of a wavefront, tied and vector fields,
values beyond 2^24, series of a batch without hits: identical to the tiled form, which the oracle tests pin."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2011_08697_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)
TILED, SPARSE = 4, 8  # FTK_DEBUG_TILED_EMIT, FTK_DEBUG_SPARSE_EMIT
KEYS = ("face_id", "pos", "mu", "type", "flags", "label")


def _same(a, b):
    assert a["n_hits"] == b["n_hits"] and a["n_trajectories"] == b["n_trajectories"]
    for k in KEYS:
        assert torch.equal(a[k], b[k]), k
    for k in ("cells_linked", "fp64_fallbacks", "degenerate_sublocations", "wide_path"):
        assert a["stats"][k] == b["stats"][k], k


def _fields(nx, ny, nt, seed):
    rng = np.random.default_rng(seed)
    white = rng.standard_normal((nt, ny, nx)).astype(np.float32)
    rare = np.broadcast_to(np.arange(nx, dtype=np.float32), (nt, ny, nx)).copy()
    rare[:, ny // 2, nx // 2] += 5.0  # a few hits in a graded field
    tied = rng.integers(-1, 2, size=(nt, 2, ny, nx)).astype(np.float32)
    return [(white, 0), (rare, 0), (tied, 1), (2.0e4 * rng.standard_normal((nt, 2, ny, nx)).astype(np.float32), 1)]


@pytest.mark.parametrize("nx,ny,nt", [(2, 2, 2), (3, 70, 4), (63, 9, 3), (64, 5, 5), (65, 4, 2), (129, 33, 6)])
def test_listed_hits_equal_the_tiled_form(nx, ny, nt):
    for f, kind in _fields(nx, ny, nt, nx):
        t = torch.from_numpy(f).to(DEV)
        a = F.track_cp2d(t, kind=kind, outputs=F.OUT_ALL, debug=TILED)
        b = F.track_cp2d(t, kind=kind, outputs=F.OUT_ALL, debug=SPARSE)
        _same(a, b)
        _same(a, F.track_cp2d(t, kind=kind, outputs=F.OUT_ALL))


def test_batch_with_empty_and_single_hit_blocks():
    rng = np.random.default_rng(9)
    fields = [np.zeros((3, 8, 70), np.float32), rng.standard_normal((4, 9, 130)).astype(np.float32),
              _fields(65, 20, 4, 1)[1][0], np.zeros((2, 2, 2), np.float32), rng.standard_normal((2, 3, 5)).astype(np.float32)]
    ts = [torch.from_numpy(f).to(DEV) for f in fields]
    a = F.track_cp2d_batched(ts, outputs=F.OUT_ALL, debug=TILED)
    b = F.track_cp2d_batched(ts, outputs=F.OUT_ALL, debug=SPARSE)
    for x, y, t in zip(a, b, ts):
        _same(x, y)
        _same(x, F.track_cp2d(t, outputs=F.OUT_ALL, debug=SPARSE))
