"""Batches that hold series of both 2D emission forms: dense series (tiled) beside sparse ones (listed, where they share
more than 1.5M vertices), empty and tiny series between them, values beyond 2^24, both sides of the bound: every series
as from its own call in the tiled form, which the oracle tests pin."""
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
TILED = 4  # FTK_DEBUG_TILED_EMIT
KEYS = ("face_id", "pos", "mu", "type", "flags", "label")
SHARED = 1500000  # vertices of the sparse series that pay for their launches


def _noise(nt, ny, nx, seed, scale=1.0, comps=0):
    shape = (nt, comps, ny, nx) if comps else (nt, ny, nx)
    return (scale * np.random.default_rng(seed).standard_normal(shape)).astype(np.float32)


def _few(nt, ny, nx, seed):
    """A ramp with bumps: few hits for its vertices."""
    f = np.broadcast_to(np.arange(nx, dtype=np.float32), (nt, ny, nx)).copy()
    rng = np.random.default_rng(seed)
    for _ in range(nt * 6):
        f[rng.integers(nt), rng.integers(ny), rng.integers(nx)] += 5.0
    return f


def _few_vectors(nt, ny, nx, seed, scale):
    u = np.zeros((nt, 2, ny, nx), np.float32)
    u[:, 0] = 1.0
    rng = np.random.default_rng(seed)
    for _ in range(nt * 4):
        y, x = rng.integers(ny - 8), rng.integers(nx - 8)
        u[rng.integers(nt), :, y:y + 6, x:x + 6] = scale * rng.standard_normal((2, 6, 6))
    return u


BATCHES = {
    "mixed": (0, lambda: [_few(3, 700, 400, 1), _noise(9, 75, 131, 2), np.zeros((3, 8, 70), np.float32),
                          _few(4, 300, 500, 3), _noise(2, 3, 5, 4), _few(2, 333, 131, 5), _noise(4, 33, 64, 6)]),
    "blobs": (0, lambda: [synth.moving_gaussians_2d(200, 150, 12, 12, seed=1, noise_std=1e-3),
                          synth.moving_gaussians_2d(300, 200, 27, 24, seed=3)]),
    "wide": (1, lambda: [_few_vectors(5, 400, 500, 1, 2.0e4), _noise(6, 33, 70, 2, 2.0e4, 2), _few_vectors(3, 300, 700, 3, 1.0)]),
    # 1500 * 500 * 2 vertices are the bound itself: all tiled; a step more, both forms
    "at_the_bound": (0, lambda: [_noise(4, 40, 90, 1), _few(2, 1500, 500, 2)]),
    "beyond_the_bound": (0, lambda: [_noise(4, 40, 90, 1), _few(3, 1500, 500, 2)]),
}


@pytest.mark.parametrize("name", sorted(BATCHES))
def test_both_forms_in_one_batch(name):
    kind, make = BATCHES[name]
    ts = [torch.from_numpy(np.ascontiguousarray(f)).to(DEV) for f in make()]
    one = [F.track_cp2d(t, kind=kind, outputs=F.OUT_ALL, debug=TILED) for t in ts]
    vertices = [t.numel() // (2 if kind else 1) for t in ts]
    few = [4 * r["n_hits"] < v for r, v in zip(one, vertices)]
    listed = sum(v for v, s in zip(vertices, few) if s)
    assert any(few) and not all(few)  # both forms, where the sparse series suffice for theirs
    assert (listed > SHARED) == (name != "at_the_bound")
    assert (one[0]["stats"]["wide_path"] == 1) == (name == "wide")
    for outputs in (F.OUT_ALL, F.OUT_POS):
        got = F.track_cp2d_batched(ts, kind=kind, outputs=outputs)
        for g, r in zip(got, one):
            assert g["n_hits"] == r["n_hits"] and g["n_trajectories"] == r["n_trajectories"]
            for k in KEYS:
                if outputs == F.OUT_ALL or k in ("face_id", "pos"):
                    assert torch.equal(g[k], r[k]), k
            for k in ("cells_linked", "fp64_fallbacks", "degenerate_sublocations"):
                assert g["stats"][k] == r["stats"][k], k


def test_mixed_batch_matches_the_oracle():
    fields = [_noise(5, 20, 70, 2), _few(2, 1100, 700, 3)]
    ts = [torch.from_numpy(f).to(DEV) for f in fields]
    for f, r in zip(fields, F.track_cp2d_batched(ts)):
        assert_full_parity(r, O.track(f))
