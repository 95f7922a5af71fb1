"""The post-processing at the edges of its parts, against the oracle: results dense enough for a lookup entry per vertex
and results that search vertex rows, more trajectories than a loop filter's samples, smoothing windows around and beyond
the tile's halo, loops of one type (no run start), runs over many words of 64 positions."""
import numpy as np
import pytest

from oracle import oracle as O
from oracle import post as P
from paper_2011_08697_amd import synth
from test_gpu_post import _check_simplified, _check_table, _dims, _track

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2011_08697_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)


def _white(shape, seed):
    return np.random.default_rng(seed).standard_normal(shape).astype(np.float32)


CASES = {
    "dense_2d": lambda: (_white((11, 75, 131), 1), 2),       # entries for labels and hits
    "mixed_2d": lambda: (synth.moving_gaussians_2d(150, 90, 9, 9, seed=3, noise_std=2e-4), 2),
    "dense_3d": lambda: (_white((4, 9, 11, 13), 2), 3),
    "sparse_3d": lambda: (synth.moving_gaussians_3d(30, 21, 19, 6, 5, seed=4), 3),
    "thin_2d": lambda: (_white((70, 2, 3), 5), 2),           # every face near a boundary hyperplane
}


@pytest.mark.parametrize("case", list(CASES))
def test_post_processing_matches_oracle_at_the_edges(case):
    f, n = CASES[case]()
    dims = _dims(f, n)
    g = _track(f, n)
    tr = O.track(f, n=n, kind=0)
    assert g["n_hits"] == tr.n_hits and tr.n_hits > 0
    tab_o, tab_g = P.traj_table(tr, n, dims), F.trajectory_table(g, dims)
    _check_table(tab_g, tab_o)
    if case == "dense_2d":
        assert tab_o["n"] > 8192
    for c in (0.0, 0.7501, 1e9):
        ext = np.abs((tab_o["t_max"] - tab_o["t_min"]) - c)
        got, want = F.filter_loops(g, tab_g, c).cpu().numpy(), P.filter_loops(tr, tab_o, c)
        near = np.isin(tr.label, tab_o["label"][ext < 1e-3])  # FP32 extents may fall on either side there
        assert np.array_equal(got[~near], want[~near]), c
    order_o, off_o = P.traj_order(tr, n, dims, tab_o)
    order_g, off_g = F.trajectory_order(g, dims, tab_g)
    assert np.array_equal(off_g.cpu().numpy(), off_o)
    assert np.array_equal(order_g.cpu().numpy(), order_o)
    loop = tab_o["n_ends"] == 0
    t = tr.pos[:, n]
    rng = np.random.default_rng(23)
    one = np.full(tr.n_hits, 2, np.uint8)
    rare = one.copy()
    rare[rng.integers(0, tr.n_hits, size=max(1, tr.n_hits // 200))] = 1  # long runs, loops with none, one and two
    planted = rng.integers(1, 3, size=tr.n_hits).astype(np.uint8)
    for types in (one, rare, planted):
        tg = torch.from_numpy(types).to(DEV)
        for half in (0, 1, 5, 64, 65, 200):
            want = P.smooth_types(order_o, off_o, loop, types, half)
            got = F.smooth_types(g, tab_g, order_g, off_g, half, types=tg).cpu().numpy()
            assert np.array_equal(got, want), half
        got = F.simplify_types(g, tab_g, order_g, off_g, 1.0, types=tg).cpu().numpy()
        _check_simplified(got, order_o, off_o, loop, types, t, 1.0)
