"""The extruded-mesh pass where its words end, against the oracle: numbers of steps around the widths of a row of lanes
and of a 64-step chunk, faces around a word and a workgroup of them, tied values, values beyond 24 bits, a vertex of no
triangle (its values are not read as the mesh's)."""
import numpy as np
import pytest

from oracle import mesh as M
from paper_2011_08697_amd import synth
from parity import assert_pos_close
from test_gpu_mesh import F, _run

pytestmark = pytest.mark.gpu


def _check(xy, tri, field):
    g = _run(xy, tri, field)
    o = M.track_cp_mesh(xy, tri, field)
    assert g["n_hits"] == o.n_hits and g["n_trajectories"] == o.n_traj
    assert np.array_equal(g["face_id"].cpu().numpy(), o.face_id)
    assert np.array_equal(g["label"].cpu().numpy(), o.label)
    assert_pos_close(g["pos"].cpu().numpy(), o.pos)
    return o.n_hits


@pytest.mark.parametrize("nt", [2, 3, 4, 5, 31, 32, 33, 63, 64, 65, 128, 130])
def test_steps_around_the_word_widths(nt):
    xy, tri = synth.kuhn_grid_mesh(5, 4)
    rng = np.random.default_rng(nt)
    assert _check(xy, tri, rng.standard_normal((nt, 2, len(xy))).astype(np.float32)) > 0
    _check(xy, tri, rng.integers(-1, 2, size=(nt, 2, len(xy))).astype(np.float32) / 2 ** 20)


@pytest.mark.parametrize("points", [3, 4, 9, 12, 23, 44, 90])
def test_faces_around_the_words(points):
    xy, tri = (np.array([[0, 0], [1, 0], [0, 1]], np.float32), np.array([[0, 1, 2]], np.int32)) if points == 3 else \
        synth.delaunay_mesh(points, seed=points)
    rng = np.random.default_rng(points)
    for scale in (1.0, 300.0):  # 2^20 steps a unit: the second reaches 30 of the 31 bits allowed
        _check(xy, tri, (scale * rng.standard_normal((7, 2, len(xy)))).astype(np.float32))


def test_values_of_an_unused_vertex_are_not_checked():
    xy, tri = synth.delaunay_mesh(30, seed=6)
    rng = np.random.default_rng(2)
    f = rng.standard_normal((5, 2, len(xy))).astype(np.float32)
    want = _run(xy, tri, f)
    xy1 = np.concatenate([xy, np.array([[0.5, 0.25]], np.float32)])
    f1 = np.concatenate([f, np.full((5, 2, 1), np.nan, np.float32)], axis=2)
    got = _run(xy1, tri, f1)
    assert got["n_hits"] == want["n_hits"] > 0
    for k in ("face_id", "pos", "label"):
        assert np.array_equal(got[k].cpu().numpy(), want[k].cpu().numpy()), k
    for v, code in ((np.nan, "non-finite"), (3.0e38, None), (1.0e9, None)):
        bad = f.copy()
        bad[3, 1, 11] = v
        with pytest.raises(F.FtkError):
            _run(xy, tri, bad)
