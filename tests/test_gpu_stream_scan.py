"""Offsets of a pushed step at the sizes where their scan changes form (one block up to 16384 rows of 64 vertices, a
multiple of its round, one more), hits in every push, room grown while steps are open: streaming equals the one-shot
call; and the errors of a push: a non-finite step fails that push and closes the tracker."""
import numpy as np
import pytest

from test_gpu_stream import _same, _stream

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2011_08697_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)


@pytest.mark.parametrize("ny", [2, 7, 8191, 8192, 8193, 16384, 16385])
def test_stream_offsets_equal_one_shot(ny):
    f = np.random.default_rng(ny).standard_normal((5, ny, 3)).astype(np.float32)
    one = F.track_cp2d(torch.from_numpy(f).to(DEV))
    assert ny == 2 or one["n_hits"] > 0
    _same(_stream(f, 2), one)


@pytest.mark.parametrize("scale", [1.0, 1024.0])  # the second beyond the narrow form of the 3D tests
def test_stream_3d_dense(scale):
    f = (scale * np.random.default_rng(3).standard_normal((6, 7, 9, 19))).astype(np.float32)
    _same(_stream(f, 3), F.track_cp3d(torch.from_numpy(f).to(DEV)))


@pytest.mark.parametrize("n,bad", [(2, 0), (2, 2), (2, 3), (3, 1)])
def test_non_finite_step_fails_its_push(n, bad):
    shape = (5, 40, 70) if n == 2 else (4, 8, 9, 20)
    f = torch.from_numpy(np.random.default_rng(1).standard_normal(shape).astype(np.float32)).to(DEV)
    f[bad].view(-1)[17] = float("nan")
    tr = F.Tracker(n, list(shape[1:][::-1]))
    failed = -1
    for t in range(shape[0]):
        try:
            tr.push(f[t].contiguous())
        except F.FtkError:
            failed = t
            break
    assert failed == max(bad, 1)  # detected with the step after a first one
    with pytest.raises(F.FtkError):
        tr.push(f[0].contiguous())
    tr.close()
