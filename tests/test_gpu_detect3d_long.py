"""3D series longer than the steps that one lane plans (16), with runs of tested steps shorter than, as long as and longer
than a workgroup's slab, against the oracle; and a series of more planes than one launch of the sign facts takes (2^23),
nearly all of them flat, against small calls on its patches."""
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


@pytest.mark.parametrize("nt", [15, 16, 17, 31, 33, 50])
@pytest.mark.parametrize("kind", ["noise", "bursts"])
def test_long_series(nt, kind):
    rng = np.random.default_rng(nt)
    f = 1e-2 * rng.normal(size=(nt, 5, 9, 18))
    if kind == "bursts":  # flat but for stretches of steps of several lengths, ends of the series among them
        for t in range(nt):
            if (t // 3) % 2 and not 20 <= t < 29 and t != nt - 1:
                f[t] = 0.0
    f = f.astype(np.float32)
    ref = O.track(f, n=3, kind=0)
    assert ref.n_hits > 0
    for slab in (0, 1, 3, 7, 16):
        assert_full_parity(F.track_cp3d(torch.from_numpy(f).to(DEV), slab_depth=slab), ref)


def test_more_planes_than_a_launch():
    nt = 2 ** 24 + 5
    f = torch.zeros((nt, 2, 2, 2), device=DEV)
    rng = np.random.default_rng(4)
    ids, labels, pos = [], [], []
    for t0, n, rim in ((0, 6, (0, 1)), (2 ** 23 - 4, 9, (1, 1)), (nt - 7, 7, (1, 0))):
        p = np.zeros((n, 2, 2, 2), np.float32)
        p[rim[0]:n - rim[1]] = rng.standard_normal((n - sum(rim), 2, 2, 2))
        p = torch.from_numpy(p).to(DEV)
        f[t0:t0 + n] = p
        r = F.track_cp3d(p)
        assert r["n_hits"] > 0
        ids.append(r["face_id"] + t0 * 8 * 60)
        labels.append(r["label"] + t0 * 8 * 60)
        pos.append(r["pos"].double() + torch.tensor([0.0, 0.0, 0.0, t0], device=DEV))
    g = F.track_cp3d(f)
    assert torch.equal(g["face_id"], torch.cat(ids)) and torch.equal(g["label"], torch.cat(labels))
    # binary32 times below 2^24 + 5: sums of four products, each rounded to a unit of at most 2
    assert bool(((g["pos"].double() - torch.cat(pos)).abs() <= 8.0).all())
    assert bool(((g["pos"][:, :3].double() - torch.cat(pos)[:, :3]).abs() <= 1e-5).all())
