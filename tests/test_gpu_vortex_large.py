"""Vortex surfaces on a grid whose rows fill more 64-vertex words than one launch takes (2^25): a uniform field but for
three patches, at both ends and across the words where a launch ends, against small calls on each patch with a rim of
the uniform field."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2011_08697_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)


def test_more_words_than_a_launch():
    big = (16, 513, 8192, 2)  # nt, nz, ny, nx: one word a row
    assert big[0] * big[1] * big[2] > 2 ** 26
    psi = torch.zeros((big[0], 2) + big[1:], device=DEV)
    psi[:, 0] = 1.0
    rng = np.random.default_rng(3)
    ids, labels, pos, parts = [], [], [], 0
    # first vertex (t, z, y) of boxes that hold a patch and its rim; rows t * 513 + z = 4096 begin the second launch
    for lo, shape in (((0, 0, 0), (4, 5, 6)), ((6, 502, 0), (4, 6, 7)), ((12, 508, 8186), (4, 5, 6))):
        box = np.zeros((shape[0], 2) + shape[1:] + (2,), np.float32)
        box[:, 0] = 1.0
        inner = tuple(slice(0 if lo[a] == 0 else 1, shape[a] if lo[a] + shape[a] == big[a] else shape[a] - 1) for a in range(3))
        at = (inner[0], slice(None), inner[1], inner[2])
        box[at] = rng.standard_normal(box[at].shape)
        b = torch.from_numpy(box).to(DEV)
        psi[lo[0]:lo[0] + shape[0], :, lo[1]:lo[1] + shape[1], lo[2]:lo[2] + shape[2]] = b
        r = F.track_vortex3d(b)
        assert r["n_hits"] > 100

        def there(i):  # the same triangle's id on the large grid
            v, ty = i // 50, i % 50
            x, v = v % 2, v // 2
            y, v = v % shape[2] + lo[2], v // shape[2]
            z, t = v % shape[1] + lo[1], v // shape[1] + lo[0]
            return (((t * big[1] + z) * big[2] + y) * 2 + x) * 50 + ty

        ids.append(there(r["tri_id"].cpu().numpy()))
        labels.append(there(r["label"].cpu().numpy()))
        pos.append(r["pos"].cpu().numpy().astype(np.float64) + np.array([0, lo[2], lo[1], lo[0]]))
        parts += r["n_components"]
    g = F.track_vortex3d(psi)
    assert np.array_equal(g["tri_id"].cpu().numpy(), np.concatenate(ids))
    assert np.array_equal(g["label"].cpu().numpy(), np.concatenate(labels))
    assert g["n_components"] == parts
    # binary32 points: half a unit of their last place on each side (coordinates below 8192)
    assert np.all(np.abs(g["pos"].cpu().numpy() - np.concatenate(pos)) <= 2.0 ** -11)
