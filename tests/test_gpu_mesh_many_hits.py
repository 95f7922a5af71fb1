"""The unions of the extruded-mesh pass where their form changes (eight lanes a hit up to 2^17 hits, then one) and beyond
2^29 hits, where eight lanes a hit pass the 2^32 lanes of a launch: copies of one small mesh side by side, each of which
must give the small mesh's result, which the oracle checks."""
import numpy as np
import pytest

from oracle import mesh as M
from paper_2011_08697_amd import synth
from parity import assert_pos_close

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2011_08697_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)


@pytest.mark.parametrize("nt,hits", [(5, 2 ** 17 - 1500), (5, 2 ** 17 + 1500), (200, 2 ** 29 + 1000)])
def test_copies_of_a_mesh(nt, hits):
    xy, tri = synth.delaunay_mesh(60, seed=5)
    nv, nf = len(xy), len(tri)
    f = np.random.default_rng(nt).standard_normal((nt, 2, nv)).astype(np.float32)
    o = M.track_cp_mesh(xy, tri, f[:5])
    xy, tri, f = (torch.from_numpy(np.ascontiguousarray(a)).to(DEV) for a in (xy.astype(np.float32), tri.astype(np.int32), f))
    r = F.track_cp_mesh2d(xy, tri, f[:5].contiguous())
    assert np.array_equal(r["face_id"].cpu().numpy(), o.face_id) and np.array_equal(r["label"].cpu().numpy(), o.label)
    assert_pos_close(r["pos"].cpu().numpy(), o.pos)
    if nt > 5:
        r = F.track_cp_mesh2d(xy, tri, f)
    S, ne, h = r["faces_per_step"], r["n_edges"], r["n_hits"]
    copies = -(-hits // h) if hits > 2 ** 17 else hits // h
    first = torch.arange(copies, device=DEV, dtype=torch.int32)[:, None, None] * nv
    g = F.track_cp_mesh2d(xy.repeat(copies, 1), (tri[None] + first).reshape(-1, 3).contiguous(), f.repeat(1, 1, copies))
    assert g["n_hits"] == copies * h and g["n_trajectories"] == copies * r["n_trajectories"]
    assert (g["n_hits"] > hits) == (hits > 2 ** 17)
    # the small mesh's hit of every face, or -1
    row = torch.full((S * nt,), -1, dtype=torch.int64, device=DEV)
    row[r["face_id"]] = torch.arange(h, device=DEV)

    def copy_and_face(i):
        t, l = i // (S * copies), i % (S * copies)
        c = torch.empty_like(l)
        for lo, n, lo0 in ((0, nf, 0), (nf, 2 * ne, nf), (nf + 2 * ne, 2 * nf, nf + 2 * ne)):
            at = (l >= lo * copies) & (l < (lo + n) * copies)
            k = l[at] - lo * copies
            c[at] = k // n
            l[at] = lo0 + k % n
        return c, t * S + l

    last = -1
    for b in range(0, g["n_hits"], 1 << 25):
        ids = g["face_id"][b:b + (1 << 25)]
        assert int(ids[0]) > last and bool((ids[1:] > ids[:-1]).all())
        last = int(ids[-1])
        c, i0 = copy_and_face(ids)
        k = row[i0]
        assert bool((k >= 0).all())
        cl, l0 = copy_and_face(g["label"][b:b + (1 << 25)])
        assert torch.equal(cl, c) and torch.equal(l0, r["label"][k])
        assert torch.equal(g["pos"][b:b + (1 << 25)], r["pos"][k])
