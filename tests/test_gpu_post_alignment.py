"""Caller-owned order arrays that begin at an entry of a larger buffer (aligned to 8 bytes only) hold what aligned ones do,
and the entries around them stay untouched."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2011_08697_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)


@pytest.mark.parametrize("first", [1, 2, 3])
def test_order_into_a_part_of_a_buffer(first):
    f = np.random.default_rng(2).standard_normal((20, 61, 90)).astype(np.float32)
    r = F.track_cp2d(torch.from_numpy(f).to(DEV))
    dims = (90, 61, 20)
    table = F.trajectory_table(r, dims)
    want, offsets = F.trajectory_order(r, dims, table)
    n, m = r["n_hits"], table["n"]
    buf = torch.full((n + 8,), -7, dtype=torch.int64, device=DEV)
    obuf = torch.full((m + 9,), -7, dtype=torch.int64, device=DEV)
    order, off = buf[first:first + n], obuf[first:first + m + 1]
    o, res, t = F._options(None), F._as_result(r), F._table_struct(table)
    d = (ctypes.c_int64 * 3)(*dims)
    F._check(F.lib().ftk_traj_order(ctypes.byref(res), 2, d, ctypes.byref(t), ctypes.byref(o), F._stream_handle(DEV),
                                    F._ptr(order), F._ptr(off)))
    torch.cuda.synchronize()
    assert torch.equal(order, want) and torch.equal(off, offsets)
    for b, k in ((buf, n), (obuf, m + 1)):
        assert bool((b[:first] == -7).all()) and bool((b[first + k:] == -7).all())
