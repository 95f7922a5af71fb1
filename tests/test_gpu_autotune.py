"""Tuning never leaves a later default call with a slower detection than the untuned one: where the shape's own rule takes
shorter slabs than the candidates, and for another length than the tuned one."""
import statistics

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2011_08697_amd as F  # noqa: E402

DEV = torch.device("cuda", 0)


def _detection_ms(f):
    return statistics.median(F.track_cp2d(f, profile=1)["stats"]["t_detect_ms"] for _ in range(41))


@pytest.mark.parametrize("nx,ny,nt,tuned_nt", [(72, 64, 12, 12), (136, 88, 10, 10), (80, 64, 6, 600)])
def test_tuning_does_not_slow_the_default_call(nx, ny, nt, tuned_nt):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(nx)
    f = torch.randn((nt, ny, nx), generator=gen, device=DEV)
    g = torch.randn((tuned_nt, ny, nx), generator=gen, device=DEV)
    before = _detection_ms(f)
    want = F.track_cp2d(f)
    ty, tt = F.autotune_cp2d(g)
    assert ty in (8, 16, 32) and tt in (8, 16, 32, min(16, tuned_nt), min(32, tuned_nt))
    # a slab of 8 steps takes three to four times as long as the rule's here
    assert _detection_ms(f) <= 2.0 * before
    r = F.track_cp2d(f)
    assert r["n_hits"] == want["n_hits"] and torch.equal(r["label"], want["label"])
