"""The choice between the middle path and the 512-row tiles."""
import pytest

from paper_2608_24070_amd import slim
from tests.plans import plan


# Calls that the middle path slowed down (its time over the 512-row tiles': 1.02 to 1.4 on the GPU), and neighbours
# that it speeds up (0.56 to 0.95)
@pytest.mark.parametrize("kind,m,rows,red,r,mid", [
    ("fwd", 8192, 1024, 2048, 0, False), ("fwd", 7963, 1024, 640, 0, False), ("fwd", 4096, 2048, 4096, 0, False),
    ("fwd", 16000, 512, 1024, 0, False), ("fwd", 4797, 1024, 768, 0, False), ("fwd", 3142, 2176, 2176, 0, False),
    ("fwd", 2048, 4096, 4096, 0, True), ("fwd", 1024, 8192, 8192, 0, True), ("fwd", 512, 16384, 4096, 0, True),
    ("fwd", 4140, 1408, 5120, 0, True), ("fwd", 5376, 896, 1792, 0, True), ("fwd", 3000, 1152, 6656, 0, True),
    ("dx", 4715, 1024, 640, 0, False), ("dx", 7168, 1024, 2048, 0, False), ("dx", 3584, 2048, 4096, 0, False),
    ("dx", 663, 8320, 13824, 0, True), ("dx", 5105, 896, 3200, 0, True), ("dx", 448, 14336, 4096, 0, True),
    ("fwd", 2250, 2432, 3968, 224, False), ("fwd", 3368, 1536, 512, 32, False), ("fwd", 3954, 1152, 2816, 96, False),
    ("fwd", 3500, 2048, 9216, 192, False), ("fwd", 2246, 3328, 1280, 128, False),
    ("fwd", 512, 11008, 4096, 384, True), ("fwd", 333, 5120, 5120, 512, True), ("fwd", 250, 28672, 8192, 512, True),
    ("fwd", 899, 5248, 10624, 512, True), ("fwd", 1300, 4096, 4096, 384, True),
    ("dx", 1280, 4096, 4096, 384, False), ("dx", 1326, 3200, 8320, 320, False), ("dx", 2203, 1920, 640, 64, False),
    ("dx", 333, 13824, 5120, 512, True), ("dx", 200, 4096, 4096, 384, True), ("dx", 632, 7552, 2304, 224, True)])
def test_middle_path_where_it_is_faster(kind, m, rows, red, r, mid):
    n, k = (red, rows) if kind == "dx" else (rows, red)
    assert plan(kind, m, n, k, r).mid == mid


# Sizes past the no-allocation entry point's scratch on the 512-row tiles too: it does not choose between the plans
@pytest.mark.parametrize("kind,m,rows,red,r", [
    ("fwd", 4096, 512, 14336, 0), ("fwd", 2048, 2048, 14336, 192), ("fwd", 3000, 1024, 13824, 96),
    ("dx", 4096, 512, 14336, 0), ("dx", 2048, 2048, 14336, 192), ("fwd", 2048, 5120, 13824, 512)])
def test_scratch_decides_nothing_past_it(kind, m, rows, red, r):
    n, k = (red, rows) if kind == "dx" else (rows, red)
    p = plan(kind, m, n, k, r)
    assert plan(kind, m, n, k, r, 0).total > slim.SLIM_NOALLOC_SCRATCH_BYTES
    assert p.mid or p.ad_tn


def test_scratch_keeps_what_fits_it():
    # the 512-row tiles fit the scratch, the middle path's partials do not
    p = plan("fwd", 1000, 4096, 11008, 384)
    assert not p.mid and p.total <= slim.SLIM_NOALLOC_SCRATCH_BYTES
