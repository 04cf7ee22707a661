"""The correspondence launch's time around the number of packs from which
workgroups no longer share one: sharing pays only while there is not a pack
for every CU."""
import pytest

from gpu_common import gpu_lib
from test_gpu_segment_grams import _model, _stream

pytestmark = pytest.mark.gpu

CORR = 2                     # stage number


@pytest.fixture(scope="module")
def swgn():
    return gpu_lib()


def test_a_launch_of_more_packs_than_cus_does_not_share_them(swgn):
    """470 packs of 60 to 70 segments: about half of what 2.4 times as many
    take (two thirds when their surfels are seen twice)."""
    m = _model(1600, 7, 1, w=320, h=240, f=300.0)
    sts = [_stream(swgn, m) for _ in range(24)]
    lay = sts[0].layout()
    few = 470 // lay["packs"]
    many = (1128 + lay["packs"] - 1) // lay["packs"]
    assert lay["segments"] > 30 * lay["packs"] and many <= len(sts)
    bx = swgn.Batch()
    us = {}
    for k in (few, many):
        bx.solve(sts[:k], [m[3]] * k)
        us[k] = min(bx.profile_stage(sts[:k], CORR, 200) for _ in range(5))
    print(few * lay["packs"], "packs", us[few], "us;", many * lay["packs"], "packs", us[many], "us")
    for x in sts + [bx]:
        x.close()
    assert us[few] < 0.63 * us[many]
