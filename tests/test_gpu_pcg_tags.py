"""The exchange words of the linear solve in one launch carry tags that come
again after 2^19 folds (swgn_frame.h): a word left behind that long must not
pass for a new one. The folds between are replayed, as a stream whose frames
are solved step by step for hours would run them."""
import numpy as np
import pytest

from gpu_common import gpu_lib
from test_gpu_pcg_solve import _same, _stream, _surface

pytestmark = pytest.mark.gpu

TAG_FOLDS = 1 << 19          # 2^32 tags / 8192 per solve
FOLD = 8                     # stage number


@pytest.fixture(scope="module")
def swgn():
    return gpu_lib()


def test_words_of_a_solve_long_past_are_not_taken_for_new(swgn):
    """Two PCG iterations, so that a solve's first words are its last. Streams
    of 65 workgroups, one per CU: the fourth's start at different times, and
    the early ones look for the words of those that have not started."""
    scenes = [_surface(4100, k) for k in range(5)]
    first = [s["depth"] for s in scenes]
    other = [(d + np.float32(0.01)).astype(np.float32) for d in first]
    sides = [[_stream(swgn, s, pcg_iters=2, gn_iters=1) for s in scenes] for _ in range(2)]
    bx = swgn.Batch()
    for sts in sides:
        bx.solve(sts, first)
    for n in [100001] * 5 + [TAG_FOLDS - 1 - 5 * 100001]:           # (a replay is reps launches and one before)
        bx.profile_stage(sides[0][3:4], FOLD, reps=n - 1)
    got, want = ([(r, st.node_se3()) for r, st in zip(bx.solve(sts, other)[0], sts)] for sts in sides)
    for k in range(5):
        _same(got[k], want[k], k)
    bx.close()
    for st in sides[0] + sides[1]:
        st.close()
