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


# a solve's last words: the sums of its only iteration; those and u, v of its last two
@pytest.mark.parametrize("pcg,n_nodes", [(1, 200), (10, 300)])
def test_words_of_a_solve_long_past_are_not_taken_for_new(swgn, pcg, n_nodes):
    s = _surface(n_nodes, n_nodes)
    other = (s["depth"] + np.float32(0.01)).astype(np.float32)
    want = _stream(swgn, s, pcg_iters=pcg, gn_iters=1, stage_timing=1)
    st = _stream(swgn, s, pcg_iters=pcg, gn_iters=1, stage_timing=1)
    bx = swgn.Batch()
    for x in (want, st):
        assert x.solve_frame(s["depth"])["stage_us"][3] > 0      # (whole)
    folds = [100001] * 5 + [TAG_FOLDS - 1 - 5 * 100001]             # (a replay is reps launches and one before)
    for n in folds:
        bx.profile_stage([st], FOLD, reps=n - 1)
    _same((st.solve_frame(other), st.node_se3()), (want.solve_frame(other), want.node_se3()), pcg)
    bx.close()
    want.close()
    st.close()
