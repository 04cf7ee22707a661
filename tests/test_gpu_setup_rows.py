"""The block pattern and the rows listed from it, at node counts around the
words and waves of its bitmaps, against the pattern's plain definition; the
segment layout that follows from it against the sequential walk."""
import numpy as np
import pytest

from gpu_common import expected_pattern, gpu_lib

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def swgn():
    return gpu_lib()


def _stream(swgn, pos, nodes):
    st = swgn.Stream(swgn.sw_config_default(width=64, height=48, fx=50.0, fy=50.0, cx=32.0, cy=24.0, node_sigma=0.1))
    nrm = np.zeros_like(pos)
    nrm[:, 2] = -1.0
    st.set_reference_surfels(pos, nrm)
    st.set_node_graph(nodes)
    return st


# a bitmap row of 1 word, 2 words, one wave of words (2048 nodes), more than one; many nodes per row in a volume
@pytest.mark.parametrize("n_nodes,n_surfels,flat", [(9, 100, True), (32, 500, False), (33, 4097, True),
                                                    (64, 4096, False), (65, 700, True), (2047, 9000, True),
                                                    (2048, 3000, False), (2049, 8193, False), (4100, 30000, True)])
def test_pattern_is_its_definition(swgn, n_nodes, n_surfels, flat):
    rng = np.random.default_rng(n_nodes)
    nodes = rng.uniform(0, 1, (n_nodes, 3)).astype(np.float32)
    pos = rng.uniform(0, 1, (n_surfels, 3)).astype(np.float32)
    if flat:
        nodes[:, 2] *= 0.01
        pos[:, 2] *= 0.01
    st = _stream(swgn, pos, nodes)
    idx, _ = st.skinning()
    nbr = st.node_graph().reshape(n_nodes, 8)
    rp, ci = st.pattern()
    wrp, wci = expected_pattern(idx.reshape(-1, 4), nbr, n_nodes)
    assert np.array_equal(rp, wrp) and np.array_equal(ci, wci)
    assert all(v == 0 for v in st.check_layout().values())
    st.close()


# surfels of one node set: one bucket, at the edges of how it is sorted
# (counted, bitonic of 512 to 2048, more than a bucket holds)
@pytest.mark.parametrize("n_surfels", [1, 2, 255, 256, 257, 512, 513, 2047, 2048, 2049, 6000])
def test_surfels_of_one_node_set_are_ordered(swgn, n_surfels):
    rng = np.random.default_rng(n_surfels)
    nodes = np.array([[0, 0, 1], [0.1, 0, 1], [0, 0.1, 1], [0.1, 0.1, 1]] + [[2 + k, 2, 1] for k in range(8)],
                     np.float32)
    pos = (np.array([0.02, 0.02, 1.0]) + rng.uniform(-0.004, 0.004, (n_surfels, 3))).astype(np.float32)
    st = _stream(swgn, pos, nodes)
    assert st.layout()["node_sets"] == 1
    assert all(v == 0 for v in st.check_layout().values())
    st.close()


# few nodes, many surfels: thousands of segments in a block (9 nodes: more
# than are ordered on chip), buckets of every size
@pytest.mark.parametrize("n_nodes,n_surfels", [(9, 2000000), (12, 60000), (40, 150000), (200, 100000)])
def test_layout_of_many_surfels_on_few_nodes(swgn, n_nodes, n_surfels):
    rng = np.random.default_rng(n_nodes)
    nodes = rng.uniform(0, 1, (n_nodes, 3)).astype(np.float32)
    pos = rng.uniform(0, 1, (n_surfels, 3)).astype(np.float32)
    st = _stream(swgn, pos, nodes)
    assert all(v == 0 for v in st.check_layout().values())
    st.close()


def test_models_in_turn_on_one_stream_equal_fresh_streams(swgn, scene_cache):
    """A model takes over the device memory of the last one unless it is much
    smaller or larger; either way it solves, fuses and grows as on a fresh stream."""
    s = scene_cache("c1")
    n = len(s.surfel_pos)

    def step(st, m):
        st.set_reference_surfels(s.surfel_pos[:m], s.surfel_nrm[:m])
        st.set_node_graph(s.node_pos)
        out = [st.solve_frame(s.depth)["e_data"], st.node_se3()]
        st.fuse_frame(s.depth, 1)
        st.update_geometry()
        return out + list(st.reference_surfels()) + list(st.surfel_attributes()) + [st.check_layout()]

    st = swgn.Stream(swgn.config_for(s))
    for m in (n, (3 * n) // 5, n, n // 8, n // 6, n, n):
        fresh = swgn.Stream(swgn.config_for(s))
        got, want = step(st, m), step(fresh, m)
        fresh.close()
        assert all(v == 0 for v in got.pop().values()) and want.pop()
        for k, (a, b) in enumerate(zip(got, want)):
            assert np.array_equal(a, b), (m, k)
    st.close()
