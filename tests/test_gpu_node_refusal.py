"""Node sets with a node that has no 8 neighbours (a position that is not
finite, or too far off for the FP32 square of a distance) are refused, and the
stream takes the next one."""
import numpy as np
import pytest

from gpu_common import gpu_lib

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def swgn():
    return gpu_lib()


@pytest.mark.parametrize("n_nodes", [9, 70, 2100])
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf, 1e30])
@pytest.mark.parametrize("device", [False, True])
def test_a_node_without_neighbours_is_refused(swgn, n_nodes, value, device):
    import torch
    rng = np.random.default_rng(n_nodes)
    nodes = rng.uniform(0, 1, (n_nodes, 3)).astype(np.float32)
    pos = rng.uniform(0, 1, (3000, 3)).astype(np.float32)
    nrm = np.tile(np.array([[0, 0, -1]], np.float32), (3000, 1))
    bad = nodes.copy()
    bad[n_nodes // 2, 1] = value
    cfg = dict(width=64, height=48, fx=50.0, fy=50.0, cx=32.0, cy=24.0, node_sigma=0.1)
    st, ref = (swgn.Stream(swgn.sw_config_default(**cfg)) for _ in range(2))
    for x in (st, ref):
        x.set_reference_surfels(pos, nrm)
    with pytest.raises(swgn.SwError) as e:
        st.set_node_graph(torch.from_numpy(bad).cuda() if device else bad)
    assert e.value.status == swgn.SW_EINVAL
    with pytest.raises(swgn.SwError):
        st.solve_frame(np.ones((48, 64), np.float32))
    st.set_node_graph(nodes)
    ref.set_node_graph(nodes)
    assert np.array_equal(st.skinning()[0], ref.skinning()[0]) and np.array_equal(st.node_graph(), ref.node_graph())
    assert all(v == 0 for v in st.check_layout().values())
    st.close()
    ref.close()
