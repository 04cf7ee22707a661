"""The segment Gram matrices at the sizes where their kernel changes its way:
segments from 1 to 232 rows (the last MFMA's partial rows, tiles dealt to the
waves or a whole segment per wave) and packs shared by several workgroups
against one workgroup each. A captured iteration's system is compared with
the sums of its own Jacobian rows in 64 bits, and a stream's result alone
(few packs: shared) with its result in a batch of many packs (not shared)."""
import numpy as np
import pytest

from gpu_common import gpu_lib

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def swgn():
    return gpu_lib()


def _model(n_nodes, run, seed, w=160, h=120, f=150.0):
    """A plane at 1 m: nodes on a grid, surfels in clusters of `run` around
    points between the nodes (a cluster shares its nearest nodes, so the
    segments have about `run` rows), and a frame 2 mm behind, with noise."""
    rng = np.random.default_rng(seed)
    side = int(np.ceil(np.sqrt(n_nodes)))
    g = (np.stack(np.meshgrid(np.arange(side), np.arange(side)), -1).reshape(-1, 2)[:n_nodes] - side / 2) * 0.03
    g = g + rng.uniform(-0.004, 0.004, g.shape)
    nodes = np.concatenate([g, np.ones((n_nodes, 1))], 1).astype(np.float32)
    xy = (g[:, None] + [0.009, 0.006] + rng.uniform(-0.002, 0.002, (n_nodes, run, 2))).reshape(-1, 2)
    pos = np.concatenate([xy, np.ones((len(xy), 1))], 1).astype(np.float32)
    nrm = np.tile(np.array([[0.0, 0.0, -1.0]], np.float32), (len(pos), 1))
    depth = (1.002 + rng.normal(0, 5e-4, (h, w))).astype(np.float32)
    cfg = dict(width=w, height=h, fx=f, fy=f, cx=w / 2, cy=h / 2, node_sigma=0.03, gn_iters=2)
    return pos, nrm, nodes, depth, cfg


def _stream(swgn, m, **cfg):
    st = swgn.Stream(swgn.sw_config_default(**{**m[4], **cfg}))
    st.set_reference_surfels(m[0], m[1])
    st.set_node_graph(m[2])
    return st


@pytest.mark.parametrize("n_nodes,run", [(300, 1), (64, 3), (64, 4), (60, 5), (50, 15), (50, 16), (50, 17), (40, 31),
                                         (40, 33), (30, 48), (20, 100), (16, 231), (16, 232), (9, 500)])
def test_system_is_the_sum_over_the_captured_rows(swgn, n_nodes, run):
    """Tolerance: FP32 sums of at most 500 products per block and surfel set,
    well conditioned (squares on the diagonal): 500 x 2^-24 = 3e-5 relative."""
    m = _model(n_nodes, run, n_nodes + run)
    st = _stream(swgn, m, debug_iter=0, lambda_reg=0.0, damping=0.0)
    try:
        st.solve_frame(m[3])
    except swgn.SwError as e:                     # (a node no surfel sees has an empty block: not solvable, still captured)
        assert e.status == swgn.SW_ENUMERIC
    r, J = (a.astype(np.float64) for a in st.last_jacobian())
    idx = st.skinning()[0]
    blocks, g, _ = st.last_system()
    rp, ci = st.pattern()
    st.close()
    nn = n_nodes
    H = np.zeros((nn, nn, 6, 6))
    want_g = np.zeros((nn, 6))
    for a in range(4):
        np.add.at(want_g, idx[:, a], J[:, a] * r[:, None])
        for b in range(4):
            np.add.at(H, (idx[:, a], idx[:, b]), J[:, a, :, None] * J[:, b, None, :])
    scale = np.abs(H).max()
    assert scale > 0
    for k in range(nn):
        for e in range(rp[k], rp[k + 1]):
            assert np.abs(blocks[e] - H[k, ci[e]]).max() <= 3e-5 * scale, (k, ci[e])
    assert np.abs(g - want_g).max() <= 3e-5 * np.abs(want_g).max()


@pytest.mark.parametrize("n_nodes,run", [(900, 1), (700, 2), (400, 9)])
def test_shared_packs_equal_whole_ones(swgn, n_nodes, run):
    m = _model(n_nodes, run, 3)
    big = _model(2500, 60, 4, w=320, h=240, f=300.0)            # enough packs that none is shared
    alone = _stream(swgn, m)
    assert alone.layout()["segments"] > 8 * alone.layout()["packs"]
    a = [alone.solve_frame(m[3]) for _ in range(2)][-1], alone.node_se3()
    st, other, bx = _stream(swgn, m), _stream(swgn, big), swgn.Batch()
    assert other.layout()["packs"] > 512
    for _ in range(2):
        stats, _ = bx.solve([st, other], [m[3], big[3]])
    assert np.array_equal(a[1], st.node_se3())
    for k in ("e_data", "e_reg", "n_corr", "pcg_resid"):
        assert a[0][k] == stats[0][k], k
    bx.close()
    for x in (alone, st, other):
        x.close()
