"""The geometry update and the append selection where the survivors' scan runs
in many tiles and its N flags, N + 1 positions and scratch lie end to end in
device memory (N = 63 mod 64: a position too many would be the scratch's first
word): kept and appended surfels against the selection done on the host."""
import numpy as np
import pytest

from gpu_common import gpu_lib
from oracle import append as A

pytestmark = pytest.mark.gpu

T_NOW = 45


@pytest.fixture(scope="module")
def swgn():
    return gpu_lib()


def _model(n_surfels, w, h, seed):
    """A wavy sheet in front of a w x h camera: n_surfels surfels of the left
    four fifths of the image, a grid of nodes, the frame of the whole sheet."""
    rng = np.random.default_rng(seed)
    f, z0 = 0.9 * w, 1.0

    def sheet(u, v):
        x, y = (u - w / 2) / f * z0, (v - h / 2) / f * z0
        return np.stack([x, y, z0 + 0.02 * np.sin(6 * x) * np.cos(5 * y)], -1)

    pos = sheet(rng.uniform(2, 0.8 * w, n_surfels), rng.uniform(2, h - 2, n_surfels))
    d = np.stack([0.12 * np.cos(6 * pos[:, 0]) * np.cos(5 * pos[:, 1]),
                  -0.1 * np.sin(6 * pos[:, 0]) * np.sin(5 * pos[:, 1]), -np.ones(n_surfels)], -1)
    nrm = d / np.linalg.norm(d, axis=1, keepdims=True)
    gu, gv = np.meshgrid(np.linspace(0, w, 16), np.linspace(0, h, 12))
    nodes = sheet(gu.ravel(), gv.ravel())
    v, u = np.mgrid[0:h, 0:w].astype(np.float64)
    X, Y = (u - w / 2) / f * z0, (v - h / 2) / f * z0
    depth = z0 + 0.02 * np.sin(6 * X) * np.cos(5 * Y)
    cfg = dict(width=w, height=h, fx=f, fy=f, cx=w / 2, cy=h / 2, node_sigma=0.08, gn_iters=1)
    return (a.astype(np.float32) for a in (pos, nrm, nodes, depth)), cfg


# surfels and pixels 63 mod 64 and their neighbours, in two and in many tiles of the scan
@pytest.mark.parametrize("n_surfels,w,h", [(4159, 333, 251), (4160, 333, 252), (20031, 333, 251), (60031, 127, 97),
                                           (60030, 640, 480), (4158, 127, 33)])
def test_update_keeps_and_appends_what_the_host_selects(swgn, n_surfels, w, h):
    (pos, nrm, nodes, depth), cfg = _model(n_surfels, w, h, n_surfels)
    rng = np.random.default_rng(1)
    st = swgn.Stream(swgn.sw_config_default(**cfg))
    st.set_reference_surfels(pos, nrm)
    st.set_node_graph(nodes)
    st.set_surfel_attributes(None, rng.uniform(1.0, 20.0, n_surfels).astype(np.float32), None,
                             rng.integers(0, 40, n_surfels).astype(np.int32))
    for _ in range(4):
        st.fuse_frame(depth, T_NOW)
        match = st.last_fusion()[0]
        pos0, nrm0 = st.reference_surfels()
        rad0, conf0, tob0, ti0 = st.surfel_attributes(with_t_init=True)
        app = st.append_candidates()
        # the survivors: unmatched pixels in row-major order, as many as were neither far nor compressive
        assert app["n_appended"] == app["n_written"] == app["pixel"].size > 0
        assert app["n_appended"] == app["n_candidates"] - app["n_far"] - app["n_compressive"]
        assert np.all(np.diff(app["pixel"]) > 0) and np.all(match.ravel()[app["pixel"]] == -1)
        # with every node at rest a survivor is its pixel's point (FP32: a few ulp of about 1 m)
        y, x = np.divmod(app["pixel"], w)
        z = depth.ravel()[app["pixel"]].astype(np.float64)
        V = np.stack([(x - cfg["cx"]) / cfg["fx"] * z, (y - cfg["cy"]) / cfg["fy"] * z, z], -1)
        assert np.max(np.abs(app["pos"] - V)) < 1e-5
        keep = ~A.unstable(conf0, ti0, T_NOW, 10.0, 30)
        g = st.update_geometry()
        na = app["n_appended"]
        assert g["n_removed"] == int((~keep).sum()) and g["n_surfels"] == int(keep.sum()) + na
        pos1, nrm1 = st.reference_surfels()
        rad1, conf1, tob1, ti1 = st.surfel_attributes(with_t_init=True)
        new = np.full(na, T_NOW, np.int32)
        for got, old, more in ((pos1, pos0, app["pos"]), (nrm1, nrm0, app["nrm"]), (rad1, rad0, app["radius"]),
                               (conf1, conf0, app["confidence"]), (tob1, tob0, new), (ti1, ti0, new)):
            assert np.array_equal(got, np.concatenate([old[keep], more]))
        # the same model again, for the next turn
        st.set_reference_surfels(pos0, nrm0)
        st.set_node_graph(nodes)
        st.set_surfel_attributes(rad0, conf0, tob0, ti0)
    st.close()
