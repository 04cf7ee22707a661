"""The linear solve in one launch (workgroups of a stream exchanging their
sums and products) against a product and a finish launch per PCG iteration:
the same operations in the same order, so every result must be identical, at
the sizes where its tiling changes, with a launch of many streams, where the
node set does not fit it, and where it gives up waiting."""
import threading

import numpy as np
import pytest

from gpu_common import gpu_lib

pytestmark = pytest.mark.gpu

STEP_SLOTS = (5, 6)          # stage_us: PCG products and finishes of the step-wise solve


@pytest.fixture(scope="module")
def swgn():
    return gpu_lib()


def _surface(n_nodes, seed, volume=False, w=320, h=240, f=285.0):
    """Nodes on a wavy surface (or in a volume in front of it), one surfel per
    second pixel, and a frame of the surface moved and noised."""
    rng = np.random.default_rng(seed)
    spacing = min(0.03, np.sqrt(0.9 / n_nodes))
    side = int(np.ceil(np.sqrt(n_nodes * 1.4)))
    gx, gy = np.meshgrid(np.arange(side) - side / 2, np.arange(side) - side / 2)
    xy = np.stack([gx.ravel() * 1.15, gy.ravel() * 0.87], 1)
    xy = (xy[np.argsort(np.hypot(*xy.T))[:n_nodes]] + rng.uniform(-0.2, 0.2, (n_nodes, 2))) * spacing
    z = 1.2 + 0.03 * np.sin(9 * xy[:, 0]) * np.cos(7 * xy[:, 1])
    if volume:
        z = z - rng.uniform(0.0, 8 * spacing, n_nodes)
    nodes = np.stack([xy[:, 0], xy[:, 1], z], 1).astype(np.float32)
    v, u = np.mgrid[2:h - 2:2, 2:w - 2:2].astype(np.float64)
    x, y = (u - w / 2) / f * 1.2, (v - h / 2) / f * 1.2
    d = 1.2 + 0.03 * np.sin(9 * x) * np.cos(7 * y)
    pos = np.stack([x, y, d], -1).reshape(-1, 3)
    nrm = np.stack([0.27 * np.cos(9 * x) * np.cos(7 * y), -0.21 * np.sin(9 * x) * np.sin(7 * y), -np.ones_like(x)], -1)
    nrm = (nrm / np.linalg.norm(nrm, axis=-1, keepdims=True)).reshape(-1, 3)
    near = np.min(np.hypot(pos[:, None, 0] - xy[None, ::max(1, n_nodes // 64), 0],
                           pos[:, None, 1] - xy[None, ::max(1, n_nodes // 64), 1]), axis=1) < 0.3
    pos, nrm = pos[near], nrm[near]
    V, U = np.mgrid[0:h, 0:w].astype(np.float64)
    X, Y = (U - w / 2) / f * 1.2, (V - h / 2) / f * 1.2
    depth = 1.205 + 0.03 * np.sin(9 * X + 0.05) * np.cos(7 * Y - 0.04) + rng.normal(0, 1e-3, (h, w))
    return dict(pos=pos.astype(np.float32), nrm=nrm.astype(np.float32), nodes=nodes, depth=depth.astype(np.float32),
                cfg=dict(width=w, height=h, fx=f, fy=f, cx=w / 2, cy=h / 2, node_sigma=float(spacing), gn_iters=3))


def _stream(swgn, s, **cfg):
    st = swgn.Stream(swgn.sw_config_default(**{**s["cfg"], **cfg}))
    st.set_reference_surfels(s["pos"], s["nrm"])
    st.set_node_graph(s["nodes"])
    return st


def _same(a, b, what):
    for k in ("n_corr", "e_data", "e_reg", "pcg_resid"):
        assert a[0][k] == b[0][k], (what, k)
    assert np.array_equal(a[1], b[1]), what


def _steps(swgn, s, frames=1, **cfg):
    """The step-wise result."""
    st, bx = _stream(swgn, s, **cfg), swgn.Batch(pcg="split")
    for _ in range(frames):
        stats, _ = bx.solve([st], [s["depth"]])
    out = stats[0], st.node_se3()
    bx.close()
    st.close()
    return out


def _whole(stats):
    return stats["stage_us"][3] > 0 and all(stats["stage_us"][k] == 0 for k in STEP_SLOTS)


# 9: the fewest nodes; 32 and 64 rows per workgroup of 4 and 8 waves, one
# workgroup or several; 2049 parts' leaves taken in a second round
@pytest.mark.parametrize("n_nodes,pcg", [(9, 10), (31, 10), (32, 3), (33, 10), (40, 1), (63, 10), (64, 2), (65, 10),
                                         (257, 25), (2047, 10), (2049, 10), (4100, 4)])
def test_whole_solve_equals_steps(swgn, n_nodes, pcg):
    s = _surface(n_nodes, n_nodes)
    want = _steps(swgn, s, pcg_iters=pcg)
    st = _stream(swgn, s, pcg_iters=pcg, stage_timing=1)
    got = st.solve_frame(s["depth"]), st.node_se3()
    st.close()
    assert _whole(got[0])
    _same(got, want, n_nodes)


def test_node_set_that_does_not_fit_is_solved_in_steps(swgn):
    """Nodes through a volume: rows and foreign columns beyond what a workgroup holds."""
    s = _surface(1500, 5, volume=True)
    want = _steps(swgn, s, damping=1.0)
    st = _stream(swgn, s, stage_timing=1, damping=1.0)
    got = st.solve_frame(s["depth"]), st.node_se3()
    st.close()
    assert not _whole(got[0])
    _same(got, want, "volume")


@pytest.mark.parametrize("sizes,graph", [((4100, 33, 4100, 700), False),          # workgroups of 8 waves
                                         ((4100, 65, 4000, 9, 3900, 4100), True)])  # more than the chip holds at once
def test_many_streams_in_one_launch(swgn, sizes, graph):
    scenes = [_surface(n, 100 + k) for k, n in enumerate(sizes)]
    want = [_steps(swgn, s, frames=2) for s in scenes]
    sts = [_stream(swgn, s) for s in scenes]
    bx = swgn.Batch(graph=graph)
    for _ in range(2):
        stats, _ = bx.solve(sts, [s["depth"] for s in scenes])
    for k, st in enumerate(sts):
        _same((stats[k], st.node_se3()), want[k], sizes[k])
        st.close()
    bx.close()


def test_two_threads_share_the_device(swgn):
    """Batches that together need more workgroups than the device holds, from
    two threads: whoever finds too few left solves in steps, with equal results."""
    scenes = [[_surface(n, 7 * k + 1) for n in (4100, 3000)] for k in range(2)]
    want = [[_steps(swgn, s, frames=4) for s in group] for group in scenes]
    got, errors = [None, None], []

    def work(k):
        try:
            sts = [_stream(swgn, s) for s in scenes[k]]
            bx = swgn.Batch()
            for _ in range(4):
                stats, _ = bx.solve(sts, [s["depth"] for s in scenes[k]])
            got[k] = [(stats[i], st.node_se3()) for i, st in enumerate(sts)]
        except Exception as e:                                  # (reported by the main thread)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k in range(2):
        for a, b in zip(got[k], want[k]):
            _same(a, b, k)


def test_a_solve_that_gives_up_waiting_is_done_again_in_steps(swgn, monkeypatch):
    """With no patience at all the first word that is not there yet ends the
    wait: the frame comes out right all the same, alone, batched and served."""
    scenes = [_surface(n, n) for n in (300, 900)]
    want = [_steps(swgn, s, frames=2) for s in scenes]
    monkeypatch.setenv("SWGN_PCG_WAIT_US", "-1")
    st = _stream(swgn, scenes[0], stage_timing=1)
    for _ in range(2):
        stats = st.solve_frame(scenes[0]["depth"])
    assert not _whole(stats)
    _same((stats, st.node_se3()), want[0], "alone")
    st.close()
    sts = [_stream(swgn, s) for s in scenes]
    bx = swgn.Batch()
    for _ in range(2):
        stats, status = bx.solve(sts, [s["depth"] for s in scenes])
    assert status == [swgn.SW_OK] * 2
    for k, st in enumerate(sts):
        _same((stats[k], st.node_se3()), want[k], "batch")
        st.close()
    bx.close()
    sts = [_stream(swgn, s) for s in scenes]
    sv = swgn.Server()
    for st in sts:
        sv.attach(st)
    for _ in range(2):
        tickets = [sv.submit(st, s["depth"]) for st, s in zip(sts, scenes)]
        done = [sv.poll(t) for t in tickets]
    for k, st in enumerate(sts):
        assert done[k][1]["status"] == swgn.SW_OK
        _same((done[k][0], st.node_se3()), want[k], "served")
    sv.close()
    for st in sts:
        st.close()


# a nearly flat sheet, whose node order jumps about in it: 148 and 201 foreign
# columns in a tile of 32 rows, so 6 and 8 sets of local nodes, one workgroup per CU
@pytest.mark.parametrize("n_nodes", [600, 1000])
def test_workgroups_with_many_foreign_columns_equal_steps(swgn, n_nodes):
    s = _surface(n_nodes, n_nodes)
    s["nodes"][:, 2] = 1.2 - np.random.default_rng(1).uniform(0, 0.1 * s["cfg"]["node_sigma"], n_nodes)
    want = _steps(swgn, s, frames=2)
    st = _stream(swgn, s, stage_timing=1)
    for _ in range(2):
        stats = st.solve_frame(s["depth"])
    assert _whole(stats)
    _same((stats, st.node_se3()), want, n_nodes)
    st.close()
    # beside a stream whose tiles have few of them
    pair = [s, _surface(900, 3)]
    want = [_steps(swgn, q, frames=2) for q in pair]
    sts = [_stream(swgn, q) for q in pair]
    bx = swgn.Batch()
    for _ in range(2):
        stats, _ = bx.solve(sts, [q["depth"] for q in pair])
    for k, st in enumerate(sts):
        _same((stats[k], st.node_se3()), want[k], (n_nodes, k))
        st.close()
    bx.close()
