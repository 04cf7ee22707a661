"""Which way the linear solves run, by the stream's own counts: batches (with
and without a HIP graph), two threads and the serving loop take whole solves,
and where one gives up waiting its frame is done again step by step."""
import threading

import numpy as np
import pytest

from gpu_common import gpu_lib
from test_gpu_pcg_solve import _same, _steps, _stream, _surface

pytestmark = pytest.mark.gpu

GN = 3                                                              # (of the scenes)


@pytest.fixture(scope="module")
def swgn():
    return gpu_lib()


def _solves(st):
    c = st.solve_counts()
    return c["whole"], c["stepwise"], c["redone"]


@pytest.mark.parametrize("sizes,graph", [((4100, 33, 4100, 700), False), ((4100, 65, 4000, 9, 3900, 4100), False),
                                         ((4100, 65, 4000, 9, 3900, 4100), True)])
def test_a_batch_alone_on_the_device_solves_whole(swgn, sizes, graph):
    scenes = [_surface(n, 100 + k) for k, n in enumerate(sizes)]
    sts = [_stream(swgn, s) for s in scenes]
    bx = swgn.Batch(graph=graph)
    for _ in range(3):
        bx.solve(sts, [s["depth"] for s in scenes])
    for st in sts:
        assert _solves(st) == (3 * GN, 0, 0)
        assert st.solve_counts()["captures"] == (1 if graph else 0)
        st.close()
    bx.close()


def test_a_fixed_schedule_and_a_node_set_that_does_not_fit_solve_in_steps(swgn):
    st, bx = _stream(swgn, _surface(300, 300)), swgn.Batch(pcg="split")
    bx.solve([st], [_surface(300, 300)["depth"]])
    assert _solves(st) == (0, GN, 0)
    s = _surface(1500, 5, volume=True)
    big = _stream(swgn, s, damping=1.0)
    big.solve_frame(s["depth"])
    assert _solves(big) == (0, GN, 0)
    for x in (bx, st, big):
        x.close()


def test_threads_beside_each_other_take_whole_solves(swgn):
    scenes = [[_surface(n, 7 * k + 1) for n in (4100, 3000)] for k in range(2)]
    counts, errors = [None, None], []

    def work(k):
        try:
            sts = [_stream(swgn, s) for s in scenes[k]]
            bx = swgn.Batch()
            for _ in range(8):
                bx.solve(sts, [s["depth"] for s in scenes[k]])
            counts[k] = [st.solve_counts() for st in sts]
        except Exception as e:                                      # (reported by the main thread)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for c in (c for group in counts for c in group):
        assert c["whole"] > 0 and c["whole"] + c["stepwise"] == 8 * GN and c["redone"] == 0


@pytest.mark.parametrize("how", ["alone", "batch", "graph", "served"])
def test_a_wait_given_up_redoes_the_frame(swgn, monkeypatch, how):
    monkeypatch.setenv("SWGN_PCG_WAIT_US", "-1")
    scenes = [_surface(n, n) for n in (300, 900)]
    sts = [_stream(swgn, s) for s in scenes]
    depths = [s["depth"] for s in scenes]
    if how == "alone":
        stats = [st.solve_frame(d) for st, d in zip(sts, depths)]
    elif how == "served":
        sv = swgn.Server()
        for st in sts:
            sv.attach(st)
        stats = [sv.poll(t)[0] for t in [sv.submit(st, d) for st, d in zip(sts, depths)]]
        sv.close()
    else:
        bx = swgn.Batch(graph=how == "graph")
        stats, _ = bx.solve(sts, depths)
        bx.close()
    counts = [st.solve_counts() for st in sts]
    for st, s, r, c in zip(sts, scenes, stats, counts):
        _same((r, st.node_se3()), _steps(swgn, s), how)
        assert (c["waits"] > 0) == (c["redone"] > 0)
        assert c["stepwise"] == GN or (how == "served" and c["stepwise"] > GN)
        st.close()
    # (served: a frame that another's given-up wait overtakes goes on in steps, and its own is redone or not)
    assert [c["redone"] for c in counts] == [1, 1] or (how == "served" and sum(c["redone"] for c in counts) == 1)


@pytest.mark.parametrize("how", ["alone", "batch"])
def test_a_frame_waits_once(swgn, monkeypatch, how):
    """Once a wave has given up, nothing of the frame waits any more: the waits
    given up are at most the waves of one solve, not those of every iteration."""
    monkeypatch.setenv("SWGN_PCG_WAIT_US", "-1")
    s = _surface(900, 900)
    st = _stream(swgn, s, gn_iters=16)
    if how == "alone":
        st.solve_frame(s["depth"])
    else:
        bx = swgn.Batch()
        bx.solve([st], [s["depth"]])
        bx.close()
    c = st.solve_counts()
    st.close()
    assert c["redone"] == 1 and c["whole"] == 16
    assert 0 < c["waits"] <= -(-900 // 8)                           # (8 rows per wave)


@pytest.mark.parametrize("how", ["alone", "batch", "served"])
def test_whole_solves_are_tried_again_after_a_wait_given_up(swgn, monkeypatch, how):
    """A wait given up (forced on one node graph only) costs the next 64
    frames the whole solve, not all that follow."""
    s = _surface(300, 300)
    monkeypatch.setenv("SWGN_PCG_WAIT_US", "-1")
    bad, st = _stream(swgn, s), None
    monkeypatch.delenv("SWGN_PCG_WAIT_US")
    st = _stream(swgn, s)
    if how == "alone":
        st.close()
        st = bad
        solve = lambda x: x.solve_frame(s["depth"])
        solve(bad)
        bad.set_node_graph(s["nodes"])                              # (with patience)
    elif how == "batch":
        ex = swgn.Batch()
        solve = lambda x: ex.solve([x], [s["depth"]])
        solve(bad)
    else:
        ex = swgn.Server()
        ex.attach(bad)
        ex.attach(st)
        solve = lambda x: ex.poll(ex.submit(x, s["depth"]))
        solve(bad)
    assert bad.solve_counts()["redone"] == 1
    before = st.solve_counts()
    for _ in range(60):
        solve(st)
    c = st.solve_counts()
    assert c["whole"] == before["whole"] and c["stepwise"] == before["stepwise"] + 60 * GN
    for _ in range(400):                                            # (served: a frame's most iterations count, not its own)
        solve(st)
    c = st.solve_counts()
    assert c["whole"] > before["whole"] and c["redone"] == before["redone"]
    if how != "alone":
        ex.close()
        bad.close()
    st.close()


def test_waits_given_up_again_and_again_become_rare(swgn, monkeypatch):
    monkeypatch.setenv("SWGN_PCG_WAIT_US", "-1")
    s = _surface(300, 300)
    st = _stream(swgn, s, gn_iters=1)
    for _ in range(500):                                            # frames 1, 65, 193, 449 (and their second solves)
        st.solve_frame(s["depth"])
    c = st.solve_counts()
    st.close()
    assert 3 <= c["redone"] <= 4


def test_mixed_workgroups_from_many_threads_never_wait_in_vain(swgn):
    """Executors whose solves take a CU per workgroup (a full batch; a sheet
    whose tiles have many foreign columns), share CUs, or are one workgroup:
    beside each other no solve gives up waiting, and the smallest need no room."""
    sheet = _surface(1000, 1000)
    sheet["nodes"][:, 2] = 1.2 - np.random.default_rng(1).uniform(0, 0.1 * sheet["cfg"]["node_sigma"], 1000)
    groups = [[_surface(4100, k) for k in range(5)], [sheet], [_surface(2000, 1)], [_surface(1700, 2), _surface(900, 3)],
              [_surface(40, 4)], [_surface(3500, 5)]]
    want = [[_steps(swgn, s, frames=30) for s in g] for g in groups]
    got, counts, errors = {}, {}, []
    start = threading.Barrier(len(groups))

    def work(k):
        try:
            sts = [_stream(swgn, s) for s in groups[k]]
            bx = swgn.Batch()
            start.wait()
            for _ in range(30):
                stats, _ = bx.solve(sts, [s["depth"] for s in groups[k]])
            got[k] = [(r, st.node_se3()) for r, st in zip(stats, sts)]
            counts[k] = [st.solve_counts() for st in sts]
        except Exception as e:                                      # (reported by the main thread)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(groups))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k, g in enumerate(groups):
        for i in range(len(g)):
            _same(got[k][i], want[k][i], (k, i))
            c = counts[k][i]
            assert c["redone"] == c["waits"] == 0 and c["whole"] + c["stepwise"] == 30 * GN
    assert counts[4][0]["stepwise"] == 0
    assert sum(c["whole"] for g in counts.values() for c in g) > 0


def test_graphs_beside_other_executors_are_captured_once_per_way_of_launching(swgn):
    """What a graph executor may launch at once varies with what others hold;
    the graph follows the launches, not the number: a pair of streams has both
    in one launch, one after the other, or in steps."""
    scenes = [_surface(n, n) for n in (4100, 4090)]
    want = [_steps(swgn, s, frames=60) for s in scenes]
    sts = [_stream(swgn, s) for s in scenes]
    done, errors = threading.Event(), []

    def beside(k):
        try:
            s = _surface((3000, 3300, 900)[k], k)
            st, bx = _stream(swgn, s), swgn.Batch()
            while not done.is_set():
                bx.solve([st], [s["depth"]])
            bx.close()
            st.close()
        except Exception as e:                                      # (reported by the main thread)
            errors.append(e)

    threads = [threading.Thread(target=beside, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    bx = swgn.Batch(graph=True)
    try:
        for _ in range(60):
            stats, _ = bx.solve(sts, [s["depth"] for s in scenes])
    finally:
        done.set()
        for t in threads:
            t.join()
    assert not errors, errors
    for st, r, w in zip(sts, stats, want):
        _same((r, st.node_se3()), w, "graph")
        assert 1 <= st.solve_counts()["captures"] <= 3 and st.solve_counts()["redone"] == 0
        st.close()
    bx.close()


def test_a_single_pcg_iteration_runs_in_steps(swgn):
    """(Faster than a solve whose workgroups exchange its only sums.)"""
    s = _surface(300, 300)
    for pcg in (1, 2):
        st = _stream(swgn, s, pcg_iters=pcg)
        got = st.solve_frame(s["depth"]), st.node_se3()
        assert _solves(st) == ((0, GN, 0) if pcg == 1 else (GN, 0, 0))
        _same(got, _steps(swgn, s, pcg_iters=pcg), pcg)
        st.close()
