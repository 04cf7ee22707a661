"""Device memory that a stream keeps from one model for the next: bounded by
the model it has, whatever came before it."""
import numpy as np
import pytest

from gpu_common import gpu_lib

pytestmark = pytest.mark.gpu

MIB = 1 << 20


@pytest.fixture(scope="module")
def swgn():
    return gpu_lib()


def _free():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def _cloud(n_surfels, n_nodes, seed=0):
    rng = np.random.default_rng(seed)
    pos = rng.uniform(0, 1, (n_surfels, 3)).astype(np.float32)
    nodes = rng.uniform(0, 1, (n_nodes, 3)).astype(np.float32)
    pos[:, 2] *= 0.02
    nodes[:, 2] *= 0.02
    nrm = np.zeros_like(pos)
    nrm[:, 2] = -1.0
    return pos, nrm, nodes


def _new_stream(swgn):
    return swgn.Stream(swgn.sw_config_default(width=64, height=48, fx=50.0, fy=50.0, cx=32.0, cy=24.0, node_sigma=0.05))


def _install(st, model):
    st.set_reference_surfels(model[0], model[1])
    st.set_node_graph(model[2])


# surfels, nodes of models that shrink by less than four times each
@pytest.mark.parametrize("models", [[(1200000, 600), (400000, 600), (120000, 600), (40000, 600)],
                                    [(60000, 24000), (50000, 8000), (50000, 2500), (50000, 700)]])
def test_a_model_after_larger_ones_holds_memory_of_its_own_size(swgn, models):
    clouds = [_cloud(*m) for m in models]
    one = _new_stream(swgn)
    _install(one, clouds[-1])                       # (whatever the first install of a process allocates once)
    before = _free()
    fresh = _new_stream(swgn)
    _install(fresh, clouds[-1])
    alone = before - _free()
    before = _free()
    st = _new_stream(swgn)
    for c in clouds:
        _install(st, c)
    held = before - _free()
    want = fresh.skinning(), fresh.pattern()
    got = st.skinning(), st.pattern()
    for a, b in zip(got, want):
        assert all(np.array_equal(x, y) for x, y in zip(a, b))
    for x in (one, fresh, st):
        x.close()
    # (a model up to four times as large may still be held, and chunks are rounded up)
    assert held <= 4 * alone + 64 * MIB, (held // MIB, alone // MIB)


def test_a_first_model_does_not_wait_for_other_streams(swgn):
    """Surfels set on a fresh stream reuse no memory, so they wait for no work
    of the device but their own."""
    import torch
    pos, nrm, nodes = _cloud(5000, 60)
    warm, st = _new_stream(swgn), _new_stream(swgn)
    _install(warm, (pos, nrm, nodes))
    side, done = torch.cuda.Stream(), torch.cuda.Event()
    with torch.cuda.stream(side):
        torch.cuda._sleep(20_000_000)                               # (loads the kernel)
        side.synchronize()
        torch.cuda._sleep(2_000_000_000)
        done.record()
    st.set_reference_surfels(pos, nrm)
    running = not done.query()
    side.synchronize()
    st.set_node_graph(nodes)
    assert running
    assert np.array_equal(st.skinning()[0], warm.skinning()[0])
    st.close()
    warm.close()


def test_a_model_that_fits_without_the_kept_memory_is_installed(swgn):
    """A model of less than twice the last one's surfels takes over its memory;
    where the two together are more than the device has left, what was kept is
    given back and the model still fits, as on a fresh stream."""
    import torch
    first, second = _cloud(1500000, 2500, 1), _cloud(2900000, 2500, 2)
    warm = _new_stream(swgn)
    _install(warm, _cloud(5000, 60))
    before = _free()
    fresh = _new_stream(swgn)
    _install(fresh, second)
    alone = before - _free()
    want = fresh.skinning()[0], fresh.layout()
    fresh.close()
    before = _free()
    both = _new_stream(swgn)
    _install(both, first)
    _install(both, second)
    together = before - _free()
    both.close()
    assert together > alone + 100 * MIB
    # fill the device so that `second` fits with half of the difference to spare
    spare = alone + (together - alone) // 2
    fill = []
    while (left := _free() - spare) > 2 * MIB:
        try:
            fill.append(torch.empty(min(left, 32 << 30) // (2 * MIB) * (2 * MIB), dtype=torch.uint8, device="cuda"))
        except torch.cuda.OutOfMemoryError:                         # (what is left is in pieces)
            break
    st = _new_stream(swgn)
    try:
        _install(st, first)
        _install(st, second)
        got = st.skinning()[0], st.layout()
    finally:
        st.close()
        del fill
        torch.cuda.empty_cache()
        warm.close()
    assert np.array_equal(got[0], want[0]) and got[1] == want[1]


def test_the_footprint_is_the_memory_held(swgn):
    """What the stream reports is what the device has less for it, after
    each step that allocates (within the device's own rounding of allocations)."""
    pos, nrm, nodes = _cloud(300000, 2000)
    depth = np.full((48, 64), 2.0, np.float32)
    warm = _new_stream(swgn)
    _install(warm, _cloud(5000, 60))
    warm.solve_frame(depth)
    warm.fuse_frame(depth, 1)
    warm.update_geometry()
    before = _free()
    st = _new_stream(swgn)

    def check(what):
        held, told = before - _free(), sum(st.footprint())
        assert abs(held - told) <= 24 * MIB, (what, held // MIB, told // MIB)

    _install(st, (pos, nrm, nodes))
    check("a model")
    for k in range(2):
        st.fuse_frame(depth, 1 + k)
        st.update_geometry()
        check("an update")
    _install(st, (pos[:100000], nrm[:100000], nodes))
    check("a smaller model")
    st.close()
    warm.close()
