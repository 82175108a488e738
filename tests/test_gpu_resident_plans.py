"""Resident time loops over grids whose plans differ in planes per thread and
thread groups, against the half-step launches: equal bit for bit."""
import numpy as np
import pytest

from tests.test_resident_plan import GRIDS
from workloads import configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def emm():
    from paper_2304_00233_amd import emm as m
    return m


@pytest.mark.parametrize("shape,rd,nb,ne,planes,several", GRIDS)
def test_every_plan_equals_half_step_launches(emm, shape, rd, nb, ne, planes, several):
    w = configs.small_case(seed=sum(shape), shape=shape, rd=rd, nb=nb, ne=ne, nt=47)
    print(f"[gpu] resident {shape} r{rd} planes {planes} several groups {several}", flush=True)
    with emm.Model(w, src_order=0) as m:
        ref = m.forward()
        assert m.info()["resident"] == 0
    with emm.Model(w) as m:
        assert np.array_equal(m.forward(), ref) and m.info()["resident"] == planes
        assert np.array_equal(m.forward(noalloc=True), ref) and m.info()["resident"] == planes
    opt = dict(checkpoint_every=16)                # recomputed, E of every step to the snapshots
    bar = np.ones((1, 7, 6, 2), complex)
    with emm.Model(w, src_order=0, **opt) as m:
        g0, _, _ = m.gradient(g_bar=bar)
    with emm.Model(w, **opt) as m:
        g1, _, _ = m.gradient(g_bar=bar)
        assert m.info()["resident"] == planes
    assert np.array_equal(g0, g1)


def test_which_loops_run_resident(emm):
    """One plane per thread: one and two sources; more: one source; every
    option that is set selects the half-step launches."""
    w = configs.small_case(seed=3, shape=(24, 22, 20), nt=20, nsrc=3)
    two = dict(sources=w.sources[:2], src_comp=w.src_comp[:2])
    one = dict(sources=w.sources[:1], src_comp=w.src_comp[:1])
    with emm.Model(w) as m:
        for kw, planes in ((one, 1), (two, 1), ({}, 0), (one, 1)):
            m.forward(**kw)
            assert m.info()["resident"] == planes
        emm.forward_models([m])
        assert m.info()["resident"] == 0
        m.gradient(g_bar=np.ones((1, 7, 6, 2), complex), **one)        # E of every step kept
        assert m.info()["resident"] == 1
    for opt in (dict(tile_kz=4), dict(tile_x=64), dict(tile_rows=1), dict(nontemporal=0), dict(ce_table=0),
                dict(src_order=0), dict(profile=1), dict(fused=1), dict(converge_tol=1e-9)):
        with emm.Model(w, **opt) as m:
            m.forward(**one)
            assert m.info()["resident"] == 0, opt


def test_profiled_gradient_with_every_step_kept(emm):
    """profile = 1 times the stencil launches of a gradient's forward also when
    that keeps E of every step."""
    w = configs.small_case(seed=4, shape=(24, 22, 20), nt=53)
    bar = np.ones((1, 7, 6, 2), complex)
    with emm.Model(w) as m:
        ref, _, _ = m.gradient(g_bar=bar)
    for opt in ({}, dict(checkpoint_every=20)):
        with emm.Model(w, profile=1, **opt) as m:
            g, _, _ = m.gradient(g_bar=bar)
            i = m.info()
        assert np.array_equal(g, ref) and i["resident"] == 0
        assert i["e_launches"] == i["h_launches"] == 4
        assert 0 < i["e_kernel_ms"] < i["forward_ms"] and 0 < i["h_kernel_ms"] < i["forward_ms"]


def test_resident_loops_of_several_threads(emm):
    """One model per thread, each on its own stream: cooperative launches take
    turns, half-step launches of other threads run beside them."""
    import threading
    w = configs.small_case(seed=5, shape=(30, 28, 26), nt=80)
    with emm.Model(w, src_order=0) as m:
        ref = m.forward()
    got = []

    def work(opt):
        with emm.Model(w, **opt) as m:
            for _ in range(4):
                got.append((np.array_equal(m.forward(), ref), m.info()["resident"] > 0))

    print("[gpu] resident loops of three threads beside one of launches", flush=True)
    threads = [threading.Thread(target=work, args=(opt,)) for opt in ({}, {}, {}, dict(src_order=0))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(got) == 16 and all(same for same, _ in got)
    assert sum(resident for _, resident in got) == 12
