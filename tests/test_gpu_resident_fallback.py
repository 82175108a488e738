"""The way back from resident time loops: a wait that gives up (no patience)
or a cooperative launch that is refused sends the run to the half-step
launches, with the same results, and the model keeps to them."""
import ctypes as C

import numpy as np
import pytest

from workloads import configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def emm():
    from paper_2304_00233_amd import emm as m
    m._lib.emm_test_resident.argtypes = [C.c_void_p, C.c_double, C.c_int]
    m._lib.emm_test_tuned.argtypes = [C.c_void_p]
    return m


@pytest.fixture(scope="module")
def w():
    return configs.small_case(seed=61, shape=(24, 21, 19), rd=2, nb=5, nt=70)


BAR = np.ones((1, 7, 6, 2), complex)
# no patience; the first, third launch refused
LIMITS = [(0.0, -1), (2.0, 0), (2.0, 2)]


@pytest.fixture(scope="module")
def ref(emm, w):
    with emm.Model(w, src_order=0) as m:
        G = m.forward()
        return G, m.gradient(g_bar=BAR)[0]


def _limit(emm, m, patience, launches):
    assert emm._lib.emm_test_resident(m.h, patience, launches) == 0


@pytest.mark.parametrize("patience,launches", LIMITS)
@pytest.mark.parametrize("noalloc", [False, True])
def test_forward(emm, w, ref, patience, launches, noalloc):
    opt = {} if noalloc else dict(checkpoint_every=20)       # four launches
    print(f"[gpu] forward, patience {patience} launches {launches} noalloc {noalloc}", flush=True)
    with emm.Model(w, **opt) as m:
        _limit(emm, m, patience, launches)
        for _ in range(3):
            assert np.array_equal(m.forward(noalloc=noalloc), ref[0])
        assert m.info()["resident"] == 0
        _limit(emm, m, 2.0, -1)
        assert np.array_equal(m.forward(noalloc=noalloc), ref[0]) and m.info()["resident"] == 0


@pytest.mark.parametrize("patience,launches", LIMITS[:2])
def test_gradient_with_every_step_kept(emm, w, ref, patience, launches):
    print(f"[gpu] gradient, every step kept, patience {patience} launches {launches}", flush=True)
    with emm.Model(w) as m:
        _limit(emm, m, patience, launches)
        g, G, _ = m.gradient(g_bar=BAR)
        assert np.array_equal(G, ref[0]) and np.array_equal(g, ref[1]) and m.info()["resident"] == 0


@pytest.mark.parametrize("patience,launches", LIMITS)
@pytest.mark.parametrize("every,inner", [(16, 0), (30, 7)])
def test_gradient_recompute(emm, w, ref, patience, launches, every, inner):
    """The forward runs resident; its segments' recomputation gives up."""
    print(f"[gpu] recompute, patience {patience} launches {launches} every {every} inner {inner}", flush=True)
    with emm.Model(w, checkpoint_every=every, checkpoint_inner=inner) as m:
        assert np.array_equal(m.forward(), ref[0]) and m.info()["resident"] > 0
        _limit(emm, m, patience, launches)
        g, G, _ = m.gradient(g_bar=BAR)
        assert np.array_equal(G, ref[0]) and np.array_equal(g, ref[1])


@pytest.mark.parametrize("every,inner", [(16, 0), (30, 7)])
def test_gradient_gives_up_then_is_refused(emm, w, ref, every, inner):
    """The first recomputed stretch runs out of patience, the next launch is
    refused: what the first left behind does not count."""
    print(f"[gpu] recompute gives up, then refused, every {every} inner {inner}", flush=True)
    with emm.Model(w, checkpoint_every=every, checkpoint_inner=inner) as m:
        assert np.array_equal(m.forward(), ref[0]) and m.info()["resident"] > 0
        _limit(emm, m, 0.0, 1)
        g, G, _ = m.gradient(g_bar=BAR)
        assert np.array_equal(G, ref[0]) and np.array_equal(g, ref[1])


def test_autotuned_where_the_launches_run(emm, w, ref):
    """tile_kz = -1 measures the launches when a time loop uses them: not
    before a resident loop, but after its refusal, and for a checkpointed
    forward, whose launch shapes the gradient's reverse sweep takes."""
    print("[gpu] autotuning beside resident loops", flush=True)
    with emm.Model(w, tile_kz=-1) as m:
        assert np.array_equal(m.forward(), ref[0]) and m.info()["resident"] > 0
        assert emm._lib.emm_test_tuned(m.h) == 0
        _limit(emm, m, 2.0, 0)
        assert np.array_equal(m.forward(), ref[0]) and m.info()["resident"] == 0
        assert emm._lib.emm_test_tuned(m.h) == 1
        assert np.array_equal(m.forward(), ref[0]) and emm._lib.emm_test_tuned(m.h) == 1
    with emm.Model(w, tile_kz=-1, checkpoint_every=20) as m:
        assert np.array_equal(m.forward(), ref[0]) and m.info()["resident"] > 0
        assert emm._lib.emm_test_tuned(m.h) == 1
        assert np.array_equal(m.gradient(g_bar=BAR)[0], ref[1])


def test_no_model_tries_for_a_while_after_a_refusal(emm, w, ref):
    emm._lib.emm_test_refusal.argtypes = [C.c_int, C.c_double]
    print("[gpu] resident loops after a refusal by the device", flush=True)
    try:
        assert emm._lib.emm_test_refusal(0, 100.0) == 0
        for _ in range(2):
            with emm.Model(w) as m:
                assert np.array_equal(m.forward(), ref[0]) and m.info()["resident"] == 0
                assert np.array_equal(m.gradient(g_bar=BAR)[0], ref[1])
    finally:
        emm._lib.emm_test_refusal(0, 0.0)
    with emm.Model(w) as m:
        assert np.array_equal(m.forward(), ref[0]) and m.info()["resident"] > 0
