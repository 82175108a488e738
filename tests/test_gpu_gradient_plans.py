"""Gradients whose checkpoint intervals the planner chose (E of every step kept
out by a share of zero): one level, reused, in groups of sources, on multiples
of the graph length, each equal bit for bit to the gradient with E of every
step kept."""
import ctypes as C

import numpy as np
import pytest

from workloads import configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def emm():
    from paper_2304_00233_amd import emm as m
    m._lib.emm_test_snapshots.argtypes = [C.c_void_p, C.c_double]
    return m


@pytest.mark.parametrize("rd,nsrc,opt", [(2, 1, {}), (2, 1, dict(graph_steps=8)), (4, 1, {}), (2, 3, dict(src_group=2)),
                                         (1, 3, dict(src_group=2, graph_steps=8)), (2, 2, dict(checkpoint_inner=5))])
def test_planned_intervals_give_the_same_gradient(emm, rd, nsrc, opt):
    w = configs.small_case(seed=80 + rd, shape=(22, 21, 20), rd=rd, nb=5, ne=rd + 2, nt=53, nsrc=nsrc)
    bar = np.ones((nsrc, 7, 6, 2), complex)
    print(f"[gpu] planned gradient r{rd} nsrc{nsrc} {opt}", flush=True)
    with emm.Model(w) as m:
        ref, G, _ = m.gradient(g_bar=bar)
        assert m.info()["ckpt_outer"] == m.info()["ckpt_inner"] == 53
    with emm.Model(w, **opt) as m:
        assert emm._lib.emm_test_snapshots(m.h, 0.0) == 0
        for _ in range(2):                       # the second reuses the run where all sources are in one group
            g, G1, _ = m.gradient(g_bar=bar)
            i = m.info()
            assert 0 < i["ckpt_inner"] <= i["ckpt_outer"] < 53 or "checkpoint_inner" in opt
            if "graph_steps" in opt:
                assert i["ckpt_outer"] % 8 == 0
            assert np.array_equal(G1, G) and np.array_equal(g, ref)
        assert emm._lib.emm_test_snapshots(m.h, 0.125) == 0
        m.gradient(g_bar=bar[:1], sources=w.sources[:1])             # from planned to whole, another layout
        g, G1, _ = m.gradient(g_bar=bar)
        assert np.array_equal(G1, G) and np.array_equal(g, ref)
