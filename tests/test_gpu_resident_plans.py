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
    with emm.Model(w) as m:
        assert np.array_equal(m.forward(), ref)
    opt = dict(checkpoint_every=16)                # recomputed, E of every step to the snapshots
    bar = np.ones((1, 7, 6, 2), complex)
    with emm.Model(w, src_order=0, **opt) as m:
        g0, _, _ = m.gradient(g_bar=bar)
    with emm.Model(w, **opt) as m:
        g1, _, _ = m.gradient(g_bar=bar)
    assert np.array_equal(g0, g1)
