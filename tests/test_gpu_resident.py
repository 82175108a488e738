"""Whole time loops in one launch (small grids, one or two sources) against
the launch-per-half-step kernels, which any launch option selects: the same
arithmetic in the same order, so the results are equal bit for bit."""
import numpy as np
import pytest

from workloads import configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def emm():
    from paper_2304_00233_amd import emm as m
    return m


# shape, rd, nb, ne, sources: tiles of uneven rows and planes, one plane per
# thread and (48^3) five, no CPML, the smallest grids; the plans between are in
# test_gpu_resident_plans.py
CASES = [((30, 26, 22), 2, 6, 4, 1), ((37, 29, 23), 1, 10, 6, 1), ((48, 48, 48), 2, 10, 7, 1),
         ((48, 48, 48), 1, 10, 6, 1), ((21, 19, 33), 3, 5, 4, 1), ((14, 15, 13), 2, 0, 3, 2),
         ((70, 12, 11), 2, 4, 3, 2), ((9, 60, 40), 1, 3, 2, 1), ((33, 9, 50), 3, 2, 3, 2)]


@pytest.mark.parametrize("shape,rd,nb,ne,nsrc", CASES)
@pytest.mark.parametrize("dft", [0, 1])
def test_resident_equals_half_step_launches(emm, shape, rd, nb, ne, nsrc, dft):
    w = configs.small_case(seed=sum(shape) + rd, shape=shape, rd=rd, nb=nb, ne=ne, nsrc=nsrc, nt=61,
                           src_comp=np.arange(nsrc) % 3).with_(dft_mode=dft)
    print(f"[gpu] resident {shape} r{rd} nb{nb} nsrc{nsrc} dft{dft}", flush=True)
    with emm.Model(w, src_order=0) as m:
        ref = m.forward()
    with emm.Model(w) as m:
        assert np.array_equal(m.forward(), ref)
        assert np.array_equal(m.forward(), ref)              # again on the same mailbox
        assert np.array_equal(m.forward(noalloc=True), ref)
    with emm.Model(w, checkpoint_every=20) as m:             # several launches
        assert np.array_equal(m.forward(), ref)


@pytest.mark.parametrize("rd,every,inner", [(1, 16, 0), (2, 25, 0), (2, 30, 7), (3, 20, 0)])
def test_gradient_recomputed_resident(emm, rd, every, inner):
    w = configs.small_case(seed=40 + rd, shape=(24, 21, 19), rd=rd, nb=5, ne=rd + 2, nt=70)
    opt = dict(checkpoint_every=every, checkpoint_inner=inner)
    print(f"[gpu] resident gradient r{rd} every {every} inner {inner}", flush=True)
    with emm.Model(w, src_order=0, **opt) as m:
        g0, G0, _ = m.gradient(g_bar=np.ones((1, 7, 6, 2), complex))
    with emm.Model(w, **opt) as m:
        g1, G1, _ = m.gradient(g_bar=np.ones((1, 7, 6, 2), complex))
    assert np.array_equal(G0, G1) and np.array_equal(g0, g1)


@pytest.mark.parametrize("rd,nsrc,opt", [(2, 1, {}), (2, 1, dict(src_order=0)), (2, 3, dict(graph_steps=8)),
                                         (4, 2, {}), (1, 2, {})])
def test_gradient_with_every_step_kept(emm, rd, nsrc, opt):
    """Planned intervals keep E of every step when it is small: the same
    gradient as from checkpoints, also when the next call reuses the run and
    when another source has used the snapshots in between."""
    w = configs.small_case(seed=50 + rd, shape=(22, 21, 20), rd=rd, nb=5, ne=rd + 2, nt=53, nsrc=nsrc)
    bar = np.ones((nsrc, 7, 6, 2), complex)
    print(f"[gpu] gradient, every step kept r{rd} nsrc{nsrc} {opt}", flush=True)
    with emm.Model(w, checkpoint_every=20, **opt) as m:
        g0, G0, _ = m.gradient(g_bar=bar)
    with emm.Model(w, **opt) as m:
        g1, G1, _ = m.gradient(g_bar=bar)
        i = m.info()
        assert i["ckpt_outer"] == i["ckpt_inner"] == 53 and i["ckpt_bytes"] > 0
        g2, G2, _ = m.gradient(g_bar=bar)
        m.gradient(g_bar=bar[:1], sources=w.sources[:1])
        g3, G3, _ = m.gradient(g_bar=bar)
    for g, G in ((g1, G1), (g2, G2), (g3, G3)):
        assert np.array_equal(G0, G) and np.array_equal(g0, g)
