"""Seeded random accepted forms (grids, orders, paddings down to none, edge
receivers, source counts, frequencies, accumulators, checkpoints, the
allocation-free entry) with default options, which run resident where they
can, against the half-step launches: equal bit for bit."""
import numpy as np
import pytest

from workloads import configs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def emm():
    from paper_2304_00233_amd import emm as m
    return m


def _draw(seed):
    g = np.random.default_rng(seed)
    rd = int(g.choice([1, 2, 2, 3, 4]))
    low = 2 * rd + 1
    shape = tuple(int(v) for v in np.maximum(low, np.exp(g.uniform(np.log(low), np.log(60), 3))))
    nsrc = int(g.choice([1, 1, 2, 3]))
    w = configs.small_case(seed=seed, shape=shape, rd=rd, nb=int(g.choice([0, 1, 3, 6, 10])),
                           ne=int(g.choice([0, 1, 3, 7])), nt=int(g.choice([1, 2, 17, 40])), nsrc=nsrc,
                           nrec=int(g.choice([1, 7, 40])), freqs=tuple(np.geomspace(0.3, 2.5, int(g.choice([1, 3, 70])))),
                           nu_axes=tuple(bool(v) for v in g.integers(0, 2, 3)), src_comp=g.integers(0, 3, nsrc))
    rec = w.receivers.copy()
    for a, ax in enumerate((w.x1, w.x2, w.x3)):          # some on the outermost cells
        q = g.random(len(rec))
        rec[q < 0.2, a] = ax[rd - 1] + 1e-3 * (ax[rd] - ax[rd - 1])
        rec[q > 0.8, a] = ax[-rd - 1] - 1e-3 * (ax[-rd - 1] - ax[-rd - 2])
    return w.with_(receivers=rec, chan_mask=int(g.choice([1, 7, 0x38, 0x3F])), dft_mode=int(g.integers(0, 2))), g


def _accepted(emm, w):
    with emm.Model(w, nt=1, src_order=0) as m:
        ok = np.ones(len(w.receivers), bool)
        for q, p in enumerate(w.receivers):
            try:
                m.forward(receivers=p[None])
            except emm.EmmError as e:
                assert e.status == -4
                ok[q] = False
    return w.with_(receivers=w.receivers[ok]) if ok.any() else None


def test_random_forms_equal_half_step_launches(emm):
    resident = 0
    for seed in range(150):
        w, g = _draw(seed)
        w = _accepted(emm, w)
        if w is None:
            continue
        print(f"[gpu] resident random {seed}: {w.name} nb{w.nb} ne{w.ne} nt{w.nt} src{len(w.sources)} "
              f"rec{len(w.receivers)} freq{len(w.freqs)} mask{w.chan_mask} dft{w.dft_mode}", flush=True)
        every = int(g.choice([0, 7, 16]))
        bar = g.normal(size=(len(w.sources), len(w.receivers), len(w.channels), len(w.freqs))) + 0j
        with emm.Model(w, src_order=0, src_group=-1) as m:
            ref = m.forward()
            grad, _, _ = m.gradient(g_bar=bar)
        with emm.Model(w, checkpoint_every=every) as m:
            assert np.array_equal(m.forward(), ref)
            resident += m.info()["resident"] > 0
            if every == 0:
                assert np.array_equal(m.forward(noalloc=True), ref)
            assert np.array_equal(m.gradient(g_bar=bar)[0], grad)
    assert resident >= 50
