"""The fold of the padded gradient onto the input cells: very long x rows (a
padded and an input row together exceed the LDS of a block) and few nodes
across, and padding thinner than the stencil, whose outer input cells are
never updated; against the FP64 oracle's adjoint, and over two source groups
against one (bit for bit)."""
import numpy as np
import pytest

from oracle import forward as F
from workloads import configs

pytestmark = pytest.mark.gpu

# the bound of the small grids in test_gpu_adjoint.py: relative L2 of the field
L2_TOL = 1e-4


@pytest.fixture(scope="module")
def emm():
    from paper_2304_00233_amd import emm as E
    return E


def long_rows():
    w = configs.small_case(seed=70, shape=(10300, 6, 5), rd=1, nb=1, ne=1, nt=200, nsrc=2,
                           nu_axes=(False, True, True))
    x = w.x1[[3, 5150]] + 40.0                       # one source at the low end of the rows
    src = w.sources.copy()
    src[:, 0] = x
    rec = np.concatenate([np.repeat(x[:, None], 3, 0) + np.array([-110.0, 30.0, 180.0] * 2)[:, None],
                          w.receivers[:6, 1:]], 1)
    return w.with_(sources=src, receivers=rec, chan_mask=1)


def test_gradient_on_very_long_rows(emm):
    w = long_rows()
    print(f"[gpu] adjoint {w.name}", flush=True)
    one = w.with_(sources=w.sources[:1], src_comp=w.src_comp[:1], receivers=w.receivers[:3])
    s = np.float32(1.3)
    st = F.make_setup(one, 2.0 * np.sqrt(max(w.freqs)))
    G_obs, _ = F.forward(one.with_(rho11=w.rho11 * s, rho22=w.rho22 * s, rho33=w.rho33 * s), dt_override=st.dt)
    _, g_o, _ = F.misfit_gradient(one, G_obs, frozen=st)
    with emm.Model(one) as m:
        g, _, _ = m.gradient(g_obs=G_obs)
    l2 = np.linalg.norm(g - g_o) / np.linalg.norm(g_o)
    print(f"[adjoint] {w.name}: rel L2 {l2:.2e}", flush=True)
    assert l2 <= L2_TOL
    bar = np.ones((2, 6, 1, 2), complex)
    out = []
    for group in (-1, 1):
        with emm.Model(w, src_group=group) as m:
            out.append(m.gradient(g_bar=bar)[0])
    assert np.array_equal(out[0], out[1])


@pytest.mark.parametrize("rd,nb,ne", [(2, 0, 0), (2, 0, 1), (3, 1, 1), (1, 0, 0), (1, 0, 1), (4, 2, 1)])
def test_gradient_with_padding_thinner_than_the_stencil(emm, rd, nb, ne):
    w = configs.small_case(seed=71 + rd, shape=(21, 19, 18), rd=rd, nb=nb, ne=ne, nt=200, nsrc=2).with_(chan_mask=1)
    print(f"[gpu] adjoint, thin padding {w.name} nb{nb} ne{ne}", flush=True)
    s = np.float32(1.3)
    st = F.make_setup(w, 2.0 * np.sqrt(max(w.freqs)))
    G_obs, _ = F.forward(w.with_(rho11=w.rho11 * s, rho22=w.rho22 * s, rho33=w.rho33 * s), dt_override=st.dt)
    _, g_o, _ = F.misfit_gradient(w, G_obs, frozen=st)
    out = []
    for group in (-1, 1):
        with emm.Model(w, src_order=0, src_group=group) as m:
            out.append(m.gradient(g_obs=G_obs)[0])
    l2 = np.linalg.norm(out[0] - g_o) / np.linalg.norm(g_o)
    print(f"[adjoint] {w.name}: rel L2 {l2:.2e}", flush=True)
    assert l2 <= L2_TOL and np.array_equal(out[0], out[1])
    off = np.ones(g_o.shape, bool)                   # input cells off the update set
    m = rd - nb - ne
    off[:, m:-m, m:-m, m:-m] = False
    assert not np.any(out[0][off]) if m > 0 else True
