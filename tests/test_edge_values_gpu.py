"""Values at the edge of the site body's correction: NaN and infinite
populations stay where they are (no rule of the negative correction hides
them, no finite site is touched), and a population of -0 counts as empty."""
import numpy as np
import pytest

import synth_inputs as SI

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

NX, NY = 70, 12
MODELS = {"passive": 0, "mips": 1, "cil": 2}


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_00530_amd as lib
    return lib


def _step(L, q, model, tau, f):
    p = L.make_params(NX, NY, MODELS[model], tau=tau, sigma=0.01, A=0.125, B=0.3, C=6.25, rho_star=1.6, u_max=0.3,
                      seed=91, lattice=L.LBM_D2Q9 if q == 9 else L.LBM_D2Q7)
    lat = L.Lattice(p)
    lat.set_state(torch.from_numpy(f.astype(np.float32)).cuda())
    lat.step(1)
    out = lat.state.cpu().numpy().copy()
    lat.close()
    return out


@pytest.mark.parametrize("tau", [1.0, 2.0])
@pytest.mark.parametrize("model", sorted(MODELS))
@pytest.mark.parametrize("q", [7, 9])
def test_nonfinite_populations_stay_local(L, q, model, tau):
    """A NaN and an infinity in the rest population of two sites (the noise
    drives corrections everywhere): after one step exactly those sites (MIPS:
    and the neighbours whose density gradient reads them) hold non-finite
    populations; every other site equals the clean run bit for bit."""
    f = SI.near_negative_populations(NX, NY, 5, q=q)
    clean = _step(L, q, model, tau, f)
    assert np.isfinite(clean).all()
    bad = f.copy()
    sites = [(3, 20), (8, 64)]
    bad[0, 3, 20] = np.nan
    bad[0, 8, 64] = np.inf
    got = _step(L, q, model, tau, bad)
    hit = ~np.isfinite(got).all(axis=0)
    for y, x in sites:
        assert hit[y, x]
    near = np.zeros_like(hit)
    for y, x in sites:
        near[y - 1:y + 2, x - 1:x + 2] = True
    if model != "mips":
        assert hit.sum() == 2
    assert not hit[~near].any()
    assert np.array_equal(got[:, ~hit], clean[:, ~hit])


@pytest.mark.parametrize("q", [7, 9])
def test_minus_zero_is_empty(L, q):
    """-0 in place of +0 changes nothing beyond the rescale's rounding (one
    step's bound, 1e-6 of the population scale), and results stay >= 0."""
    f = SI.near_negative_populations(NX, NY, 6, q=q)
    f[:, 4, :] = 0.0
    minus = f.copy()
    minus[:, 4, :] = -0.0
    a, b = _step(L, q, "cil", 1.0, f), _step(L, q, "cil", 1.0, minus)
    assert (a >= 0).all() and (b >= 0).all()
    assert np.abs(a - b).max() <= 1e-6 * np.abs(a).max()
