"""Batches of small lattices in the several-steps-per-launch form (tile_rows 0
lets the tuning take it): members equal single lattices stepped one step per
launch bit for bit, with samples, density ramps, captured graphs, direct
launches and chunks past 1024 steps, and a workspace that serves another model
or a subset of the lattices afterwards."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_00530_amd as lib
    return lib


KW = {"cil": dict(tau=1.0, sigma=4.0 / 70.0, A=0.125, B=0.3),
      "mips": dict(tau=2.0, sigma=8.0 / 70.0, C=6.25, rho_star=1.6, u_max=0.3),
      "passive": dict(tau=1.5, sigma=0.0)}
CODE = {"passive": 0, "mips": 1, "cil": 2}
SIZES = [(90, 30), (64, 64), (3, 4), (65, 18), (180, 60), (31, 8)]


def _setup(L, q, model, storage, sizes):
    ps = [L.make_params(nx, ny, CODE[model], seed=500 + l, storage=storage, rho_ref=0.9 if storage else 0.0,
                        lattice=L.LBM_D2Q9 if q == 9 else L.LBM_D2Q7, **KW[model])
          for l, (nx, ny) in enumerate(sizes)]
    b, lats = L.Batch(ps), []
    for l, p in enumerate(ps):
        lat = L.Lattice(p, init=L.make_init(mode=1, rho_mean=0.9, rho_spread=0.2, u_mag=0.1, pop_noise=1e-3))
        b.set_state(l, lat.state)
        lats.append(lat)
    return b, lats


def _bits(t):
    return t.view(torch.int32 if t.dtype == torch.float32 else torch.int16)


def _advance(lats, n):
    for lat in lats:
        for _ in range(n):
            lat.step(1)


def _check(b, lats):
    torch.cuda.synchronize()
    for l, lat in enumerate(lats):
        assert torch.equal(_bits(b.state(l)), _bits(lat.state)), l


@pytest.mark.parametrize("use_graph", [0, 1])
@pytest.mark.parametrize("q,model", [(7, "cil"), (7, "mips"), (7, "passive"), (9, "cil"), (9, "mips")])
def test_members_equal_single_steps(L, q, model, use_graph):
    b, lats = _setup(L, q, model, L.LBM_F32, SIZES)
    for n in (7, 16, 1, 2, 23):
        b.run(n, use_graph=use_graph)
        _advance(lats, n)
        _check(b, lats)


@pytest.mark.parametrize("storage", [1, 2, 3])
@pytest.mark.parametrize("model", ["cil", "mips"])
def test_16_bit(L, model, storage):
    b, lats = _setup(L, 7, model, storage, SIZES[:4])
    b.run(13)
    _advance(lats, 13)
    _check(b, lats)


def test_samples_ramp_and_chunks(L):
    b, lats = _setup(L, 7, "cil", L.LBM_F32, [(64, 30), (66, 30)])
    out = b.run(2200, sample_every=1100, drho=[0.01, -0.005])
    for k in range(2):
        _advance(lats, 1100)
        for l, lat in enumerate(lats):
            o = lat.observables()
            assert abs(out[l][k]["M"] - o["M"]) <= 1e-12 * o["M"] and abs(out[l][k]["drho"] - o["drho"]) <= 1e-12
            lat.add_density([0.01, -0.005][l])
    _check(b, lats)


def test_workspace_serves_another_model_and_a_subset(L):
    """The tile list kept in a workspace belongs to one geometry: another model
    on the same lattices, and a subset of them, get their own."""
    b, lats = _setup(L, 7, "cil", L.LBM_F32, [(90, 30)] * 12)
    b.run(8)
    _advance(lats, 8)
    _check(b, lats)
    other, olats = _setup(L, 7, "mips", L.LBM_F32, [(90, 30)] * 12)
    for l in range(12):
        b.params[l] = other.params[l]
        b.set_state(l, olats[l].state)
    b.step_index = 0
    b.run(9)
    _advance(olats, 9)
    _check(b, olats)
    b.step_index = 9
    b.run(6, subset=[1, 4, 5])
    _advance([olats[l] for l in (1, 4, 5)], 6)
    _check(b, olats)
