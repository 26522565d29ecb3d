"""Batches large enough for the two-step tiles, as the tuning runs them (tile_rows
0: possibly each lattice group as two branches of a graph, D2Q9 MIPS possibly
on 64 x 24 tiles): states and samples equal those of a named tile shape on one
branch bit for bit, over repeated replays with the caller's own work between
them, odd step counts and samples; and the shape reported for such a batch is
one that tile_rows names."""
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
      "mips": dict(tau=2.0, sigma=8.0 / 70.0, C=6.25, rho_star=1.6, u_max=0.3)}
SIDES = (128, 192, 256, 384, 512)
MIXED = [(SIDES[(7 * l + 1) % 5], SIDES[(3 * l + l // 5) % 5]) for l in range(30)]


def _batch(L, q, model, sizes):
    ps = [L.make_params(nx, ny, {"mips": 1, "cil": 2}[model], seed=70 + l,
                        lattice=L.LBM_D2Q9 if q == 9 else L.LBM_D2Q7, **KW[model])
          for l, (nx, ny) in enumerate(sizes)]
    return L.Batch(ps), ps


@pytest.mark.parametrize("q,model,sizes", [(7, "cil", MIXED), (7, "mips", MIXED), (9, "cil", MIXED[:9]),
                                           (9, "mips", MIXED), (7, "cil", [(1024, 1024)] * 5),
                                           (7, "cil", [(300, 210), (900, 602)]), (9, "mips", [(1000, 751)])])
def test_tuned_equals_named(L, q, model, sizes):
    tuned, ps = _batch(L, q, model, sizes)
    named, _ = _batch(L, q, model, sizes)
    for l, p in enumerate(ps):
        lat = L.Lattice(p, init=L.make_init(mode=1, rho_mean=0.9, rho_spread=0.2, u_mag=0.1, pop_noise=1e-3))
        tuned.set_state(l, lat.state)
        named.set_state(l, lat.state)
        lat.close()
    for n, every in ((6, 3), (5, 0), (6, 3), (6, 3), (7, 0)):
        a = tuned.run(n, sample_every=every)
        b = named.run(n, sample_every=every, tile_rows=16)
        assert a == b
        for l in range(len(sizes)):
            assert torch.equal(tuned.state(l), named.state(l)), (n, l)
    assert L.lbm_sweep_tile_rows(tuned.params, tuned.n) in (1, 2, 4, 8, 16)
    with pytest.raises(L.LbmError):
        tuned.run(2, tile_rows=24)
