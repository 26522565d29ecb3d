"""The lattices of a batch in two orders, one after the other in one workspace:
128 x 512 and 256 x 256 sites are as many step tiles and half as many sampling
tiles, so a captured graph of one order must not be replayed for the other.
Samples and states equal those of a batch of its own, bit for bit."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_00530_amd as lib
    return lib


def _batch(L, sizes):
    ps = [L.make_params(nx, ny, L.LBM_MIPS, seed=300 + l, tau=2.0, sigma=8.0 / 70.0, C=6.25, rho_star=1.6, u_max=0.3)
          for l, (nx, ny) in enumerate(sizes)]
    b = L.Batch(ps)
    for l, p in enumerate(ps):
        lat = L.Lattice(p, init=L.make_init(mode=1, rho_mean=0.9, rho_spread=0.2, u_mag=0.1, pop_noise=1e-3))
        b.set_state(l, lat.state)
        lat.close()
    return b


# two lattice groups one after the other; one group (as two branches where the
# tuning takes them)
@pytest.mark.parametrize("n,tile_rows,steps", [(100, 16, 4), (20, 0, 40), (20, 16, 40)])
def test_two_orders(L, n, tile_rows, steps):
    sizes = [(128, 512)] * (n // 2) + [(256, 256)] * (n // 2)
    one, two = _batch(L, sizes), _batch(L, sizes)
    there, back = list(range(n)), list(range(n // 2, n)) + list(range(n // 2))
    if n == 100:
        assert L.lbm_sweep_groups(one.params, n) == 2
    for order in (there, back, there, back):
        a = one.run(steps, tile_rows=tile_rows, subset=order)
        b = two.run(steps, tile_rows=tile_rows, subset=there)
        for k, l in enumerate(order):
            assert a[k] == b[l], (order[0], l)
        for l in range(n):
            assert torch.equal(one.state(l), two.state(l)), (order[0], l)
