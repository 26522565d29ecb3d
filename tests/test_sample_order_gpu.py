"""A lattice's samples do not depend on its batch: the FP64 sums run in one order,
whether the batch's tiles are few (four rows a lane) or many (sixteen), and
lbm_moments' sums in the same one.  Bit for bit, at the edges of the sampling
tiles, and lattices of more columns than the closing launch has lanes."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_00530_amd as lib
    return lib


OWN = [(300, 210), (256, 16), (3, 4), (257, 34), (1025, 18), (1024, 66), (2100, 30), (513, 400)]
MANY = [(130, 4000)] * 8  # 250 tiles each: more than 1024 in a lattice group


@pytest.mark.parametrize("q,model,storage", [(7, "cil", 0), (7, "mips", 0), (9, "cil", 0), (7, "cil", 1)])
def test_samples_alone_and_in_company(L, q, model, storage):
    kw = dict(tau=1.0, sigma=4.0 / 70.0, A=0.125, B=0.3) if model == "cil" else dict(
        tau=2.0, sigma=8.0 / 70.0, C=6.25, rho_star=1.6, u_max=0.3)
    ps = [L.make_params(nx, ny - (1 if q == 9 and ny == 34 else 0), L.LBM_CIL if model == "cil" else L.LBM_MIPS,
                        seed=80 + l, storage=storage, rho_ref=0.9 if storage else 0.0,
                        lattice=L.LBM_D2Q9 if q == 9 else L.LBM_D2Q7, **kw) for l, (nx, ny) in enumerate(OWN + MANY)]
    lats = [L.Lattice(p, init=L.make_init(mode=1, rho_mean=0.9, rho_spread=0.2, u_mag=0.1, pop_noise=1e-3)) for p in ps]
    n = len(OWN)

    def samples(which):
        b = L.Batch([ps[l] for l in which])
        for k, l in enumerate(which):
            b.set_state(k, lats[l].state)
        return dict(zip(which, b.run(2, sample_every=1)))

    together = samples(list(range(len(ps))))
    few = samples(list(range(n)))
    turned = samples(list(range(n))[::-1])
    assert few == turned == {l: together[l] for l in range(n)}
    for l in (0, 4, 7):
        assert samples([l])[l] == few[l]
    for l in range(len(ps)):
        for k in range(2):
            lats[l].step(1)
            assert lats[l].observables() == together[l][k], (l, k)
