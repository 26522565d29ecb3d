"""Fields, observables and coarse fields at the edges of their tiles (256 columns
x 16 rows, four rows a lane; coarse cells by the row), on states with a
different value at every site, against float64 sums of the float32 site
values."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_00530_amd as lib
    return lib


def _lattice(L, q, nx, ny, seed, storage=0):
    p = L.make_params(nx, ny, L.LBM_CIL, tau=1.0, sigma=4.0 / 70.0, A=0.125, B=0.3, seed=seed, storage=storage,
                      rho_ref=0.9 if storage else 0.0, lattice=L.LBM_D2Q9 if q == 9 else L.LBM_D2Q7)
    return L.Lattice(p, init=L.make_init(mode=1, rho_mean=0.9, rho_spread=0.2, u_mag=0.1, pop_noise=1e-3))


@pytest.mark.parametrize("q,storage", [(7, 0), (9, 0), (7, 1), (7, 3)])
@pytest.mark.parametrize("nx,ny", [(2, 2), (255, 16), (256, 14), (257, 18), (513, 34), (1300, 30)])
def test_observables_are_the_sums_of_the_fields(L, q, storage, nx, ny):
    lat = _lattice(L, q, nx, ny, 3, storage)
    lat.step(2)
    rho, ux, uy, obs = lat.fields()
    r, x, y = rho.double(), (rho.double() * ux.double()), (rho.double() * uy.double())
    eps = 2.0 ** -22  # u is one division, rho u one product away from j, float32 each
    scale = (x * x + y * y).sqrt().sum().item()
    n = r.sum().item()
    assert abs(obs["M"] - n) <= 1e-13 * n
    assert abs(obs["Jx"] - x.sum().item()) <= eps * scale and abs(obs["Jy"] - y.sum().item()) <= eps * scale
    assert abs(obs["mean_speed"] - scale / n) <= eps * scale / n
    assert abs(obs["drho"] - r.mean(0).std(unbiased=False).item()) <= 1e-12
    assert obs["nonfinite"] == 0 and lat.observables() == obs
    # a batch of this lattice samples the same sums
    if q == 7 or storage == 0:
        b = L.Batch([lat.params])
        b.set_state(0, lat.state)
        s = b.run(0)[0][0]
        for k in ("M", "Jx", "Jy", "phi", "mean_speed", "drho"):
            assert abs(s[k] - obs[k]) <= 1e-13 * max(abs(obs[k]), 1.0), k
    # a non-finite population is counted wherever it is
    lat.state.view(torch.uint8).reshape(-1)[-4:] = 0xFF
    assert lat.observables(check=False)["nonfinite"] >= 1


@pytest.mark.parametrize("nx,ny,c", [(64, 32, 1), (300, 6, 1), (512, 8, 2), (258, 12, 6), (264, 24, 12), (320, 64, 32),
                                     (1024, 512, 256), (640, 640, 320), (520, 40, 4)])
def test_coarse_fields(L, nx, ny, c):
    lats = [_lattice(L, 7, nx, ny, 10 + k) for k in range(3)]
    h, w = ny // c, nx // c
    out = torch.full((3, 4, h, w), -1.0, device="cuda")
    ptrs = torch.tensor([lat.state.data_ptr() for lat in lats], dtype=torch.int64, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    L.lbm_coarsen_many(lats[0].params, 3, ptrs.data_ptr(), c, out.data_ptr(), 4 * h * w, st)
    one = torch.empty((3, h, w), device="cuda")
    for k, lat in enumerate(lats):
        rho, ux, uy, _ = lat.fields()
        f = torch.stack([rho, rho * ux, rho * uy]).double()
        ref = f.view(3, h, c, w, c).mean((2, 4))
        # float32 sums of c^2 terms in turn: c^2 roundings of 2^-24 of the sum at
        # most, and the two of u and rho u
        tol = (c * c + 4) * 2.0 ** -24 * f.abs().view(3, h, c, w, c).mean((2, 4)) + 1e-12
        assert ((out[k, :3].double() - ref).abs() <= tol).all()
        assert (out[k, 3] == -1.0).all()
        L.lbm_coarsen(lat.params, lat.state.data_ptr(), c, one.data_ptr(), st)
        assert torch.equal(one, out[k, :3])


def test_results_to_the_host_from_threads_and_streams(L):
    """Samples from several threads, each on its own stream, more of them at once
    than the pinned slots hold in places (a batch of 700 samples): every call
    gets its own."""
    import threading
    lats = [_lattice(L, 7, 40 + 2 * k, 18, 40 + k) for k in range(4)]
    want = [lat.observables() for lat in lats]
    torch.cuda.synchronize()
    bad = []

    def work(k):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            p = lats[k].params
            lat = L.Lattice(p)
            lat.set_state(lats[k].state)
            b = L.Batch([p])
            for _ in range(20):
                if lat.observables() != want[k]:
                    bad.append(k)
                b.set_state(0, lats[k].state)
                b.step_index = 0
                out = b.run(700, sample_every=1)[0]
                if len(out) != 700 or [o["step"] for o in out] != list(range(1, 701)):
                    bad.append(-k)
            lat.close()

    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
    assert lats[0].params.nx == 40 and L.Batch([lats[0].params]).run(0, sample_every=1) == [[]]
