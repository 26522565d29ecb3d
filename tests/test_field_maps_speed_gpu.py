"""Two calls where a form of a kernel was taken beyond the sizes it is faster at.
Coarse fields in cells of one or two sites, which take a lane each: not slower than in
larger cells of the same sites, and right at the edges of a block.  Sums of many
sampling tiles: a lattice of 1024 tiles, four rows a lane once, takes the time of
one of 1032, sixteen.  Best of several timings of captured graphs."""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_00530_amd as lib
    return lib


def _lattice(L, nx, ny, storage=0, q=7):
    p = L.make_params(nx, ny, L.LBM_CIL, tau=1.0, sigma=4.0 / 70.0, A=0.125, B=0.3, seed=9, storage=storage,
                      rho_ref=0.9 if storage else 0.0, lattice=L.LBM_D2Q9 if q == 9 else L.LBM_D2Q7)
    return L.Lattice(p, init=L.make_init(mode=1, rho_mean=0.9, rho_spread=0.2, u_mag=0.1, pop_noise=1e-3))


def _us(stream, call):
    stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        for _ in range(4):
            call()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    best = float("inf")
    for _ in range(16):
        e0.record(stream)
        g.replay()
        e1.record(stream)
        e1.synchronize()
        best = min(best, e0.elapsed_time(e1) * 250.0)
    return best


@pytest.mark.parametrize("nx,ny,c,larger", [(4096, 4096, 1, 2), (16, 30000, 1, 4), (16, 30000, 2, 4),
                                            (64, 8192, 2, 4)])
def test_small_cells(L, nx, ny, c, larger):
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        lat = _lattice(L, nx, ny)
        out = torch.empty((3, ny, nx), device="cuda")
        us = [_us(s, lambda: L.lbm_coarsen(lat.params, lat.state.data_ptr(), k, out.data_ptr(), s.cuda_stream))
              for k in (c, larger)]
        lat.close()
    # at c = 1 a third more is written (4096^2: 672 MB against 520)
    assert us[0] <= (1.35 if c == 1 else 1.15) * us[1], us


@pytest.mark.parametrize("nx,ny,c", [(257, 34, 1), (2, 2, 1), (256, 4, 1), (514, 36, 2), (2, 60, 2), (62, 36, 2),
                                     (60, 64, 4), (4, 8, 4), (64, 8, 4), (68, 32, 4)])
def test_small_cell_values(L, nx, ny, c):
    lat = _lattice(L, nx, ny)
    out = torch.full((3, ny // c, nx // c), -1.0, device="cuda")
    L.lbm_coarsen(lat.params, lat.state.data_ptr(), c, out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    rho, ux, uy, _ = lat.fields()
    f = torch.stack([rho, rho * ux, rho * uy]).double().view(3, ny // c, c, nx // c, c)
    # float32 sums of c^2 terms in turn: c^2 roundings of 2^-24 of the sum at most, and
    # the two of u and rho u
    tol = (c * c + 4) * 2.0 ** -24 * f.abs().mean((2, 4)) + 1e-12
    assert ((out.double() - f.mean((2, 4))).abs() <= tol).all()
    if c == 1:
        assert torch.equal(out[0], rho)
    lat.close()


@pytest.mark.parametrize("q,storage", [(7, 0), (7, 1), (9, 0)])
def test_sums_of_many_tiles(L, q, storage):
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        us = []
        for ny in (2048, 2064):
            lat = _lattice(L, 2048, ny, storage, q)
            r = torch.empty((ny, 2048), device="cuda")
            us.append(_us(s, lambda: L.lbm_moments(lat.ctx, r.data_ptr(), None, None, want_obs=False)))
            lat.close()
    assert us[0] <= 1.06 * us[1], us
