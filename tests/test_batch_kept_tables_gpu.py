"""One workspace with its tables kept (keep_tables), then another model on the
same lattice sizes in either order: the samples, the density ramp and the
states are those of single lattices.  The sizes are such that the models' lists
of several-steps tiles differ in length, so that a table placed behind that list
moves with the model."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_00530_amd as lib
    return lib


KW = {1: dict(tau=2.0, sigma=8.0 / 70.0, C=6.25, rho_star=1.6, u_max=0.3),
      2: dict(tau=1.0, sigma=4.0 / 70.0, A=0.125, B=0.3)}


def _lattices(L, model, q, sizes):
    ps = [L.make_params(nx, ny, model, seed=40 + l, lattice=L.LBM_D2Q9 if q == 9 else L.LBM_D2Q7, **KW[model])
          for l, (nx, ny) in enumerate(sizes)]
    return ps, [L.Lattice(p, init=L.make_init(mode=1, rho_mean=0.9, rho_spread=0.2, u_mag=0.1, pop_noise=1e-3))
                for p in ps]


def _sweep(L, ps, bufs, ws, steps, every, step0, keep, drho):
    """Samples of a sweep through the C interface, on the caller's workspace."""
    n = len(ps)
    arr = (L.lbm_params * n)(*ps)
    out = (L.lbm_obs * (n * (steps // every)))()
    opts = L.lbm_sweep_opts(steps, every, step0, 0, 1)
    opts.keep_tables = keep
    dr = (ctypes.c_double * n)(*drho)
    opts.drho = dr
    ptrs = (ctypes.c_void_p * (2 * n))(*[b.data_ptr() for pair in bufs for b in pair])
    L.lbm_sweep_batch(arr, n, opts, ptrs, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream, out)
    return [[out[l * (steps // every) + k].as_dict() for k in range(steps // every)] for l in range(n)]


@pytest.mark.parametrize("q,sizes", [(7, [(128, 128)] * 20), (7, [(96, 34)] * 9),
                                     (9, [(128, 127)] * 12)])
@pytest.mark.parametrize("order", [(1, 2, 1), (2, 1, 2)])
def test_model_swap(L, q, sizes, order):
    n = len(sizes)
    both = {m: _lattices(L, m, q, sizes) for m in (1, 2)}
    ws = torch.empty(1 << 20 | max(L.lbm_sweep_workspace_bytes((L.lbm_params * n)(*both[m][0]), n, 2) for m in (1, 2)),
                     dtype=torch.uint8, device="cuda")
    bufs = [[torch.empty((q, ny, nx), device="cuda") for _ in range(2)] for nx, ny in sizes]
    drho = [0.004 * (l % 5) - 0.006 for l in range(n)]
    done = {1: 0, 2: 0}
    for turn, m in enumerate(order):
        ps, lats = both[m]
        for pair, lat in zip(bufs, lats):
            pair[0].copy_(lat.state)
        got = _sweep(L, ps, bufs, ws, 8, 4, done[m], 1 if turn else 0, drho)
        for l, lat in enumerate(lats):
            for k in range(2):
                lat.step(4)
                o = lat.observables()
                for key in ("M", "phi", "mean_speed"):
                    assert abs(got[l][k][key] - o[key]) <= 1e-12 * max(1.0, abs(o[key])), (turn, l, k, key)
                assert abs(got[l][k]["drho"] - o["drho"]) <= 1e-12 and got[l][k]["step"] == o["step"]
                lat.add_density(drho[l])
            assert torch.equal(bufs[l][0], lat.state), (turn, l)
        done[m] += 8
