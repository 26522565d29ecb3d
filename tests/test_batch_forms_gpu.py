"""Every form that the tuning of a batch may choose, each set by hand, so that it
is reached whatever this machine's timings are: the tile shapes on one and on two
branches of a graph, the lattices resident in LDS, several steps per launch on
small tiles.  States and samples equal those of 64 x 16 tiles on one branch bit
for bit: even, odd and single steps, samples, density ramps, direct launches,
more than one lattice group."""
import ctypes

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# shapes 0 .. 4 of the local models, 3, 4 (two steps, 64 x 8 and 64 x 16), 6 (64 x 4)
# and, on D2Q9, 7 (64 x 24) of MIPS; resident, several steps
RESIDENT, MULTI = 8, 9


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1902_00530_amd as lib
    return lib


KW = {"cil": dict(tau=1.0, sigma=4.0 / 70.0, A=0.125, B=0.3),
      "mips": dict(tau=2.0, sigma=8.0 / 70.0, C=6.25, rho_star=1.6, u_max=0.3), "passive": dict(tau=1.5, sigma=0.0)}
SMALL = [(64, 48), (3, 4), (65, 18), (70, 44), (31, 8)]
MIXED = [(130, 70), (257, 94), (64, 200), (300, 48), (96, 96), (65, 34), (510, 50)]
WIDE = [(1000, 752), (700, 1002), (1024, 1024), (900, 602)] * 2


def _batch(L, q, model, sizes, storage=0):
    ps = [L.make_params(nx, ny, {"passive": 0, "mips": 1, "cil": 2}[model], seed=600 + l, storage=storage,
                        rho_ref=0.9 if storage else 0.0,
                        lattice=L.LBM_D2Q9 if q == 9 else L.LBM_D2Q7, **KW[model]) for l, (nx, ny) in enumerate(sizes)]
    both = L.Batch(ps), L.Batch(ps)
    for l, p in enumerate(ps):
        lat = L.Lattice(p, init=L.make_init(mode=1, rho_mean=0.9, rho_spread=0.2, u_mag=0.1, pop_noise=1e-3))
        for b in both:
            b.set_state(l, lat.state)
        lat.close()
    return both


def _set(L, b, form, split):
    assert L._lib.lbm_test_tune(b.params, b.n, form, split) == L.LBM_OK, L.lbm_last_error()


def _tuned(L, b):
    form, split = ctypes.c_int32(-1), ctypes.c_int32(-1)
    assert L._lib.lbm_test_tuned(b.params, b.n, ctypes.byref(form), ctypes.byref(split)) >= 1
    return form.value, split.value


def _forms(q, model, sizes):
    shapes = {("cil", 7): [0, 1, 2, 3, 4], ("mips", 7): [6, 3, 4], ("mips", 9): [3, 4, 7]}[
        "mips" if model == "mips" else "cil", q if model == "mips" else 7]
    two = [k for k in shapes if k in (3, 4, 7)]
    out = [(k, 0) for k in shapes] + [(k, 1) for k in two]
    if max(x * y for x, y in sizes) <= 3072:
        out.append((RESIDENT, 0))
    if sum(x * y for x, y in sizes) <= 1 << 20:
        out.append((MULTI, 0))
    return out


@pytest.mark.parametrize("sizes", [SMALL, MIXED, WIDE], ids=["small", "mixed", "wide"])
@pytest.mark.parametrize("q,model", [(7, "cil"), (7, "mips"), (7, "passive"), (9, "cil"), (9, "mips")])
def test_each_form(L, q, model, sizes):
    if sizes is WIDE and model == "passive":
        pytest.skip("as the CIL case")
    got, ref = _batch(L, q, model, sizes)
    if sizes is WIDE:
        assert L.lbm_sweep_groups(got.params, got.n) > 1
    ramp = [0.002 * (l % 3) - 0.002 for l in range(len(sizes))]
    for form, split in _forms(q, model, sizes):
        for n, every, kw in ((24, 12, dict(drho=ramp)), (23, 0, {}), (1, 0, {}), (26, 0, {}), (26, 0, {}),
                             (7, 0, dict(use_graph=0))):
            _set(L, got, form, split)
            a = got.run(n, sample_every=every, **kw)
            assert _tuned(L, got) == (form, split)
            b = ref.run(n, sample_every=every, tile_rows=16, **kw)
            assert a == b, (form, split, n)
            for l in range(len(sizes)):
                assert torch.equal(got.state(l), ref.state(l)), (form, split, n, l)


@pytest.mark.parametrize("storage", [1, 2, 3])
@pytest.mark.parametrize("model", ["cil", "mips"])
def test_each_form_16_bit(L, model, storage):
    got, ref = _batch(L, 7, model, SMALL, storage)
    for form, split in _forms(7, model, SMALL):
        for n in (22, 9):
            _set(L, got, form, split)
            assert got.run(n) == ref.run(n, tile_rows=16), (form, split, n)
            for l in range(len(SMALL)):
                assert torch.equal(got.state(l).view(torch.int16), ref.state(l).view(torch.int16)), (form, split, n, l)


def test_two_orders_on_two_branches(L):
    """As tests/test_batch_orders_gpu.py, the branches set by hand."""
    n = 20
    sizes = [(128, 512)] * 10 + [(256, 256)] * 10
    one, two = _batch(L, 7, "mips", sizes)
    there, back = list(range(n)), list(range(10, n)) + list(range(10))
    for order in (there, back, there, back):
        _set(L, one, 4, 1)
        a = one.run(40, subset=order)
        b = two.run(40, subset=there, tile_rows=16)
        for k, l in enumerate(order):
            assert a[k] == b[l], (order[0], l)
        for l in range(n):
            assert torch.equal(one.state(l), two.state(l)), (order[0], l)


def test_direct_launches_first(L):
    """What a call without graphs has tuned, which times no branches, is not what
    graphs run by afterwards; a call without graphs after that takes no branches."""
    got, ref = _batch(L, 7, "cil", [(200, 130), (330, 94), (128, 100)])
    form, split = ctypes.c_int32(-1), ctypes.c_int32(-1)
    for use_graph, known in ((0, 1), (0, 1), (1, 2), (0, 2), (1, 2)):
        a = got.run(20, use_graph=use_graph)
        assert L._lib.lbm_test_tuned(got.params, got.n, ctypes.byref(form), ctypes.byref(split)) == known
        assert a == ref.run(20, tile_rows=16)
        for l in range(3):
            assert torch.equal(got.state(l), ref.state(l)), (use_graph, l)


def test_first_call(L):
    """A batch's first call times the forms, each a few times at most: two 4096 x 4096
    lattices, where that is nearly all GPU time, within 20 calls' time (36 with six
    replays of every form and its branches)."""
    import time
    ps = [L.make_params(4096, 4096, L.LBM_CIL, seed=l, **KW["cil"]) for l in range(2)]
    b = L.Batch(ps)
    for l in range(2):
        b.buffers[2 * l].fill_(0.1)
    took = []
    for _ in range(6):
        torch.cuda.synchronize()
        t = time.perf_counter()
        b.run(20)
        took.append(time.perf_counter() - t)
    assert took[0] <= 20 * min(took[1:]), took


def test_refused_forms(L):
    b, _ = _batch(L, 7, "cil", WIDE[:2])
    for form, split in ((RESIDENT, 0), (MULTI, 0), (5, 0), (6, 0), (7, 0), (0, 1), (10, 0), (-1, 0), (3, 2)):
        assert L._lib.lbm_test_tune(b.params, b.n, form, split) == L.LBM_EINVAL
