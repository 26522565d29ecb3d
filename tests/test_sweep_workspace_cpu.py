"""Workspace sizes of batched sweeps: part of a batch never needs more than the
batch (a program sizes one workspace and runs parts of the batch in it, as a
surrogate sweep does), and the size does not depend on the model.  Around the
sizes where the list of several-steps tiles appears, changes its geometry and
ends (2^20 sites)."""
import random

import pytest

KW = {0: dict(tau=1.5), 1: dict(tau=2.0, sigma=8.0 / 70.0, C=6.25, rho_star=1.6, u_max=0.3),
      2: dict(tau=1.0, sigma=4.0 / 70.0, A=0.125, B=0.3)}


def _need(L, sizes, model, q=7, samples=1):
    ps = (L.lbm_params * len(sizes))(*[
        L.make_params(nx, ny, model, lattice=L.LBM_D2Q9 if q == 9 else L.LBM_D2Q7, **KW[model]) for nx, ny in sizes])
    return L.lbm_sweep_workspace_bytes(ps, len(sizes), samples)


@pytest.mark.parametrize("q", [7, 9])
@pytest.mark.parametrize("side,most", [(128, 70), (64, 262), (32, 1030), (256, 20), (300, 14)])
def test_fewer_equal_lattices(side, most, q):
    import paper_1902_00530_amd as L
    for model in (1, 2):
        sizes = [_need(L, [(side, side)] * n, model, q) for n in range(1, most, 1 if most < 300 else 3)]
        assert all(a <= b for a, b in zip(sizes, sizes[1:]))


def test_parts_of_mixed_batches():
    import paper_1902_00530_amd as L
    rng = random.Random(7)
    for _ in range(60):
        sizes = [(rng.randint(2, 400), 2 * rng.randint(1, 200)) for _ in range(rng.randint(2, 60))]
        model = rng.choice([0, 1, 2])
        whole = _need(L, sizes, model)
        for _ in range(20):
            part = rng.sample(sizes, rng.randint(1, len(sizes)))
            assert _need(L, part, model) <= whole


def test_same_for_every_model():
    import paper_1902_00530_amd as L
    for sizes in ([(128, 128)] * 20, [(90, 30)] * 12, [(96, 34)] * 9, [(64, 64)] * 300, [(1024, 1024)] * 5):
        assert len({_need(L, sizes, m) for m in (0, 1, 2)}) == 1
