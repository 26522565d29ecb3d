"""Performance cases: the calls a program makes of this library, over the sizes
it makes them at.

    lattice   Lattice.step(n): one lattice of the method
    fields    Lattice.fields(): rho, u and the FP64 observables of a state
    batch     Batch.run(): many lattices together, with samples and density ramps
    judge     FieldSampler.judge_from(): lift, k steps, coarsen (the surrogate's data)
    train     Surrogate.train_step(): one Adam step on a mini-batch
    predict   Surrogate.predict(): one network evaluation

prepare() makes the inputs from a seed and the objects a program keeps, run() is
one call, exact() the same results in float64 from plain torch.
"""
import math

import torch
import torch.nn.functional as F

import paper_1902_00530_amd as L
from paper_1902_00530_amd import surrogate as S

STORAGES = {"f32": L.LBM_F32, "bf16": L.LBM_BF16_DEV, "f16": L.LBM_F16_DEV, "bf16r32": L.LBM_BF16_DEV_R32}
MODELS = {"mips": L.LBM_MIPS, "cil": L.LBM_CIL}
# the density scale of the repository's workloads (4 for CIL, 8 for MIPS) of
# the paper's constants; "paper" takes them as printed
CIL = dict(tau=1.0, sigma=4.0 / 70.0, A=0.125, B=0.3)
MIPS = dict(tau=2.0, sigma=8.0 / 70.0, C=6.25, rho_star=1.6, u_max=0.3)
MIPS_PAPER = dict(tau=2.0, sigma=1.0 / 70.0, C=50.0, rho_star=0.2, u_max=0.3)
CIL_PAPER = dict(tau=1.0, sigma=1.0 / 70.0, A=2.0, B=0.3)
SIDES = (128, 192, 256, 384, 512)  # the sides of a phase sweep's lattices


def listed():
    return [
        # the paper's box: a launch-bound lattice, stepped in long runs
        dict(name="lattice_mips_64", kind="lattice", q=7, model="mips", storage="f32", nx=64, ny=64, steps=100),
        # the precision run: a lattice far larger than the caches
        dict(name="lattice_cil_4096", kind="lattice", q=7, model="cil", storage="f32", nx=4096, ny=4096, steps=20),
        # the same in 16-bit storage
        dict(name="lattice_cil_4096_bf16", kind="lattice", q=7, model="cil", storage="bf16", nx=4096, ny=4096,
             steps=20),
        # the square lattice at an ordinary, ragged size with an odd row count
        dict(name="lattice_q9_mips_1000x751", kind="lattice", q=9, model="mips", storage="f32", nx=1000, ny=751,
             steps=24),
        # fields and observables of an ordinary lattice
        dict(name="fields_1024", kind="fields", q=7, model="cil", storage="f32", nx=1024, ny=1024, steps=0),
        # five mean densities at 1024 x 1024, one sample at the end of 20 steps
        dict(name="batch_cil_5x1024", kind="batch", q=7, model="cil", storage="f32", n=5, nx=1024, ny=1024, steps=20,
             sample_every=0, ramp=False),
        # a phase sweep over lattices of mixed sizes
        dict(name="batch_phase_sweep_48", kind="batch", q=7, model="cil", storage="f32", n=48, nx=0, ny=0, steps=100,
             sample_every=50, ramp=False),
        # the paper's MIPS noise ramp: twelve 90 x 30 lattices, long sample periods
        dict(name="protocol_mips_12x90x30", kind="batch", q=7, model="mips", storage="f32", n=12, nx=90, ny=30,
             steps=500, sample_every=500, ramp=False),
        # the paper's hysteresis experiment: fifty 180 x 60 lattices, the density up and down
        dict(name="protocol_cil_50x180x60", kind="batch", q=7, model="cil", storage="f32", n=50, nx=180, ny=60,
             steps=1000, sample_every=500, ramp=True),
        # one round of the surrogate's training pairs (and a sweep's check)
        dict(name="judge_64x256", kind="judge", n=64, side=256, coarse=8, k=50),
        # one optimiser step of the surrogate's training
        dict(name="train_64x32x32", kind="train", n=64, h=32, w=32),
        # one network jump of a surrogate sweep
        dict(name="predict_64x32x32", kind="predict", n=64, h=32, w=32),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["lattice", "lattice", "fields", "batch", "batch", "judge", "train", "predict"])
    if kind in ("lattice", "fields"):
        q = rng.choice([7, 7, 9])
        model = rng.choice(["mips", "cil"])
        storage = rng.choice(["f32", "f32", "bf16", "f16"] + (["bf16r32"] if q == 7 else []))
        nx, ny = _log_int(rng, 48, 4000), _log_int(rng, 32, 4000)
        if q == 7:
            ny += ny & 1
        steps = 0 if kind == "fields" else rng.randint(1, 100 if nx * ny < 1 << 20 else 20)
        return dict(kind=kind, q=q, model=model, storage=storage, nx=nx, ny=ny, steps=steps)
    if kind == "batch":
        if rng.random() < 0.4:  # a protocol's lattices: small, many steps, sampled, ramped
            model = rng.choice(["mips", "cil"])
            nx, ny = _log_int(rng, 60, 200), 2 * _log_int(rng, 15, 40)
            every = rng.randint(50, 500)
            return dict(kind="batch", q=7, model=model, storage="f32", n=rng.randint(4, 60), nx=nx, ny=ny,
                        steps=2 * every, sample_every=every, ramp=rng.random() < 0.5)
        q = rng.choice([7, 7, 9])
        storage = rng.choice(["f32", "f32", "bf16", "f16", "bf16r32"]) if q == 7 else "f32"
        mixed = rng.random() < 0.5
        nx, ny = (0, 0) if mixed else (_log_int(rng, 128, 1400), 2 * _log_int(rng, 64, 600))
        return dict(kind="batch", q=q, model=rng.choice(["mips", "cil", "cil"]), storage=storage,
                    n=rng.randint(8, 30 if storage == "bf16r32" else 56) if mixed else rng.randint(1, 12), nx=nx, ny=ny, steps=rng.randint(4, 60),
                    sample_every=0, ramp=False)
    if kind == "judge":
        coarse = rng.choice([8, 16, 32])
        return dict(kind="judge", n=rng.randint(4, 64), side=coarse * rng.randint(4, 256 // coarse), coarse=coarse,
                    k=rng.randint(10, 50))
    return dict(kind=kind, n=rng.randint(3, 64), h=rng.randint(8, 40), w=rng.randint(8, 40))


# ------------------------------------------------------------------ inputs

def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _rng(seed):
    # drawn on the host, so that every machine draws the same
    return torch.Generator().manual_seed(int(seed))


def _uniform(g, shape, lo=0.0, hi=1.0):
    return (torch.rand(shape, generator=g) * (hi - lo) + lo).to(_device()).double()


E7 = [(0.0, 0.0)] + [(math.cos(k * math.pi / 3.0), math.sin(k * math.pi / 3.0)) for k in range(6)]
E9 = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]
W7 = [0.5] + [1.0 / 12.0] * 6
W9 = [4.0 / 9.0] + [1.0 / 9.0] * 4 + [1.0 / 36.0] * 4


def _steady(q, rho, ux, uy):
    """xi(rho, u) in float64, [q, ...]."""
    c = 4.0 if q == 7 else 3.0  # 1 / c_s^2
    out = []
    for (ex, ey), w in zip(E7 if q == 7 else E9, W7 if q == 7 else W9):
        eu = ex * ux + ey * uy
        out.append(w * rho * (1.0 + c * eu + 0.5 * c * c * eu * eu - 0.5 * c * (ux * ux + uy * uy)))
    return torch.stack(out)


def _lattices(case, seed):
    """Per lattice (constants, noise seed, nx, ny, mean density) and the float32 start."""
    n = case.get("n", 1)
    g = _rng(seed * 1000003 + 17)
    out = []
    for l in range(n):
        nx, ny = case["nx"], case["ny"]
        if nx == 0:  # mixed sides, the same for every seed (a program's batch keeps its shapes)
            nx, ny = SIDES[(7 * l + 1) % 5], SIDES[(3 * l + l // 5) % 5]
        small = case["kind"] == "batch" and nx * ny <= 16000
        frac = (l + 0.5) / n
        if case["model"] == "cil":
            k = dict(CIL_PAPER if small else CIL)
            rho_mean = (0.09 + 0.25 * frac) if small else (0.74 if n == 1 else 0.5 + frac)
            spread, mag = 0.1, None
        else:
            k = dict(MIPS_PAPER if small else MIPS)
            rho_mean = (0.06 + 0.12 * frac) if small else 1.0
            spread, mag = (0.1, 0.01) if small else (0.0, 0.1)
        rho = rho_mean * (1.0 + spread * _uniform(g, (ny, nx), -1.0, 1.0))
        if case["model"] == "cil":
            mag = (k["B"] - k["A"] * rho * rho).clamp_min(0.0)
        if case["model"] == "cil" and not small:  # an ordered state, its direction about +x
            th = 0.05 * torch.randn((ny, nx), generator=g).to(_device()).double()
        else:
            th = _uniform(g, (ny, nx), 0.0, 2.0 * math.pi)
        f = _steady(case["q"], rho, mag * torch.cos(th), mag * torch.sin(th))
        if case["model"] == "mips" and not small:
            f = f + _uniform(g, f.shape, -1e-3, 1e-3)
        out.append((k, int(torch.randint(1 << 40, (1,), generator=g)), nx, ny, rho_mean, f.float()))
    return out


def _params(case, k, seed, nx, ny, rho_mean):
    return L.make_params(nx, ny, MODELS[case["model"]], seed=seed, storage=STORAGES[case["storage"]],
                         rho_ref=0.0 if case["storage"] == "f32" else rho_mean,
                         lattice=L.LBM_D2Q9 if case["q"] == 9 else L.LBM_D2Q7, **k)


def _references(case, rho_mean):
    """The values r_i the deviation storages subtract, [q] floats."""
    dt = {"f32": None, "bf16": torch.bfloat16, "f16": torch.float16, "bf16r32": torch.bfloat16}[case["storage"]]
    if dt is None:
        return [0.0] * case["q"]
    r = [float(torch.tensor(w * rho_mean, dtype=torch.float32).to(dt)) for w in (W7 if case["q"] == 7 else W9)]
    if case["storage"] == "bf16r32":
        r[0] = 0.0
    return r


def _stored(case, f, rho_mean):
    """The buffer a program holds for float32 populations f."""
    if case["storage"] == "f32":
        return f
    r = torch.tensor(_references(case, rho_mean), device=f.device).view(-1, 1, 1)
    if case["storage"] == "bf16r32":
        rest = f[0].contiguous().view(torch.int16).reshape(2, f.shape[1], f.shape[2])
        return torch.cat([rest, (f[1:] - r[1:]).to(torch.bfloat16).view(torch.int16)])
    return (f - r).to(torch.bfloat16 if case["storage"] == "bf16" else torch.float16)


def _as_numbers(case, state):
    """A state as floating tensors (bf16r32: its float32 plane and its bf16 planes)."""
    if case["storage"] != "bf16r32":
        return state
    ny, nx = state.shape[1:]
    return [state[:2].reshape(-1).view(torch.float32).reshape(ny, nx), state[2:].view(torch.bfloat16)]


def _judge_inputs(case, seed):
    """Coarse fields (n, 4, h, w) with the lattices' constants and noise seeds."""
    g = _rng(seed * 1000003 + 29)
    n, h = case["n"], case["side"] // case["coarse"]
    act = [0.3 * ((l % 8) + 1) / 8.0 for l in range(n)]
    mean = torch.tensor([0.3 + 1.5 * ((l * 5) % n) / max(1, n - 1) for l in range(n)]).view(n, 1, 1).to(_device())
    rho = mean * _uniform(g, (n, h, h), 0.97, 1.03)
    b = torch.tensor(act, device=rho.device).view(n, 1, 1)
    mag = (b - CIL["A"] * rho * rho).clamp_min(0.0)
    th = 2.0 * math.pi * torch.rand((n, 1, 1), generator=g).to(_device()) + _uniform(g, (n, h, h), -0.3, 0.3)
    x = torch.stack([rho, rho * mag * torch.cos(th), rho * mag * torch.sin(th), b.expand(n, h, h)], 1)
    seeds = [int(torch.randint(1 << 40, (1,), generator=g)) for _ in range(n)]
    return x.float().contiguous(), act, seeds


POOL = 8  # mini-batches in the pool of training pairs
LR = 1e-3


def _network_inputs(case, seed):
    """Fields, targets, sample order and a network in mid-training: weights,
    biases and their Adam moments."""
    g = _rng(seed * 1000003 + 31)
    n, h, w = case["n"], case["h"], case["w"]
    total = n * POOL if case["kind"] == "train" else n
    c = torch.randn((total, 4, 1, 1), generator=g)
    x = 0.1 * torch.randn((total, 4, h, w), generator=g) + torch.cat([1.0 + 0.2 * c[:, :1], 0.1 * c[:, 1:3], 0.15 + 0.05 * c[:, 3:]], 1)
    x[:, 3] = x[:, 3, :1, :1]
    t = x + 0.05 * torch.randn((total, 4, h, w), generator=g)
    shapes = [(32, 4, 3, 3), (32,), (32, 32, 3, 3), (32,), (3, 32, 3, 3), (3,)]
    theta, m, v = [], [], []
    for s in shapes:
        lim = math.sqrt(6.0 / (9 * s[1])) if len(s) == 4 else 0.05
        theta.append((torch.rand(s, generator=g) * 2.0 - 1.0) * lim)
        m.append(1e-4 * torch.randn(s, generator=g))
        v.append(1e-6 * (0.5 + torch.rand(s, generator=g)))
    perm = torch.randperm(total, generator=g).to(torch.int32)
    return x, t, perm, theta, m, v


def _block_views(sur):
    """theta, m, v and the bf16 weights as views of the surrogate's parameter block."""
    view = L.lbm_surrogate_view_of(sur.handle)
    base = sur.params.data_ptr()

    def at(ptr, count, dt):
        o = ptr - base
        return sur.params[o:o + count * (2 if dt == torch.bfloat16 else 4)].view(dt)

    f32 = [[at(p[k], view.count[k], torch.float32) for k in range(6)] for p in (view.theta, view.m, view.v)]
    return f32, [at(view.w_bf16[k], view.count[2 * k], torch.bfloat16) for k in range(3)]


# ------------------------------------------------------- what a program does

def prepare(case, seed):
    kind = case["kind"]
    if kind in ("lattice", "fields"):
        (k, noise, nx, ny, rho_mean, f), = _lattices(case, seed)
        lat = L.Lattice(_params(case, k, noise, nx, ny, rho_mean))
        lat.set_state(_stored(case, f, rho_mean))
        return dict(case=case, lat=lat)
    if kind == "batch":
        lats = _lattices(case, seed)
        b = L.Batch([_params(case, k, noise, nx, ny, r) for k, noise, nx, ny, r, _ in lats])
        for l, (_, _, _, _, r, f) in enumerate(lats):
            b.set_state(l, _stored(case, f, r))
        return dict(case=case, batch=b)
    if kind == "judge":
        x, act, seeds = _judge_inputs(case, seed)
        k = dict(CIL)
        ps = [L.make_params(case["side"], case["side"], L.LBM_CIL, seed=s, **dict(k, B=a)) for s, a in zip(seeds, act)]
        return dict(case=case, sampler=S.FieldSampler(ps, case["coarse"], case["k"]), x=x)
    x, t, perm, theta, m, v = _network_inputs(case, seed)
    sur = S.Surrogate(case["h"], case["w"], 8, 50, case["n"])
    f32, wb = _block_views(sur)
    for dst, src in zip(f32, (theta, m, v)):
        for d, s in zip(dst, src):
            d.copy_(s.reshape(-1))
    for j in range(3):
        wb[j].copy_(theta[2 * j].reshape(-1))
    x, t, perm = x.cuda(), t.cuda(), perm.cuda()
    sur.fit_normalisation(x)
    return dict(case=case, sur=sur, x=x, t=t, perm=perm, f32=f32, at=0)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "lattice":
        lat = state["lat"]
        lat.step(case["steps"])
        return _as_numbers(case, lat.state)
    if kind == "fields":
        rho, ux, uy, obs = state["lat"].fields()
        return [rho, ux, uy, obs]
    if kind == "batch":
        b = state["batch"]
        if case["ramp"]:  # a density step up after each sample, then back down
            obs = b.run(case["steps"], sample_every=case["sample_every"], drho=0.0025)
            back = b.run(case["steps"], sample_every=case["sample_every"], drho=-0.0025)
            obs = [u + d for u, d in zip(obs, back)]
        else:
            obs = b.run(case["steps"], sample_every=case["sample_every"])
        table = torch.tensor([[list(o.values()) for o in lat] for lat in obs], dtype=torch.float64)
        return [table] + [_as_numbers(case, b.state(l)) for l in range(b.n)]
    if kind == "judge":
        return state["sampler"].judge_from(state["x"], torch.cuda.current_stream().cuda_stream)
    if kind == "train":
        n, at = case["n"], state["at"]
        state["at"] = (at + n) % (n * POOL)
        loss = state["sur"].train_step(state["x"], state["t"], state["perm"][at:at + n], LR)
        return [loss, state["f32"]]
    return state["sur"].predict(state["x"])


def work(case):
    """The state read and written once (a longer run reads and writes it no
    more often than that in principle), and the arithmetic of every step: about
    100 flops per site on seven populations, 130 on nine (the noise's integer
    products not counted)."""
    kind = case["kind"]
    if kind in ("lattice", "fields", "batch"):
        n = case.get("n", 1)
        if case["nx"] == 0:
            sites = sum(SIDES[(7 * l + 1) % 5] * SIDES[(3 * l + l // 5) % 5] for l in range(n))
        else:
            sites = n * case["nx"] * case["ny"]
        per = {"f32": 4 * case["q"], "bf16": 2 * case["q"], "f16": 2 * case["q"], "bf16r32": 16}[case["storage"]]
        if kind == "fields":
            return dict(bytes=sites * (per + 12), flops=sites * 20)
        return dict(bytes=2 * sites * per, flops=sites * case["steps"] * (2 if case.get("ramp") else 1) * (100 if case["q"] == 7 else 130))
    if kind == "judge":
        h = case["side"] // case["coarse"]
        return dict(bytes=case["n"] * h * h * 32, flops=case["n"] * case["side"] ** 2 * case["k"] * 100)
    px = case["n"] * case["h"] * case["w"]
    forward = 2 * px * 9 * (4 * 32 + 32 * 32 + 32 * 3)
    if kind == "predict":
        return dict(bytes=px * 32, flops=forward)
    # the weight gradients of three layers, the input gradients of two
    return dict(bytes=px * 28 + 6 * 4 * 11299, flops=2 * forward + 2 * px * 9 * (32 * 32 + 32 * 3))


# ---------------------------------------------------------------- float64

def _philox(site, step, seed):
    """Philox4x32-10 of counters (site, step, 0, 0) and per-lattice keys, four
    32-bit words in int64 tensors."""
    mask = 0xFFFFFFFF
    c = [site & mask, torch.zeros_like(site) + (step & mask), torch.zeros_like(site) + (step >> 32),
         torch.zeros_like(site)]
    k0, k1 = seed & mask, seed >> 32 & mask
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [(p1 >> 32 & mask) ^ c[1] ^ k0, p1 & mask, (p0 >> 32 & mask) ^ c[3] ^ k1, p0 & mask]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return c


def _stream(f, q):
    """Population i of a site from the site at minus e_i; f [q, n, ny, nx]."""
    g = [f[0]]
    if q == 9:
        return torch.stack([torch.roll(f[i], (E9[i][1], E9[i][0]), (-2, -1)) for i in range(9)])
    odd = (torch.arange(f.shape[-2], device=f.device) & 1).bool().view(-1, 1)
    up, dn = [torch.roll(f[i], 1, -2) for i in (2, 3)], [torch.roll(f[i], -1, -2) for i in (5, 6)]
    g.append(torch.roll(f[1], 1, -1))
    g.append(torch.where(odd, up[0], torch.roll(up[0], 1, -1)))
    g.append(torch.where(odd, torch.roll(up[1], -1, -1), up[1]))
    g.append(torch.roll(f[4], -1, -1))
    g.append(torch.where(odd, torch.roll(dn[0], -1, -1), dn[0]))
    g.append(torch.where(odd, dn[1], torch.roll(dn[1], 1, -1)))
    return torch.stack(g)


def _fields(f, q):
    e = E7 if q == 7 else E9
    return f.sum(0), sum(f[i] * e[i][0] for i in range(1, q)), sum(f[i] * e[i][1] for i in range(1, q))


def _gradient(rho, q):
    """Isotropic stencil (1 / c_s^2) sum_i w_i e_i rho(r + e_i)."""
    if q == 9:
        nb = [torch.roll(rho, (-E9[i][1], -E9[i][0]), (-2, -1)) for i in range(9)]
        return (sum(3.0 * W9[i] * E9[i][k] * nb[i] for i in range(1, 9)) for k in (0, 1))
    odd = (torch.arange(rho.shape[-2], device=rho.device) & 1).bool().view(-1, 1)
    r = lambda v, s: torch.roll(v, s, -1)  # noqa: E731
    hi, lo = torch.roll(rho, -1, -2), torch.roll(rho, 1, -2)
    nb = [rho, r(rho, -1), torch.where(odd, r(hi, -1), hi), torch.where(odd, hi, r(hi, 1)), r(rho, 1),
          torch.where(odd, lo, r(lo, 1)), torch.where(odd, r(lo, -1), lo)]
    return (sum(4.0 * W7[i] * E7[i][k] * nb[i] for i in range(1, 7)) for k in (0, 1))


def _steps(f, q, model, c, seeds, first, count):
    """`count` steps of the method on f [q, n, ny, nx] float64; c: its constants
    (numbers or [n, 1, 1] tensors), seeds [n, 1, 1] int64."""
    ny, nx = f.shape[-2:]
    site = torch.arange(nx * ny, device=f.device, dtype=torch.int64).view(1, ny, nx)
    pairs = [(1, 4), (2, 5), (3, 6)] if q == 7 else [(1, 3), (2, 4), (5, 7), (6, 8)]
    for t in range(first, first + count):
        f = _stream(f, q)
        rho, jx, jy = _fields(f, q)
        if model == "cil":
            j = torch.sqrt(jx * jx + jy * jy)
            s = torch.where(j > 0, (c["B"] - c["A"] * rho * rho).clamp_min(0.0) / j.clamp_min(1e-300), 0.0)
            ux, uy = s * jx, s * jy
        else:
            gx, gy = _gradient(rho, q)
            s = c["C"] * (1.0 - rho / c["rho_star"]).clamp_min(0.0)
            ux, uy = s * gx, s * gy
            u = torch.sqrt(ux * ux + uy * uy)
            s = torch.where(u > c["u_max"], c["u_max"] / u.clamp_min(1e-300), 1.0)
            ux, uy = s * ux, s * uy
        f = f + (_steady(q, rho, ux, uy) - f) / c["tau"]
        w = _philox(site, t, seeds)
        if q == 7:
            h = torch.stack([w[i // 2] >> 16 * (i % 2) & 0xFFFF for i in range(7)]).double()
            h = c["sigma"] * (2.0 * (h + 0.5) / 65536.0 - 1.0)
        else:
            h = []
            for i in range(9):
                k, o = divmod(14 * i, 32)
                v = w[k] >> o
                if o > 18:
                    v = v | w[k + 1] << 32 - o
                h.append(v & 0x3FFF)
            h = c["sigma"] * (2.0 * (torch.stack(h).double() + 0.5) / 16384.0 - 1.0)
        f = f + (h - h.mean(0))
        del h, w
        # negative correction
        fired = f[0] < 0
        f[0].clamp_min_(0.0)
        for a, b in pairs:
            bad = (f[a] < 0) | (f[b] < 0)
            d = f[a] - f[b]
            f[a] = torch.where(bad, d.clamp_min(0.0), f[a])
            f[b] = torch.where(bad, (-d).clamp_min(0.0), f[b])
            fired |= bad
        s = f.sum(0)
        f *= torch.where(fired, torch.where(s > 0, rho / s.clamp_min(1e-300), 0.0), 1.0)
    return f


def _observables(f, q, c, step):
    """One row per lattice: step, M, Jx, Jy, phi, mean speed, zeta, banding, nonfinite."""
    rho, jx, jy = _fields(_stream(f, q), q)
    m, x, y = (v.sum((-2, -1)) for v in (rho, jx, jy))
    speed = torch.sqrt(jx * jx + jy * jy).sum((-2, -1)) / m
    col = rho.mean(-2)
    return torch.stack([torch.full_like(m, step), m, x, y, torch.sqrt(x * x + y * y) / m, speed, c.get("B", 0.0) - speed,
                        col.std(-1, unbiased=False), torch.zeros_like(m)], -1)


def _start64(case, f, rho_mean):
    """Float64 populations of the stored start and the references r_i."""
    s = _stored(case, f, rho_mean)
    r = torch.tensor(_references(case, rho_mean), dtype=torch.float64, device=f.device).view(-1, 1, 1)
    if case["storage"] == "bf16r32":
        a, b = _as_numbers(case, s)
        return torch.cat([a.double()[None], b.double() + r[1:]]), r
    return s.double() + r, r


def _conv64(x, w, b):
    return F.conv2d(F.pad(x, (1, 1, 1, 1), mode="circular"), w, b)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("lattice", "fields"):
        (k, noise, nx, ny, rho_mean, f), = _lattices(case, seed)
        f, r = _start64(case, f, rho_mean)
        seeds = torch.tensor([noise], device=f.device).view(1, 1, 1)
        f = _steps(f[:, None], case["q"], case["model"], k, seeds, 0, case["steps"])
        if kind == "fields":
            rho, jx, jy = _fields(_stream(f, case["q"])[:, 0], case["q"])
            o = _observables(f, case["q"], k, 0)[0].tolist()
            keys = ("step", "M", "Jx", "Jy", "phi", "mean_speed", "zeta", "drho", "nonfinite")
            obs = dict(zip(keys, o))
            obs["step"], obs["nonfinite"] = int(obs["step"]), int(obs["nonfinite"])
            return [rho, torch.where(rho != 0, jx / rho, 0.0), torch.where(rho != 0, jy / rho, 0.0), obs]
        d = f[:, 0] - r
        return [d[0], d[1:]] if case["storage"] == "bf16r32" else d
    if kind == "batch":
        if case["steps"] > 500 or case["ramp"] or case["nx"] == 0:
            return None  # a long chaotic run, or many shapes
        lats = _lattices(case, seed)
        both = [_start64(case, f, r) for *_, r, f in lats]
        f = torch.stack([a for a, _ in both], 1)
        seeds = torch.tensor([x[1] for x in lats], device=f.device).view(-1, 1, 1)
        k = lats[0][0]
        every = case["sample_every"] or case["steps"]
        rows = []
        for t in range(0, case["steps"], every):
            f = _steps(f, case["q"], case["model"], k, seeds, t, every)
            rows.append(_observables(f, case["q"], k, t + every))
        out = [torch.stack(rows, 1)]
        for l in range(len(lats)):
            d = f[:, l] - both[l][1]
            out.append([d[0], d[1:]] if case["storage"] == "bf16r32" else d)
        return out
    if kind == "judge":
        x, act, seeds = _judge_inputs(case, seed)
        c, n = case["coarse"], case["n"]
        big = x[:, :3].double().repeat_interleave(c, 2).repeat_interleave(c, 3)
        rho = big[:, 0]
        f = _steady(7, rho, big[:, 1] / rho, big[:, 2] / rho)
        k = dict(CIL, B=torch.tensor(act, dtype=torch.float32, device=f.device).double().view(n, 1, 1))
        f = _steps(f, 7, "cil", k, torch.tensor(seeds, device=f.device).view(n, 1, 1), 0, case["k"])
        out = torch.stack(_fields(_stream(f, 7), 7), 1)
        h = case["side"] // c
        out = out.view(n, 3, h, c, h, c).mean((3, 5))
        return torch.cat([out, x[:, 3:].double()], 1)
    x, t, perm, theta, m, v = _network_inputs(case, seed)
    x, t = x.double(), t.double()
    mean = x.mean((0, 2, 3)).view(1, 4, 1, 1)
    std = x.std((0, 2, 3), unbiased=False).view(1, 4, 1, 1)
    par = [(p.to(torch.bfloat16) if p.dim() == 4 else p).double().requires_grad_() for p in theta]
    at = perm[:case["n"]].long() if kind == "train" else torch.arange(case["n"])
    xn = ((x - mean) / std)[at]
    a1 = torch.relu(_conv64(xn, par[0], par[1]))
    a2 = torch.relu(_conv64(a1, par[2], par[3]))
    y = xn[:, :3] + _conv64(a2, par[4], par[5])
    if kind == "predict":
        return torch.cat([(y * std[:, :3] + mean[:, :3]).detach(), x[:, 3:]], 1)
    tn = ((t - mean) / std)[at][:, :3]
    loss = ((y - tn) ** 2).mean()
    grads = torch.autograd.grad(loss, par)
    out = [[], [], []]
    for th, mk, vk, g in zip(theta, m, v, grads):
        mk, vk = 0.9 * mk.double() + 0.1 * g, 0.999 * vk.double() + 0.001 * g * g
        th = th.double() - LR * (mk / (1.0 - 0.9)) / (torch.sqrt(vk / (1.0 - 0.999)) + 1e-8)
        for o, val in zip(out, (th, mk, vk)):
            o.append(val.reshape(-1))
    return [loss.detach().reshape(1), out]
