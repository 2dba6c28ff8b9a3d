"""Timed cases of the library's main paths, each through its public entry
points, from calls bound by latency to the largest inputs.

A case is a dict of plain values; its "path" says what one pass does:
  forces   NBody.forces(): tree, lists, forces and results at the current
           positions (open boundaries, or TreePM in a periodic box)
  step     NBody.step(): one kick-drift-kick step, which holds a forces()
  compute  bhq_compute on resident lists, and the results in input order
  batch    one list build over many independent systems, forces, results
  pm       bhq_pm_compute alone
  lists    the caller's own groups and lists through the set calls for
           device memory, forces, results

The FP32 kernels' accelerations and potentials are FP32 values that the
library hands over in FP64 arrays; a pass returns them as FP32 (the same
values).  Everything else is returned as it is.
"""
import math

import numpy as np
import torch

from paper_1812_07313_amd import bhq
from paper_1812_07313_amd.nbody import NBody

KERNELS = {"mono": bhq.MONO, "quad": bhq.QUAD, "soft": bhq.QUAD_SOFT,
           "split": bhq.SPLIT_QUAD, "split_mono": bhq.SPLIT_MONO}
DEV = "cuda"
F64 = torch.float64


def listed():
    return [
        # the smallest systems that are integrated on their own: latency
        dict(name="plummer_2k", path="forces", dist="plummer", n=2048, eps=1 / 32, theta=0.5,
             ncrit=64, kernel="quad", fp64=False),
        # the Plummer sphere of the small benchmark configuration
        dict(name="plummer_16k", path="forces", dist="plummer", n=16384, eps=1 / 64, theta=0.5,
             ncrit=64, kernel="quad", fp64=False),
        # time steps of a mid-sized sphere in equilibrium, an odd particle count
        dict(name="plummer_100k_step", path="step", dist="plummer", n=100003, eps=2.0 ** -8,
             theta=0.65, ncrit=256, kernel="quad", fp64=False, sort=0, dt=2.0 ** -10),
        # FP64 forces, as a reference run uses them
        dict(name="plummer_131k_fp64", path="forces", dist="plummer", n=131071, eps=1 / 128,
             theta=0.5, ncrit=64, kernel="soft", fp64=True),
        # the uniform cube of the benchmark: the force kernel on resident
        # lists, and a whole force evaluation
        dict(name="cube_1m_compute", path="compute", dist="cube", n=1 << 20, eps=1e-3, theta=0.5,
             ncrit=256, kernel="quad", fp64=False),
        dict(name="cube_1m", path="forces", dist="cube", n=1 << 20, eps=1e-3, theta=0.5,
             ncrit=256, kernel="quad", fp64=False),
        # strongly clustered particles: deep trees, uneven lists
        dict(name="clustered_4m", path="forces", dist="clustered", n=1 << 22, eps=2e-4, theta=0.5,
             ncrit=256, kernel="quad", fp64=False),
        # many independent systems in one call
        dict(name="batch_256", path="batch", nsys=256, lo=10.0, hi=16.0, theta=0.6, ncrit=128,
             kernel="quad", fp64=False),
        # TreePM forces all in FP64, a side that is no power of two
        dict(name="treepm_60_fp64", path="forces", dist="lattice", n=60 ** 3, side=60, mesh=60,
             theta=0.5, ncrit=128, kernel="split", fp64=True),
        # the largest: a TreePM step of the 2^24 lattice
        dict(name="treepm_256_step", path="step", dist="lattice", n=1 << 24, side=256, mesh=256,
             theta=0.5, ncrit=128, kernel="split", fp64=False, sort=8, dt=1e-3),
        # the particle mesh alone, unsorted particles
        dict(name="pm_128", path="pm", n=2000003, mesh=128),
        # the caller's own groups and lists, monopole cells
        dict(name="own_lists_mono", path="lists", ng=301, ni=57, np=711, nc=905, kernel="mono",
             fp64=False),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(2.0 ** rng.uniform(math.log2(lo), math.log2(hi))))


def draw(rng):
    path = rng.choice(("forces", "forces", "forces", "step", "step", "compute", "batch", "treepm",
                       "treepm", "pm", "lists"))
    fp64 = rng.random() < 0.25
    if path in ("forces", "step", "compute"):
        n = _log_uniform(rng, 1000, 1 << 21 if fp64 else 3 << 20)
        c = dict(path=path, dist=rng.choice(("plummer", "cube", "sphere", "clustered")), n=n,
                 eps=round(0.4 / n ** (1 / 3), 6), theta=round(rng.uniform(0.5, 0.8), 3),
                 ncrit=rng.choice((64, 128, 256)), kernel=rng.choice(("quad", "quad", "soft",
                                                                      "mono")), fp64=fp64)
        if path == "step":
            c.update(dist="plummer", sort=rng.choice((0, 8)), dt=2.0 ** -10)
        return c
    if path == "batch":
        return dict(path="batch", nsys=rng.randint(5, 200), lo=10.0, hi=round(rng.uniform(12, 16),
                                                                             2),
                    theta=round(rng.uniform(0.5, 0.8), 3), ncrit=rng.choice((64, 128)),
                    kernel=rng.choice(("quad", "mono")), fp64=fp64)
    if path == "treepm":
        side = _log_uniform(rng, 48, 110 if fp64 else 200)
        c = dict(path=rng.choice(("forces", "step")), dist="lattice", n=side ** 3, side=side,
                 mesh=side + side % 2, theta=round(rng.uniform(0.5, 0.7), 3),
                 ncrit=rng.choice((64, 128)), kernel=rng.choice(("split", "split", "split_mono")),
                 fp64=fp64)
        if c["path"] == "step":
            c.update(sort=rng.choice((0, 8)), dt=1e-3)
        return c
    if path == "pm":
        mesh = 2 * _log_uniform(rng, 16, 110)
        return dict(path="pm", n=int(mesh ** 3 * rng.uniform(0.3, 1.5)) + 1, mesh=mesh)
    return dict(path="lists", ng=_log_uniform(rng, 40, 3000), ni=rng.randint(20, 150),
                np=rng.randint(100, 1500), nc=rng.randint(100, 1500),
                kernel=rng.choice(("mono", "quad")), fp64=fp64)


# --- inputs -------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, dtype=F64, device=DEV)


def _direction(g, n):
    v = torch.randn(n, 3, generator=g, dtype=F64, device=DEV)
    return v / v.norm(dim=1, keepdim=True)


def _plummer(g, n):
    """Unit scale radius, cut at the radius that holds 0.999 of the mass."""
    r = (((0.999 * _rand(g, n)).clamp_min(1e-12)) ** (-2 / 3) - 1.0) ** -0.5
    return r[:, None] * _direction(g, n)


def _positions(c, g):
    n, dist = c["n"], c["dist"]
    if dist == "plummer":
        return _plummer(g, n)
    if dist == "cube":
        return _rand(g, n, 3).float().double()
    if dist == "sphere":
        return _rand(g, n, 1) ** (1 / 3) * _direction(g, n)
    if dist == "clustered":
        # 512 Plummer spheres with dN/dM ~ M^-1.9 on [1, 1000] and a scale
        # radius of 0.02 (M / M_max)^(1/3), over a 10 % uniform background
        nb = n // 10
        mass = (1.0 + _rand(g, 512) * (1000.0 ** -0.9 - 1.0)) ** (-1 / 0.9)
        which = torch.multinomial(mass, n - nb, replacement=True, generator=g)
        radius = 0.02 * (mass / mass.max()) ** (1 / 3)
        x = _plummer(g, n - nb) * radius[which, None] + _rand(g, 512, 3)[which]
        return torch.cat([x, _rand(g, nb, 3)])
    s = c["side"]  # a lattice with displacements, in the periodic unit box
    i = (torch.arange(s, dtype=F64, device=DEV) + 0.5) / s
    x = torch.stack(torch.meshgrid(i, i, i, indexing="ij"), -1).reshape(-1, 3)
    x = (x + 0.02 * torch.randn(n, 3, generator=g, dtype=F64, device=DEV)) % 1.0
    return torch.where(x >= 1.0, torch.zeros_like(x), x)


def _particles(c, seed):
    g = _gen(seed)
    x = _positions(c, g)
    n = c["n"]
    m = torch.full((n,), 1.0 / n, dtype=F64, device=DEV)
    # isotropic velocities: the Plummer model's dispersion at each radius, so
    # that a sphere stays as it is over many steps; a lattice moves by a
    # tenth of its spacing per step
    v = torch.randn(n, 3, generator=g, dtype=F64, device=DEV)
    if c["dist"] == "lattice":
        v *= 0.1 / c["side"] / 1e-3
    else:
        v *= (1.0 + (x * x).sum(1, keepdim=True)) ** -0.25 / math.sqrt(6.0)
    return x, v, m


def _split(c):
    """Split scale of 1.25 lattice spacings and the cutoff at 4.5 of it."""
    rs = 1.25 / c["side"]
    return rs, 4.5 * rs


def _systems(c, seed):
    """Independent Plummer systems, their sizes log-uniform (the case's own),
    and softening."""
    sizes = torch.round(2.0 ** (c["lo"] + (c["hi"] - c["lo"]) * _rand(_gen(c["nsys"]), c["nsys"])))
    sizes = sizes.to(torch.int64)
    x = _plummer(_gen(seed), int(sizes.sum()))
    each = torch.repeat_interleave(sizes.to(F64), sizes)
    off = np.concatenate([[0], np.cumsum(sizes.cpu().numpy())]).astype(np.int64)
    return off, x, 1.0 / each, (0.25 / each ** (1 / 3)) ** 2


def _own_lists(c, seed):
    """Groups of particles in small cubes, and lists of particles and cells
    around each; sizes vary from group to group about the case's."""
    g, sizes = _gen(seed), _gen(c["ng"])
    ng = c["ng"]

    def offsets(k):
        cnt = (k * (0.5 + _rand(sizes, ng))).to(torch.int64) + 1
        return torch.cat([cnt.new_zeros(1), cnt.cumsum(0)]), cnt

    s = dict(centre=_rand(g, ng, 3))
    for key, k, w in (("i", c["ni"], 0.02), ("jp", c["np"], 0.1), ("jc", c["nc"], 1.0)):
        off, cnt = offsets(k)
        t = int(off[-1])
        s[key + "_off"] = off
        d = _rand(g, t, 3) - 0.5
        if key == "jc":  # accepted cells lie away from the group
            d = d + 0.2 * d / d.norm(dim=1, keepdim=True)
        s[key] = (torch.repeat_interleave(s["centre"], cnt, 0) + w * d).contiguous()
    s["jp_m"] = (0.5 + _rand(g, len(s["jp"]))) / len(s["jp"])
    s["jc_m"] = (0.5 + _rand(g, len(s["jc"]))) / len(s["jc"])
    a = 0.03 * (_rand(g, len(s["jc"]), 3) - 0.5)
    q = 3.0 * a[:, :, None] * a[:, None, :]
    q = (q - torch.eye(3, dtype=F64, device=DEV) * (a * a).sum(1)[:, None, None])
    q = q * s["jc_m"][:, None, None]
    s["jc_q"] = torch.stack([q[:, 0, 0], q[:, 0, 1], q[:, 0, 2], q[:, 1, 1], q[:, 1, 2],
                             q[:, 2, 2]], 1).contiguous()
    return s


OWN_EPS = 1e-3


# --- states ---------------------------------------------------------------------

class State:
    """The handles and arrays a program holds; handles closed with it."""

    def __init__(self, case):
        self.case = case
        self.nb = self.ctx = self.pm = None

    def __del__(self):
        torch.cuda.synchronize()
        if self.nb is not None:
            self.nb.close()
        if self.ctx is not None:
            bhq.bhq_destroy(self.ctx)
        if self.pm is not None:
            bhq.bhq_pm_destroy(self.pm)


def _precision(c):
    return bhq.FP64 if c["fp64"] else bhq.FP32_OFS64


def prepare(case, seed):
    c = case
    s = State(c)
    path = c["path"]
    if path == "pm":
        g = _gen(seed)
        s.x = _rand(g, c["n"], 3)
        s.m = (0.5 + _rand(g, c["n"])) / c["n"]
        s.a = torch.zeros_like(s.x)
        s.pot = torch.zeros_like(s.m)
        s.pm = bhq.bhq_pm_create(c["mesh"], 1.0, 1.25 / c["mesh"])
        return s
    if path == "lists":
        s.l = _own_lists(c, seed)
        s.ctx = bhq.bhq_create(0, KERNELS[c["kernel"]], _precision(c))
        s.a = torch.zeros_like(s.l["i"])
        s.pot = torch.zeros(len(s.a), dtype=F64, device=DEV)
        return s
    if path == "batch":
        s.off, s.x, s.m, s.eps2 = _systems(c, seed)
        s.ctx = bhq.bhq_create(0, KERNELS[c["kernel"]], _precision(c))
        s.a = torch.zeros_like(s.x)
        s.pot = torch.zeros_like(s.m)
        return s
    x, v, m = _particles(c, seed)
    if path == "compute":
        s.ctx = bhq.bhq_create(0, KERNELS[c["kernel"]], _precision(c))
        bhq.bhq_set_eps(s.ctx, c["eps"])
        bhq.bhq_build_lists_device(s.ctx, x, m, c["theta"], c["ncrit"])
        s.a = torch.zeros_like(x)
        s.pot = torch.zeros_like(m)
        return s
    more = {}
    if c["dist"] == "lattice":
        rs, rcut = _split(c)
        more = dict(box=1.0, rs=rs, rcut=rcut, pm_mesh=c["mesh"])
    s.nb = NBody(x, v, m, c.get("eps", 0.0), c["theta"], c["ncrit"], kernel=KERNELS[c["kernel"]],
                 precision=_precision(c), sort_every=c.get("sort", 0), **more)
    if path == "step":
        s.nb.forces()  # a run has the forces of its last step in hand
    return s


def run(state):
    s, c = state, state.case
    path = c["path"]
    if path == "step":
        s.nb.step(c["dt"])
        return {"x": s.nb.x, "v": s.nb.v, "a": s.nb.a if c["fp64"] else s.nb.a.float()}
    if path == "forces":
        s.nb.forces()
        a, pot = s.nb.a, s.nb.pot
    elif path == "pm":
        bhq.bhq_pm_compute(s.pm, s.x, s.m, s.a, s.pot)
        return {"a": s.a, "pot": s.pot}
    else:
        if path == "batch":
            bhq.bhq_build_lists_device_batch(s.ctx, s.off, s.x, s.m, c["theta"], c["ncrit"],
                                             eps2=s.eps2)
        elif path == "lists":
            t = s.l
            bhq.bhq_set_groups_dev(s.ctx, t["i_off"], t["centre"], t["jp_off"], t["jc_off"])
            bhq.bhq_set_i_dev(s.ctx, t["i"])
            bhq.bhq_set_eps(s.ctx, OWN_EPS)
            bhq.bhq_set_jp_dev(s.ctx, 0, t["jp"], t["jp_m"])
            bhq.bhq_set_jc_dev(s.ctx, 0, t["jc"], t["jc_m"], t["jc_q"])
        bhq.bhq_compute(s.ctx)
        bhq.bhq_get_result_device(s.ctx, s.a, s.pot)
        a, pot = s.a, s.pot
    if not c["fp64"]:
        a, pot = a.float(), pot.float()
    return {"a": a, "pot": pot}


# --- what a pass cannot do without -----------------------------------------------

def work(case):
    """Bytes: particles in (position and mass) and results out, once; flops:
    the interactions of an average particle at the case's opening angle
    (for the open trees about 1270 cells and 1100 particles at 0.5; for the
    split kernels the particles within the cutoff), 20 per particle term and
    53 per cell term."""
    c = case
    path = c["path"]
    if path == "pm":
        n3 = c["mesh"] ** 3
        return {"bytes": 64.0 * c["n"], "flops": 300.0 * c["n"] + 12.5 * n3 * math.log2(n3)}
    if path == "lists":
        ni, npp, nc = c["ng"] * c["ni"], c["np"], c["nc"]
        quad = c["kernel"] == "quad"
        return {"bytes": c["ng"] * (32.0 * npp + (80.0 if quad else 32.0) * nc) + 56.0 * ni,
                "flops": ni * (20.0 * npp + (53.0 if quad else 20.0) * nc)}
    if path == "batch":
        n = c["nsys"] * (2.0 ** c["hi"] - 2.0 ** c["lo"]) / ((c["hi"] - c["lo"]) * math.log(2.0))
    else:
        n = c["n"]
    cell = 20.0 if c["kernel"] in ("mono", "split_mono") else 53.0
    if c.get("dist") == "lattice":
        inside = 4.0 / 3.0 * math.pi * (4.5 * 1.25) ** 3  # particles within the cutoff
        flops = n * inside * 36.0
        if c["mesh"]:
            flops += 300.0 * n + 12.5 * c["mesh"] ** 3 * math.log2(c["mesh"] ** 3)
    else:
        pairs, cells = 1100.0 * (0.5 / c["theta"]) ** 1.5, 1270.0 * (0.5 / c["theta"]) ** 3
        flops = n * (20.0 * min(n, pairs) + cell * min(0.2 * n, cells))
    return {"bytes": 64.0 * n + (96.0 * n if path == "step" else 0.0), "flops": flops}


# --- the same in 64 bits -----------------------------------------------------------

PAIRS = 6e10       # direct sums up to this many pairs
CHUNK = 1 << 25    # pairs at a time


def _direct(xi, x, m, eps2):
    """Softened direct sum over all particles at xi (eps2: one value or one
    per xi)."""
    a = torch.empty_like(xi)
    p = torch.empty(len(xi), dtype=F64, device=DEV)
    step = max(1, CHUNK // len(x))
    e2 = eps2 if isinstance(eps2, torch.Tensor) else torch.full((len(xi),), eps2, dtype=F64,
                                                                device=DEV)
    for k in range(0, len(xi), step):
        t = xi[k:k + step]
        d = [x[None, :, q] - t[:, None, q] for q in range(3)]
        ri = (d[0] * d[0] + d[1] * d[1] + d[2] * d[2] + e2[k:k + step, None]).rsqrt_()
        mr = m * ri
        p[k:k + step] = -mr.sum(1)
        mr *= ri
        mr *= ri
        for q in range(3):
            a[k:k + step, q] = (mr * d[q]).sum(1)
    return a, p


def _short(x, m, rs, rcut):
    """Periodic short-range sum inside the cutoff (unit box)."""
    order = torch.argsort(x[:, 0])
    xs, ms = x[order], m[order]
    a, p = torch.empty_like(x), torch.empty_like(m)
    step = 256
    for k in range(0, len(xs), step):
        t = xs[k:k + step]
        lo, hi = float(t[0, 0]) - rcut, float(t[-1, 0]) + rcut
        u = xs[:, 0]
        near = ((u >= lo) & (u <= hi)) | (u >= lo + 1.0) | (u <= hi - 1.0)
        y, w = xs[near], ms[near]
        d = y[None] - t[:, None]
        d -= torch.round(d)
        r2 = (d * d).sum(2)
        keep = (r2 > 0.0) & (r2 < rcut * rcut)
        r = torch.where(keep, r2, torch.ones_like(r2)).sqrt()
        z = r / (2.0 * rs)
        e = torch.erfc(z)
        g = e + z * torch.exp(-z * z) * (2.0 / math.sqrt(math.pi))
        mk = torch.where(keep, w / r, torch.zeros_like(r))
        p[order[k:k + step]] = -(mk * e).sum(1)
        a[order[k:k + step]] = ((mk * g / (r * r))[:, :, None] * d).sum(1)
    return a, p


def _mesh(x, m, n, rs):
    """Long-range part by the particle-mesh method (unit box)."""
    u = x * n
    i0 = torch.floor(u + 0.5)
    d = u - i0
    w = torch.stack([0.5 * (0.5 - d) ** 2, 0.75 - d * d, 0.5 * (0.5 + d) ** 2])  # [3, n, axis]
    i0 = i0.to(torch.int64)

    def points():
        for ox in range(3):
            for oy in range(3):
                for oz in range(3):
                    i = [(i0[:, q] + o - 1) % n for q, o in enumerate((ox, oy, oz))]
                    yield (i[0] * n + i[1]) * n + i[2], w[ox, :, 0] * w[oy, :, 1] * w[oz, :, 2]

    rho = torch.zeros(n ** 3, dtype=F64, device=DEV)
    for at, wt in points():
        rho.index_add_(0, at, m * wt)
    rk = torch.fft.rfftn(rho.reshape(n, n, n) * n ** 3)
    f = torch.fft.fftfreq(n, d=1.0 / n, dtype=F64, device=DEV)
    k = [2.0 * math.pi * f[:, None, None], 2.0 * math.pi * f[None, :, None],
         2.0 * math.pi * f[None, None, :n // 2 + 1].abs()]
    k2 = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
    k2[0, 0, 0] = 1.0
    win = torch.ones_like(k2)
    for q in k:
        win = win * torch.sinc(q / (2.0 * math.pi * n)) ** 6
    green = -4.0 * math.pi * torch.exp(-k2 * rs * rs) / k2 / win
    green[0, 0, 0] = 0.0
    phi = green * rk
    nyq = 2.0 * math.pi * (n // 2)
    fields = [torch.fft.irfftn(-1j * torch.where(q.abs() == nyq, torch.zeros_like(q), q) * phi,
                               s=(n, n, n)).reshape(-1) for q in k]
    fields.append(torch.fft.irfftn(phi, s=(n, n, n)).reshape(-1))
    out = torch.zeros(len(x), 4, dtype=F64, device=DEV)
    for at, wt in points():
        for q in range(4):
            out[:, q] += wt * fields[q][at]
    return out[:, :3].contiguous(), out[:, 3].contiguous()


def _forces(c, x, m):
    if c["dist"] == "lattice":
        rs, rcut = _split(c)
        a, p = _short(x, m, rs, rcut)
        al, pl = _mesh(x, m, c["mesh"], rs)
        return a + al, p + pl
    return _direct(x, x, m, c["eps"] ** 2)


def exact(case, seed):
    c = case
    path = c["path"]
    if path == "pm":
        g = _gen(seed)
        x = _rand(g, c["n"], 3)
        m = (0.5 + _rand(g, c["n"])) / c["n"]
        a, p = _mesh(x, m, c["mesh"], 1.25 / c["mesh"])
        return {"a": a, "pot": p}
    if path == "lists":
        return _exact_lists(c, _own_lists(c, seed))
    if path == "batch":
        off, x, m, eps2 = _systems(c, seed)
        if float(((off[1:] - off[:-1]).astype(float) ** 2).sum()) > PAIRS:
            return None
        parts = [_direct(x[b:e], x[b:e], m[b:e], eps2[b:e]) for b, e in zip(off[:-1], off[1:])]
        return {"a": torch.cat([a for a, _ in parts]), "pot": torch.cat([p for _, p in parts])}
    if float(c["n"]) ** 2 > PAIRS:
        return None
    x, v, m = _particles(c, seed)
    if path != "step":
        a, p = _forces(c, x, m)
        return {"a": a, "pot": p}
    if c["sort"]:  # the rows are in tree order
        return None
    dt = c["dt"]
    v = v + 0.5 * dt * _forces(c, x, m)[0]
    x = x + dt * v
    if c["dist"] == "lattice":
        x = x - torch.floor(x)
    a = _forces(c, x, m)[0]
    return {"x": x, "v": v + 0.5 * dt * a, "a": a}


def _exact_lists(c, s):
    a, p = torch.empty_like(s["i"]), torch.empty(len(s["i"]), dtype=F64, device=DEV)
    io, po, co = (s[k].tolist() for k in ("i_off", "jp_off", "jc_off"))
    quad = c["kernel"] == "quad"
    for g in range(c["ng"]):
        i, jp, jc = (slice(o[g], o[g + 1]) for o in (io, po, co))
        t = s["i"][i]
        ag, pg = _direct(t, s["jp"][jp], s["jp_m"][jp], OWN_EPS ** 2)
        ac, pc = _direct(t, s["jc"][jc], s["jc_m"][jc], OWN_EPS ** 2)
        ag, pg = ag + ac, pg + pc
        if quad:
            d = s["jc"][jc][None] - t[:, None]
            q = s["jc_q"][jc][:, [0, 1, 2, 1, 3, 4, 2, 4, 5]].reshape(-1, 3, 3)
            qd = (q[None] * d[:, :, None, :]).sum(3)
            dqd = (qd * d).sum(2)
            ri = ((d * d).sum(2) + OWN_EPS ** 2).rsqrt()
            r5 = ri ** 5
            pg = pg - (0.5 * dqd * r5).sum(1)
            ag = ag + ((2.5 * dqd * r5 * ri * ri)[:, :, None] * d - r5[:, :, None] * qd).sum(1)
        a[i], p[i] = ag, pg
    return {"a": a, "pot": p}
