"""The work that a simulation has this framework do, as cases to time.

A case is one call (or one pair of calls) through the public entry points of
``paper_2512_12629_amd`` on particles that look like those of a run: a lattice
displaced by a k^-2 Zel'dovich field, part of it moved into Plummer spheres
(halos), or plain uniform positions.  ``op`` says which call:

  force      Cube2.force           PM of every level + PP, once per time step
  backward   Cube2.force_backward  its adjoint, once per step of a gradient
  kick       Cube2.kick_drift      kick, drift and re-sort, once per time step
  pack       Cube2.pack            quantise and sort new positions
  velocity   Cube2.vel_encode + vel_decode   16-bit velocities of the stored state
  force64    Cube2.force_f64       the FP64 form that FP32 forces are checked with
  tiles      Cube2Tiled.force      the tile+buffer force of a sharded box

Case fields: n_p (lattice side, N = n_p^3), n_fine (mesh side), ratio (coarse
spacing, 0 = one level), spheres and per_sphere (halos), uniform, tsc,
isolated, b_fine, b_pp, move (rms drift of a step in fine cells), and for the
tiles tile and buffer.
"""
import math

import torch

import paper_2512_12629_amd as cube2

B_COARSE = 14.0
KICK = 0.5


def _case(name, op, n_p, n_fine, ratio=0, spheres=0, per_sphere=2048, uniform=False, tsc=False,
          isolated=False, b_fine=2.0, b_pp=0.2, move=0.25, tile=64, buffer=32):
    c = dict(op=op, n_p=n_p, n_fine=n_fine, ratio=ratio, spheres=spheres, per_sphere=per_sphere,
             uniform=uniform, tsc=tsc, isolated=isolated, b_fine=b_fine, b_pp=b_pp, move=move,
             tile=tile, buffer=buffer)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest box of the tests, one level: launches and latency count
        _case("force_small", "force", 32, 64, uniform=True),
        # one level, a lattice before halos form: an ordinary small run
        _case("force_one_level", "force", 128, 256),
        # two levels with halos: the middle of the range of a production run
        _case("force_two_level", "force", 256, 512, 4, 1000),
        # one GPU's tile of a large run: the benchmark's workload
        _case("force_largest", "force", 512, 1024, 4, 8000),
        # the paper's own settings (TSC, beta = 3.5) with a ragged particle number
        _case("force_paper", "force", 201, 512, 4, 300, tsc=True, b_fine=3.5, b_pp=0.0625),
        # the force adjoint of the gradient runs (one level, 128^3 on 256^3)
        _case("backward_one_level", "backward", 128, 256),
        # the force adjoint of the benchmark's workload
        _case("backward_largest", "backward", 512, 1024, 4, 8000),
        # the other half of a time step: kick, drift and re-sort
        _case("kick_largest", "kick", 512, 1024, 4, 8000),
        # positions read from initial conditions or a snapshot, ragged number
        _case("pack_ragged", "pack", 301, 512, 4, 1000),
        # storing and restoring the 16-bit velocities of the state
        _case("velocity", "velocity", 256, 512, 4, 1000),
        # the FP64 form, which a user checks FP32 forces against
        _case("force64", "force64", 128, 256),
        # the tile+buffer force over a whole small box: many calls on small local boxes
        _case("tiles", "tiles", 128, 256, 4, 60),
    ]


def draw(rng):
    op = rng.choice(["force"] * 5 + ["backward"] * 3 + ["kick"] * 2 + ["pack", "velocity", "force64", "tiles"])
    if op == "tiles":
        return _case(None, op, rng.randrange(60, 129), rng.choice([128, 256]), 4, rng.randrange(0, 60),
                     per_sphere=rng.choice([512, 1000, 2048]))
    n_fine = rng.choice([64, 128, 256] if op == "force64" else [32, 64, 128, 256, 512, 512, 1024])
    ratio = rng.choice([0, 2, 4, 4, 8]) if n_fine >= 64 else 0
    lo, hi = n_fine * 0.3, n_fine * 0.5
    n_p = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    n = n_p ** 3
    per = rng.choice([256, 700, 1500, 2048, 3001])
    spheres = int(n * rng.uniform(0.0, 0.12) / per)
    uniform = rng.random() < 0.15
    wide = op in ("force", "force64") and n_fine <= 512 and rng.random() < 0.3
    b_fine, b_pp = rng.choice([(3.5, 0.0625), (3.0, 0.3)]) if wide else rng.choice([(2.0, 0.2), (2.0, 0.2), (1.5, 0.1)])
    return _case(None, op, n_p, n_fine, ratio, 0 if uniform else spheres, per, uniform,
                 tsc=op != "pack" and rng.random() < 0.25, isolated=rng.random() < 0.1, b_fine=b_fine,
                 b_pp=b_pp, move=rng.choice([0.05, 0.25, 1.0, 3.0]))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _positions(case, seed):
    """float32 (3, N) box-unit positions in a caller's order, on the GPU."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(1000003 * seed + 12629)
    n_p = case["n_p"]
    n = n_p ** 3
    if case["uniform"]:
        x = torch.rand((3, n), generator=gen, device=dev, dtype=torch.float32)
    else:
        noise = torch.randn((n_p, n_p, n_p), generator=gen, device=dev, dtype=torch.float32)
        nk = torch.fft.rfftn(noise)
        del noise
        f = torch.fft.fftfreq(n_p, device=dev) * n_p
        r = torch.fft.rfftfreq(n_p, device=dev) * n_p
        k2 = f[:, None, None] ** 2 + f[None, :, None] ** 2 + r[None, None, :] ** 2
        k2[0, 0, 0] = 1.0
        nk *= k2 ** -1.5
        nk[0, 0, 0] = 0.0
        del k2
        x = torch.empty((3, n), device=dev, dtype=torch.float32)
        var = 0.0
        for d, k in enumerate((r[None, None, :], f[None, :, None], f[:, None, None])):
            psi = torch.fft.irfftn(1j * k * nk, s=(n_p, n_p, n_p))
            x[d] = psi.reshape(-1)
            var += float(psi.double().square().mean())
            del psi
        del nk
        x *= 0.25 / math.sqrt(max(var, 1e-30))
        g = torch.arange(n_p, device=dev, dtype=torch.float32) + 0.5
        v = x.view(3, n_p, n_p, n_p)
        v[0] += g[None, None, :]
        v[1] += g[None, :, None]
        v[2] += g[:, None, None]
        x /= n_p
    k = case["spheres"] * case["per_sphere"]
    if k:
        # one particle from each of k stretches of the lattice order
        step = n // k
        idx = (torch.arange(k, device=dev) * step
               + torch.randint(0, step, (k,), generator=gen, device=dev))
        centre = torch.rand((3, case["spheres"]), generator=gen, device=dev)
        # Plummer radii by the inverse of the enclosed mass, truncated at 10 a
        top = (1.0 + 0.01) ** -1.5
        u = torch.rand(k, generator=gen, device=dev).clamp_(min=1e-6) * top
        rad = (0.5 / case["n_fine"]) / torch.sqrt(u ** (-2.0 / 3.0) - 1.0)
        dirs = torch.randn((3, k), generator=gen, device=dev)
        dirs /= dirs.norm(dim=0, keepdim=True)
        x[:, idx] = centre.repeat_interleave(case["per_sphere"], dim=1) + dirs * rad
    x -= torch.floor(x)
    x[x >= 1.0] = 0.0
    if case["isolated"]:
        x *= 0.5
    return x.contiguous()


def _random(case, seed, n):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7919 * seed + 17)
    return torch.randn((3, n), generator=gen, device="cuda")


def _config(case):
    flags = 0
    if case["tsc"]:
        flags |= cube2.CUBE2_ASSIGN_TSC
    if case["isolated"]:
        flags |= cube2.CUBE2_ISOLATED
    if case["op"] == "force64":
        flags |= cube2.CUBE2_FP64_FORM
    return cube2.Config(n_fine=case["n_fine"], coarse_ratio=case["ratio"], b_coarse=B_COARSE,
                        b_fine=case["b_fine"], b_pp=case["b_pp"], flags=flags)


def prepare(case, seed):
    x = _positions(case, seed)
    n = x.shape[1]
    op = case["op"]
    if op == "tiles":
        tiled = cube2.Cube2Tiled(_config(case), case["tile"], case["buffer"], n)
        pos, cs, _ = tiled.g.pack(x)
        return {"op": op, "sim": tiled, "pos": pos, "cs": cs}
    sim = cube2.Cube2(_config(case), n)
    if op == "pack":
        return {"op": op, "sim": sim, "x": x}
    pos, cs, _ = sim.pack(x)
    s = {"op": op, "sim": sim, "pos": pos, "cs": cs}
    if op == "backward":
        s["acc_bar"] = _random(case, seed, n)
    elif op == "kick":
        v = _random(case, seed, 2 * n)
        s["vel"] = v[:, :n].contiguous()
        s["acc"] = v[:, n:].contiguous()
        s["drift"] = case["move"] / math.sqrt(3.0 * (1.0 + KICK * KICK))
    elif op == "velocity":
        s["vel"] = _random(case, seed, n)
    return s


def run(s):
    op, sim = s["op"], s["sim"]
    if op in ("force", "tiles"):
        return sim.force(s["pos"], s["cs"])
    if op == "backward":
        return sim.force_backward(s["pos"], s["cs"], s["acc_bar"])
    if op == "kick":
        return sim.kick_drift(s["pos"], s["cs"], s["vel"], s["acc"], KICK, s["drift"])
    if op == "pack":
        return sim.pack(s["x"])
    if op == "velocity":
        coded = sim.vel_encode(s["pos"], s["cs"], s["vel"])
        return coded, sim.vel_decode(s["pos"], s["cs"], *coded)
    return sim.force_f64(s["pos"], s["cs"])


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

def work(case):
    n = case["n_p"] ** 3
    nf = case["n_fine"]
    cells = (nf // 2) ** 3
    op = case["op"]
    ios = 6 * n + 4 * (cells + 1)
    if op == "pack":
        return {"bytes": 12 * n + ios + 4 * n, "flops": 3 * n}
    if op == "kick":
        return {"bytes": 2 * ios + 12 * n + 24 * n + 4 * n, "flops": 12 * n}
    if op == "velocity":
        bulk = 12 * (nf // (case["ratio"] or 4)) ** 3
        return {"bytes": 2 * (ios + 6 * n + 12 * n + bulk), "flops": 18 * n}
    levels = [nf] + ([nf // case["ratio"]] if case["ratio"] else [])
    # each level: a real transform forth and back, the product with G, and a
    # particle's assignment, differences and interpolation
    nodes = 27 if case["tsc"] else 8
    mesh = sum(2 * 2.5 * m ** 3 * 3 * math.log2(m) + m ** 3 + 2 * n * nodes + 6 * 8 * n for m in levels)
    # ordered pairs within the cutoff: the even part by its density, and the
    # share of a truncated Plummer sphere's pairs (a = 0.5) closer than b_fine
    vol = nf ** 3 * (0.125 if case["isolated"] else 1.0)
    near = {1.5: 0.7, 2.0: 0.82, 3.0: 0.91, 3.5: 0.94}.get(case["b_fine"], 0.8)
    pairs = n * (n / vol) * 4.19 * case["b_fine"] ** 3 + near * case["spheres"] * case["per_sphere"] ** 2
    if op == "backward":
        return {"bytes": ios + 24 * n, "flops": 2 * mesh + 6 * nodes * n + 52 * pairs}
    return {"bytes": ios + (24 if op == "force64" else 12) * n, "flops": mesh + 28 * pairs}


# ---------------------------------------------------------------------------
# The same results in 64 bits
# ---------------------------------------------------------------------------

F64 = torch.float64


def _sinc(x):
    return torch.sinc(x / math.pi)


def _profile_k(k, b):
    """Transform of the softened profile (eq. 13), 12/u^4 (2 - 2 cos u - u sin u)."""
    u = 0.5 * k * b
    s = torch.zeros_like(u)
    u2 = u * u
    for j in range(11, 1, -1):
        s = s * u2 + 12.0 * (-1) ** j * (2 * j - 2) / math.factorial(2 * j)
    far = u.clamp(min=1.0)
    return torch.where(u < 1.5, s, 12.0 / far ** 4 * (2.0 - 2.0 * torch.cos(far) - far * torch.sin(far)))


def _green(n, b, b_prev, order, iso, nmax=2):
    """Eq. 11 on the octant [mz][my][mx]."""
    h = n // 2 + 1
    m = torch.arange(h, device="cuda", dtype=F64)
    k = 2.0 * math.pi * m / n

    def sinm(j):
        v = torch.sin(2.0 * math.pi * (j % n) / n)
        return torch.where((2 * j) % n == 0, torch.zeros_like(v), v)

    d = 4.0 / 3.0 * sinm(m) - sinm(2 * m) / 6.0
    al = [k + 2.0 * math.pi * a for a in range(-nmax, nmax + 1)]
    w2 = [_sinc(0.5 * q) ** (2 * order) for q in al]
    u1 = sum(w2)
    dd = d[:, None, None] ** 2 + d[None, :, None] ** 2 + d[None, None, :] ** 2
    big = torch.zeros((h, h, h), device="cuda", dtype=F64)
    for z in range(2 * nmax + 1):
        for y in range(2 * nmax + 1):
            for x in range(2 * nmax + 1):
                kk = al[z][:, None, None] ** 2 + al[y][None, :, None] ** 2 + al[x][None, None, :] ** 2
                kd = (al[z] * d)[:, None, None] + (al[y] * d)[None, :, None] + (al[x] * d)[None, None, :]
                kd *= w2[z][:, None, None]
                kd *= w2[y][None, :, None]
                kd *= w2[x][None, None, :]
                kd /= kk.clamp(min=1e-300)
                mag = kk.sqrt()
                t = _profile_k(mag, b) ** 2
                if b_prev:
                    t -= _profile_k(mag, b_prev) ** 2
                if iso:
                    t *= 1.0 - _sinc(mag * iso)
                big += torch.where(kk > 0, kd * t, torch.zeros_like(t))
    u = u1[:, None, None] * u1[None, :, None] * u1[None, None, :]
    return torch.where(dd > 0, -4.0 * math.pi * big / (dd.clamp(min=1e-300) * u * u), torch.zeros_like(big))


def _solve(rho, g):
    n = rho.shape[0]
    s = torch.fft.rfftn(rho)
    i = torch.arange(n, device="cuda")
    i = torch.minimum(i, n - i)
    for z in range(n):
        s[z] *= g[i[z]][i]
    return torch.fft.irfftn(s, s=(n, n, n))


def _diff(phi, axis):
    """D of eq. 7 along axis (0 = x): the 4-point difference."""
    a = 2 - axis
    return (2.0 / 3.0 * (torch.roll(phi, -1, a) - torch.roll(phi, 1, a))
            - (torch.roll(phi, -2, a) - torch.roll(phi, 2, a)) / 12.0)


def _weights(y, tsc):
    """First node, weights and slopes per axis of level coordinates y (truncated to 2^-15)."""
    lo = torch.floor(y)
    f = torch.floor((y - lo) * 32768.0) / 32768.0
    if not tsc:
        one = torch.ones_like(f)
        return lo.long(), [1.0 - f, f], [-one, one]
    up = f >= 0.5
    d = torch.where(up, f - 1.0, f)
    m = d * 32768.0
    w0 = torch.floor(((16384.0 - m) ** 2 + 16384.0) / 32768.0) / 65536.0
    w2 = torch.floor(((16384.0 + m) ** 2 + 16384.0) / 32768.0) / 65536.0
    return (lo + up).long() - 1, [w0, 1.0 - w0 - w2, w2], [d - 0.5, -2.0 * d, d + 0.5]


STRETCH = 1 << 22


def _nodes(x, h, n, tsc):
    """(slice, node index, weight, its three slopes in 1/fine cell) for every node of every stretch."""
    for a in range(0, x.shape[1], STRETCH):
        at = slice(a, min(a + STRETCH, x.shape[1]))
        lo, w, s = _weights(x[:, at] / h, tsc)
        k = len(w)
        for z in range(k):
            for y in range(k):
                for q in range(k):
                    i = (torch.remainder(lo[2] + z, n) * n + torch.remainder(lo[1] + y, n)) * n + torch.remainder(lo[0] + q, n)
                    wx, wy, wz = w[q][0], w[y][1], w[z][2]
                    yield at, i, wx * wy * wz, (s[q][0] * wy * wz / h, wx * s[y][1] * wz / h, wx * wy * s[z][2] / h)


def _deposit(x, h, n, tsc, value=None):
    rho = torch.zeros(n ** 3, device="cuda", dtype=F64)
    for at, i, w, _ in _nodes(x, h, n, tsc):
        rho.index_add_(0, i, w if value is None else w * value[at])
    return rho.view(n, n, n)


def _level(x, case, level, n_fine, out, bar=None):
    """Adds one level's mesh force of positions x, or its adjoint for the cotangents bar, to out."""
    two, tsc = bool(case["ratio"]), case["tsc"]
    h = case["ratio"] if level else 1
    n = n_fine // h
    b, prev = (B_COARSE / h, 0.0) if level else (case["b_fine"], B_COARSE if two else 0.0)
    iso = n / 2 if case["isolated"] and not prev else 0.0
    g = _green(n, b, prev, 3 if tsc else 2, iso)
    phi = _solve(_deposit(x, h, n, tsc), g)
    c = 1.0 / (h * h)
    field = [-_diff(phi, d).reshape(-1) * c for d in range(3)]
    if bar is None:
        for at, i, w, _ in _nodes(x, h, n, tsc):
            for d in range(3):
                out[d, at] += w * field[d][i]
        return
    pb = torch.zeros((n, n, n), device="cuda", dtype=F64)
    for d in range(3):
        pb += _diff(_deposit(x, h, n, tsc, bar[d] * c), d)
    rb = _solve(pb, g).reshape(-1)
    for at, i, _, s in _nodes(x, h, n, tsc):
        v = rb[i]
        for d in range(3):
            v = v + bar[d, at] * field[d][i]
        for d in range(3):
            out[d, at] += s[d] * v


def _r_over_r(r, b):
    """R(r, b) / r of eq. 2 and its derivative."""
    t = r / b

    def poly(c):
        p, q = torch.zeros_like(t), torch.zeros_like(t)
        for k in reversed(range(len(c))):
            q = q * t + p
            p = p * t + c[k]
        return p, q

    p1, q1 = poly([64 / 5, 0.0, -256 / 5, 32.0, 1536 / 35, -192 / 5])
    p2, q2 = poly([256 / 5, -96.0, 256 / 5, 32.0, -1536 / 35, 64 / 5])
    p2, q2 = p2 + 3 / 35 / t ** 3 - 32 / 5 / t, q2 - 9 / 35 / t ** 4 + 32 / 5 / t ** 2
    p = torch.where(t < 0.5, p1, torch.where(t < 1.0, p2, t ** -3))
    q = torch.where(t < 0.5, q1, torch.where(t < 1.0, q2, -3.0 * t ** -4))
    return p / b ** 3, q / b ** 4


def _pair_law(r, case):
    """g = [R(r, b_pp) - R(r, b_fine)] / r and dg/dr."""
    bf, bp = case["b_fine"], case["b_pp"]
    p, dp = _r_over_r(r, bp)
    f, df = _r_over_r(r, bf)
    q = 1.0 - r / bf
    c = (1344 / 35, -2912 / 35, 2048 / 35, -64 / 5)
    pol = c[0] + q * (c[1] + q * (c[2] + q * c[3]))
    dpol = c[1] + q * (2 * c[2] + 3 * q * c[3])
    g = q ** 5 * pol / r ** 3
    dg = -(5 * q ** 4 * pol + q ** 5 * dpol) / (bf * r ** 3) - 3.0 * g / r
    tail = (r >= bp) & (2 * r >= bf)
    return torch.where(tail, g, p - f), torch.where(tail, dg, dp - df)


def _pairs(x, case, n_fine, out, bar=None):
    """Adds the pair sum of positions x (or its adjoint) to out."""
    n = x.shape[1]
    side = n_fine // 2
    c = (x / 2.0).long()
    key = (c[2] * side + c[1]) * side + c[0]
    order = torch.argsort(key)
    first = torch.zeros(side ** 3 + 1, device="cuda", dtype=torch.long)
    first[1:] = torch.cumsum(torch.bincount(key, minlength=side ** 3), 0)
    xs = x[:, order].contiguous()
    bs = bar[:, order].contiguous() if bar is not None else None
    cc = c[:, order]
    del c, key
    total = torch.zeros_like(xs)
    reach = 1 if case["b_fine"] <= 2.0 else 2
    span = range(-reach, reach + 1)
    most = 1 << 25
    for oz in span:
        for oy in span:
            for ox in span:
                nb = ((torch.remainder(cc[2] + oz, side) * side + torch.remainder(cc[1] + oy, side)) * side
                      + torch.remainder(cc[0] + ox, side))
                start = first[nb]
                count = first[nb + 1] - start
                ends = torch.cumsum(count, 0)
                all_pairs = int(ends[-1])
                bounds = torch.searchsorted(ends, torch.arange(1, all_pairs // most + 1, device="cuda") * most)
                cuts = [0] + bounds.tolist() + [n]
                for a, b in zip(cuts, cuts[1:]):
                    if b <= a:
                        continue
                    cnt = count[a:b]
                    i = torch.repeat_interleave(torch.arange(a, b, device="cuda"), cnt)
                    if not i.numel():
                        continue
                    base = int(ends[a] - count[a])
                    j = torch.arange(i.numel(), device="cuda") + base - (ends[i] - count[i]) + start[i]
                    d = [xs[k, j] - xs[k, i] for k in range(3)]
                    d = [v - n_fine * torch.round(v / n_fine) for v in d]
                    r2 = d[0] * d[0] + d[1] * d[1] + d[2] * d[2]
                    keep = torch.nonzero((r2 > 0) & (r2 < case["b_fine"] ** 2)).flatten()
                    i, j, r = i[keep], j[keep], r2[keep].sqrt()
                    d = [v[keep] for v in d]
                    g, dg = _pair_law(r, case)
                    if bar is None:
                        v = [g * d[k] for k in range(3)]
                    else:
                        u = [bs[k, j] - bs[k, i] for k in range(3)]
                        du = (d[0] * u[0] + d[1] * u[1] + d[2] * u[2]) * dg / r
                        v = [g * u[k] + du * d[k] for k in range(3)]
                    for k in range(3):
                        total[k].index_add_(0, i, v[k])
    out[:, order] += total


def _ordered(case, seed):
    """Quantised fine-cell positions of the sorted particles, and the order."""
    nf = case["n_fine"]
    q = torch.floor(_positions(case, seed).double() * (nf * 32768)).long()
    order = torch.argsort(_key(q, nf), stable=True)
    return q[:, order], order


def _key(q, nf):
    c = q >> 16
    t, u = c >> 3, c & 7
    nt = nf // 16
    return ((t[2] * nt + t[1]) * nt + t[0]) * 512 + (u[2] * 8 + u[1]) * 8 + u[0]


def exact(case, seed):
    op, nf = case["op"], case["n_fine"]
    if op == "pack":
        return None
    if nf > 512:
        return None
    q, _ = _ordered(case, seed)
    n = q.shape[1]
    if op == "kick":
        v = _random(case, seed, 2 * n).double()
        v, a = v[:, :n], v[:, n:]
        v = v + KICK * a
        drift = case["move"] / math.sqrt(3.0 * (1.0 + KICK * KICK))
        q = torch.remainder(q + torch.round(drift * v.float().double() * 32768.0).long(), nf * 32768)
        return [None, None, v[:, torch.argsort(_key(q, nf), stable=True)], None]
    if op == "velocity":
        v = _random(case, seed, n).double()
        h = case["ratio"] or 4
        nb = nf // h
        c = (q >> 15) // h
        cell = (c[2] * nb + c[1]) * nb + c[0]
        cnt = torch.bincount(cell, minlength=nb ** 3).clamp(min=1).double()
        bulk = torch.stack([torch.zeros(nb ** 3, device="cuda", dtype=F64).index_add_(0, cell, v[d]) / cnt
                            for d in range(3)])
        dev = v - bulk[:, cell]
        step = dev.abs().max() / 32767.0
        back = bulk[:, cell] + step * torch.round(dev / step)
        return (None, bulk.view(3, nb, nb, nb), step.reshape(1)), back
    x = q.double() / 32768.0
    out = torch.zeros((3, n), device="cuda", dtype=F64)
    if op == "tiles":
        return _tiled(x, case, out)
    bar = _random(case, seed, n).double() if op == "backward" else None
    for level in range(2 if case["ratio"] else 1):
        _level(x, case, level, nf, out, bar)
    _pairs(x, case, nf, out, bar)
    return out


def _tiled(x, case, out):
    """The coarse level on the whole box; the fine level on each tile's box; all pairs."""
    nf, tile, buf = case["n_fine"], case["tile"], case["buffer"]
    _level(x, case, 1, nf, out)
    _pairs(x, case, nf, out)
    side = tile + 2 * buf
    for z in range(0, nf, tile):
        for y in range(0, nf, tile):
            for q in range(0, nf, tile):
                org = torch.tensor([[q - buf], [y - buf], [z - buf]], device="cuda", dtype=F64)
                local = torch.remainder(x - org, nf)
                idx = torch.nonzero((local < side).all(0)).flatten()
                if not idx.numel():
                    continue
                loc = local[:, idx]
                f = torch.zeros_like(loc)
                _level(loc, case, 0, side, f)
                own = torch.nonzero(((loc >= buf) & (loc < buf + tile)).all(0)).flatten()
                out[:, idx[own]] += f[:, own]
    return out
