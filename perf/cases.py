"""Performance cases of the Ahmad-Cohen block step: what a direct N-body program
has the library do, from the one-body block to the full block of a million
bodies, each through the package's public entry points.

Inputs are Plummer spheres with Kroupa masses (optionally 5% of the bodies in
tight binaries), drawn on the GPU from the seed alone, with neighbour radii
that hold about 64 bodies.  Outputs of the force calls go to the caller's
tensors, as in a stepping loop.  ``exact`` is plain torch in float64.
"""
import math
import random

import torch

import paper_1504_03687_amd as nb

PLUMMER_B = 3.0 * math.pi / 16.0     # scale length of a Plummer sphere in N-body units
NEIGHBOURS = 64                      # the neighbour number that the radii aim at
FLOPS_FORCE = 40                     # per pair: force and jerk
FLOPS_ADJOINT = 110                  # per pair: both sides' gradients, shared geometry once
FLOPS_POTENTIAL = 11                 # per pair
EXACT_PAIRS = 3.0e10                 # pairs that the float64 reference can do in a few seconds


def listed():
    return [
        # the deepest step levels: one body due, then a few (latency, launches, one j-set read)
        {"name": "one_row_n1m", "kind": "force", "n": 1 << 20, "rows": 1, "precision": "fp64",
         "cap": 1024, "binaries": True},
        {"name": "rows32_n131072", "kind": "force", "n": 131072, "rows": 32, "precision": "mixed",
         "cap": 512, "binaries": False},
        # a small cluster, every body due on a shared step
        {"name": "cluster_n1024", "kind": "force", "n": 1024, "rows": 1024, "precision": "fp64",
         "cap": 256, "binaries": False},
        # ordinary blocks of a mid-size cluster, even and ragged
        {"name": "rows1024_n131072", "kind": "force", "n": 131072, "rows": 1024,
         "precision": "mixed", "cap": 512, "binaries": False},
        {"name": "rows16001_n100003", "kind": "force", "n": 100003, "rows": 16001,
         "precision": "fp64", "cap": 256, "binaries": False},
        # the most frequent block of the million-body cluster's step levels
        {"name": "rows1272_n1m", "kind": "force", "n": 1 << 20, "rows": 1272,
         "precision": "mixed", "cap": 1024, "binaries": True},
        # the full block of the million-body cluster
        {"name": "full_n1m", "kind": "force", "n": 1 << 20, "rows": 1 << 20, "precision": "mixed",
         "cap": 160, "binaries": True},
        # a whole block step: predict, regular and irregular force, correct, next radii
        {"name": "step4099_n131072", "kind": "step", "n": 131072, "rows": 4099,
         "precision": "mixed", "cap": 256, "binaries": True},
        # an ensemble of uneven clusters in one call
        {"name": "ensemble96", "kind": "ensemble", "clusters": 96, "n_lo": 1024, "n_hi": 32768,
         "precision": "mixed", "cap": 256},
        # differentiable step: forward and backward through the autograd function
        {"name": "grad_n20011", "kind": "grad", "n": 20011, "rows": 20011, "precision": "fp64"},
        # energy check of a run
        {"name": "potential_n131072", "kind": "potential", "n": 131072},
        # step scheduler: full sort by step level, then the re-sort after a block
        {"name": "sched_n1m", "kind": "sched", "n": 1 << 20, "level": 10, "k_max": 20},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["force", "force", "force", "force", "step", "ensemble", "grad", "potential",
                       "sched"])
    if kind in ("force", "step"):
        n = _log_int(rng, 1024, 1 << 20)
        rows = _log_int(rng, 1, n if kind == "force" else max(1, n // 8))
        return {"kind": kind, "n": n, "rows": rows,
                "precision": rng.choice(["mixed", "fp64"]) if rows < 600000 else "mixed",
                "cap": rng.choice([128, 200, 256]), "binaries": rng.random() < 0.5}
    if kind == "ensemble":
        return {"kind": kind, "clusters": _log_int(rng, 4, 160),
                "n_lo": _log_int(rng, 600, 3000), "n_hi": _log_int(rng, 4000, 32768),
                "precision": rng.choice(["mixed", "fp64"]), "cap": rng.choice([128, 256])}
    if kind == "grad":
        n = _log_int(rng, 1024, 65536)
        return {"kind": kind, "n": n, "rows": _log_int(rng, max(1, n // 64), n),
                "precision": rng.choice(["mixed", "fp64"])}
    if kind == "potential":
        return {"kind": kind, "n": _log_int(rng, 1024, 1 << 18)}
    return {"kind": kind, "n": _log_int(rng, 1024, 1 << 20), "level": rng.randint(4, 14),
            "k_max": 20}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _uniform(g, *shape):
    return torch.rand(shape, generator=g, dtype=torch.float64, device="cuda")


def _isotropic(g, n):
    z = 2.0 * _uniform(g, n) - 1.0
    f = 2.0 * math.pi * _uniform(g, n)
    s = torch.sqrt((1.0 - z * z).clamp_min(0.0))
    return torch.stack((s * torch.cos(f), s * torch.sin(f), z))


def _kroupa(g, n):
    """Two-segment power law, m^-1.3 on [0.08, 0.5) and m^-2.3 on [0.5, 100]."""
    def integral(a, lo, hi):
        return (hi ** (1 - a) - lo ** (1 - a)) / (1 - a)

    def inverse(a, lo, hi, u):
        e = 1 - a
        return (lo ** e + u * (hi ** e - lo ** e)) ** (1 / e)

    w1, w2 = integral(1.3, 0.08, 0.5), 0.5 * integral(2.3, 0.5, 100.0)
    seg, u = _uniform(g, n), _uniform(g, n)
    return torch.where(seg < w1 / (w1 + w2), inverse(1.3, 0.08, 0.5, u),
                       inverse(2.3, 0.5, 100.0, u))


_SPEED = {}


def _speed_fraction(g, n):
    """Speed over escape speed, density q^2 (1 - q^2)^(7/2), by its tabulated
    cumulative distribution."""
    if "table" not in _SPEED:
        q = torch.linspace(0.0, 1.0, 4097, dtype=torch.float64, device="cuda")
        c = torch.cumsum(q * q * (1.0 - q * q).clamp_min(0.0) ** 3.5, 0)
        _SPEED["table"] = (q, c / c[-1])
    q, c = _SPEED["table"]
    u = _uniform(g, n)
    k = torch.searchsorted(c, u).clamp(1, 4096)
    t = (u - c[k - 1]) / (c[k] - c[k - 1]).clamp_min(1e-300)
    return q[k - 1] + t.clamp(0.0, 1.0) * (q[k] - q[k - 1])


def _cluster(g, n, binaries=False):
    """x, v (3, n), m (n) of a Plummer sphere and the squared neighbour radii
    (n): the sphere that holds NEIGHBOURS bodies at the local density."""
    X = 0.999 * _uniform(g, n).clamp_min(1e-12)
    r = 1.0 / torch.sqrt(X ** (-2.0 / 3.0) - 1.0)
    x = PLUMMER_B * r * _isotropic(g, n)
    v = (_speed_fraction(g, n) * math.sqrt(2.0) * (1.0 + r * r) ** -0.25 *
         _isotropic(g, n)) / math.sqrt(PLUMMER_B)
    m = _kroupa(g, n)
    m = m / m.sum()
    if binaries:
        # pairs (2k, 2k+1) of 5% of the bodies: a circular orbit around the first one's place
        k = n // 40
        a = 1e-5 * 100.0 ** _uniform(g, k)
        d = _isotropic(g, k)
        e = _isotropic(g, k)
        e = e - (e * d).sum(0) * d
        e = e / e.square().sum(0).sqrt()
        mb = m[0:2 * k:2] + m[1:2 * k:2]
        rel_x, rel_v = a * d, torch.sqrt(mb / a) * e
        f = m[1:2 * k:2] / mb
        cx, cv = x[:, 0:2 * k:2].clone(), v[:, 0:2 * k:2].clone()
        x[:, 0:2 * k:2] = cx + f * rel_x
        x[:, 1:2 * k:2] = cx - (1.0 - f) * rel_x
        v[:, 0:2 * k:2] = cv + f * rel_v
        v[:, 1:2 * k:2] = cv - (1.0 - f) * rel_v
    r = x.square().sum(0).sqrt() / PLUMMER_B
    rs = PLUMMER_B * (NEIGHBOURS / n) ** (1.0 / 3.0) * (1.0 + r * r) ** (5.0 / 6.0)
    rs = torch.minimum(rs, 0.5 * PLUMMER_B * (1.0 + r))
    return x.contiguous(), v.contiguous(), m, rs * rs


def _field(x, v):
    """Plummer acceleration and its derivative: stand-ins for the last step's."""
    r2 = x.square().sum(0) + PLUMMER_B ** 2
    r3 = r2 ** 1.5
    return -x / r3, -v / r3 + 3.0 * (x * v).sum(0) * x / (r3 * r2)


def _block(g, n, rows):
    """rows distinct bodies; in random order unless all bodies are due."""
    if rows == n:
        return torch.arange(n, dtype=torch.int32, device="cuda")
    return torch.randperm(n, generator=g, device="cuda")[:rows].to(torch.int32)


def _ensemble_sizes(case):
    """(bodies, rows) of each cluster: log-uniform sizes, 1% to all bodies due; the sizes are
    the ensemble's own, the bodies come from the seed."""
    r = random.Random(case["clusters"] * 1000003 + case["n_lo"] * 101 + case["n_hi"])
    for _ in range(case["clusters"]):
        n = _log_int(r, case["n_lo"], case["n_hi"])
        yield n, max(1, round(r.uniform(0.01, 1.0) * n))


def _outputs(rows, cap):
    f = dict(dtype=torch.float64, device="cuda")
    i = dict(dtype=torch.int32, device="cuda")
    return (torch.zeros((3, rows), **f), torch.zeros((3, rows), **f), torch.zeros(rows, **i),
            torch.zeros((rows, cap), **i), torch.zeros(1, **i))


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1504036870 + 7919 * int(seed))
    s = {"kind": case["kind"], "precision": case.get("precision")}
    kind = case["kind"]
    if kind == "ensemble":
        parts, j_off, i_off = [], [0], [0]
        for n, rows in _ensemble_sizes(case):
            x, v, m, rs2 = _cluster(g, n)
            ib = torch.randperm(n, generator=g, device="cuda")[:rows]
            parts.append((x, v, m, rs2[ib], (ib + j_off[-1]).to(torch.int32)))
            j_off.append(j_off[-1] + n)
            i_off.append(i_off[-1] + rows)
        s.update(j_off=j_off, i_off=i_off, cap=case["cap"],
                 x=torch.cat([p[0] for p in parts], 1).contiguous(),
                 v=torch.cat([p[1] for p in parts], 1).contiguous(),
                 m=torch.cat([p[2] for p in parts]), rs2=torch.cat([p[3] for p in parts]),
                 ib=torch.cat([p[4] for p in parts]), out=_outputs(i_off[-1], case["cap"]))
        return s
    n = case["n"]
    if kind == "sched":
        # a bulk of step levels around 2^-6 and a tail of close pairs down to the finest
        k = torch.round(6.0 + 1.5 * torch.randn(n, generator=g, dtype=torch.float64,
                                                device="cuda"))
        deep = _uniform(g, n) < 0.05
        k = torch.where(deep, torch.floor(7.0 + 14.0 * _uniform(g, n)), k)
        level = k.clamp(3, case["k_max"]).to(torch.int32)
        # after the block of this level: most steps kept, some one coarser or up to three finer
        L = case["level"]
        u = _uniform(g, n)
        d = torch.where(u < 0.7, 0.0, torch.where(u < 0.85, -1.0,
                                                  1.0 + torch.floor(3.0 * _uniform(g, n))))
        new = torch.where(level >= L, (level + d).clamp(L, case["k_max"]), level.double())
        s.update(level=level, new=new.to(torch.int32), L=L, k_max=case["k_max"],
                 due=int((level >= L).sum()))
        return s
    x, v, m, rs2 = _cluster(g, n, case.get("binaries", False))
    s.update(x=x, v=v, m=m)
    if kind == "potential":
        return s
    rows = case["rows"]
    ib = _block(g, n, rows)
    s.update(ib=ib, rs2=rs2[ib.long()].contiguous())
    if kind == "force":
        s.update(cap=case["cap"], out=_outputs(rows, case["cap"]))
    elif kind == "grad":
        s["w_a"] = torch.randn((3, rows), generator=g, dtype=torch.float64, device="cuda")
        s["w_j"] = torch.randn((3, rows), generator=g, dtype=torch.float64, device="cuda")
        for k in ("x", "v", "m"):
            s[k].requires_grad_()
    else:
        a, jk = _field(x, v)
        h = 2.0 ** -torch.floor(6.0 + 4.0 * _uniform(g, n))
        s.update(a=a, jk=jk, t=2.0 ** -4, t0=2.0 ** -4 - h, h=h, cap=case["cap"],
                 last=torch.cat((x, v, a, jk)), xp=torch.empty_like(x), vp=torch.empty_like(v),
                 out=_outputs(rows, case["cap"]))
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    kind = s["kind"]
    if kind == "force":
        return nb.regular_force(s["x"], s["v"], s["m"], s["ib"], s["rs2"], s["cap"],
                                s["precision"], out=s["out"])
    if kind == "step":
        nb.predict(s["x"], s["v"], s["a"], s["jk"], s["t0"], s["t"], out=(s["xp"], s["vp"]))
        acc, jerk, cnt, lst, ovf = nb.regular_force(s["xp"], s["vp"], s["m"], s["ib"], s["rs2"],
                                                    s["cap"], s["precision"], out=s["out"])
        ia, ij = nb.irregular_force(s["xp"], s["vp"], s["m"], s["ib"], s["cap"], cnt, lst)
        ib = s["ib"].long()
        b = s["last"].index_select(1, ib)
        x1, v1, a2, a3 = nb.hermite_correct(s["h"][ib], b[0:3], b[3:6], b[6:9], b[9:12],
                                            acc + ia, jerk + ij)
        rs2 = nb.radius_update(cnt, s["rs2"], NEIGHBOURS)
        return s["xp"], s["vp"], acc, jerk, cnt, lst, ovf, ia, ij, x1, v1, a2, a3, rs2
    if kind == "ensemble":
        return nb.regular_force_batched(s["j_off"], s["i_off"], s["x"], s["v"], s["m"], s["ib"],
                                        s["rs2"], s["cap"], s["precision"], out=s["out"])
    if kind == "grad":
        # no lists wanted here (capacity 0): the force, the counts and the gradients
        acc, jerk, cnt, _, _ = nb.RegularForce.apply(s["x"], s["v"], s["m"], s["ib"], s["rs2"], 0,
                                                     s["precision"])
        gx, gv, gm = torch.autograd.grad((acc, jerk), (s["x"], s["v"], s["m"]),
                                         (s["w_a"], s["w_j"]))
        return acc.detach(), jerk.detach(), cnt, gx, gv, gm
    if kind == "potential":
        return nb.potential(s["x"], s["m"])
    order, level_end = nb.sched_build(s["level"], s["k_max"])
    nb.sched_update(order, level_end, s["due"], s["L"], s["new"], s["k_max"])
    return order, level_end


def work(case):
    kind = case["kind"]
    if kind == "ensemble":
        sizes = list(_ensemble_sizes(case))
        return {"bytes": sum(56.0 * n + rows * (64.0 + 4.0 * NEIGHBOURS) for n, rows in sizes),
                "flops": float(FLOPS_FORCE * sum(n * rows for n, rows in sizes))}
    n = float(case["n"])
    if kind == "potential":
        return {"bytes": 40.0 * n, "flops": FLOPS_POTENTIAL * n * n}
    if kind == "sched":
        # list and levels read and written once for the sort, once more for the due share
        return {"bytes": 12.0 * n, "flops": 4.0 * n}
    rows = float(case["rows"])
    force = {"bytes": 56.0 * n + rows * (64.0 + 4.0 * NEIGHBOURS),
             "flops": FLOPS_FORCE * n * rows}
    if kind == "grad":
        return {"bytes": force["bytes"] + 112.0 * n + 96.0 * rows,
                "flops": (FLOPS_FORCE + FLOPS_ADJOINT) * n * rows}
    if kind == "step":
        return {"bytes": force["bytes"] + 152.0 * n + rows * (60.0 * NEIGHBOURS + 248.0 + 168.0),
                "flops": force["flops"] + rows * (FLOPS_FORCE * NEIGHBOURS + 120.0)}
    return force


# ---------------------------------------------------------------------------
# float64 reference (torch alone)
# ---------------------------------------------------------------------------
def _neighbours(dx, rs2, self_pair):
    """The library's neighbour rule: float32 of the float64 differences, squares
    summed with single roundings as by fused multiply-adds."""
    f = [d.float().double() for d in dx]
    r2 = (f[0] * f[0]).float().double()
    r2 = (f[1] * f[1] + r2).float().double()
    r2 = (f[2] * f[2] + r2).float()
    return (r2 < rs2.float()[:, None]) & ~self_pair


def _force_chunks(x, v, ib, first, last, budget=4.0e7):
    """Row chunks (b0, b1, dx, du, self pair) of the pairs with bodies [first, last)."""
    step = max(1, int(budget / max(1, last - first)))
    j = torch.arange(first, last, device=x.device)
    for b0 in range(0, ib.numel(), step):
        i = ib[b0:b0 + step].long()
        yield (b0, b0 + i.numel(), [x[k, first:last][None, :] - x[k, i][:, None] for k in range(3)],
               [v[k, first:last][None, :] - v[k, i][:, None] for k in range(3)],
               j[None, :] == i[:, None])


def _pair_sums(w3, w5, dx, du, su):
    acc = torch.stack([(w3 * dx[k]).sum(1) for k in range(3)])
    jerk = torch.stack([(w3 * du[k] - 3.0 * w5 * su * dx[k]).sum(1) for k in range(3)])
    return acc, jerk


def _exact_force(x, v, m, ib, rs2, first=0, last=None, irregular=False):
    """acc, jerk, count (and the neighbours' acc, jerk) of the rows ib."""
    last = x.shape[1] if last is None else last
    rows = ib.numel()
    out = [torch.empty((3, rows), dtype=torch.float64, device=x.device) for _ in range(4)]
    cnt = torch.empty(rows, dtype=torch.int32, device=x.device)
    for b0, b1, dx, du, me in _force_chunks(x, v, ib, first, last):
        nbr = _neighbours(dx, rs2[b0:b1], me)
        r2 = dx[0] * dx[0] + dx[1] * dx[1] + dx[2] * dx[2]
        r2 = torch.where(me, torch.ones_like(r2), r2)
        w3 = torch.where(me, 0.0, m[None, first:last] / (r2 * r2.sqrt()))
        su = dx[0] * du[0] + dx[1] * du[1] + dx[2] * du[2]
        reg = torch.where(nbr, 0.0, w3)
        out[0][:, b0:b1], out[1][:, b0:b1] = _pair_sums(reg, reg / r2, dx, du, su)
        if irregular:
            w3 = torch.where(nbr, w3, 0.0)
            out[2][:, b0:b1], out[3][:, b0:b1] = _pair_sums(w3, w3 / r2, dx, du, su)
        cnt[b0:b1] = nbr.sum(1).to(torch.int32)
    return out, cnt


def exact(case, seed):
    kind = case["kind"]
    if kind == "sched" or work(case)["flops"] > FLOPS_FORCE * EXACT_PAIRS:
        return None
    s = prepare(case, seed)
    if kind == "force":
        (acc, jerk, _, _), cnt = _exact_force(s["x"], s["v"], s["m"], s["ib"], s["rs2"])
        return acc, jerk, cnt, None, None
    if kind == "ensemble":
        acc, jerk, cnt = [], [], []
        for c in range(len(s["j_off"]) - 1):
            i0, i1 = s["i_off"][c], s["i_off"][c + 1]
            out, k = _exact_force(s["x"], s["v"], s["m"], s["ib"][i0:i1], s["rs2"][i0:i1],
                                  s["j_off"][c], s["j_off"][c + 1])
            acc.append(out[0])
            jerk.append(out[1])
            cnt.append(k)
        return torch.cat(acc, 1), torch.cat(jerk, 1), torch.cat(cnt), None, None
    if kind == "step":
        dt = s["t"] - s["t0"]
        xp = s["x"] + dt * (s["v"] + dt * (s["a"] / 2 + dt * (s["jk"] / 6)))
        vp = s["v"] + dt * (s["a"] + dt * (s["jk"] / 2))
        (acc, jerk, ia, ij), cnt = _exact_force(xp, vp, s["m"], s["ib"], s["rs2"], irregular=True)
        ib = s["ib"].long()
        h = s["h"][ib]
        x0, v0, a0, j0 = s["last"][:, ib].reshape(4, 3, -1)
        a1, j1 = acc + ia, jerk + ij
        v1 = v0 + h / 2 * (a0 + a1) + h * h / 12 * (j0 - j1)
        x1 = x0 + h / 2 * (v0 + v1) + h * h / 12 * (a0 - a1)
        a3 = (12 * (a0 - a1) + 6 * h * (j0 + j1)) / h ** 3
        a2 = (-6 * (a0 - a1) - h * (4 * j0 + 2 * j1)) / h ** 2 + h * a3
        f = (NEIGHBOURS / cnt.clamp_min(1).double()) ** (2.0 / 3.0)
        return (xp, vp, acc, jerk, cnt, None, None, ia, ij, x1, v1, a2, a3,
                s["rs2"] * f.clamp(0.5, 2.0))
    if kind == "grad":
        x, v, m = (s[k].detach() for k in ("x", "v", "m"))
        (acc, jerk, _, _), cnt = _exact_force(x, v, m, s["ib"], s["rs2"])
        gx, gv, gm = torch.zeros_like(x), torch.zeros_like(v), torch.zeros_like(m)
        for b0, b1, dx, du, me in _force_chunks(x, v, s["ib"], 0, x.shape[1], 2.0e7):
            drop = _neighbours(dx, s["rs2"][b0:b1], me) | me
            A = [s["w_a"][k, b0:b1][:, None] for k in range(3)]
            B = [s["w_j"][k, b0:b1][:, None] for k in range(3)]
            r2 = dx[0] * dx[0] + dx[1] * dx[1] + dx[2] * dx[2]
            r2 = torch.where(drop, torch.ones_like(r2), r2)
            r3 = torch.where(drop, 0.0, 1.0 / (r2 * r2.sqrt()))
            r5 = r3 / r2
            su = dx[0] * du[0] + dx[1] * du[1] + dx[2] * du[2]
            ab = sum(A[k] * dx[k] + B[k] * du[k] for k in range(3))
            br = sum(B[k] * dx[k] for k in range(3))
            gm += (ab * r3 - 3.0 * su * br * r5).sum(0)
            i = s["ib"][b0:b1].long()
            c = 15.0 * su * br * r5 / r2 - 3.0 * r5 * ab
            for k in range(3):
                t = m * (A[k] * r3 - 3.0 * r5 * (su * B[k] + br * du[k]) + c * dx[k])
                gx[k] += t.sum(0)
                gx[k].index_add_(0, i, -t.sum(1))
                t = m * (B[k] * r3 - 3.0 * br * r5 * dx[k])
                gv[k] += t.sum(0)
                gv[k].index_add_(0, i, -t.sum(1))
        return acc, jerk, cnt, gx, gv, gm
    phi = torch.empty_like(s["m"])
    ib = torch.arange(case["n"], device="cuda")
    for b0, b1, dx, _, me in _force_chunks(s["x"], s["x"], ib, 0, case["n"]):
        r2 = dx[0] * dx[0] + dx[1] * dx[1] + dx[2] * dx[2]
        phi[b0:b1] = -torch.where(me, 0.0, s["m"] / torch.where(me, 1.0, r2).sqrt()).sum(1)
    return phi, 0.5 * (s["m"] * phi).sum().reshape(1)
