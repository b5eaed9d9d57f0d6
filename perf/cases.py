"""The work that programs have this framework do, as cases whose time is measured.

Every case goes through the public entry points, with the positions and forces of the
workloads (perturbed cubic lattices in a cube or a spherical drop, straight bead chains in
a dilute cloud) and the seeded stand-in networks. The families:

  step      one full step of a simulation: tree, partition, ACA and product (hmatvec);
  product   products on one configuration's kept factors, as an iterative solver or a
            serving loop takes them (H @ F, or the product that allocates nothing);
  grad      one training step: forward and backward through autograd (dX, dF, dtheta);
  batch     many small systems in one handle, replayed from its graph;
  filaments one time step of a filament suspension with the short-range terms;
  rotation  one full step of the 6N product with torques.
"""
import math

import numpy as np
import torch

import paper_2505_08174_amd as hh

BUDGET = 64 << 30   # device memory for ACA factors; above half of it the product streams them
TYPES = {"fp64": (torch.float64, torch.float64), "fp32": (torch.float32, torch.float32),
         "bf16": (torch.float32, torch.float64), "bf16_split": (torch.float32, torch.float64)}


def _case(name, family, n, kernel, prec, geom="cube", phi=0.15, forces="normal", c_leaf=128,
          eps=1e-4, eta=1.0, inp="direction", systems=1, noalloc=False):
    return {"name": name, "family": family, "n": n, "kernel": kernel, "prec": prec, "geom": geom,
            "phi": phi, "forces": forces, "c_leaf": c_leaf, "eps": eps, "eta": eta, "inp": inp,
            "systems": systems, "noalloc": noalloc}


def listed():
    return [
        # the smallest calls: a product of a serving loop on a small system (latency)
        _case("serve_mlp_bf16_500", "product", 500, "mlp", "bf16", phi=0.1, noalloc=True),
        # a full step of the small FP64 validation suspension
        _case("step_rpy_fp64_2k", "step", 2000, "rpy", "fp64", phi=0.1, c_leaf=64, eps=1e-6),
        # a full step of a small suspension in the plain FP32 form, odd size
        _case("step_mlp_fp32_5k", "step", 5003, "mlp", "fp32"),
        # an ordinary step: medium suspension, BF16 with hi + lo near field
        _case("step_mlp_split_30k", "step", 30001, "mlp", "bf16_split", phi=0.2),
        # the plain FP32 workload at its full size, factors stored
        _case("step_mlp_fp32_100k", "step", 100000, "mlp", "fp32", phi=0.2),
        # a sedimenting drop in the BF16 form, streamed factors: the largest step here
        _case("step_mlp_bf16_250k", "step", 250000, "mlp", "bf16", geom="drop", phi=0.1,
              forces="gravity"),
        # products of an iterative solver on kept factors (far field and near field re-applied)
        _case("solver_rpy_fp32_60k", "product", 60000, "rpy", "fp32", phi=0.2),
        # a training step on a small suspension, all three gradients
        _case("grad_mlp_fp32_2k", "grad", 2011, "mlp", "fp32", c_leaf=64),
        # a training step on a larger one
        _case("grad_mlp_fp32_16k", "grad", 16000, "mlp", "fp32"),
        # many small systems of ragged sizes in one graph
        _case("batch_mlp_bf16_24sys", "batch", 48000, "mlp", "bf16", systems=24),
        # a time step of filaments and free particles with the short-range terms
        _case("filaments_bf16_21k", "filaments", 21504, "mlp", "bf16", geom="chains",
              forces="gravity", eps=0.02),
        # the 6N product with torques
        _case("rotation_fp32_40k", "rotation", 40000, "rpy6", "fp32", phi=0.2, forces="normal",
              c_leaf=64, eps=1e-5),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["step", "step", "product", "grad", "batch", "filaments", "rotation"])
    geom = rng.choice(["cube", "drop"])
    phi = round(rng.uniform(0.05, 0.25), 3)
    forces = rng.choice(["normal", "gravity"])
    c_leaf = rng.choice([64, 96, 128])
    eta = rng.choice([1.0, 1.0, 0.8])
    if family in ("step", "product"):
        kernel, prec, hi = rng.choice([("rpy", "fp64", 60000), ("rpy", "fp32", 100000),
                                       ("mlp", "fp32", 60000), ("mlp", "bf16", 150000),
                                       ("mlp", "bf16_split", 100000)])
        n = _size(rng, 500, hi)
        noalloc = family == "product" and rng.random() < 0.5
        eps = rng.choice([1e-6, 1e-5, 1e-4]) if prec == "fp64" else rng.choice([1e-3, 1e-4, 1e-4])
        if family == "product":
            n = min(n, 60000)
        return {k: v for k, v in _case("", family, n, kernel, prec, geom, phi, forces, c_leaf, eps,
                                       eta, noalloc=noalloc).items() if k != "name"}
    if family == "grad":
        c = _case("", family, _size(rng, 1000, 16000), "mlp", "fp32", geom, phi, "normal", c_leaf)
    elif family == "batch":
        s = rng.randint(3, 32)
        c = _case("", family, s * _size(rng, 300, 2000), "mlp", rng.choice(["bf16", "bf16_split"]),
                  "cube", phi, "normal", c_leaf, systems=s)
    elif family == "filaments":
        c = _case("", family, 42 * rng.randint(24, 700), "mlp", rng.choice(["bf16", "fp32"]),
                  "chains", 0.0, "gravity", c_leaf, rng.choice([0.02, 1e-2]))
    else:
        c = _case("", family, _size(rng, 1000, 40000), "rpy6", rng.choice(["fp32", "fp32", "fp64"]),
                  geom, phi, "normal", rng.choice([32, 64]), rng.choice([1e-4, 1e-5]))
        if c["prec"] == "fp64":
            c["n"] = min(c["n"], 20000)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs


def _lattice(n, phi, drop, rng):
    """n points of a primitive cubic lattice of volume fraction phi (the nearest to the centre
    for a drop, row by row for a cube), each coordinate jittered; centres stay 2.05 apart."""
    s = (4.0 * math.pi / (3.0 * phi)) ** (1.0 / 3.0)
    jit = max(0.0, min(0.25, (s - 2.05) / (2.0 * math.sqrt(3.0))))
    if drop:
        m = int(math.ceil((3.0 * n / (4.0 * math.pi)) ** (1.0 / 3.0))) + 2
        r = np.arange(-m, m + 1)
        g = np.stack(np.meshgrid(r, r, r, indexing="ij"), -1).reshape(-1, 3)
        g = g[np.argsort((g * g).sum(1), kind="stable")[:n]]
    else:
        m = int(math.ceil(n ** (1.0 / 3.0)))
        i = np.arange(n)
        g = np.stack([i % m, (i // m) % m, i // (m * m)], 1)
    return g * s + rng.uniform(-jit, jit, (n, 3))


def _chains(n, rng, beads=21, bond=3.0, gap=2.1):
    """Straight chains of 21 beads in the inner half of a dilute ball and as many free
    particles in its outer shell; objects that come closer than `gap` are drawn again."""
    nf = n // (2 * beads)
    free = n - nf * beads
    # the density of 5,120 chains and 107,520 free particles in the ball of radius
    # 4 * 10^(1/3) * 20 bonds
    r_out = 4.0 * 10.0 ** (1.0 / 3.0) * (beads - 1) * bond * (nf / 5120.0) ** (1.0 / 3.0)
    r_out = max(r_out, 1.5 * (beads - 1) * bond)
    r_in = 0.5 ** (1.0 / 3.0) * r_out
    off = (np.arange(beads) - 0.5 * (beads - 1)) * bond

    def ball(k, lo, hi):
        d = rng.standard_normal((k, 3))
        d /= np.linalg.norm(d, axis=1)[:, None]
        return d * (lo ** 3 + rng.random((k, 1)) * (hi ** 3 - lo ** 3)) ** (1.0 / 3.0)

    def draw_obj(ids):
        c = ids[ids < nf]
        u = rng.standard_normal((c.size, 3))
        u /= np.linalg.norm(u, axis=1)[:, None]
        mid = ball(c.size, 0.0, max(r_in - 0.5 * (beads - 1) * bond, 0.3 * r_in))
        X[:nf * beads].reshape(nf, beads, 3)[c] = mid[:, None] + off[None, :, None] * u[:, None]
        f = ids[ids >= nf]
        X[nf * beads + f - nf] = ball(f.size, r_in, r_out)

    X = np.empty((n, 3))
    obj = np.concatenate([np.repeat(np.arange(nf), beads), nf + np.arange(free)])
    draw_obj(np.arange(nf + free))
    ob = torch.from_numpy(obj).cuda()
    for _ in range(60):
        Xd = torch.from_numpy(X).cuda()
        bad = []
        for s in range(0, n, 4096):
            d = torch.cdist(Xd[s:s + 4096], Xd, compute_mode="donot_use_mm_for_euclid_dist")
            hit = (d < gap) & (ob[s:s + 4096, None] > ob[None, :])
            bad.append(ob[s:s + 4096][hit.any(1)])
        bad = np.unique(torch.cat(bad).cpu().numpy())
        if bad.size == 0:
            break
        draw_obj(bad)
    return X, nf


def _weights(seed, widths):
    """Glorot-uniform weights and biases U(+-1/sqrt(fan_in)), fixed as a trained net's are."""
    r = np.random.default_rng([seed, 77])
    Ws, bs = [], []
    for i, o in zip(widths[:-1], widths[1:]):
        lim = math.sqrt(6.0 / (i + o))
        Ws.append(r.uniform(-lim, lim, (o, i)))
        bs.append(r.uniform(-1.0, 1.0, o) / math.sqrt(i))
    return Ws, bs


KNET = (1, (3, 64, 64, 64, 9))
SNET = (11, (3, 64, 64, 64, 9))
GNET = (12, (6, 64, 64, 64, 18))


def _inputs(case, seed):
    """Positions, forces (and torques), cotangents, offsets: host FP64 arrays."""
    rng = np.random.default_rng([seed, 5])
    n, off, nf = case["n"], None, 0
    if case["geom"] == "chains":
        X, nf = _chains(n, rng)
    elif case["systems"] > 1:
        # ragged: sizes log-uniform within a factor of five, the same for every seed, summing to n
        w = np.exp(np.random.default_rng([n, 9]).uniform(0, math.log(5.0), case["systems"]))
        size = np.maximum(1, np.floor(w / w.sum() * n).astype(np.int64))
        size[-1] += n - size.sum()
        off = np.concatenate([[0], np.cumsum(size)])
        X = np.concatenate([_lattice(int(m), case["phi"], False, rng) for m in size])
    else:
        X = _lattice(n, case["phi"], case["geom"] == "drop", rng)
    F = rng.standard_normal((n, 6 if case["kernel"] == "rpy6" else 3))
    if case["forces"] == "gravity":
        F *= math.sqrt(0.1)
        F[:, 2] -= 1.0
    return X, F, rng.standard_normal((n, 3)), off, nf


def _kernel(ctx, case):
    if case["kernel"] == "rpy":
        return hh.Kernel.rpy(ctx)
    if case["kernel"] == "rpy6":
        return hh.Kernel.rpy6(ctx)
    return hh.Kernel.mlp(ctx, _weights(*KNET), case["inp"])


def prepare(case, seed):
    X, F, dU, off, nf = _inputs(case, seed)
    tf, tu = TYPES[case["prec"]]
    ctx = hh.Context(0)
    ctx.set_budget(BUDGET)
    s = {"case": case, "ctx": ctx, "X": torch.from_numpy(X).cuda(),
         "F": torch.from_numpy(F).to(tf).cuda()}
    family = case["family"]
    if family == "grad":
        s["theta"] = torch.from_numpy(hh.pack_mlp(_weights(*KNET)))
        s["dU"] = torch.from_numpy(dU).to(tu).cuda()
        for k in ("X", "F", "theta"):
            s[k].requires_grad_(True)
        return s
    s["kern"] = _kernel(ctx, case)
    if family == "product":
        s["H"] = hh.HMatrix(ctx, s["X"], s["kern"], case["c_leaf"], case["eta"], case["eps"],
                            case["prec"])
        s["U"] = torch.empty_like(s["F"], dtype=tu)
    elif family == "batch":
        s["H"] = hh.Batch(ctx, s["X"], off, s["kern"], case["c_leaf"], case["eta"], case["eps"],
                          case["prec"])
        s["U"] = torch.empty_like(s["F"], dtype=tu)
    elif family == "filaments":
        s["sim"] = hh.Suspension(ctx, s["X"], s["kern"], case["prec"], dt=0.002, n_fil=nf,
                                 n_beads=21, c_leaf=case["c_leaf"], eps=case["eps"],
                                 short=(_weights(*SNET), _weights(*GNET), 5.0))
    return s


def run(s):
    case, family = s["case"], s["case"]["family"]
    if family in ("step", "rotation"):
        return hh.hmatvec(s["ctx"], s["X"], s["F"], s["kern"], case["c_leaf"], case["eta"],
                          case["eps"], case["prec"])
    if family == "product":
        H = s["H"]
        if case["noalloc"]:
            return hh.matvec_noalloc(s["ctx"], H.tree, H.part, H.lr, s["kern"], s["F"], s["U"],
                                     case["prec"])
        return H @ s["F"]
    if family == "batch":
        return s["H"].matvec(s["F"], s["U"])
    if family == "filaments":
        U = s["sim"].step()
        return {"U": U, "X": s["X"]}
    U = hh.hmatvec_autograd(s["ctx"], s["X"], s["F"], s["theta"], c_leaf=case["c_leaf"],
                            eta=case["eta"], eps=case["eps"], prec=case["prec"],
                            input_mode=case["inp"])
    dX, dF, dth = torch.autograd.grad(U, (s["X"], s["F"], s["theta"]), s["dU"])
    return {"U": U.detach(), "dX": dX, "dF": dF, "dtheta": dth}


def work(case):
    """Kernel entries that the H-matrix cannot do without: near pairs of neighbouring leaves
    and the columns and rows of the cross approximation, by counts fitted to the workloads
    (about 8,000 near sources per particle at leaves of 128, and about 2,800 samples per
    particle and doubling of n beyond that)."""
    n = case["n"] // case["systems"]
    rows = case["n"] * (2 if case["kernel"] == "rpy6" else 1)
    n = n * (2 if case["kernel"] == "rpy6" else 1)
    reach = 8000.0 * (case["c_leaf"] / 128.0) * (2 if case["kernel"] == "rpy6" else 1)
    if case["geom"] == "chains":
        reach *= 0.6
    near = min(float(n), reach)
    far = max(0.0, 2800.0 * math.log2(max(n / reach, 1.0)))
    entry = 17920.0 if case["kernel"] == "mlp" else 60.0
    es = 8.0 if case["prec"] == "fp64" else 4.0
    if case["family"] == "grad":
        flops = rows * (near + far) * 3.0 * entry
    elif case["family"] == "product":
        flops = rows * (near * (entry + 18.0) + 18.0 * far)
    else:
        flops = rows * (near + far) * (entry + 18.0)
    kept = 36.0 * far * rows if case["family"] == "product" else 0.0   # factors read once
    return {"bytes": rows * (24.0 + 3 * es + 3 * 8.0) + kept * es / 4.0, "flops": flops}


# ------------------------------------------------- the same in 64 bits, dense


def _net(seed_widths, v):
    Ws, bs = _weights(*seed_widths)
    h = v
    for k, (W, b) in enumerate(zip(Ws, bs)):
        h = h @ torch.from_numpy(W).cuda().T + torch.from_numpy(b).cuda()
        if k < len(Ws) - 1:
            h = torch.tanh(h)
    return h


def _sym(O):
    return 0.5 * (O + O.transpose(-1, -2))


def _entries(case, r):
    """K(r) for displacements r [..., 3] (two-body translational entries)."""
    d2 = (r * r).sum(-1)
    d = d2.sqrt()
    if case["kernel"] == "mlp":
        v = r / d[..., None] if case["inp"] == "direction" else r
        O = _net(KNET, v.reshape(-1, 3)).reshape(r.shape[:-1] + (3, 3))
        return _sym(O) / (8.0 * math.pi * d)[..., None, None]
    far = d >= 2.0
    ci = torch.where(far, (1 + 2.0 / (3.0 * d2)) / (8 * math.pi * d),
                     (1 - 9.0 * d / 32.0) / (6 * math.pi))
    co = torch.where(far, (1 - 2.0 / d2) / (8 * math.pi * d), (3.0 * d / 32.0) / (6 * math.pi))
    eye = torch.eye(3, dtype=r.dtype, device=r.device)
    return ci[..., None, None] * eye + (co / d2)[..., None, None] * r[..., :, None] * r[..., None, :]


def _dense(case, X, F, i0, i1, j0, j1):
    """Rows i0..i1 against the sources j0..j1 (their own pairs left out)."""
    r = X[i0:i1, None, :] - X[None, j0:j1, :]
    own = torch.arange(i0, i1, device=X.device)[:, None] == torch.arange(j0, j1, device=X.device)
    r = torch.where(own[..., None], torch.ones((), dtype=r.dtype, device=r.device), r)
    f = torch.where(own[..., None], torch.zeros((), dtype=r.dtype, device=r.device),
                    F[None, j0:j1, :])
    if case["kernel"] != "rpy6":
        return (_entries(case, r) * f[..., None, :]).sum(-1).sum(1)
    d2 = (r * r).sum(-1)
    id3 = d2 ** -1.5 / (8 * math.pi)
    ff, tt = f[..., :3], f[..., 3:]
    u = (_entries(case, r) * ff[..., None, :]).sum(-1) + \
        id3[..., None] * torch.linalg.cross(tt, r, dim=-1)
    w = id3[..., None] * torch.linalg.cross(ff, r, dim=-1) - 0.5 * id3[..., None] * \
        (tt - 3.0 * r * (r * tt).sum(-1, keepdim=True) / d2[..., None])
    return torch.cat([u, w], -1).sum(1)


def _product(case, X, F, off):
    U = F / (6 * math.pi)
    if case["kernel"] == "rpy6":
        U = torch.cat([F[:, :3] / (6 * math.pi), F[:, 3:] / (8 * math.pi)], 1)
    pairs = (1 << 19) if case["kernel"] == "mlp" else (1 << 22)
    for a, b in zip(off[:-1], off[1:]):
        a, b = int(a), int(b)
        per = max(1, pairs // (b - a))
        for i in range(a, b, per):
            U[i:min(b, i + per)] += _dense(case, X, F, i, min(b, i + per), a, b)
    return U


def _short(X, F, rc=5.0):
    """The short-range terms: neighbours within rc, then every pair (j, k) with k a neighbour
    of i and j a neighbour of k, j != i."""
    n = X.shape[0]
    ii, jj = [], []
    for s in range(0, n, 2048):
        d = X[s:s + 2048, None, :] - X[None]
        near = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2] < rc * rc
        a, b = near.nonzero(as_tuple=True)
        keep = a + s != b
        ii.append(a[keep] + s)
        jj.append(b[keep])
    i, k = torch.cat(ii), torch.cat(jj)                # k in N(i), ordered by i
    U = torch.zeros_like(F)
    d = X[k] - X[i]
    r = d.norm(dim=1)
    K = _sym(_net(SNET, d / r[:, None]).reshape(-1, 3, 3)) / (8 * math.pi * r)[:, None, None]
    U.index_add_(0, i, (K * F[i][:, None, :]).sum(-1))
    deg = torch.bincount(i, minlength=n)
    start = torch.cumsum(deg, 0) - deg
    for s in range(0, i.numel(), 1 << 15):
        a, b = i[s:s + (1 << 15)], k[s:s + (1 << 15)]
        p = torch.repeat_interleave(torch.arange(a.numel(), device=X.device), deg[b])
        q = torch.arange(p.numel(), device=X.device) - torch.repeat_interleave(
            torch.cumsum(deg[b], 0) - deg[b], deg[b])
        j = k[start[b[p]] + q]
        keep = j != a[p]
        j, ti, tk = j[keep], a[p[keep]], b[p[keep]]
        dj, dk = X[j] - X[ti], X[tk] - X[ti]
        o = _net(GNET, torch.cat([dj, dk], 1) / rc)
        sc = 1.0 / (8 * math.pi * (dj - dk).norm(dim=1) * dk.norm(dim=1))
        As = _sym(o[:, :9].reshape(-1, 3, 3)) * sc[:, None, None]
        At = _sym(o[:, 9:].reshape(-1, 3, 3)) * sc[:, None, None]
        U.index_add_(0, ti, (As * F[ti][:, None, :]).sum(-1) + (At * F[j][:, None, :]).sum(-1))
    return U


def _filament_forces(X, nf, beads=21, kt=20.0, l0=3.0, kb=50.0):
    F = torch.zeros_like(X)
    F[:, 2] = -1.0
    C = X[:nf * beads].reshape(nf, beads, 3)
    G = F[:nf * beads].reshape(nf, beads, 3)
    r = C[:, 1:] - C[:, :-1]
    d = r.norm(dim=-1, keepdim=True)
    t = kt * (d - l0) * r / d
    G[:, :-1] += t
    G[:, 1:] -= t
    u = r / d
    t1, t2 = u[:, :-1], u[:, 1:]
    c = torch.linalg.cross(t1, t2, dim=-1)
    T = -kb * c * c.norm(dim=-1, keepdim=True)
    prev, nxt = torch.linalg.cross(T, t1, dim=-1), -torch.linalg.cross(T, t2, dim=-1)
    G[:, :-2] += prev
    G[:, 2:] += nxt
    G[:, 1:-1] -= prev + nxt
    return F


def _gradients(case, X, F, W, theta):
    """U and the gradients of sum W . U of the dense product, by row chunks through autograd."""
    n = X.shape[0]
    X = X.clone().requires_grad_(True)
    F = F.clone().requires_grad_(True)
    th = theta.cuda().requires_grad_(True)
    U = torch.empty_like(W)
    per = max(1, (1 << 18) // n)
    eye = torch.arange(n, device=X.device)
    for i in range(0, n, per):
        e = min(n, i + per)
        r = X[i:e, None, :] - X[None]
        own = eye[i:e, None] == eye[None]
        r = torch.where(own[..., None], torch.ones((), dtype=r.dtype, device=r.device), r)
        d = (r * r).sum(-1).sqrt()
        h = (r / d[..., None] if case["inp"] == "direction" else r).reshape(-1, 3)
        at = 0
        for fi, fo in ((3, 64), (64, 64), (64, 64), (64, 9)):
            A = th[at:at + fi * fo].reshape(fo, fi)
            h = torch.addmm(th[at + fi * fo:at + fi * fo + fo], h, A.T)
            at += fi * fo + fo
            if fo == 64:
                h = torch.tanh(h)
        K = _sym(h.reshape(e - i, n, 3, 3)) / (8 * math.pi * d)[..., None, None]
        K = torch.where(own[..., None, None], torch.zeros((), dtype=K.dtype, device=K.device), K)
        u = F[i:e] / (6 * math.pi) + (K * F[None, :, None, :]).sum(-1).sum(1)
        U[i:e] = u.detach()
        (u * W[i:e]).sum().backward()
    return {"U": U, "dX": X.grad, "dF": F.grad, "dtheta": th.grad.cpu()}


def exact(case, seed):
    # the dense sum over kernel MLP entries in 64 bits takes too long beyond these sizes
    if case["kernel"] == "mlp" and case["n"] // case["systems"] > 40000:
        return None
    X, F, dU, off, nf = _inputs(case, seed)
    X = torch.from_numpy(X).cuda()
    F = torch.from_numpy(F).to(TYPES[case["prec"]][0]).double().cuda()
    off = [0, case["n"]] if off is None else off
    if case["family"] == "grad":
        W = torch.from_numpy(dU).to(TYPES[case["prec"]][1]).double().cuda()
        return _gradients(case, X, F, W, torch.from_numpy(hh.pack_mlp(_weights(*KNET))))
    if case["family"] != "filaments":
        return _product(case, X, F, off)
    F = _filament_forces(X, nf)
    F = F.to(TYPES[case["prec"]][0]).double()
    U = _product(case, X, F, off) + _short(X, F)
    return {"U": U, "X": X + 0.002 * U}
