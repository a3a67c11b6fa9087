"""Performance cases: the work that a program using this sampler has it do.

Every case goes through the package's public entry points: `Box.sample` and
`Box.sample_seeded` (noise -> MINRES solve -> projection onto the tet mesh) over
boxes of 8^3 to 256^3 cells and batches of 1 to 128 samples, in both precisions,
with constant and cell-wise coefficients; the stateless transfer product
`csr_apply`; the construction of the transfer `build_transfer_device`; and a
burst of requests through the serving loop.  Sizes are those of the benchmark
workloads and the serving mix, and odd ones in between.

`exact` gives the same results in float64 from plain torch: the spectral solve
of the constant-coefficient box, a conjugate-gradient solve for cell-wise
coefficients, the flux by dense line solves, the projection by clipping every
tet against the cells it crosses, and the counter-based generator from its
published definition.
"""
import math

import numpy as np
import torch

import paper_1712_06758_amd as P

DEV = torch.device("cuda")
F64 = torch.float64

# Kuhn split of a cube into 6 tets (corner number = x + 2 y + 4 z).
KUHN = np.array([(0, 1, 3, 7), (0, 1, 5, 7), (0, 2, 3, 7), (0, 2, 6, 7), (0, 4, 5, 7), (0, 4, 6, 7)])


# ---------------------------------------------------------------------------
# the cases


def _sample(name, n, batch, precision, kappa, m, noise="given", out="tet", coef="const", refine=0.0):
    """A sampling call: box n^3, `batch` samples, mesh of 6 m^3 tets (0: none).
    noise: "given" (a tensor), "event" (drawn on the device), "coupled" (drawn
    as the coarse sample of a fine event).  out: "tet", "box", "tet+box",
    "box+sigma".  coef: constant or cell-wise kappa and g.  refine: target of
    the iterative refinement (0: off)."""
    c = {"kind": "sample", "n": n, "batch": batch, "precision": precision, "kappa": kappa, "m": m,
         "noise": noise, "out": out, "coef": coef, "refine": refine}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # One draw on the smallest box of the workload set: a test, a first call, latency alone.
        _sample("box16 b1 fp64", 16, 1, "fp64", 10.0, 10, out="tet+box"),
        # The coarse halves of a multilevel estimator: many small boxes at once, noise from the event.
        _sample("box32 b24 mixed coupled", 32, 24, "mixed", 20.0, 16, noise="coupled"),
        # One field at a time on a middle box, with its flux, as a flow model takes it.
        _sample("box64 b1 mixed flux", 64, 1, "mixed", 10.0, 0, out="box+sigma"),
        # The 64^3 workload: 32 vectors onto 303,918 tets.
        _sample("box64 b32 fp64", 64, 32, "fp64", 10.0, 37),
        # An odd batch in mixed precision refined to float64 accuracy.
        _sample("box64 b7 refined", 64, 7, "mixed", 15.0, 20, noise="event", out="box", refine=1e-11),
        # The headline workload: 64 vectors at 128^3 onto 2,431,344 tets.
        _sample("box128 b64 mixed", 128, 64, "mixed", 20.0, 74),
        # The same box, one sample in full precision.
        _sample("box128 b1 fp64", 128, 1, "fp64", 20.0, 74),
        # Space-dependent correlation length and variance, an odd batch.
        _sample("box128 b13 cellwise", 128, 13, "mixed", 20.0, 0, out="box", coef="cell"),
        # The largest box of the workload set.
        _sample("box256 b8 mixed", 256, 8, "mixed", 50.0, 0, noise="event", out="box"),
        # Fields that are there already, projected with an explicit matrix.
        {"name": "transfer 64 b20", "kind": "transfer", "n": 64, "batch": 20, "m": 37},
        # A new mesh: the transfer matrix of the 128^3 workload.
        {"name": "build 128", "kind": "build", "n": 128, "m": 74},
        # A burst of coupled requests through the serving loop, 32^3 and 64^3 levels.
        {"name": "serve burst", "kind": "serve", "r32": 32, "r64": 12},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    kind = rng.choice(["sample"] * 7 + ["transfer", "transfer", "build", "serve"])
    if kind == "serve":
        return {"kind": "serve", "r32": _log_int(rng, 1, 38), "r64": _log_int(rng, 1, 12)}
    if kind == "build":
        n = rng.choice([16, 32, 64, 128])
        return {"kind": "build", "n": n, "m": _log_int(rng, max(2, n // 6), min(74, n * 5 // 8))}
    if kind == "transfer":
        n = rng.choice([16, 32, 64, 128])
        return {"kind": "transfer", "n": n, "batch": _log_int(rng, 1, 64 if n < 128 else 40),
                "m": _log_int(rng, max(2, n // 6), min(64, n * 5 // 8))}
    n = rng.choice([8, 16, 32, 32, 64, 64, 128, 128, 256])
    most = {8: 128, 16: 128, 32: 128, 64: 64, 128: 32, 256: 3}[n]
    precision = rng.choice(["fp64", "mixed"])
    batch = _log_int(rng, 1, most)
    kappa = round(math.exp(rng.uniform(math.log(5.0), math.log(50.0))), 3)
    out = rng.choice(["tet", "tet", "box", "tet+box", "box+sigma"])
    m = _log_int(rng, max(2, n // 6), min(64, n * 5 // 8)) if "tet" in out else 0
    coef = rng.choice(["const", "const", "cell"])
    noise = rng.choice(["given", "given", "event", "coupled"])
    refine = 1e-11 if precision == "mixed" and n < 256 and rng.random() < 0.2 else 0.0
    return _sample(None, n, batch, precision, kappa, m, noise, out, coef, refine)


# ---------------------------------------------------------------------------
# inputs


def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + salt) & ((1 << 62) - 1))
    return g


def _randn(shape, seed, salt):
    return torch.randn(shape, generator=_gen(seed, salt), device=DEV, dtype=F64)


def _mesh(lo, hi, m, seed):
    """Jittered Kuhn-tet mesh of the cube [lo, hi]^3: (xyz [V, 3], tets [6 m^3, 4])."""
    ht = (hi - lo) / m
    g = lo + ht * np.arange(m + 1)
    X, Y, Z = np.meshgrid(g, g, g, indexing="ij")
    xyz = np.stack([X.ravel(), Y.ravel(), Z.ravel()], axis=1)
    xyz = xyz + np.random.default_rng(seed).uniform(-0.2 * ht, 0.2 * ht, size=xyz.shape)
    i, j, k = (a.ravel() for a in np.meshgrid(np.arange(m), np.arange(m), np.arange(m), indexing="ij"))
    corner = np.stack([(k + (b >> 2 & 1)) + (m + 1) * ((j + (b >> 1 & 1)) + (m + 1) * (i + (b & 1)))
                       for b in range(8)], axis=1)
    return np.ascontiguousarray(xyz), corner[:, KUHN].reshape(-1, 4).astype(np.int32)


def _smooth(n, lo, hi, seed):
    """A smooth positive cell field spanning [lo, hi], x fastest."""
    rng = np.random.default_rng(seed)
    x = (np.arange(n) + 0.5) / n
    Z, Y, X = np.meshgrid(x, x, x, indexing="ij")
    f = np.zeros_like(X)
    for _ in range(4):
        a, b, c = rng.uniform(0.5, 2.5, 3)
        p = rng.uniform(0, 2 * np.pi, 3)
        f += np.cos(np.pi * a * X + p[0]) * np.cos(np.pi * b * Y + p[1]) * np.cos(np.pi * c * Z + p[2])
    f = (f - f.min()) / (f.max() - f.min())
    return torch.tensor((lo * (hi / lo) ** f).reshape(-1), device=DEV)


def _coefficients(case, seed):
    """(kappa, g) cell fields of a cell-wise case."""
    kap = _smooth(case["n"], 0.5 * case["kappa"], 2.0 * case["kappa"], seed)
    return kap, torch.sqrt(8.0 * math.pi * kap)


def _event0(seed):
    return (int(seed) * 7919) & ((1 << 40) - 1)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "sample":
        n, B = case["n"], case["batch"]
        box = P.Box(n, case["kappa"], precision=case["precision"], max_batch=B)
        if case["m"]:
            box.set_mesh(*_mesh(0.1, 0.9, case["m"], seed), builder="device" if n >= 128 else "host")
        if case["coef"] == "cell":
            box.set_coefficients(*_coefficients(case, seed))
        if case["refine"]:
            box.set_refinement(case["refine"])
        s = {"case": case, "box": box, "event0": _event0(seed)}
        if case["noise"] == "given":
            s["xi"] = _randn((B, n ** 3), seed, 1)
        return s
    if kind == "transfer":
        n = case["n"]
        rp, ci, cv = P.build_transfer_device(n, *_mesh(0.1, 0.9, case["m"], seed))
        order = torch.as_tensor(P.transfer_chunk_order(n, rp.cpu().numpy(), ci.cpu().numpy())).to(DEV)
        return {"case": case, "rp": rp, "ci": ci, "cv": cv, "order": order,
                "x": _randn((case["batch"], n ** 3), seed, 2)}
    if kind == "build":
        # the seed moves the first tet only: the number of entries stays that of the mesh
        xyz, tets = _mesh(0.1, 0.9, case["m"], 1)
        tets = np.roll(tets, 1 + int(seed) * 7919 % (tets.shape[0] - 1), axis=0)
        return {"case": case, "xyz": torch.tensor(xyz, device=DEV), "tets": torch.tensor(tets, device=DEV)}
    from paper_1712_06758_amd import serve
    srv = serve.build_gpu_server(levels=(32, 64), corr_len=0.05, keep_results=True, hbm_budget=1 << 36)
    first = _event0(seed)
    arrivals = [(0.0, 32, first + r) for r in range(case["r32"])] + [(0.0, 64, first + r) for r in range(case["r64"])]
    return {"case": case, "srv": srv, "arrivals": arrivals}


# ---------------------------------------------------------------------------
# one pass


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "sample":
        want = dict(u_tet="tet" in case["out"], u_box="box" in case["out"], sigma="sigma" in case["out"])
        if case["noise"] == "given":
            r = state["box"].sample(state["xi"], **want)
        else:
            r = state["box"].sample_seeded(2024, state["event0"], case["batch"], coupled=case["noise"] == "coupled",
                                           **want)
        return {k: r[k] for k in ("u_tet", "u_box", "sigma") if k in r}
    if kind == "transfer":
        return P.csr_apply(state["rp"], state["ci"], state["cv"], state["x"], state["rp"].numel() - 1,
                           order=state["order"])
    if kind == "build":
        rp, ci, cv = P.build_transfer_device(case["n"], state["xyz"], state["tets"])
        return {"row_ptr": rp, "cols": ci, "vals": cv}
    srv = state["srv"]
    srv.done = []
    srv.run(state["arrivals"])
    # every part of every request, in the order of the arrivals
    return [p.result for r in sorted(srv.done, key=lambda r: r.rid) for p in r.parts]


def work(case):
    """Inputs read once, outputs written once.  The operations of a solve are
    those of its MINRES iterations (about 36 in mixed precision and 47 in
    float64): the operator, the recurrences and one V-cycle, about 200 a cell."""
    kind = case["kind"]
    if kind == "serve":
        b = f = 0.0
        for level, count in ((32, case["r32"]), (64, case["r64"])):
            for n in ((32,) if level == 32 else (64, 32)):
                b += count * 8.0 * (n ** 3 + 6 * (level // 2) ** 3)
                f += count * 36 * 200.0 * n ** 3
        return {"bytes": b, "flops": f}
    n, nc = case["n"], float(case["n"] ** 3)
    ntet = 6.0 * case["m"] ** 3
    # cells a tet crosses, estimated from the ratio of the mesh width to h
    nnz = ntet * (1.0 + 1.35 * 0.8 * n / max(1, case["m"])) ** 2
    if kind == "build":
        return {"bytes": 24.0 * (case["m"] + 1) ** 3 + 16.0 * ntet + 8.0 * ntet + 12.0 * nnz, "flops": 300.0 * nnz}
    B = case["batch"]
    if kind == "transfer":
        return {"bytes": 8.0 * B * (nc + ntet) + 12.0 * nnz + 8.0 * ntet, "flops": 2.0 * B * nnz}
    b = 8.0 * B * nc * ((case["noise"] == "given") + ("box" in case["out"]) + 3.0 * ("sigma" in case["out"]))
    if "tet" in case["out"]:
        b += 8.0 * B * ntet + 12.0 * nnz + 8.0 * ntet
    if case["coef"] == "cell":
        b += 16.0 * nc
    its = (36 if case["precision"] == "mixed" else 47) + (15 if case["refine"] else 0)
    return {"bytes": max(b, 8.0 * B * nc), "flops": its * 200.0 * nc * B}


# ---------------------------------------------------------------------------
# the same in 64 bits, without the package's code


def _dct(n):
    """Orthonormal DCT-II matrix and the eigenvalues of one direction of
    B M^-1 B^T on a line of n cells (times h)."""
    i = torch.arange(n, device=DEV, dtype=F64)
    C = torch.cos(math.pi * (i[None, :] + 0.5) * i[:, None] / n) * math.sqrt(2.0 / n)
    C[0] = math.sqrt(1.0 / n)
    lam = 12.0 * torch.sin(math.pi * i / (2 * n)) ** 2 / (2.0 + torch.cos(math.pi * i / n))
    return C, lam / n


def _along(A, u):
    """A applied along x, y and z of u [B, n, n, n] (x last), in turn."""
    B, nz, ny, nx = u.shape
    u = torch.matmul(u, A.t())
    u = torch.matmul(A, u)
    return torch.matmul(A, u.reshape(B, nz, -1)).reshape(B, -1, u.shape[2], u.shape[3])


def _spectral(n, kappa, f):
    """(kappa^2 W + B M^-1 B^T)^-1 f for f [B, n^3]."""
    C, lam = _dct(n)
    d = kappa * kappa / n ** 3 + lam[:, None, None] + lam[None, :, None] + lam[None, None, :]
    return _along(C.t(), _along(C, f.reshape(-1, n, n, n)) / d).reshape(f.shape)


def _cellwise(n, kap, f):
    """The same with cell-wise kappa, by conjugate gradients on the exact
    Schur complement, preconditioned by the constant-coefficient solve."""
    C, lam = _dct(n)
    K = C.t() @ torch.diag(lam) @ C
    k2 = kap * kap / n ** 3
    ref = float(torch.sqrt(kap.min() * kap.max()))

    def S(u):
        w = u.reshape(-1, n, n, n)
        y = torch.matmul(w, K) + torch.matmul(K, w) + torch.matmul(K, w.reshape(-1, n, n * n)).reshape(w.shape)
        return y.reshape(u.shape) + k2 * u

    x = torch.zeros_like(f)
    r = f.clone()
    z = _spectral(n, ref, r)
    p = z.clone()
    rz = (r * z).sum(1, keepdim=True)
    rz0 = rz.clone()
    for _ in range(200):
        q = S(p)
        a = rz / (p * q).sum(1, keepdim=True)
        x += a * p
        r -= a * q
        z = _spectral(n, ref, r)
        new = (r * z).sum(1, keepdim=True)
        if bool((new <= 1e-30 * rz0).all()):
            break
        p = z + (new / rz) * p
        rz = new
    return x


def _flux(n, u):
    """sigma = -M^-1 B^T u on the full face layout, [B, 3 n^2 (n + 1)]."""
    T = torch.zeros((n - 1, n - 1), device=DEV, dtype=F64)
    T += torch.diag(torch.full((n - 1,), 2.0 / 3.0, device=DEV, dtype=F64))
    o = torch.full((n - 2,), 1.0 / 6.0, device=DEV, dtype=F64)
    T += torch.diag(o, 1) + torch.diag(o, -1)
    D = torch.zeros((n - 1, n), device=DEV, dtype=F64)
    i = torch.arange(n - 1, device=DEV)
    D[i, i + 1], D[i, i] = float(n), -float(n)
    G = torch.zeros((n + 1, n), device=DEV, dtype=F64)
    G[1:n] = torch.linalg.solve(T, D)
    w = u.reshape(-1, n, n, n)
    B = w.shape[0]
    sx = torch.matmul(w, G.t()).reshape(B, -1)
    sy = torch.matmul(G, w).reshape(B, -1)
    sz = torch.matmul(G, w.reshape(B, n, n * n)).reshape(B, -1)
    return torch.cat([sx, sy, sz], 1)


M32 = 0xFFFFFFFF


def _i64(v):
    v &= (1 << 64) - 1
    return v - (1 << 64) if v >> 63 else v


def _mulhilo(a, b):
    """High and low words of the 64 x 64-bit product of the constant a and the tensor b (bit patterns)."""
    al, ah = a & M32, a >> 32
    bl, bh = b & M32, (b >> 32) & M32
    ll, lh, hl, hh = al * bl, al * bh, ah * bl, ah * bh
    mid = ((ll >> 32) & M32) + (lh & M32) + (hl & M32)
    return hh + ((lh >> 32) & M32) + ((hl >> 32) & M32) + ((mid >> 32) & M32), b * _i64(a)


def _noise(n, seed, event):
    """The field of an event on the n^3 box: Philox4x64-10 (Salmon et al., SC 2011) and Box-Muller."""
    c0 = torch.arange(n ** 3 // 4, device=DEV, dtype=torch.int64)
    c1, c2, c3 = torch.full_like(c0, n), torch.zeros_like(c0), torch.zeros_like(c0)
    k0, k1 = int(seed), int(event)
    for r in range(10):
        h0, l0 = _mulhilo(0xD2E7470EE14C6C93, c0)
        h1, l1 = _mulhilo(0xCA5A826395121157, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ _i64(k0), l1, h0 ^ c3 ^ _i64(k1), l0
        k0, k1 = k0 + 0x9E3779B97F4A7C15, k1 + 0xBB67AE8584CAA73B
    out = torch.empty((c0.numel(), 4), device=DEV, dtype=F64)
    m53 = (1 << 53) - 1
    for q, (a, b) in enumerate(((c0, c1), (c2, c3))):
        u = (((a >> 11) & m53) + 1).to(F64) * 2.0 ** -53
        t = ((b >> 11) & m53).to(F64) * 2.0 ** -53
        rad = torch.sqrt(-2.0 * torch.log(u))
        out[:, 2 * q] = rad * torch.cos(2 * math.pi * t)
        out[:, 2 * q + 1] = rad * torch.sin(2 * math.pi * t)
    return out.reshape(-1)


def _restrict(xf, n):
    return xf.reshape(n, 2, n, 2, n, 2).sum((1, 3, 5)).reshape(-1) / math.sqrt(8.0)


def _event_noise(n, seed, event, coupled):
    return _restrict(_noise(2 * n, seed, event), n) if coupled else _noise(n, seed, event)


def _clip(T, own, d, plane, sign):
    """The parts of the tets T [N, 4, 3] with sign (x_d - plane) >= 0, split into
    tets again, and the owners of the parts."""
    f = sign * (T[:, :, d] - plane[:, None])
    f, o = torch.sort(f, dim=1, descending=True)
    T = torch.gather(T, 1, o[:, :, None].expand(-1, -1, 3))
    k = (f > 0).sum(1)

    def cut(s, a, b):
        t = (f[s, a] / (f[s, a] - f[s, b]))[:, None]
        return T[s, a] + t * (T[s, b] - T[s, a])

    def prism(a, b):
        return [torch.stack(v, 1) for v in ((a[0], a[1], a[2], b[0]), (a[1], a[2], b[0], b[1]),
                                            (a[2], b[0], b[1], b[2]))]

    s4, s1, s2, s3 = k == 4, k == 1, k == 2, k == 3
    parts, owners = [T[s4]], [own[s4]]
    parts.append(torch.stack([T[s1, 0], cut(s1, 0, 1), cut(s1, 0, 2), cut(s1, 0, 3)], 1))
    owners.append(own[s1])
    parts += prism((T[s2, 0], cut(s2, 0, 2), cut(s2, 0, 3)), (T[s2, 1], cut(s2, 1, 2), cut(s2, 1, 3)))
    parts += prism((T[s3, 0], T[s3, 1], T[s3, 2]), (cut(s3, 0, 3), cut(s3, 1, 3), cut(s3, 2, 3)))
    owners += [own[s2]] * 3 + [own[s3]] * 3
    return torch.cat(parts), torch.cat(owners)


def _volume(T):
    return torch.linalg.det(T[:, 1:] - T[:, :1]).abs() / 6.0


def _project(n, mesh, u):
    """Averages of the box fields u [B, n^3] over the tets, from exact overlaps."""
    xyz = torch.tensor(mesh[0], device=DEV)
    tets = torch.tensor(mesh[1], device=DEV).long()
    out = torch.empty((u.shape[0], tets.shape[0]), device=DEV, dtype=F64)
    for t0 in range(0, tets.shape[0], 100000):
        V = xyz[tets[t0:t0 + 100000]]
        T, own = V, torch.arange(V.shape[0], device=DEV)[:, None]      # owner: tet, then cell indices
        for d in range(3):
            lo = torch.floor(T[:, :, d].min(1).values * n).long().clamp(0, n - 1)
            hi = torch.floor(T[:, :, d].max(1).values * n).long().clamp(0, n - 1)
            rep = hi - lo + 1
            src = torch.repeat_interleave(torch.arange(T.shape[0], device=DEV), rep)
            at = torch.arange(src.numel(), device=DEV) - torch.repeat_interleave(torch.cumsum(rep, 0) - rep, rep)
            i = lo[src] + at
            T, own = T[src], torch.cat([own[src], i[:, None]], 1)
            T, own = _clip(T, own, d, own[:, -1].to(F64) / n, 1.0)
            T, own = _clip(T, own, d, (own[:, -1] + 1).to(F64) / n, -1.0)
        vol = _volume(T)
        cell = own[:, 1] + n * (own[:, 2] + n * own[:, 3])
        key, inv = torch.unique(own[:, 0] * n ** 3 + cell, return_inverse=True)
        w = torch.zeros(key.numel(), device=DEV, dtype=F64).index_add_(0, inv, vol)
        row, col = key // n ** 3, key % n ** 3
        w = w / _volume(V)[row]
        for b in range(u.shape[0]):
            out[b, t0:t0 + V.shape[0]] = torch.zeros(V.shape[0], device=DEV, dtype=F64).index_add_(0, row, w * u[b, col])
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "build":
        return None      # which overlaps of rounding size are listed is the clipper's choice
    if kind == "transfer":
        return _project(case["n"], _mesh(0.1, 0.9, case["m"], seed), _randn((case["batch"], case["n"] ** 3), seed, 2))
    if kind == "serve":
        kappa, first, got = 20.0, _event0(seed), []
        g = math.sqrt(8.0 * math.pi * kappa)
        for level, count in ((32, case["r32"]), (64, case["r64"])):
            mesh = _mesh(0.1, 0.9, level // 2, 1)
            parts = []
            for n in ((32,) if level == 32 else (64, 32)):
                xi = torch.stack([_event_noise(n, 2024, (level << 40) | (first + r), n != level)
                                  for r in range(count)])
                parts.append(_project(n, mesh, _spectral(n, kappa, g * n ** -1.5 * xi)))
            got += [p[r] for r in range(count) for p in parts]
        return got
    n, B, kappa = case["n"], case["batch"], case["kappa"]
    if case["noise"] == "given":
        xi = _randn((B, n ** 3), seed, 1)
    else:
        xi = torch.stack([_event_noise(n, 2024, _event0(seed) + b, case["noise"] == "coupled") for b in range(B)])
    if case["coef"] == "cell":
        kap, g = _coefficients(case, seed)
        u = _cellwise(n, kap, g * n ** -1.5 * xi)
    else:
        u = _spectral(n, kappa, math.sqrt(8.0 * math.pi * kappa) * n ** -1.5 * xi)
    res = {}
    if "tet" in case["out"]:
        res["u_tet"] = _project(n, _mesh(0.1, 0.9, case["m"], seed), u)
    if "box" in case["out"]:
        res["u_box"] = u
    if "sigma" in case["out"]:
        res["sigma"] = _flux(n, u)
    return res
