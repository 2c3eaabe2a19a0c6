"""The work that is timed: what a DMRG program has this library do, step by step.

One growth step of a DMRG run projects the superblock's vector (alone, and
inside Davidson), forms the density matrices of the ground state, diagonalizes
them and takes the block's operators to the kept basis; the orthogonalization
products and the adjoint of the projection are called by themselves too.  The
sizes are those of the repository's workloads (Heisenberg m = 32 to 2048,
Hubbard m = 2048, J1-J2 m = 1024, a batch of 64 members of m = 256 to 2048,
tall-skinny products of 1e5 to 4e6 rows), ragged as the sector sizes are.
"""
from math import comb

import numpy as np
import torch

import paper_1309_5571_amd as dm


def listed():
    return [
        # a superblock early in a chain's growth: one latency-bound call
        {"name": "project_heisenberg_m32", "kind": "project", "model": "heisenberg", "m": 32, "count": 1},
        # the headline superblock: many small two-label sectors (largest block 36)
        {"name": "project_hubbard_m2048", "kind": "project", "model": "hubbard", "m": 2048, "count": 1},
        # one superblock with medium sectors (largest block 180)
        {"name": "project_heisenberg_m1024", "kind": "project", "model": "heisenberg", "m": 1024, "count": 1},
        # many chains or parameter points side by side: the largest projection
        {"name": "project_batch64", "kind": "project", "model": "heisenberg", "m": 2048, "m_lo": 256, "count": 64},
        # forward and backward of the differentiable projection (fitting J1, J2)
        {"name": "grad_j1j2_m1024", "kind": "grad", "model": "j1j2", "m": 1024, "count": 1},
        # the headline solve: FP32 phase, then FP64 to the tolerance
        {"name": "davidson_hubbard_m2048_f32", "kind": "davidson", "model": "hubbard", "m": 2048, "count": 1,
         "prec": "f32", "tol": 1e-11},
        # the default solve of one superblock, FP64 only
        {"name": "davidson_heisenberg_m1024", "kind": "davidson", "model": "heisenberg", "m": 1024, "count": 1,
         "prec": "f64", "tol": 1e-11},
        # a batched solve with a BF16 phase
        {"name": "davidson_batch16_bf16", "kind": "davidson", "model": "heisenberg", "m": 1536, "m_lo": 256,
         "count": 16, "prec": "bf16", "tol": 1e-11},
        # one Gram-Schmidt pair on a long basis: s = V^T x and p = V s
        {"name": "gram_schmidt_n4000000_k20", "kind": "gram_schmidt", "n": 4000000, "k": 20},
        # both blocks' density matrices of a large superblock's state
        {"name": "density_heisenberg_m2048", "kind": "density", "model": "heisenberg", "m": 2048, "count": 1},
        # eigenpairs of one block's density matrix, sector by sector (largest order 180)
        {"name": "eigh_heisenberg_m1024", "kind": "eigh", "model": "heisenberg", "m": 1024, "count": 1},
        # an enlarged block's operators taken to half as many kept states
        {"name": "renormalize_heisenberg_m1024", "kind": "renormalize", "model": "heisenberg", "m": 1024, "keep": 512},
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["project", "project", "project", "grad", "davidson", "davidson", "gram_schmidt", "density",
                       "eigh", "renormalize"])
    if kind == "gram_schmidt":
        return {"kind": kind, "n": _log(rng, 100000, 4000000), "k": rng.randint(1, 32)}
    if kind == "renormalize":
        m = _log(rng, 64, 2048)
        return {"kind": kind, "model": "heisenberg", "m": m, "keep": int(m * rng.uniform(0.3, 0.9))}
    if kind == "grad":
        return {"kind": kind, "model": "j1j2", "m": _log(rng, 64, 1536), "count": 1}
    if kind == "eigh":
        return {"kind": kind, "model": rng.choice(["heisenberg", "hubbard"]), "m": _log(rng, 64, 1536), "count": 1}
    case = {"kind": kind, "model": rng.choice(["heisenberg", "hubbard"]), "count": 1}
    if case["model"] == "hubbard":
        case["m"] = _log(rng, 512, 2048)
    elif kind != "density" and rng.random() < 0.4:
        case["count"] = rng.randint(2, 32 if kind == "project" else 12)
        case["m_lo"] = _log(rng, 32, 512)
        case["m"] = rng.randint(2 * case["m_lo"], 1536)
    else:
        case["m"] = _log(rng, 32 if kind == "project" else 128, 2048)
    if kind == "davidson":
        case["prec"] = rng.choice(["f64", "f64", "f32", "bf16"])
        case["tol"] = 1e-11
    return case


# ------------------------------------------------------------------ superblocks


class _Space:
    def __init__(self, labels, dims):
        self.labels, self.dims = np.asarray(labels, np.int32), np.asarray(dims, np.int64)
        self.index = {tuple(int(v) for v in lab): i for i, lab in enumerate(self.labels)}


class _Op:
    """An operator by its pattern: kind, and for dense ones (src, dst) pairs; values come with a generator."""

    def __init__(self, kind, pairs=(), blocks=None, diag=None):
        self.kind, self.blocks, self.diag = kind, blocks, diag
        self.src, self.dst = np.array([a for a, _ in pairs], np.int32), np.array([b for _, b in pairs], np.int32)


class _Problem:
    pass


def _apportion(weights, m):
    """Integer sizes that sum to m, in proportion to the weights (largest remainders)."""
    quota = m * np.asarray(weights, float) / np.sum(weights)
    dims = np.floor(quota).astype(np.int64)
    dims[np.argsort(-(quota - dims), kind="stable")[: m - int(dims.sum())]] += 1
    return dims


def _space(model, m):
    if model == "hubbard":  # (N_up, N_dn) about the filling, a Gaussian profile
        labels = [(a, b) for a in range(-9, 10) for b in range(-9, 10)]
        weights = [np.exp(-(a * a + b * b) / 18.0) for a, b in labels]
    else:  # 2 S^z, a binomial profile
        labels = [(q,) for q in range(-10, 11)]
        weights = [comb(20, 10 + q) for (q,) in labels]
    dims = _apportion(weights, m)
    return _Space([lab for lab, d in zip(labels, dims) if d], [d for d in dims if d])


def _dense(space, shift, m, rng, symmetric=False):
    """N(0, 1) / sqrt(m) blocks q -> q + shift; a block Hamiltonian is symmetric with levels over [-50, 0]."""
    pairs = [(s, space.index[t]) for s, lab in enumerate(space.labels)
             if (t := tuple(int(a) + b for a, b in zip(lab, shift))) in space.index]
    if rng is None:
        return _Op("dense", pairs)
    blocks = [rng.standard_normal((space.dims[d], space.dims[s])) / np.sqrt(m) for s, d in pairs]
    if symmetric:
        blocks = [np.triu(b) + np.triu(b, 1).T + np.diag(rng.uniform(-50.0, 0.0, len(b))) for b in blocks]
    return _Op("dense", pairs, blocks)


def _transposed(op):
    pairs = list(zip(op.dst.tolist(), op.src.tolist()))
    return _Op("dense", pairs, None if op.blocks is None else [np.ascontiguousarray(b.T) for b in op.blocks])


def _side(model, space, m, rng):
    """Operators of one block: identity, H, then the diagonal and ladder operators of the model."""
    def diagonal():
        return _Op("diag", diag=None if rng is None else rng.uniform(0.0, 1.0, m))

    rank = space.labels.shape[1]
    ops = [_Op("identity"), _dense(space, (0,) * rank, m, rng, symmetric=True)]
    if model == "hubbard":
        ops += [diagonal() for _ in range(3)]
        for shift in ((1, 0), (0, 1)):
            up = _dense(space, shift, m, rng)
            ops += [up, _transposed(up)]
        return ops
    for _ in range(2 if model == "j1j2" else 1):
        up = _dense(space, (1,), m, rng)
        ops += [_Op("diag", diag=np.repeat(space.labels[:, 0] / 2.0, space.dims)), up, _transposed(up)]
    return ops


_TERMS = {
    "heisenberg": ([(1, 0), (0, 1), (3, 4), (4, 3), (2, 2)], [1.0, 1.0, 0.5, 0.5, 1.0]),
    "j1j2": ([(1, 0), (0, 1), (3, 4), (4, 3), (2, 2), (6, 4), (7, 3), (5, 2)],
             [1.0, 1.0, 0.5, 0.5, 1.0, 0.25, 0.25, 0.5]),
    "hubbard": ([(1, 0), (0, 1), (2, 0), (0, 2), (3, 0), (0, 3), (4, 0), (0, 4), (5, 6), (6, 5), (7, 8), (8, 7)],
                [1.0, 1.0, 4.0, 4.0, -2.0, -2.0, -2.0, -2.0, -1.0, -1.0, -1.0, -1.0]),
}


def _problem(model, m, rng):
    p = _Problem()
    p.left = p.right = _space(model, m)
    p.target = np.zeros(p.left.labels.shape[1], np.int32)
    p.ops_left = _side(model, p.left, m, rng)
    p.ops_right = _side("heisenberg" if model == "j1j2" else model, p.right, m, rng)
    terms, coef = _TERMS[model]
    p.terms, p.coef = np.array(terms, np.int32), np.array(coef)
    return p


def _rng(seed):
    return np.random.Generator(np.random.PCG64(seed))


def _sizes(case):
    """Members' m: the case's own, or spread over [m_lo, m] (their logarithm evenly) for a batch."""
    count = case["count"]
    if count == 1:
        return [case["m"]]
    lo, hi = case["m_lo"], case["m"]
    return [int(round(lo * (hi / lo) ** (i / (count - 1)))) for i in range(count)]


def _problems(case, seed, values=True):
    return [_problem(case["model"], m, _rng(seed + 7919 * (i + 1)) if values else None)
            for i, m in enumerate(_sizes(case))]


def _pairs(p):
    """(left sector, right sector) of every block of psi, in the layout's order."""
    out = []
    for s, lab in enumerate(p.left.labels):
        r = p.right.index.get(tuple(int(t) - int(v) for t, v in zip(p.target, lab)))
        if r is not None:
            out.append((s, r))
    return out


def _length(p):
    return sum(int(p.left.dims[a] * p.right.dims[b]) for a, b in _pairs(p))


def _vector(case, seed):
    n = sum(_length(p) for p in _problems(case, seed, values=False))
    return _rng(seed).standard_normal(n)


# ------------------------------------------------------------------ plain evaluation


def _records(p):
    """(term, input pair, output pair, left block index, right block index) of every product of the projection."""
    pairs = _pairs(p)
    index = {a: i for i, (a, _) in enumerate(pairs)}

    def images(op):  # source sector -> (destination, block)
        if op.kind != "dense":
            return None
        return {int(s): (int(d), k) for k, (s, d) in enumerate(zip(op.src, op.dst))}

    left, right = [images(o) for o in p.ops_left], [images(o) for o in p.ops_right]
    for t, (a, b) in enumerate(p.terms):
        for i, (sl, sr) in enumerate(pairs):
            dl, bl = (sl, -1) if left[a] is None else left[a].get(sl, (None, None))
            dr, br = (sr, -1) if right[b] is None else right[b].get(sr, (None, None))
            if dl is not None and dr is not None:
                yield t, i, index[dl], bl, br


def _blocks(p, v):
    out, o = [], 0
    for a, b in _pairs(p):
        r, c = int(p.left.dims[a]), int(p.right.dims[b])
        out.append(v[o:o + r * c].reshape(r, c))
        o += r * c
    return out


def _factor(op, space, sector, block, x, left, transpose):
    """One factor of a term applied to x from its side."""
    if op.kind == "identity":
        return x
    if op.kind == "diag":
        o = int(space.dims[:sector].sum())
        d = op.diag[o:o + int(space.dims[sector])]
        return d[:, None] * x if left else x * d
    m = op.blocks[block].T if transpose else op.blocks[block]
    return m @ x if left else x @ m.T


def _apply(p, v, adjoint=False):
    """H v (or its adjoint), block by block."""
    x, pairs = _blocks(p, v), _pairs(p)
    y = [np.zeros_like(b) for b in x]
    for t, i, o, bl, br in _records(p):
        a, b = p.terms[t]
        src, dst = (o, i) if adjoint else (i, o)
        z = _factor(p.ops_left[a], p.left, pairs[i][0], bl, x[src], True, adjoint)
        y[dst] += p.coef[t] * _factor(p.ops_right[b], p.right, pairs[i][1], br, z, False, adjoint)
    return np.concatenate([b.reshape(-1) for b in y])


def _coef_gradient(p, v, g):
    x, gb, pairs = _blocks(p, v), _blocks(p, g), _pairs(p)
    out = np.zeros(len(p.terms))
    for t, i, o, bl, br in _records(p):
        a, b = p.terms[t]
        z = _factor(p.ops_left[a], p.left, pairs[i][0], bl, x[i], True, False)
        out[t] += np.sum(gb[o] * _factor(p.ops_right[b], p.right, pairs[i][1], br, z, False, False))
    return out


def _diagonal(p):
    """diag(H), for the preconditioner of the plain solve."""
    pairs = _pairs(p)
    d = [np.zeros((int(p.left.dims[a]), int(p.right.dims[b]))) for a, b in pairs]

    def along(op, space, sector, block):
        if op.kind == "identity":
            return np.ones(int(space.dims[sector]))
        o = int(space.dims[:sector].sum())
        return op.diag[o:o + int(space.dims[sector])] if op.kind == "diag" else np.diag(op.blocks[block])

    for t, i, o, bl, br in _records(p):
        if i == o:
            a, b = p.terms[t]
            d[i] += p.coef[t] * np.outer(along(p.ops_left[a], p.left, pairs[i][0], bl),
                                         along(p.ops_right[b], p.right, pairs[i][1], br))
    return np.concatenate([b.reshape(-1) for b in d])


def _energy(p, v):
    """Lowest eigenvalue in the target sector: a plain Davidson iteration in NumPy."""
    diag = _diagonal(p)
    basis, images = [v / np.linalg.norm(v)], []
    for _ in range(60):
        images.append(_apply(p, basis[-1]))
        V, W = np.array(basis), np.array(images)
        e, y = np.linalg.eigh(V @ W.T)
        r = y[:, 0] @ W - e[0] * (y[:, 0] @ V)
        if np.linalg.norm(r) <= 1e-9:  # the energy's error is of the order of its square
            break
        gap = diag - min(e[0], diag.min())
        t = r / np.maximum(gap, 1e-3)
        for _ in range(2):
            t -= V.T @ (V @ t)
        basis.append(t / np.linalg.norm(t))
    return e[0]


# ------------------------------------------------------------------ inputs


def _spectrum_blocks(case, seed):
    """One side's density-matrix blocks: eigenvalues falling over four decades, random eigenvectors."""
    rng = _rng(seed)
    space = _space(case["model"], case["m"])
    blocks = []
    for d in space.dims:
        q = np.linalg.qr(rng.standard_normal((d, d)))[0]
        w = 10.0 ** (-4.0 * (np.arange(d) + rng.uniform(0.0, 0.5, d)) / max(d, 8))
        a = (q * w) @ q.T / case["m"]
        blocks.append((a + a.T) / 2)
    return space.dims, blocks


def _kept_basis(case, seed):
    """An enlarged block's operators H, S+, S- and S^z, eigenvectors of every sector and the states kept."""
    rng = _rng(seed)
    space = _space(case["model"], case["m"])
    ops = _side("heisenberg", space, case["m"], rng)[1:]
    u = [np.linalg.qr(rng.standard_normal((d, d)))[0] for d in space.dims]
    return space, ops, u, np.minimum(_apportion(space.dims, case["keep"]), space.dims)


def _renormalize_inputs(case, seed):
    space, ops, u, keep = _kept_basis(case, seed)
    dims = space.dims
    u_off = np.concatenate([[0], np.cumsum(dims * dims)])
    data, blocks, pos, out = [], [], 0, 0
    for op in ops:
        if op.kind == "diag":
            pairs = [(s, s, op.diag[o:o + d]) for s, (o, d) in enumerate(zip(np.cumsum(dims) - dims, dims))]
        else:
            pairs = list(zip(op.src.tolist(), op.dst.tolist(), op.blocks))
        for s, d, b in pairs:
            blocks.append((pos, int(u_off[d]), int(u_off[s]), out, int(dims[d]), int(dims[s]), int(keep[d]),
                           int(keep[s]), int(op.kind == "diag")))
            data.append(b.reshape(-1))
            pos += b.size
            out += int(keep[d] * keep[s])
    return np.concatenate(data), np.concatenate([x.reshape(-1) for x in u]), blocks, out


def _tall(case, seed):
    """Nearly orthonormal columns (row j of the tensor is column j) and a vector."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    n, k = case["n"], case["k"]
    v = torch.randn(k, n, dtype=torch.float64, device="cuda", generator=g) / n ** 0.5
    return v, torch.randn(n, dtype=torch.float64, device="cuda", generator=g)


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case}
    if kind == "gram_schmidt":
        s["V"], s["x"] = _tall(case, seed)
        s["p"] = torch.empty_like(s["x"])
    elif kind == "eigh":
        s["dims"], blocks = _spectrum_blocks(case, seed)
        s["a"] = _gpu(np.concatenate([b.reshape(-1) for b in blocks]))
    elif kind == "renormalize":
        data, u, s["blocks"], s["out_len"] = _renormalize_inputs(case, seed)
        s["data"], s["u"] = _gpu(data), _gpu(u)
    else:
        s["plan"] = dm.Plan(_problems(case, seed), prec=case.get("prec", "f64"))
        s["psi"] = _gpu(_vector(case, seed))
        if kind == "project":
            s["y"] = torch.empty_like(s["psi"])
        elif kind == "grad":
            s["psi"].requires_grad_(True)
            s["coef"] = s["plan"].coef.clone().requires_grad_(True)
            s["gbar"] = _gpu(_rng(seed + 1).standard_normal(s["plan"].n))
        elif kind == "density":
            s["psi"] /= s["psi"].norm()
            left, right = s["plan"].density_layout()
            s["rho"] = tuple(torch.empty(int(o[-1]), dtype=torch.float64, device="cuda") for o in (left, right))
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "project":
        return s["plan"].project_raw(s["psi"], out=s["y"])
    if kind == "grad":
        y = dm.project(s["plan"], s["psi"], s["coef"])
        return (y, *torch.autograd.grad(y, (s["psi"], s["coef"]), s["gbar"]))
    if kind == "davidson":
        psi, energies, _, _ = s["plan"].davidson(s["psi"], tol=case["tol"], prec=case["prec"])
        return psi, energies
    if kind == "gram_schmidt":
        coefficients = dm.gemv_t(s["V"], s["x"])
        return coefficients, dm.gemv_n(s["V"], coefficients, s["p"])
    if kind == "density":
        return s["plan"].density(s["psi"], out=s["rho"])
    if kind == "eigh":
        return dm.eigh_blocks(s["a"], s["dims"])
    return dm.renormalize(s["data"], s["u"], s["blocks"], s["out_len"])


# ------------------------------------------------------------------ what a pass cannot do without


def _projection_work(p):
    """Operator blocks and diagonals read once, psi read and y written once; the cheaper order of each product."""
    n = _length(p)
    pairs, flops, read = _pairs(p), 0, {}
    for t, i, o, bl, br in _records(p):
        a, b = (int(v) for v in p.terms[t])
        r, c = int(p.left.dims[pairs[i][0]]), int(p.right.dims[pairs[i][1]])
        ro, co = int(p.left.dims[pairs[o][0]]), int(p.right.dims[pairs[o][1]])
        if bl >= 0 and br >= 0:
            flops += 2 * min(ro * r * c + ro * c * co, r * c * co + ro * r * co)
        elif bl >= 0 or br >= 0:
            flops += 2 * ro * co * (r if bl >= 0 else c)
        else:
            flops += 2 * r * c
        if p.ops_left[a].kind != "identity":
            read["left", a, pairs[i][0]] = ro * r if bl >= 0 else r
        if p.ops_right[b].kind != "identity":
            read["right", b, pairs[i][1]] = co * c if br >= 0 else c
    return {"bytes": 8 * (2 * n + sum(read.values())), "flops": flops}


def work(case):
    kind = case["kind"]
    if kind == "gram_schmidt":
        n, k = case["n"], case["k"]
        return {"bytes": 8 * (n * k + 2 * n + 2 * k), "flops": 4 * n * k}
    if kind == "eigh":
        d = _space(case["model"], case["m"]).dims
        # eigenpairs of a symmetric matrix through its tridiagonal form: 4/3 d^3 each to reduce and to transform
        # back, and the eigenvectors of the tridiagonal form
        return {"bytes": 8 * int(np.sum(2 * d * d + d)), "flops": int(np.sum(4 * d ** 3))}
    if kind == "renormalize":
        space = _space(case["model"], case["m"])
        keep = np.minimum(_apportion(space.dims, case["keep"]), space.dims)
        read, flops = int(np.sum(space.dims * keep)), 0
        for op in _side("heisenberg", space, case["m"], None)[1:]:
            for s in range(len(space.dims)) if op.kind == "diag" else range(len(op.src)):
                a, b = (s, s) if op.kind == "diag" else (int(op.src[s]), int(op.dst[s]))
                r, c, kr, kc = (int(v) for v in (space.dims[b], space.dims[a], keep[b], keep[a]))
                read += (r if op.kind == "diag" else r * c) + kr * kc
                flops += 2 * (0 if op.kind == "diag" else r * c * kc) + 2 * r * kr * kc
        return {"bytes": 8 * read, "flops": flops}
    problems = _problems(case, 0, values=False)
    if kind == "density":
        d = [(int(p.left.dims[a]), int(p.right.dims[b])) for p in problems for a, b in _pairs(p)]
        return {"bytes": 8 * sum(r * c + r * r + c * c for r, c in d), "flops": sum(r * c * (r + c + 2) for r, c in d)}
    each = [_projection_work(p) for p in problems]
    w = {k: sum(e[k] for e in each) for k in ("bytes", "flops")}
    if kind == "grad":  # y, the adjoint product and the coefficients' inner products
        n = sum(_length(p) for p in problems)
        return {"bytes": w["bytes"] + 16 * n, "flops": 2 * w["flops"] + 2 * n * len(problems[0].terms)}
    if kind == "davidson":  # at least a handful of projections, with the basis and its images read between them
        n = sum(_length(p) for p in problems)
        return {"bytes": w["bytes"], "flops": 7 * w["flops"] + 7 * 7 * 8 * n}
    return w


# ------------------------------------------------------------------ the same in plain NumPy / torch


def exact(case, seed):
    kind = case["kind"]
    if kind == "gram_schmidt":
        v, x = _tall(case, seed)
        coefficients = v @ x
        return coefficients, coefficients @ v
    if kind == "eigh":
        w, u = [], []
        for b in _spectrum_blocks(case, seed)[1]:
            e, q = np.linalg.eigh(b)
            q = q[:, ::-1]
            q = q * np.sign(q[np.argmax(np.abs(q), axis=0), np.arange(len(e))])
            w.append(e[::-1])
            u.append(q.reshape(-1))
        return np.concatenate(w), np.concatenate(u)
    if kind == "renormalize":
        space, ops, u, keep = _kept_basis(case, seed)
        k = [x[:, :n] for x, n in zip(u, keep)]
        out = []
        for op in ops:
            if op.kind == "diag":
                o = np.cumsum(space.dims) - space.dims
                out += [(k[s].T * op.diag[o[s]:o[s] + d]) @ k[s] for s, d in enumerate(space.dims)]
            else:
                out += [k[d].T @ b @ k[s] for s, d, b in zip(op.src, op.dst, op.blocks)]
        return np.concatenate([b.reshape(-1) for b in out])
    problems = _problems(case, seed)
    psi = _vector(case, seed)
    cut = np.cumsum([_length(p) for p in problems])[:-1]
    parts = np.split(psi, cut)
    if kind == "project":
        return np.concatenate([_apply(p, v) for p, v in zip(problems, parts)])
    if kind == "density":
        x = [b for p, v in zip(problems, parts) for b in _blocks(p, v / np.linalg.norm(psi))]
        return (np.concatenate([(b @ b.T).reshape(-1) for b in x]), np.concatenate([(b.T @ b).reshape(-1) for b in x]))
    if kind == "grad":
        p, g = problems[0], _rng(seed + 1).standard_normal(len(psi))
        return _apply(p, psi), _apply(p, g, adjoint=True), _coef_gradient(p, psi, g)
    # the solve: its energies (an eigenvector has no sign of its own); many members take too long
    if len(problems) > 4 or len(psi) > 200000:
        return None
    return None, np.array([_energy(p, v) for p, v in zip(problems, parts)])
