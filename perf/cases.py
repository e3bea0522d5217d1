"""The work that a program built on this framework has it do, as timed cases.

A case names a kind of work and its sizes.  `prepare` makes the inputs on the
GPU from the seed (and the plan, workspace or model that a program keeps),
`run` is one pass through the public entry points, `exact` is the same result
in 64 bits from plain torch, and `work` is the bytes and operations that the
result cannot do without.
"""
import math

import numpy as np
import torch

import paper_1905_01330_amd as tn
from paper_1905_01330_amd import inputs

DEV = "cuda:0"
F64 = torch.float64


def listed():
    return [
        # one edge between two small nodes (a gate, the end of a chain): launch latency
        {"name": "edge-16", "kind": "edge", "left": 16, "mid": 1, "bond": 16, "right": 16, "edges": 1, "prec": "fp32"},
        # two parallel edges and a permuted result at bonds that no tile divides
        {"name": "edge-odd-333", "kind": "edge", "left": 333, "mid": 3, "bond": 333, "right": 331, "edges": 2,
         "prec": "fp32"},
        # the bulk-site contraction of a chi = 1024 chain with a bond-5 operator
        {"name": "edge-1024", "kind": "edge", "left": 1024, "mid": 5, "bond": 1024, "right": 1024, "edges": 1,
         "prec": "split_bf16"},
        # operator environments of a transverse-field Ising chain, both directions
        {"name": "sweep-tfim-256", "kind": "sweep", "model": "tfim", "sites": 30, "chi": 256, "prec": "fp32"},
        # operator environments of an XXZ chain at the benchmark's bond
        {"name": "sweep-xxz-1024", "kind": "sweep", "model": "xxz", "sites": 24, "chi": 1024, "prec": "split_bf16"},
        # one overlap of two chains, an ordinary bond that is not a power of two
        {"name": "inner-100", "kind": "inner", "sites": 100, "chi": 100, "prec": "split_bf16"},
        # overlaps of many chains of uneven length and bond in one call
        {"name": "batch-32", "kind": "batch", "chains": 32, "sites": 128, "chi": 512, "prec": "fp32"},
        # classifying a large batch of 28 x 28 images
        {"name": "classify-4096", "kind": "classify", "sites": 784, "chi": 64, "batch": 4096, "train": False},
        # one training step: scores, loss and every weight gradient
        {"name": "train-1024", "kind": "classify", "sites": 784, "chi": 128, "batch": 1024, "train": True},
        # bringing an updated chain back to the left-canonical gauge (FP64)
        {"name": "gauge-1024", "kind": "gauge", "sites": 28, "chi": 1024},
        # truncating a two-site node of a chi = 256 chain back to its bond
        {"name": "split-256", "kind": "split", "left": 256, "right": 256, "keep": 256},
        # the effective Hamiltonian of a two-site DMRG update on its node
        {"name": "heff-256", "kind": "heff", "chi": 256, "right": 256, "model": "tfim", "prec": "split_bf16"},
    ]


def _between(rng, lo, hi):
    """A whole number, spread evenly over the logarithm; every other one made odd."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 0.5:
        v |= 1
    return max(lo, min(hi, v))


def draw(rng):
    kind = rng.choice(["edge", "edge", "sweep", "inner", "batch", "classify", "train", "gauge", "split", "heff"])
    prec = rng.choice(["fp32", "split_bf16"])
    if kind == "edge":
        return {"kind": "edge", "left": _between(rng, 8, 1024), "mid": rng.randint(1, 5), "bond": _between(rng, 8, 1024),
                "right": _between(rng, 8, 1024), "edges": rng.randint(1, 2), "prec": prec}
    if kind == "sweep":
        return {"kind": "sweep", "model": rng.choice(["tfim", "xxz"]), "sites": rng.randint(12, 30),
                "chi": _between(rng, 16, 700), "prec": prec}
    if kind == "inner":
        return {"kind": "inner", "sites": rng.randint(16, 100), "chi": _between(rng, 16, 1024), "prec": "split_bf16"}
    if kind == "batch":
        return {"kind": "batch", "chains": rng.randint(4, 32), "sites": _between(rng, 16, 128),
                "chi": _between(rng, 16, 500), "prec": prec}
    if kind in ("classify", "train"):
        return {"kind": "classify", "sites": rng.choice([64, 196, 400, 784]), "chi": _between(rng, 8, 128),
                "batch": _between(rng, 16, 1024), "train": kind == "train"}
    if kind == "gauge":
        return {"kind": "gauge", "sites": rng.randint(14, 28), "chi": _between(rng, 16, 900)}
    if kind == "split":
        left, right = _between(rng, 8, 256), _between(rng, 8, 256)
        return {"kind": "split", "left": left, "right": right, "keep": max(1, min(left, right) - rng.randint(0, 7))}
    return {"kind": "heff", "chi": _between(rng, 16, 512), "right": _between(rng, 16, 512),
            "model": rng.choice(["tfim", "xxz"]), "prec": prec}


# ---------------------------------------------------------------------------
# inputs


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _randn(gen, *shape, dtype=torch.float32):
    return torch.randn(*shape, generator=gen, device=DEV, dtype=dtype)


def _isometry(gen, rows, cols):
    """Orthonormal columns, FP64."""
    x = _randn(gen, rows, cols, dtype=F64)
    if rows < 2 * cols:
        return torch.linalg.qr(x.cpu())[0].to(DEV)
    for _ in range(2):      # a tall Gaussian is well conditioned: its Gram matrix will do, twice
        g = torch.linalg.cholesky(x.T @ x)
        x = torch.linalg.solve_triangular(g, x.T.contiguous(), upper=False).T.contiguous()
    return x


def _canonical_sites(gen, n, chi):
    """A left-canonical chain: every site [D, 2, D'] an isometry from (D, 2) to D' (FP64)."""
    dims = inputs.bond_dims(n, 2, chi)
    return [_isometry(gen, dims[k] * 2, dims[k + 1]).reshape(dims[k], 2, dims[k + 1]) for k in range(n)]


def _mpo(model, n, dtype=torch.float32):
    ops = inputs.xxz_mpo(n, 0.5) if model == "xxz" else inputs.tfim_mpo(n)
    return [torch.tensor(w, dtype=dtype, device=DEV) for w in ops]


def _edge_inputs(case, seed):
    gen = _gen(seed)
    a, w, b, c = case["left"], case["mid"], case["bond"], case["right"]
    site = _randn(gen, b, 2, c) / math.sqrt(2 * b)
    if case["edges"] == 1:
        return _randn(gen, a, w, b), site, [2], [0]
    return _randn(gen, b, 2, w, a), site, [0, 1], [0, 1]


def _edge_out(case):
    a, w, c = case["left"], case["mid"], case["right"]
    if case["edges"] == 1:
        return torch.empty(a, w, 2, c, device=DEV)
    return torch.empty(c, w, a, device=DEV)      # the environment layout [bra, operator, ket]


def _chain_pair(gen, n, chi):
    """A chain and a copy of it with a tenth of noise (FP32), each one buffer of sites."""
    dims = inputs.bond_dims(n, 2, chi)
    sizes = [dims[k] * 2 * dims[k + 1] for k in range(n)]
    flat = _randn(gen, sum(sizes)) / math.sqrt(2 * chi)
    other = flat + 0.1 * _randn(gen, sum(sizes)) / math.sqrt(2 * chi)

    def cut(x):
        return [s.view(dims[k], 2, dims[k + 1]) for k, s in enumerate(x.split(sizes))]

    return cut(flat), cut(other)


def _batch_shapes(case):
    rng = np.random.default_rng(case["chains"] * 1000003 + case["sites"] * 1009 + case["chi"])
    return [(int(rng.integers(8, case["sites"] + 1)), int(rng.integers(8, case["chi"] + 1)))
            for _ in range(case["chains"])]


LABELS = 10


def _classify_inputs(case, seed):
    gen = _gen(seed)
    n, chi, batch = case["sites"], case["chi"], case["batch"]
    dims = [1] + [chi] * (n - 1) + [1]
    shapes = [(dims[k], 2, LABELS, dims[k + 1]) if k == n // 2 else (dims[k], 2, dims[k + 1]) for k in range(n)]
    sizes = [math.prod(s) for s in shapes]
    flat = _randn(gen, sum(sizes)) / math.sqrt(chi)
    sites = [x.view(s) for x, s in zip(flat.split(sizes), shapes)]
    pixels = torch.rand(batch, n, generator=gen, device=DEV)
    labels = torch.randint(0, LABELS, (batch,), generator=gen, device=DEV)
    return sites, pixels, labels, shapes, sizes


def _gauge_inputs(case, seed):
    """A left-canonical chain after an update of a tenth of its size."""
    gen = _gen(seed)
    sites = _canonical_sites(gen, case["sites"], case["chi"])
    return [s + 0.1 * _randn(gen, *s.shape, dtype=F64) / math.sqrt(2 * max(s.shape[0], s.shape[2])) for s in sites]


def _split_inputs(case, seed):
    """A two-site node [left, 2, 2, right] with the decaying spectrum of a ground state (FP32)."""
    gen = _gen(seed)
    m, n = 2 * case["left"], 2 * case["right"]
    k = min(m, n)
    u = torch.linalg.qr(_randn(gen, m, k, dtype=F64).cpu())[0]
    v = torch.linalg.qr(_randn(gen, n, k, dtype=F64).cpu())[0]
    s = torch.exp(-torch.arange(k, dtype=F64) * (10.0 / k))
    node = (u * (s / torch.linalg.norm(s))) @ v.T
    return node.reshape(case["left"], 2, 2, case["right"]).float().to(DEV)


def _heff_inputs(case, seed):
    gen = _gen(seed)
    dl, dr = case["chi"], case["right"]
    mpo = _mpo(case["model"], 6)
    wl, wr = mpo[2].shape[0], mpo[3].shape[1]
    left = _randn(gen, dl, wl, dl) / math.sqrt(dl)
    right = _randn(gen, dr, wr, dr) / math.sqrt(dr)
    theta = _randn(gen, dl, 2, 2, dr) / math.sqrt(4 * dl * dr)
    return left, right, mpo[2], mpo[3], theta


def prepare(case, seed):
    kind = case["kind"]
    if kind == "edge":
        a, b, ia, ib = _edge_inputs(case, seed)
        return {"kind": kind, "a": a, "b": b, "ia": ia, "ib": ib, "out": _edge_out(case), "prec": case["prec"],
                "edges": case["edges"]}
    if kind == "sweep":
        psi = [s.float().contiguous() for s in _canonical_sites(_gen(seed), case["sites"], case["chi"])]
        return {"kind": kind, "sweep": tn.EnvSweep(psi, _mpo(case["model"], case["sites"]), prec=case["prec"])}
    if kind == "inner":
        psi, phi = _chain_pair(_gen(seed), case["sites"], case["chi"])
        return {"kind": kind, "psi": psi, "phi": phi, "prec": case["prec"]}
    if kind == "batch":
        gen = _gen(seed)
        chains = [_chain_pair(gen, n, chi) for n, chi in _batch_shapes(case)]
        return {"kind": kind, "batch": tn.BatchedInner(chains, prec=case["prec"])}
    if kind == "classify":
        sites, pixels, labels, shapes, sizes = _classify_inputs(case, seed)
        model = tn.MPSClassifier(case["sites"], case["sites"] // 2, LABELS, case["chi"], case["batch"])
        grad = torch.empty(sum(sizes), device=DEV) if case["train"] else None
        return {"kind": kind, "model": model, "sites": sites, "pixels": pixels, "labels": labels, "grad": grad,
                "dsites": [x.view(s) for x, s in zip(grad.split(sizes), shapes)] if case["train"] else None}
    if kind == "gauge":
        sites = _gauge_inputs(case, seed)
        sizes = [s.numel() for s in sites]
        flat = torch.cat([s.reshape(-1) for s in sites])
        work = torch.empty_like(flat)
        return {"kind": kind, "flat": flat, "work": work,
                "sites": [x.view(s.shape) for x, s in zip(work.split(sizes), sites)]}
    if kind == "split":
        return {"kind": kind, "node": _split_inputs(case, seed), "keep": case["keep"]}
    left, right, w1, w2, theta = _heff_inputs(case, seed)
    return {"kind": kind, "args": (left, right, w1, w2, theta), "out": torch.empty_like(theta), "prec": case["prec"]}


# ---------------------------------------------------------------------------
# one pass


def run(state):
    kind = state["kind"]
    if kind == "edge":
        # two edges: the result is written straight into its permuted layout
        out = state["out"] if state["edges"] == 1 else state["out"].permute(1, 2, 0)
        tn.contract_between(state["a"], state["b"], state["ia"], state["ib"], out=out, prec=state["prec"])
        return state["out"]
    if kind == "sweep":
        # the environments between the sites, which the next updates read
        s = state["sweep"].run()
        return {"L": s.L[1:-1], "R": s.R[1:-1]}
    if kind == "inner":
        # mantissa and log scale, kept in the program's own single precision
        return tn.mps_inner(state["psi"], state["phi"], prec=state["prec"]).float()
    if kind == "batch":
        return state["batch"].run().float()
    if kind == "classify":
        logits = state["model"].forward(state["sites"], state["pixels"])
        if state["dsites"] is None:
            return logits
        _, dlogits = tn.softmax_xent(logits, state["labels"])
        state["model"].backward(state["sites"], state["pixels"], dlogits, state["dsites"])
        return {"logits": logits, "dlogits": dlogits, "grad": state["grad"]}
    if kind == "gauge":
        # the call works in place: the program keeps the chain it came from
        state["work"].copy_(state["flat"])
        return {"lognorm": tn.mps_left_canonicalize(state["sites"]), "sites": state["work"]}
    if kind == "split":
        # the factors are unique up to signs only: the truncated node is what they stand for
        left, right, trun = tn.split_node(state["node"], [0, 1], [2, 3], max_singular_values=state["keep"])
        return {"node": tn.contract_between(left, right, [2], [0]), "dropped": trun}
    return tn.dmrg_apply_heff(*state["args"], out=state["out"], prec=state["prec"])


# ---------------------------------------------------------------------------
# the same in 64 bits


def _log_overlap(psi, phi):
    """(mantissa in [0.5, 1), natural log of its power of two) of the overlap."""
    env, log2 = torch.ones(1, 1, dtype=F64, device=DEV), 0.0
    for a, b in zip(psi, phi):
        t = torch.tensordot(env, b.double(), ([1], [0]))
        env = torch.tensordot(a.double(), t, ([0, 1], [0, 1]))
        top = float(env.abs().max())
        env, log2 = env / top, log2 + math.log2(top)
    v = float(env[0, 0])
    log2 += math.log2(abs(v))
    e = math.floor(log2) + 1
    return [math.copysign(2.0 ** (log2 - e), v), e * math.log(2.0)]


def _scores(sites, pixels, label_site):
    """Class scores of FP64 sites, one sample a row."""
    angle = 0.5 * math.pi * pixels.double()
    phi = torch.stack([torch.cos(angle), torch.sin(angle)], dim=2)      # [B, N, 2]

    def step(v, a, k):       # v[B, l], a[l, 2, r]
        t = torch.tensordot(v, a, ([1], [0]))
        return phi[:, k, 0, None] * t[:, 0] + phi[:, k, 1, None] * t[:, 1]

    n, one = len(sites), torch.ones(len(pixels), 1, dtype=F64, device=pixels.device)
    left, right = one, one
    for k in range(label_site):
        left = step(left, sites[k], k)
    for k in range(n - 1, label_site, -1):
        right = step(right, sites[k].permute(2, 1, 0), k)
    w = sites[label_site]                                                # [l, 2, labels, r]
    out = []
    for q in range(w.shape[2]):
        out.append((step(left, w[:, :, q], label_site) * right).sum(1))
    return torch.stack(out, dim=1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "edge":
        a, b, ia, ib = _edge_inputs(case, seed)
        r = torch.tensordot(a.double(), b.double(), (ia, ib))
        return r if case["edges"] == 1 else r.permute(2, 0, 1).contiguous()
    if kind == "sweep":
        psi = [s.float().double() for s in _canonical_sites(_gen(seed), case["sites"], case["chi"])]
        mpo, n = _mpo(case["model"], case["sites"], F64), case["sites"]
        env, lefts = torch.ones(1, 1, 1, dtype=F64, device=DEV), []
        for k in range(n - 1):
            t = torch.tensordot(env, psi[k], ([2], [0]))                  # a' u s b
            t = torch.tensordot(mpo[k], t, ([0, 3], [1, 2]))              # v t a' b
            env = torch.tensordot(psi[k], t, ([0, 1], [2, 1]))            # b' v b
            lefts.append(env)
        env, rights = torch.ones(1, 1, 1, dtype=F64, device=DEV), []
        for k in range(n - 1, 0, -1):
            t = torch.tensordot(psi[k], env, ([2], [2]))                  # a s b' v
            t = torch.tensordot(mpo[k], t, ([1, 3], [3, 1]))              # u t a b'
            env = torch.tensordot(psi[k], t, ([1, 2], [1, 3]))            # a' u a
            rights.append(env)
        return {"L": lefts, "R": rights[::-1]}
    if kind == "inner":
        return torch.tensor(_log_overlap(*_chain_pair(_gen(seed), case["sites"], case["chi"])), dtype=F64)
    if kind == "batch":
        gen = _gen(seed)
        return torch.tensor([_log_overlap(*_chain_pair(gen, n, chi)) for n, chi in _batch_shapes(case)], dtype=F64)
    if kind == "classify":
        sites, pixels, labels, _, _ = _classify_inputs(case, seed)
        sites = [s.double().requires_grad_(case["train"]) for s in sites]
        scores = _scores(sites, pixels, case["sites"] // 2)
        if not case["train"]:
            return scores
        scores.retain_grad()
        torch.nn.functional.cross_entropy(scores, labels).backward()
        return {"logits": scores.detach(), "dlogits": scores.grad,
                "grad": torch.cat([s.grad.reshape(-1) for s in sites])}
    if kind == "gauge":
        carry, out = torch.ones(1, 1, dtype=F64), []
        for s in _gauge_inputs(case, seed):
            x = torch.tensordot(carry, s.cpu(), ([1], [0]))
            q, r = torch.linalg.qr(x.reshape(-1, x.shape[2]))
            sign = torch.where(torch.diagonal(r) < 0, -1.0, 1.0).double()
            out.append((q * sign).reshape(-1))
            carry = r * sign[:, None]
        return {"lognorm": torch.log(carry[0]), "sites": torch.cat(out)}
    if kind == "split":
        node = _split_inputs(case, seed).double().cpu()
        u, s, v = torch.linalg.svd(node.reshape(2 * case["left"], 2 * case["right"]), full_matrices=False)
        k = min(case["keep"], len(s))
        return {"node": ((u[:, :k] * s[:k]) @ v[:k]).reshape(node.shape), "dropped": s[k:]}
    left, right, w1, w2, theta = (x.double() for x in _heff_inputs(case, seed))
    t = torch.tensordot(left, theta, ([2], [0]))                          # a' u s1 s2 b
    t = torch.tensordot(t, w1, ([1, 2], [0, 3]))                          # a' s2 b v t1
    t = torch.tensordot(t, w2, ([3, 1], [0, 3]))                          # a' b t1 x t2
    t = torch.tensordot(t, right, ([1, 3], [2, 1]))                       # a' t1 t2 b'
    return t.contiguous()


# ---------------------------------------------------------------------------
# what a pass cannot do without


def _chain_work(n, chi, copies):
    """Bytes of the sites and operations of one overlap."""
    dims = inputs.bond_dims(n, 2, chi)
    flops = sum(4 * dims[k] * dims[k + 1] * (dims[k] + dims[k + 1]) for k in range(n))
    return 4 * copies * sum(dims[k] * 2 * dims[k + 1] for k in range(n)), flops


def work(case):
    kind = case["kind"]
    if kind == "edge":
        a, w, b, c = case["left"], case["mid"], case["bond"], case["right"]
        m, k, n = (a * w, b, 2 * c) if case["edges"] == 1 else (a * w, 2 * b, c)
        return {"bytes": 4 * (m * k + k * n + m * n), "flops": 2 * m * n * k}
    if kind == "sweep":
        n, dims = case["sites"], inputs.bond_dims(case["sites"], 2, case["chi"])
        bond = 5 if case["model"] == "xxz" else 3
        w = [1] + [bond] * (n - 1) + [1]
        size = [4 * dims[k] * w[k] * dims[k] for k in range(n + 1)]
        flops = 0
        for k in range(n):
            a, b, u, v = dims[k], dims[k + 1], w[k], w[k + 1]
            flops += 4 * a * a * u * b + 4 * b * b * v * a + 8 * a * b * u * v     # one direction
            flops += 4 * a * b * b * v + 4 * a * a * b * u + 8 * a * b * u * v     # the other
        sites = 4 * sum(dims[k] * 2 * dims[k + 1] for k in range(n))
        return {"bytes": 2 * (sites + sum(size)), "flops": flops}
    if kind == "inner":
        b, f = _chain_work(case["sites"], case["chi"], 2)
        return {"bytes": b + 8, "flops": f}
    if kind == "batch":
        parts = [_chain_work(n, chi, 2) for n, chi in _batch_shapes(case)]
        return {"bytes": sum(b for b, _ in parts), "flops": sum(f for _, f in parts)}
    if kind == "classify":
        n, chi, batch = case["sites"], case["chi"], case["batch"]
        weights = (n - 3) * 2 * chi * chi + 4 * chi + 2 * LABELS * chi * chi
        # per sample and weight: a product and a sum forward, the same twice backward
        passes = 3 if case["train"] else 1
        return {"bytes": 4 * (weights * (2 if case["train"] else 1) + batch * (n + LABELS)),
                "flops": 2 * passes * batch * weights}
    if kind == "gauge":
        dims = inputs.bond_dims(case["sites"], 2, case["chi"])
        flops = nbytes = 0
        for k in range(case["sites"]):
            m, n = 2 * dims[k], dims[k + 1]
            # the carried triangle's product, the factorisation, and forming Q
            flops += dims[k] * m * n + 2 * (2 * m * n * n - 2 * n * n * n // 3)
            nbytes += 2 * 8 * m * n
        return {"bytes": nbytes, "flops": flops}
    if kind == "split":
        m, n, k = 2 * case["left"], 2 * case["right"], case["keep"]
        lo, hi = min(m, n), max(m, n)
        return {"bytes": 4 * 2 * m * n, "flops": 4 * hi * lo * lo + 17 * lo * lo * lo + 2 * m * n * k}
    l, r, w = case["chi"], case["right"], 5 if case["model"] == "xxz" else 3
    flops = 2 * l * l * w * 4 * r + 2 * l * r * 2 * (2 * w) * (2 * w) * 2 + 2 * l * 4 * r * w * r
    return {"bytes": 4 * (l * w * l + r * w * r + 8 * l * r), "flops": flops}
