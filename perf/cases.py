"""Performance cases: the calls a user of this framework makes, through its public entry points.

A case is a dict of plain values; ``listed()`` names the ones that are followed, ``draw(rng)`` gives further ones of
the same ranges.  ``prepare`` makes a case's inputs on the GPU, ``run`` is one pass, ``exact`` the same outputs in
64 bits by plain torch, ``work`` what a pass cannot do without.

Kinds and their ranges:

  product  C ~ max_k A_ik B_kj of uniform or log-normal operands, FP64 or BF16 path, FP32 or FP64 storage, batched or
           not, optionally balanced over the inner index; every dimension 32 ... 8192, up to 8192^3 multiply-adds
  grad     forward and backward of a batch of products (uniform operands, normal cotangent), every dimension 48 ... 768
  apsp     all-pairs shortest distances: sparse random digraphs on the FP64 path (256 ... 2048 vertices), random
           geometric graphs on the BF16 path (512 ... 4096 vertices), plain root or r = 1 projection
  maxconv  max-convolutions of b vector pairs, FP32 or FP64, 16 ... 8192 points each
  xy_topk  the k largest x_i + y_j with their indices, lists of 256 ... 8192, k 16 ... 256, plain or paired queue
"""

import math

import torch

import paper_1511_05690_amd as mt

DEV = "cuda"


def listed():
    return [
        # The smallest configuration the benchmark has: one product in FP64, a matter of latency.
        dict(name="product_256_fp64", kind="product", path="fp64", dtype="f64", b=1, m=256, k=256, n=256, dist="uniform",
             pmax=64, balance=False),
        # The smallest multi-tile call with no round size in it: launches and latency on the BF16 path.
        dict(name="product_ragged_small_bf16", kind="product", path="bf16", dtype="f32", b=1, m=257, k=513, n=255,
             dist="uniform", pmax=64, balance=False),
        # An everyday product, odd in every dimension, too small to fill the GPU with large tiles.
        dict(name="product_ragged_mid_bf16", kind="product", path="bf16", dtype="f32", b=1, m=1500, k=2050, n=1777,
             dist="lognormal", pmax=128, balance=False),
        # The headline product.
        dict(name="product_8192_bf16", kind="product", path="bf16", dtype="f32", b=1, m=8192, k=8192, n=8192,
             dist="lognormal", pmax=128, balance=False),
        # The accurate path at an ordinary large size.
        dict(name="product_4096_fp64", kind="product", path="fp64", dtype="f32", b=1, m=4096, k=4096, n=4096,
             dist="lognormal", pmax=128, balance=False),
        # A training step through the product: the batched gradient configuration, p* selected.
        dict(name="grad_64x512_bf16", kind="grad", path="bf16", dtype="f32", b=64, m=512, k=512, n=512, pmax=64),
        # A small accurate gradient with odd sizes.
        dict(name="grad_ragged_fp64", kind="grad", path="fp64", dtype="f64", b=6, m=300, k=257, n=201, pmax=64),
        # All-pairs shortest paths of a sparse random digraph on the accurate path (11 squarings).
        dict(name="apsp_er2048_fp64", kind="apsp", path="fp64", graph="er", n=2048, pmax=512, projection=""),
        # Shortest paths of a geometric graph on the fast path, the projected estimate its long paths need.
        dict(name="apsp_rgg3500_bf16_r1", kind="apsp", path="bf16", graph="rgg", n=3500, pmax=128, projection="r1"),
        # Max-product inference: many pairs of probability vectors.
        dict(name="maxconv_8192x2048_fp64", kind="maxconv", dtype="f64", b=8192, n=2048, m=2048, dist="distribution",
             pmax=64),
        # A few long vectors of odd lengths.
        dict(name="maxconv_long_fp32", kind="maxconv", dtype="f32", b=48, n=6001, m=3500, dist="uniform", pmax=64),
        # The top 256 of x + y at the larger list size of the paper, indices from the paired queue.
        dict(name="xy_topk_8192_paired", kind="xy_topk", dtype="f64", n=8192, k=256, spread=1.0, paired=True),
    ]


def _size(rng, lo, hi):
    """A size of lo ... hi, even over its logarithm; most are odd or not a multiple of a tile."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return min(hi, max(lo, v if rng.random() < 0.8 else (v + 31) // 32 * 32))


def draw(rng):
    kind = rng.choice(["product", "product", "product", "grad", "apsp", "maxconv", "xy_topk"])
    if kind == "product":
        path = rng.choice(["bf16", "bf16", "fp64"])
        most = 8192 if path == "bf16" else 4096
        b = rng.choice([1, 1, 1, 4, 16])
        while True:
            m, k, n = (_size(rng, 32, most) for _ in range(3))
            if b * m * k * n <= most ** 3 and b * (m * k + k * n + m * n) <= 3 * 8192 ** 2:
                break
        return dict(kind=kind, path=path, dtype=rng.choice(["f32", "f64"]) if path == "fp64" else "f32", b=b, m=m, k=k,
                    n=n, dist=rng.choice(["uniform", "lognormal"]), pmax=rng.choice([64, 128]),
                    balance=rng.random() < 0.15)
    if kind == "grad":
        path = rng.choice(["bf16", "fp64"])
        m, k, n = (_size(rng, 48, 768) for _ in range(3))
        return dict(kind=kind, path=path, dtype="f32" if path == "bf16" else "f64", b=_size(rng, 1, 32 if path == "bf16" else 8),
                    m=m, k=k, n=n, pmax=64)
    if kind == "apsp":
        path = rng.choice(["bf16", "fp64"])
        return dict(kind=kind, path=path, graph="rgg" if path == "bf16" else "er",
                    n=_size(rng, 512, 4000) if path == "bf16" else _size(rng, 256, 2047),
                    pmax=128 if path == "bf16" else 512, projection=rng.choice(["", "r1"]))
    if kind == "maxconv":
        n, m = _size(rng, 16, 8192), _size(rng, 16, 8192)
        most = max(1, min(8192, 2 ** 24 // (n + m) if n + m - 1 <= 4096 else 2 ** 20 // (n + m)))
        return dict(kind=kind, dtype=rng.choice(["f32", "f64"]), b=_size(rng, 1, most), n=n, m=m,
                    dist=rng.choice(["uniform", "distribution"]), pmax=64)
    return dict(kind=kind, dtype=rng.choice(["f32", "f64"]), n=_size(rng, 256, 8192), k=_size(rng, 16, 256), spread=1.0,
                paired=rng.random() < 0.5)


# ------------------------------------------------------------------ inputs
def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _dtype(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


def _uniform(shape, g):
    return 1.0 - torch.rand(shape, generator=g, device=DEV, dtype=torch.float64)  # (0, 1]


def _operands(case, g):
    """The operands of a product: uniform on (0, 1], or exp(N(0, 2^2)) up to 10^6; where they are to be balanced,
    their inner index carries 16 decades of scale, in A and against it in B."""
    shape_a, shape_b = (case["b"], case["m"], case["k"]), (case["b"], case["k"], case["n"])
    if case["b"] == 1:
        shape_a, shape_b = shape_a[1:], shape_b[1:]
    if case.get("dist", "uniform") == "lognormal":
        a, b = (torch.randn(s, generator=g, device=DEV, dtype=torch.float64).mul_(2.0).exp_().clamp_(max=1e6)
                for s in (shape_a, shape_b))
    else:
        a, b = _uniform(shape_a, g), _uniform(shape_b, g)
    if case.get("balance"):
        scale = 10.0 ** (16.0 * torch.rand(case["k"], generator=g, device=DEV, dtype=torch.float64) - 8.0)
        a, b = a * scale, b / scale[:, None]
    return a.to(_dtype(case)), b.to(_dtype(case))


def _graph(case, g):
    """Weights of a digraph with edges of weight U[0, 10) at probability 0.05, or of a geometric graph in the unit
    square whose vertices have about 20 neighbours, weight 100 x length."""
    n = case["n"]
    inf = torch.full((), math.inf, device=DEV)
    if case["graph"] == "er":
        edge = torch.rand((n, n), generator=g, device=DEV) < 0.05
        w = torch.where(edge, 10.0 * torch.rand((n, n), generator=g, device=DEV), inf)
    else:
        pts = torch.rand((n, 2), generator=g, device=DEV, dtype=torch.float64)
        d = ((pts[:, None, 0] - pts[None, :, 0]) ** 2 + (pts[:, None, 1] - pts[None, :, 1]) ** 2).sqrt_()
        w = torch.where(d < 2.56 / math.sqrt(n), (100.0 * d).float(), inf)
    w.fill_diagonal_(0.0)
    return w.float()


def _vectors(case, g):
    shapes = (case["b"], case["n"]), (case["b"], case["m"])
    if case["dist"] == "distribution":  # Dirichlet(1) rows
        v = [torch.rand(s, generator=g, device=DEV, dtype=torch.float64).clamp_(min=1e-300).log_().neg_() for s in shapes]
        v = [t / t.sum(-1, keepdim=True) for t in v]
    else:
        v = [_uniform(s, g) for s in shapes]
    return [t.to(_dtype(case)) for t in v]


def _lists(case, g):
    return [(case["spread"] * torch.rand(case["n"], generator=g, device=DEV, dtype=torch.float64)).to(_dtype(case))
            for _ in range(2)]


def _scale(case):
    """The transform scale s of exp(-s w): 1, or 0.35 where the distances reach about 140."""
    return 1.0 if case["graph"] == "er" else 0.35


def prepare(case, seed):
    g = _generator(seed)
    s = {"case": case, "P": mt.pfamily(case["pmax"]) if "pmax" in case else None}
    if case["kind"] == "product":
        s["A"], s["B"] = _operands(case, g)
    elif case["kind"] == "grad":
        a, b = _operands(case, g)
        s["A"], s["B"] = a.requires_grad_(), b.requires_grad_()
        shape = a.shape[:-1] + b.shape[-1:]
        s["G"] = torch.randn(shape, generator=g, device=DEV, dtype=torch.float64).to(_dtype(case))
    elif case["kind"] == "apsp":
        s["W"] = _graph(case, g)
    elif case["kind"] == "maxconv":
        s["x"], s["y"] = _vectors(case, g)
    else:
        s["x"], s["y"] = _lists(case, g)
    return s


# ------------------------------------------------------------------ one pass
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "product":
        return mt.estimate(state["A"], state["B"], P=state["P"], path=case["path"], balance=case["balance"])
    if kind == "grad":
        c = mt.estimate(state["A"], state["B"], P=state["P"], path=case["path"])
        da, db = torch.autograd.grad(c, (state["A"], state["B"]), state["G"])
        return {"C": c.detach(), "dA": da, "dB": db}
    if kind == "apsp":
        return mt.apsp(state["W"], s=_scale(case), P=state["P"], path=case["path"], projection=case["projection"] or None)
    if kind == "maxconv":
        return mt.maxconv(state["x"], state["y"], P=state["P"])
    v, i, j = mt.xy_topk(state["x"], state["y"], case["k"], paired=case["paired"])
    return {"values": v, "i": i, "j": j}


# ------------------------------------------------------------------ the same in 64 bits
TAU = {"bf16": 1e-30, "fp64": 1e-290}
TAU_CONV = 1e-12


def _power(x, p):
    """x ** p for a power of two p."""
    while p > 1:
        x = x * x
        p //= 2
    return x


def _ratio(x, s):
    return torch.where(s > 0, x / torch.where(s > 0, s, 1.0), 0.0)


def _largest_stable(ring, family, tau, projection=""):
    """S^(1/p) at the largest p of the family with S = ring(p) >= tau (at the smallest p where there is none) and
    that p; with projection "r1" (S_p / S_q)^(1 / (p - q)) with the next smaller p, q, in its place."""
    out = chosen = above = None
    for p in sorted(family, reverse=True):
        s = ring(p)
        if out is None:
            out, chosen = torch.zeros_like(s), torch.zeros(s.shape, dtype=torch.int32, device=s.device)
        if above is not None:  # entries chosen at the p above, now that S at the next smaller one is known
            q, s_above = above
            fix = (chosen == q) & (s > 0)
            out = torch.where(fix, (s_above / s.clamp(min=1e-320)) ** (1.0 / (q - p)), out)
        take = (chosen == 0) & ((s >= tau) | (p == min(family)))
        out = torch.where(take, s.clamp(min=0.0) ** (1.0 / p), out)
        chosen = torch.where(take, p, chosen)
        above = (p, s) if projection == "r1" else None
    return out, chosen


def _scaled_product(a, b, family, tau):
    """The estimate of max_k a_ik b_kj and the p of each entry."""
    r, c = a.amax(-1, keepdim=True), b.amax(-2, keepdim=True)
    a, b = _ratio(a, r), _ratio(b, c)
    root, p = _largest_stable(lambda p: torch.matmul(_power(a, p), _power(b, p)), family, tau)
    return r, c, a, b, root, p


def _exact_product(case, state):
    a, b = state["A"].double(), state["B"].double()
    if case["balance"]:
        am, bm = a.amax(-2), b.amax(-1)
        d = torch.where((am > 0) & (bm > 0), (bm / am).sqrt(), 1.0)
        a, b = a * d[..., None, :], b / d[..., :, None]
    r, c, _, _, root, _ = _scaled_product(a, b, state["P"], TAU[case["path"]])
    return r * c * root


def _exact_grad(case, state):
    a, b, g = state["A"].detach().double(), state["B"].detach().double(), state["G"].double()
    r, c, a, b, root, p = _scaled_product(a, b, state["P"], TAU[case["path"]])
    da, db = torch.zeros_like(a), torch.zeros_like(b)
    for q in state["P"]:
        w = torch.where((p == q) & (root > 0), g * root.clamp(min=1e-300) ** (1.0 - q), 0.0)
        if bool((w != 0).any()):
            da += a ** (q - 1) * torch.matmul(w * c, _power(b, q).transpose(-1, -2))
            db += b ** (q - 1) * torch.matmul(_power(a, q).transpose(-1, -2), w * r)
    return {"C": r * c * root, "dA": da, "dB": db}


def _exact_apsp(case, state):
    x = torch.exp(-_scale(case) * state["W"].double())
    for _ in range(max(0, (case["n"] - 1).bit_length())):
        root, _ = _largest_stable(lambda p: _power(x, p) @ _power(x, p), state["P"], TAU[case["path"]],
                                  case["projection"])
        x = root.clamp(max=1.0).fill_diagonal_(1.0)
    return -torch.log(x) / _scale(case)


def _exact_maxconv(case, state):
    x, y = state["x"].double(), state["y"].double()
    n, m = case["n"], case["m"]
    rows = max(1, (1 << 29) // (n * (n + m - 1)))  # pairs at a time: their windows take 4 GiB
    out = []
    for at in range(0, case["b"], rows):
        u, v = x[at:at + rows], y[at:at + rows]
        ux, vy = u.amax(-1, keepdim=True), v.amax(-1, keepdim=True)
        u, v = u / ux, v / vy

        def ring(p):  # sum_i u_i^p v_(t-i)^p, by its definition
            windows = torch.nn.functional.pad(_power(v, p), (n - 1, n - 1)).unfold(-1, n, 1)
            return torch.matmul(windows, _power(u, p).flip(-1)[..., None])[..., 0]

        out.append(ux * vy * _largest_stable(ring, state["P"], TAU_CONV)[0])
    return torch.cat(out)


def _exact_topk(case, state):
    """The k largest sums themselves: the queue's values estimate them.  The indices have no 64-bit counterpart."""
    x, y = state["x"].double(), state["y"].double()
    top = torch.topk(x, min(case["k"], case["n"])).values[:, None] + torch.topk(y, min(case["k"], case["n"])).values
    return {"values": torch.topk(top.flatten(), case["k"]).values, "i": None, "j": None}


def exact(case, seed):
    state = prepare(case, seed)
    return {"product": _exact_product, "grad": _exact_grad, "apsp": _exact_apsp, "maxconv": _exact_maxconv,
            "xy_topk": _exact_topk}[case["kind"]](case, state)


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    """One ring product (or convolution) at each entry's own p: the operands read and the result written once."""
    size = 8 if case.get("dtype") == "f64" else 4
    if case["kind"] in ("product", "grad"):
        b, m, k, n = (case[t] for t in "bmkn")
        values, products = b * (m * k + k * n + m * n), b * m * k * n
        if case["kind"] == "grad":  # A, B, G read; C, dA, dB written; the products for C, dA and dB
            return {"bytes": 2 * size * values, "flops": 6 * products}
        return {"bytes": size * values, "flops": 2 * products}
    if case["kind"] == "apsp":
        n = case["n"]
        return {"bytes": 8 * n * n, "flops": 2 * n ** 3 * max(1, (n - 1).bit_length())}
    n, m = case["n"], case.get("m", case["n"])
    log = max(4, (n + m - 2).bit_length())
    transforms = 3 * 2.5 * (1 << log) * log  # three real transforms of one convolution
    if case["kind"] == "maxconv":
        return {"bytes": size * case["b"] * (n + m + n + m - 1), "flops": transforms * case["b"]}
    return {"bytes": size * 2 * n + 16 * case["k"], "flops": transforms * len(mt.XY_FAMILY)}
