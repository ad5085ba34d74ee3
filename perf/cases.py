"""The work that a program has this library do, as measurable cases.

Every case goes through the package's public entry points on inputs made on
the GPU from a seed: Gaussian random fields whose per-mode power falls as
k^-3 (the shape of the simulation outputs the method is meant for) or, for
the FP64 fields, k^-11/3 with a sharp front, with two boxes (or the strongest
gradients) held to a tight bound and the rest to a loose one.

Kinds of pass (``case["kind"]``):

=============  ==============================================================
``quantize``   a field to codes: ``Plan.decompose_quantize``
``restore``    codes to a field: ``Plan.dequantize_recompose``
``step``       both, one after the other
``insitu``     both under a tolerance map made anew in the pass
``transform``  ``Plan.decompose`` and ``Plan.recompose`` without quantization
``grad``       the autograd form: decompose, recompose and both backwards
``qoi``        per-node widths for a quantity of interest, then codes
``batch``      a list of fields of mixed shapes: ``Batch``, graph replay
``paper8``     both directions of the 8^3 block form: ``Paper8Plan``
``compress``   a field to a container in a pinned buffer the program keeps
``decompress`` such a container to a field
=============  ==============================================================
"""
import math
import random

import torch

from paper_2609_00205_amd import Batch, Paper8Plan, Plan, autograd, decompress

DTYPES = {"f32": torch.float32, "f64": torch.float64}
ESIZE = {"f32": 4, "f64": 8}


def _case(kind, shape, dtype="f32", block=17, L=1, M=2, nested=False, pad="clamp", kept=False, name=None, **more):
    c = {"kind": kind, "nz": shape[0], "ny": shape[1], "nx": shape[2], "dtype": dtype, "block": block, "L": L, "M": M,
         "nested": nested, "pad": pad, "kept": kept}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The plain method on a small field, every level global: the smallest
        # call, bound by launches and latency.
        _case("step", (65, 65, 65), L=0, M=6, name="step-65-global"),
        # One variable of a small simulation, its region of interest moving
        # from step to step: the map is made and propagated in each pass.
        _case("insitu", (129, 129, 129), name="insitu-129"),
        # The default workload, each direction by itself: 512^3 FP32, one
        # block level and two global levels, the map fixed over the run.
        _case("quantize", (512, 512, 512), kept=True, name="quantize-512"),
        _case("restore", (512, 512, 512), kept=True, name="restore-512"),
        # A field whose dims tile nothing, transform only, deeper hierarchy.
        _case("transform", (98, 1200, 1200), L=2, M=2, name="transform-98x1200x1200"),
        # Training or sensitivity analysis through the transform, ragged dims.
        _case("grad", (100, 500, 500), name="grad-100x500x500"),
        # Bounds for a mean over a box of the field.
        _case("qoi", (384, 384, 256), name="qoi-384x384x256"),
        # Many fields of mixed sizes at once, replayed from a graph.
        _case("batch", (257, 257, 257), L=-1, M=0, fields=32, name="batch-32"),
        # The largest: a double-precision turbulence field with a front, the
        # steepest voxels held tight, block level only.
        _case("step", (1024, 1024, 512), dtype="f64", L=1, M=0, name="step-f64-1024x1024x512"),
        # The disjoint 8^3 block form with its hybrid hierarchy.
        _case("paper8", (512, 512, 512), L=1, M=2, name="paper8-512"),
        # Whole containers, writing and reading.
        _case("compress", (256, 384, 384), dtype="f64", L=1, M=2, name="compress-f64-256x384x384"),
        _case("decompress", (512, 512, 512), name="decompress-512"),
    ]


#: Kinds drawn, and the most voxels of each (less than its listed case, or than
#: the largest listed pass would take).
_DRAWN = {"step": 512 ** 3, "insitu": 512 ** 3, "quantize": 512 ** 3, "restore": 512 ** 3, "transform": 512 ** 3,
          "grad": 300 ** 3, "qoi": 300 ** 3, "batch": 257 ** 3, "paper8": 400 ** 3, "compress": 300 ** 3,
          "decompress": 320 ** 3}


def _shape(rng, most):
    """Dims whose product is spread over its logarithm between 33^3 and
    `most`, of uneven sides, each between 20 and 1100."""
    v = math.exp(rng.uniform(math.log(33 ** 3), math.log(0.9 * most)))
    side = v ** (1.0 / 3.0)
    a, b = math.exp(rng.uniform(-0.6, 0.6)), math.exp(rng.uniform(-0.6, 0.6))
    dims = [side * a, side * b, side / (a * b)]
    rng.shuffle(dims)
    dims = [min(1100, max(20, int(round(d)))) for d in dims]
    while dims[0] * dims[1] * dims[2] > most:
        k = dims.index(max(dims))
        dims[k] = max(20, int(0.9 * dims[k]))
    return tuple(dims)


def draw(rng):
    kind = rng.choice(sorted(_DRAWN))
    dtype = rng.choice(["f32", "f32", "f64"])
    shape = _shape(rng, _DRAWN[kind] // (2 if dtype == "f64" else 1))
    if kind == "paper8":
        return _case(kind, shape, dtype=dtype, L=rng.choice([1, 1, 2, 3]), M=rng.choice([0, 2]))
    if kind == "batch":
        return _case(kind, (257, 257, 257), dtype=dtype, block=17, L=-1, M=rng.choice([0, 0, 1]),
                     nested=rng.random() < 0.2, fields=rng.randint(4, 24), shapes=rng.randint(1, 10 ** 6))
    block = rng.choice([17, 17, 17, 17, 9, 33])
    L, M = rng.choice([1, 1, 1, 2]), rng.choice([0, 1, 2, 2, 3])
    if rng.random() < 0.15 and shape[0] * shape[1] * shape[2] <= 256 ** 3:
        L, M = 0, rng.choice([2, 3, 4])
    nested = block == 17 and L == 2 and rng.random() < 0.5
    return _case(kind, shape, dtype=dtype, block=block, L=L, M=M, nested=nested,
                 pad="zero" if rng.random() < 0.1 else "clamp", kept=kind != "insitu" and rng.random() < 0.5)


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------


def _field(shape, dtype, gen, front=False):
    """Mean 0, std 1, per-mode power k^-3 (or, with a front, k^-11/3 plus
    2 tanh across a random plane)."""
    f = torch.fft.rfftn(torch.randn(shape, dtype=dtype, device="cuda", generator=gen))
    k2 = sum((torch.fft.fftfreq(n, 1.0 / n, device="cuda", dtype=dtype) if a < 2 else
              torch.fft.rfftfreq(n, 1.0 / n, device="cuda", dtype=dtype)).square().reshape([-1 if i == a else 1
                                                                                          for i in range(3)])
             for a, n in enumerate(shape))
    k2[0, 0, 0] = 1.0
    f *= k2.pow_(-(11.0 / 12.0 if front else 0.75))
    f[0, 0, 0] = 0.0
    del k2
    x = torch.fft.irfftn(f, s=shape)
    del f
    x -= x.mean()
    x /= x.std()
    if front:
        nv = torch.randn(3, dtype=torch.float64, device="cuda", generator=gen)
        nv = (nv / nv.norm()).tolist()
        r = [(torch.arange(n, device="cuda", dtype=dtype) - (n - 1) / 2.0) * v for n, v in zip(shape, nv)]
        x += 2.0 * torch.tanh((r[0][:, None, None] + r[1][None, :, None] + r[2][None, None, :]) / 2.0)
    return x.contiguous()


def _boxes(shape, rng, count, part):
    """`count` boxes of 1/part of each side at random origins."""
    out = []
    for _ in range(count):
        e = [max(4, n // part) for n in shape]
        o = [rng.randrange(0, max(1, n - k + 1)) for n, k in zip(shape, e)]
        out.append(tuple(o) + tuple(a + k for a, k in zip(o, e)))
    return out


def _steep(x):
    """Voxels above the 95th percentile of |grad x|."""
    g = torch.zeros_like(x)
    for a in range(3):
        n = x.shape[a]
        d = (x.narrow(a, 2, n - 2) - x.narrow(a, 0, n - 2)).mul_(0.5)
        g.narrow(a, 1, n - 2).add_(d.square_())
    some = g.reshape(-1)[:: max(1, g.numel() // 1000003)]
    return g > torch.sort(some).values[int(0.95 * some.numel())]


def _tols(case, boxes, scale):
    """(tight boxes with their bound, loose bound) of a case."""
    tight = 1e-6 if case["dtype"] == "f64" else 1e-5
    loose = 1e-3 if case["dtype"] == "f64" or case["kind"] == "batch" else 1e-2
    return [b + (tight * scale,) for b in boxes], loose * scale


def _batch_shapes(case):
    r = random.Random(case.get("shapes", 4))
    return [tuple(r.choice([33, 65, 129, 257]) for _ in range(3)) for _ in range(case["fields"])]


def _inputs(case, seed):
    """(field, other inputs, tight boxes, loose bound) of a case on one field."""
    gen, rng = torch.Generator(device="cuda"), random.Random(seed)
    gen.manual_seed(seed)
    shape, dtype = (case["nz"], case["ny"], case["nx"]), DTYPES[case["dtype"]]
    x = _field(shape, dtype, gen, _steep_kind(case))
    more = {}
    if case["kind"] == "grad":
        full = [_padded(n, case) for n in shape]
        more = {"gc": torch.randn(full, dtype=dtype, device="cuda", generator=gen),
                "gx": torch.randn(shape, dtype=dtype, device="cuda", generator=gen)}
    return (x, more) + _tols(case, _boxes(shape, rng, 2, 8), float(x.abs().max()))


def _steep_kind(case):
    """The FP64 steps run on turbulence with a front, its steepest voxels held tight."""
    return case["kind"] == "step" and case["dtype"] == "f64"


def _prepare_batch(case, seed):
    gen, rng = torch.Generator(device="cuda"), random.Random(seed)
    gen.manual_seed(seed)
    shapes, dtype = _batch_shapes(case), DTYPES[case["dtype"]]
    b = Batch(shapes, dtype=dtype, block=case["block"], L=None if case["L"] < 0 else case["L"], M=case["M"],
              nested=case["nested"])
    xs = [_field(s, dtype, gen) for s in shapes]
    tols = [p.tolmap_from_boxes(*_tols(case, _boxes(p.shape, rng, 1, 4), float(x.abs().max())))
            for p, x in zip(b.plans, xs)]
    return {"kind": "batch", "batch": b, "xs": xs, "tols": tols, "outs": [torch.empty_like(x) for x in xs],
            "codes": [torch.empty(p.coeff_shape, dtype=torch.int32, device="cuda") for p in b.plans]}


def prepare(case, seed):
    kind, dtype, shape = case["kind"], DTYPES[case["dtype"]], (case["nz"], case["ny"], case["nx"])
    if kind == "batch":
        return _prepare_batch(case, seed)
    x, more, boxes, loose = _inputs(case, seed)
    st = {"kind": kind, "x": x, **more}
    if kind == "paper8":
        st["plan"] = p = Paper8Plan(shape, dtype=dtype, L=case["L"], M=case["M"])
        vt = torch.full(shape, loose, dtype=torch.float64, device="cuda")
        for z0, y0, x0, z1, y1, x1, t in boxes:
            vt[z0:z1, y0:y1, x0:x1] = t
        st.update(tol=p.tolmap_from_voxels(vt), out=torch.empty_like(x),
                  codes=torch.empty(p.coeff_size, dtype=torch.int32, device="cuda"))
        return st
    st["plan"] = p = Plan(shape, dtype=dtype, block=case["block"], L=case["L"], M=case["M"], pad_mode=case["pad"],
                          nested=case["nested"])
    if kind == "grad":
        x.requires_grad_()
        return st
    if kind in ("transform", "qoi"):
        st["coeff"] = torch.empty(p.coeff_shape, dtype=dtype, device="cuda")
    if kind == "transform":
        st["out"] = torch.empty_like(x)
        return st
    if kind == "insitu":
        st.update(boxes=boxes, loose=loose)
    elif kind == "qoi":
        scale = float(x.abs().max())
        g = torch.zeros_like(x)
        box = tuple(slice(3 * n // 8, 5 * n // 8) for n in shape)
        g[box] = 1.0 / g[box].numel()
        st.update(g=g, tol_q=1e-6 * scale, tol=p.tolmap_from_boxes([], 1e-3 * scale))
    elif _steep_kind(case):
        st["tol"] = p.tolmap_from_voxels(torch.where(_steep(x), boxes[0][6], loose).to(torch.float64))
    else:
        st["tol"] = p.tolmap_from_boxes(boxes, loose)
    if case["kept"]:
        p.quant_prepare(st["tol"])
    if kind in ("compress", "decompress"):
        room = math.prod(p.coeff_shape) * x.element_size() * 5 // 4 + st["tol"].numel() * 8 + (1 << 20)
        st["host"] = host = torch.zeros(room, dtype=torch.uint8, pin_memory=True)
        if kind == "decompress":
            st["buf"] = host[: p.compress(x, st["tol"], out=host).nbytes]
            del st["x"], st["host"]
        return st
    st["codes"] = torch.empty(p.coeff_shape, dtype=torch.int32, device="cuda")
    if kind == "restore":
        p.decompose_quantize(x, st["tol"], codes=st["codes"], check=False)
        del st["x"]
    if kind not in ("quantize", "qoi"):
        st["out"] = torch.empty(shape, dtype=dtype, device="cuda")
    return st


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------


def run(st):
    kind, p = st["kind"], st.get("plan")
    if kind == "quantize":
        return p.decompose_quantize(st["x"], st["tol"], codes=st["codes"], check=False)
    if kind == "restore":
        return p.dequantize_recompose(st["codes"], st["tol"], out=st["out"])
    if kind == "step":
        p.decompose_quantize(st["x"], st["tol"], codes=st["codes"], check=False)
        return st["codes"], p.dequantize_recompose(st["codes"], st["tol"], out=st["out"])
    if kind == "insitu":
        tol = p.tolmap_from_boxes(st["boxes"], st["loose"])
        p.decompose_quantize(st["x"], tol, codes=st["codes"], check=False)
        return tol, st["codes"], p.dequantize_recompose(st["codes"], tol, out=st["out"])
    if kind == "transform":
        p.decompose(st["x"], out=st["coeff"])
        return st["coeff"], p.recompose(st["coeff"], out=st["out"])
    if kind == "grad":
        c = autograd.decompose(st["x"], p)
        gx, = torch.autograd.grad(c, st["x"], st["gc"])
        leaf = c.detach().requires_grad_()
        y = autograd.recompose(leaf, p)
        gc, = torch.autograd.grad(y, leaf, st["gx"])
        return c.detach(), gx, y.detach(), gc
    if kind == "qoi":
        delta, n = p.qoi_deltas(st["g"], st["tol_q"], st["tol"])
        p.decompose(st["x"], out=st["coeff"])
        codes, _ = p.quantize_delta(st["coeff"], delta, codes=st["codes"], stats=False)
        return delta, n, codes
    if kind == "batch":
        st["batch"].decompose_quantize(st["xs"], st["tols"], codes=st["codes"], use_graph=True)
        st["batch"].dequantize_recompose(st["codes"], st["tols"], outs=st["outs"], use_graph=True)
        return st["codes"], st["outs"]
    if kind == "paper8":
        p.decompose_quantize(st["x"], st["tol"], codes=st["codes"])
        return st["codes"], p.dequantize_recompose(st["codes"], st["tol"], out=st["out"])
    if kind == "compress":
        return p.compress(st["x"], st["tol"], out=st["host"]).nbytes, st["host"]  # the bytes after the container are 0
    return decompress(st["buf"])


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------


def _padded(n, case):
    """Smallest length >= n that the case's block levels tile and its global
    levels halve."""
    b, L, M = case["block"], max(0, case["L"]), case["M"]
    unit = 1 if L == 0 else (b - 1) if case["nested"] else (b - 1) << (L - 1)
    m = max(n, b if L else 1)
    while True:
        k = (m - 1) // (1 << L) + 1
        ok = (m - 1) % unit == 0
        for _ in range(M):
            if k > 2 and k % 2 == 0:
                ok = False
            k = k if k <= 2 else (k + 1) // 2
        if ok:
            return m
        m += 1


def work(case):
    """Each input read and each output written once; about 20 operations per
    node and direction (interpolation, restriction and solve of three axes)."""
    es, kind = ESIZE[case["dtype"]], case["kind"]
    shape = (case["nz"], case["ny"], case["nx"])
    if kind == "batch":
        n = npad = sum(a * b * c for a, b, c in _batch_shapes(case))
    elif kind == "paper8":
        n, npad, dims = math.prod(shape), 0, shape
        for _ in range(case["L"]):
            dims = [8 * ((d + 7) // 8) for d in dims]
            npad += math.prod(dims)
            dims = [d // 8 * 5 for d in dims]
        npad += math.prod(dims)
    else:
        n, npad = math.prod(shape), math.prod(_padded(d, case) for d in shape)
    once = n * es + 4 * npad
    byt, dirs = {"quantize": (once, 1), "restore": (once, 1), "transform": (2 * es * (n + npad), 2),
                 "grad": (4 * es * (n + npad), 4), "qoi": (2 * es * n + 12 * npad, 2),
                 "compress": (n * es + 1.3 * npad, 1), "decompress": (n * es + 1.3 * npad, 1)}.get(kind, (2 * once, 2))
    return {"bytes": byt, "flops": 20 * npad * dirs}


# --------------------------------------------------------------------------
# the transform in 64 bits, by dense matrices per axis
# --------------------------------------------------------------------------


def _even(n):
    """Indices of the coarse nodes of an n-node axis."""
    return list(range(n)) if n <= 2 else sorted(set(range(0, n, 2)) | {n - 1})


def _ops(dims, fixed, device):
    """Per axis (coarse indices, P, K) of one level on unit-spaced nodes:
    linear interpolation from the even nodes and the last, and the L2
    correction K = Mc^-1 P^T M (its end rows zero where the ends are fixed)."""
    out = []
    for n in dims:
        idx = _even(n)
        m = len(idx)
        P, K = torch.zeros(n, m, dtype=torch.float64), torch.zeros(m, n, dtype=torch.float64)

        def mass(c):
            h = torch.tensor(c, dtype=torch.float64).diff()
            d = torch.zeros(len(c), dtype=torch.float64)
            d[:-1] += h / 3.0
            d[1:] += h / 3.0
            return torch.diag(d) + torch.diag(h / 6.0, 1) + torch.diag(h / 6.0, -1)

        if n <= 2:
            P, K = torch.eye(n, dtype=torch.float64), torch.eye(n, dtype=torch.float64)
        else:
            for j, (lo, hi) in enumerate(zip(idx, idx[1:])):
                for i in range(lo, hi + 1):
                    P[i, j], P[i, j + 1] = (hi - i) / (hi - lo), (i - lo) / (hi - lo)
            P[idx] = torch.eye(m, dtype=torch.float64)
            rows = slice(1, m - 1) if fixed else slice(0, m)
            K[rows] = torch.linalg.solve(mass(idx)[rows, rows], (P.T @ mass(list(range(n))))[rows])
        out.append((torch.tensor(idx, device=device), P.to(device), K.to(device)))
    return out


def _three(ops, which, t):
    """An operator of each of the last three axes applied."""
    for a in (2, 1, 0):
        t = (t.movedim(a - 3, -1) @ ops[a][which].T).movedim(-1, a - 3)
    return t


def _pick(t, ops):
    for a in range(3):
        t = t.index_select(t.dim() + a - 3, ops[a][0])
    return t


def _put(t, c, ops):
    """t with c at the coarse nodes."""
    keep = torch.ones(t.shape[-3:], dtype=torch.bool, device=t.device)
    keep[torch.meshgrid(*(o[0] for o in ops), indexing="ij")] = False
    for a in range(3):
        shape = list(c.shape)
        shape[a - 3] = t.shape[a - 3]
        c = c.new_zeros(shape).index_add(c.dim() + a - 3, ops[a][0], c)
    return torch.where(keep, t, c)


def _level_down(u, fixed):
    """Details with the corrected values at the coarse nodes, on the last three axes."""
    ops = _ops(u.shape[-3:], fixed, u.device)
    uc = _pick(u, ops)
    w = _put(u - _three(ops, 1, uc), torch.zeros_like(uc), ops)
    return _put(w, uc + _three(ops, 2, w), ops)


def _level_up(o, fixed):
    ops = _ops(o.shape[-3:], fixed, o.device)
    c = _pick(o, ops)
    w = _put(o, torch.zeros_like(c), ops)
    return _three(ops, 1, c - _three(ops, 2, w)) + w


def _blocks(fn, u, b):
    """fn on every b^3 block of a grid whose blocks share their faces."""
    t = fn(u.unfold(0, b, b - 1).unfold(1, b, b - 1).unfold(2, b, b - 1)).permute(0, 3, 1, 4, 2, 5)
    for a in (4, 2, 0):  # joined along each axis: all but the last node of every block, then the far face
        t = torch.cat([t.narrow(a + 1, 0, b - 1).flatten(a, a + 1), t.select(a, -1).narrow(a, b - 1, 1)], a)
    return t


def _level(fn, t, case, s):
    if s >= case["L"]:
        return fn(t, False)
    return _blocks(lambda u: fn(u, True), t, ((case["block"] - 1) >> (s if case["nested"] else 0)) + 1)


def _coarse_ops(shape, device):
    return [(torch.tensor(_even(n), device=device),) for n in shape]


def _down(x, case):
    for a, n in enumerate(x.shape):
        m = _padded(n, case)
        if case["pad"] == "zero":
            x = torch.cat([x, x.new_zeros(x.shape[:a] + (m - n,) + x.shape[a + 1:])], a)
        else:
            x = x.index_select(a, torch.arange(m, device=x.device).clamp(max=n - 1))
    parts = []
    for s in range(case["L"] + case["M"]):
        parts.append(_level(_level_down, x, case, s))
        x = _pick(parts[-1], _coarse_ops(x.shape, x.device))
    for g in reversed(parts):
        x = _put(g, x, _coarse_ops(g.shape, g.device))
    return x


def _up(c, case, shape):
    grids = [c]
    for _ in range(case["L"] + case["M"]):
        grids.append(_pick(grids[-1], _coarse_ops(grids[-1].shape, c.device)))
    x = grids.pop()
    for s in reversed(range(case["L"] + case["M"])):
        g = grids.pop()
        x = _level(_level_up, _put(g, x, _coarse_ops(g.shape, g.device)), case, s)
    return x[: shape[0], : shape[1], : shape[2]]


def exact(case, seed):
    """The transform's and its gradients' values in 64 bits.  Codes are whole
    numbers, and a field restored from codes, a map of widths or a container
    depends on them, so these have no such value."""
    if case["kind"] not in ("transform", "grad"):
        return None
    x, more, _, _ = _inputs(case, seed)
    x = x.double()
    if case["kind"] == "transform":
        return _down(x, case), x
    x.requires_grad_()
    co = _down(x, case)
    gx, = torch.autograd.grad(co, x, more["gc"].double())
    leaf = co.detach().requires_grad_()
    y = _up(leaf, case, x.shape)
    gc, = torch.autograd.grad(y, leaf, more["gx"].double())
    return co.detach(), gx, y.detach(), gc
