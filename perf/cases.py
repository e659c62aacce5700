"""Performance cases: the work that programs have this library do, through its
public entry points, with the sizes of the repository's own workloads.

    listed()            the named cases, smallest calls to the largest
    draw(rng)           one more case of the same ranges, without a name
    prepare(case, seed) what a program holds before the call (inputs on the GPU,
                        output buffers, context, resident streams)
    run(state)          one pass; returns its outputs whole
    work(case)          bytes and operations one pass cannot do without
    exact(case, seed)   the outputs in 64 bits where they are computed numbers

Inputs are coefficient levels with Laplace(0, 2^-l) values (level l, coarsest
first; sizes by 3D dyadic coarsening), or for the decomposition of a field a
smooth one of 16 random-phase sinusoids with 1% Gaussian noise.
"""
import ctypes
import math

import numpy as np
import torch

import paper_2505_00227_amd as mdr

def _case(op, dtype, shape, nlevels, nplanes=None, m=4, **more):
    c = {"op": op, "dtype": dtype, "n0": shape[0], "n1": shape[1], "n2": shape[2], "nlevels": nlevels,
         "nplanes": nplanes or (32 if dtype == "f32" else 64), "m": m, "huf_chunk": 256, "concat": False}
    c.update(more)
    return c


def listed():
    cases = []

    def add(name, *a, **k):
        c = _case(*a, **k)
        c["name"] = name
        cases.append(c)

    # the smallest useful call: 32768 values, refactored and read back once (latency and launches)
    add("tiny_f32", "progressive", "f32", (32, 32, 32), 5, tols="1e-3")
    # the plain workload: one level of 2^20 values, a stream per plane (the encoder's general form),
    # refactored and refined three times
    add("plain_1m_f32", "progressive", "f32", (1, 1, 1 << 20), 1, m=1, tols="1e-1,1e-3,1e-6")
    # a 512^3 field's levels as the decomposition leaves them, back to back: one refactor, then six
    # refinements, each into a buffer of its own that the recomposition could take
    add("field512_f32", "progressive", "f32", (512, 512, 512), 9, concat=True, tols="1e-1,1e-2,1e-3,1e-4,1e-5,1e-6")
    # one 256 MiB slab of a resident 1024^3 f64 field, read by a new reader (retrieval latency)
    add("slab_fetch_f64", "fetch", "f64", (32, 1024, 1024), 9, tols="1e-4")
    # the whole 1024^3 f64 field as 32 slabs: one batched refactor, every plane read back (tolerance 0)
    add("field1024_f64", "batch", "f64", (32, 1024, 1024), 9, nvars=32, uneven=False, tols="0")
    # 256 variables of uneven size in one batch, read back at 1e-3
    add("batch256_f32", "batch", "f32", (256, 256, 256), 5, nvars=256, uneven=True, tols="1e-3")
    # storage: a variable refactored, serialized to host bytes, loaded again and read at 1e-5
    add("archive_2m_f32", "archive", "f32", (128, 128, 128), 6, tols="1e-5")
    # the field side of the path: multilevel decomposition, and recomposition of a ragged f64 grid
    add("decompose512_f32", "decompose", "f32", (512, 512, 512), 9)
    add("recompose_f64", "recompose", "f64", (301, 402, 503), 8)
    # squared-L2 tables of a 512^3 field's levels (L2-driven retrieval's preparation)
    add("l2_512_f32", "l2", "f32", (512, 512, 512), 9)
    # three velocity components read until V_total = vx^2 + vy^2 + vz^2 is within 1e-4
    add("qoi_256_f32", "qoi", "f32", (256, 256, 256), 7, nvars=3, family="sumsq", tols="1e-4")
    # a field in host memory through the chunked pipeline: refactor, then read at 1e-6, both over PCIe
    add("pipeline_f64", "pipeline", "f64", (32, 256, 256), 7, nchunks=8, tols="1e-6")
    return cases


# ---------------------------------------------------------------- drawn cases
def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng, lo, hi):
    """Three edges whose product is about a log-uniform draw from [lo, hi]."""
    n = _log_int(rng, lo, hi)
    e = n ** (1.0 / 3.0)
    a = max(1, int(e * rng.uniform(0.5, 1.5)))
    b = max(1, int(e * rng.uniform(0.5, 1.5)))
    return a, b, max(1, min(n // (a * b), 4096 if a * b > 1 else n))


def draw(rng):
    op = rng.choice(["progressive", "progressive", "progressive", "fetch", "fetch", "batch", "batch", "archive",
                     "decompose", "recompose", "l2", "qoi", "pipeline"])
    dtype = rng.choice(["f32", "f64"])
    W = 32 if dtype == "f32" else 64
    half = 1 if dtype == "f32" else 2
    if op in ("decompose", "recompose"):
        shape = _shape(rng, 1 << 12, (1 << 27) // half)
        if rng.random() < 0.4:  # whole 16-byte rows
            shape = (shape[0], shape[1], max(4, shape[2] // 4 * 4))
        return _case(op, dtype, shape, rng.randint(2, 9))
    nplanes = W if rng.random() < 0.6 else rng.randint(8, W)
    m = 4 if rng.random() < 0.6 else rng.choice([1, 2, 3, 5, 8])
    chunk = 256 if rng.random() < 0.7 else rng.choice([512, 1024, 2048, 4096])
    tol = "%.3g" % math.exp(rng.uniform(math.log(1e-7), math.log(1e-1)))
    more = {"nplanes": nplanes, "m": m, "huf_chunk": chunk, "tols": tol, "concat": rng.random() < 0.3}
    nlev = rng.randint(1, 9)
    if op == "progressive":
        k = rng.randint(1, 4)
        t = sorted((math.exp(rng.uniform(math.log(1e-7), math.log(1e-1))) for _ in range(k)), reverse=True)
        more["tols"] = ",".join("%.3g" % v for v in t)
        return _case(op, dtype, _shape(rng, 1 << 10, (1 << 26) // half), nlev, **more)
    if op == "fetch":
        if rng.random() < 0.3:
            more["tols"] = "0"
        return _case(op, dtype, _shape(rng, 1 << 12, (1 << 26) // half), nlev, **more)
    if op == "batch":
        return _case(op, dtype, _shape(rng, 1 << 12, 1 << 21), rng.randint(1, 6), nvars=rng.randint(2, 96),
                     uneven=True, **more)
    if op == "archive":
        return _case(op, dtype, _shape(rng, 1 << 10, 1 << 21), nlev, **more)
    if op == "l2":
        return _case(op, dtype, _shape(rng, 1 << 12, (1 << 26) // half), nlev, nplanes=nplanes, m=m)
    if op == "qoi":
        fam = rng.choice(["sumsq", "magnitude", "product"])
        more["tols"] = "%.3g" % math.exp(rng.uniform(math.log(1e-5), math.log(1e-1)))
        return _case(op, dtype, _shape(rng, 1 << 12, (1 << 24) // half), nlev,
                     nvars=2 if fam == "product" else rng.randint(1, 3), family=fam, **more)
    return _case(op, dtype, _shape(rng, 1 << 12, 1 << 21), nlev, nchunks=rng.randint(2, 8), **more)


# ---------------------------------------------------------------- inputs
def _torch_dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.float64


def _edges(case):
    return case["n0"], case["n1"], case["n2"]


def _level_sizes(edges, nlevels):
    """Values per level, coarsest first: the nodes each halving of the grid spacing adds."""
    pts = [math.prod(((d - 1) >> j) + 1 for d in edges) for j in range(nlevels)][::-1]
    return [pts[0]] + [b - a for a, b in zip(pts, pts[1:])]


def _variables(case):
    """Grid edges of each variable of the case."""
    e = _edges(case)
    nv = case.get("nvars", 1)
    if not case.get("uneven"):
        return [e] * nv
    # uneven variables: edges uniform in [edge / 16, edge], the same for every seed
    rng = np.random.default_rng(case["n0"] * 1000003 + nv)
    return [tuple(int(rng.integers(max(1, d // 16), d + 1)) for d in e) for _ in range(nv)]


def _split(case, edges, flat):
    """The levels of a flat buffer: back to back (concat: the form the multilevel
    decomposition writes and the recomposition reads), else each from a 64-value boundary."""
    out, at = [], 0
    for n in _level_sizes(edges, case["nlevels"]):
        out.append(flat[at:at + n])
        at += n if case["concat"] else (n + 63) // 64 * 64
    return out


def _flat(case, edges):
    """A zeroed buffer that holds a grid's levels."""
    sizes = _level_sizes(edges, case["nlevels"])
    n = sum(sizes) if case["concat"] else sum((k + 63) // 64 * 64 for k in sizes)
    return torch.zeros(n, dtype=_torch_dtype(case), device="cuda")


def _levels(case, edges, gen):
    """Laplace(0, 2^-l) coefficient levels of a grid, drawn in f64."""
    out = _split(case, edges, _flat(case, edges))
    for l, n in enumerate(_level_sizes(edges, case["nlevels"])):
        t = torch.rand(n, dtype=torch.float64, device="cuda", generator=gen)
        t.sub_(0.5)
        mag = torch.log1p(t.abs().mul_(-2.0).clamp_(min=-1.0 + 2.0 ** -53)).mul_(-(2.0 ** -l))
        out[l].copy_(torch.copysign(mag, t))
        del t, mag
    return out


def _smooth_field(case, seed):
    """16 random-phase sinusoids (wavevectors in [1, 8]^3, amplitude 1/|k|) and 1% noise."""
    rng = np.random.default_rng(seed)
    ks, ph = rng.integers(1, 9, size=(16, 3)), rng.uniform(0.0, 2.0 * math.pi, 16)
    ax = [torch.arange(n, dtype=torch.float64, device="cuda") * (2.0 * math.pi / n) for n in _edges(case)]
    u = torch.zeros(_edges(case), dtype=torch.float64, device="cuda")
    for k, p in zip(ks, ph):
        # sin(a + b) by the product rule, so that only lines and planes take sines
        yz = (ax[1] * int(k[1]))[:, None] + (ax[2] * int(k[2]) + float(p))[None, :]
        a = 1.0 / math.sqrt(sum(int(c) * int(c) for c in k))
        x = ax[0] * int(k[0])
        u.addcmul_((a * torch.sin(x))[:, None, None], torch.cos(yz)[None])
        u.addcmul_((a * torch.cos(x))[:, None, None], torch.sin(yz)[None])
    gen = torch.Generator("cuda").manual_seed(seed)
    u.add_(torch.randn(u.shape, dtype=torch.float64, device="cuda", generator=gen), alpha=0.01 * float(u.std()) + 1e-30)
    return u.to(_torch_dtype(case))


def _tols(case):
    return [float(t) for t in case["tols"].split(",")]


def _params(case):
    return mdr.default_params(group_planes=case["m"], huf_chunk=case["huf_chunk"])


def _numbers(infos):
    """Info records as two arrays: byte counts and flags (exact), and bounds."""
    ints = [[i[k] for k in i if isinstance(i[k], int)] for i in infos]
    flts = [[x for k in i if not isinstance(i[k], int) for x in (i[k] if isinstance(i[k], list) else [i[k]])]
            for i in infos]
    return np.array(ints, np.int64), np.array(flts, np.float64)


def _inputs(case, seed):
    """Every variable's levels, made from the seed alone."""
    gen = torch.Generator("cuda").manual_seed(seed)
    return [_levels(case, e, gen) for e in _variables(case)]


def _host_chunks(case, seed):
    """The pipeline's field: every chunk's levels concatenated, in pinned host memory."""
    gen = torch.Generator("cuda").manual_seed(seed)
    per = case["n0"] * case["n1"] * case["n2"]
    host = torch.empty(per * case["nchunks"], dtype=_torch_dtype(case), pin_memory=True)
    for c in range(case["nchunks"]):
        host[c * per:(c + 1) * per].copy_(torch.cat(_levels(case, _edges(case), gen)))
    return host


def prepare(case, seed):
    op = case["op"]
    st = {"case": case, "ctx": mdr.Context(0)}
    if op in ("decompose", "recompose"):
        st["steps"] = case["nlevels"] - 1
        if op == "decompose":
            st["field"] = _smooth_field(case, seed)
            st["coeffs"] = torch.empty(st["field"].numel(), dtype=st["field"].dtype, device="cuda")
        else:
            st["coeffs"] = torch.cat(_inputs(case, seed)[0])
            st["field"] = torch.empty(_edges(case), dtype=st["coeffs"].dtype, device="cuda")
        return st
    st["params"] = _params(case)
    if op == "pipeline":
        st["host"] = _host_chunks(case, seed)
        st["host_out"] = torch.empty(st["host"].shape, dtype=st["host"].dtype, pin_memory=True)
        st["pipe"] = mdr.Pipeline(st["ctx"], case["nchunks"], _level_sizes(_edges(case), case["nlevels"]),
                                  _torch_dtype(case), case["nplanes"], st["params"])
        return st
    variables = _inputs(case, seed)
    edges = _variables(case)
    if op in ("progressive", "archive"):
        st["levels"] = variables[0]
        st["flat"] = [_flat(case, edges[0]) for _ in _tols(case)]
        st["outs"] = [_split(case, edges[0], f) for f in st["flat"]]
        if op == "archive":  # the host buffer a program that stores variables keeps
            s = 4 if case["dtype"] == "f32" else 8
            n = sum(t.numel() for t in variables[0])
            st["blob"] = np.zeros(2 * n * s + 65536 * case["nlevels"], np.uint8)
    elif op == "batch":
        # every variable's values in one buffer; views and output pointers marshalled once, as a
        # program that repeats a batch keeps them
        sizes = [_flat(case, e).numel() for e in edges]
        pad = [(n + 63) // 64 * 64 for n in sizes]
        st["flat"] = torch.zeros(sum(pad), dtype=_torch_dtype(case), device="cuda")
        at = np.concatenate([[0], np.cumsum(pad)])
        st["views"] = mdr.BatchViews(variables)
        st["outs"] = mdr.BatchOutputs([_split(case, e, st["flat"][int(a):int(a) + n])
                                       for e, a, n in zip(edges, at, sizes)])
    elif op == "l2":
        st["levels"] = variables[0]
        st["r"] = mdr.refactor(st["ctx"], variables[0], case["nplanes"], mdr.default_params(group_planes=case["m"]))
    else:  # fetch, qoi: the refactored fields are resident, their values are not kept
        st["rs"] = [mdr.refactor(st["ctx"], v, case["nplanes"], st["params"]) for v in variables]
        st["flat"] = [_flat(case, e) for e in edges]
        st["outs"] = [_split(case, e, f) for e, f in zip(edges, st["flat"])]
    return st


# ---------------------------------------------------------------- one pass
def run(state):
    case, ctx = state["case"], state["ctx"]
    op, B = case["op"], case["nplanes"]
    if op == "progressive":
        r = mdr.refactor(ctx, state["levels"], B, state["params"])
        rt = mdr.Retriever(ctx, r)
        infos = [rt.retrieve(t, o) for t, o in zip(_tols(case), state["outs"])]
        counts, bounds = _numbers(infos)
        tables = np.array([r.info(l)["E"] for l in range(r.nlevels)])
        return {"tables": tables, "counts": counts, "bounds": bounds, "values": state["flat"]}
    if op == "fetch":
        info = mdr.Retriever(ctx, state["rs"][0]).retrieve(_tols(case)[0], state["outs"][0])
        return [*_numbers([info]), *state["flat"]]
    if op == "batch":
        rs = mdr.refactor_batch(ctx, state["views"], B, state["params"])
        rts = [mdr.Retriever(ctx, r) for r in rs]
        infos = mdr.retrieve_batch(rts, [_tols(case)[0]] * len(rts), state["outs"])
        return [*_numbers(infos), state["flat"]]
    if op == "archive":
        r = mdr.refactor(ctx, state["levels"], B, state["params"])
        blob, used, h = state["blob"], ctypes.c_uint64(), ctypes.c_void_p()
        host = ctypes.c_void_p(blob.ctypes.data)
        if mdr.mdr_serialize(r.handle, host, blob.size, ctypes.byref(used)) != mdr.MDR_OK:
            raise RuntimeError(mdr.mdr_last_error().decode())
        if mdr.mdr_deserialize(ctx.handle, host, used.value, ctypes.byref(h)) != mdr.MDR_OK:
            raise RuntimeError(mdr.mdr_last_error().decode())
        info = mdr.Retriever(ctx, mdr.Refactored(ctx, h)).retrieve(_tols(case)[0], state["outs"][0])
        return [blob, *_numbers([info]), *state["flat"]]
    if op == "decompose":
        mdr.decompose(state["field"], state["steps"], state["coeffs"])
        return state["coeffs"]
    if op == "recompose":
        mdr.recompose(state["coeffs"], state["steps"], state["field"])
        return state["field"]
    if op == "l2":
        r = state["r"]
        r.l2_table(state["levels"])
        return np.array([r.l2(l) for l in range(r.nlevels)])
    if op == "qoi":
        rts = [mdr.Retriever(ctx, r) for r in state["rs"]]
        info = mdr.retrieve_qoi(case["family"], rts, _tols(case)[0], state["outs"], relative=True)
        return [*_numbers([info]), *state["flat"]]
    a = state["pipe"].refactor(state["host"])
    b = state["pipe"].retrieve(_tols(case)[0], state["host_out"])
    return [np.array([a["stream_bytes"], b["stream_bytes"]]), state["host_out"]]


# ---------------------------------------------------------------- what a pass needs
def work(case):
    op = case["op"]
    s = 4 if case["dtype"] == "f32" else 8
    n = sum(a * b * c for a, b, c in _variables(case))
    planes = n * (case["nplanes"] + 1) // 8  # a sign and nplanes magnitude bits per value
    if op in ("decompose", "recompose"):
        return {"bytes": 2 * n * s, "flops": 2 * n}
    if op == "l2":  # a difference, a square and a sum per value and table entry
        return {"bytes": n * s, "flops": 3 * n * (case["nplanes"] + 1)}
    if op == "progressive":  # values in, planes out, then each refinement's values
        return {"bytes": n * s + planes + n * s * len(_tols(case)), "flops": n}
    if op == "fetch":
        return {"bytes": n * s, "flops": n}
    if op == "qoi":  # values written, and read once for the estimate
        return {"bytes": 2 * n * s, "flops": 6 * n}
    if op == "pipeline":
        return {"bytes": case["nchunks"] * (2 * n * s + 2 * planes), "flops": n * case["nchunks"]}
    return {"bytes": 2 * n * s + 2 * planes, "flops": n}  # batch, archive: values in, planes out and in, values out


# ---------------------------------------------------------------- 64-bit results
def _refine(u, shape):
    """Multilinear refinement of a stride-2 grid's values to `shape`, axis by axis (n2, n1, n0)."""
    for ax in (2, 1, 0):
        n = shape[ax]
        out_shape = list(u.shape)
        out_shape[ax] = n
        out = torch.empty(out_shape, dtype=torch.float64, device=u.device)
        ev, od = [slice(None)] * 3, [slice(None)] * 3
        ev[ax], od[ax] = slice(0, n, 2), slice(1, n, 2)
        out[tuple(ev)] = u
        if n > 1:
            k = n // 2
            left = u.narrow(ax, 0, k)
            right = u.narrow(ax, 1, min(k, u.shape[ax] - 1))
            o = left.clone()
            o.narrow(ax, 0, right.shape[ax]).add_(right).mul_(0.5)
            out[tuple(od)] = o
        u = out
    return u


def _new_nodes(shape):
    """Mask of a grid's nodes that are not on its stride-2 grid."""
    odd = [torch.arange(d, device="cuda") % 2 == 1 for d in shape]
    return odd[0][:, None, None] | odd[1][None, :, None] | odd[2][None, None, :]


def _grids(case):
    """Grid shapes of the strides 2^0 .. 2^(nlevels - 1)."""
    return [tuple(((d - 1) >> j) + 1 for d in _edges(case)) for j in range(case["nlevels"])]


def exact(case, seed):
    op = case["op"]
    if op == "decompose":
        u = _smooth_field(case, seed).double()
        grids = _grids(case)
        parts = []
        for j in range(case["nlevels"] - 1):
            coarse = u[::2, ::2, ::2]
            parts.append((u - _refine(coarse, grids[j]))[_new_nodes(grids[j])])
            u = coarse
        return torch.cat([u.reshape(-1)] + parts[::-1])
    if op == "recompose":
        c, grids = torch.cat(_inputs(case, seed)[0]).double(), _grids(case)
        n = math.prod(grids[-1])
        u, at = c[:n].reshape(grids[-1]), n
        for j in range(case["nlevels"] - 2, -1, -1):
            new = _new_nodes(grids[j])
            k = int(new.sum())
            u = _refine(u, grids[j])
            u[new] += c[at:at + k]
            at += k
        return u
    if op == "l2":
        out = []
        for t in _inputs(case, seed)[0]:
            a = t.double().abs()
            e = math.frexp(float(a.max()))[1] if a.numel() else 0
            row = []
            for k in range(case["nplanes"] + 1):
                s = a * 2.0 ** (k - e)
                s = (s - torch.floor(s)) * 2.0 ** (e - k)
                row.append(float((s * s).sum()))
            out.append(row)
        return np.array(out)
    return None
