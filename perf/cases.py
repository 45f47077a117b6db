"""Performance cases: the work a user of this library has it do, through its public entry
points, over the range of sizes, trees, types and directions it serves.

A case is one of seven kinds of work:

  sketch   a dense tensor in device memory is sketched whole (reset + update); the
           stream's sketches (every R_t and the root's) are read back
  step     the same followed by the recovery: reset + update + enqueued assembly -> cores
  box      one additive box, read in place from a resident tensor, on a resident stream
  streams  rounds of batched packed boxes, one a stream and round, over many small streams
  rank1    a group of rank-1 terms on a resident stream (the group form the server uses)
  round    rounding of a tensor given in tree format (Khatri-Rao maps): reset + update_ttn
           + enqueued assembly -> cores
  recon    the dense tensor of a set of cores

FP32 and BF16 plans accumulate in FP64 what FP32 arithmetic gives; their sketches are
handed on as FP32.  `exact` evaluates the method's formulas in FP64 with plain torch,
the Gaussian maps included (a counter-based generator and Box-Muller).
"""
import math
import random

import numpy as np
import torch

import paper_2412_06111_amd as P

TREES = {
    "t3": ((1, 2), 3),
    "t4": ((1, 2), (3, 4)),
    "t5": (((1, 2), 3), (4, 5)),
    "t6": (((1, 2), 3), 4, (5, 6)),      # the index tree of the 6-D experiments
    "tucker4": (1, 2, 3, 4),
}
TORCH_OF = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
SIZE_OF = {"f64": 8, "f32": 4, "bf16": 2}


# ---------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest problem of the accuracy experiments: launches and latency only
        dict(name="step_16x4_ttnn_f64", kind="step", tree="t4", dims="16,16,16,16", r=6, p=3, variant="ttnn",
             dtype="f64", data="ttn", e=4, noise=1e-3),
        # the headline workload: 268M entries in one pass, FP32
        dict(name="sketch_128x4_sttnn_f32", kind="sketch", tree="t4", dims="128,128,128,128", r=32, p=16,
             variant="sttnn", dtype="f32", data="ttn", e=24, noise=1e-4),
        # the reduced-precision run at its largest rank
        dict(name="sketch_128x4_sttnn_bf16_r64", kind="sketch", tree="t4", dims="128,128,128,128", r=64, p=32,
             variant="sttnn", dtype="bf16", data="ttn", e=24, noise=1e-4),
        # the plain method on the same tensor (every leaf map spans the other three modes)
        dict(name="sketch_128x4_ttnn_f32", kind="sketch", tree="t4", dims="128,128,128,128", r=32, p=16,
             variant="ttnn", dtype="f32", data="ttn", e=24, noise=1e-4),
        # the FP64 path of the same comparison, recovery included
        dict(name="step_128x4_sttnn_f64", kind="step", tree="t4", dims="128,128,128,128", r=32, p=16,
             variant="sttnn", dtype="f64", data="ttn", e=24, noise=1e-4),
        # a user's own data: no mode a power of two, mode 1 odd, an odd rank
        dict(name="sketch_ragged_ttnn_f32", kind="sketch", tree="t4", dims="97,113,61,75", r=21, p=10,
             variant="ttnn", dtype="f32", data="ttn", e=24, noise=1e-4),
        # the 6-D accuracy experiment at its largest rank
        dict(name="sketch_hilbert_20x6_sttnn_f64", kind="sketch", tree="t6", dims="20,20,20,20,20,20", r=13, p=3,
             variant="sttnn", dtype="f64", data="hilbert", e=0, noise=0.0),
        # single-stream serving: a sub-block of the resident order-5 tensor
        dict(name="box_64x5_ttnn_f32", kind="box", tree="t5", dims="64,64,64,64,64", ext="33,21,47,40,26",
             off="13,40,9,22,35", r=24, p=12, variant="ttnn", dtype="f32"),
        # many-stream serving: one round after another of one box a stream
        dict(name="streams_16x8_ttnn_f32", kind="streams", tree="t4", streams=16, rounds=8, shapes=1000, nlo=32,
             nhi=160, elo=4, ehi=48, variant="ttnn", dtype="f32"),
        # single-stream serving: a full group of rank-1 terms
        dict(name="rank1_64x5_16_f32", kind="rank1", tree="t5", dims="64,64,64,64,64", terms=16, r=24, p=12,
             variant="ttnn", dtype="f32"),
        # the rounding experiment (TTN ranks 70, quadratic decay)
        dict(name="round_500x6_r32", kind="round", tree="t6", n=500, s=70, r=32, p=10),
        # the dense approximant, as for the error metric
        dict(name="recon_128x4_f32", kind="recon", tree="t4", dims="128,128,128,128", r=32, p=16, dtype="f32"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng: random.Random):
    kind = rng.choice(["sketch", "sketch", "sketch", "step", "step", "box", "box", "streams", "rank1", "round", "recon"])
    if kind in ("sketch", "step"):
        dtype = "f64" if kind == "step" else rng.choice(["f64", "f32", "f32", "bf16"])
        tree = rng.choice(["t3", "t4", "t4", "t5", "t6", "tucker4"])
        d = {"t3": 3, "t5": 5, "t6": 6}.get(tree, 4)
        total = _log(rng, 4e4 if d > 4 else 4e3, 2.5e7 if dtype == "f64" else 6e7)
        dims = _shape(rng, d, total)
        r = max(3, min(int(_log(rng, 4, 16 if tree == "tucker4" else 64)), min(dims), int(2e9 / total)))
        hil = kind == "sketch" and dtype == "f64" and rng.random() < 0.3
        return dict(kind=kind, tree=tree, dims=_txt(dims), r=r, p=rng.choice([3, max(1, r // 2)]),
                    variant=rng.choice(["ttnn", "sttnn"]), dtype=dtype, data="hilbert" if hil else "ttn",
                    e=max(2, min(min(dims), r - 2 if r > 6 else r)), noise=1e-3)
    if kind == "box":
        tree = rng.choice(["t4", "t5"])
        n = rng.randint(40, 64) if tree == "t5" else rng.randint(48, 160)
        dims = [max(24, n - rng.randint(0, 8)) for _ in range(5 if tree == "t5" else 4)]
        hi = 40 if tree == "t5" else 96
        ext = [rng.randint(8, min(hi, x)) for x in dims]
        off = [rng.randint(0, x - e) for x, e in zip(dims, ext)]
        r = rng.choice([16, 24, 32])
        return dict(kind="box", tree=tree, dims=_txt(dims), ext=_txt(ext), off=_txt(off), r=min(r, 24), p=r // 2,
                    variant=rng.choice(["ttnn", "ttnn", "sttnn"]), dtype=rng.choice(["f32", "f32", "f64", "bf16"]))
    if kind == "streams":
        nlo = rng.randint(24, 64)
        return dict(kind="streams", tree="t4", streams=rng.randint(2, 24), rounds=rng.randint(1, 5),
                    shapes=rng.randint(1, 10 ** 6), nlo=nlo, nhi=nlo + rng.randint(0, 90), elo=4,
                    ehi=rng.randint(8, 48), variant=rng.choice(["ttnn", "ttnn", "sttnn"]),
                    dtype=rng.choice(["f32", "f32", "f64", "bf16"]))
    if kind == "rank1":
        tree = rng.choice(["t4", "t5"])
        d, hi = (5, 48) if tree == "t5" else (4, 128)
        dims = [int(_log(rng, 12, hi)) for _ in range(d)]
        r = rng.randint(6, 12)
        return dict(kind="rank1", tree=tree, dims=_txt(dims), terms=rng.choice([1, 2, 5, 8, 16]), r=r, p=r // 2,
                    variant=rng.choice(["ttnn", "ttnn", "sttnn"]), dtype=rng.choice(["f32", "f32", "f64", "bf16"]))
    if kind == "round":
        n = int(_log(rng, 60, 500))
        s = rng.randint(20, min(60, n))
        return dict(kind="round", tree=rng.choice(["t4", "t5", "t6"]), n=n, s=s, r=rng.randint(6, min(30, s - 6)), p=10)
    d = rng.choice([3, 4, 5])
    dims = _shape(rng, d, _log(rng, 1e4, 1.2e8))
    return dict(kind="recon", tree={3: "t3", 4: "t4", 5: "t5"}[d], dims=_txt(dims), r=max(3, min(int(_log(rng, 4, 40)), min(dims))),
                p=3, dtype=rng.choice(["f32", "f64"]))


def _shape(rng, d, total):
    w = [rng.uniform(0.75, 1.25) for _ in range(d)]
    n = [max(4, int(round(math.exp(math.log(total) * x / sum(w))))) for x in w]
    return [min(x, 1500) for x in n]


def _txt(v):
    return ",".join(str(x) for x in v)


def _ints(text):
    return tuple(int(x) for x in text.split(","))


# ---------------------------------------------------------------- trees and sizes
class _Node:
    def __init__(self, modes, parent):
        self.modes, self.parent, self.kids = modes, parent, []


def _modes(s):
    return (s,) if isinstance(s, int) else tuple(m for c in s for m in _modes(c))


def _nodes(spec):
    """Nodes level by level (the numbering of the maps), root first."""
    out, queue = [], [(spec, -1)]
    while queue:
        nxt = []
        for s, par in queue:
            out.append(_Node(_modes(s), par))
            if par >= 0:
                out[par].kids.append(len(out) - 1)
            if not isinstance(s, int):
                nxt += [(c, len(out) - 1) for c in s]
        queue = nxt
    return out


def _reuse(nodes, t):
    """Groups contracted before node t is sketched sequentially: the earlier siblings of
    its ancestors and its own, outermost first."""
    path = []
    while t > 0:
        path.append(t)
        t = nodes[t].parent
    out = []
    for v in reversed(path):
        kids = nodes[nodes[v].parent].kids
        out += kids[:kids.index(v)]
    return out


def _prod(v):
    return math.prod(int(x) for x in v)


def _contraction_work(spec, dims, r, p, variant, ext=None):
    """(flops, map entries, sketch entries) of one pass over a tensor (or box of extent ext)."""
    nodes, k, ext = _nodes(spec), r + p, ext or dims
    flops, maps, outs, seen = 0, 0, 0, set()

    def size(S):
        e = list(ext)
        for s in S:
            for j, m in enumerate(nodes[s].modes):
                e[m - 1] = k if j == 0 else 1
        return _prod(e)

    def chain(S):
        for j in range(len(S)):
            if tuple(S[:j + 1]) not in seen:
                seen.add(tuple(S[:j + 1]))
                yield 2 * size(S[:j]) * k, _prod(ext[m - 1] for m in nodes[S[j]].modes) * k

    for t in range(1, len(nodes)):
        S = _reuse(nodes, t) if variant == "sttnn" else []
        for f, m in chain(S):
            flops, maps = flops + f, maps + m
        nt = _prod(ext[m - 1] for m in nodes[t].modes)
        flops += 2 * size(S) * r
        maps += size(S) // nt * r
        outs += nt * r
    for f, m in chain(nodes[0].kids):
        flops, maps = flops + f, maps + m
    return flops, maps, outs + k ** len(nodes[0].kids)


def work(case):
    kind, spec = case["kind"], TREES[case["tree"]]
    nodes = _nodes(spec)
    if kind in ("sketch", "step", "box"):
        dims, s = _ints(case["dims"]), SIZE_OF[case["dtype"]]
        ext = _ints(case["ext"]) if kind == "box" else dims
        f, m, o = _contraction_work(spec, dims, case["r"], case["p"], case["variant"], ext)
        return {"bytes": _prod(ext) * s + m * s + (2 if kind == "box" else 1) * o * 8, "flops": f}
    if kind == "streams":
        s, total, flops = SIZE_OF[case["dtype"]], 0, 0
        for pr in _stream_problems(case):
            for _, ext in pr["boxes"]:
                f, m, o = _contraction_work(spec, pr["dims"], pr["r"], pr["p"], case["variant"], ext)
                total, flops = total + _prod(ext) * s + m * s + 2 * o * 8, flops + f
        return {"bytes": total, "flops": flops}
    if kind == "rank1":
        dims, s, r, k = _ints(case["dims"]), SIZE_OF[case["dtype"]], case["r"], case["r"] + case["p"]
        maps = outs = 0
        for t in range(1, len(nodes)):
            S = _reuse(nodes, t) if case["variant"] == "sttnn" else []
            e = list(dims)
            for g in S:
                for j, m in enumerate(nodes[g].modes):
                    e[m - 1] = k if j == 0 else 1
            nt = _prod(dims[m - 1] for m in nodes[t].modes)
            maps, outs = maps + _prod(e) // nt * r, outs + nt * r
            if nodes[t].parent == 0 or any(t in _reuse(nodes, v) for v in range(1, len(nodes)) if case["variant"] == "sttnn"):
                maps += nt * k
        return {"bytes": maps * s + 2 * outs * 8, "flops": 2 * case["terms"] * (maps + outs)}
    if kind == "round":
        n, s, r, k = case["n"], case["s"], case["r"], case["r"] + case["p"]
        cores = flops = outs = 0
        for t, nd in enumerate(nodes):
            size = (n if not nd.kids else s ** len(nd.kids)) * (s if t else 1)
            cores += size
            flops += 2 * size * ((r + k) if t else 0) + 2 * size * r * max(1, len(nd.kids)) + 2 * size * k
            outs += (n * r if not nd.kids else r ** len(nd.kids) * (r if t else 1)) + (2 * k * r if t else 0)
        return {"bytes": 8 * (cores + outs + len(_modes(spec)) * n * (r + k)), "flops": flops}
    dims, r = _ints(case["dims"]), case["r"]
    N = _prod(dims)
    flops = 2 * N * r + sum(2 * _prod(dims[m - 1] for m in nd.modes) * r * r for t, nd in enumerate(nodes) if t and nd.kids)
    return {"bytes": N * SIZE_OF[case["dtype"]] + 8 * sum(dims) * r, "flops": flops}


# ---------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFF)
    return g


def _haar(n, k, g):
    q, r = np.linalg.qr(g.standard_normal((n, k)))
    return q * np.sign(np.diag(r))[None, :]


def _decay_core(shape, sigma, g):
    """Superdiagonal core with entries sigma, rotated by a Haar matrix on every mode."""
    c = np.zeros(shape)
    for i in range(min(shape)):
        c[(i,) * len(shape)] = sigma[i]
    for ax, n in enumerate(shape):
        c = np.moveaxis(np.tensordot(_haar(n, n, g), c, axes=([1], [ax])), 0, ax)
    return c


def _ttn_cores(spec, dims, e, sigma, seed):
    """Tree-format cores by level-order node id: Haar leaves, rotated superdiagonal cores."""
    g, out = np.random.Generator(np.random.PCG64(int(seed))), []
    for t, nd in enumerate(_nodes(spec)):
        if not nd.kids:
            out.append(_haar(_prod(dims[m - 1] for m in nd.modes), e, g))
        else:
            out.append(_decay_core((e,) * (len(nd.kids) + (1 if t else 0)), sigma, g))
    return out


def _mode_step(H, pos, M):
    """Contract position `pos` of H (positions slowest first, as in memory) with M's rows."""
    sh = list(H.shape)
    Q, n, L = _prod(sh[:pos]), sh[pos], _prod(sh[pos + 1:])
    if Q * n * L == 0:
        return H.new_zeros(sh[:pos] + [M.shape[1]] + sh[pos + 1:])
    H = H.reshape(Q, n, L)
    if L == 1:
        out = H.reshape(Q, n) @ M
    elif Q == 1:
        out = M.t().contiguous() @ H.reshape(n, L)
    else:
        out = (H.transpose(1, 2).reshape(Q * L, n) @ M).reshape(Q, L, M.shape[1]).transpose(1, 2)
    return out.reshape(sh[:pos] + [M.shape[1]] + sh[pos + 1:])


def _dense(spec, cores):
    """The tensor of tree-format cores (device FP64 arrays, first index first): memory
    order with mode 1 fastest, flat."""
    nodes = _nodes(spec)
    U = [None] * len(nodes)
    for t in range(len(nodes) - 1, -1, -1):
        if not nodes[t].kids:
            U[t] = cores[t]
            continue
        c = cores[t]
        H = c.permute(*reversed(range(c.dim()))).contiguous()          # last index slowest
        m = len(nodes[t].kids)
        for q in range(m):
            H = _mode_step(H, H.dim() - 1 - q, U[nodes[t].kids[q]].t().contiguous())
        U[t] = H.reshape(-1) if t == 0 else H.reshape(H.shape[0], -1).t().contiguous()
    return U[0]


def _whole(case, seed):
    """The whole tensor of a sketch or step case, flat, in the plan's type."""
    spec, dims = TREES[case["tree"]], _ints(case["dims"])
    if case["data"] == "hilbert":
        s = torch.zeros(tuple(reversed(dims)), dtype=torch.float64, device="cuda")
        for mu, n in enumerate(dims):
            shape = [1] * len(dims)
            shape[len(dims) - 1 - mu] = n
            s += torch.arange(n, dtype=torch.float64, device="cuda").view(shape)
        return (1.0 / (s + (1 + len(dims)))).reshape(-1).to(TORCH_OF[case["dtype"]])
    cores = _ttn_cores(spec, dims, case["e"], 0.8 ** np.arange(case["e"]), seed)
    T = _dense(spec, [torch.from_numpy(np.ascontiguousarray(c)).cuda() for c in cores])
    T *= math.sqrt(T.numel()) / torch.linalg.vector_norm(T)
    T += case["noise"] * torch.randn(T.numel(), generator=_gen(seed + 1), device="cuda", dtype=torch.float64)
    return T.to(TORCH_OF[case["dtype"]])


def _gauss_tensor(spec, dims, e, seed, dtype):
    """A random tree-format tensor with N(0,1) cores at about unit RMS, flat."""
    g = np.random.Generator(np.random.PCG64(int(seed)))
    cores = []
    for t, nd in enumerate(_nodes(spec)):
        n = _prod(dims[m - 1] for m in nd.modes) if not nd.kids else 0
        shape = (n, e) if not nd.kids else (e,) * (len(nd.kids) + (1 if t else 0))
        cores.append(torch.from_numpy(g.standard_normal(shape) / math.sqrt(_prod(shape[:-1]) if nd.kids else 1)).cuda())
    return _dense(spec, cores).to(TORCH_OF[dtype])


def _stream_problems(case):
    """Shapes, ranks and boxes of the streams, from the case alone."""
    out = []
    for s in range(case["streams"]):
        g = random.Random(case["shapes"] * 1000 + s)
        dims = tuple(g.randint(case["nlo"], case["nhi"]) for _ in range(4))
        r = g.choice([16, 32])
        boxes = []
        for _ in range(case["rounds"]):
            ext = tuple(min(n, g.randint(case["elo"], case["ehi"])) for n in dims)
            boxes.append((tuple(g.randint(0, n - e) for n, e in zip(dims, ext)), ext))
        out.append(dict(dims=dims, r=r, p=r // 2, boxes=boxes))
    return out


def _stream_blocks(case, seed, s, pr):
    """The packed boxes of one stream: slices of one random tree-format tensor."""
    g = np.random.Generator(np.random.PCG64([int(seed), s]))
    e, dims, spec = int(g.integers(8, 33)), pr["dims"], TREES[case["tree"]]
    leaves = [torch.from_numpy(g.standard_normal((n, e))).cuda() for n in dims]
    inner = [torch.from_numpy(g.standard_normal((e,) * q) / e).cuda() for q in (2, 3, 3)]
    blocks = []
    for off, ext in pr["boxes"]:
        cut = [u[o:o + x].contiguous() for u, o, x in zip(leaves, off, ext)]
        blocks.append(_dense(spec, inner + cut).mul_(1.0 / e).to(TORCH_OF[case["dtype"]]))
    return blocks


def _map_seed(seed):
    return 1 + int(seed) % (1 << 40)


def _plan(case, seed):
    return P.Plan(TREES[case["tree"]], _ints(case["dims"]), case["r"], case["p"], variant=case["variant"],
                  dtype=case["dtype"], seed=_map_seed(seed))


def _factors(case, seed):
    dims, g = _ints(case["dims"]), _gen(seed + 2)
    return [[torch.randn(n, generator=g, device="cuda", dtype=torch.float64) for n in dims]
            for _ in range(case["terms"])]


def _round_cores(case, seed):
    n = case["n"]
    dims = (n,) * len(_modes(TREES[case["tree"]]))
    return _ttn_cores(TREES[case["tree"]], dims, case["s"], 1.0 / np.arange(1, case["s"] + 1) ** 2, seed)


def _recon_cores(case, seed):
    r = case["r"]
    return _ttn_cores(TREES[case["tree"]], _ints(case["dims"]), r, 0.9 ** np.arange(r), seed)


def _by_modes(spec, cores):
    """Column-major flat device copies of level-order cores, keyed by the nodes' modes."""
    return {nd.modes: torch.from_numpy(np.ascontiguousarray(c.reshape(-1, order="F"))).cuda()
            for nd, c in zip(_nodes(spec), cores)}


def prepare(case, seed):
    kind, spec = case["kind"], TREES[case["tree"]]
    st = {"kind": kind, "case": case}
    if kind in ("sketch", "step"):
        st["plan"], st["x"] = _plan(case, seed), _whole(case, seed)
        st["cores"] = st["plan"].alloc_cores() if kind == "step" else None
    elif kind == "box":
        dims, ext, off = _ints(case["dims"]), _ints(case["ext"]), _ints(case["off"])
        T = _gauss_tensor(spec, dims, 16, seed, case["dtype"]).view(*reversed(dims))
        st["block"] = T[tuple(slice(o, o + e) for o, e in zip(reversed(off), reversed(ext)))]
        st["plan"], st["ext"], st["off"] = _plan(case, seed), ext, off
    elif kind == "streams":
        probs = _stream_problems(case)
        st["plans"] = [P.Plan(spec, pr["dims"], pr["r"], pr["p"], variant=case["variant"], dtype=case["dtype"],
                              seed=_map_seed(seed) + s) for s, pr in enumerate(probs)]
        blocks = [_stream_blocks(case, seed, s, pr) for s, pr in enumerate(probs)]
        st["rounds"] = [[(plan, b[k], pr["boxes"][k][1], pr["boxes"][k][0], 1.0)
                         for plan, b, pr in zip(st["plans"], blocks, probs)] for k in range(case["rounds"])]
    elif kind == "rank1":
        st["plan"], st["terms"] = _plan(case, seed), _factors(case, seed)
        st["plan"].set_rank1_form("grouped")
        st["alphas"] = [1.0 if y % 2 == 0 else -0.5 for y in range(case["terms"])]
    elif kind == "round":
        dims = (case["n"],) * len(_modes(spec))
        st["plan"] = P.Plan(spec, dims, case["r"], case["p"], variant="kr", seed=_map_seed(seed))
        st["in"] = _by_modes(spec, _round_cores(case, seed))
        st["cores"] = st["plan"].alloc_cores()
        st["work"] = torch.empty(st["plan"].update_ttn_work_bytes(case["s"]), dtype=torch.uint8, device="cuda")
    else:
        dims = _ints(case["dims"])
        st["plan"] = P.Plan(spec, dims, case["r"], case["p"], variant="sttnn", dtype="f64", seed=_map_seed(seed))
        by = _by_modes(spec, _recon_cores(case, seed))
        st["cores"] = [by[m] for m in st["plan"].node_modes]
        st["out"] = torch.empty(_prod(dims), dtype=TORCH_OF[case["dtype"]], device="cuda")
    return st


# ---------------------------------------------------------------- one pass
def _snapshot(plan):
    """Every accumulated sketch of a plan: R_t of the nodes, Psi of the root."""
    return [plan.read_sketch(v, P.SK_PSI if v == 0 else P.SK_R) for v in range(plan.num_nodes)]


def _handed_on(sketches, dtype):
    return sketches if dtype == "f64" else [x.to(torch.float32) for x in sketches]


def run(st):
    kind, case = st["kind"], st["case"]
    if kind == "sketch":
        st["plan"].reset()
        st["plan"].update(st["x"])
        return _handed_on(_snapshot(st["plan"]), case["dtype"])
    if kind == "step":
        st["plan"].reset()
        st["plan"].update(st["x"])
        return st["plan"].assemble_async(st["cores"])
    if kind == "box":
        st["plan"].update(st["block"], extent=st["ext"], offset=st["off"])
        return _handed_on(_snapshot(st["plan"]), case["dtype"])
    if kind == "streams":
        for items in st["rounds"]:
            P.update_batched(items)
        return _handed_on([torch.cat([x.t().reshape(-1) for x in _snapshot(plan)]) for plan in st["plans"]],
                          case["dtype"])
    if kind == "rank1":
        st["plan"].update_rank1_batched(st["terms"], st["alphas"])
        return _snapshot(st["plan"])
    if kind == "round":
        st["plan"].reset()
        st["plan"].update_ttn(st["in"], case["s"], work=st["work"])
        return st["plan"].assemble_async(st["cores"])
    return st["plan"].reconstruct(st["cores"], out=st["out"], out_dtype=P.F32 if case["dtype"] == "f32" else P.F64)


# ---------------------------------------------------------------- the same in FP64, plain torch
def _mul32(a, b):
    """High and low halves of the 64-bit product of 32-bit values (int64 arithmetic)."""
    p = a * b
    return (p >> 32) & 0xFFFFFFFF, p & 0xFFFFFFFF


def _gauss_rows(seed, tag, row0, rows, cols):
    """Rows [row0, row0 + rows) of the N(0,1) map `tag`: Philox4x32-10 on (row, column,
    tag), Box-Muller on two 53-bit uniforms."""
    row = torch.arange(row0, row0 + rows, dtype=torch.int64, device="cuda")[:, None]
    col = torch.arange(cols, dtype=torch.int64, device="cuda")[None, :]
    c0, c1 = (row & 0xFFFFFFFF).expand(rows, cols), (row >> 32).expand(rows, cols)
    c2, c3 = col.expand(rows, cols), torch.full((1, 1), tag, dtype=torch.int64, device="cuda").expand(rows, cols)
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for i in range(10):
        if i:
            k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
        h0, l0 = _mul32(c0, 0xD2511F53)
        h1, l1 = _mul32(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
    a, b = (c1 << 21) | (c0 >> 11), (c3 << 21) | (c2 >> 11)
    u1, u2 = (a + 1).to(torch.float64) * 2.0 ** -53, b.to(torch.float64) * 2.0 ** -53
    return torch.sqrt(-2.0 * torch.log(u1)) * torch.cos((2.0 * math.pi) * u2)


def _stored(x, dtype):
    if dtype == "f64":
        return x
    x = x.to(torch.float32)
    return (x.to(torch.bfloat16) if dtype == "bf16" else x).to(torch.float64)


def _map_chunks(seed, tag, rows, cols, dtype):
    step = max(1, (1 << 24) // cols)
    for r0 in range(0, rows, step):
        yield r0, _stored(_gauss_rows(seed, tag, r0, min(step, rows - r0), cols), dtype)


def _map(seed, tag, rows, cols, dtype):
    out = torch.empty((rows, cols), dtype=torch.float64, device="cuda")
    for r0, x in _map_chunks(seed, tag, rows, cols, dtype):
        out[r0:r0 + x.shape[0]] = x
    return out


def _exact_sketch(spec, H, r, p, variant, dtype, seed):
    """Every R_t and the root's Psi (by level-order id) of the FP64 tensor H (mode 1 last)."""
    nodes, k = _nodes(spec), r + p
    dims = tuple(reversed(H.shape))
    Y = {t: _map(seed, 2 * t + 1, _prod(dims[m - 1] for m in nodes[t].modes), k, dtype) for t in range(1, len(nodes))}
    done = {(): (H, [(m,) for m in range(len(dims), 0, -1)])}

    def contracted(S):
        S = tuple(S)
        if S not in done:
            Z, lab = contracted(S[:-1])
            mod = nodes[S[-1]].modes
            at = [i for i, x in enumerate(lab) if x[0] in mod]
            sh = list(Z.shape)
            Z = Z.reshape(sh[:at[0]] + [_prod(sh[at[0]:at[-1] + 1])] + sh[at[-1] + 1:])
            done[S] = (_mode_step(Z, at[0], Y[S[-1]]), lab[:at[0]] + [mod] + lab[at[-1] + 1:])
        return done[S]

    out = {0: contracted(nodes[0].kids)[0].reshape(-1, 1)}
    for t in range(1, len(nodes)):
        Z, lab = contracted(_reuse(nodes, t) if variant == "sttnn" else [])
        at = [i for i, x in enumerate(lab) if x[0] in nodes[t].modes]
        sh = Z.shape
        Q, n, L = _prod(sh[:at[0]]), _prod(sh[at[0]:at[-1] + 1]), _prod(sh[at[-1] + 1:])
        A = Z.reshape(Q, n, L).transpose(0, 1).reshape(n, Q * L)
        R = torch.zeros((n, r), dtype=torch.float64, device="cuda")
        for r0, x in _map_chunks(seed, 2 * t, Q * L, r, dtype):
            R += A[:, r0:r0 + x.shape[0]] @ x
        out[t] = R
        del A
    return out, Y


def _exact_cores(spec, dims, sk, Y, psi=None, om=None):
    """Cores (by level-order id, column-major flat) from the sketches, by signed QR and
    the truncated inverse."""
    nodes = _nodes(spec)
    Q, inv = {}, {}
    for t in range(1, len(nodes)):
        o = (om[t] if om else Y[t].t().contiguous() @ sk[t]).cpu().numpy()
        q, rr = np.linalg.qr(o)
        s = np.where(np.diag(rr) < 0, -1.0, 1.0)
        u, d, v = np.linalg.svd(rr * s[:, None])
        keep = d > 10 * 2.0 ** -52 * d[0]
        Q[t] = torch.from_numpy(q * s[None, :]).cuda()
        inv[t] = torch.from_numpy((v[keep].T / d[keep]) @ u[:, keep].T).cuda()
    out = {}
    for t, nd in enumerate(nodes):
        if not nd.kids:
            out[t] = (sk[t] @ inv[t]).t().reshape(-1)
            continue
        if psi is not None or t == 0:
            H = (psi[t] if psi is not None else sk[0]).reshape([1 if t == 0 else Q[t].shape[1]] + [Q[c].shape[0] for c in reversed(nd.kids)])
        else:
            H = sk[t].t().reshape([sk[t].shape[1]] + [Y[c].shape[0] for c in reversed(nd.kids)])
            for q, c in enumerate(nd.kids):
                H = _mode_step(H, len(nd.kids) - q, Y[c])
        for q, c in enumerate(nd.kids):
            H = _mode_step(H, len(nd.kids) - q, Q[c])
        out[t] = (H if t == 0 else _mode_step(H, 0, inv[t])).reshape(-1)
    return out


def _caller_order(spec):
    """Level-order ids in the order of the plan's own node numbering (depth first)."""
    nodes = _nodes(spec)
    out = []

    def walk(t):
        out.append(t)
        for c in nodes[t].kids:
            walk(c)

    walk(0)
    return out


def _exact_round(case, seed):
    spec, s, r, k = TREES[case["tree"]], case["s"], case["r"], case["r"] + case["p"]
    nodes, n = _nodes(spec), case["n"]
    B = [torch.from_numpy(np.ascontiguousarray(c)).cuda() for c in _round_cores(case, seed)]
    ms = _map_seed(seed)
    X = {m: _map(ms, 2 * (64 + m - 1), n, r, "f64") for m in _modes(spec)}
    Y = {m: _map(ms, 2 * (64 + m - 1) + 1, n, k, "f64") for m in _modes(spec)}

    def joined(core, vecs, keep):
        """sum of core over every index but `keep`, index q weighted by column j of vecs[q]."""
        T = torch.movedim(core, keep, -1).unsqueeze(0)                  # (j, ..., keep)
        for q in [i for i in range(core.dim()) if i != keep]:
            v = vecs[q].t()
            T = (T * v.reshape(v.shape[0], v.shape[1], *([1] * (T.dim() - 2)))).sum(1)
        return T.t().contiguous()                                       # (keep, j)

    dx, dy, up = {}, {}, {}
    for t in range(len(nodes) - 1, 0, -1):
        for d, F in ((dx, X), (dy, Y)):
            d[t] = B[t].t().contiguous() @ F[nodes[t].modes[0]] if not nodes[t].kids else joined(
                B[t], [d[c] for c in nodes[t].kids], B[t].dim() - 1)
    for t, nd in enumerate(nodes):
        for q, c in enumerate(nd.kids):
            up[c] = joined(B[t], [dx[g] for g in nd.kids] + ([up[t]] if t else []), q)
    om = {t: dy[t].t().contiguous() @ up[t] for t in range(1, len(nodes))}
    sk, psi = {}, {}
    for t, nd in enumerate(nodes):
        if not nd.kids:
            sk[t] = B[t] @ up[t]
            continue
        H = B[t].permute(*reversed(range(B[t].dim()))).contiguous()
        if t == 0:
            H = H.unsqueeze(0)
        for q, c in enumerate(nd.kids):
            H = _mode_step(H, H.dim() - 1 - q, dy[c])
        psi[t] = (H if t == 0 else _mode_step(H, 0, up[t])).reshape(-1)
    cores = _exact_cores(spec, None, sk, None, psi=psi, om=om)
    return [cores[t] for t in _caller_order(spec)]


def exact(case, seed):
    kind, spec = case["kind"], TREES[case["tree"]]
    order = _caller_order(spec)
    if kind == "round":
        return _exact_round(case, seed)
    if kind == "recon":
        return _dense(spec, [torch.from_numpy(np.ascontiguousarray(c)).cuda() for c in _recon_cores(case, seed)])
    if kind == "streams":
        out = []
        for s, pr in enumerate(_stream_problems(case)):
            H = torch.zeros(tuple(reversed(pr["dims"])), dtype=torch.float64, device="cuda")
            for (off, ext), b in zip(pr["boxes"], _stream_blocks(case, seed, s, pr)):
                H[tuple(slice(o, o + e) for o, e in zip(reversed(off), reversed(ext)))] += b.double().view(*reversed(ext))
            sk, _ = _exact_sketch(spec, H, pr["r"], pr["p"], case["variant"], case["dtype"], _map_seed(seed) + s)
            out.append(torch.cat([sk[t].t().reshape(-1) for t in order]))
        return out
    dims = _ints(case["dims"])
    r, p, variant, dtype, ms = case["r"], case["p"], case["variant"], case["dtype"], _map_seed(seed)
    if kind == "rank1":
        return _exact_rank1(case, seed, spec, dims, ms, order)
    if kind == "box":
        ext, off = _ints(case["ext"]), _ints(case["off"])
        T = _gauss_tensor(spec, dims, 16, seed, dtype).view(*reversed(dims))
        at = tuple(slice(o, o + e) for o, e in zip(reversed(off), reversed(ext)))
        H = torch.zeros(T.shape, dtype=torch.float64, device="cuda")
        H[at] = T[at].double()
        del T
    else:
        H = _whole(case, seed).double().view(*reversed(dims))
    sk, Y = _exact_sketch(spec, H, r, p, variant, dtype, ms)
    if kind == "step":
        cores = _exact_cores(spec, dims, sk, Y)
        return [cores[t] for t in order]
    return [sk[t] for t in order]


def _exact_rank1(case, seed, spec, dims, ms, order):
    nodes, r, k, dtype = _nodes(spec), case["r"], case["r"] + case["p"], case["dtype"]
    terms, m = _factors(case, seed), case["terms"]
    F = [torch.stack([t[mu] for t in terms]) for mu in range(len(dims))]        # (term, n)

    def kron(vs, r0=0, rows=None):
        """Rows of the terms' Kronecker vectors (first factor fastest): (term, rows)."""
        total = _prod(v.shape[1] for v in vs)
        i = torch.arange(r0, r0 + (total if rows is None else rows), device="cuda")
        out = torch.ones((m, i.numel()), dtype=torch.float64, device="cuda")
        for v in vs:
            out *= v[:, i % v.shape[1]]
            i = torch.div(i, v.shape[1], rounding_mode="floor")
        return out

    def group(t):
        """Y_t^T of the group's Kronecker vector, per term."""
        vs, w = [F[q - 1] for q in nodes[t].modes], 0.0
        for r0, y in _map_chunks(ms, 2 * t + 1, _prod(v.shape[1] for v in vs), k, dtype):
            w = w + kron(vs, r0, y.shape[0]) @ y
        return w

    a = torch.tensor([1.0 if y % 2 == 0 else -0.5 for y in range(m)], dtype=torch.float64, device="cuda")
    g, out = {}, {}
    for t in range(1, len(nodes)):
        S, vs = _reuse(nodes, t) if case["variant"] == "sttnn" else [], []
        for mu in range(1, len(dims) + 1):
            s = next((q for q in S if mu in nodes[q].modes), None)
            if mu in nodes[t].modes or (s is not None and mu != nodes[s].modes[0]):
                continue
            if s is not None and s not in g:
                g[s] = group(s)
            vs.append(F[mu - 1] if s is None else g[s])
        w = torch.zeros((m, r), dtype=torch.float64, device="cuda")
        for r0, x in _map_chunks(ms, 2 * t, _prod(v.shape[1] for v in vs), r, dtype):
            w += kron(vs, r0, x.shape[0]) @ x
        out[t] = (kron([F[q - 1] for q in nodes[t].modes]) * a[:, None]).t().contiguous() @ w
    for c in nodes[0].kids:
        if c not in g:
            g[c] = group(c)
    out[0] = (kron([g[c] for c in nodes[0].kids]) * a[:, None]).sum(0).reshape(-1, 1)
    return [out[t] for t in order]
