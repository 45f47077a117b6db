"""Edges of the generic contraction's tile: row tiles of 16, 32 and 64 with remainders,
one to three column blocks and a second column tile, contractions of one value, of one
step more or less than a whole one, and past one offset table; rows along memory (node
1), contraction along memory (node 2) and the left form (root), packed and in place."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_util import TOL_ARITH, failures, sketch_errors, to_device

pytestmark = pytest.mark.gpu

# (extent 1, extent 2, r, p)
SHAPES = [(1, 1, 1, 0), (15, 33, 3, 1), (16, 31, 16, 1), (17, 64, 17, 15), (32, 257, 15, 1), (33, 255, 32, 1),
          (64, 513, 31, 17), (65, 32, 33, 15), (40, 1030, 48, 1), (130, 70, 49, 48)]


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("e1,e2,r,p", SHAPES)
def test_tile_edges(e1, e2, r, p, dtype):
    import paper_2412_06111_amd as P
    spec, dims, off = (1, 2), (e1 + 3, e2 + 2), (2, 1)
    g = np.random.default_rng(7 * e1 + e2)
    full = np.zeros(dims)
    full[2:2 + e1, 1:1 + e2] = g.standard_normal((e1, e2))
    dev, consumed = to_device(full, dtype)
    view = dev.view(dims[1], dims[0])[1:1 + e2, 2:2 + e1]
    tree = O.Tree(spec, dims, r, p)
    sk = O.sketch(consumed, tree, O.DRMs(tree, 5, "ttnn", dtype), "ttnn")
    for block in (view, view.contiguous().reshape(-1)):
        plan = P.Plan(spec, dims, r, p, variant="ttnn", dtype=dtype, seed=5)
        plan.update(block, extent=(e1, e2), offset=off)
        torch.cuda.synchronize()
        errs = sketch_errors(plan, tree, sk)
        assert not failures(errs, TOL_ARITH[dtype]), errs
        plan.close()


def test_tile_ignores_values_past_the_box():
    """Rows, columns and contraction values past the end are masked: infinities and NaN
    around a box read in place do not reach its sketch."""
    import paper_2412_06111_amd as P
    spec, dims, ext, off = ((1, 2), 3), (21, 19, 23), (17, 13, 9), (2, 3, 5)
    g = np.random.default_rng(3)
    box = g.standard_normal(ext)
    t = torch.full(tuple(reversed(dims)), float("nan"), dtype=torch.float32, device="cuda")
    t[::2] = float("inf")
    at = tuple(slice(o, o + e) for o, e in zip(reversed(off), reversed(ext)))
    t[at] = torch.from_numpy(np.ascontiguousarray(box.T)).float().cuda()
    full = np.zeros(dims)
    full[tuple(slice(o, o + e) for o, e in zip(off, ext))] = t[at].double().cpu().numpy().T
    tree = O.Tree(spec, dims, 5, 3)
    sk = O.sketch(full, tree, O.DRMs(tree, 9, "ttnn", "f32"), "ttnn")
    plan = P.Plan(spec, dims, 5, 3, variant="ttnn", dtype="f32", seed=9)
    plan.update(t[at], extent=ext, offset=off)
    torch.cuda.synchronize()
    errs = sketch_errors(plan, tree, sk)
    assert not failures(errs, TOL_ARITH["f32"]), errs


# the reconstruction's last step (all modes but the last by the last): fewer rows or
# columns than a wave's 64 x 32 tile, edges moved back inside it, ranks no multiple of 4,
# and past the 1,024 rows of an XCD's share
@pytest.mark.parametrize("dims,r", [((3, 5, 4), 1), ((9, 11, 37), 5), ((13, 5, 33), 4), ((16, 4, 32), 3),
                                    ((64, 2, 31), 7), ((71, 19, 65), 18)])
@pytest.mark.parametrize("out", ["f64", "f32"])
def test_reconstruct_edges(dims, r, out):
    import paper_2412_06111_amd as P
    spec = (1, 2, 3)
    tree = O.Tree(spec, dims, r, 0)
    g = np.random.default_rng(sum(dims) + r)
    cores = {n.id: g.standard_normal(O.core_shape(tree, n.id)) for n in tree.nodes}
    want = O.reconstruct({i: c.ravel(order="F") if i == 0 else c for i, c in cores.items()}, tree)
    plan = P.Plan(spec, dims, r, 0, variant="ttnn", dtype="f64", seed=1)
    dev = [None] * plan.num_nodes
    for n in tree.nodes:
        dev[plan.node(n.modes)] = torch.from_numpy(cores[n.id].ravel(order="F").copy()).cuda()
    got = plan.reconstruct(dev, out_dtype=P.F32 if out == "f32" else P.F64)
    torch.cuda.synchronize()
    err = np.linalg.norm(got.double().cpu().numpy() - want.ravel(order="F")) / np.linalg.norm(want)
    assert err < (1e-12 if out == "f64" else 1e-7), err       # FP64 sums; FP32: one rounding of the result
    plan.close()


def reconstruction(spec, dims, r, out):
    """A plan, random cores on the device and the oracle's tensor of them."""
    import paper_2412_06111_amd as P
    tree = O.Tree(spec, dims, r, 0)
    g = np.random.default_rng(sum(dims) + r)
    cores = {n.id: g.standard_normal(O.core_shape(tree, n.id)) for n in tree.nodes}
    plan = P.Plan(spec, dims, r, 0, variant="ttnn", dtype="f64", seed=1)
    dev = [None] * plan.num_nodes
    for n in tree.nodes:
        dev[plan.node(n.modes)] = torch.from_numpy(cores[n.id].ravel(order="F").copy()).cuda()
    return plan, dev, P.F32 if out == "f32" else P.F64, tree, cores


@pytest.mark.parametrize("out", ["f64", "f32"])
@pytest.mark.parametrize("dims", [(3, 23, 40), (16, 40, 50), (64, 33, 9), (65, 5, 6), (129, 30, 31), (1100, 8, 9), (1100, 5, 5)], ids=str)
def test_reconstruct_splits(dims, out):
    """The last step's splits over waves and XCDs: first halves from below one wave's rows to
    several tiles an XCD, second halves from one tile on."""
    plan, dev, kind, tree, cores = reconstruction((1, (2, 3)), dims, 3, out)
    want = O.reconstruct({i: c.ravel(order="F") if i == 0 else c for i, c in cores.items()}, tree)
    got = plan.reconstruct(dev, out_dtype=kind)
    torch.cuda.synchronize()
    err = np.linalg.norm(got.double().cpu().numpy() - want.ravel(order="F")) / np.linalg.norm(want)
    assert err < (1e-12 if out == "f64" else 1e-7), err       # FP64 sums; FP32: one rounding of the result
    plan.close()


def test_reconstruct_time_either_way_round():
    """A tensor whose first half is one mode takes about what the same entries take from even
    halves (the last step's work is the same; with the XCDs split along the first half only it
    took 348 us for 78).  Three times: the forming of the larger half is in it as well."""
    us = {}
    for spec, dims in (((1, (2, 3)), (128, 512, 512)), (((1, 2), (3, 4)), (64, 64, 64, 128))):
        plan, dev, kind, _, _ = reconstruction(spec, dims, 32, "f32")
        out = torch.empty(int(np.prod(dims)), dtype=torch.float32, device="cuda")
        best = float("inf")
        for _ in range(12):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(5):
                plan.reconstruct(dev, out=out, out_dtype=kind)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 200)
        us[spec] = best
        plan.close()
    a, b = us.values()
    assert a < 3 * b, us


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("ext", [(2, 37, 19), (3, 18, 40), (4, 50, 9), (5, 33, 21), (7, 16, 30), (33, 65, 5)], ids=str)
def test_tile_groups_across_runs(ext, dtype):
    """Contractions along memory whose runs (mode 1) are shorter than, as long as and no
    multiple of a thread's group of values, on blocks that start one entry past an aligned
    address, packed and read in place in another order of modes."""
    import paper_2412_06111_amd as P
    spec, dims, off = ((1, 2), 3), tuple(e + 1 for e in ext), (1, 0, 1)
    g = np.random.default_rng(sum(ext))
    dev, consumed = to_device(g.standard_normal(ext), dtype)
    shifted = torch.empty(dev.numel() + 1, dtype=dev.dtype, device="cuda")[1:]
    shifted.copy_(dev)
    swapped = dev.view(*reversed(ext)).transpose(0, 2).contiguous().transpose(0, 2)   # mode 3 fastest in memory
    full = np.zeros(dims)
    full[1:, :-1, 1:] = consumed
    tree = O.Tree(spec, dims, 9, 4)
    sk = O.sketch(full, tree, O.DRMs(tree, 5, "ttnn", dtype), "ttnn")
    for block in (shifted, swapped):
        plan = P.Plan(spec, dims, 9, 4, variant="ttnn", dtype=dtype, seed=5)
        plan.update(block, extent=ext, offset=off)
        torch.cuda.synchronize()
        errs = sketch_errors(plan, tree, sk)
        assert not failures(errs, TOL_ARITH[dtype]), errs
        plan.close()
