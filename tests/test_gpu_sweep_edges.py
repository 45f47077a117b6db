"""The role-split sweeps at r = 32 (FP64 Z1-out, FP32 Z1-out and TTNN), two slabs and 32
columns a sub-tile, at the edges of their range: one slab pair, an odd number of pairs, one
column block a tile, several tiles a column band, Y rows short of the padded 48."""
import numpy as np
import pytest

import oracle as O
from gpu_util import TOL_ARITH, failures, sketch_errors, to_device

pytestmark = pytest.mark.gpu

SHAPES = [(128, 2, 16, 64), (128, 6, 8, 32), (128, 10, 24, 24), (128, 34, 16, 64)]


@pytest.mark.parametrize("dims", SHAPES, ids=str)
@pytest.mark.parametrize("p", [1, 16])
@pytest.mark.parametrize("variant,dtype", [("sttnn", "f64"), ("sttnn", "f32"), ("ttnn", "f32")])
def test_role_split_sweep_edges(dims, p, variant, dtype):
    import paper_2412_06111_amd as P
    T = np.random.default_rng(21).standard_normal(dims)
    dev, consumed = to_device(T, dtype)
    plan = P.Plan(O.T4, dims, 32, p, variant=variant, dtype=dtype, seed=9)
    plan.update(dev, alpha=0.5)
    plan.update(dev, alpha=0.5)
    tree = O.Tree(O.T4, dims, 32, p)
    sk = O.sketch(consumed, tree, O.DRMs(tree, 9, variant, dtype), variant)
    bad = failures(sketch_errors(plan, tree, sk), TOL_ARITH[dtype])
    assert not bad, bad


@pytest.mark.parametrize("dims", [(128, 4, 16, 64), (128, 12, 24, 24), (128, 6, 8, 32), (128, 68, 16, 64)], ids=str)
@pytest.mark.parametrize("p", [1, 32])
def test_bf16_sweep_edges(dims, p):
    """BF16 at r = 64: four slabs a tile where n_2 allows, else two."""
    import paper_2412_06111_amd as P
    T = np.random.default_rng(22).standard_normal(dims)
    dev, consumed = to_device(T, "bf16")
    plan = P.Plan(O.T4, dims, 64, p, variant="sttnn", dtype="bf16", seed=9)
    plan.update(dev, alpha=0.5)
    plan.update(dev, alpha=0.5)
    tree = O.Tree(O.T4, dims, 64, p)
    sk = O.sketch(consumed, tree, O.DRMs(tree, 9, "sttnn", "bf16"), "sttnn")
    bad = failures(sketch_errors(plan, tree, sk), TOL_ARITH["bf16"])
    assert not bad, bad


@pytest.mark.parametrize("dims,p", [((128, 132, 8, 32), 1), ((128, 512, 8, 24), 32), ((128, 68, 16, 64), 32), ((128, 1024, 8, 4), 32)], ids=str)
def test_bf16_sums_of_two_slabs(dims, p):
    """Sketches that follow from Z_A at BF16, r = 64, four slabs a tile (one column block a
    tile, three, two) and two (1,024 of one column block), over several tiles a sketch.  A
    product adds with an error of one FP32 rounding (2.5e-8 of the sum, rms) or two; sums of
    the eight products of two slabs, the former tiles, come out sqrt(9 / 2) to sqrt(9) times
    that, 5.3e-8 to 7.5e-8.  Sixteen products in one chain are at 1.3e-7."""
    import paper_2412_06111_amd as P
    T = np.random.default_rng(23).standard_normal(dims)
    dev, consumed = to_device(T, "bf16")
    plan = P.Plan(O.T4, dims, 64, p, variant="sttnn", dtype="bf16", seed=9)
    plan.update(dev)
    tree = O.Tree(O.T4, dims, 64, p)
    sk = O.sketch(consumed, tree, O.DRMs(tree, 9, "sttnn", "bf16"), "sttnn")
    errs = sketch_errors(plan, tree, sk)
    got = {k: errs[k][0] for k in (("psi", (1, 2, 3, 4)), ("R", (3, 4)), ("R", (3,)), ("R", (4,)))}
    print(got, flush=True)
    assert max(got.values()) <= 1e-7, got
    assert errs["R", (1, 2)][0] <= 1.5e-7 and errs["R", (1,)][0] <= 2e-7, errs


@pytest.mark.parametrize("variant,dtype", [("sttnn", "f64"), ("sttnn", "f32"), ("ttnn", "f32")])
@pytest.mark.parametrize("dims", [(128, 30, 8, 12), (128, 32, 4, 8), (128, 46, 8, 12), (128, 32, 48, 56), (128, 32, 64, 44)], ids=str)
def test_sums_of_many_tiles(dims, variant, dtype):
    """Z_A's partials summed by one thread an entry and by eight: 15, 16 and 23 tiles of two
    slabs; 252 and 264 tiles of entries for 256 compute units."""
    import paper_2412_06111_amd as P
    T = np.random.default_rng(24).standard_normal(dims)
    dev, consumed = to_device(T, dtype)
    plan = P.Plan(O.T4, dims, 32, 16, variant=variant, dtype=dtype, seed=9)
    plan.update(dev)
    tree = O.Tree(O.T4, dims, 32, 16)
    sk = O.sketch(consumed, tree, O.DRMs(tree, 9, variant, dtype), variant)
    bad = failures(sketch_errors(plan, tree, sk), TOL_ARITH[dtype])
    assert not bad, bad
