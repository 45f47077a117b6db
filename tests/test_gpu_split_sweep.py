"""The FP32 sweep at r = 32 forms its products on BF16 parts; a tile whose results leave the
range where that is exact is formed again on the FP32 matrix cores.  128 x 8 x 16 x 16 has
two slabs and one column block a tile, 128 x 8 x 64 x 32 several."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_util import TOL_ARITH, errs2, failures

pytestmark = pytest.mark.gpu

R, P_ = 32, 16
SHAPES = [(128, 8, 16, 16), (128, 8, 64, 32)]


@pytest.fixture(scope="module")
def P():
    import paper_2412_06111_amd as P
    return P


def tensor(T):
    return torch.from_numpy(np.asarray(T, dtype=np.float32).ravel(order="F").copy()).cuda()


def sketches(P, plan, T, nodes):
    plan.reset()
    plan.update(tensor(T))
    return [plan.read_sketch(plan.node(m), P.SK_R).cpu().numpy() for m in nodes]


def wide_nodes(variant):
    """Nodes whose sketch the sweep sums straight from the tensor."""
    return [(1, 2), (1,)] + ([(3, 4)] if variant == "ttnn" else [])


@pytest.mark.parametrize("variant", ["sttnn", "ttnn"])
@pytest.mark.parametrize("dims", SHAPES, ids=str)
@pytest.mark.parametrize("scale", [2.0 ** -105, 2.0 ** -70, 2.0 ** 100])
def test_powers_of_two_scale_through(P, variant, dims, scale):
    """A power of two changes no rounding: the scaled tensor's sketches are the scaled
    sketches, to the arithmetic error of the two runs, at magnitudes where parts of the
    split values would fall below the smallest BF16 number as well."""
    T = np.random.default_rng(3).standard_normal(dims).astype(np.float32)
    plan = P.Plan(O.T4, dims, R, P_, variant=variant, dtype="f32", seed=6)
    nodes = wide_nodes(variant)
    one = sketches(P, plan, T, nodes)
    big = sketches(P, plan, T * np.float32(scale), nodes)
    bad = failures({n: errs2(b / scale, a) for n, a, b in zip(nodes, one, big)}, TOL_ARITH["f32"])
    assert not bad, bad


@pytest.mark.parametrize("variant", ["sttnn", "ttnn"])
@pytest.mark.parametrize("dims", SHAPES, ids=str)
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38, 1e-33])
def test_values_at_the_ends_of_the_range(P, variant, dims, value):
    """One entry v in a tensor of zeros: the sketches are v times those of a one there, in
    FP32, infinities and overflow with their signs."""
    at = (77, 5, 9, 13)
    T = np.zeros(dims, dtype=np.float32)
    T[at] = 1.0
    plan = P.Plan(O.T4, dims, R, P_, variant=variant, dtype="f32", seed=6)
    nodes = wide_nodes(variant)
    one = sketches(P, plan, T, nodes)
    T[at] = value
    got = sketches(P, plan, T, nodes)
    for n, x, g in zip(nodes, one, got):
        with np.errstate(over="ignore", invalid="ignore"):
            want = np.where(x != 0, np.float32(value) * x.astype(np.float32), np.float32(0)).astype(np.float64)
        hit = (x != 0).any(axis=1)
        assert hit.sum() == 1
        assert np.array_equal(g[~hit], want[~hit]), n
        # one product and its sum with zeros, 2^-24 each side
        np.testing.assert_allclose(g[hit], want[hit], rtol=2.0 ** -22, atol=0, err_msg=str(n))
