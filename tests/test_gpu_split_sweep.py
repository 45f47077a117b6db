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


ALL = [(1, 2), (1,), (2,), (3, 4), (3,), (4,)]


def small(x, e):
    """x 2^e as FP32 holds it, and the same values times 2^-e (exact both ways)."""
    s = np.ldexp(np.asarray(x, dtype=np.float64), e).astype(np.float32)
    return s, np.ldexp(s.astype(np.float64), -e).astype(np.float32)


def small_tol(K, e):
    """FP32 arithmetic of two runs, and sums of K products of size 2^e that FP32 holds in
    steps of 2^-149: K roundings of up to half a step in a sum of about sqrt(K) 2^e."""
    return 2.0 ** -20 + np.sqrt(K) * 2.0 ** (-150 - e)


@pytest.mark.parametrize("variant", ["sttnn", "ttnn"])
@pytest.mark.parametrize("dims", SHAPES, ids=str)
@pytest.mark.parametrize("e", [-120, -133, -140])
def test_small_tensors(P, variant, dims, e):
    """Tensors whose split parts fall below the smallest BF16 number: the second part
    (2^-120), nearly all of the first (2^-133) and every part (2^-140, FP32 subnormals)."""
    T, up = small(np.random.default_rng(4).standard_normal(dims), e)
    plan = P.Plan(O.T4, dims, R, P_, variant=variant, dtype="f32", seed=6)
    one, got = sketches(P, plan, up, ALL), sketches(P, plan, T, ALL)
    tol = small_tol(max(np.prod(dims[:2]), np.prod(dims[2:])), e)
    bad = {n: v for n, a, b in zip(ALL, one, got) if not (v := errs2(np.ldexp(b, -e), a)[0]) <= tol}
    assert not bad, (bad, tol)


@pytest.mark.parametrize("variant", ["sttnn", "ttnn"])
@pytest.mark.parametrize("dims", SHAPES, ids=str)
@pytest.mark.parametrize("e", [-120, -140])
def test_small_rows_and_columns(P, variant, dims, e):
    """One row (i_1, i_2) and one column (i_3, i_4) of small values in a tensor of ordinary
    ones: their rows of the sketches of (1, 2) and (3, 4) are those of the values scaled up."""
    g = np.random.default_rng(5)
    T = g.standard_normal(dims).astype(np.float32)
    big = T.copy()
    T[77, 5], big[77, 5] = small(T[77, 5], e)
    col, up = small(T[:, :, 9, 13], e)
    T[:, :, 9, 13], big[:, :, 9, 13] = col, up
    T[77, 5, 9, 13] = big[77, 5, 9, 13] = 0.0
    plan = P.Plan(O.T4, dims, R, P_, variant=variant, dtype="f32", seed=6)
    row, cl = 77 + 128 * 5, 9 + dims[2] * 13
    for node, at, K in (((1, 2), row, np.prod(dims[2:])), ((3, 4), cl, np.prod(dims[:2]))):
        (a,), (b,) = (sketches(P, plan, x, [node]) for x in (big, T))
        err = np.linalg.norm(np.ldexp(b[at], -e) - a[at]) / np.linalg.norm(a[at])
        assert err <= small_tol(K, e), (node, err, small_tol(K, e))


@pytest.mark.parametrize("variant", ["sttnn", "ttnn"])
def test_rounding_has_no_direction(P, variant):
    """The sums of Y_A, Y_1 and X_B rows with the tensor (Z_A, Z_1 and R_B) are off to either
    side alike: their mean error is within five standard deviations of the mean of as many
    independent errors.  Sums that are all rounded one way add up over the 512 tiles of this
    tensor: R_B was 20 such deviations off.  Z_A is the root's sketch undone (its 32 columns times a
    32 x 48 map), Z_1's mean error a projection of R_2's errors on the columns' sums of X_2."""
    dims = (128, 1024, 32)
    g = torch.Generator(device="cuda").manual_seed(8)
    T = torch.randn(int(np.prod(dims)), generator=g, device="cuda", dtype=torch.float32)
    M = T.double().view(32, 128 * 1024).t()
    plan = P.Plan(((1, 2), 3), dims, R, P_, variant=variant, dtype="f32", seed=6)
    plan.update(T)
    A, B, one, two = (plan.node(m) for m in ((1, 2), (3,), (1,), (2,)))
    X = {v: plan.read_drm(v, 0) for v in (B, two)}
    Y = {v: plan.read_drm(v, 1) for v in (A, B, one)}
    k = R + P_
    ZA = Y[A].t() @ M
    off = {"Z_A": plan.read_sketch(0, P.SK_PSI).view(k, k).t() @ torch.linalg.pinv(Y[B]) - ZA}
    if variant == "ttnn":
        off["R_B"] = plan.read_sketch(B, P.SK_R) - M.t() @ X[B]
    else:
        Z1 = torch.einsum("cba,aj->bcj", M.t().reshape(32, 1024, 128), Y[one]).reshape(1024, -1)   # [i_2][(i_3, j)]
        X2 = X[two].view(32, k, R).reshape(32 * k, R)                                              # rows j + k i_3
        w = X2.sum(0)
        off["Z_1"] = (plan.read_sketch(two, P.SK_R) - Z1 @ X2) @ w / (w @ w)
    for name, d in off.items():
        sd = float(d.std()) / np.sqrt(d.numel())
        print(name, float(d.mean()) / sd, flush=True)
        assert abs(float(d.mean())) <= 5 * sd, (name, float(d.mean()), sd)
    plan.close()
