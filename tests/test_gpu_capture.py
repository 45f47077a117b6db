"""Whole-tensor updates of a plan without a one-pass or MFMA form pass their tables with the
launches: a captured update replays on the tensor's values of the moment, between eager
calls of the same plan and others, and gives the eager sketches bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def sketches(P, plan):
    return [plan.read_sketch(v, P.SK_PSI if v == 0 else P.SK_R) for v in range(plan.num_nodes)]


@pytest.mark.parametrize("dims,variant,dtype", [((16, 16, 16, 16), "ttnn", "f64"), ((33, 35, 37, 39), "sttnn", "f32"),
                                                ((97, 51, 61, 45), "ttnn", "bf16")], ids=str)
def test_captured_update_replays(dims, variant, dtype):
    import paper_2412_06111_amd as P
    spec = ((1, 2), (3, 4))
    n = 1
    for e in dims:
        n *= e
    tdt = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}[dtype]
    g = torch.Generator(device="cuda").manual_seed(3)
    tensors = [torch.randn(n, generator=g, device="cuda", dtype=torch.float32).to(tdt) for _ in range(4)]
    plan, other = (P.Plan(spec, dims, 6, 3, variant=variant, dtype=dtype, seed=s) for s in (4, 5))
    x = tensors[0].clone()
    plan.reset()
    plan.update(x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.reset()
        plan.update(x, alpha=0.5)
    for t in tensors:
        x.copy_(t)
        graph.replay()
        got = sketches(P, plan)
        other.update(t)                        # eager work of another plan in between
        plan.reset()
        plan.update(t, alpha=0.5)
        want = sketches(P, plan)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
