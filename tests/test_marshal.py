"""The native argument marshalling of binding.py: what it takes goes to the library with the right arguments, everything else
is left to the checks in Python, with the messages these have."""
import pytest
import torch

import paper_1805_01993_amd as L
from paper_1805_01993_amd import binding as B


def test_it_leaves_what_is_not_ordinary():
    plan = L.ccdc_plan(4, 2, 4, 12).bind(16, "f32")
    sh = plan.shapes()
    V, X, Phi = (torch.zeros(sh[k]) for k in ("V", "X", "Phi"))
    quick = plan._quickly()
    assert type(quick).__name__ == "Marshal"          # built with the library
    for args in [(B._PIPELINE, V, X, Phi), (B._PIPELINE, V, X), (B._PIPELINE, V, X, None), (B._PIPELINE,), (), (99, V, X, Phi),
                 (-1, V), ("x", V, X, Phi), (B._NODE_ENCODE, 1.0, V, X), (B._NODE_ENCODE, -2, V, X), (B._NODE_ENCODE, 1 << 40, V, X)]:
        assert quick(*args) is None                   # host tensors, wrong counts and types
    with pytest.raises(ValueError, match="V: need a contiguous device tensor"):
        plan.pipeline_fused(V, X, Phi)
    with pytest.raises(ValueError, match="X: need"):
        plan._need(V, "X", "X")
    plan.close()
    assert plan._quick is None


@pytest.mark.parametrize("node", [1 << 31, (1 << 63) - 1, 1 << 63, 1 << 64, -(1 << 63), -(1 << 63) - 1])
def test_node_numbers_that_do_not_fit_are_left(node):
    plan = L.ccdc_plan(4, 2, 4, 12).bind(16, "f32")
    sh = plan.shapes()
    V, X, Phi = (torch.zeros(sh[k]) for k in ("V", "X", "Phi"))
    assert plan._quickly()(B._NODE_ENCODE, node, V, X) is None
    with pytest.raises(ValueError, match="V: need a contiguous device tensor"):
        plan.node_encode(node, V, X)
    with pytest.raises(ValueError, match="V: need a contiguous device tensor"):
        plan.node_decode_reduce(node, V, X, Phi)
    plan.close()


def test_unbound_plans_answer_as_before():
    plan = L.ccdc_plan(4, 2, 4, 12)
    with pytest.raises(B.CcdcError):
        plan.pipeline_fused(torch.zeros(1), torch.zeros(1), torch.zeros(1))


@pytest.mark.gpu
def test_calls_reach_the_library():
    plan = L.ccdc_plan(5, 2, 5, 10).bind(40, "u32").upload()
    sh = plan.shapes()
    g = torch.Generator(device="cuda").manual_seed(1)
    V = torch.randint(-(1 << 31), 1 << 31, sh["V"], dtype=torch.int32, device="cuda", generator=g)
    new = lambda key: torch.full(sh[key], 5, dtype=torch.int32, device="cuda")
    theta = V[:, 0].clone()

    def outputs(stream):                              # stream=None: native; an explicit one: through Python
        M, Vbar, X, D, D2, X2, X3, X4, X5 = map(new, ("V", "Vbar", "X", "D", "D", "X", "X", "X", "X"))
        P = [new("Phi") for _ in range(5)]
        plan.map(V, theta, M, stream=stream)
        plan.combine(V, Vbar, stream=stream)
        plan.encode(Vbar, X, stream=stream)
        plan.decode(X, Vbar, D, stream=stream)
        plan.reduce(V, D, P[0], stream=stream)
        plan.shuffle_fused(V, X2, D2, stream=stream)
        plan.pipeline_fused(V, X3, P[1], stream=stream)
        plan.pipeline_fused_noalloc(V, X4, P[2], stream=stream)
        plan.node_encode(-1, V, X5, stream=stream)
        plan.node_decode_reduce(-1, V, X5, P[3], stream=stream)
        plan.node_decode_reduce(3, V, X5, P[4], stream=stream)
        return [M, Vbar, X, D, D2, X2, X3, X4, X5] + P

    plan._quickly()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                     # the current stream is taken
        quick = outputs(None)
    side.synchronize()
    for a, b in zip(quick, outputs(torch.cuda.current_stream())):
        assert torch.equal(a, b)


@pytest.mark.gpu
def test_modes_that_intercept_calls_see_the_tensors():
    class Seen(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            names.append(getattr(func, "__name__", ""))
            return func(*args, **(kwargs or {}))

    names = []
    plan = L.ccdc_plan(4, 2, 4, 12).bind(16, "f32").upload()
    sh = plan.shapes()
    V = torch.ones(sh["V"], device="cuda")
    X, Phi, Phi2 = (torch.zeros(sh[k], device="cuda") for k in ("X", "Phi", "Phi"))
    plan.pipeline_fused(V, X, Phi)
    assert type(plan._quick).__name__ == "Marshal"
    with Seen():
        plan.pipeline_fused(V, X, Phi2)
    assert names.count("numel") == names.count("data_ptr") == 3       # of V, X and Phi, in the checks in Python
    assert torch.equal(Phi, Phi2) and bool((Phi == 12).all())
    plan.close()


@pytest.mark.gpu
def test_refusals_are_those_of_the_checks():
    plan = L.ccdc_plan(4, 2, 4, 12).bind(16, "f32").upload()
    sh = plan.shapes()
    V, X, Phi = (torch.zeros(sh[k], device="cuda") for k in ("V", "X", "Phi"))
    plan.pipeline_fused(V, X, Phi)
    assert type(plan._quick).__name__ == "Marshal"
    wrong = [((V[:, :3], X, Phi), "V: need"), ((V.half(), X, Phi), "V: need 4-byte elements"), ((V, X.cpu(), Phi), "X: need a contiguous"),
             ((V.transpose(1, 3), X, Phi), "V: need a contiguous")]
    for args, message in wrong:
        with pytest.raises(ValueError, match=message):
            plan.pipeline_fused(*args)
    plan.pipeline_fused(torch.nn.Parameter(V), X, Phi)                # a subclass: through Python
    with pytest.raises(B.CcdcError, match="ccdc_node_encode"):
        plan.node_encode(4, V, X)                     # the library's own refusal
    jobs = L.ccdc_plan_jobs(4, 2, 4, 6).bind(16, "f32").upload()
    s2 = jobs.shapes()
    with pytest.raises(B.CcdcError, match="ccdc_pipeline_fused"):
        jobs.pipeline_fused(*(torch.zeros(s2[k], device="cuda") for k in ("V", "X", "Phi")))
    plan.bind(32, "bf16").upload()                    # sizes and elements of the new binding
    with pytest.raises(ValueError):
        plan.pipeline_fused(V, X, Phi)
    sh = plan.shapes()
    V, X, Phi = (torch.zeros(sh[k], device="cuda", dtype=torch.bfloat16) for k in ("V", "X", "Phi"))
    plan.pipeline_fused(V, X, Phi)
    plan.close()
    with pytest.raises(B.CcdcError):
        plan.pipeline_fused(V, X, Phi)
