"""ccdc_node_decode_reduce with its row lists cut by rounds (units numbered by chunk) and at the edges of that rule, against the
plain sums; a node alone has the bits of the call for all nodes.  Whole numbers of a small range: every sum is exact, so the order of
addition does not matter.  Needs a GPU."""
from math import comb

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,r,m,T,mode", [
    (16, 3, 1, 4096, "h32"),              # by round, 32 chunks, five tiles and a part of one
    (16, 4, 1, 1028, "f32"),              # one pack past a wavefront's: lane-packed, equal cuts
    (11, 5, 1, 6336, "u32"),              # by round
    (13, 4, 7, 948, "bf16"),              # eight files' sums, short last segment
    (14, 5, 1, 281, "f32"),               # one-element packs, by round
    (9, 5, 1, 40704, "h32"),              # numbered by tile
    (12, 3, 2, 3456, "f16"),
    (10, 2, 1, 3544, "u32"),              # r = 2: equal cuts
])
def test_lists_by_round(K, r, m, T, mode):
    import torch

    import paper_1805_01993_amd as L
    assert torch.cuda.is_available(), "no GPU visible"
    plan = L.ccdc_plan(K, r, K, m * comb(K, r)).bind(T, mode).upload()
    sh = plan.shapes()
    dt = {"u32": torch.int32, "f32": torch.float32, "h32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[mode]
    g = torch.Generator(device="cuda").manual_seed(7)
    V = torch.randint(-2, 3, sh["V"], device="cuda", generator=g).to(dt)
    X = torch.zeros(sh["X"], dtype=dt, device="cuda")
    Phi = [torch.full(sh["Phi"], 77, dtype=dt, device="cuda") for _ in range(3)]
    plan.node_encode(-1, V, X)
    for _ in range(2):                     # twice: nothing is left over from a call
        plan.node_decode_reduce(-1, V, X, Phi[0])
        plan.node_decode_reduce(-1, V, X, Phi[1])
        assert torch.equal(Phi[0], Phi[1])
    for k in range(K):
        plan.node_decode_reduce(k, V, X, Phi[2])
    assert torch.equal(Phi[0].view(torch.int16), Phi[2].view(torch.int16))
    if mode == "u32":
        want = V[:, 0].clone()
        for n in range(1, V.shape[1]):
            want ^= V[:, n]
        assert torch.equal(Phi[0], want)
    else:
        # sums of at most 12000 numbers of -2..2 are whole numbers under 2^24; 16 bits round them once
        want = V.float().sum(1).to(dt)
        assert torch.equal(Phi[0], want)
    plan.close()
