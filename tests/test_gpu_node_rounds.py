"""ccdc_node_decode_reduce with its row lists cut by rounds (units numbered by chunk) and at the edges of that rule, against the
plain sums; a node alone has the bits of the call for all nodes.  Whole numbers of a small range first: every sum is exact, so the order
of addition does not matter.  Then numbers that round in every addition: it does.  Needs a GPU."""
from math import comb

import pytest

pytestmark = pytest.mark.gpu

# K, r, m, T, mode, whether lists are cut by rounds (test_sanitized_geometry.py asks the library)
LISTS = [
    (16, 3, 1, 4096, "h32", True),        # 32 chunks, five tiles and a part of one
    (16, 4, 1, 1028, "f32", False),       # one pack past a wavefront's: lane-packed, equal cuts
    (11, 5, 1, 6336, "u32", True),
    (13, 4, 7, 948, "bf16", True),        # seven files' sums, short last segment
    (13, 3, 1, 1280, "bf16", False),      # chunks of over twice the mean
    (14, 5, 1, 281, "f32", True),         # one-element packs
    (14, 3, 1, 6735, "f16", True),        # packs at any element
    (9, 5, 1, 40704, "h32", False),       # numbered by tile
    (10, 4, 4, 4096, "f16", True),
    (10, 2, 1, 3544, "u32", False),       # r = 2: equal cuts
]


@pytest.mark.parametrize("K,r,m,T,mode", [case[:5] for case in LISTS])
def test_lists_by_round(K, r, m, T, mode):
    import torch

    import paper_1805_01993_amd as L
    assert torch.cuda.is_available(), "no GPU visible"
    plan = L.ccdc_plan(K, r, K, m * comb(K, r)).bind(T, mode).upload()
    sh = plan.shapes()
    dt = {"u32": torch.int32, "f32": torch.float32, "h32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[mode]
    bits = torch.int16 if dt.itemsize == 2 else torch.int32
    X = torch.zeros(sh["X"], dtype=dt, device="cuda")

    def run(V):
        """Outputs of the call for all nodes, twice, and of the calls for each."""
        Phi = [torch.full(sh["Phi"], 77, dtype=dt, device="cuda") for _ in range(3)]
        plan.node_encode(-1, V, X)
        plan.node_decode_reduce(-1, V, X, Phi[0])
        plan.node_decode_reduce(-1, V, X, Phi[1])
        for k in range(K):
            plan.node_decode_reduce(k, V, X, Phi[2])
        assert torch.equal(Phi[0].view(bits), Phi[1].view(bits))
        assert torch.equal(Phi[0].view(bits), Phi[2].view(bits))
        return Phi[0]

    for seed in (7, 8):                    # other values in the same buffers: nothing is left over from a call
        g = torch.Generator(device="cuda").manual_seed(seed)
        V = torch.randint(-2, 3, sh["V"], device="cuda", generator=g).to(dt)
        Phi = run(V)
        if mode == "u32":
            want = V[:, 0].clone()
            for n in range(1, V.shape[1]):
                want ^= V[:, n]
            assert torch.equal(Phi, want)
        else:
            # sums of at most 12000 numbers of -2..2 are whole numbers under 2^24; 16 bits round them once
            assert torch.equal(Phi, V.float().sum(1).to(dt))
    if mode != "u32":
        V.normal_(generator=g)
        Phi = run(V).double()
        n = V.shape[1]
        want = torch.zeros(sh["Phi"], dtype=torch.float64, device="cuda")
        for file in V.unbind(1):
            want += file.double()
        # Errors of sums of n standard normal numbers in fp32: each addition rounds to within 2^-24 of a partial sum of sqrt(n) or so, as do
        # coding and decoding (r numbers); 8 sqrt(n) bounds the partial sums, and errors add up like sqrt(n).  A batch's sum and the
        # output are rounded to 16 bits once each.
        tol = 8 * n * 2.0 ** -24
        if dt.itemsize == 2:
            unit = 2.0 ** -8 if mode == "bf16" else 2.0 ** -11
            tol += unit * (want.abs() + 8 * (n if m > 1 else 0) ** 0.5)
        assert bool(((Phi - want).abs() <= tol).all())
    plan.close()
