"""The node-local calls on inputs large enough to be read past the caches (files only, or all of it), for all nodes and for
each alone.  Packets and outputs against the fused calls, which share their row order.  Field elements, or sparse ones in
16 bits: exact.  Needs a GPU."""
from math import comb

import pytest
import torch

import paper_1805_01993_amd as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,r,m,T,mode", [
    (4, 1, 1, 1_600_000, "u32"),          # r = 1: from 64 MB of values on
    (4, 1, 3, 700_008, "bf16"),
    (4, 2, 1, 3_200_000, "u32"),          # r = 2: 256 MB
    (4, 2, 1, 3_200_004, "u32"),          # rows and segments begin inside a line
    (4, 2, 2, 2_900_000, "f16"),
    (5, 3, 1, 3_400_000, "u32"),          # r = 3: 512 MB; a node alone: 640 MB
    (6, 4, 1, 2_400_000, "u32"),
    (6, 5, 1, 7_700_000, "u32"),
    (4, 2, 1, 6_700_001, "u32"),          # packs at any element, a node alone past the caches
    (26, 4, 1, 495, "u32"),               # one-element packs (segments of under 32 packs), the same
    (7, 6, 1, 3_400_000, "u32"),          # the lane-packed kernels, the same
])
def test_large_inputs(K, r, m, T, mode):
    N, dt = m * comb(K, r), {"u32": torch.int32, "bf16": torch.bfloat16, "f16": torch.float16}[mode]
    plan = L.ccdc_plan(K, r, K, N).bind(T, mode).upload()
    sh = plan.shapes()
    values = N * K * T * dt.itemsize
    assert values > {1: 64e6, 2: 256e6, 3: 512e6, 4: 768e6, 5: 1024e6}.get(r, 640e6)
    g = torch.Generator(device="cuda").manual_seed(T)
    if mode == "u32":
        V = torch.randint(-(1 << 31), 1 << 31, sh["V"], dtype=dt, device="cuda", generator=g)
    else:
        V = (torch.rand(sh["V"], device="cuda", generator=g) < 4.0 / N).to(dt)
    new = lambda key: torch.full(sh[key], 77, dtype=dt, device="cuda")
    X, D, Phi, Xn, Phin = new("X"), new("D"), new("Phi"), new("X"), new("Phi")
    plan.shuffle_fused(V, X, D)
    plan.reduce(V, D, Phi)
    del D
    bits = torch.int16 if dt.itemsize == 2 else torch.int32
    plan.node_encode(-1, V, Xn)
    plan.node_decode_reduce(-1, V, Xn, Phin)
    assert torch.equal(Xn.view(bits), X.view(bits)) and torch.equal(Phin, Phi)
    Xn.fill_(5), Phin.fill_(5)
    for k in range(K):
        plan.node_encode(k, V, Xn)
    for k in range(K):
        plan.node_decode_reduce(k, V, Xn, Phin)
    assert torch.equal(Xn.view(bits), X.view(bits)) and torch.equal(Phin, Phi)
    plan.close()
