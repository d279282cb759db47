"""ccdc_pipeline_fused and ccdc_node_decode_reduce on small inputs, where a workgroup makes outputs of one node.  Packets
against ccdc_shuffle_fused's bit for bit, outputs against ccdc_shuffle_fused + ccdc_reduce on whole numbers of a small range (field elements; sparse ones in 16
bits), which are exact in every order; and the lines between this form and the one-pass kernel.  Needs a GPU."""
from math import comb

import pytest
import torch

import paper_1805_01993_amd as L

pytestmark = pytest.mark.gpu
BY_RECEIVER = 4                                      # flag of pipeline_launch()
DTYPES = {"u32": torch.int32, "bf16": torch.bfloat16, "f16": torch.float16}


def run(K, r, c, m, T, mode, shift=0):
    N, dt = m * comb(K, r), DTYPES.get(mode, torch.float32)
    plan = L.ccdc_plan(K, r, c * K, N).bind(T, mode).upload()
    sh, launch, sums = plan.shapes(), plan.pipeline_launch(), plan.reduce_launch()
    g = torch.Generator(device="cuda").manual_seed(T)

    def buf(key, fill):                              # `shift` elements past an aligned address, the same around it
        n = torch.Size(sh[key]).numel()
        whole = torch.full((n + shift + 8,), fill, dtype=dt, device="cuda")
        return whole, whole[shift:shift + n].view(sh[key])

    V = buf("V", 0)[1]
    if mode == "u32":
        V.copy_(torch.randint(-(1 << 31), 1 << 31, sh["V"], dtype=dt, device="cuda", generator=g))
    elif dt.itemsize == 2:
        V.copy_((torch.rand(sh["V"], device="cuda", generator=g) < 8.0 / N).to(dt))      # sums stay far below 2^8
    else:
        V.copy_(torch.randint(-8, 9, sh["V"], device="cuda", generator=g).to(dt))
    (Xall, X), (Pall, Phi), (_, want_X), (_, want), (_, D) = (buf(key, 77) for key in ("X", "Phi", "X", "Phi", "D"))
    plan.shuffle_fused(V, want_X, D)
    plan.reduce(V, D, want)
    bits = torch.int16 if dt.itemsize == 2 else torch.int32
    for call in (plan.pipeline_fused, plan.pipeline_fused_noalloc):
        X.fill_(55), Phi.fill_(55)
        call(V, X, Phi)
        assert torch.equal(X.view(bits), want_X.view(bits)), "X differs"
        assert torch.equal(Phi, want), "Phi differs"
    Phi.fill_(55)
    plan.node_decode_reduce(-1, V, want_X, Phi)
    assert torch.equal(Phi, want), "node-local Phi differs"
    Phi.fill_(55)
    for k in range(K):                               # each node reads its own files and the packets sent to it
        plan.node_decode_reduce(k, V, want_X, Phi)
    assert torch.equal(Phi, want), "one node's Phi differs"
    for whole, inner in ((Xall, X), (Pall, Phi)):    # nothing outside the outputs was written
        assert bool((whole[:shift] == 77).all()) and bool((whole[shift + inner.numel():] == 77).all())
    plan.close()
    return bool(launch[3] & BY_RECEIVER), sums[3] > 0


# K, r, functions a node, files a batch, T, mode: plans of this form, in node-local decoding too but for two of many rounds or files
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("K,r,c,m,T,mode", [
    (9, 1, 1, 1, 64, "f32"), (13, 1, 1, 1, 1168, "u32"), (24, 1, 1, 1, 1036, "f16"),      # one pack a coded pack
    (21, 1, 1, 5, 101, "bf16"), (20, 1, 1, 10, 729, "u32"), (19, 1, 1, 4, 876, "h32"),    # several files
    (9, 2, 1, 1, 193, "bf16"), (10, 2, 2, 1, 340, "f16"), (11, 2, 1, 1, 512, "u32"), (11, 2, 1, 1, 5536, "h32"),
    (6, 2, 1, 6, 1366, "u32"), (5, 2, 1, 8, 5184, "h32"),
    (7, 3, 1, 1, 64, "f32"), (7, 3, 1, 1, 211, "f32"), (7, 3, 1, 1, 212, "bf16"), (8, 3, 1, 1, 2048, "h32"),
    (6, 3, 1, 5, 892, "u32"), (5, 3, 1, 5, 2666, "bf16"),
    (7, 4, 1, 1, 223, "bf16"), (7, 4, 2, 1, 1726, "u32"), (6, 4, 2, 2, 2956, "u32"), (8, 4, 1, 1, 2922, "h32"),
    (7, 5, 1, 1, 464, "bf16"), (7, 5, 2, 8, 202, "h32"), (9, 5, 1, 1, 1344, "f16"),
])
def test_by_receiver(K, r, c, m, T, mode, shift):
    assert run(K, r, c, m, T, mode, shift) == (True, (K, r) not in ((20, 1), (9, 5)))


@pytest.mark.parametrize("K,r,c,T,mode,receiver", [
    (20, 1, 2, 7500, "h32", True),        # r = 1: 48.0 MB moved, and more
    (20, 1, 2, 7510, "h32", False),
    (11, 2, 1, 6900, "u32", True),        # 23.8 MB, and 24.2
    (11, 2, 1, 7000, "u32", False),
    (17, 3, 1, 134, "u32", False),        # small, but a node is in 560 rounds
])
def test_where_the_line_lies(K, r, c, T, mode, receiver):
    assert run(K, r, c, 1, T, mode)[0] == receiver


# files a batch are summed; a plan by receiver in both calls or in neither, packs of one and of four elements
@pytest.mark.parametrize("K,r,m,T", [(5, 2, 2, 64), (6, 3, 3, 256), (4, 1, 5, 640), (7, 4, 2, 260), (5, 2, 2, 37), (6, 2, 9, 259),
                                     (7, 3, 2, 40000), (6, 2, 5, 60001)])
def test_numbers_beside_nans(K, r, m, T):
    """h32: a batch may sum NaNs of several patterns.  Every call codes the same pattern for it, so it comes out of a coded packet
    whole and what is decoded beside it stays the number that it is."""
    N = m * comb(K, r)
    plan = L.ccdc_plan(K, r, K, N).bind(T, "h32").upload()
    sh = plan.shapes()
    g = torch.Generator(device="cuda").manual_seed(T)
    V = torch.randint(-8, 9, sh["V"], device="cuda", generator=g).float()
    bits, pick = V.view(torch.int32), torch.rand(sh["V"], device="cuda", generator=g)
    for i, pattern in enumerate((0x7FC12345, 0x7F800001, 0xFFC54321 - (1 << 32), 0x7FC00000, 0x80000000 - (1 << 32))):
        bits[(pick >= 0.01 * i) & (pick < 0.01 * (i + 1))] = pattern
    Vbar, X, X2, X3, X4, D, D2, P1, P2, P3, P4 = (torch.empty(sh[k], device="cuda")
                                                  for k in "Vbar X X X X D D Phi Phi Phi Phi".split())
    same = lambda a, b: torch.equal(a.view(torch.int32), b.view(torch.int32))  # noqa: E731
    plan.combine(V, Vbar), plan.encode(Vbar, X), plan.decode(X, Vbar, D), plan.reduce(V, D, P1)
    plan.shuffle_fused(V, X2, D2), plan.pipeline_fused(V, X3, P2)
    plan.node_encode(-1, V, X4), plan.node_decode_reduce(-1, V, X, P3)
    for k in range(K):
        plan.node_decode_reduce(k, V, X, P4)
    assert same(D, Vbar) and same(D2, Vbar)
    assert same(X2, X) and same(X4, X) and same(X3, X)
    nan = V.isnan().any(1)
    want = V.sum(1)
    for Phi in (P1, P2, P3, P4):
        assert torch.equal(Phi.isnan(), nan) and torch.equal(Phi[~nan], want[~nan])
    plan.close()
