"""Value lengths that no pack divides, on inputs large enough for 16-byte packs at any element, and pointers that are only aligned to
an element: every call against plain sums and against each other.  Whole numbers of a small range, so every sum is exact.  Needs a GPU."""
from math import comb

import pytest

pytestmark = pytest.mark.gpu


def tensors(torch, plan, T, mode, shift):
    """new(key, fill): a tensor of the plan's shape that begins `shift` elements into a buffer, between guards."""
    sh = plan.shapes()
    dt = {"u32": torch.int32, "bf16": torch.bfloat16, "f16": torch.float16}.get(mode, torch.float32)
    whole = []

    def new(key, fill=77):
        n = torch.Size(sh[key]).numel()
        buf = torch.full((n + 16,), fill, dtype=dt, device="cuda")
        whole.append((buf, shift, n, fill))
        return buf[shift:shift + n].view(sh[key])

    def intact():
        return all(bool((b[:s] == f).all()) and bool((b[s + n:] == f).all()) for b, s, n, f in whole)
    return new, intact, dt


def plain(torch, V, mode, dt):
    if mode != "u32":
        return V.float().sum(1).to(dt)
    want = V[:, 0].clone()
    for n in range(1, V.shape[1]):
        want ^= V[:, n]
    return want


# K, r, c, m, T, mode and which calls are made of 16-byte packs at any element, where pointers are aligned to their elements only: map,
# combine, encode, decode, reduce, fused shuffle, node-local sending and decoding, those two for one node (test_sanitized_geometry.py asks the
# library).  Lists that are not cut and cut ones, by round and in equal parts; segments that fill wavefronts and (19 nodes) that do not; last
# segments one element short of a pack, one long, of whole packs; several files; r beyond what decoding by sender is unrolled for; a length
# that packs divide, for the pointers alone.
CODED = [
    (6, 2, 1, 1, 140001, "bf16", "1111011010"), (6, 2, 1, 1, 90002, "f32", "1111001000"), (7, 3, 1, 1, 150003, "u32", "1111101100"),
    (5, 1, 1, 1, 420003, "f16", "1111111110"), (5, 1, 2, 2, 150001, "h32", "1111101110"), (7, 4, 1, 3, 40005, "bf16", "1111000000"),
    (8, 6, 1, 1, 60001, "bf16", "1110001000"), (13, 3, 1, 5, 6031, "bf16", "1111101101"), (14, 3, 1, 1, 6735, "f16", "1111111111"),
    (14, 3, 1, 1, 6735, "u32", "1111101101"), (19, 4, 1, 1, 525, "u32", "1111101101"), (7, 3, 1, 2, 360003, "f16", "1111111110"),
    (9, 5, 2, 4, 3381, "f16", "1110100101"), (6, 2, 1, 1, 140000, "f16", "1111011010"), (7, 5, 2, 1, 3011, "h32", "1100000000"),
]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("K,r,c,m,T,mode", [case[:6] for case in CODED])
def test_calls_of_coded_plans(K, r, c, m, T, mode, shift):
    import torch

    import paper_1805_01993_amd as L
    assert torch.cuda.is_available(), "no GPU visible"
    plan = L.ccdc_plan(K, r, c * K, m * comb(K, r)).bind(T, mode).upload()
    new, intact, dt = tensors(torch, plan, T, mode, shift)
    g = torch.Generator(device="cuda").manual_seed(T + shift)
    V = new("V")
    V.copy_(torch.randint(-2, 3, V.shape, device="cuda", generator=g))
    X, Xf, Xn, Vbar, D, Df = (new(k) for k in "X X X Vbar D D".split())
    Phi, Pf, Pn, P1 = (new("Phi") for _ in range(4))
    plan.combine(V, Vbar), plan.encode(Vbar, X), plan.decode(X, Vbar, D), plan.reduce(V, D, Phi)
    plan.shuffle_fused(V, Xf, Df), plan.reduce(V, Df, Pf)
    plan.node_encode(-1, V, Xn), plan.node_decode_reduce(-1, V, Xn, Pn)
    for k in range(K):
        plan.node_decode_reduce(k, V, Xn, P1)
    bits = lambda t: t.view(torch.int16 if t.element_size() == 2 else torch.int32)  # noqa: E731
    assert torch.equal(bits(D), bits(Vbar)) and torch.equal(bits(Df), bits(Vbar))
    assert torch.equal(bits(Xf), bits(X)) and torch.equal(bits(Xn), bits(X))
    want = plain(torch, V, mode, dt)
    for got in (Phi, Pf, Pn, P1):
        assert torch.equal(got, want)
    files, theta, out = new("V"), new("Phi"), new("V")
    files.copy_(torch.randint(-2, 3, V.shape, device="cuda", generator=g))
    theta.copy_(torch.randint(-2, 3, theta.shape, device="cuda", generator=g))
    plan.map(files, theta, out)
    want = theta.unsqueeze(1) ^ files if mode == "u32" else theta.unsqueeze(1) - files
    assert torch.equal(out, want)
    plan.map(files, theta, files)          # in place
    assert torch.equal(files, want)
    assert intact()
    plan.close()


# K, r, N, T (f32), the same for map, combine and reduce
UNCODED = [(13, 3, 26, 90001, "111"), (5, 1, 40, 220003, "111"), (9, 5, 18, 120002, "111"), (9, 5, 18, 50002, "100"), (24, 2, 144, 7003, "110")]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("K,r,N,T", [case[:4] for case in UNCODED])
def test_uncoded_plans(K, r, N, T, shift):
    import torch

    import paper_1805_01993_amd as L
    assert torch.cuda.is_available(), "no GPU visible"
    plan = L.ccdc_plan_compression(K, r, K, N).bind(T, "f32").upload()
    new, intact, dt = tensors(torch, plan, T, "f32", shift)
    V, Vbar, Phi = new("V"), new("Vbar"), new("Phi")
    V.copy_(torch.randint(-2, 3, V.shape, device="cuda"))
    plan.combine(V, Vbar), plan.reduce(V, Vbar, Phi)
    assert torch.equal(Phi, V.sum(1))
    assert intact()
    plan.close()
