"""Reads through and past the caches: the calls choose between the two by the bytes they move and by where rows begin,
so every call is run on either side of those lines, on rows that begin on whole cache lines and on rows that do not.
Field elements: every result is exact."""
import math

import pytest
import torch

import paper_1805_01993_amd as L

pytestmark = pytest.mark.gpu


def xor(t, dim):
    out = torch.zeros_like(t.select(dim, 0))
    for part in t.unbind(dim):
        out ^= part
    return out


# K, r, files a batch, T.  Four nodes, r = 2, one file a batch: an element of T stands for 24 of V, 12 of Vbar and D, 6 of X
# and 4 of Phi, so the limits of 64 MB (of what a stage reads and writes, map: reads) and 128 MB (the one-pass kernel) lie at
# T = 380952 for ccdc_shuffle_fused, 400000 for ccdc_reduce, 444444 for ccdc_combine, 571429 for ccdc_map, 941176 for
# ccdc_pipeline_fused.  That of 100 MB for one-element packets, which lengths take that four does not divide and whose segments
# have under 32 packs, lies at T = 243.5 for 60 nodes (102660 packets).
SHAPES = [(4, 2, 1, 8192), (4, 2, 1, 8190), (4, 2, 1, 8191), (4, 2, 1, 700_000), (4, 2, 1, 700_004),
          (4, 2, 1, 800_000), (4, 2, 1, 860_000), (4, 2, 1, 1_048_576), (4, 2, 1, 1_048_580),
          (4, 2, 1, 1_048_575), (4, 1, 2, 1_048_576), (4, 1, 2, 1_048_574), (4, 1, 2, 4096),
          (12, 3, 1, 8_192), (12, 3, 1, 8_196), (12, 3, 1, 8_193),
          (4, 2, 1, 380_928), (4, 2, 1, 380_960), (4, 2, 1, 399_968), (4, 2, 1, 400_032), (4, 2, 1, 444_416),
          (4, 2, 1, 444_448), (4, 2, 1, 571_424), (4, 2, 1, 571_456), (4, 2, 1, 941_152), (4, 2, 1, 941_184),
          (60, 2, 1, 243), (60, 2, 1, 245)]


def test_the_shapes_lie_on_both_sides():
    at = {"shuffle": (24 + 6 + 12, 64e6), "reduce": (24 + 12 + 4, 64e6), "combine": (24 + 12, 64e6), "map": (24 + 4, 64e6),
          "pipeline": (24 + 6 + 4, 128e6)}
    lengths = [T for K, r, m, T in SHAPES if (K, r, m) == (4, 2, 1)]
    for per, limit in at.values():
        near = [T for T in lengths if abs(T * per * 4 / limit - 1) < 2e-4 and T % 32 == 0]
        assert {T * per * 4 <= limit for T in near} == {True, False}
    one_element = [T for K, r, m, T in SHAPES if K == 60]
    assert all(T % 4 and (-(-T // 2) + 3) // 4 < 32 for T in one_element)
    assert {T * 3 * math.comb(60, 3) * 4 <= 100e6 for T in one_element} == {True, False}


@pytest.mark.parametrize("K,r,m,T", SHAPES)
def test_results_on_either_side_of_the_lines(K, r, m, T):
    N = m * math.comb(K, r)
    plan = L.ccdc_plan(K, r, K, N).bind(T, "u32").upload()
    sh = plan.shapes()
    g = torch.Generator(device="cuda").manual_seed(T)

    def values(shape):
        return torch.randint(-(1 << 31), 1 << 31, shape, dtype=torch.int32, device="cuda", generator=g)

    files, theta = values(sh["V"]), values(sh["Phi"])

    def new(name):
        return torch.full(sh[name], 7, dtype=torch.int32, device="cuda")

    V = new("V")
    plan.map(files, theta, V)
    assert torch.equal(V, files ^ theta.unsqueeze(1))
    del files
    want = xor(V, 1)
    X, Phi = new("X"), new("Phi")
    plan.pipeline_fused(V, X, Phi)
    assert torch.equal(Phi, want)
    Xs, D, Phi = new("X"), new("D"), new("Phi")
    plan.shuffle_fused(V, Xs, D)
    plan.reduce(V, D, Phi)
    assert torch.equal(Xs, X) and torch.equal(Phi, want)
    Vbar, Xe, De, Phi = new("Vbar"), new("X"), new("D"), new("Phi")
    plan.combine(V, Vbar)
    plan.encode(Vbar, Xe)
    plan.decode(Xe, Vbar, De)
    assert torch.equal(Xe, X) and torch.equal(De, Vbar) and torch.equal(D, Vbar)
    Xn = new("X")
    plan.node_encode(-1, V, Xn)
    plan.node_decode_reduce(-1, V, Xn, Phi)
    assert torch.equal(Xn, X) and torch.equal(Phi, want)
    plan.close()
