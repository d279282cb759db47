"""Batches of several files whose packs are asked for together (packs of less than 16 bytes): every count of files around the
steps of four, two and one, segments that fill wavefronts and that do not, one output pack more or less.  Whole numbers of a
small range, exact in every order: decoded packets against combined ones, coded packets of the three calls that make them
against each other, outputs against the sum of V over the files.  Plans of several jobs, which never decode by receiver.  Needs a
GPU."""
import pytest
import torch

import paper_1805_01993_amd as L

pytestmark = pytest.mark.gpu
DTYPES = {"u32": torch.int32, "bf16": torch.bfloat16, "f16": torch.float16}


def values(sh, mode):
    dt = DTYPES.get(mode, torch.float32)
    g = torch.Generator(device="cuda").manual_seed(sh["V"][-1])
    low, high = (-(1 << 31), 1 << 31) if mode == "u32" else (-1, 2)
    V = torch.randint(low, high, sh["V"], device="cuda", generator=g, dtype=torch.int32)
    if mode == "u32":
        want = V[:, 0].clone()
        for n in range(1, V.shape[1]):
            want ^= V[:, n]
        return V, want
    if dt.itemsize == 2:                             # packets of up to 9 files, coded of up to 5: below 2^8; sums as well
        V *= torch.rand(sh["V"], device="cuda", generator=g) < 30.0 / sh["V"][1]
    return V.to(dt), V.sum(1).to(dt)


MODES = ["u32", "f32", "h32", "bf16", "f16"]
LENGTHS = [1, 2, 71, 259, 646, 1030, 2049]
FILES = [(1, 2), (1, 7), (2, 2), (2, 3), (2, 6), (3, 2), (3, 5), (4, 2), (4, 3), (4, 9), (5, 2), (5, 4), (6, 3)]      # r, files a batch


@pytest.mark.parametrize("T", LENGTHS)
@pytest.mark.parametrize("r,m", FILES)
def test_coded_plans(r, m, T):
    K, mode = r + 2, MODES[(FILES.index((r, m)) + LENGTHS.index(T)) % 5]
    plan = L.ccdc_plan_jobs(K, r, K, m * (r + 1)).bind(T, mode).upload()
    assert plan.reduce_launch()[2:] == (0, 0)
    sh = plan.shapes()
    V, want = values(sh, mode)
    new = lambda key: torch.full(sh[key], 55, dtype=V.dtype, device="cuda")  # noqa: E731
    Vbar, X, X2, X3, D, Phi = (new(k) for k in ("Vbar", "X", "X", "X", "D", "Phi"))
    plan.combine(V, Vbar)
    plan.encode(Vbar, X)
    plan.shuffle_fused(V, X2, D)
    plan.node_encode(-1, V, X3)
    bits = torch.int16 if V.dtype.itemsize == 2 else torch.int32       # coded words may be NaN
    assert torch.equal(X.view(bits), X2.view(bits)) and torch.equal(X.view(bits), X3.view(bits))
    assert torch.equal(D, Vbar)
    plan.reduce(V, D, Phi)
    assert torch.equal(Phi, want)
    Phi.fill_(55)
    plan.node_decode_reduce(-1, V, X, Phi)
    assert torch.equal(Phi, want)
    Phi.fill_(55)
    for k in range(K):
        plan.node_encode(k, V, X3.fill_(55) if k == 0 else X3)
        plan.node_decode_reduce(k, V, X, Phi)
    assert torch.equal(X.view(bits), X3.view(bits)) and torch.equal(Phi, want)
    plan.close()


@pytest.mark.parametrize("T", [1, 259, 2050])
@pytest.mark.parametrize("K,r,N", [(4, 3, 40), (5, 1, 40), (13, 3, 26), (24, 2, 96)])     # batches of several sizes
def test_uncoded_plans(K, r, N, T):
    plan = L.ccdc_plan_compression(K, r, K, N).bind(T, "u32").upload()
    sh = plan.shapes()
    V, want = values(sh, "u32")
    Vbar, Phi = (torch.full(sh[k], 55, dtype=V.dtype, device="cuda") for k in ("Vbar", "Phi"))
    plan.combine(V, Vbar)
    plan.reduce(V, Vbar, Phi)
    assert torch.equal(Phi, want)
    plan.close()
