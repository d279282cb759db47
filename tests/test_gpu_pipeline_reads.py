"""ccdc_pipeline_fused on either side of the lines between its ways to read V and to number its workgroups.  X against
ccdc_encode's, Phi against the sum of V over the files.  Field elements, whole numbers of a small range, or sparse ones in
16 bits: exact.  Needs a GPU."""
from math import comb

import pytest
import torch

import paper_1805_01993_amd as L

pytestmark = pytest.mark.gpu


def moved(sh, eb):
    return sum(torch.Size(sh[key]).numel() for key in ("V", "X", "Phi")) * eb


def run(K, r, m, T, mode):
    """Runs the pass, checks it, and returns the plan's shapes and launch."""
    N, dt = m * comb(K, r), {"u32": torch.int32, "bf16": torch.bfloat16, "f16": torch.float16}.get(mode, torch.float32)
    plan = L.ccdc_plan(K, r, K, N).bind(T, mode).upload()
    sh, launch = plan.shapes(), plan.pipeline_launch()
    g = torch.Generator(device="cuda").manual_seed(T)
    if mode == "u32":
        V = torch.randint(-(1 << 31), 1 << 31, sh["V"], dtype=dt, device="cuda", generator=g)
    elif dt.itemsize == 2:
        V = (torch.rand(sh["V"], device="cuda", generator=g) < 8.0 / N).to(dt)      # sums stay far below 2^8
    else:
        V = torch.randint(-8, 9, sh["V"], device="cuda", generator=g).to(dt)
    X, Phi, want_X = (torch.full(sh[key], 77, dtype=dt, device="cuda") for key in ("X", "Phi", "X"))
    Vbar = torch.empty(sh["Vbar"], dtype=dt, device="cuda")
    plan.combine(V, Vbar)
    plan.encode(Vbar, want_X)
    del Vbar
    plan.pipeline_fused(V, X, Phi)
    bits = torch.int16 if dt.itemsize == 2 else torch.int32
    assert torch.equal(X.view(bits), want_X.view(bits)), "X differs from ccdc_encode's"
    if mode == "u32":
        want = V[:, 0].clone()
        for n in range(1, N):
            want ^= V[:, n]
        assert torch.equal(Phi, want)
    else:
        assert torch.equal(Phi.float(), V.float().sum(1))
    plan.close()
    return sh, launch, dt.itemsize


@pytest.mark.parametrize("K,r,m,T,mode", [
    (5, 1, 1, 100_003, "f32"),            # r = 1, one file a batch: the XCDs on runs of 16 tiles, the last runs shorter
    (5, 1, 1, 8_200, "u32"),              # 33 tiles of four-element packs: shorter runs throughout
    (6, 1, 1, 1_100_004, "u32"),          # the same on a large input
    (5, 1, 2, 100_003, "h32"),            # several files, r = 2: contiguous ranges of tiles
    (6, 2, 1, 100_003, "f32"),
    (5, 2, 1, 250_002, "bf16"),
])
def test_orders_of_the_workgroups(K, r, m, T, mode):
    _, launch, _ = run(K, r, m, T, mode)
    assert launch[2] == 1                 # one chunk
