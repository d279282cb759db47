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


# K, r, files a batch, T, mode, whether packs of 16 bytes; each moves more than the 128 MB that are always read through the caches
PAST = [
    (8, 2, 1, 400_000, "f32", True),      # rows on whole lines
    (7, 3, 1, 480_000, "u32", True),
    (7, 4, 1, 409_600, "h32", True),
    (6, 5, 1, 1_041_600, "f32", True),
    (4, 1, 10, 320_000, "f32", True),     # one step in flight
    (6, 2, 4, 320_000, "u32", True),
    (5, 3, 12, 409_152, "h32", True),
    (8, 2, 1, 300_002, "h32", True),      # wide packs whose tiles share sectors, up to 1.4 GB
    (7, 3, 1, 300_001, "f32", True),
    (5, 4, 1, 3_000_004, "u32", True),
    (6, 5, 1, 1_841_604, "f32", True),
    (9, 5, 1, 100_003, "u32", True),      # the same in chunks
    (6, 3, 10, 125_001, "h32", True),
    (6, 2, 12, 70_002, "f32", True),
    (8, 2, 1, 800_000, "bf16", False),    # narrow packs on whole lines
    (7, 3, 1, 480_000, "f16", False),
    (8, 4, 1, 320_000, "bf16", False),
    (7, 5, 1, 800_000, "f16", False),
    (6, 3, 8, 96_000, "bf16", False),
    (6, 1, 4, 704_000, "f16", False),
    (10, 4, 8, 2048, "f32", False),
]
KEPT = [
    (8, 2, 1, 400_001, "bf16", False),    # narrow packs whose tiles share lines
    (7, 3, 1, 480_004, "f16", False),
    (6, 3, 8, 96_001, "bf16", False),
    (9, 4, 8, 4100, "u32", False),
    (18, 1, 1, 51_921, "f32", True),      # wide ones up to 200 MB, r <= 2
    (24, 2, 1, 3373, "u32", True),
    (5, 2, 1, 6_485_985, "f32", True),    # wide ones from 1.4 GB on
    (7, 3, 1, 1_380_769, "u32", True),
]


@pytest.mark.parametrize("K,r,m,T,mode,wide", PAST + KEPT)
def test_large_inputs(K, r, m, T, mode, wide):
    sh, launch, eb = run(K, r, m, T, mode)
    assert (launch[0] * eb == 16) == wide
    size, shares = moved(sh, eb), T * eb % (32 if wide else 128) or sh["X"][2] * eb % (32 if wide else 128)
    assert size > 128e6
    assert ((K, r, m, T, mode, wide) in KEPT) == bool(shares and (not wide or size >= 1.4e9 or r <= 2 and size <= 200e6))
