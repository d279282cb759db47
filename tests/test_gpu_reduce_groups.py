"""ccdc_reduce where one workgroup sums a whole row list (few outputs): short and long lists, one pack more or less than a
workgroup covers, the pack widths, and the lines to the split form.  The path up to the decoded packets, then the outputs
against the sum of V over the files.  Field elements, or sparse ones in 16 bits: exact.  Needs a GPU."""
from math import comb

import pytest
import torch

import paper_1805_01993_amd as L

pytestmark = pytest.mark.gpu


def run(plan, T, mode, whole_lists):
    plan.bind(T, mode).upload()
    split, waves = plan.reduce_launch()[:2]
    assert (waves > 0) == (split > 1 and whole_lists)
    sh, dt = plan.shapes(), {"u32": torch.int32, "bf16": torch.bfloat16, "f16": torch.float16}[mode]
    g = torch.Generator(device="cuda").manual_seed(T)
    if mode == "u32":
        V = torch.randint(-(1 << 31), 1 << 31, sh["V"], dtype=dt, device="cuda", generator=g)
        want = V[:, 0].clone()
        for n in range(1, V.shape[1]):
            want ^= V[:, n]
    else:
        V = (torch.rand(sh["V"], device="cuda", generator=g) < 8.0 / V_files(sh)).to(dt)      # sums stay far below 2^8
        want = V.double().sum(1).to(dt)
    n = torch.Size(sh["Phi"]).numel()
    whole = torch.full((n + 16,), 7, dtype=dt, device="cuda")
    Phi = whole[8:8 + n].view(sh["Phi"])
    if plan.compression:
        D = torch.empty(sh["Vbar"], dtype=dt, device="cuda")
        plan.combine(V, D)
    else:
        X, D = (torch.empty(sh[k], dtype=dt, device="cuda") for k in ("X", "D"))
        plan.shuffle_fused(V, X, D)
    plan.reduce(V, D, Phi)
    assert torch.equal(Phi, want)
    assert bool((whole[:8] == 7).all()) and bool((whole[8 + n:] == 7).all())
    plan.close()


def V_files(sh):
    return sh["V"][1]


LENGTHS = [1, 3, 64, 66, 256, 260, 511, 512, 2048, 2056]
SHAPES = [(4, 1, 1), (5, 2, 3), (7, 3, 1), (10, 4, 2), (11, 5, 2)]      # K, r, files a batch: 4 to 672 rows a list


@pytest.mark.parametrize("T", LENGTHS)
@pytest.mark.parametrize("K,r,m", SHAPES)
def test_lists_of_coded_plans(K, r, m, T):
    mode = ["u32", "bf16", "f16"][(SHAPES.index((K, r, m)) + LENGTHS.index(T)) % 3]
    rows = m * comb(K - 1, r - 1) + comb(K - 1, r)
    run(L.ccdc_plan(K, r, K, m * comb(K, r)), T, mode, rows <= 640)


@pytest.mark.parametrize("T", [1, 63, 64, 65, 1024, 1028, 20002])
@pytest.mark.parametrize("K,r,N", [(4, 3, 40), (5, 1, 40), (13, 3, 26), (24, 2, 96)])             # batches of several sizes
def test_lists_of_uncoded_plans(K, r, N, T):
    run(L.ccdc_plan_compression(K, r, K, N), T, "u32", True)


@pytest.mark.parametrize("T", [5, 256, 1000])
@pytest.mark.parametrize("K,r,N", [(5, 2, 6), (6, 3, 8), (8, 2, 9)])
def test_lists_of_many_jobs(K, r, N, T):
    run(L.ccdc_plan_jobs(K, r, K, N), T, "u32", True)


@pytest.mark.parametrize("K,T", [(8, 131068), (8, 131072), (8, 131076)])      # 2^18 packs of all outputs, one launch from there on
def test_where_outputs_fill_the_chip(K, T):
    run(L.ccdc_plan_compression(K, 2, K, 16), T, "u32", True)
