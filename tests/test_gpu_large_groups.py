"""Workgroups of the one-pass kernel that take more than 64 KB of LDS (up to the 160 KB of a compute unit): plans with
many running outputs a lane, packs of every width the choice gives, a packet's last segment whole, short and one that a
pack straddles.  Field elements, or whole numbers of a small range (sparse ones in 16 bits): sums are exact."""
from math import comb

import pytest
import torch

import paper_1805_01993_amd as L

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,r,c,m,T,mode", [
    (16, 3, 1, 1, 4096, "f32"),          # short last segment
    (16, 3, 1, 1, 3072, "h32"),          # whole segments
    (16, 3, 1, 1, 4098, "u32"),          # a pack straddles the packet's end
    (16, 3, 1, 8, 762, "f16"),           # several files a batch
    (16, 4, 1, 6, 257, "bf16"),
    (24, 3, 1, 2, 2048, "f32"),
    (22, 4, 1, 1, 88, "h32"),
    (14, 4, 2, 1, 879, "f32"),
    (19, 4, 1, 1, 861, "bf16"),
    (15, 5, 1, 1, 192, "f32"),
    (17, 5, 1, 1, 235, "u32"),
    (18, 2, 1, 1, 57076, "f16"),         # r = 2, a large input
    (24, 3, 1, 8, 432, "bf16"),          # large inputs with several files
    (22, 4, 1, 6, 576, "f16"),
])
def test_workgroups_over_64_kilobytes(K, r, c, m, T, mode):
    N = m * comb(K, r)
    plan = L.ccdc_plan(K, r, c * K, N).bind(T, mode).upload()
    pack, waves = plan.pipeline_launch()[:2]
    assert 64 * 1024 < waves * pack * K * r * 256 <= 160 * 1024
    dt = {"u32": torch.int32, "bf16": torch.bfloat16, "f16": torch.float16}.get(mode, torch.float32)
    sh = plan.shapes()
    g = torch.Generator(device="cuda").manual_seed(T)
    if dt.itemsize == 2:
        V = (torch.rand(sh["V"], device="cuda", generator=g) < 8.0 / N).to(dt)      # sums stay far below 2^8
    else:
        V = torch.randint(-8, 9, sh["V"], device="cuda", generator=g).to(dt)
    X, Phi, X2, Phi2, Vbar, want_X = (torch.full(sh[key], 77, dtype=dt, device="cuda")
                                      for key in ("X", "Phi", "X", "Phi", "Vbar", "X"))
    plan.combine(V, Vbar)
    plan.encode(Vbar, want_X)
    plan.pipeline_fused(V, X, Phi)
    plan.pipeline_fused_noalloc(V, X2, Phi2)
    bits = torch.int16 if dt.itemsize == 2 else torch.int32
    assert torch.equal(X.view(bits), want_X.view(bits)) and torch.equal(X2.view(bits), want_X.view(bits))
    if mode == "u32":
        total = V[:, 0].clone()
        for n in range(1, N):
            total ^= V[:, n]
        assert torch.equal(Phi, total)
    else:
        assert torch.equal(Phi.float(), V.float().sum(1))
    assert torch.equal(Phi2, Phi)
    plan.close()


@pytest.mark.parametrize("K,r,m,T,mode", [(13, 2, 1, 502358, "bf16"), (8, 2, 6, 247552, "bf16"), (8, 2, 1, 2068872, "bf16")])
def test_r2_with_a_tile_for_every_compute_unit_keeps_to_64_kilobytes(K, r, m, T, mode):
    """Larger workgroups were up to 16 % slower there."""
    plan = L.ccdc_plan(K, r, K, m * comb(K, r)).bind(T, mode).upload()
    pack, waves = plan.pipeline_launch()[:2]
    assert -(-(T // r) // (64 * pack)) >= torch.cuda.get_device_properties(0).multi_processor_count
    assert waves * pack * K * r * 256 <= 64 * 1024
    plan.close()


@pytest.mark.parametrize("K,r,m,T,mode", [(24, 3, 8, 432, "bf16"), (24, 3, 12, 448, "bf16"), (22, 4, 6, 576, "f16"), (19, 4, 4, 600, "f16")])
def test_large_inputs_avoid_a_nearly_empty_second_tile(K, r, m, T, mode):
    """As two tiles of two-element packs, the second with 8 to 12 of 64 lanes at work, these ran up to 1.8 times as long."""
    plan = L.ccdc_plan(K, r, K, m * comb(K, r)).bind(T, mode).upload()
    pack = plan.pipeline_launch()[0]
    lanes = plan.seg_len // pack
    assert lanes % 64 == 0 or lanes % 64 > 12
    plan.close()
