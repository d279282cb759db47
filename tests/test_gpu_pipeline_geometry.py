"""ccdc_pipeline_fused where its launch geometry and its packs have edges.  SHAPES: value lengths that no
pack width divides, packets shorter than a pack or a segment, several files per batch, one to many column
tiles, pointers that are only element-aligned; nearly all of them run one-element packs.  X against
ccdc_encode's bit for bit, Phi against eq. (1) from the oracle.  WIDE: shapes that the library sends to
wide packs, each with the geometry that makes it one of the kernel's forms.  (The CPU build runs every form
by force, test_sanitized_geometry.py.)  Needs a GPU."""
from math import comb

import numpy as np
import pytest

import oracle as O
from workloads import generate_numpy

pytestmark = pytest.mark.gpu

# K, r, c, files per batch, T
SHAPES = [
    (4, 2, 1, 2, 1), (4, 3, 1, 1, 2), (7, 5, 1, 1, 3), (5, 4, 2, 3, 7),            # packets shorter than their segments
    (5, 1, 1, 1, 255), (5, 1, 1, 7, 257), (6, 2, 1, 1, 513), (6, 2, 2, 10, 258),    # a tile and an element more or less
    (7, 3, 1, 1, 1543), (7, 3, 1, 2, 1030), (8, 4, 1, 1, 4097), (7, 5, 1, 3, 1287),
    (12, 4, 1, 1, 66), (16, 5, 1, 1, 131), (16, 3, 1, 1, 1021), (24, 2, 1, 1, 70),  # few columns, many rounds
    (5, 2, 1, 1, 70001), (4, 1, 1, 2, 200003),                                       # many tiles, one chunk
]


@pytest.fixture(scope="module")
def torch():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    torch.cuda.set_device(0)
    return torch


@pytest.mark.parametrize("mode", ["f32", "u32", "h32"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "-".join(map(str, s)))
@pytest.mark.parametrize("shift", [0, 1], ids=["aligned", "element-aligned"])
def test_pipeline_edges(torch, shape, mode, shift):
    import paper_1805_01993_amd as L
    K, r, c, m, T = shape
    Q, N = c * K, m * comb(K, r)
    plan = L.ccdc_plan(K, r, Q, N).bind(T, mode).upload()
    sh = plan.shapes()
    Vh = generate_numpy(1, N, Q, T, 5, "u32" if mode == "u32" else "f32")
    host = torch.from_numpy(Vh.view(np.int32) if mode == "u32" else Vh)
    poison = -1 if mode == "u32" else float("nan")

    def buf(key):                       # the buffer starts `shift` elements past an aligned address, poison around it
        n = int(np.prod(sh[key]))
        t = torch.full((n + 2 * shift + 8,), poison, dtype=host.dtype, device="cuda")
        return t, t[shift:shift + n].view(sh[key])

    (Vall, V), (Xall, X), (Pall, Phi), (_, Vbar), (_, want_X) = map(buf, ("V", "X", "Phi", "Vbar", "X"))
    V.copy_(host.view(sh["V"]))
    plan.combine(V, Vbar)
    plan.encode(Vbar, want_X)
    plan.pipeline_fused(V, X, Phi)
    torch.cuda.synchronize()
    assert torch.equal(X.view(torch.int32), want_X.view(torch.int32)), "X differs from ccdc_encode's"
    want = O.direct(O.build_plan(K, r, Q, N), T, Vh).reshape(-1)
    got = Phi.cpu().numpy().reshape(-1)
    if mode == "u32":
        assert np.array_equal(got.view(np.uint32), want)
    else:
        assert np.abs(got.astype(np.float64) - want).max() <= 1e-5 * np.abs(want).max()
    # nothing outside the outputs was written
    for whole, inner in ((Xall, X), (Pall, Phi)):
        edge = torch.cat([whole[:shift], whole[shift + inner.numel():]])
        assert bool((edge == -1).all() if mode == "u32" else torch.isnan(edge).all())
    plan.close()


@pytest.mark.parametrize("mode", ["bf16", "f16"])
@pytest.mark.parametrize("shape", [s for s in SHAPES if s[4] > 1], ids=lambda s: "-".join(map(str, s)))
def test_pipeline_edges_16bit(torch, shape, mode):
    """Buffers at odd element offsets (2-byte alignment); the outputs are small whole numbers, exact in every order."""
    import paper_1805_01993_amd as L
    K, r, c, m, T = shape
    Q, N = c * K, m * comb(K, r)
    plan = L.ccdc_plan(K, r, Q, N).bind(T, mode).upload()
    sh = plan.shapes()
    dt = torch.bfloat16 if mode == "bf16" else torch.float16
    new = lambda key: torch.full((int(np.prod(sh[key])) + 1,), float("nan"), dtype=dt, device="cuda")[1:].view(sh[key])
    V, X, Phi, Vbar, want_X = map(new, ("V", "X", "Phi", "Vbar", "X"))
    g = torch.Generator(device="cuda").manual_seed(9)
    V.copy_((torch.rand(sh["V"], device="cuda", generator=g) < 8.0 / N).to(dt))      # sums stay far below 2^8
    plan.combine(V, Vbar)
    plan.encode(Vbar, want_X)
    plan.pipeline_fused(V, X, Phi)
    torch.cuda.synchronize()
    assert torch.equal(X.view(torch.int16), want_X.view(torch.int16)), "X differs from ccdc_encode's"
    assert torch.equal(Phi.double(), V.double().sum(1))
    plan.close()


# Large shapes that ran slower than with one wavefront a workgroup and at most N/8 chunks, and the geometry each gets
# since (pack, wavefronts, chunks), with the measured times.
LAUNCHES = [
    ((22, 4, 1, 1, 344), "h32", (2, 1, 768)),        # 101 -> 77 us
    ((8, 5, 1, 1, 111788), "u32", (2, 3, 2)),        # 66 -> 57
    ((11, 4, 1, 1, 138064), "u32", (4, 1, 5)),       # 545 -> 478
    ((10, 4, 1, 1, 132616), "f32", (4, 1, 7)),       # 321 -> 282
    ((9, 5, 1, 1, 100000), "f32", (4, 1, 9)),        # 113 -> 104
    ((22, 4, 1, 1, 2139), "f16", (2, 1, 128)),       # odd length: two-byte accesses would be 317 us, these are 242
    ((11, 1, 1, 2, 892808), "f32", (4, 1, 1)),       # 278 -> 256, with one step in flight
    ((12, 1, 1, 2, 426920), "u32", (4, 1, 1)),       # 154 -> 140, the same
]
ONE_STEP = 2                                         # flag of pipeline_launch()


@pytest.mark.parametrize("shape,mode,want", LAUNCHES, ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else v)
def test_launch_of_large_inputs(torch, shape, mode, want):
    import paper_1805_01993_amd as L
    K, r, c, m, T = shape
    plan = L.ccdc_plan(K, r, c * K, m * comb(K, r)).bind(T, mode).upload()
    assert plan.pipeline_launch()[:3] == want
    assert bool(plan.pipeline_launch()[3] & ONE_STEP) == (r == 1)
    plan.close()


# shape, mode, (pack, wavefronts, chunks, flags): what makes it a form of its own
WIDE = [
    ((7, 3, 1, 1, 100003), "f32", (4, 3, 1, 0)),     # a pack straddles the packet's end, r = 3, one chunk
    ((10, 2, 1, 1, 20001), "u32", (4, 3, 3, 0)),     # the same with chunks, and more rounds than three times those in flight
    ((10, 3, 1, 1, 10001), "h32", (2, 4, 9, 0)),     # two-element packs, chunks
    ((6, 4, 1, 1, 60001), "f32", (2, 5, 1, 0)),      # r = 4
    ((6, 5, 1, 1, 150001), "u32", (2, 4, 1, 0)),     # r = 5; wavefronts without a round
    ((9, 4, 1, 1, 20002), "f32", (2, 3, 6, 0)),      # last segment short, whole packs
    ((9, 4, 1, 1, 20002), "f16", (2, 3, 6, 0)),
    ((9, 2, 1, 3, 20001), "f32", (4, 3, 6, 0)),      # three files a batch, 14 steps a wavefront, three in flight
    ((9, 2, 1, 3, 20001), "bf16", (2, 7, 3, 0)),
    ((6, 1, 1, 12, 60002), "h32", (4, 8, 1, 0)),     # r = 1, 22 steps, six in flight
    ((5, 2, 1, 8, 60001), "bf16", (4, 6, 1, 0)),
    ((8, 5, 1, 1, 111788), "f32", (2, 3, 2, 1)),     # equal shares of the rounds
    ((9, 5, 1, 1, 100000), "u32", (4, 1, 9, 1)),
]


@pytest.mark.parametrize("shape,mode,want", WIDE, ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else v)
def test_wide_packs(torch, shape, mode, want):
    """Whole numbers of a small range: sums are exact in every order (in 16 bits: sparse ones, sums far below 2^8)."""
    import paper_1805_01993_amd as L
    K, r, c, m, T = shape
    N = m * comb(K, r)
    plan = L.ccdc_plan(K, r, c * K, N).bind(T, mode).upload()
    assert plan.pipeline_launch() == want
    sh, dt = plan.shapes(), {"u32": torch.int32, "bf16": torch.bfloat16, "f16": torch.float16}.get(mode, torch.float32)
    g = torch.Generator(device="cuda").manual_seed(6)
    if dt.itemsize == 2:
        V = (torch.rand(sh["V"], device="cuda", generator=g) < 8.0 / N).to(dt)
    else:
        V = torch.randint(-8, 9, sh["V"], device="cuda", generator=g).to(dt)
    X, Phi, Vbar, want_X = (torch.full(sh[key], 77, dtype=dt, device="cuda") for key in ("X", "Phi", "Vbar", "X"))
    plan.combine(V, Vbar)
    plan.encode(Vbar, want_X)
    plan.pipeline_fused(V, X, Phi)
    bits = torch.int16 if dt.itemsize == 2 else torch.int32
    assert torch.equal(X.view(bits), want_X.view(bits)), "X differs from ccdc_encode's"
    if mode == "u32":
        total = V[:, 0].clone()
        for n in range(1, N):
            total ^= V[:, n]
        assert torch.equal(Phi, total)
    else:
        assert torch.equal(Phi.float(), V.float().sum(1))
    plan.close()


@pytest.mark.parametrize("mode", ["f32", "u32", "h32"])
@pytest.mark.parametrize("T", [310003, 310004])
def test_one_step_in_flight(torch, T, mode):
    """r = 1, ten files a batch, packets long enough for the form with one step in flight, with and without an end
    that a pack straddles.  Whole numbers of a small range: sums are exact in every order."""
    import paper_1805_01993_amd as L
    plan = L.ccdc_plan(4, 1, 4, 40).bind(T, mode).upload()
    assert plan.pipeline_launch()[0] == 4 and plan.pipeline_launch()[3] & ONE_STEP
    sh, dt = plan.shapes(), torch.int32 if mode == "u32" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(4)
    V = torch.randint(-8, 9, sh["V"], device="cuda", generator=g).to(dt)
    X, Phi, Vbar, want_X = (torch.full(sh[key], 77, dtype=dt, device="cuda") for key in ("X", "Phi", "Vbar", "X"))
    plan.combine(V, Vbar)
    plan.encode(Vbar, want_X)
    plan.pipeline_fused(V, X, Phi)
    assert torch.equal(X.view(torch.int32), want_X.view(torch.int32)), "X differs from ccdc_encode's"
    if mode == "u32":
        want = V[:, 0].clone()
        for n in range(1, V.shape[1]):
            want ^= V[:, n]
    else:
        want = V.sum(1)
    assert torch.equal(Phi, want)
    plan.close()
