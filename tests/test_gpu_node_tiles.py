"""The node-local calls' kernels by wavefront and by packed lanes at the edges of their tiles: segments of a few packs, of one
wavefront, one pack more or less, and where the rule between the two changes.  Plans of the J-job
schedule, which never decode by receiver.  Packets against ccdc_encode's and outputs against
ccdc_reduce's, whose row order they share (XOR: bit for bit).  Needs a GPU."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    torch.cuda.set_device(0)
    return torch


@pytest.mark.parametrize("mode", ["u32", "f32", "bf16"])
@pytest.mark.parametrize("K,r,m", [(2, 1, 1), (6, 2, 3), (4, 3, 1), (7, 4, 2), (6, 5, 1), (7, 6, 1)])
@pytest.mark.parametrize("packs", [1, 47, 48, 64, 65, 96, 97, 130])
def test_node_calls_at_tile_edges(torch, K, r, m, packs, mode):
    import paper_1805_01993_amd as L
    lanes = 8 if mode == "bf16" else 4
    T = r * packs * lanes
    plan = L.ccdc_plan_jobs(K, r, K, m * (r + 1)).bind(T, mode).upload()
    assert plan.reduce_launch()[2:] == (0, 0)
    sh = plan.shapes()
    dt = {"u32": torch.int32, "f32": torch.float32, "bf16": torch.bfloat16}[mode]
    g = torch.Generator(device="cuda").manual_seed(3)
    # whole numbers of a small range: every sum is exact in fp32, so the order of addition does not matter
    V = torch.randint(-8, 9, sh["V"], device="cuda", generator=g).to(dt)
    new = lambda key: torch.full(sh[key], 77, dtype=dt, device="cuda")
    X, D, Phi, Xn, Phin = new("X"), new("D"), new("Phi"), new("X"), new("Phi")
    plan.shuffle_fused(V, X, D)
    plan.reduce(V, D, Phi)
    plan.node_encode(-1, V, Xn)
    plan.node_decode_reduce(-1, V, Xn, Phin)
    assert torch.equal(Xn.view(torch.int16), X.view(torch.int16))       # packets are bit patterns
    assert torch.equal(Phin, Phi)
    one = new("Phi")
    k = K - 1
    plan.node_decode_reduce(k, V, X, one)
    assert torch.equal(one[:, k], Phin[:, k])
    assert bool((one[:, :k] == 77).all())
    plan.close()
