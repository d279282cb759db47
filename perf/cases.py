"""The work a user of this library has it do, as measurable cases: whole passes of the shuffle path through
`paper_1805_01993_amd`'s entry points, over the sizes, payload modes and routes that are used in earnest.

A case names a route (which calls one pass makes), the problem (K nodes, replication r, Q functions, N files per
job), the elements T of one intermediate value and the payload mode.  Routes:

  pipeline   ccdc_pipeline_fused: the whole path in one pass (the route a program takes unless it needs D)
  files      ccdc_map, then ccdc_pipeline_fused: a step that starts from files and a model
  shuffle    ccdc_shuffle_fused, then ccdc_reduce (the only fused route for the J-job schedule)
  stages     ccdc_combine, ccdc_encode, ccdc_decode, ccdc_reduce one after the other
  node       ccdc_node_encode, then ccdc_node_decode_reduce, for every node of the cluster
  uncoded    the compression-only comparison scheme: ccdc_combine, then ccdc_reduce
"""
from __future__ import annotations

import itertools
import math

import torch

import paper_1805_01993_amd as L

HALF = {"bf16": torch.bfloat16, "f16": torch.float16}
XOR_CODED = ("u32", "h32", "bf16", "f16")       # modes whose packets are bit patterns


def _case(route, K, r, c, m, T, mode, sigma=1.0):
    """m files per batch: N = m batches' worth of files for the schedule the route uses."""
    jobs = route == "shuffle"
    per = r + 1 if jobs else math.comb(K, r)
    return {"route": route, "K": K, "r": r, "Q": c * K, "N": m * per, "T": T, "mode": mode, "sigma": sigma}


def listed():
    return [
        # smallest call: a control-plane-sized exchange on four nodes (two files per batch); latency and launches
        {"name": "tiny_f32", **_case("pipeline", 4, 2, 1, 2, 256, "f32")},
        # small ordinary job on ten nodes, 20 MB of integer payload coded in the field
        {"name": "k10_u32", **_case("pipeline", 10, 3, 1, 1, 4096, "u32")},
        # ordinary job on sixteen nodes, 1820 short rounds, 147 MB
        {"name": "k16_f32", **_case("pipeline", 16, 3, 1, 1, 4096, "f32")},
        # distributed gradient descent: a 25.6M-parameter gradient cut eight ways, 2.9 GB
        {"name": "gradient_f32", **_case("pipeline", 8, 2, 1, 1, 3_200_000, "f32", 0.01)},
        # many nodes, 42504 rounds of short values, 2.1 GB, and the same job with 16-bit payload
        {"name": "k24_f32", **_case("pipeline", 24, 4, 1, 1, 2048, "f32")},
        {"name": "k24_bf16", **_case("pipeline", 24, 4, 1, 1, 2048, "bf16")},
        # a training step that starts from data files: Map, then the shuffle, 16-bit gradients
        {"name": "gradient_files_bf16", **_case("files", 8, 2, 1, 1, 3_200_000, "bf16", 0.01)},
        # more files than subsets: ten files pre-combined into each packet, two functions per node
        {"name": "batches_h32", **_case("pipeline", 8, 2, 2, 10, 25_000, "h32", 0.01)},
        # a value length that divides by nothing
        {"name": "ragged_f32", **_case("pipeline", 7, 3, 1, 1, 100_003, "f32")},
        # the paper's own schedule: 56 jobs on eight nodes, two stages, decoded packets kept
        {"name": "jobs_k8_u32", **_case("shuffle", 8, 2, 1, 3, 150_000, "u32")},
        # the four stages called one by one (a program that looks at every intermediate), several files per batch
        {"name": "stages_f16", **_case("stages", 12, 3, 1, 2, 6_000, "f16")},
        # every node for itself, from its own files and the packets it receives: what a real cluster runs
        {"name": "node_k16_h32", **_case("node", 16, 3, 1, 1, 4096, "h32")},
    ]


def draw(rng):
    """One more case of the same ranges: 4 to 24 nodes, every replication the one-pass kernel takes, 64 KB to 2.9 GB
    of intermediate values, one to twelve files per batch, any value length."""
    while True:
        route = rng.choices(["pipeline", "files", "shuffle", "stages", "node", "uncoded"], [10, 2, 3, 2, 2, 1])[0]
        mode = rng.choice(["f32", "u32"] if route == "uncoded" else ["f32", "f32", "u32", "h32", "bf16", "bf16", "f16"])
        eb = 2 if mode in HALF else 4
        r = rng.randint(1, 5)
        K = rng.randint(max(4, r + 1), 8 if route == "shuffle" else 24)
        c = rng.choice([1, 1, 1, 2])
        m = rng.choice([1, 1, 1, rng.randint(2, 12)])
        case = _case(route, K, r, c, m, 1, mode, rng.choice([1.0, 0.01]))
        if route == "uncoded":               # batches of mu*N files: N a multiple of 2K is whole for every mu
            case["N"] = 2 * K * rng.randint(1, 8)
        jobs = math.comb(K, r + 1) if route == "shuffle" else 1
        rounds = math.comb(K, r + 1) * (K - r if route == "shuffle" else 1)
        values = jobs * case["N"] * case["Q"]
        T = int(math.exp(rng.uniform(math.log(64e3), math.log(2.9e9))) / (values * eb))
        grain = rng.choice([1, 1, 4, 8, 64])
        T = T // grain * grain
        if T < 64 or rounds > 50_000 or case["N"] < K:
            continue
        case["T"] = T
        # what a pass may move: as much as the largest listed case (a node on its own re-reads the packets it cancels)
        if _moved(case) * (1 + (r - 1) / 2 if route == "node" else 1) <= 4.0e9:
            return case


# ------------------------------------------------------------------ sizes of a case
def _sizes(case):
    K, r, Q, N, T = (case[k] for k in ("K", "r", "Q", "N", "T"))
    W = Q // K * T
    if case["route"] == "uncoded":
        num, den = (r, K) if 2 * r <= K else (1, 2)
        nb = -(-den // num)
        batch = [N * num // den] * (nb - 1)
        batch.append(N - sum(batch))
        combined = sum(N - batch[k % nb] for k in range(K)) * W          # every node gets every batch but its own
        rows = K * (nb - 1) * W
        return {"V": N * Q * T, "combined": combined, "packets": rows, "X": 0, "Phi": Q * T}
    jobs = math.comb(K, r + 1) if case["route"] == "shuffle" else 1
    rounds = math.comb(K, r + 1) * (K - r if case["route"] == "shuffle" else 1)
    ell = W // r if W % (4 * r) == 0 else (-(-W // r) + 3) // 4 * 4
    m = N // (r + 1 if case["route"] == "shuffle" else math.comb(K, r))
    packets = rounds * (r + 1)
    return {"V": jobs * N * Q * T, "combined": packets * m * W, "packets": packets * W, "X": packets * ell,
            "Phi": jobs * Q * T}


def _elements(case):
    """Elements each call of a pass has to read and write, each input once and each output once."""
    s = _sizes(case)
    own = s["V"] - s["combined"]                 # values that their own reducer adds
    return {
        "pipeline": s["V"] + s["X"] + s["Phi"],
        "files": (s["V"] + s["Phi"] + s["V"]) + (s["V"] + s["X"] + s["Phi"]),
        "shuffle": (s["combined"] + s["X"] + s["packets"]) + (own + s["packets"] + s["Phi"]),
        "stages": (s["combined"] + s["packets"]) + (s["packets"] + s["X"]) + (s["X"] + 2 * s["packets"])
        + (own + s["packets"] + s["Phi"]),
        "node": (s["combined"] + s["X"]) + (s["V"] + s["X"] + s["Phi"]),
        "uncoded": (s["combined"] + s["packets"]) + (own + s["packets"] + s["Phi"]),
    }[case["route"]]


def _moved(case):
    return _elements(case) * (2 if case["mode"] in HALF else 4)


def work(case):
    s, r = _sizes(case), case["r"]
    coding = 0 if case["route"] == "uncoded" else (r - 1) * (s["X"] + s["packets"])      # encode and decode
    return {"bytes": _moved(case), "flops": s["V"] + coding + (s["V"] if case["route"] == "files" else 0)}


def tolerance(case):
    """Whole numbers and XOR-coded packets (compared as patterns) are exact in every mode.  A sum is taken in 32 bits in
    an order of the implementation's choosing: against the same sums in 64 bits the paths were at most 2.6e-7 off (2-norm)
    and 1.3e-6 at the worst value.  Stored in 16 bits, a sum next to a rounding boundary may go to the neighbour, one
    unit in the last place (2^-7 of the value in bf16, 2^-10 in f16), one in a few hundred values at most."""
    if case["mode"] == "u32":
        return "exact"
    if case["mode"] == "bf16":
        return {"rel": 5e-4, "max": 8e-3}
    if case["mode"] == "f16":
        return {"rel": 6e-5, "max": 1e-3}
    return {"rel": 1.2e-6, "max": 8e-6}


# ------------------------------------------------------------------ one pass
def _values(shape, case, g):
    if case["mode"] == "u32":
        return torch.randint(-(1 << 31), 1 << 31, shape, dtype=torch.int32, device="cuda", generator=g)
    dtype = HALF.get(case["mode"], torch.float32)
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(0.0, case["sigma"], generator=g)


def _inputs(case, seed):
    """The values (or the files) [J][N][Q][T], and the model [J][Q][T] of a step from files."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    J = math.comb(case["K"], case["r"] + 1) if case["route"] == "shuffle" else 1
    V = _values((J, case["N"], case["Q"], case["T"]), case, g)
    return V, _values((J, case["Q"], case["T"]), case, g) if case["route"] == "files" else None


def prepare(case, seed):
    """The plan, uploaded; the values (or files and model) in device memory; the buffers a program keeps for results."""
    route = case["route"]
    plan = L.Plan(case["K"], case["r"], case["Q"], case["N"], jobs=route == "shuffle", compression=route == "uncoded")
    plan.bind(case["T"], case["mode"]).upload()
    V, theta = _inputs(case, seed)
    shapes = plan.shapes()
    state = {"plan": plan, "route": route, "mode": case["mode"], "V": V}
    if route == "files":
        state["files"], state["V"], state["theta"] = V, torch.empty_like(V), theta
    kept = {"pipeline": (), "files": (), "node": (), "shuffle": ("D",), "stages": ("Vbar", "D"), "uncoded": ("Vbar",)}
    for name in ("X", "Phi") + kept[route]:
        if route == "uncoded" and name == "X":
            continue
        state[name] = torch.zeros(shapes[name], dtype=V.dtype, device="cuda")
    return state


def _packets(t, mode):
    """XOR-coded packets are bit patterns, not numbers."""
    if mode not in XOR_CODED or not t.is_floating_point():
        return t
    return t.view(torch.int16 if t.element_size() == 2 else torch.int32)


def run(state):
    plan, route, mode = state["plan"], state["route"], state["mode"]
    V, Phi = state["V"], state["Phi"]
    if route == "uncoded":
        plan.combine(V, state["Vbar"])
        plan.reduce(V, state["Vbar"], Phi)
        return {"packets": state["Vbar"], "Phi": Phi}
    X = state["X"]
    out = {"X": _packets(X, mode), "Phi": Phi}
    if route == "pipeline":
        plan.pipeline_fused(V, X, Phi)
    elif route == "files":
        plan.map(state["files"], state["theta"], V)
        plan.pipeline_fused(V, X, Phi)
        out["V"] = V
    elif route == "shuffle":
        plan.shuffle_fused(V, X, state["D"])
        plan.reduce(V, state["D"], Phi)
        out["D"] = state["D"]
    elif route == "stages":
        plan.combine(V, state["Vbar"])
        plan.encode(state["Vbar"], X)
        plan.decode(X, state["Vbar"], state["D"])
        plan.reduce(V, state["D"], Phi)
        out["Vbar"], out["D"] = state["Vbar"], state["D"]
    else:
        plan.node_encode(-1, V, X)
        plan.node_decode_reduce(-1, V, X, Phi)
    return out


# ------------------------------------------------------------------ the same pass in 64 bits
def _schedule(case):
    """Per round and member: the member's node, and the file (over all jobs) its batch starts at."""
    K, r, N = case["K"], case["r"], case["N"]
    groups = list(itertools.combinations(range(K), r + 1))
    member, first = [], []
    if case["route"] != "shuffle":           # one job: batch p lives on the p-th r-subset of the nodes
        rank = {P: p for p, P in enumerate(itertools.combinations(range(K), r))}
        m = N // len(rank)
        for S in groups:
            member.append(S)
            first.append([rank[S[:b] + S[b + 1:]] * m for b in range(r + 1)])
        return member, first
    m = N // (r + 1)
    job = {S: j for j, S in enumerate(groups)}

    def start(S, dropped):                   # the batch of the job on S that the node `dropped` misses
        return job[S] * N + (r - S.index(dropped)) * m

    for S in groups:
        member.append(S)
        first.append([start(S, s) for s in S])
        for i in range(K):                   # second stage: one round per node outside the group
            if i not in S:
                member.append(S)
                first.append([start(tuple(sorted(set(S) - {s} | {i})), i) for s in S])
    return member, first


def exact(case, seed):
    """Plain sums in 64 bits: outputs, pre-combined and decoded packets, and coded packets where they are numbers."""
    if case["mode"] == "u32":
        return None                          # whole numbers: compared bit for bit
    route, K, r, Q, N, T = (case[k] for k in ("route", "K", "r", "Q", "N", "T"))
    V, theta = _inputs(case, seed)
    V = V.double() if theta is None else theta.double().unsqueeze(1) - V.double()
    out = {"Phi": V.sum(1)}
    W, files = Q // K * T, V.reshape(-1, K, Q // K * T)
    if route == "files":
        out["V"] = V
    if route == "uncoded":
        num, den = (r, K) if 2 * r <= K else (1, 2)
        nb, per = -(-den // num), N * num // den
        batch = [files[t * per:(t + 1) * per if t < nb - 1 else N].sum(0) for t in range(nb)]
        out["packets"] = torch.stack([batch[t][k] for k in range(K) for t in range(nb) if t != k % nb])
        return out
    coded = case["mode"] == "f32"
    if not coded and route not in ("shuffle", "stages"):
        out["X"] = None                      # bit patterns
        return out
    member, first = (torch.tensor(t, device="cuda") for t in _schedule(case))
    m = N // (r + 1 if route == "shuffle" else math.comb(K, r))
    ell = W // r if W % (4 * r) == 0 else (-(-W // r) + 3) // 4 * 4
    packets, X = [], []
    step = max(1, (1 << 27) // ((r + 1) * r * ell))
    for u in range(0, len(member), step):
        who, at = member[u:u + step], first[u:u + step]
        P = sum(files[at + f, who] for f in range(m))                    # [rounds][r+1][W]
        if route in ("shuffle", "stages"):
            packets.append(P)
        if coded:
            seg = torch.nn.functional.pad(P, (0, r * ell - W)).view(-1, r + 1, r, ell)
            X.append(torch.stack([sum(seg[:, b, a - (a > b)] for b in range(r + 1) if b != a)
                                  for a in range(r + 1)], 1))
    out["X"] = torch.cat(X) if coded else None
    if packets:
        out["D"] = torch.cat(packets)
        if route == "stages":
            out["Vbar"] = out["D"]
    return out
