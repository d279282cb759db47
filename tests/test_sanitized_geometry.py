"""The one-pass kernel's launch geometries and the node-local kernels' two forms on the CPU build of the kernels, under
ASan and UBSan (see test_sanitized_host_code.py): every path's outputs against the plain sum and the paths' packets
against each other.  CASES run every path as the library launches it, and with row lists split and decoded by node.hip's kernels, which
small inputs do not take.  The forms of the one-pass kernel (pack width,
end of a packet, several files a batch, wavefronts, chunks, how the rounds are shared out, more and fewer steps than
the kernel keeps in flight) are not left to what the library would choose: FORMS forces each into the plan."""
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor
from math import comb

import pytest

import test_gpu_any_length as any_length
import test_gpu_node_rounds as node_rounds
from test_sanitized_host_code import ENV, kernel_driver  # noqa: F401  (the fixture)

# K, r, Q, N, T, mode (0 f32, 1 u32, 2 h32, 3 bf16, 4 f16), jobs, compute units, wavefronts a unit holds
CASES = [
    (5, 1, 5, 15, 259, 0, 0, 8, 8),       # r = 1, three files a batch, odd length
    (6, 2, 6, 30, 517, 2, 0, 2, 8),       # two files a batch, odd length, two compute units
    (7, 3, 7, 35, 1023, 1, 0, 256, 8),    # odd length, many compute units
    (6, 4, 12, 15, 401, 3, 0, 40, 8),     # 16-bit, two functions a node
    (7, 5, 7, 42, 333, 4, 0, 8, 4),       # r = 5, two files a batch
    (5, 4, 5, 5, 3, 0, 0, 8, 8),          # a packet shorter than its segments
    (5, 2, 5, 10, 512, 1, 0, 8, 8),       # node-local: segments of exactly one wavefront of packs
    (6, 3, 6, 20, 804, 2, 0, 8, 8),       # node-local: one pack past a wavefront (lane-packed kernels)
    (4, 2, 4, 6, 400, 0, 1, 8, 8),        # the J-job schedule: node-local kernels over several jobs
    (9, 5, 9, 126, 333, 0, 0, 256, 8),    # more than 40 running outputs a lane
    (14, 3, 14, 364, 192, 3, 0, 256, 8),
]


SPLIT = {"SHIM_NODE": "0,0", "SHIM_REDUCE": "0"}


@pytest.mark.parametrize("forms", [{}, SPLIT], ids=["chosen", "split"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_geometries_under_sanitizers(kernel_driver, case, forms):  # noqa: F811
    res = subprocess.run([kernel_driver] + [str(v) for v in case], capture_output=True, text=True,
                         env=dict(os.environ, **ENV, **forms), timeout=600)
    assert res.returncode == 0, res.stdout + res.stderr
    assert " 0 mismatches" in res.stdout, res.stdout
    if forms:
        assert ",0,0,0\n" in res.stdout[res.stdout.index("reduce "):], res.stdout


# Value lengths, per r: whole segments of 264 elements (66 four-element packs: a full column tile and a part one), a
# last segment four elements short, one that no pack width divides, whole segments on whole cache lines.
LENGTHS = {"whole": lambda r: 264 * r, "short": lambda r: 264 * r - 4 if r > 1 else 260, "split": lambda r: 264 * r - 3,
           "lines": lambda r: 320 * r}
# pack, wavefronts, chunks, flags (1: equal shares, 2: one step in flight where the kernel has that form)
FORMS = ["4,1,1,3", "4,2,3,2", "4,1,1,1", "4,1,1,0", "4,2,1,1", "4,1,3,0", "2,1,1,1", "2,3,1,0", "2,2,2,1", "2,1,5,0", "1,1,1,1", "1,6,1,0", "1,2,3,1"]


@pytest.mark.parametrize("past", [False, True], ids=["kept", "past"])
@pytest.mark.parametrize("m", [1, 3])
@pytest.mark.parametrize("r", [1, 2, 3, 4, 5])
def test_forms_of_the_one_pass_kernel(kernel_driver, r, m, past):  # noqa: F811
    """C(7, r+1) rounds: one wavefront alone has 7 to 35 rounds, or 21 to 105 steps of one file, one of six has one or
    two rounds; up to six steps are in flight.  As small inputs are read and as large ones are."""
    K = 7
    env = dict(os.environ, **ENV, **({"SHIM_PAST": "1"} if past else {}))

    def run(k, end):
        T, mode = LENGTHS[end](r), (r + k + m) % 5
        forms = []
        for f in FORMS:
            pack, waves, chunks, _ = map(int, f.split(","))
            if K * r * 256 * pack * waves <= 65536 and chunks <= comb(K, r + 1) and not (pack == 4 and r == 5 and m > 1):
                forms.append(f)                              # (r = 5 with several files has no four-element packs)
        assert any(f[0] == "4" for f in forms) or (r == 5 and m > 1)
        assert any(f[0] == "2" for f in forms)
        args = (K, r, K, m * comb(K, r), T, mode, 0, 8, 8)
        res = subprocess.run([kernel_driver] + [str(v) for v in args] + forms, capture_output=True, text=True,
                             env=env, timeout=600)
        assert res.returncode == 0, res.stdout + res.stderr
        assert " 0 mismatches" in res.stdout, res.stdout
        streamed = {l.split()[1]: int(l.split()[2]) for l in res.stdout.splitlines() if l.startswith("streamed")}
        for f in forms:                      # past the caches: whole lines, and packs of 16 bytes wherever rows begin
            assert (streamed[f] > 0) == (past and (end == "lines" or (f[0] == "4" and mode < 3)))

    with ThreadPoolExecutor(4) as pool:
        list(pool.map(run, range(4), LENGTHS))


# What each call reads past the caches when no input counts as small (a small one is read through them by every call).
# Cases as above; the calls that make non-temporal loads.
NODES = "node-encode node-decode one-node-encode one-node-decode"
STAGES = "combine reduce shuffle map"
PAST = [
    ((4, 2, 4, 6, 512, 0, 0, 8, 8), f"{STAGES} {NODES} pipeline"),
    ((4, 1, 4, 8, 512, 3, 0, 8, 8), f"{STAGES} {NODES} pipeline"),
    ((6, 5, 6, 6, 1280, 1, 0, 8, 8), f"{STAGES} {NODES} pipeline"),
    ((6, 3, 6, 40, 1536, 4, 0, 8, 8), f"{STAGES} {NODES} pipeline"),
    ((4, 2, 4, 6, 511, 0, 0, 8, 8), "combine map one-node-encode one-node-decode"),        # one-element packs
    ((5, 4, 10, 20, 33, 2, 0, 8, 8), "combine map one-node-encode one-node-decode"),
    ((4, 2, 4, 240, 3, 0, 0, 8, 8), "combine map one-node-encode one-node-decode"),        # 40 files a batch, a wavefront a packet
    ((6, 3, 6, 20, 96, 2, 0, 8, 8), f"{STAGES} one-node-encode one-node-decode pipeline"),        # segments of 8 packs: lane-packed
    ((4, 2, 4, 6, 512, 0, 1, 8, 8), f"{STAGES} {NODES}"),        # several jobs
]


@pytest.mark.parametrize("args,calls", PAST, ids=lambda v: "-".join(map(str, v)) if isinstance(v, tuple) else "")
def test_reads_past_the_caches(kernel_driver, args, calls):  # noqa: F811
    for past in (False, True):
        res = subprocess.run([kernel_driver] + [str(v) for v in args], capture_output=True, text=True,
                             env=dict(os.environ, **ENV, **({"SHIM_PAST": "1"} if past else {})), timeout=600)
        assert res.returncode == 0, res.stdout + res.stderr
        assert " 0 mismatches" in res.stdout, res.stdout
        streamed = {l.split()[1]: int(l.split()[2]) for l in res.stdout.splitlines() if l.startswith("streamed")}
        assert {c for c, n in streamed.items() if n} == (set(calls.split()) if past else set())
    if "node-decode" in calls.split() and args[1] > 1:        # for all nodes, the coded packets stay in the caches
        assert streamed["node-decode"] < streamed["one-node-decode"]


# Workgroups of 64 to 160 KB of LDS
LARGE_GROUPS = [
    ((9, 5, 9, 126, 5 * 264 - 3, 0), ["4,2,1,0", "4,3,2,1", "2,6,1,0", "2,7,3,1"]),
    ((9, 5, 9, 252, 5 * 264 - 4, 1), ["2,3,1,0", "2,7,2,0"]),
    ((14, 3, 14, 364, 3 * 264, 4), ["4,2,3,0", "4,3,1,1", "2,7,1,0"]),
    ((14, 3, 14, 728, 3 * 264 - 3, 2), ["4,3,2,0", "2,4,1,0"]),
]


@pytest.mark.parametrize("args,forms", LARGE_GROUPS, ids=lambda v: "-".join(map(str, v)))
def test_large_workgroups_under_sanitizers(kernel_driver, args, forms):  # noqa: F811
    K, r = args[:2]
    for f in forms:
        pack, waves, _, _ = map(int, f.split(","))
        assert 65536 < K * r * 256 * pack * waves <= 160 * 1024
    res = subprocess.run([kernel_driver] + [str(v) for v in args + (0, 8, 8)] + forms, capture_output=True, text=True,
                         env=dict(os.environ, **ENV), timeout=600)
    assert res.returncode == 0, res.stdout + res.stderr
    assert " 0 mismatches" in res.stdout, res.stdout


# The form for small inputs, by receiver: pack, wavefronts, no chunks, flags
RECEIVER = ["1,1,0,0", "1,3,0,0", "2,2,0,0", "2,5,0,0", "4,2,0,0", "4,3,0,0"]


@pytest.mark.parametrize("m", [1, 3])
@pytest.mark.parametrize("r", [1, 2, 3, 4, 5])
def test_forms_by_receiver(kernel_driver, r, m):  # noqa: F811
    """As above, one tile of 64 packs and a part of one, ends of a packet that the packs divide, packets shorter than their
    segments; 6 to 20 rounds a node, one and several stages of them and of own files, wavefronts without any."""
    K = 7

    def run(k, T):
        args = (K, r, K, m * comb(K, r), T, (r + k + m) % 5, 0, 8, 8)
        forms = [f for f in RECEIVER if T % int(f[0]) == 0 and T >= int(f[0])] if T > 3 else ["1,2,0,0", "1,16,0,0"]
        res = subprocess.run([kernel_driver] + [str(v) for v in args] + forms, capture_output=True, text=True,
                             env=dict(os.environ, **ENV), timeout=600)
        assert res.returncode == 0, res.stdout + res.stderr
        assert " 0 mismatches" in res.stdout, res.stdout

    with ThreadPoolExecutor(4) as pool:
        list(pool.map(run, range(5), [264 * r, 264 * r - 4 if r > 1 else 260, 264 * r - 2, 68 * r - 3, 3]))


# Node-local decoding by receiver (pack, wavefronts) and lists summed whole (wavefronts)
@pytest.mark.parametrize("m", [1, 3])
@pytest.mark.parametrize("r", [1, 2, 3, 4, 5])
def test_forms_of_the_reductions(kernel_driver, r, m):  # noqa: F811
    """K = r+2; for all nodes and for each alone; the ends of a packet as above, one and several stages of rounds, own files and rows,
    wavefronts without any."""
    K = r + 2
    ends = [(260 if r == 1 else 264 * r - 4, "4,3", "3"), (264 * r - 2, "2,2", "16"), (68 * r - 3, "1,16", "2"), (3, "1,2", "5")]

    def run(k, case):
        T, node, waves = case
        args = (K, r, K, m * comb(K, r), T, (r + k + m) % 5, 0, 8, 8)
        res = subprocess.run([kernel_driver] + [str(v) for v in args], capture_output=True, text=True,
                             env=dict(os.environ, SHIM_NODE=node, SHIM_REDUCE=waves, **ENV), timeout=600)
        assert res.returncode == 0, res.stdout + res.stderr
        assert " 0 mismatches" in res.stdout, res.stdout
        assert f",{waves},{node}\n" in res.stdout, res.stdout

    with ThreadPoolExecutor(4) as pool:
        list(pool.map(run, range(4), ends))


def plan_only(kernel_driver, K, r, N, T, mode, jobs=0, c=1):
    """What a plan takes on 256 compute units."""
    res = subprocess.run([kernel_driver] + [str(v) for v in (K, r, c * K, N, T, mode, jobs, 256, 16)], capture_output=True, text=True,
                         env=dict(os.environ, SHIM_PLAN_ONLY="1", **ENV), timeout=600)
    assert res.returncode == 0, res.stdout + res.stderr
    return dict(l.split() for l in res.stdout.splitlines())


def choices(kernel_driver, K, r, N, T, mode):
    """Of it CCDC_Q_PIPELINE_LAUNCH and CCDC_Q_REDUCE_LAUNCH."""
    said = plan_only(kernel_driver, K, r, N, T, mode)
    return [[int(v) for v in said[k].split(",")] for k in ("launch", "reduce")]


# K, r, files a batch, T, mode; whether node-local decoding is by receiver, for one node as for all
@pytest.mark.parametrize("K,r,m,T,mode,receiver", [
    (15, 1, 1, 680, 1, True), (9, 2, 1, 8128, 4, True), (6, 4, 6, 7200, 0, True), (20, 1, 1, 64, 0, True),
    (12, 4, 1, 1624, 0, False),        # one node 9.2 us with its rounds spread over 108 chunks, by receiver 26
    (15, 3, 1, 1104, 2, False),        # 11.6 and 20.0
    (13, 4, 1, 1048, 1, False),        # 15.0 and 47.3
    (20, 3, 1, 388, 3, False),
    (18, 2, 1, 64, 1, False),          # 6.8 and 9.4; all nodes 8.0 and 11.3
])
def test_node_local_form_fits_one_node_and_all(kernel_driver, K, r, m, T, mode, receiver):  # noqa: F811
    assert (choices(kernel_driver, K, r, m * comb(K, r), T, mode)[1][3] > 0) == receiver


@pytest.mark.parametrize("K,r,m,T,mode,receiver", [
    (24, 1, 1, 376, 2, True), (7, 3, 1, 212, 0, True), (10, 2, 1, 680, 4, True), (11, 2, 1, 5536, 1, True),
    (4, 1, 1, 50119, 0, False),        # 3136 workgroups that load four packs each: 4.0 us by the one-pass kernel, 6.6
    (12, 2, 2, 1377, 2, False),        # 264 workgroups of 12 wavefronts: two generations on 256 compute units, 9.4 and 12.9
    (17, 3, 1, 134, 1, False),
])
def test_one_pass_form_of_small_inputs(kernel_driver, K, r, m, T, mode, receiver):  # noqa: F811
    assert bool(choices(kernel_driver, K, r, m * comb(K, r), T, mode)[0][3] & 4) == receiver


# The last two were one-element packs with 2 wavefronts and the split form before packs at any element: 33.9 and 28.7 us; now 27.7 and 21.3
# (in packs at any element 2 wavefronts 27.3, the split form 24.1).
@pytest.mark.parametrize("K,r,T,mode,waves", [
    (12, 3, 6000, 4, 10), (14, 3, 6736, 4, 8), (14, 3, 2735, 1, 5), (14, 3, 2735, 4, 0), (14, 3, 1735, 4, 7), (16, 3, 1735, 4, 0),
    (14, 3, 6735, 1, 8), (14, 3, 6735, 4, 8),
])
def test_reduce_of_narrow_packs(kernel_driver, K, r, T, mode, waves):  # noqa: F811
    """One-element packs of 16 bits with over 64 rows a wavefront keep the split form; packs at any element are wide ones."""
    m = 2 if K == 12 else 1
    assert choices(kernel_driver, K, r, m * comb(K, r), T, mode)[1][1] == waves


# K, r, m, T, mode, whether node-local lists are cut by rounds, however unequal the chunks: edges of the rest of the rule (replication,
# one-element packs, segments that leave lanes idle, a list that is not cut)
BY_ROUND = [
    (7, 3, 2, 768, 2, 1), (6, 4, 1, 1024, 0, 1), (6, 5, 3, 1280, 1, 1), (6, 3, 3, 1536, 3, 1), (7, 3, 1, 765, 1, 1),
    (7, 3, 5, 759, 0, 1), (6, 2, 1, 512, 2, 0), (7, 3, 2, 804, 2, 0), (6, 5, 1, 4100, 4, 1),
]


@pytest.mark.parametrize("case", BY_ROUND, ids=lambda c: "-".join(map(str, c)))
def test_lists_by_round(kernel_driver, case):  # noqa: F811
    """Every row once, whatever the chunks: the sums are whole numbers, and a node alone has the bits of all nodes."""
    K, r, m, T, mode, by_round = case
    args = (K, r, K, m * comb(K, r), T, mode, 0, 256, 8)
    res = subprocess.run([kernel_driver] + [str(v) for v in args], capture_output=True, text=True,
                         env=dict(os.environ, **ENV, SHIM_NODE="0,0", SHIM_REDUCE="0", SHIM_ROUNDS="1"), timeout=600)
    assert res.returncode == 0, res.stdout + res.stderr
    assert f"lists by round {by_round}\n" in res.stdout, res.stdout
    assert " 0 mismatches" in res.stdout, res.stdout


# The same at the sizes where it matters: chunks of up to 1.4 times the mean (several files: twice), lists that are not cut or numbered by tile
@pytest.mark.parametrize("K,r,m,T,mode,by_round", [
    (16, 3, 1, 4096, 2, True), (11, 5, 1, 6336, 1, True), (14, 5, 1, 281, 0, True),
    (15, 3, 1, 4480, 2, True),         # 1.19 (with the rounds dealt in turn 1.70: a node alone 16.0 us, in equal cuts 13.3)
    (19, 3, 1, 1408, 2, True),         # 1.25 (1.97)
    (12, 3, 1, 6464, 3, False),        # 1.48: a node alone 10.8 us, in equal cuts 9.6
    (13, 3, 1, 1280, 3, False),        # 2.27
    (6, 5, 10, 62272, 1, False),       # one round, whose packets are in one chunk: 36 and 53 us for all nodes
    (4, 3, 10, 120000, 0, False), (8, 5, 12, 19008, 0, True), (9, 5, 1, 40704, 2, False), (10, 2, 1, 3544, 1, False),
])
def test_which_lists_are_cut_by_round(kernel_driver, K, r, m, T, mode, by_round):  # noqa: F811
    assert plan_only(kernel_driver, K, r, m * comb(K, r), T, mode)["by_round"] == str(int(by_round))


# K, r, Q, N, T, mode, jobs: lengths that no pack divides, last segments a few elements long, one pack and less
ANY = [
    (5, 1, 5, 15, 259, 0, 0), (6, 2, 6, 30, 517, 2, 0), (7, 3, 7, 35, 1023, 1, 0), (6, 4, 12, 15, 401, 3, 0), (7, 5, 7, 42, 333, 4, 0),
    (5, 4, 5, 5, 3, 0, 0), (5, 2, 5, 10, 9, 3, 0), (5, 3, 5, 10, 31, 0, 0), (5, 3, 5, 30, 46, 4, 0), (4, 2, 4, 6, 401, 3, 1), (5, 2, 5, 9, 203, 0, 1),
    (8, 6, 8, 28, 131, 0, 0), (6, 2, 6, 15, 262, 3, 0),
]


@pytest.mark.parametrize("past", [False, True], ids=["kept-groups", "past-split"])
@pytest.mark.parametrize("case", ANY, ids=lambda c: "-".join(map(str, c)))
def test_packs_at_any_element(kernel_driver, case, past):  # noqa: F811
    """Every call in 16-byte packs where the value length does not divide by them, as small inputs are read, with whole lists summed in
    one launch, and as large ones are, with split lists."""
    env = dict(os.environ, **ENV, SHIM_ANY="1", SHIM_NODE="0,0", **({"SHIM_PAST": "1", "SHIM_REDUCE": "0"} if past else {}))
    res = subprocess.run([kernel_driver] + [str(v) for v in case + (8, 8)], capture_output=True, text=True, env=env, timeout=600)
    assert res.returncode == 0, res.stdout + res.stderr
    assert " 0 mismatches" in res.stdout, res.stdout


# K, r, N, T, mode, jobs (2: uncoded): lengths that no pack divides
@pytest.mark.parametrize("K,r,N,T,mode,jobs,wide", [
    (14, 3, 364, 6735, 4, 0, True),            # 69 MB, one-element packs would be cut too
    (14, 3, 364, 6735, 1, 0, True),
    (14, 3, 364, 2735, 4, 0, False),           # 28 MB
    (24, 1, 24 * 9, 3871, 3, 0, False),        # r = 1: 40 MB of values, 6 MB of lists
    (4, 2, 6, 6700001, 1, 0, True),            # over 262144 packs
    (24, 2, 288, 14345, 1, 2, False),          # 397 MB of values, 48 MB of lists
    (13, 3, 26, 30001, 0, 2, False), (13, 3, 26, 90001, 0, 2, True),
])
def test_which_lists_are_wide(kernel_driver, K, r, N, T, mode, jobs, wide):  # noqa: F811
    assert plan_only(kernel_driver, K, r, N, T, mode, jobs)["wide_lists"] == str(int(wide))


MODES = ["f32", "u32", "h32", "bf16", "f16"]


@pytest.mark.parametrize("K,r,c,m,T,mode,calls", any_length.CODED)
def test_which_calls_take_packs_at_any_element(kernel_driver, K, r, c, m, T, mode, calls):  # noqa: F811
    """The GPU test's plans lie on the sides of the lines that it says they do."""
    assert plan_only(kernel_driver, K, r, m * comb(K, r), T, MODES.index(mode), c=c)["any_element"] == calls


@pytest.mark.parametrize("K,r,m,T,mode,by_round", node_rounds.LISTS)
def test_which_lists_of_the_gpu_test_are_cut_by_round(kernel_driver, K, r, m, T, mode, by_round):  # noqa: F811
    assert plan_only(kernel_driver, K, r, m * comb(K, r), T, MODES.index(mode))["by_round"] == str(int(by_round))


@pytest.mark.parametrize("K,r,N,T,calls", any_length.UNCODED)
def test_which_uncoded_calls_take_packs_at_any_element(kernel_driver, K, r, N, T, calls):  # noqa: F811
    taken = plan_only(kernel_driver, K, r, N, T, 0, jobs=2)["any_element"]
    assert taken[:2] + taken[4] == calls


@pytest.mark.parametrize("K,r,T,packs", [(8, 6, 1024, 256), (6, 2, 300, 75), (5, 3, 1040, 260)])
def test_row_packs_of_lane_packed_decoding(kernel_driver, K, r, T, packs):  # noqa: F811
    """A row has the packs of its elements, not of r whole segments: a workgroup for every 256 of them, output and chunk."""
    args = (K, r, K, comb(K, r), T, 1, 0, 8, 8)
    res = subprocess.run([kernel_driver] + [str(v) for v in args], capture_output=True, text=True,
                         env=dict(os.environ, **ENV, SHIM_ANY="1", **SPLIT), timeout=600)
    assert res.returncode == 0, res.stdout + res.stderr
    assert " 0 mismatches" in res.stdout, res.stdout
    split = int(res.stdout[res.stdout.index("reduce ") + 7:].split(",")[0])
    assert split > 1 and f"workgroups node-decode {K * split * -(-packs // 256)}\n" in res.stdout, res.stdout


# K, r, Q, N, T, jobs: segments that do not fill a wavefront's lanes and segments that do, packets shorter than their segments, one file a
# batch and several, several jobs, r beyond what decoding is unrolled for
ALONE = [
    (3, 1, 3, 3, 72, 0), (6, 2, 6, 15, 64, 0), (5, 3, 5, 10, 72, 0), (5, 4, 5, 5, 400, 0), (6, 5, 6, 6, 90, 0), (5, 4, 5, 5, 3, 0),
    (5, 2, 5, 10, 512, 0), (6, 3, 6, 20, 786, 0), (5, 3, 5, 20, 72, 0), (5, 2, 5, 6, 203, 1), (8, 6, 8, 28, 60, 0),
]


@pytest.mark.parametrize("any_element", [False, True], ids=["", "any"])
@pytest.mark.parametrize("case", ALONE, ids=lambda c: "-".join(map(str, c)))
def test_a_node_alone_keeps_to_its_files(kernel_driver, case, any_element):  # noqa: F811
    """Calls for one node touch only the files it stores, the packets it sends or is sent and its own outputs: the driver puts the rest out of
    reach for every call of one node, and the sanitizer reports an access to it.  The kernels of node.hip (SHIM_NODE), lists split."""
    for mode in (1, 3):
        K, r, Q, N, T, jobs = case
        res = subprocess.run([kernel_driver] + [str(v) for v in (K, r, Q, N, T, mode, jobs, 8, 8)], capture_output=True, text=True,
                             env=dict(os.environ, **ENV, **SPLIT, **({"SHIM_ANY": "1"} if any_element else {})), timeout=600)
        assert res.returncode == 0, res.stdout + res.stderr
        assert " 0 mismatches" in res.stdout, res.stdout
