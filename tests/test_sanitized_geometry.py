"""The one-pass kernel's launch geometries and the node-local kernels' two forms on the CPU build of the kernels, under
ASan and UBSan (see test_sanitized_host_code.py): every path's outputs against the plain sum and the paths' packets
against each other, where packs straddle the end of a packet, batches have several files, workgroups several
wavefronts and a segment a wavefront or more of packs."""
import os
import subprocess

import pytest

from test_sanitized_host_code import ENV, kernel_driver  # noqa: F401  (the fixture)

# K, r, Q, N, T, mode (0 f32, 1 u32, 2 h32, 3 bf16, 4 f16), jobs, compute units, wavefronts a unit holds
CASES = [
    (5, 1, 5, 15, 259, 0, 0, 8, 8),       # r = 1, three files a batch, three elements past the last wide pack
    (6, 2, 6, 30, 517, 2, 0, 2, 8),       # two files a batch, odd length, few compute units: several generations
    (7, 3, 7, 35, 1023, 1, 0, 256, 8),    # chunks of single rounds
    (6, 4, 12, 15, 401, 3, 0, 40, 8),     # 16-bit packs at 2-byte alignment, two functions a node
    (7, 5, 7, 42, 333, 4, 0, 8, 4),       # r = 5, two files a batch
    (5, 4, 5, 5, 3, 0, 0, 8, 8),          # a packet shorter than its segments
    (5, 2, 5, 10, 512, 1, 0, 8, 8),       # node-local: segments of exactly one wavefront of packs
    (6, 3, 6, 20, 804, 2, 0, 8, 8),       # node-local: one pack past a wavefront (lane-packed kernels)
    (4, 2, 4, 6, 400, 0, 1, 8, 8),        # the J-job schedule: node-local kernels over several jobs
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "-".join(map(str, c)))
def test_geometries_under_sanitizers(kernel_driver, case):  # noqa: F811
    res = subprocess.run([kernel_driver] + [str(v) for v in case], capture_output=True, text=True,
                         env=dict(os.environ, **ENV), timeout=600)
    assert res.returncode == 0, res.stdout + res.stderr
    assert " 0 mismatches" in res.stdout, res.stdout
