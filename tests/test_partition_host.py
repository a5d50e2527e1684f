"""lesasm_sfc_partition on the host: coefficients of more parts than travel with
the launch need no memory of their own, so a call with little left returns an
error code like any other and throws nothing through the C boundary."""
import os
import subprocess
import sys

import pytest

from paper_2005_05899_amd import build

SCRIPT = """
import ctypes, resource
import numpy as np
from paper_2005_05899_amd import lesasm
lib = lesasm.load()
parts = 50_000_000
lam = np.ones(parts)
lib.lesasm_sfc_partition(1, 256, None, 300, lam.ctypes.data, 1, 256, 1 << 62, 256, None)  # (loads what the runtime needs)
size = 4096 * int(open("/proc/self/statm").read().split()[0])
resource.setrlimit(resource.RLIMIT_AS, (size + (100 << 20), resource.RLIM_INFINITY))
print("status", lib.lesasm_sfc_partition(1, 256, None, parts, lam.ctypes.data, 1, 256, 1 << 62, 256, None))
"""


def test_no_memory_for_many_coefficients():
    import torch
    if torch.cuda.device_count():
        pytest.skip("its device pointers are numbers: only where no GPU would follow them")
    r = subprocess.run([sys.executable, "-c", SCRIPT], cwd=build.ROOT, capture_output=True, text=True, timeout=120,
                       env={**os.environ, "OMP_NUM_THREADS": "1"})
    assert r.returncode == 0 and "status -4" in r.stdout, (r.returncode, r.stdout, r.stderr[-500:])


@pytest.mark.gpu
@pytest.mark.parametrize("parts", [256, 257, 4095, 4096, 4097, 8192, 10000])
def test_coefficients_in_pieces(parts):
    import numpy as np
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import partition as op
    from paper_2005_05899_amd import lesasm
    rng = np.random.default_rng(parts)
    c = rng.uniform(0.0, 1.0, (30000, 3))
    w = rng.integers(1, 100, len(c)).astype(np.int32)
    lam = rng.uniform(0.0, 2.0, parts)
    lam *= parts / lam.sum()
    got = lesasm.sfc_partition(torch.from_numpy(c).cuda(), torch.from_numpy(w).cuda(), parts, lam, 5)
    assert np.array_equal(got.cpu().numpy(), op.sfc_partition(c, w, parts, lam=lam, level=5)[0])
