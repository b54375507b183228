"""CPU-only: the threads per division that a plan picks, read from the line that
BIGINT_DEBUG prints (256 CUs are assumed where there is no GPU)."""
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# divisions, dividend limbs (one size, or bounds of log-uniform ones), divisor
# limbs over dividend limbs, threads
PLANS = [
    (1, (2048, 2048), 0.5, 256),
    (4096, (2048, 2048), 0.5, 64),      # all at once on one wave each
    (512, (2048, 8192), 0.5, 512),
    (1500, (8192, 8192), 0.75, 256),    # more with fewer threads, but each 2.2 times as long
    (2048, (8192, 8192), 0.5, 256),
    (700, (16384, 16384), 0.5, 512),
    (2500, (4096, 4096), 0.5, 64),
    (600, (64, 16384), 0.5, 512),       # done when the largest is
    (1000, (64, 16384), 0.5, 512),
    (600, (1000, 3000), 0.5, 256),      # no two fit beside the largest
    (10000, (16, 1000), 0.5, 64),
]


def test_threads_of_plans():
    if not os.path.exists(os.path.join(ROOT, "paper_2607_28897_amd", "_lib", "libbigint_rocm.so")):
        pytest.skip("library not built")
    code = ("import sys; sys.path.insert(0, %r); import numpy as np; import paper_2607_28897_amd as m\n"
            "m.lib()\n"
            "for n, (lo, hi), f, _ in %r:\n"
            "    u = np.round(lo * (hi / lo) ** (np.arange(n) / max(n - 1, 1))).astype(np.int64)\n"
            "    try:\n        m.DivPlan(u, np.maximum((u * f).astype(np.int64), 1))\n"
            "    except m.BigIntError:\n        pass\n" % (ROOT, PLANS))
    r = subprocess.run([sys.executable, "-c", code], env=dict(os.environ, BIGINT_DEBUG="1"), capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    got = [int(x) for x in re.findall(r"^bigint: plan of \d+ divisions: .* (\d+) threads per division", r.stderr, re.M)]
    assert got == [p[3] for p in PLANS], list(zip(got, PLANS))
