"""How many kernels a call of the fused pass enqueues, on the CPU: the built library in a child process in which
hipLaunchKernel only counts.  A step whose plan needs one round of units is the fused pass and the merge, greedy or drawn, also
where the plan's bound is far above the rows: whatever a launch ahead of the pass prepares, a step of few rows under a loose
plan pays for it (2 of 19 us)."""
import ctypes
import os
import subprocess
import sys

import pytest

from paper_2601_06562_amd import binding

STUB = r"""
struct dim3 { unsigned x, y, z; };
static int launches;
int hipLaunchKernel(const void* kernel, struct dim3 grid, struct dim3 block, void** args, unsigned long lds, void* stream) {
  (void)kernel, (void)grid, (void)block, (void)args, (void)lds, (void)stream;
  ++launches;
  return 0;
}
int counted(void) { const int n = launches; launches = 0; return n; }
"""


def child(stub, cases):
    counter = ctypes.CDLL(stub, mode=ctypes.RTLD_GLOBAL)            # ahead of the library, so that its launches come here
    L = binding.lib()
    for T, bound, d, V, tau in cases:
        plan = binding.mosaic_plan_workspace(T, bound, d, V, 0, 256, tau > 0)
        p = 1 << 20                                                 # a device address that nobody looks at
        rc = L.mosaic_masked_logits_sample(p, T, d, d, p, V, p, p, p, bound, tau, 1, p, p, p, ctypes.byref(plan), p, 1 << 60, 0)
        assert rc == 0, rc
        print(counter.counted())


# (T, bound, d, V, temperature) -> launches
WIDE = (4 << 30) // (2 * 4096) + 1                                   # a hidden tensor beyond 4 GiB: the check of the list
CASES = {(16384, bound, d, V, tau): 2 for d, V in ((512, 8192), (1024, 32000), (2048, 65536), (3584, 152064), (4096, 126464))
         for bound in (16, 200, 512, 2048, 4096) for tau in (0.0, 0.7)}
CASES.update({(131072, 60000, 4096, 126464, tau): 3 for tau in (0.0, 0.7)})        # several rounds of units: their counters
CASES.update({(WIDE, 1000, 4096, 126464, tau): 4 for tau in (0.0, 0.7)})           # and a launch of the kernel for such lists


def test_launches_of_a_step(tmp_path):
    if not os.path.exists(binding.LIB_PATH):
        pytest.skip("the library is not built")
    src, so = tmp_path / "count.c", str(tmp_path / "count.so")
    src.write_text(STUB)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", so, str(src)], check=True)
    code = f"import test_launch_counts as t; t.child({so!r}, list(t.CASES))"
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, "-c", code], cwd=os.path.join(root, "tests"), stdout=subprocess.PIPE, text=True, timeout=120,
                         env=dict(os.environ, PYTHONPATH=root))
    assert res.returncode == 0
    counts = [int(x) for x in res.stdout.split()]
    assert len(counts) == len(CASES)
    wrong = {case: (n, want) for (case, want), n in zip(CASES.items(), counts) if n != want}
    assert not wrong, wrong
