"""Host memory that runs out inside the library is a status of the call, not an
exception that passes its C boundary (host only, in a child process)."""
import os
import subprocess
import sys

from conftest import ROOT

CHILD = """
import resource
from paper_1904_11563_amd import bpx
code = bpx.Code.identity(64, 128)
keep = [bpx.Plan(code, list(range(64)), 0, bpx.MODE_STRAGGLER, 8192, 64, 64)]
used = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
resource.setrlimit(resource.RLIMIT_AS, (used + (48 << 20),) * 2)
seen = 0
for _ in range(2000):
    try:
        keep.append(bpx.Plan(code, list(range(64)), 0, bpx.MODE_STRAGGLER, 8192, 64, 64))
    except bpx.BpxError as e:
        assert e.status == bpx.E_NOMEM, e
        seen += 1
        if seen == 3:
            break
assert seen == 3, len(keep)
del keep[1:]
bpx.Plan(code, list(range(64)), 0, bpx.MODE_STRAGGLER, 8192, 64, 64)
print("out of memory", seen, "times")
"""


def test_no_host_memory_is_a_status():
    env = dict(os.environ, PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, env=env, capture_output=True,
                       text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout[-500:], r.stderr[-1500:])
    assert "out of memory 3 times" in r.stdout
