"""A mesh whose set-up does not fit the memory at hand is an error of the call,
and the process goes on."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import resource
from paper_1610_02258_amd import inputs as I, rdx
model = I.model_abc().as_dict()
small, large = I.box_mesh(2, 2, 2, 1e-6).as_dict(), I.box_mesh(40, 40, 60, 1e-6).as_dict()
rdx.setup_geometry(small, model)
had = rdx.setup_geometry(large, model)["tau"]
size = int(open("/proc/self/statm").read().split()[0]) * resource.getpagesize()
# the call's outputs (88 bytes a tet) fit, its working arrays do not
resource.setrlimit(resource.RLIMIT_AS, (size + 120 * len(large["tets"]), resource.RLIM_INFINITY))
try:
    rdx.setup_geometry(large, model)
    print("no error")
except rdx.RdxError as e:
    print("status", e.status)
rdx.setup_geometry(small, model)
resource.setrlimit(resource.RLIMIT_AS, (resource.RLIM_INFINITY, resource.RLIM_INFINITY))
print(rdx.setup_geometry(large, model)["tau"] == had)
"""


def test_set_up_out_of_memory():
    p = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stderr
    assert p.stdout.split("\n")[:2] == ["status -4", "True"]
