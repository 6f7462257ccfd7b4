"""A read of results on a stream under graph capture is refused and ends the
capture, also where the copy would go through pinned buffers (from 4 MB on):
the caller must not be left with a valid graph that writes into them."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

# in a process of its own: a capture that ended in error stays with its stream
# and thread
CODE = """
import ctypes
from paper_2211_05009_amd import lbm
hip = ctypes.CDLL("libamdhip64.so.7")       # the runtime loaded already
st, graph = ctypes.c_void_p(), ctypes.c_void_p()
assert hip.hipStreamCreate(ctypes.byref(st)) == 0
c = lbm.Cavity({nx}, {ny}, 1000.0)
c.set_stream(st.value)
c.step(20)
c.moments()                                 # the buffers it needs exist
assert hip.hipStreamBeginCapture(st, 1) == 0
try:
    c.moments()
    print("accepted")
except lbm.LbmError as e:
    print("refused", e)
print("end", hip.hipStreamEndCapture(st, ctypes.byref(graph)), flush=True)
"""


@pytest.mark.parametrize("nx,ny", [(200, 100), (500, 500)])   # 0.5 MB, 6 MB
def test_reads_under_capture_are_refused(nx, ny):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    out = subprocess.run([sys.executable, "-c", CODE.format(nx=nx, ny=ny)], cwd=root,
                         capture_output=True, text=True, timeout=100)
    lines = out.stdout.splitlines()
    assert out.returncode == 0 and len(lines) == 2, out.stdout + out.stderr
    assert lines[0].startswith("refused")
    assert lines[1].startswith("end ") and lines[1] != "end 0"
