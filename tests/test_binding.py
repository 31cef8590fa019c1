"""The Python binding before and beside the library: what a process meets that has made no call yet (no GPU needed)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def in_a_fresh_process(code):
    """what `code` prints in a process that has imported the package and nothing else of it"""
    r = subprocess.run([sys.executable, "-c", "import paper_2505_18663_amd as dvdq, torch\n" + code], cwd=ROOT, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return r.stdout.strip()


def test_the_first_call_of_a_process_may_be_a_controllers_step():
    """A controller that was unpickled there: __init__ has not run, the library is not loaded."""
    out = in_a_fresh_process("""
ctl = dvdq.GbsController.__new__(dvdq.GbsController)
ctl.delta, ctl.b_low, ctl.b_high = 0.1, 4, 8
ctl.state, ctl.workspace = torch.zeros(16, dtype=torch.uint8), torch.zeros(64, dtype=torch.uint8)
f = torch.zeros(8, dtype=torch.bfloat16)
try:
    ctl.step(f, f)
except Exception as e:
    print(type(e).__name__, e)
""")
    assert out == "TypeError f_t: expected a CUDA/HIP tensor"
