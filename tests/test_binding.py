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


def test_the_native_module_is_the_one_built_for_this_python_and_torch():
    out = in_a_fresh_process("import os; dvdq.lib(); print(os.path.basename(dvdq._marshal.__file__))")
    import torch
    assert out == f"_marshal.{sys.implementation.cache_tag}.torch-{torch.__version__}.so"


def test_without_a_native_module_calls_go_through_ctypes():
    """Another torch than the one at hand when the native module was built: no such file."""
    out = in_a_fresh_process("""
import warnings
torch.__version__ = "0.0.0"
import importlib; importlib.reload(dvdq)
with warnings.catch_warnings(record=True) as w:
    warnings.simplefilter("always")
    print(dvdq.version() >= 100, [x.category.__name__ for x in w])
assert not hasattr(dvdq._marshal, "bind")
for f in (lambda x: dvdq.rotate_quant(x, 128, 8), lambda x: dvdq.rotate_quant_blockwise(x, 128, 4, 128), lambda x: dvdq.qlinear(x, x, x, 128, 8),
          lambda x: dvdq.w4ax_gemm(x, x, x, x, 8), lambda x: dvdq.GbsController.step(type("C", (), dict(delta=0., b_low=4, b_high=8, state=x, workspace=x))(), x, x)):
    try:
        f(torch.zeros(8, 128))
    except TypeError as e:
        print(e)
""")
    assert out.splitlines() == ["True ['RuntimeWarning']"] + [f"{n}: expected a CUDA/HIP tensor" for n in ("x", "x", "x", "codes", "f_t")]
