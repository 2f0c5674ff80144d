"""Generated kernels do not depend on which process compiles them; no device needed."""
import glob
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

COMPILE = """
import sys
{first}
sys.path[:0] = [{root!r}, {root!r} + "/tests"]
import unit_graphs as U
from paper_2108_13342_amd import api
assert api.precompile_spec(U.attention_block(1, 2, 96, 96, 64, dtype="bf16"), cache_dir={out!r}, attention=1) > 0
"""


def test_a_kernel_is_the_same_whether_torch_was_loaded_first(tmp_path):
    """(torch brings a hipRTC of another version than the system's; the kernel cache is filled by processes that run nothing.)"""
    code = []
    for first in ("", "import torch"):
        out = str(tmp_path / (first.split() or ["none"])[-1])
        subprocess.run([sys.executable, "-c", COMPILE.format(first=first, root=ROOT, out=out)], check=True, timeout=240)
        code.append({os.path.basename(f): open(f, "rb").read() for f in glob.glob(out + "/*.hsaco")})
    assert code[0] and code[0] == code[1]
