"""Kernels whose state has to stay in registers use no scratch memory: the one-workgroup
levels in single precision keep a thread's coefficients there through every sweep of the
coarsest level, and reading them back from memory made a sweep a third slower than one that
forms them again.  Read from the metadata of the library's own object file."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LLVM = "/opt/rocm/llvm/bin"


def _scratch(obj, tmp):
    run = lambda *a: subprocess.run(a, check=True, capture_output=True, text=True).stdout  # noqa: E731
    bundle, code = str(tmp / "bundle"), str(tmp / "code")
    run(f"{LLVM}/llvm-objcopy", f"--dump-section=.hip_fatbin={bundle}", obj, str(tmp / "rest.o"))
    run(f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o",
        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={bundle}", f"--output={code}")
    notes = run(f"{LLVM}/llvm-readelf", "--notes", code)
    return {m[0]: int(m[1]) for m in
            re.findall(r"\.name: +(\S+)\n +\.private_segment_fixed_size: +(\d+)", notes)}


def test_small_levels_in_single_precision_use_no_scratch(tmp_path):
    obj = os.path.join(ROOT, "paper_2307_01797_amd", "_build", "field.o")
    if not (os.path.exists(obj) and os.path.exists(f"{LLVM}/llvm-readelf")):
        pytest.skip("needs the built object file and the LLVM tools")
    s = {k: v for k, v in _scratch(obj, tmp_path).items() if "k_small_levelIf" in k}
    assert len(s) >= 4
    assert all(v == 0 for v in s.values()), s
