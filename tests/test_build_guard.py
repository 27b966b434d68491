"""What the compiler reports of the kernels' registers (CPU only): the build refuses
values in accumulation registers, and the looping hop does not spill."""
import json
import os

import pytest

from paper_1811_08095_amd import build_lib

KERNEL = """
#include <hip/hip_runtime.h>
__global__ void __launch_bounds__(256) k(float* p) {
  float v = p[threadIdx.x];
%s
  p[threadIdx.x] = v;
}
"""


def _compile(tmp_path, monkeypatch, body):
    (tmp_path / "k.hip").write_text(KERNEL % body)
    monkeypatch.setattr(build_lib, "CSRC", str(tmp_path))
    return build_lib._compile("k.hip", False, str(tmp_path), ())


def test_accumulation_registers_are_refused(tmp_path, monkeypatch):
    body = '  asm volatile("v_accvgpr_write_b32 a0, %0" ::"v"(v) : "a0");'
    with pytest.raises(RuntimeError, match="accumulation registers"):
        _compile(tmp_path, monkeypatch, body)


def test_vector_registers_pass(tmp_path, monkeypatch, capfd):
    _compile(tmp_path, monkeypatch, "  v += 1.0f;")
    assert "remark" not in capfd.readouterr().err


def test_looping_hop_does_not_spill():
    """Its time with work to do is that of the hop it stands for."""
    path = os.path.join(build_lib.BUILD, "hop_fp64.scratch.json")
    if not os.path.exists(path):
        pytest.skip("the library was not built here")
    with open(path) as f:
        scratch = {k: v for k, v in json.load(f).items() if "hop_loop_kernel" in k}
    assert len(scratch) == 8 and set(scratch.values()) == {0}, scratch
