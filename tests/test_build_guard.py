"""The build refuses kernels whose values lie in accumulation registers (CPU only)."""
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
