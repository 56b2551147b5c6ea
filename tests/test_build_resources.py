"""What the compiler made of the residual projections' GEMM kernels, of both attention kernels and of the fp32 GEMM, read
from the built library's own metadata: none may spill vector registers.  The GEMM epilogue runs once per tile with the
accumulators live, so state that only the narrow tiles need has to stay out of the wide ones (a run-time choice there cost
the persistent 256x256 kernel two spills); k_attn_wide has 128 registers, so that two workgroups fit a compute unit; k_attn_mfma
needs 242 and more of its 256."""
import os
import shutil
import subprocess

import pytest
import yaml

from paper_2602_12957_amd.build import LIB_PATH, build_library

LLVM = "/opt/rocm/llvm/bin"


def _kernels(tmp_path):
    tools = [os.path.join(LLVM, t) for t in ("llvm-objdump", "llvm-readelf")]
    if not all(os.path.exists(t) for t in tools):
        pytest.skip("no LLVM tools to read the library with")
    if not os.path.exists(LIB_PATH):
        build_library()
    shutil.copy(LIB_PATH, tmp_path / "lib.so")
    subprocess.run([tools[0], "--offloading", "lib.so"], cwd=tmp_path, check=True, capture_output=True)
    code = [f for f in os.listdir(tmp_path) if f.endswith("gfx950")]
    assert len(code) == 1, code
    notes = subprocess.run([tools[1], "--notes", code[0]], cwd=tmp_path, check=True, capture_output=True, text=True).stdout
    return yaml.safe_load(notes.split("---\n", 1)[1].split("\n...", 1)[0])["amdhsa.kernels"]


def test_residual_gemm_kernels_do_not_spill(tmp_path):
    gemms = {k[".name"]: k[".vgpr_spill_count"] for k in _kernels(tmp_path) if "k_gemm_mfma" in k[".name"] and "EpiResidual" in k[".name"]}
    for form in ("k_gemm_mfma8", "k_gemm_mfma8p", "k_gemm_mfma_ws", "k_gemm_mfma_d", "k_gemm_mfma_r"):
        assert any(f"{len(form)}{form}I" in name for name in gemms), form
    assert {n: s for n, s in gemms.items() if s} == {}


def test_wide_attention_does_not_spill(tmp_path):
    forms = {k[".name"]: k[".vgpr_spill_count"] + k[".private_segment_fixed_size"] for k in _kernels(tmp_path) if "11k_attn_wideI" in k[".name"]}
    assert len(forms) == 4 and {n: s for n, s in forms.items() if s} == {}


@pytest.mark.parametrize("name, number", [("11k_attn_mfmaI", 24), ("10k_gemm_f32I", 15)])
def test_general_attention_and_fp32_gemm_do_not_spill(tmp_path, name, number):
    forms = {k[".name"]: k[".vgpr_spill_count"] + k[".private_segment_fixed_size"] for k in _kernels(tmp_path) if name in k[".name"]}
    assert len(forms) == number and {n: s for n, s in forms.items() if s} == {}
