"""The stage update's buffers that are one and the same in some stages (c and Xin in the first, Xin and xs64 in
the others) must not be declared free of aliases: one wave writes what another reads, and only the order of
the two, which such a declaration lets the compiler change, keeps them apart.  Read from the device IR."""
import os
import re
import subprocess

import pytest

from paper_2601_16949_amd import build as B

SRC = os.path.join(B.CSRC, "kernels.hip")


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not available")
def test_stage_update_buffers_may_alias(tmp_path):
    src = open(SRC).read()
    args = re.search(r"\bk_epilogue\((.*?)\)\s*\{", src, re.S).group(1)
    names = [re.search(r"(\w+)\s*$", a).group(1) for a in args.split(",")]
    ir = str(tmp_path / "kernels.ll")
    subprocess.run([B.HIPCC, *B.FLAGS, "-O0", "--cuda-device-only", "-S", "-emit-llvm", "-Xclang",
                    "-disable-llvm-passes", "-o", ir, SRC], check=True, capture_output=True)
    kernels = [ln for ln in open(ir) if ln.startswith("define") and "amdgpu_kernel" in ln and "k_epilogue" in ln]
    assert len(kernels) >= 2  # FP32 and split BF16
    for ln in kernels:
        params = re.sub(r"\([^()]*\)", "", ln[ln.index("(") + 1:])  # (attributes' own arguments)
        params = params[:params.index(")")].split(",")
        assert len(params) == len(names), (params, names)
        by_name = dict(zip(names, params))
        assert "noalias" in by_name["acc"]  # the attribute is where this looks for it
        for n in ("Xin", "c", "xs64"):
            assert "noalias" not in by_name[n], (n, by_name[n])
