"""The main loop of the bf16 linear kernels as compiled: LDS reads and scalar loads share a counter, so a scalar load that is still
pending when the loop starts makes the compiler wait for every fragment of a step in front of its first MFMA."""
import re
import subprocess

import pytest

from paper_2506_05096_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "linear_bf16.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "-S", "--cuda-device-only", str(build.CSRC / "linear_bf16.hip"), "-o", str(out)],
                   check=True, capture_output=True)
    parts = out.read_text().split("; -- Begin function ")[1:]
    return {m[1]: p for p in parts if (m := re.match(r"_ZN\S*linear_bf16_kernelILi(\w+?)EEEv", p))}


@pytest.mark.parametrize("shape", [s + g for s in ("4ELi2ELi256", "2ELi3ELi256", "2ELi2ELi256", "2ELi1ELi128") for g in ("ELb0", "ELb1")])
def test_first_mfma_of_a_step_waits_for_its_own_fragments_only(kernels, shape):
    body = kernels[shape]
    loop = body[body.index("Loop Header"):]
    first = re.search(r"lgkmcnt\((\d+)\)", loop[:loop.index("v_mfma")])
    assert first and int(first[1]) > 0, first
