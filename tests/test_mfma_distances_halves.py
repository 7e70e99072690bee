"""The distances of test_mfma_distances.py in the attention kernel whose waves take 16 queries: its chunks are half as
long, so a result is read four of them after its last MFMA instead of two (no GPU)."""
import os
import subprocess

import pytest

import test_mfma_distances as whole
from paper_2512_07090_amd import build

SRC = "attend_bf16_halves.hip"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "k.s")
    subprocess.run([build.HIPCC, *build.FLAGS, *build.FILE_FLAGS[SRC], "-S", "--cuda-device-only",
                    os.path.join(build.CSRC, SRC), "-o", out], check=True, capture_output=True)
    found = {k: v for k, v in whole._kernels(open(out).read()).items() if "attend_bf16_kernel" in k}
    assert len(found) == 1 and all(sum(i[1].startswith("v_mfma") and i[3] for i in v) > 75 for v in found.values())
    return found


def test_results_are_left_alone_until_they_are_written(kernels):
    whole.test_results_are_left_alone_until_they_are_written(kernels)


def test_operands_are_written_before_they_are_read(kernels):
    whole.test_operands_are_written_before_they_are_read(kernels)
