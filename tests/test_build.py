"""The sources' build-time constants (CPU: the preprocessor only)."""

import os
import shutil
import subprocess

import pytest

from paper_1509_02615_amd import build as B


def test_workgroup_size_of_the_weights_is_fixed():
    """The workgroup kernel of the weights is written for four wavefronts
    (columns, reduction slots, the monomial table's threads): no build macro may
    give it another number."""
    hipcc = B.HIPCC if os.path.exists(B.HIPCC) else shutil.which("hipcc")
    if not hipcc:
        pytest.skip("needs hipcc")
    out = subprocess.run([hipcc, "-E", "--cuda-host-only", "-std=c++17", "-DRBFFD_W_THREADS=128",
                          os.path.join(B.CSRC, "weights.hip")], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr
    assert "constexpr int W_THREADS = 256;" in out.stdout
