"""The blocks of a row that the resident select samples (sample.h, compiled for
the host): for every number of waves and of vectors per thread that its kernels
have, one block out of every vn consecutive ones, one to a wave."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_24593_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.fixture(scope="module")
def vector(tmp_path_factory):
    if not shutil.which(HIPCC):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("sample")
    (d / "shim.hip").write_text('#include "sample.h"\n'
                                'extern "C" int vec(int w, int waves, int vn) { return pivot::sampled_vector(w, waves, vn); }\n')
    subprocess.run([HIPCC, "--offload-host-only", "-O2", "-std=c++17", "-fPIC", "-shared", "-I" + CSRC,
                    str(d / "shim.hip"), "-o", str(d / "shim.so")], check=True)
    return ctypes.CDLL(str(d / "shim.so")).vec


@pytest.mark.parametrize("waves", [8, 16])
@pytest.mark.parametrize("vn", range(1, 17))
def test_one_block_per_stratum(vector, waves, vn):
    v = [vector(w, waves, vn) for w in range(waves)]
    assert all(0 <= x < vn for x in v)
    blocks = sorted(x * waves + w for w, x in enumerate(v))
    assert [b // vn for b in blocks] == list(range(waves)), blocks
    # on average the middle block of a stratum, over the whole row and over either half
    off = np.array(blocks) - vn * np.arange(waves) - (vn - 1) / 2
    assert max(abs(off.mean()), abs(off[:waves // 2].mean()), abs(off[waves // 2:].mean())) <= 1, off
