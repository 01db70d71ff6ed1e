"""The rules between the tile shapes, compiled for the host from kernels.h: the
cases of the GPU tests lie on the sides of the lines that they claim."""
import ctypes
import os
import re
import subprocess

import pytest

from paper_2606_27866_amd import flexmoe as fm
from tests.test_prefill_tiles_gpu import ONE_LAUNCH


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    src = open(os.path.join(os.path.dirname(fm.__file__), "csrc", "kernels.h")).read()
    body = re.search(r"constexpr double kMidSharedFlops.*?^}$", src, re.S | re.M).group(0)
    d = tmp_path_factory.mktemp("rules")
    (d / "r.cpp").write_text(body + '\nextern "C" int one_launch(int T, int d, int s) { return mid_one_launch(T, d, s); }\n')
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(d / "r.so"), str(d / "r.cpp")], check=True)
    return ctypes.CDLL(str(d / "r.so"))


def test_shared_expert_in_one_launch(rules):
    for T, d, I_s, small in ONE_LAUNCH:
        assert bool(rules.one_launch(T, d, I_s)) == small
    assert rules.one_launch(1 << 20, 1000, 0)       # without a shared expert there is nothing to bound
    assert rules.one_launch(1000, 2048, 5632)       # the Qwen1.5-MoE shape, whose rows are whole lines
    assert not rules.one_launch(572, 1840, 8560)    # 54 GFLOP, 28 % slower with the small tiles
