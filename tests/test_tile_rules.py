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
    body = "\n".join(re.search(r"^%s.*?^}$" % start, src, re.S | re.M).group(0)
                     for start in ("constexpr double kMidSharedFlops", "inline bool mid_nt_all"))
    d = tmp_path_factory.mktemp("rules")
    (d / "r.cpp").write_text(body + """
extern "C" int one_launch(int T, int d, int s) { return mid_one_launch(T, d, s); }
extern "C" int nt_all(int E, int I, int d, int s) { return mid_nt_all(E, I, d, s); }
""")
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(d / "r.so"), str(d / "r.cpp")], check=True)
    return ctypes.CDLL(str(d / "r.so"))


def test_shared_expert_in_one_launch(rules):
    for T, d, I_s, small in ONE_LAUNCH:
        assert bool(rules.one_launch(T, d, I_s)) == small
    assert rules.one_launch(1 << 20, 1000, 0)       # without a shared expert there is nothing to bound
    assert rules.one_launch(1000, 2048, 5632)       # the Qwen1.5-MoE shape, whose rows are whole lines
    assert not rules.one_launch(572, 1840, 8560)    # 54 GFLOP, 28 % slower with the small tiles


def test_hint_on_rows_that_share_lines(rules):
    assert rules.nt_all(51, 328, 3656, 1320) and rules.nt_all(51, 648, 3656, 1320)  # the shared expert ends later
    assert not rules.nt_all(30, 2024, 3664, 1040) and not rules.nt_all(61, 968, 1144, 488)
    # the GPU test of the small tiles runs the hint on such rows beside a shared expert, and without one not
    assert rules.nt_all(13, 264, 72, 136) and rules.nt_all(13, 264, 200, 2056)
