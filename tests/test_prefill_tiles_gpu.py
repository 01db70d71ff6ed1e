"""Edges of the prefill tiles: segments of every row count around the 64-row
steps of the MFMA work, reductions of one, two, three and four K tiles with
and without a remainder, and channel counts around the tile's 128 channels."""
import numpy as np
import pytest

from paper_2606_27866_amd import synth
from tests.gpu_util import BF16_TOL, GpuLayer, check_route, check_y, mini_layer, oracle_ref, say

pytestmark = pytest.mark.gpu

ROWS = [1, 63, 64, 65, 127, 128, 129, 191, 193, 255, 256, 257, 513]
KEEP = [1, 7, 8, 63, 64, 65, 127, 128, 129, 192, 255, 256, 264]


def skewed_logits(rows, seed):
    """Logits that send rows[e] tokens to expert e (top-1), in shuffled order."""
    rng = np.random.Generator(np.random.PCG64(seed))
    lg = rng.standard_normal((sum(rows), len(rows))).astype(np.float32)
    expert = rng.permutation(np.repeat(np.arange(len(rows)), rows))
    lg[np.arange(len(expert)), expert] += 20.0
    return lg


@pytest.mark.parametrize("d,I_s", [(64, 0), (72, 136), (136, 0), (256, 72)])
@pytest.mark.parametrize("keep", [KEEP, KEEP[::-1]])
def test_segment_and_reduction_edges(d, I_s, keep):
    say("prefill edges d", d, "I_s", I_s, "keep", keep)
    E = len(ROWS)
    cfg, x, _, w, s = mini_layer("edges", sum(ROWS), d, E, 264, 1, I_s, config_id=91)
    lg = skewed_logits(ROWS, d)
    keep = np.array(keep, np.int32)
    g = GpuLayer(d, E, 264, 1, I_s, synth.BF16, cfg.norm_topk, cfg.T, *w, *s)
    y, r = g.forward(x, lg, keep)
    ref, rr = oracle_ref(cfg, x, lg, w, s, keep)
    assert rr["counts"].tolist() == ROWS
    check_route(r, rr)
    check_y(y, ref, BF16_TOL)
