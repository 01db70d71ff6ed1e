"""Routing on both dispatch paths where the ranking branches: expert counts
around 16 (ranked with ties at once), 64, 128 and 256 (keys per lane), token
counts that leave a wave one, two, three and four tokens, and logits with ties,
NaN and infinities next to tokens without any."""
import numpy as np
import pytest

from paper_2606_27866_amd import synth
from tests.gpu_util import BF16_TOL, GpuLayer, check_route, check_y, mini_layer, oracle_ref, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,k", [(8, 2), (16, 4), (17, 3), (60, 8), (64, 1), (65, 16), (200, 4), (256, 8)])
@pytest.mark.parametrize("T", [1, 17, 33, 64, 90])
def test_ties_and_special_logits(E, k, T):
    say("route E", E, "k", k, "T", T)
    cfg, x, lg, w, s = mini_layer("rt", T, 64, E, 16, k, 0, dtype=synth.BF16, norm=0, config_id=98)
    rng = np.random.Generator(np.random.PCG64(E * 1000 + T))
    for t in range(0, T, 2):                       # every second token: quantised, so full of ties
        lg[t] = np.round(lg[t] * 2) / 2
    for t in range(0, T, 3):
        lg[t, rng.integers(0, E, 2)] = np.nan
    for t in range(1, T, 4):
        lg[t, rng.integers(0, E)] = -np.inf
        lg[t, rng.integers(0, E, 2)] = -0.0
    keep = np.full(E, 16, np.int32)
    ref, rr = oracle_ref(cfg, x, lg, w, s, keep)
    g = GpuLayer(64, E, 16, k, 0, synth.BF16, 0, T, *w, *s)
    y, r = g.forward(x, lg, keep)
    np.testing.assert_array_equal(r["topk_idx"], rr["idx"])
    for name in ("counts", "offsets", "perm", "pos"):
        np.testing.assert_array_equal(r[name], rr[name])
    clean = ~np.isnan(lg).any(axis=1)              # NaN logits make the weights NaN on both sides
    np.testing.assert_allclose(r["topk_w"][clean], rr["w"][clean], rtol=0, atol=1e-6)
    if clean.any():
        check_y(y[clean], ref[clean], BF16_TOL)
