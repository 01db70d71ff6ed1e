"""Edges of the fp32 tiles: row counts around the 16-row fragments, the 64 rows
up to which the token rows are staged deeper and the tile's 128; reductions
of one to several 32-deep K tiles that end inside and outside a 16-byte chunk;
weights past the kept prefix that are not finite; operand blocks past the
reach of 32-bit buffer offsets."""
import numpy as np
import pytest

from paper_2606_27866_amd import flexmoe as fm
from paper_2606_27866_amd import synth
from tests.gpu_util import F32_TOL, GpuLayer, check_route, check_y, mini_layer, oracle_ref, say
from tests.test_prefill_tiles_gpu import skewed_logits

pytestmark = pytest.mark.gpu

ROWS = [1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 80, 96, 97, 112, 113, 127, 128, 129, 257]
KEEP = [1, 2, 3, 4, 5, 31, 32, 33, 63, 64, 65, 127, 128, 129, 130, 131, 200, 135, 136]


@pytest.mark.parametrize("d,I_s", [(8, 0), (24, 40), (32, 0), (40, 136), (136, 72)])
@pytest.mark.parametrize("keep", [KEEP, KEEP[::-1]])
def test_f32_segment_and_reduction_edges(d, I_s, keep):
    say("f32 edges d", d, "I_s", I_s, "keep", keep)
    E, T, I = len(ROWS), sum(ROWS), 200
    cfg, x, _, w, s = mini_layer("f32e", T, d, E, I, 1, I_s, dtype=synth.F32, config_id=96)
    lg = skewed_logits(ROWS, d)
    keep = np.array(keep, np.int32)
    ref, rr = oracle_ref(cfg, x, lg, w, s, keep)
    assert rr["counts"].tolist() == ROWS
    # what the budget cuts off is not read into the result, finite or not
    wg, wu, wd = (a.copy() for a in w)
    for e, k in enumerate(keep):
        for a, v in ((wg[e, k:], np.nan), (wu[e, k:], np.inf), (wd[e, :, k:], (np.nan, np.inf)[e % 2])):
            a[...] = v
    for weights in (w, (wg, wu, wd)):
        g = GpuLayer(d, E, I, 1, I_s, synth.F32, cfg.norm_topk, T, *weights, *s)
        y, r = g.forward(x, lg, keep)
        check_route(r, rr)
        check_y(y, ref, F32_TOL)


@pytest.mark.parametrize("T", [65535, 65536])
def test_f32_operand_blocks_around_2_to_the_29(T):
    """T * d just below and at 2^29 elements: the matrix-core tiles, then the
    vector-ALU tiles they give way to, against torch in fp64."""
    import torch
    d, I = 8192, 16
    say("f32 blocks T", T, "d", d)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x = torch.empty((T, d), device="cuda").normal_(generator=g)
    lg = torch.empty((T, 2), device="cuda").normal_(generator=g)
    wg, wu = (torch.empty((2, I, d), device="cuda").normal_(0, 0.02, generator=g) for _ in range(2))
    wd = torch.empty((2, d, I), device="cuda").normal_(0, 0.02, generator=g)
    keep = [13, 16]
    layer = fm.Layer(d, 2, I, 1, 0, fm.FLEXMOE_F32, 1, max_tokens=T)
    layer.set_weights(wg, wu, wd)
    layer.set_budget(keep)
    y = layer.forward(x, lg)
    e = torch.argmax(lg, dim=1)
    err = scale = 0.0
    for t0 in range(0, T, 8192):
        xs, es = x[t0:t0 + 8192].double(), e[t0:t0 + 8192]
        ref = torch.zeros_like(xs)
        for i in (0, 1):
            h = torch.nn.functional.silu(xs @ wg[i, :keep[i]].double().T) * (xs @ wu[i, :keep[i]].double().T)
            ref += (es == i).double().unsqueeze(1) * (h @ wd[i, :, :keep[i]].double().T)
        err = max(err, (y[t0:t0 + 8192].double() - ref).abs().max().item())
        scale = max(scale, ref.abs().max().item())
    assert err <= F32_TOL * scale, "max|err| %.3e, max|ref| %.3e" % (err, scale)
