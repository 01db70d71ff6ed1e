"""Edges of the prefill tiles: segments of every row count around the 64-row
steps of the MFMA work, reductions of one, two, three and four K tiles with
and without a remainder, channel counts around the tile's 128 channels, and
both sides of the lines between the tile shapes."""
import numpy as np
import pytest

import oracle
from paper_2606_27866_amd import flexmoe as fm
from paper_2606_27866_amd import synth
from tests.gpu_util import BF16_TOL, GpuLayer, check_route, check_y, mini_layer, oracle_ref, say
from tests.test_action_gpu import BWD_TOL, check_max
from tests.test_saliency_gpu import check_scores

pytestmark = pytest.mark.gpu

ROWS = [1, 63, 64, 65, 127, 128, 129, 191, 193, 255, 256, 257, 273, 385, 513]
KEEP = [1, 7, 8, 63, 64, 65, 127, 128, 129, 192, 255, 256, 264, 200, 100]


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


# around the 32-row steps and the 128-row tiles that batches of few rows per
# expert take (mean 94 rows, 13 x 3 channel tiles)
MID_ROWS = [1, 31, 32, 33, 64, 65, 95, 97, 127, 128, 129, 160, 257]


@pytest.mark.parametrize("d,I_s,noalloc", [(64, 0, False), (72, 136, False), (136, 0, False), (200, 2056, False),
                                           (264, 2056, True), (64, 72, True)])
@pytest.mark.parametrize("keep", [KEEP[:13], KEEP[12::-1]])
def test_small_tile_edges(d, I_s, noalloc, keep):
    """noalloc: the shared expert's rows take the same tiles, with a split
    down reduction (two chunks at I_s = 2056)."""
    import torch
    say("small-tile edges d", d, "I_s", I_s, "noalloc", noalloc, "keep", keep)
    E, T = len(MID_ROWS), sum(MID_ROWS)
    cfg, x, _, w, s = mini_layer("mid", T, d, E, 264, 1, I_s, config_id=95)
    lg = skewed_logits(MID_ROWS, d)
    keep = np.array(keep, np.int32)
    ref, rr = oracle_ref(cfg, x, lg, w, s, keep)
    assert rr["counts"].tolist() == MID_ROWS
    g = GpuLayer(d, E, 264, 1, I_s, synth.BF16, cfg.norm_topk, T, *w, *s)
    y, r = g.forward(x, lg, keep)
    check_route(r, rr)
    check_y(y, ref, BF16_TOL)
    if noalloc:
        L, yd = g.layer, torch.empty((T, d), dtype=torch.bfloat16, device="cuda")
        fm.flexmoe_layer_forward_noalloc(L.desc, T, fm.to_device(x), fm.to_device(lg), L.w_gate, L.w_up, L.w_down,
                                         L.keep, L.ws_gate, L.ws_up, L.ws_down, yd)
        torch.cuda.synchronize()
        check_y(synth.bf16_bits_to_f32(fm.to_host(yd)).astype(np.float64), ref, BF16_TOL)


@pytest.mark.parametrize("d,I,I_s", [(72, 264, 0), (320, 136, 136)])
def test_backward_segment_and_reduction_edges(d, I, I_s):
    """The training and saliency backward over the same segments: their row
    counts are also the weight gradients' reduction lengths (1 to 9 K tiles)."""
    import torch
    say("backward edges d", d, "I", I, "I_s", I_s)
    E, T = len(ROWS), sum(ROWS)
    cfg, x, _, w, s = mini_layer("edges", T, d, E, I, 1, I_s, norm=0, config_id=92)
    lg = skewed_logits(ROWS, d)
    keep = np.minimum(np.array(KEEP, np.int32), I)
    tgt = synth.make_target(cfg, T)
    layer = fm.Layer(d, E, I, 1, I_s, synth.BF16, 0, max_tokens=T)
    layer.set_weights(*[fm.to_device(a) if a is not None else None for a in (*w, *s)])
    xd, ld = fm.to_device(x), fm.to_device(lg)

    learner = fm.ActionLearner(layer, T, synth.ACTION_RATIOS)
    learner.transpose_weights()
    y = learner.forward(xd, ld, keep=fm.to_device(keep))
    y_ref = oracle.layer_forward(x, lg, *w, keep, 1, 0, *s)
    check_y(synth.bf16_bits_to_f32(fm.to_host(y)).astype(np.float64), y_ref, BF16_TOL)
    dy = (y_ref - tgt).astype(np.float32)
    dx, _, dm = learner.backward(ld, fm.to_device(dy))
    torch.cuda.synchronize()
    dx_ref, _, dm_ref = oracle.masked_backward(x, lg, *w, keep, 1, 0, dy, *s)
    check_max(dx.cpu().numpy(), dx_ref, BWD_TOL, "dx")
    for e in range(E):
        check_max(dm.cpu().numpy()[e], dm_ref[e], BWD_TOL, "dmask[%d]" % e)

    sal = fm.Saliency(layer, T)
    sal.add_batch(xd, ld, fm.to_device(tgt))
    torch.cuda.synchronize()
    check_scores(sal.scores.cpu().numpy(), oracle.channel_saliency([(x, lg, tgt)], *w, 1, 0, *s))


@pytest.mark.parametrize("T", [1536, 1537, 2048, 2049])
def test_tile_rule_edges(T):
    """A layer whose large tiles fill their waves, without a shared expert: 96
    rows per expert are the last that take the small tiles (elsewhere 128)."""
    import torch
    d, E, I = 3072, 16, 2048
    say("tile rule T", T)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T)

    def rnd(*shape, std):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)

    w = [rnd(E, I, d, std=0.02), rnd(E, I, d, std=0.02), rnd(E, d, I, std=0.02)]
    x, lg = rnd(T, d, std=1.0), torch.randn((T, E), device="cuda", generator=gen)
    keep = np.array([I, 0, 1, 127, 128, 129, 1000, I - 1] * 2, np.int32)
    layer = fm.Layer(d, E, I, 1, 0, synth.BF16, 0, max_tokens=T)
    layer.set_weights(*w)
    layer.set_budget(keep)
    y = layer.forward(x, lg).float()
    check_y(y.cpu().numpy(), top1_ref(x, lg, w, keep).cpu().numpy(), BF16_TOL)


def top1_ref(x, lg, w, keep):
    """The routed part of a top-1 layer in fp32 on the device."""
    import torch
    p, silu = torch.softmax(lg, 1), torch.nn.functional.silu
    ref = torch.zeros(x.shape, device="cuda")
    for e in range(lg.shape[1]):
        n, t = int(keep[e]), torch.nonzero(lg.argmax(1) == e).squeeze(1)
        xe = x[t].float()
        h = silu(xe @ w[0][e, :n].float().T) * (xe @ w[1][e, :n].float().T)
        ref[t] = p[t, e].unsqueeze(1) * (h @ w[2][e, :, :n].float().T)
    return ref


# 6 T d I_shared flops: 993 and 994 tokens are the sides of 50e9 at hidden size
# 1000 and 8392 channels, whose weight rows end inside a cache line
ONE_LAUNCH = [(993, 1000, 8392, True), (994, 1000, 8392, False), (994, 1024, 8448, True)]


@pytest.mark.parametrize("T,d,I_s,small", ONE_LAUNCH)
def test_shared_rule_edges(T, d, I_s, small):
    """The forward whose one launch covers the shared expert too: the routed
    experts (62 rows each) take its tiles."""
    import torch
    E, I = 16, 136
    say("shared rule T", T, "d", d, "I_s", I_s)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(T + d)

    def rnd(*shape, std=0.02):
        return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)

    w = [rnd(E, I, d), rnd(E, I, d), rnd(E, d, I)]
    s = [rnd(I_s, d), rnd(I_s, d), rnd(d, I_s)]
    x, lg = rnd(T, d, std=1.0), torch.randn((T, E), device="cuda", generator=gen)
    keep = np.array([I, 0, 1, 127, 128, 129, 100, I - 1] * 2, np.int32)
    layer = fm.Layer(d, E, I, 1, I_s, synth.BF16, 0, max_tokens=T)
    layer.set_weights(*w, *s)
    layer.set_budget(keep)
    y = torch.empty_like(x)
    fm.flexmoe_layer_forward_noalloc(layer.desc, T, x, lg, *w, layer.keep, *s, y)
    xf = x.float()
    h = torch.nn.functional.silu(xf @ s[0].float().T) * (xf @ s[1].float().T)
    ref = top1_ref(x, lg, w, keep) + h @ s[2].float().T
    check_y(y.float().cpu().numpy(), ref.cpu().numpy(), BF16_TOL)
