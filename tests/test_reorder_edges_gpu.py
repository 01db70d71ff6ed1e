"""Edges of the ranking, the column gather and the export: channel counts
around a workgroup's 256 channels, a chunk of 2048 keys and the rows that fit
in LDS; ties, zeros of both signs, infinities and NaN; a down matrix that is
not 16-byte aligned."""
import numpy as np
import pytest

import oracle
from paper_2606_27866_amd import flexmoe as fm
from paper_2606_27866_amd import synth
from tests.gpu_util import mini_layer, say

pytestmark = pytest.mark.gpu


def special_scores(E, I, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    s = rng.standard_normal((E, I)).astype(np.float32)
    s[0] = np.round(s[0] * 2) / 2                       # ties, zeros of both signs
    s[0][rng.integers(0, I, I // 8 + 1)] = -0.0
    for v in (np.nan, -np.nan, np.inf, -np.inf, 0.0):   # scattered special values, several of each
        s[E - 1][rng.integers(0, I, I // 16 + 2)] = v
    return s


@pytest.mark.parametrize("dtype,E,I,d,offset", [
    (synth.BF16, 3, 8, 8, 0), (synth.BF16, 2, 256, 24, 0), (synth.BF16, 2, 264, 72, 0), (synth.BF16, 2, 2048, 16, 0),
    (synth.BF16, 2, 2056, 40, 0), (synth.BF16, 2, 4360, 24, 0), (synth.BF16, 1, 32776, 8, 0),
    (synth.BF16, 2, 264, 72, 1), (synth.F32, 2, 520, 24, 0), (synth.F32, 1, 16392, 8, 0), (synth.F32, 2, 264, 72, 1),
    # rows of W_down per workgroup: 5 and 3 with a remainder, one, and one that fills 64 KB of LDS
    (synth.BF16, 2, 2400, 24, 0), (synth.BF16, 2, 3800, 16, 0), (synth.BF16, 2, 14336, 24, 0),
    (synth.BF16, 1, 32768, 8, 0), (synth.F32, 2, 7168, 24, 0), (synth.F32, 1, 16384, 8, 0)])
def test_rank_reorder_edges(dtype, E, I, d, offset):
    import torch
    say("reorder dtype", dtype, "E", E, "I", I, "d", d, "offset", offset)
    cfg, _, _, w, _ = mini_layer("rr", 8, d, E, I, 1, 0, dtype=dtype, config_id=93)
    scores = special_scores(E, I, I)
    ref = oracle.rank_reorder(scores, *w)
    desc = fm.make_desc(d, E, I, 1, 0, dtype, 1, 8)
    dev = [fm.to_device(a) for a in w]
    outs = [torch.empty_like(t) for t in dev]

    def shifted(t):  # the same values `offset` elements past an aligned address
        big = torch.zeros(t.numel() + offset, dtype=t.dtype, device=t.device)
        v = big[offset:].view(t.shape)
        v.copy_(t)
        return v

    dev[2], outs[2] = shifted(dev[2]), shifted(outs[2])
    perm = torch.empty((E, I), dtype=torch.int32, device="cuda")
    fm.flexmoe_rank_reorder(desc, fm.to_device(scores), *dev, *outs, perm)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(perm.cpu().numpy(), ref[3])
    for o, r in zip(outs, ref):
        assert np.array_equal(fm.to_host(o), r)


@pytest.mark.parametrize("dtype", [synth.BF16, synth.F32])
def test_export_edges(dtype):
    """Widths around a 16-byte chunk and a padded row, down to nothing."""
    import torch
    E, I, d = 12, 520, 72
    keep = np.array([0, 1, 3, 4, 5, 7, 8, 9, 255, 513, 519, 520], np.int32)
    cfg, _, _, w, _ = mini_layer("ex", 8, d, E, I, 1, 0, dtype=dtype, config_id=94)
    layer = fm.Layer(d, E, I, 1, 0, dtype, 1, max_tokens=8)
    layer.set_weights(*[fm.to_device(a) for a in w])
    cw = layer.export_clipped(keep)
    torch.cuda.synchronize()
    n = cw.packed_channels * d
    for got, ref in zip((cw.w_gate_c, cw.w_up_c, cw.w_down_c), oracle.export_clipped(keep, *w)):
        assert np.array_equal(fm.to_host(got)[:n], ref)
