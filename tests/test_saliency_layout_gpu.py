"""The saliency's transposed copies start every segment on a 64-row boundary
when the caller brings the transposed down weights, the wider copies fit the
reported workspace and the experts have rows enough (48 on average, with many
channels 20), else on an 8-row boundary: both give the oracle's scores, in a
workspace of exactly the reported size that is followed by guard bytes.  Which
one a call took is read from the workspace, where the transposed x is found by
its first row."""
import numpy as np
import pytest

import oracle
from paper_2606_27866_amd import flexmoe as fm
from paper_2606_27866_amd import synth
from tests.gpu_util import mini_layer, say
from tests.test_prefill_tiles_gpu import skewed_logits
from tests.test_saliency_gpu import check_scores

pytestmark = pytest.mark.gpu

ROWS = [0, 1, 63, 64, 65, 7, 128, 200]
MORE_ROWS = [0, 1, 63, 64, 65, 7, 129, 700]  # 129 on average


@pytest.mark.parametrize("d,I", [(512, 512),   # the wider copies take the room of the down weights
                                 (64, 72)])    # too small for that: 8-row boundaries either way
@pytest.mark.parametrize("own_transpose", [True, False])
@pytest.mark.parametrize("rows", [ROWS, MORE_ROWS])
def test_both_segment_alignments(d, I, own_transpose, rows):
    import torch
    say("saliency layout d", d, "I", I, "own transpose", own_transpose, "rows", rows)
    E, T = len(rows), sum(rows)
    cfg, x, _, w, s = mini_layer("sl", T, d, E, I, 1, 0, norm=0, config_id=97)
    lg = skewed_logits(rows, d)
    tgt = synth.make_target(cfg, T)
    layer = fm.Layer(d, E, I, 1, 0, synth.BF16, 0, max_tokens=T)
    layer.set_weights(*[fm.to_device(a) for a in w])
    sal = fm.Saliency(layer, T, transpose_once=own_transpose)
    n = sal.workspace.numel()
    guarded = torch.full((n + 4096,), 0xA5, dtype=torch.uint8, device="cuda")
    sal.workspace = guarded[:n]
    assert n == fm.flexmoe_saliency_workspace_bytes(sal.desc, T)
    sal.add_batch(fm.to_device(x), fm.to_device(lg), fm.to_device(tgt))
    torch.cuda.synchronize()
    check_scores(sal.scores.cpu().numpy(), oracle.channel_saliency([(x, lg, tgt)], *w, 1, 0, *s))
    assert bool((guarded[n:] == 0xA5).all())


def transposed_row(x, lg, pad):
    """Row 0 of x^T in the dispatched order: every expert's tokens, then zeros
    up to a multiple of `pad` rows (after the last expert, of 8)."""
    expert, parts = lg.argmax(1), []
    for e in range(lg.shape[1]):
        t = np.nonzero(expert == e)[0]
        step = pad if e + 1 < lg.shape[1] else 8
        parts += [x[t, 0], np.zeros(-len(t) % step, x.dtype)]
    return np.concatenate(parts)


@pytest.mark.parametrize("d,I,rows,own_transpose,pad", [
    (512, 512, MORE_ROWS, True, 64),                  # the wider copies take the room of the down weights
    (512, 512, MORE_ROWS, False, 8),                  # that room is taken
    (64, 72, MORE_ROWS, True, 8),                     # they do not fit
    (512, 512, [48, 47, 49, 48], True, 64),           # 48 rows on average
    (512, 512, [48, 47, 48, 48], True, 8),            # just below
    (176, 4096, [17, 20, 23], True, 64),              # 20 rows on average, 16 channel tiles
    (176, 4096, [17, 20, 22], True, 8),               # just below
    (176, 3840, [17, 20, 23], True, 8)])              # 15 channel tiles
def test_segment_alignment_taken(d, I, rows, own_transpose, pad):
    import torch
    say("saliency alignment d", d, "I", I, "rows", rows, "own transpose", own_transpose)
    E, T = len(rows), sum(rows)
    cfg, x, _, w, s = mini_layer("sa", T, d, E, I, 1, 0, norm=0, config_id=99)
    lg = skewed_logits(rows, d)
    tgt = synth.make_target(cfg, T)
    layer = fm.Layer(d, E, I, 1, 0, synth.BF16, 0, max_tokens=T)
    layer.set_weights(*[fm.to_device(a) for a in w])
    sal = fm.Saliency(layer, T, transpose_once=own_transpose)
    sal.workspace.fill_(0xA5)  # nothing left of an earlier call
    sal.add_batch(fm.to_device(x), fm.to_device(lg), fm.to_device(tgt))
    torch.cuda.synchronize()
    check_scores(sal.scores.cpu().numpy(), oracle.channel_saliency([(x, lg, tgt)], *w, 1, 0, *s))
    held = sal.workspace.cpu().numpy().tobytes()
    for p in (8, 64):
        found = transposed_row(x, lg, p).tobytes() in held
        assert found == (p == pad), "pad %d %s" % (p, "found" if found else "not found")
