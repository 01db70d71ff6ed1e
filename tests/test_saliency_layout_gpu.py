"""The saliency's transposed copies start every segment on a 64-row boundary
when the caller brings the transposed down weights and the wider copies fit
the reported workspace, else on an 8-row boundary: both give the oracle's
scores, in a workspace of exactly the reported size that is followed by
guard bytes."""
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


@pytest.mark.parametrize("d,I", [(512, 512),   # the wider copies take the room of the down weights
                                 (64, 72)])    # too small for that: 8-row boundaries either way
@pytest.mark.parametrize("own_transpose", [True, False])
def test_both_segment_alignments(d, I, own_transpose):
    import torch
    say("saliency layout d", d, "I", I, "own transpose", own_transpose)
    E, T = len(ROWS), sum(ROWS)
    cfg, x, _, w, s = mini_layer("sl", T, d, E, I, 1, 0, norm=0, config_id=97)
    lg = skewed_logits(ROWS, d)
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
