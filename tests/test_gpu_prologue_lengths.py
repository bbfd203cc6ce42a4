"""Key lengths from the prologue on masks that are not trailing pads: the last
unmasked key of a sequence wherever it lies, sequences shorter and longer than
a wavefront's run of tokens, none unmasked, against the mask itself.
"""
import numpy as np
import pytest
import torch

import synth

from test_gpu_parity import check_logits, f64, gpu_model
from oracle import OracleModel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch,seq", [(1, 1), (5, 7), (3, 64), (2, 65), (7, 200), (40, 33)])
def test_scattered_masks(batch, seq):
    cfg = synth.reduced("encoder_1024").replace(
        n_layers=1, d_model=128, n_heads=2, d_ff=128, batch=batch, seq=seq, vocab=200,
        max_pad=0, dtype="f32")
    w = synth.make_weights(cfg, 3)
    ids, _ = synth.make_inputs(cfg, 1)
    rng = np.random.default_rng(seq)
    m = gpu_model(cfg, w)
    for share in (1.0, 0.5, 0.05):
        mask = (rng.random((batch, seq)) < share).astype(np.int32)
        mask[0, 0] = 1
        out = m.new_logits(batch, seq)
        m.forward(torch.from_numpy(ids).cuda(), torch.from_numpy(mask).cuda(), out)
        torch.cuda.synchronize()
        res = OracleModel(cfg, w).forward(ids, mask)
        check_logits(f64(out), res.logits_f64, cfg.dtype, f"masks {batch}x{seq} {share}")
        d = m.decisions()
        assert d["pad_any"] == bool((mask == 0).any()) and d["need"] == seq
    m.close()
