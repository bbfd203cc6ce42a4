"""GPU parity of fp32 attention (tiles of 32 queries x 32 keys, keys split over
4 wavefronts) at the edges of its tiles: sequence lengths around 32 and 128,
each head size, causal and bidirectional, with and without padded keys (up to
all but one key of a sequence), and cross-attention with unequal lengths.
Logits over every position against the oracle at 1e-4.
"""
import pytest

import synth

from test_gpu_kernel_paths import _compare
from test_gpu_seq2seq import case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("heads", [8, 4, 2])
@pytest.mark.parametrize("batch,seq,pad", [(1, 1, 0), (2, 31, 30), (2, 33, 0), (3, 129, 128),
                                           (1, 160, 40)])
def test_tiles(causal, heads, batch, seq, pad):
    _compare(synth.reduced("causal_lm_768").replace(
        n_layers=1, d_model=256, n_heads=heads, d_ff=256, batch=batch, seq=seq, vocab=300,
        max_pad=pad, causal=causal, dtype="f32"))


@pytest.mark.parametrize("src,tgt", [(65, 7), (40, 33)])
def test_cross_attention(src, tgt):
    cfg = synth.reduced("seq2seq_768").replace(
        n_layers=1, n_dec_layers=1, d_model=128, n_heads=2, d_ff=192, batch=2, seq=src, tgt_seq=tgt,
        vocab=300, max_pad=src // 2, tgt_max_pad=tgt // 2, dtype="f32")
    w = synth.make_weights(cfg, 5)
    m = case(cfg, w, *synth.make_inputs(cfg, 2), *synth.make_target_inputs(cfg, 2), "cross fp32")[0]
    m.close()
