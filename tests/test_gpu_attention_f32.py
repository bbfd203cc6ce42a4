"""GPU parity of fp32 attention (tiles of 32 queries x 32 keys, keys split over
4 wavefronts; a wavefront per query for up to 6 keys) at the edges of its tiles:
sequence lengths around 6, 32 and 128, each head size, causal and bidirectional,
with and without padded keys (up to all but one key of a sequence), and
cross-attention with unequal lengths.  Logits over every position against the
oracle at 1e-4.

A token whose key and value rows are NaN does not reach a query that may not
see it: the logits of those queries are those of a run with a finite token in
its place (1e-5 of the largest logit: the same products, summed tile by tile in
one run and key by key in the other).
"""
import numpy as np
import pytest

import synth

from test_gpu_kernel_paths import _compare
from test_gpu_parity import f64, gpu_model, run
from test_gpu_seq2seq import case, run_s2s, s2s_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("heads", [8, 4, 2])
@pytest.mark.parametrize("batch,seq,pad", [(1, 1, 0), (3, 6, 4), (2, 7, 3), (2, 31, 30), (2, 33, 0), (3, 129, 128),
                                           (1, 160, 40)])
def test_tiles(causal, heads, batch, seq, pad):
    _compare(synth.reduced("causal_lm_768").replace(
        n_layers=1, d_model=256, n_heads=heads, d_ff=256, batch=batch, seq=seq, vocab=300,
        max_pad=pad, causal=causal, dtype="f32"))


@pytest.mark.parametrize("src,tgt", [(65, 7), (40, 33), (6, 6), (7, 5)])
def test_cross_attention(src, tgt):
    cfg = synth.reduced("seq2seq_768").replace(
        n_layers=1, n_dec_layers=1, d_model=128, n_heads=2, d_ff=192, batch=2, seq=src, tgt_seq=tgt,
        vocab=300, max_pad=src // 2, tgt_max_pad=tgt // 2, dtype="f32")
    w = synth.make_weights(cfg, 5)
    m = case(cfg, w, *synth.make_inputs(cfg, 2), *synth.make_target_inputs(cfg, 2), "cross fp32")[0]
    m.close()


def _finite_and_nan(cfg, w, forward):
    """Logits of ``forward()`` with the last token of the vocabulary embedded
    as it is, and as NaN."""
    finite = forward()
    w.globals["tok_emb"][-1] = np.nan
    return finite, forward()


def _same(got, ref):
    assert np.isfinite(ref).all() and np.isfinite(got).all()
    assert np.abs(got - ref).max() <= 1e-5 * np.abs(ref).max()


@pytest.mark.parametrize("heads", [8, 4, 2])
@pytest.mark.parametrize("seq,bad", [(3, 2), (7, 4), (40, 39), (40, 5), (150, 90), (150, 149)])
def test_nan_at_a_later_position(heads, seq, bad):
    cfg = synth.reduced("decoder_4096").replace(
        n_layers=2, d_model=256, n_heads=heads, d_ff=256, batch=2, seq=seq, vocab=300, dtype="f32")
    w = synth.make_weights(cfg, 4)
    ids, mask = synth.make_inputs(cfg, 2)
    ids = np.minimum(ids, cfg.vocab - 2)
    ids[1, bad] = cfg.vocab - 1
    ref, got = _finite_and_nan(cfg, w, lambda: f64(run(gpu_model(cfg, w), ids, mask)))
    _same(got[0], ref[0])
    _same(got[1, :bad], ref[1, :bad])
    assert np.isnan(got[1, bad]).all()


@pytest.mark.parametrize("heads", [8, 4, 2])
@pytest.mark.parametrize("seq,pads", [(5, 2), (40, 3), (40, 30), (150, 20)])
def test_nan_under_the_mask(heads, seq, pads):
    cfg = synth.reduced("encoder_1024").replace(
        n_layers=2, d_model=256, n_heads=heads, d_ff=256, batch=2, seq=seq, vocab=300, max_pad=0,
        dtype="f32", tied_head=False)
    w = synth.make_weights(cfg, 4)
    ids, mask = synth.make_inputs(cfg, 2)
    ids = np.minimum(ids, cfg.vocab - 2)
    # trailing pads, and a hidden key among visible ones
    ids[1, -pads:], mask[1, -pads:] = cfg.vocab - 1, 0
    ids[0, 1], mask[0, 1] = cfg.vocab - 1, 0
    ref, got = _finite_and_nan(cfg, w, lambda: f64(run(gpu_model(cfg, w), ids, mask)))
    _same(got[mask != 0], ref[mask != 0])


def test_nan_under_the_source_mask():
    cfg = synth.reduced("seq2seq_768").replace(
        n_layers=1, n_dec_layers=1, d_model=128, n_heads=2, d_ff=192, batch=2, seq=40, tgt_seq=9,
        vocab=300, max_pad=0, tgt_max_pad=0, dtype="f32")
    w = synth.make_weights(cfg, 5)
    si, sm = synth.make_inputs(cfg, 2)
    ti, tm = synth.make_target_inputs(cfg, 2)
    si, ti = np.minimum(si, cfg.vocab - 2), np.minimum(ti, cfg.vocab - 2)
    si[1, -4:], sm[1, -4:] = cfg.vocab - 1, 0
    ref, got = _finite_and_nan(cfg, w, lambda: f64(run_s2s(s2s_model(cfg, w), si, sm, ti, tm)))
    _same(got[..., :-1], ref[..., :-1])     # (the last column: the head is tied)
