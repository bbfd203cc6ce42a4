"""GPU parity of the tiled GEMMs at the edges of their tiles: row counts just
above and below a tile, column counts that leave a partial tile, rows of odd
length (logits that start at any element), and every epilogue, for each
storage type (fp32: 32 x 32 and 64 x 64 tiles).  The 128-wide models, K of 128,
reach every tile shape with the plain epilogues and up to 64 x 64 with the
rotary and gated ones; the wide models behind them reach the others, with K of
512 and more, so that the ring of stages of the large tiles turns over.  The
model runs one layer; its logits are compared with the oracle over every position
(fp32 1e-4, 16-bit 2e-2).
"""
import pytest

import synth

from test_gpu_kernel_paths import _compare

pytestmark = pytest.mark.gpu

# batch, sequence, vocabulary of a 128-wide model: 17 .. 2048 rows
SIZES = [(1, 17, 333), (1, 32, 64), (1, 33, 65), (3, 43, 777), (2, 64, 4097), (2, 100, 9001),
         (1, 257, 2050), (4, 175, 9001), (7, 256, 9001), (8, 256, 9001)]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("batch,seq,vocab", SIZES)
def test_rows_and_odd_vocabulary(dtype, batch, seq, vocab):
    """Bias, GELU and residual epilogues; plain store to rows of odd length."""
    _compare(synth.reduced("causal_lm_768").replace(
        n_layers=1, d_model=128, n_heads=2, d_ff=192, batch=batch, seq=seq, vocab=vocab,
        max_pad=min(40, seq - 1), dtype=dtype))


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("name", ["causal_lm_768", "decoder_4096"])
@pytest.mark.parametrize("batch,seq,vocab", [(1, 19, 333), (1, 257, 2050), (7, 256, 9001),
                                             (8, 256, 9001)])
def test_one_stage(name, dtype, batch, seq, vocab):
    """K of 64: the ring holds a single stage (16-bit)."""
    _compare(synth.reduced(name).replace(
        n_layers=1, d_model=64, n_heads=1, d_ff=64, batch=batch, seq=seq, vocab=vocab,
        max_pad=0, dtype=dtype))


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("heads", [2, 4, 8])
@pytest.mark.parametrize("batch,seq", [(1, 19), (3, 43), (5, 130)])
def test_rotary_and_gated(dtype, heads, batch, seq):
    """Rotary pairs of head size 128, 64 and 32 and SwiGLU pairs (a tile may
    hold several heads or a part of one)."""
    _compare(synth.reduced("decoder_4096").replace(
        n_layers=1, d_model=256, n_heads=heads, d_ff=320, batch=batch, seq=seq, vocab=515,
        dtype=dtype))


@pytest.mark.parametrize("batch,seq", [(1, 21), (2, 97), (3, 333)])
def test_gated_gelu_with_clamp_sites(batch, seq):
    """GEGLU pairs and the clamp-site statistics of the residual epilogue."""
    _compare(synth.reduced("encoder_clamp_1024").replace(
        n_layers=1, d_model=256, n_heads=4, d_ff=448, batch=batch, seq=seq, vocab=900))


# rows, vocabulary of a 512-wide model: the head on 128 x 256 (17 and 101 rows),
# 256 x 192 and 256 x 256 tiles
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("batch,seq,vocab", [(1, 17, 33333), (1, 101, 50257), (3, 45, 33333),
                                             (3, 43, 50257)])
def test_wide_head(dtype, batch, seq, vocab):
    _compare(synth.reduced("causal_lm_768").replace(
        n_layers=1, d_model=512, n_heads=8, d_ff=704, batch=batch, seq=seq, vocab=vocab,
        max_pad=9, dtype=dtype))


# rows, FFN width of a 512-wide model: gate/up on 128 x 128, 256 x 128, 128 x 256,
# 256 x 192 and 256 x 256 tiles
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("batch,seq,ff", [(1, 17, 8448), (1, 131, 8448), (2, 137, 8448),
                                          (3, 97, 11008), (1, 523, 8448)])
def test_wide_gated(dtype, batch, seq, ff):
    _compare(synth.reduced("decoder_4096").replace(
        n_layers=1, d_model=512, n_heads=4, d_ff=ff, batch=batch, seq=seq, vocab=515,
        rope_capacity=1024, dtype=dtype))


# rows and width: QKV with the rotation on 128 x 64, 128 x 128, 256 x 128, 128 x 256,
# 256 x 192 and 256 x 256 tiles; with 2703 rows also O and down on 256 x 128
@pytest.mark.parametrize("dtype,batch,seq,d", [
    ("bf16", 1, 661, 512), ("f16", 1, 661, 512), ("bf16", 3, 437, 512), ("f16", 3, 437, 512),
    ("bf16", 5, 363, 768), ("f16", 5, 363, 768), ("bf16", 3, 687, 1280), ("bf16", 3, 643, 1408),
    ("f16", 3, 643, 1408), ("bf16", 3, 687, 1920), ("bf16", 3, 901, 1536)])
def test_wide_rotary(dtype, batch, seq, d):
    _compare(synth.reduced("decoder_4096").replace(
        n_layers=1, d_model=d, n_heads=d // 128, d_ff=704, batch=batch, seq=seq, vocab=515,
        rope_capacity=1024, dtype=dtype))
