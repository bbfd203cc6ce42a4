"""GPU parity of the tiled GEMMs at the edges of their tiles: row counts just
above and below a tile, column counts that leave a partial tile, rows of odd
length (logits that start at any element), and every epilogue, for each
storage type and for every tile shape that the sizes select (32 x 32 up to
256 x 256; fp32: 32 x 32 and 64 x 64).  The model runs one layer; its logits
are compared with the oracle over every position (fp32 1e-4, 16-bit 2e-2).
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
