"""GPU parity of the products of at most 16 rows (a decode step, a tiny
forward): every way the norm of the input rows is taken (into LDS, scaled
after the product, by its own launch), row counts from 1 to 16, column counts
that leave a partial group of 16, and the plain, gated and rotary epilogues,
for each storage type.  Logits over every position against the oracle (fp32
1e-4, 16-bit 2e-2).
"""
import pytest

import synth

from test_gpu_kernel_paths import _compare

pytestmark = pytest.mark.gpu

ROWS = [(1, 1), (1, 2), (3, 5), (1, 16), (16, 1)]


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("batch,seq", ROWS)
@pytest.mark.parametrize("d,vocab", [(64, 33), (448, 9001)])
def test_layernorm_in_lds(dtype, batch, seq, d, vocab):
    _compare(synth.reduced("causal_lm_768").replace(
        n_layers=2, d_model=d, n_heads=d // 64, d_ff=3 * d, batch=batch, seq=seq, vocab=vocab,
        max_pad=min(4, seq - 1), dtype=dtype))


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("batch,seq", ROWS)
def test_rmsnorm_of_long_rows(dtype, batch, seq):
    """d 1152: scaled after the product in fp32 and bf16, its own launch in
    fp16; rotary and SwiGLU."""
    _compare(synth.reduced("decoder_4096").replace(
        n_layers=2, d_model=1152, n_heads=9, d_ff=704, batch=batch, seq=seq, vocab=515,
        dtype=dtype))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_layernorm_of_long_rows(dtype):
    """d 1152: a LayerNorm too long for LDS takes its own launch."""
    _compare(synth.reduced("causal_lm_768").replace(
        n_layers=2, d_model=1152, n_heads=9, d_ff=704, batch=2, seq=7, vocab=515, max_pad=3,
        dtype=dtype))
