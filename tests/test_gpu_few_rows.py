"""GPU parity of the products of at most 16 rows (a decode step, a tiny
forward): every way the norm of the input rows is taken (into LDS, scaled
after the product, by its own launch), row counts from 1 to 16, column counts
that leave a partial group of 16, and the plain, gated and rotary epilogues,
for each storage type; fp32 products of at most 8 rows that are summed across
the lanes.  Logits over every position against the oracle (fp32
1e-4, 16-bit 2e-2).  A debug forward, which also stores the norms' outputs,
gives the logits and the residual stream of the ordinary forward bit for bit.
"""
import pytest
import torch

import synth

from test_gpu_kernel_paths import _compare
from test_gpu_parity import gpu_model, run

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


@pytest.mark.parametrize("batch,seq", [(1, 1), (2, 1), (1, 3), (4, 1), (1, 5), (2, 4), (3, 3)])
@pytest.mark.parametrize("d,ff,vocab", [(768, 1344, 9001), (832, 2112, 8193), (512, 1280, 8192)])
def test_fp32_lane_sums(d, ff, vocab, batch, seq):
    """1, 2, 3-4, 5-8 and 9 rows: a head of 8192 and more columns (the last
    group partial), outputs of 2048 and more and of fewer columns, K from 512
    to 2112; bias, GELU and residual."""
    _compare(synth.reduced("causal_lm_768").replace(
        n_layers=1, d_model=d, n_heads=d // 64, d_ff=ff, batch=batch, seq=seq, vocab=vocab,
        max_pad=min(1, seq - 1), dtype="f32"))


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("name,d", [("causal_lm_768", 448), ("causal_lm_768", 1152),
                                    ("decoder_4096", 448), ("decoder_4096", 1152)])
@pytest.mark.parametrize("batch,seq", [(1, 1), (3, 5), (2, 8), (1, 17)])
def test_debug_forward_has_the_same_bits(name, d, dtype, batch, seq):
    cfg = synth.reduced(name).replace(
        n_layers=2, d_model=d, n_heads=d // 64 if d == 448 else 9, d_ff=704, batch=batch, seq=seq,
        vocab=515, max_pad=0, dtype=dtype)
    w = synth.make_weights(cfg, 3)
    ids, mask = synth.make_inputs(cfg, 1)
    m = gpu_model(cfg, w)
    plain = run(m, ids, mask)
    h = m.debug_buffer(0, batch * seq, d)
    out = torch.empty_like(plain)
    dump = m.forward_layers(torch.from_numpy(ids).cuda(), torch.from_numpy(mask).cuda(), out)
    torch.cuda.synchronize()
    as_bits = torch.int32 if dtype == "f32" else torch.int16
    assert torch.equal(out.view(as_bits), plain.view(as_bits))
    assert torch.equal(dump["h_out"][-1].view(as_bits), h.view(as_bits))
    m.close()
