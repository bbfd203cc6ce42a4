"""The greedy choice of a decode step against the logits it is taken on: the
lowest index among equal values, the first NaN if any, for vocabularies
smaller than the parts a row is split into, odd ones and long ones, and
several sequences; and the sequence lengths that the same launch updates.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import TRAP_KV_CAPACITY

from test_gpu_parity import f64, gpu_model

pytestmark = pytest.mark.gpu


def _steps(cfg, w, n=3):
    m = gpu_model(cfg, w, kv_cache=True, max_seq=cfg.seq + n)
    ids, mask = synth.make_inputs(cfg, 1)
    m.forward(torch.from_numpy(ids).cuda(), torch.from_numpy(mask).cuda(), m.new_logits(*ids.shape))
    cur = torch.zeros(cfg.batch, dtype=torch.int32, device="cuda")
    out, nxt = m.new_decode_logits(cfg.batch), torch.full_like(cur, -1)
    for _ in range(n):
        m.decode(cur, out, nxt)
        torch.cuda.synchronize()
        yield f64(out), nxt.cpu().numpy()
    assert m.check_error() == (0, 0)
    m.decode(cur, out, nxt)            # the cache is full: every length was advanced n times
    torch.cuda.synchronize()
    assert m.check_error()[0] == (TRAP_KV_CAPACITY if mask[:, -1].any() else 0)
    m.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16", "f16"])
@pytest.mark.parametrize("vocab", [3, 17, 515, 9001])
def test_first_largest(dtype, vocab):
    cfg = synth.reduced("decoder_4096").replace(
        n_layers=1, d_model=128, n_heads=2, d_ff=128, batch=3, seq=5, vocab=vocab, dtype=dtype)
    for logits, nxt in _steps(cfg, synth.make_weights(cfg, 2)):
        assert np.array_equal(nxt, logits.argmax(-1))


@pytest.mark.parametrize("vocab", [5, 9001])
def test_all_equal_and_first_nan(vocab):
    cfg = synth.reduced("decoder_4096").replace(
        n_layers=1, d_model=128, n_heads=2, d_ff=128, batch=2, seq=5, vocab=vocab, dtype="f32")
    w = synth.make_weights(cfg, 2)
    w.globals["lm_head"][:] = 0
    for logits, nxt in _steps(cfg, w):
        assert np.array_equal(nxt, [0, 0])
    w.globals["lm_head"][[vocab - 2, vocab - 1]] = np.nan
    for logits, nxt in _steps(cfg, w):
        assert np.array_equal(nxt, [vocab - 2] * 2)
