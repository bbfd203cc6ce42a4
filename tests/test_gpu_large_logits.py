"""fp32 logits of more tiles than one launch has room for (2^32 threads, 512 to
64 x 64 logits: 137 GB): the first and last sequences and the one that the parts
of the head meet in against a forward of these three alone (1e-5: another tile
shape, the same products).
"""
import pytest
import torch

import synth

from test_gpu_parity import gpu_model

pytestmark = pytest.mark.gpu


def test_head_in_parts_of_rows():
    B, S, V = 1024, 1024, 33000
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("needs 160 GiB of free device memory")
    cfg = synth.reduced("causal_lm_768").replace(
        n_layers=1, d_model=64, n_heads=2, d_ff=64, vocab=V, batch=B, seq=S, max_pad=0, dtype="f32")
    rows = (2 ** 32 // 512 - 1) // -(-V // 64) * 64
    assert B * S * V > 2 ** 23 * 64 * 64 and rows < B * S
    pick = [0, rows // S, B - 1]
    w = synth.make_weights(cfg, 3)
    g = torch.Generator(device="cuda").manual_seed(5)
    ids = torch.randint(0, V, (B, S), generator=g, device="cuda", dtype=torch.int32)
    m = gpu_model(cfg, w)
    few = m.new_logits(3, S)
    m.forward(ids[pick].contiguous(), torch.ones_like(ids[pick]), few)
    out = m.new_logits(B, S)
    m.forward(ids, torch.ones_like(ids), out)
    torch.cuda.synchronize()
    for i, b in enumerate(pick):
        assert (out[b] - few[i]).abs().max() <= 1e-5 * few[i].abs().max()
    m.close()
    del out
    torch.cuda.empty_cache()
