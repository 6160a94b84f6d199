"""Attention with the keys of a query over two wavefronts, at the sizes where a key half is empty, ragged or longer than the other,
against the oracle; the bars of the attention that small and large batches share."""
import numpy as np
import pytest

from oracle import free_oracle as fo
from tests import parity_util as pu

pytestmark = pytest.mark.gpu

# one key; the second half empty (up to 32 keys), one key in it, one tile, one key more, halves of the last tile ragged; several
# samples; scores that grow along the keys, so that the two halves end with different reference maxima
@pytest.mark.parametrize("B,N,heads,dh,spread", [(1, 1, 1, 16, 1.5), (2, 32, 4, 72, 1.5), (1, 33, 2, 72, 1.5), (1, 64, 2, 64, 1.5),
                                                 (1, 65, 8, 128, 1.5), (2, 77, 2, 16, 1.5), (3, 96, 2, 72, 1.5), (2, 450, 6, 64, 1.5),
                                                 (1, 1024, 2, 72, 1.5), (1, 1061, 3, 72, 12.0), (2, 200, 2, 128, 12.0)])
def test_split_keys(B, N, heads, dh, spread):
    import torch
    from paper_2511_20390_amd import binding
    rng = np.random.default_rng(B * N + dh)
    D = heads * dh
    qkv = (rng.standard_normal((B * N, 3 * D)) * 1.5).astype(np.float32)
    if spread > 2:
        qkv[:, D:2 * D] *= np.tile(np.linspace(0.1, spread, N), B)[:, None].astype(np.float32)
    dev = pu.to_dev(qkv, torch.bfloat16)
    v = dev.float().cpu().numpy().astype(np.float64).reshape(B, N, 3, heads, dh)
    ref = np.empty((B, N, heads, dh))
    for b in range(B):
        for h in range(heads):
            ref[b, :, h] = fo.attention(v[b, :, 0, h], v[b, :, 1, h], v[b, :, 2, h])
    out = binding.op_attention_split(dev, B, N, heads, dh).float().cpu().numpy()
    assert pu.rel_l2(out, ref.reshape(B * N, D)) < 6e-3
    assert pu.row_rel_l2(out, ref, dh) < 2e-2                 # per (token, head)
    one = binding.op_attention(dev, B, N, heads, dh, "bf16").float().cpu().numpy()
    # probabilities and outputs are rounded to bf16 in both (2^-9 each, twice): no further from the exact result than the other
    assert pu.rel_l2(out, ref.reshape(B * N, D)) <= 1.1 * pu.rel_l2(one, ref.reshape(B * N, D))
