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


# fp32: the key tiles (32 keys) of 32 queries over four wavefronts (head dim 128: all keys in each); one key, whole and ragged tiles,
# wavefronts without a tile (up to 96 keys), more than one round of tiles, last queries missing; scores that grow along the keys
@pytest.mark.parametrize("B,N,heads,dh,spread", [(1, 1, 1, 16, 1.5), (2, 31, 4, 72, 1.5), (1, 33, 2, 72, 1.5), (1, 96, 2, 64, 1.5),
                                                 (1, 97, 8, 128, 1.5), (2, 129, 2, 16, 1.5), (3, 161, 3, 72, 1.5), (2, 450, 6, 64, 1.5),
                                                 (1, 1061, 3, 72, 12.0), (2, 300, 2, 128, 12.0), (8, 64, 2, 72, 1.5)])
def test_fp32_keys_over_wavefronts(B, N, heads, dh, spread):
    from paper_2511_20390_amd import binding
    rng = np.random.default_rng(B * N + dh)
    D = heads * dh
    qkv = (rng.standard_normal((B * N, 3 * D)) * 1.5).astype(np.float32)
    if spread > 2:
        qkv[:, D:2 * D] *= np.tile(np.linspace(0.1, spread, N), B)[:, None].astype(np.float32)
    v = qkv.astype(np.float64).reshape(B, N, 3, heads, dh)
    ref = np.empty((B, N, heads, dh))
    for b in range(B):
        for h in range(heads):
            ref[b, :, h] = fo.attention(v[b, :, 0, h], v[b, :, 1, h], v[b, :, 2, h])
    out = binding.op_attention(pu.to_dev(qkv), B, N, heads, dh, "fp32").cpu().numpy()
    # a score of size s, a sum of dh products in fp32, is off by up to 2^-24 s sqrt(dh) where it is one of the largest, and a probability
    # by that much of itself; the sums over the keys by a few roundings
    s = np.abs(np.einsum("bqhd,bkhd->bhqk", v[:, :, 0], v[:, :, 1])).max() / np.sqrt(dh)
    assert pu.row_rel_l2(out, ref, dh) < 2.0 ** -24 * (8 + np.sqrt(dh) * s)


@pytest.mark.parametrize("dead", [range(0, 32), range(32, 64), range(0, 160)])
def test_fp32_keys_of_no_weight(dead):
    """Keys whose score is -inf weigh nothing, also where they are all that a wavefront has."""
    from paper_2511_20390_amd import binding
    N, heads, dh = 160 + 7, 2, 72
    D = heads * dh
    rng = np.random.default_rng(5)
    qkv = rng.standard_normal((N, 3 * D)).astype(np.float32)
    qkv[:, :D] = np.abs(qkv[:, :D])
    rows = list(dead)
    qkv[rows, D:2 * D] = -np.inf
    out = binding.op_attention(pu.to_dev(qkv), 1, N, heads, dh, "fp32").cpu().numpy()
    live = [i for i in range(N) if i not in dead]
    v = qkv.astype(np.float64).reshape(N, 3, heads, dh)
    ref = np.stack([fo.attention(v[:, 0, h], v[live, 1, h], v[live, 2, h]) for h in range(heads)], 1)
    assert pu.rel_l2(out, ref.reshape(N, D)) < 2e-6


# one row and one pass of rows behind the last whole tile, with the tile's other passes past the end; a sample that is followed by another one
@pytest.mark.parametrize("mode", ["fp32", "bf16"])
@pytest.mark.parametrize("B,N,heads,dh", [(1, 33, 2, 72), (1, 40, 3, 64), (2, 65, 2, 16), (1, 129, 1, 128), (3, 450, 2, 72)])
def test_rows_behind_a_sample_are_not_used(B, N, heads, dh, mode):
    """NaN in the rows behind the last sample, and in the next sample, reaches no output."""
    import torch
    from paper_2511_20390_amd import binding
    D = heads * dh
    g = torch.Generator(device="cuda").manual_seed(N)
    room = torch.full((B * N + 256, 3 * D), float("nan"), device="cuda")
    room[:B * N] = torch.randn(B * N, 3 * D, generator=g, device="cuda")
    room = room if mode == "fp32" else room.bfloat16()
    for nan_samples in range(B):                     # the last ones
        qkv = room[:B * N].clone()
        room[(B - nan_samples) * N:] = float("nan")
        out = binding.op_attention(room[:B * N], B, N, heads, dh, mode).reshape(B, N, D)
        whole = binding.op_attention(qkv, B, N, heads, dh, mode).reshape(B, N, D)
        assert torch.equal(out[:B - nan_samples], whole[:B - nan_samples]) and torch.isfinite(out[:B - nan_samples].float()).all()
