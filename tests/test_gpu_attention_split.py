"""bf16 attention with the keys of a query block split over two wavefronts (batches of few queries) at the sizes where the
split can go wrong: exactly one tile, one key more, a second half that is all past the end in the last tile, a long loop.
Reference: softmax attention in fp32 by torch on the bf16 values."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N,heads,dh", [(1, 64, 2, 72), (1, 65, 3, 72), (2, 96, 2, 64), (1, 97, 1, 16), (2, 129, 2, 128),
                                          (1, 1000, 4, 72), (2, 1024, 16, 72), (1, 63, 2, 72)])
def test_keys_split_over_two_wavefronts(B, N, heads, dh):
    import torch
    from paper_2511_20390_amd import binding
    g = torch.Generator(device="cuda").manual_seed(B * N + dh)
    qkv = (1.5 * torch.randn(B * N, 3 * heads * dh, generator=g, device="cuda")).to(torch.bfloat16)
    qkv[N // 2:, :heads * dh] *= 4.0                          # sharp rows: the two halves' maxima differ widely
    out = binding.op_attention(qkv, B, N, heads, dh, "bf16").float()
    q, k, v = (t.contiguous() for t in qkv.float().view(B, N, 3, heads, dh).permute(2, 0, 3, 1, 4))
    p = torch.softmax(torch.matmul(q * dh ** -0.5, k.transpose(-1, -2).contiguous()), -1)
    ref = torch.matmul(p, v).permute(0, 2, 1, 3).reshape(B * N, heads * dh)
    # probabilities and output rounded to bf16: 2^-9 relative each, 2-norm below their sum
    assert ((out - ref).norm() / ref.norm()).item() < 2 * 2 ** -9
    assert ((out - ref).norm(dim=1).max() / ref.norm(dim=1).mean()).item() < 8 * 2 ** -9
