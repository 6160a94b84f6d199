"""The GEMM kernels at the sizes where their tiles and K loops can go wrong: remainders in rows and columns, one,
two and three K slices, column halves of a tile that are all padding.  Reference: the same product by torch, in fp32 on the bf16
values or in fp64 on the fp32 values."""
import pytest

pytestmark = pytest.mark.gpu

# A bf16 result is within 2^-9 of the value it rounds, so the 2-norm error is below 2^-9 = 2.0e-3 of the result; the fp32 sums
# add K 2^-24 at worst (2.7e-4 for K = 4608, sqrt(K) 2^-24 = 4e-6 where errors are independent).
BF16_TOL = 2.0e-3 + 3e-4
# fp32 residual: sums in another order only, sqrt(4608) 2^-24 = 4e-6, five times that
F32_TOL = 2e-5


def _case(M, N, K, seed=0):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed + M + N + K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    return (rnd(M, K).to(torch.bfloat16), (rnd(N, K) / K ** 0.5).to(torch.bfloat16), rnd(N),
            rnd(M, N), rnd(1, N))


def _rel(a, b):
    return ((a.double() - b.double()).norm() / b.double().norm()).item()


def check_linear(M, N, K):
    import torch
    from paper_2511_20390_amd import binding
    x, w, bias, resid, gate = _case(M, N, K)
    ref = x.float() @ w.float().T + bias
    out = binding.op_linear(x, w, bias, "bf16", binding.EPI_BIAS)
    assert _rel(out, ref) < BF16_TOL
    row = (out.float() - ref).norm(dim=1).max() / ref.norm(dim=1).mean()
    assert row.item() < 2 * BF16_TOL                           # no single row is off
    out = binding.op_linear(x, w, bias, "bf16", binding.EPI_BIAS_GELU)
    assert _rel(out, torch.nn.functional.gelu(ref, approximate="tanh")) < BF16_TOL
    got = resid.clone()
    binding.op_linear(x, w, bias, "bf16", binding.EPI_GATE_RESID, resid=got, gate=gate, rows_per_sample=M)
    ref = resid + gate * ref
    assert _rel(got, ref) < F32_TOL
    assert ((got - ref).norm(dim=1).max() / ref.norm(dim=1).mean()).item() < 5 * F32_TOL


# every tile of gemm_pipe.hip with ragged rows and columns, one to three slices and more; 1150 columns: element-wise epilogue
@pytest.mark.parametrize("M,N,K", [(700, 3464, 192), (6000, 1160, 320), (1000, 4600, 192), (8190, 1160, 128), (3000, 4600, 64),
                                   (8190, 4600, 320), (2040, 4600, 1152), (3000, 4600, 320), (8190, 4600, 1152),
                                   (12100, 4600, 1152), (300, 1150, 128)])
def test_many_rows(M, N, K):
    check_linear(M, N, K)


# the tiles of gemm_rows.hip: single rows and columns groups, fewer slices than stages, as many, one more and many
@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (65, 72, 128), (130, 200, 192), (63, 1152, 256), (190, 328, 320), (500, 1160, 384),
                                   (257, 1152, 4608), (390, 3464, 128), (390, 3464, 192), (390, 3464, 256), (300, 3464, 1152),
                                   (500, 4600, 1152), (1000, 3464, 2304)])
def test_few_rows(M, N, K):
    check_linear(M, N, K)


# fp32: the tiles of gemm_rows.hip and each of the larger ones; slices of 32, fewer than the ring's stages and more
@pytest.mark.parametrize("M,N,K", [(1, 8, 32), (65, 72, 64), (130, 200, 96), (63, 1152, 160), (257, 1152, 4608), (450, 3464, 1152),
                                   (512, 4600, 1152), (900, 3464, 1152), (1200, 2304, 768), (1000, 4600, 384), (1500, 4600, 256),
                                   (2048, 3080, 192), (2049, 1160, 64)])
def test_few_rows_fp32(M, N, K):
    import torch
    from paper_2511_20390_amd import binding
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    x, w, bias, resid, gate = rnd(M, K), rnd(N, K) / K ** 0.5, rnd(N), rnd(M, N), rnd(1, N)
    ref = x.double() @ w.double().T + bias
    assert _rel(binding.op_linear(x, w, bias, "fp32", binding.EPI_BIAS), ref) < F32_TOL
    out = binding.op_linear(x, w, bias, "fp32", binding.EPI_BIAS_GELU)
    assert _rel(out, torch.nn.functional.gelu(ref, approximate="tanh")) < F32_TOL
    got = resid.clone()
    binding.op_linear(x, w, bias, "fp32", binding.EPI_GATE_RESID, resid=got, gate=gate, rows_per_sample=M)
    ref = resid + gate * ref
    assert _rel(got, ref) < F32_TOL
    assert ((got - ref).norm(dim=1).max() / ref.norm(dim=1).mean()).item() < 5 * F32_TOL


@pytest.mark.parametrize("M,rows", [(8192, 256), (7680, 480), (12288, 1024)])
def test_residual_update_with_row_sums(M, rows):
    """z and the 128-column sums of the prepared LayerNorm from both tiles that write them (192 x 256 and 256 x 256)."""
    import torch
    from paper_2511_20390_amd import binding
    N, K = 1152, 192
    x, w, bias, resid, _ = _case(M, N, K, seed=1)
    g = torch.Generator(device="cuda").manual_seed(M)
    mod = torch.randn(M // rows, 2 * N, generator=g, device="cuda")
    gate, scale = mod[:, :N], mod[:, N:]
    got = resid.clone()
    z, stats = binding.op_linear_resid_prep(x, w, bias, got, gate, scale, rows)
    ref = resid + gate.repeat_interleave(rows, 0) * (x.float() @ w.float().T + bias)
    assert _rel(got, ref) < F32_TOL
    assert _rel(z, got * (1 + scale.repeat_interleave(rows, 0))) < BF16_TOL
    parts = got.double().view(M, N // 128, 128)
    # sums of 128 fp32 values: 128 2^-24 of the sum of magnitudes at worst
    assert (stats[..., 0] - parts.sum(-1)).abs().max().item() < 128 * 2 ** -24 * parts.abs().sum(-1).max().item()
    assert _rel(stats[..., 1], (parts ** 2).sum(-1)) < 128 * 2 ** -24
