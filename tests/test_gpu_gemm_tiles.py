"""The GEMM kernels at the sizes where their tiles and K loops can go wrong: remainders in rows and columns, few K slices
and many, column halves of a tile that are all padding.  Reference: the same product by torch, in fp32 on the bf16
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


def check_linear(M, N, K, epilogues=(0, 1, 2)):
    import torch
    from paper_2511_20390_amd import binding
    x, w, bias, resid, gate = _case(M, N, K)
    lin = x.float() @ w.float().T + bias
    if binding.EPI_BIAS in epilogues:
        out = binding.op_linear(x, w, bias, "bf16", binding.EPI_BIAS)
        assert _rel(out, lin) < BF16_TOL
        row = (out.float() - lin).norm(dim=1).max() / lin.norm(dim=1).mean()
        assert row.item() < 2 * BF16_TOL                       # no single row is off
    if binding.EPI_BIAS_GELU in epilogues:
        out = binding.op_linear(x, w, bias, "bf16", binding.EPI_BIAS_GELU)
        assert _rel(out, torch.nn.functional.gelu(lin, approximate="tanh")) < BF16_TOL
    if binding.EPI_GATE_RESID in epilogues:
        got = resid.clone()
        binding.op_linear(x, w, bias, "bf16", binding.EPI_GATE_RESID, resid=got, gate=gate, rows_per_sample=M)
        ref = resid + gate * lin
        assert _rel(got, ref) < F32_TOL
        assert ((got - ref).norm(dim=1).max() / ref.norm(dim=1).mean()).item() < 5 * F32_TOL


def check_linear_fp32(M, N, K):
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


# problems of many rows as the tile choice takes them (which tile that is per epilogue: see TILES below for chosen ones); 1150
# columns: element-wise epilogue
@pytest.mark.parametrize("M,N,K", [(700, 3464, 192), (6000, 1160, 320), (1000, 4600, 192), (8190, 1160, 128), (3000, 4600, 64),
                                   (8190, 4600, 320), (2040, 4600, 1152), (3000, 4600, 320), (8190, 4600, 1152),
                                   (12100, 4600, 1152), (300, 1150, 128)])
def test_many_rows(M, N, K):
    check_linear(M, N, K)


# problems of few rows as the tile choice takes them: a single row, a single group of columns, one to 72 slices
@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (65, 72, 128), (130, 200, 192), (63, 1152, 256), (190, 328, 320), (500, 1160, 384),
                                   (257, 1152, 4608), (390, 3464, 128), (390, 3464, 192), (390, 3464, 256), (300, 3464, 1152),
                                   (500, 4600, 1152), (1000, 3464, 2304)])
def test_few_rows(M, N, K):
    check_linear(M, N, K)


# Every tile by name, with ragged rows and columns, at each number of slices where its loop takes another way: one, one less than
# the stages of the ring, as many, one more, many (few rows: rings of 4, 3 and 4 stages); one, two, three, many (many rows: two
# stages).  (tile, epilogues, M, N, slices); what is not listed is a combination that the tile choice never makes: 128 x 128 of
# the few-row kernel is taken from 12 slices on, 192 x 256 never with GELU.
ROWS, PIPE, PLAIN, ALL = 1000000, 2000000, (0, 1), (0, 1, 2)
TILES = [
    *[(ROWS + 64064, ALL, M, N, n) for M, N, n in ((1, 8, 1), (65, 72, 3), (130, 200, 4), (63, 1160, 5), (257, 1160, 72))],
    *[(ROWS + 128064, PLAIN, 9000, N, n) for N, n in ((392, 1), (392, 2), (392, 3), (72, 4), (72, 5), (72, 36))],
    (ROWS + 128064, (2,), 9000, 72, 12), (ROWS + 128064, (2,), 9000, 72, 36),
    (ROWS + 128128, PLAIN, 9000, 200, 12), (ROWS + 128128, PLAIN, 390, 4104, 36), (ROWS + 128128, (2,), 9000, 200, 36),
    *[(PIPE + 128128, ALL, 9000, 200, n) for n in (1, 2, 3, 4)], (PIPE + 128128, (1, 2), 10000, 520, 36),
    (PIPE + 160128, PLAIN, 9000, 392, 18), (PIPE + 160128, ALL, 9000, 392, 72),
    (PIPE + 192128, (1,), 11000, 328, 1), (PIPE + 192128, PLAIN, 11000, 328, 2), (PIPE + 192128, PLAIN, 11000, 328, 3),
    (PIPE + 192128, (2,), 9000, 392, 3), (PIPE + 192128, PLAIN, 8190, 520, 36), (PIPE + 192128, (2,), 9000, 392, 36),
    (PIPE + 192256, (0,), 11000, 1000, 3), (PIPE + 192256, (0,), 11000, 1000, 18), (PIPE + 192256, (2,), 5000, 1544, 72),
    (PIPE + 256192, (1, 2), 5000, 1544, 1), (PIPE + 256192, (1, 2), 5000, 1544, 2), (PIPE + 256192, ALL, 5000, 1544, 3),
    (PIPE + 256192, ALL, 8190, 4600, 36),
    (PIPE + 256256, (1,), 10000, 1160, 1), (PIPE + 256256, (0,), 11000, 1000, 2), (PIPE + 256256, (1,), 10000, 1160, 2),
    (PIPE + 256256, (0,), 5000, 2312, 3), (PIPE + 256256, (1,), 10000, 1160, 3), (PIPE + 256256, ALL, 5000, 2312, 36),
    (PIPE + 384192, (1,), 10000, 1544, 1), (PIPE + 384192, (1,), 10000, 1544, 2), (PIPE + 384192, (1,), 10000, 1544, 3),
    (PIPE + 384192, (0,), 6500, 2312, 4), (PIPE + 384192, (2,), 10000, 1544, 6), (PIPE + 384192, ALL, 6500, 2312, 36),
]


@pytest.mark.parametrize("tile,epilogues,M,N,slices", TILES)
def test_tile(tile, epilogues, M, N, slices):
    from paper_2511_20390_amd import binding
    for epi in epilogues:
        assert binding.load().free_linear_tile(M, N, 64 * slices, binding.FREE_BF16, epi) == tile
    check_linear(M, N, 64 * slices, epilogues)


# fp32, slices of 32: as the tile choice takes them (the last one is beyond the rows of its table)
@pytest.mark.parametrize("M,N,K", [(1, 8, 32), (65, 72, 64), (130, 200, 96), (63, 1152, 160), (257, 1152, 4608), (450, 3464, 1152),
                                   (512, 4600, 1152), (900, 3464, 1152), (1200, 2304, 768), (1000, 4600, 384), (1500, 4600, 256),
                                   (2048, 3080, 192), (2049, 1160, 64)])
def test_few_rows_fp32(M, N, K):
    check_linear_fp32(M, N, K)


# the same by tile (rings of 4 and 3 stages; 0: the register-staged kernel, two stages)
@pytest.mark.parametrize("tile,M,N,slices", [
    *[(ROWS + 64064, M, N, n) for M, N, n in ((1, 8, 1), (65, 72, 3), (130, 200, 4), (63, 1160, 5), (257, 1160, 144))],
    *[(ROWS + 128064, M, N, n) for M, N, n in ((200, 8200, 1), (300, 8200, 2), (1900, 1544, 3), (1900, 1544, 4), (65, 8200, 36))],
    *[(96128, M, N, n) for M, N, n in ((450, 8200, 1), (200, 8200, 2), (200, 8200, 3), (200, 8200, 36))],
    *[(128128, M, N, n) for M, N, n in ((1200, 8200, 1), (1200, 8200, 2), (1000, 6152, 3), (1900, 1544, 36))],
    *[(160128, M, N, n) for M, N, n in ((900, 8200, 1), (1000, 8200, 2), (1000, 8200, 3), (450, 8200, 36))],
    (256256, 1500, 8200, 12)])
def test_tile_fp32(tile, M, N, slices):
    from paper_2511_20390_amd import binding
    for epi in ALL:
        assert binding.load().free_linear_tile(M, N, 32 * slices, binding.FREE_FP32, epi) == tile
    check_linear_fp32(M, N, 32 * slices)


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
