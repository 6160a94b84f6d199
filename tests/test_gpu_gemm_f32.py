"""The linear layers of fp32 models (three bf16 parts per value on the matrix cores) at the sizes where their tiles and K loop can go
wrong, against the product in 64 bits and against the fp32 instructions."""
import pytest

pytestmark = pytest.mark.gpu

# three parts carry all 24 bits and the one product left out is below 2^-30 of each: what remains are fp32 sums, sqrt(K) 2^-24 of
# the result where errors are independent (4e-6 at K = 4608); five times that, as for the fp32 instructions
F32_TOL = 2e-5


def _data(M, N, K, seed=0):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed + M + N + K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    return rnd(M, K), rnd(N, K) / K ** 0.5, rnd(N), rnd(M, N), rnd(1, N)


def _rel(a, b):
    return ((a.double() - b.double()).norm() / b.double().norm()).item()


# one row, one column group, one to 144 slices (the loop takes four per pass), ragged rows and columns, 1150 and 4597 columns:
# element-wise epilogue; the last four on 128 x 128 tiles (one round of them against four of 64 x 64, from eight slices on), the others on
# 64 x 64
@pytest.mark.parametrize("M,N,K", [(1, 8, 32), (65, 72, 64), (130, 200, 96), (63, 1152, 128), (64, 64, 160), (257, 1152, 4608),
                                   (450, 1150, 384), (512, 4608, 1152), (600, 3464, 1152), (2050, 1160, 32), (3000, 4600, 224),
                                   (770, 4600, 1152), (771, 4597, 288), (769, 4608, 320), (770, 4600, 352)])
def test_parts(M, N, K):
    import torch
    from paper_2511_20390_amd import binding
    x, w, bias, resid, gate = _data(M, N, K)
    ref = x.double() @ w.double().T + bias
    out = binding.op_linear_f32(x, w, bias)
    err = _rel(out, ref)
    assert err < F32_TOL
    if M * N >= 4096:                                    # no further off than the fp32 instructions
        assert err <= 1.02 * _rel(binding.op_linear(x, w, bias, "fp32"), ref)
    assert ((out - ref).norm(dim=1).max() / ref.norm(dim=1).mean()).item() < 5 * F32_TOL
    out = binding.op_linear_f32(x, w, bias, binding.EPI_BIAS_GELU)
    assert _rel(out, torch.nn.functional.gelu(ref, approximate="tanh")) < F32_TOL
    got = resid.clone()
    binding.op_linear_f32(x, w, bias, binding.EPI_GATE_RESID, resid=got, gate=gate, rows_per_sample=M)
    ref = resid + gate * ref
    assert _rel(got, ref) < F32_TOL
    assert ((got - ref).norm(dim=1).max() / ref.norm(dim=1).mean()).item() < 5 * F32_TOL


# 64 x 64 tiles and 128 x 128 ones; fewer and more slices than the loop takes per pass
@pytest.mark.parametrize("M,N,K", [(300, 200, 32), (513, 1152, 1152), (3000, 1160, 352)])
def test_few_terms(M, N, K):
    """Sums that no averaging helps.  One non-zero per row: every result is one product and must be it, rounded once (2^-24; the seven
    products below the leading one have sums of 2^-7 of it, each rounded: 2^-31; the ninth, left out, is below 2^-30).  A few
    non-zeros: no further off than the fp32 instructions."""
    import torch
    from paper_2511_20390_amd import binding
    x, w, bias, _, _ = _data(M, N, K, seed=2)
    bias.zero_()
    g = torch.Generator(device="cuda").manual_seed(3)
    one = torch.zeros_like(x)
    at = torch.randint(0, K, (M, 1), generator=g, device="cuda")
    one.scatter_(1, at, x.gather(1, at))
    ref = one.double() @ w.double().T
    err = (binding.op_linear_f32(one, w, bias).double() - ref).abs() / ref.abs().clamp_min(1e-300)
    assert err.max().item() <= 2 ** -24 + 8 * 2 ** -31 + 2 ** -30
    few = x * (torch.rand(M, K, generator=g, device="cuda") < 0.05)
    few[:, K // 2:] = 0
    ref = few.double() @ w.double().T
    assert _rel(binding.op_linear_f32(few, w, bias), ref) <= 1.02 * _rel(binding.op_linear(few, w, bias, "fp32"), ref)


def test_rows_do_not_depend_on_the_pack():
    """Both tiles add in the same order: 70 rows alone (64 x 64) are those of 3000 (128 x 128), bit for bit."""
    import torch
    from paper_2511_20390_amd import binding
    x, w, bias, _, _ = _data(3000, 1152, 352)
    assert torch.equal(binding.op_linear_f32(x[:70].contiguous(), w, bias), binding.op_linear_f32(x, w, bias)[:70])


# 64 x 64 tiles; 128 x 128 ones at K = 352
@pytest.mark.parametrize("M,N,K", [(100, 72, 64), (3000, 1160, 64), (3000, 1160, 352)])
def test_values_without_three_parts(M, N, K):
    """Infinities, NaN, magnitudes near both ends of fp32: what fp32 products give."""
    import torch
    from paper_2511_20390_amd import binding
    x, w, bias, _, _ = _data(M, N, K, seed=1)
    x[3, 5], x[40, 7], x[70, 0], x[71, :], w[9, 1] = float("inf"), float("nan"), 3e38, 1e-42, float("-inf")
    out, ref = binding.op_linear_f32(x, w, bias), x @ w.T + bias
    assert torch.equal(out.isnan(), ref.isnan()) and torch.equal(out.isinf(), ref.isinf())
    assert torch.equal(out[ref.isinf()], ref[ref.isinf()])
    ok = ref.isfinite()
    # K products: errors of K 2^-24 of the largest partial sum at worst
    assert ((out - ref).abs()[ok] <= K * 2 ** -24 * (x.abs() @ w.abs().T + bias.abs())[ok]).all()


@pytest.mark.parametrize("M,N,K", [(100, 72, 64), (3000, 1160, 352)])
def test_small_magnitudes(M, N, K):
    """Values whose last bits are below the smallest bf16, down to fp32's own smallest: their small sums are rounded once (in steps of
    2^-149 where fp32 has no smaller ones)."""
    import torch
    from paper_2511_20390_amd import binding
    g = torch.Generator(device="cuda").manual_seed(5)
    mant = lambda *s: (1 + torch.rand(*s, generator=g, device="cuda")).double()
    x = torch.zeros(M, K, dtype=torch.float64, device="cuda")
    at = torch.randint(0, K, (M, 1), generator=g, device="cuda")
    x.scatter_(1, at, mant(M, 1) * 2.0 ** torch.arange(-126, -100, device="cuda", dtype=torch.float64).repeat(M)[:M, None])
    for w_exp in (-20, 0, 30):
        w = (mant(N, K) * 2.0 ** w_exp).float()
        ref = x.float().double() @ w.double().T
        out = binding.op_linear_f32(x.float(), w, torch.zeros(N, device="cuda")).double()
        assert ((out - ref).abs() <= ref.abs() * 2 ** -24 + 2.0 ** -150).all(), w_exp


def test_other_rows_keep_their_bits():
    """One row whose sums are not finite or tiny sends its tile to the fp32 products; the rows beside it stay as they were."""
    import torch
    from paper_2511_20390_amd import binding
    x, w, bias, _, _ = _data(200, 136, 96, seed=4)
    ref = binding.op_linear_f32(x, w, bias)
    x[70], x[131, 3] = 1e-36, float("nan")
    out = binding.op_linear_f32(x, w, bias)
    keep = [m for m in range(200) if m not in (70, 131)]
    assert torch.equal(out[keep], ref[keep]) and out[131].isnan().all()


def test_refused():
    import torch
    from paper_2511_20390_amd import binding
    x, w, bias, _, _ = _data(4, 8, 64)
    lib, p = binding.load(), lambda t: t.data_ptr()
    call = lambda a, k, epi: lib.free_op_linear_f32(a, p(w), p(bias), 4, 8, k, epi, p(x), None, None, 0, 1, None)
    assert call(p(x), 36, 0) == binding.FREE_ERR_SHAPE and call(p(x) + 4, 64, 0) == binding.FREE_ERR_SHAPE
    assert call(p(x), 64, 3) == binding.FREE_ERR_RANGE and call(None, 64, 0) == binding.FREE_ERR_NULL
    assert call(p(x), 64, 2) == binding.FREE_ERR_NULL
