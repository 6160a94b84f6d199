"""The tile that a dense projection is given against the times of the tiles (us, launches back to back on one MI355X of 256
compute units, weights from HBM and from the caches in equal parts).  Host only."""
import pytest

from paper_2511_20390_amd import binding

BIAS, GELU, RESID = binding.EPI_BIAS, binding.EPI_BIAS_GELU, binding.EPI_GATE_RESID
ROWS, PIPE = 1000000, 2000000


@pytest.mark.parametrize("M,N,K,epi,us", [
    # a drafting step of two states of 1024 tokens: QKV, out-projection, MLP-1, MLP-2, fusion layer
    (2048, 3456, 1152, BIAS, {PIPE + 128128: 20.4, PIPE + 160128: 21.8, PIPE + 192256: 23.2}),
    (2048, 1152, 1152, RESID, {PIPE + 128128: 15.0, ROWS + 128128: 16.0, ROWS + 128064: 16.9}),
    (2048, 4608, 1152, GELU, {PIPE + 160128: 26.2, PIPE + 192128: 27.3, PIPE + 192256: 28.5}),
    (2048, 1152, 4608, RESID, {ROWS + 128128: 40.7, PIPE + 128128: 46.4, ROWS + 128064: 47.6}),
    (2048, 1152, 2304, RESID, {ROWS + 128128: 22.2, PIPE + 128128: 23.2, ROWS + 128064: 26.5}),
    # width 768, many rows
    (4000, 768, 768, RESID, {PIPE + 128128: 11.3, ROWS + 128128: 15.1, PIPE + 192128: 15.3}),
    (2700, 3072, 768, GELU, {PIPE + 160128: 19.2, PIPE + 192128: 20.4, PIPE + 192256: 21.8}),
    # few rows
    (512, 1152, 4608, RESID, {ROWS + 64064: 19.9, ROWS + 128064: 28.7}),
    (512, 3456, 1152, BIAS, {ROWS + 128064: 8.9, ROWS + 64064: 10.4, ROWS + 128128: 11.5}),
    (512, 384, 384, RESID, {ROWS + 64064: 5.0, ROWS + 128064: 6.6, PIPE + 128128: 7.1}),
])
def test_chosen_tile_is_within_4_percent_of_the_best_one(M, N, K, epi, us):
    tile = binding.load().free_linear_tile(M, N, K, binding.FREE_BF16, epi)
    assert tile in us and us[tile] <= 1.04 * min(us.values()), (tile, us)


def test_tile_query_errors():
    tile = binding.load().free_linear_tile
    assert tile(64, 64, 64, 7, BIAS) == binding.FREE_ERR_DTYPE
    assert tile(64, 64, 64, binding.FREE_BF16, 6) == binding.FREE_ERR_RANGE
    assert tile(64, 64, 64, binding.FREE_BF16, -1) == binding.FREE_ERR_RANGE
    assert tile(64, 64, 60, binding.FREE_BF16, BIAS) == binding.FREE_ERR_SHAPE      # no whole 16-byte chunks
    assert tile(64, 64, 96, binding.FREE_BF16, 3) == binding.FREE_ERR_SHAPE         # folded LayerNorm: whole slices only
    assert tile(64, 64, 64, binding.FREE_FP32, 3) == binding.FREE_ERR_SHAPE         # and bf16 only


@pytest.mark.parametrize("folded", [True, False])
def test_measured_traffic_belongs_to_the_kernels_of_the_benchmark(folded):
    """The kernel names under which bench.py looks measured HBM traffic up are those of the kernels its round launches (12288
    rows of width 1152), and the committed summary has a line for each."""
    import re

    import bench
    layers = {"gemm_qkv": (3456, 1152, 3 if folded else BIAS), "gemm_proj": (1152, 1152, 5 if folded else RESID),
              "gemm_fc1": (4608, 1152, 4 if folded else GELU), "gemm_fc2": (1152, 4608, 5 if folded else RESID)}
    names = bench.CATEGORY_SYMBOL if folded else bench.CATEGORY_SYMBOL_PLAIN
    for cat, (N, K, epi) in layers.items():
        m = re.match(r"gemm_pipe_kernel<(\d+), (\d+), \d, \d, (\d)>`", names[cat])
        assert m, names[cat]
        tile = PIPE + 1000 * int(m[1]) + int(m[2])
        assert (tile, int(m[3])) == (binding.load().free_linear_tile(12288, N, K, binding.FREE_BF16, epi), epi), cat
        t = bench.measured_traffic(cat, folded)
        assert t and 0 < t["write_MB"] <= t["fetch_MB"], cat
    for cat in ("attention", "verify_partial"):
        assert bench.measured_traffic(cat, folded), cat
