"""The output layer on the matrix cores (both weight types, every width it has), from the top feature the same forward returns: LayerNorm,
modulation, projection and the order of the pixels, against 64 bits."""
import numpy as np
import pytest

from oracle import free_oracle as fo
from paper_2511_20390_amd import synth
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


# token rows that are no multiple of a workgroup's 16, fewer than one workgroup's, several samples in one workgroup
@pytest.mark.parametrize("mode", ["fp32", "bf16"])
@pytest.mark.parametrize("hidden,heads,lat_h,lat_w,B", [(384, 6, 18, 22, 3), (768, 12, 2, 6, 1), (1024, 16, 6, 10, 2), (1152, 16, 10, 14, 3)])
def test_output_layer(hidden, heads, lat_h, lat_w, B, mode):
    # bf16 weights: activations in two bf16 parts, 2^-17 of each; fp32: sums of up to 1152 products in fp32
    assert _output_layer_error(hidden, heads, lat_h, lat_w, B, mode) < (2e-5 if mode == "bf16" else 4e-6)


# fp32: a rounding is off by 2^-24 / sqrt(3) of the value at random.  A level of a sum that is added pair by pair costs one of the sum's
# size, a chain of n products about (n + 1) / 2, the modulated value and the bias two: eight products in a chain, 4 D / 128 such chains of a lane,
# four wavefronts.  A third more for what is not random
@pytest.mark.parametrize("hidden,heads,lat_h,lat_w,B", [(384, 6, 36, 44, 2), (768, 12, 32, 32, 2), (1024, 16, 32, 32, 2), (1152, 16, 32, 32, 2)])
def test_output_layer_fp32_sums(hidden, heads, lat_h, lat_w, B):
    levels = 4.5 + np.ceil(np.log2(4 * hidden / 128)) + 2 + 2
    assert _output_layer_error(hidden, heads, lat_h, lat_w, B, "fp32") < 4 / 3 * 2.0 ** -24 / np.sqrt(3) * np.sqrt(levels)


def _output_layer_error(hidden, heads, lat_h, lat_w, B, mode):
    from paper_2511_20390_amd import binding
    cfg = synth.dit_config("tiny", hidden=hidden, heads=heads, mlp_hidden=2 * hidden, depth=1, lat_h=lat_h, lat_w=lat_w)
    w = pu.weights_for(cfg, mode, 41)
    model = binding.FreeDit(cfg, w, mode)
    rng = np.random.default_rng(42)
    x = rng.standard_normal((B, cfg["in_ch"], lat_h, lat_w)).astype(np.float32)
    t, y = (rng.integers(0, n, B).astype(np.int32) for n in (1000, cfg["num_classes"] + 1))
    eps, feat = model.dit_forward_packed(*(pu.to_dev(v) for v in (x, t, y)), want_feat=True)
    w64 = {k: np.asarray(v, np.float64) for k, v in w.items()}
    mod = fo.linear(fo.silu(fo.conditioning(w64, cfg, t, y)), w64["fin_ada_w"], w64["fin_ada_b"])
    shift, scale = mod[:, None, :hidden], mod[:, None, hidden:]
    top = feat.double().cpu().numpy().reshape(B, -1, hidden)
    tok = fo.linear(fo.layer_norm(top) * (1.0 + scale) + shift, w64["fin_w"], w64["fin_b"])
    p = cfg["patch"]
    ref = fo.unpatchify(tok, p, tok.shape[-1] // (p * p), lat_h // p, lat_w // p)
    model.close()
    return pu.rel_l2(eps.cpu().numpy().reshape(ref.shape), ref)
