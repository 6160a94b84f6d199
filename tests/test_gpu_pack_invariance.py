"""Below the row count from which the LayerNorms are folded, a state's result does not depend on what it is packed with:
every kernel adds in an order that the number of rows has no part in, whichever tile or launch it is given to."""
import numpy as np
import pytest

from paper_2511_20390_amd import synth
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["bf16", "fp32"])
@pytest.mark.parametrize("hidden,heads,lat_h,lat_w,B", [(384, 6, 36, 50, 5), (1152, 16, 32, 32, 6), (768, 12, 64, 64, 3)])
def test_alone_or_packed_same_bits(hidden, heads, lat_h, lat_w, B, mode):
    import torch
    from paper_2511_20390_amd import binding
    cfg = synth.dit_config("small", hidden=hidden, heads=heads, mlp_hidden=4 * hidden, depth=2, lat_h=lat_h, lat_w=lat_w)
    model = binding.FreeDit(cfg, pu.weights_for(cfg, mode, 11), mode)
    rng = np.random.default_rng(12)
    x = pu.to_dev(rng.standard_normal((B, cfg["in_ch"], lat_h, lat_w)).astype(np.float32))
    t, y = (pu.to_dev(rng.integers(0, n, B).astype(np.int32)) for n in (1000, cfg["num_classes"] + 1))
    eps, feat = (v.clone() for v in model.dit_forward_packed(x, t, y, want_feat=True))
    for b in range(B):
        one = [v[b:b + 1].contiguous() for v in (x, t, y)]
        eps1, feat1 = model.dit_forward_packed(*one, want_feat=True)
        assert torch.equal(eps1.reshape(-1), eps[b].reshape(-1)), b
        assert torch.equal(feat1.reshape(-1), feat.reshape(B, -1)[b]), b
    model.close()
