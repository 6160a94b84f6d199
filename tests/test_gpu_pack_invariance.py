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


# 450 tokens are no multiple of 32, 576 columns none of 128; few heads and many keys, long K of a narrow layer, both of them
@pytest.mark.parametrize("hidden,heads,lat_h,lat_w,B", [(384, 6, 36, 50, 10), (1152, 16, 36, 50, 10), (576, 8, 32, 34, 16)])
def test_never_folded_same_bits_at_every_size(hidden, heads, lat_h, lat_w, B):
    """Models whose LayerNorms are folded at no size: alone, in a pack of just under 4096 token rows and in one of more."""
    import torch
    from paper_2511_20390_amd import binding
    cfg = synth.dit_config("small", hidden=hidden, heads=heads, mlp_hidden=4 * hidden, depth=2, lat_h=lat_h, lat_w=lat_w)
    model = binding.FreeDit(cfg, pu.weights_for(cfg, "bf16", 15), "bf16")
    assert (B - 1) * synth.n_tokens(cfg) < 4096 <= B * synth.n_tokens(cfg) and not model.ln_fold_active(B)
    rng = np.random.default_rng(16)
    x = pu.to_dev(rng.standard_normal((B, cfg["in_ch"], lat_h, lat_w)).astype(np.float32))
    t, y = (pu.to_dev(rng.integers(0, n, B).astype(np.int32)) for n in (1000, cfg["num_classes"] + 1))
    eps, feat = (v.clone() for v in model.dit_forward_packed(x, t, y, want_feat=True))
    for n in (1, B - 1):
        eps1, feat1 = model.dit_forward_packed(*(v[:n].contiguous() for v in (x, t, y)), want_feat=True)
        assert torch.equal(eps1.reshape(-1), eps[:n].reshape(-1)), n
        assert torch.equal(feat1.reshape(-1), feat.reshape(B, -1)[:n].reshape(-1)), n
    model.close()


@pytest.mark.parametrize("hidden,heads,depth", [(512, 8, 44), (1152, 16, 5), (2048, 16, 3)])
def test_reading_weights_ahead_changes_no_bit(hidden, heads, depth):
    """Models whose weights do not stay in the caches have them read ahead by the LayerNorm and attention launches of small
    packs; the same states in a pack of 17, too large for that, without folded LayerNorms, give the same bits."""
    import torch
    from paper_2511_20390_amd import binding
    cfg = synth.dit_config("small", hidden=hidden, heads=heads, mlp_hidden=4 * hidden, depth=depth, lat_h=32, lat_w=32)
    assert depth * 18 * hidden * hidden * 2 >= 220 << 20 and 17 * synth.n_tokens(cfg) >= 4096
    model = binding.FreeDit(cfg, pu.weights_for(cfg, "bf16", 13), "bf16")
    model.set_ln_fold(binding.LN_FOLD_OFF)
    rng = np.random.default_rng(14)
    x = pu.to_dev(rng.standard_normal((17, cfg["in_ch"], 32, 32)).astype(np.float32))
    t, y = (pu.to_dev(rng.integers(0, n, 17).astype(np.int32)) for n in (1000, cfg["num_classes"] + 1))
    eps, feat = (v.clone() for v in model.dit_forward_packed(x, t, y, want_feat=True))
    for lo, hi in ((0, 1), (1, 4), (4, 17)):
        part = [v[lo:hi].contiguous() for v in (x, t, y)]
        eps1, feat1 = model.dit_forward_packed(*part, want_feat=True)
        assert torch.equal(eps1.reshape(-1), eps[lo:hi].reshape(-1)), lo
        assert torch.equal(feat1.reshape(-1), feat.reshape(17, -1)[lo:hi].reshape(-1)), lo
    model.close()


def test_reading_weights_ahead_with_parts_changes_no_bit():
    """The same in what small packs run by default: the LayerNorm that reads ahead also adds up the parts of the MLP's second layer (one
    and two states: one and four wavefronts per workgroup), which one workgroup per tile adds in larger packs."""
    import torch
    from paper_2511_20390_amd import binding
    cfg = synth.dit_config("small", hidden=1152, heads=16, mlp_hidden=4608, depth=5, lat_h=32, lat_w=32)
    assert 5 * 18 * 1152 * 1152 * 2 >= 220 << 20 and 15 * synth.n_tokens(cfg) < 4096
    model = binding.FreeDit(cfg, pu.weights_for(cfg, "bf16", 19), "bf16")
    rng = np.random.default_rng(20)
    x = pu.to_dev(rng.standard_normal((15, cfg["in_ch"], 32, 32)).astype(np.float32))
    t, y = (pu.to_dev(rng.integers(0, n, 15).astype(np.int32)) for n in (1000, cfg["num_classes"] + 1))
    eps, feat = (v.clone() for v in model.dit_forward_packed(x, t, y, want_feat=True))
    for lo, hi in ((0, 1), (1, 3), (3, 6), (2, 14)):
        eps1, feat1 = model.dit_forward_packed(*(v[lo:hi].contiguous() for v in (x, t, y)), want_feat=True)
        assert torch.equal(eps1.reshape(-1), eps[lo:hi].reshape(-1)), lo
        assert torch.equal(feat1.reshape(-1), feat.reshape(15, -1)[lo:hi].reshape(-1)), lo
    model.close()


def test_forced_streams_change_no_bit_of_small_batches():
    """Below 4096 token rows the sums of the split layers go through one workspace region: with two or three streams forced such a
    batch gives the bits of one stream."""
    import torch
    from paper_2511_20390_amd import binding
    cfg = synth.dit_config("small", hidden=1152, heads=16, mlp_hidden=4608, depth=2, lat_h=32, lat_w=32)
    model = binding.FreeDit(cfg, pu.weights_for(cfg, "bf16", 17), "bf16")
    rng = np.random.default_rng(18)
    for B in (2, 15):
        x = pu.to_dev(rng.standard_normal((B, cfg["in_ch"], 32, 32)).astype(np.float32))
        t, y = (pu.to_dev(rng.integers(0, n, B).astype(np.int32)) for n in (1000, cfg["num_classes"] + 1))
        res = []
        for n in (1, 2, 3):
            model.set_streams(n)
            res.append([v.clone() for v in model.dit_forward_packed(x, t, y, want_feat=True)])
        for r in res[1:]:
            assert torch.equal(r[0], res[0][0]) and torch.equal(r[1], res[0][1]), B
    model.close()


# the conditioning's linear layers take four or eight samples per pass and one to five pieces of a row at once: rows of one piece, of a whole
# number of pieces, of more than one pass; the modulation's and the embedding's launches go by the samples too (17: two
# modulation passes; larger workgroups from 10 samples on in fp32 at two blocks of width 1152, at width 1280 from 16 on and in fp32 from 4)
@pytest.mark.parametrize("mode", ["bf16", "fp32"])
@pytest.mark.parametrize("hidden,heads,t_freq,depth", [(384, 6, 256, 1), (512, 8, 64, 1), (576, 8, 260, 1), (1152, 16, 256, 1), (1152, 16, 256, 2),
                                                       (1280, 20, 256, 1), (2048, 16, 256, 1)])
def test_small_packs_of_every_size_same_bits(hidden, heads, t_freq, depth, mode):
    import torch
    from oracle import free_oracle as fo
    from paper_2511_20390_amd import binding
    cfg = synth.dit_config("tiny", hidden=hidden, heads=heads, mlp_hidden=2 * hidden, depth=depth, lat_h=2, lat_w=6, t_freq_dim=t_freq)
    w = pu.weights_for(cfg, mode, 21)
    model = binding.FreeDit(cfg, w, mode)
    rng = np.random.default_rng(22)
    x = rng.standard_normal((17, cfg["in_ch"], 2, 6)).astype(np.float32)
    t, y = (rng.integers(0, n, 17).astype(np.int32) for n in (1000, cfg["num_classes"] + 1))
    dev = [pu.to_dev(v) for v in (x, t, y)]
    eps, feat = (v.clone() for v in model.dit_forward_packed(*dev, want_feat=True))
    ref = fo.dit_forward(w, cfg, x, t, y)
    assert pu.rel_l2(eps.cpu().numpy(), ref[0]) <= pu.DIT_REL_L2[mode] and pu.rel_l2(feat.cpu().numpy(), ref[1]) <= pu.DIT_REL_L2[mode]
    for B in (1, 4, 5, 8, 9, 12, 13, 16):
        eps1, feat1 = model.dit_forward_packed(*(v[:B].contiguous() for v in dev), want_feat=True)
        assert torch.equal(eps1.reshape(-1), eps[:B].reshape(-1)), B
        assert torch.equal(feat1.reshape(-1), feat.reshape(17, -1)[:B].reshape(-1)), B
    model.close()
