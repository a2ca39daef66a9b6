"""Widths 64 and 128: the kernel that does everything of a layer after attention, 32 rows a workgroup.  Feed-forward
blocks of the fewest and the most hidden chunks, rows that end inside, at and one behind a workgroup's: a frame
is the same bit for bit alone and in a batch (whose rows lie elsewhere in the workgroups), and what the oracle gives."""
import numpy as np
import pytest

from oracle import cfdetr_oracle as O
from paper_2505_23317_amd import synth

pytestmark = pytest.mark.gpu

BAR = 2e-2


def _coarse(cfg, w, images):
    from paper_2505_23317_amd import cfdetr as K
    enc = K.Encoder(cfg, w)
    n = images.shape[0]
    out = enc.alloc_outputs(n)
    enc.coarse_encode(enc.upload_images(images), n, out["x0_cache"], out["y_coarse"])
    enc.sync_status()
    y = out["y_coarse"].reshape(n, -1, cfg.d).clone()
    enc.close()
    return y


# 5 frames: 5, 160, 165 and 4,495 rows
@pytest.mark.parametrize("cells", [(1, 1), (4, 8), (3, 11), (29, 31)])
@pytest.mark.parametrize("d, heads, ffn", [(64, 2, 128), (64, 2, 1024), (128, 4, 128), (128, 4, 896)])
def test_rows_alone_and_in_a_batch(d, heads, ffn, cells):
    import torch

    frames = 5
    cfg = synth.Config("small", frames, 8 * cells[0], 8 * cells[1], (8,), d, heads, 3, ffn, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 29)
    images = synth.bf16_round(np.random.default_rng(7).normal(0.5, 0.25, (frames, 3, cfg.H, cfg.W)).astype(np.float32))
    many = _coarse(cfg, w, images)
    assert torch.isfinite(many).all()
    for f in (0, frames - 1):
        assert torch.equal(_coarse(synth.replace(cfg, B=1), w, images[f:f + 1])[0], many[f]), f
    ref = np.asarray(O.coarse_encode(images[frames - 1:], cfg.patch, w, cfg.heads)[-1]).reshape(-1, d)
    assert float(np.abs(many[-1].cpu().numpy() - ref).max() / np.abs(ref).max()) <= BAR


# the largest hidden block there is, two workgroups a CU: 32,000 rows are two rounds of them and more
@pytest.mark.parametrize("d, heads", [(64, 2), (128, 4)])
def test_largest_hidden_block_over_many_rows(d, heads):
    import torch

    frames = 32
    cfg = synth.Config("small", frames, 8 * 8, 8 * 125, (8,), d, heads, 2, 1024, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 29)
    images = synth.bf16_round(np.random.default_rng(7).normal(0.5, 0.25, (frames, 3, cfg.H, cfg.W)).astype(np.float32))
    many = _coarse(cfg, w, images)
    assert torch.isfinite(many).all()
    for f in (0, frames // 2, frames - 1):
        assert torch.equal(_coarse(synth.replace(cfg, B=1), w, images[f:f + 1])[0], many[f]), f
    ref = np.asarray(O.coarse_encode(images[frames - 1:], cfg.patch, w, cfg.heads)[-1]).reshape(-1, d)
    assert float(np.abs(many[-1].cpu().numpy() - ref).max() / np.abs(ref).max()) <= BAR
