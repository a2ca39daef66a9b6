"""Attention work items of 256 queries (64 per wavefront, taken where there are many query rows)
against items of 128: every query's result must be the same bit for bit, in the ordinary path and
where the sums of probabilities leave the exponent range.  899 tokens a frame: a ragged last key
tile and a last item that is neither empty nor full in either form; 64 frames x 2 heads are just
beyond the line between the forms, one frame is far below it.  One frame is checked against the
oracle."""
import numpy as np
import pytest

from oracle import cfdetr_oracle as O
from paper_2505_23317_amd import synth

pytestmark = pytest.mark.gpu

BAR = 2e-2
FRAMES = 64


@pytest.mark.parametrize("offset_log2", [0.0, 180.0, -200.0])
def test_item_size_does_not_change_a_result(offset_log2):
    import torch
    from paper_2505_23317_amd import cfdetr as K

    cfg = synth.Config("items", FRAMES, 232, 248, (8,), 128, 2, 1, 128, "bf16", box_rule="poisson")
    assert FRAMES * cfg.n_cells(0) * cfg.heads > 3500 * 32
    w = synth.make_weights(cfg, 5)
    if offset_log2:
        # every base-2 logit near offset: constant queries and keys (plus the keys' own part)
        w["w_qkv"][0, : cfg.d, :] = 0.0
        w["b_qkv"][0, : cfg.d] = np.float32(1.0 / (1.4426950408889634 * np.sqrt(cfg.d_head)))
        w["b_qkv"][0, cfg.d: 2 * cfg.d] = np.float32(offset_log2)
    rng = np.random.default_rng(3)
    images = synth.bf16_round(rng.normal(0.5, 0.25, (FRAMES, 3, cfg.H, cfg.W)).astype(np.float32))
    enc = K.Encoder(cfg, w)
    out = enc.alloc_outputs(FRAMES)
    enc.coarse_encode(enc.upload_images(images), FRAMES, out["x0_cache"], out["y_coarse"])
    enc.sync_status()
    many = out["y_coarse"].reshape(FRAMES, -1, cfg.d)
    assert torch.isfinite(many).all()
    one = K.Encoder(synth.replace(cfg, B=1), w)
    o1 = one.alloc_outputs(1)
    for f in (0, 31, FRAMES - 1):
        one.coarse_encode(one.upload_images(images[f:f + 1]), 1, o1["x0_cache"], o1["y_coarse"])
        one.sync_status()
        assert torch.equal(o1["y_coarse"], many[f]), f
    y = O.coarse_encode(images[:1], cfg.patch, w, cfg.heads)[-1]
    ref = np.asarray(y).reshape(-1, cfg.d)
    err = float(np.abs(many[0].cpu().numpy() - ref).max() / np.abs(ref).max())
    print("items of 256 against the oracle:", err, flush=True)
    assert err <= BAR
    one.close()
    enc.close()
