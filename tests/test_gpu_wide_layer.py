"""The fused layer kernel of widths 256 and 384: workgroups of 32, 64 and 96 rows (chosen by the number of
rows) give every row the same bits, down to a single row, for feed-forward blocks of one hidden
chunk, several, and as many as it takes; and they give what the oracle gives.  899 tokens a frame
(rows no tile height divides): one frame is in the first range of the rule, 10, 19 and 28 frames
are just inside the others."""
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


@pytest.mark.parametrize("ffn, frames", [(128, 10), (640, 19), (2048, 28)])
def test_rows_per_workgroup_do_not_change_a_result(ffn, frames):
    import torch

    cfg = synth.Config("wide", frames, 232, 248, (8,), 384, 6, 2, ffn, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 7)
    rng = np.random.default_rng(3)
    images = synth.bf16_round(rng.normal(0.5, 0.25, (frames, 3, cfg.H, cfg.W)).astype(np.float32))
    many = _coarse(cfg, w, images)
    assert torch.isfinite(many).all()
    for f in (0, frames - 1):
        assert torch.equal(_coarse(synth.replace(cfg, B=1), w, images[f:f + 1])[0], many[f]), f
    ref = np.asarray(O.coarse_encode(images[:1], cfg.patch, w, cfg.heads)[-1]).reshape(-1, cfg.d)
    err = float(np.abs(many[0].cpu().numpy() - ref).max() / np.abs(ref).max())
    print("fused layer against the oracle:", err, flush=True)
    assert err <= BAR


@pytest.mark.parametrize("rows", [(1, 1), (1, 31), (3, 11), (5, 13)])
def test_few_rows(rows):
    cfg = synth.Config("narrow", 1, 8 * rows[0], 8 * rows[1], (8,), 384, 6, 1, 256, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 9)
    images = synth.bf16_round(np.random.default_rng(5).normal(0.5, 0.25, (1, 3, cfg.H, cfg.W)).astype(np.float32))
    y = _coarse(cfg, w, images)[0].cpu().numpy()
    ref = np.asarray(O.coarse_encode(images, cfg.patch, w, cfg.heads)[-1]).reshape(-1, cfg.d)
    assert float(np.abs(y - ref).max() / np.abs(ref).max()) <= BAR


@pytest.mark.parametrize("ffn, frames", [(256, 10), (1024, 19), (2048, 28)])
def test_rows_per_workgroup_at_width_256(ffn, frames):
    """One frame has workgroups of 32 rows, 10 and 28 frames of 64, 19 frames of 96."""
    import torch

    cfg = synth.Config("wide256", frames, 232, 248, (8,), 256, 8, 2, ffn, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 11)
    rng = np.random.default_rng(4)
    images = synth.bf16_round(rng.normal(0.5, 0.25, (frames, 3, cfg.H, cfg.W)).astype(np.float32))
    many = _coarse(cfg, w, images)
    assert torch.isfinite(many).all()
    for f in (0, frames - 1):
        assert torch.equal(_coarse(synth.replace(cfg, B=1), w, images[f:f + 1])[0], many[f]), f
    ref = np.asarray(O.coarse_encode(images[:1], cfg.patch, w, cfg.heads)[-1]).reshape(-1, cfg.d)
    assert float(np.abs(many[0].cpu().numpy() - ref).max() / np.abs(ref).max()) <= BAR


@pytest.mark.parametrize("rows", [(1, 1), (1, 31), (3, 11), (5, 13)])
def test_few_rows_at_width_256(rows):
    cfg = synth.Config("narrow256", 1, 8 * rows[0], 8 * rows[1], (8,), 256, 8, 1, 512, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 13)
    images = synth.bf16_round(np.random.default_rng(6).normal(0.5, 0.25, (1, 3, cfg.H, cfg.W)).astype(np.float32))
    y = _coarse(cfg, w, images)[0].cpu().numpy()
    ref = np.asarray(O.coarse_encode(images, cfg.patch, w, cfg.heads)[-1]).reshape(-1, cfg.d)
    assert float(np.abs(y - ref).max() / np.abs(ref).max()) <= BAR


@pytest.mark.parametrize("d", [256, 384])
def test_last_tile_at_the_capacity_stays_inside_its_buffer(d):
    """9,696 rows, all that the context has room for: the last workgroup's 64 rows end 32 rows past a
    multiple of 96.  What lies behind (packed weights) is read by the passes of one frame."""
    import torch
    from paper_2505_23317_amd import cfdetr as K

    cfg = synth.Config("full", 8, 48, 808, (8,), d, d // 64 if d == 384 else 8, 2, 256, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 21)
    images = synth.bf16_round(np.random.default_rng(7).normal(0.5, 0.25, (cfg.B, 3, cfg.H, cfg.W)).astype(np.float32))
    enc = K.Encoder(cfg, w)
    out = enc.alloc_outputs(cfg.B)
    img = enc.upload_images(images)
    assert enc.max_tokens == cfg.B * 606

    def one_frame():
        enc.coarse_encode(img, 1, out["x0_cache"], out["y_coarse"])
        enc.sync_status()
        return out["y_coarse"].reshape(-1, d)[:606].clone()

    before = one_frame()
    b, t, o = enc.upload_boxes(np.zeros((0, 4), np.int32), np.zeros(0, np.uint8), np.zeros(cfg.B + 1, np.int32))
    for _ in range(2):
        enc.multilevel_batch(img, cfg.B, b, t, o, out)
        enc.sync_status()
        assert torch.equal(out["y_coarse"].reshape(-1, d)[:606], before)
        assert torch.equal(out["y_mixed"].reshape(-1, d)[:4848], out["y_coarse"].reshape(-1, d)[:4848])
    assert torch.equal(one_frame(), before)
    enc.close()
