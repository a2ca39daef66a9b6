"""Patch embedding.  Frames in fp32: a tile by four groups of wavefronts (few tiles), by one group,
and tiles of 128 x 128 give every token the same bits (K is summed in quarters by all), for
patches of 8 (no quarters), 16, 32 and 64 pixels, and the oracle's values.  Frames in bf16: the same of the forms for patches of 64 pixels."""
import numpy as np
import pytest

from oracle import cfdetr_oracle as O
from paper_2505_23317_amd import synth

pytestmark = pytest.mark.gpu


def _embed(cfg, w, images):
    from paper_2505_23317_amd import cfdetr as K
    enc = K.Encoder(cfg, w)
    n = images.shape[0]
    out = enc.alloc_outputs(n)
    enc.coarse_encode(enc.upload_images(images), n, out["x0_cache"], out["y_coarse"])
    enc.sync_status()
    x = out["x0_cache"].reshape(n, -1, cfg.d).clone()
    enc.close()
    return x


# frames of the largest batch: 64 x 64 tiles beyond the CUs, 128 x 128 tiles from 256 on
@pytest.mark.parametrize("patch, rows, cols, d, frames", [
    (8, 37, 41, 128, (1, 6, 24)), (16, 37, 41, 128, (1, 6, 24)), (32, 13, 17, 256, (1, 32, 64)),
    (64, 5, 3, 768, (1, 40)), (16, 1, 1, 64, (1, 2))])
def test_every_form_gives_the_same_bits(patch, rows, cols, d, frames):
    import torch

    cfg = synth.Config("fp32", max(frames), rows * patch, cols * patch, (patch,), d, d // 32 if d < 768 else 12, 1, 128, "f32",
                       box_rule="poisson")
    w = synth.make_weights(cfg, 17)
    images = np.random.default_rng(8).random((max(frames), 3, cfg.H, cfg.W), dtype=np.float32)
    few = _embed(synth.replace(cfg, B=1), w, images[:1])
    ref = np.asarray(O.coarse_encode(images[:1], cfg.patch, w, cfg.heads)[0]).reshape(-1, d)
    # pixels round to bf16 (2^-9), K products of them add up in fp32: relative to the largest value
    assert float(np.abs(few[0].cpu().numpy() - ref).max() / np.abs(ref).max()) <= 2.0 ** -8
    for n in frames[1:]:
        assert torch.equal(_embed(synth.replace(cfg, B=n), w, images[:n])[0], few[0]), n


# few tokens: 2 x 12 tiles of 64 x 64 and smaller; 35 and 40 frames: the kernel with packed weights (gemm_bf16_patch_kernel)
@pytest.mark.parametrize("frames", [(1, 35, 40)])
def test_bf16_frames_with_large_patches(frames):
    import torch

    cfg = synth.Config("bf16", max(frames), 8 * 64, 9 * 64, (64,), 768, 12, 1, 128, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 19)
    images = synth.bf16_round(np.random.default_rng(9).random((max(frames), 3, cfg.H, cfg.W), dtype=np.float32))
    few = _embed(synth.replace(cfg, B=1), w, images[:1])
    ref = np.asarray(O.coarse_encode(images[:1], cfg.patch, w, cfg.heads)[0]).reshape(-1, cfg.d)
    assert float(np.abs(few[0].cpu().numpy() - ref).max() / np.abs(ref).max()) <= 2.0 ** -8
    for n in frames[1:]:
        x = _embed(synth.replace(cfg, B=n), w, images[:n])
        assert torch.equal(x[0], few[0]) and torch.isfinite(x).all(), n


# 221 tokens a frame: 32 x 32 tiles for one and four frames, 32 x 64 for eight, 64 x 64 for sixteen, 64 x 128 with packed
# weights (gemm_bf16_patch_kernel) for forty
@pytest.mark.parametrize("patch", [16, 32])
def test_bf16_frames_by_tile(patch):
    import torch

    cfg = synth.Config("bf16", 40, 13 * patch, 17 * patch, (patch,), 256, 8, 1, 256, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 23)
    images = synth.bf16_round(np.random.default_rng(10).random((40, 3, cfg.H, cfg.W), dtype=np.float32))
    few = _embed(synth.replace(cfg, B=1), w, images[:1])
    ref = np.asarray(O.coarse_encode(images[:1], cfg.patch, w, cfg.heads)[0]).reshape(-1, cfg.d)
    assert float(np.abs(few[0].cpu().numpy() - ref).max() / np.abs(ref).max()) <= 2.0 ** -8
    for n in (4, 8, 16, 40):
        x = _embed(synth.replace(cfg, B=n), w, images[:n])
        assert torch.equal(x[0], few[0]) and torch.isfinite(x).all(), n


# Levels in between each other: a tile of 64 tokens holds some of its level, none, or nothing else.  Room for 20,480 tokens
# sends both levels to gemm_bf16_patch_kernel (more 64 x 64 tiles than CUs), a context of its own a frame to the small tiles.
@pytest.mark.parametrize("fractions", [(0.0, 1.0, 0.3), (0.05, 0.6, 0.0)])
def test_levels_in_one_tile(fractions):
    import torch
    from paper_2505_23317_amd import cfdetr as K

    cfg = synth.Config("levels", 3, 32 * 13, 32 * 17, (32, 16), 256, 8, 1, 256, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 29)
    images = synth.bf16_round(np.random.default_rng(11).random((3, 3, cfg.H, cfg.W), dtype=np.float32))
    tok = []
    for f, part in enumerate(fractions):   # cells picked at random, each one token or its four children
        fine = np.random.default_rng(40 + f).random((13, 17)) < part
        tok.append([t for r in range(13) for c in range(17) for t in
                    ([(1, 2 * r + i, 2 * c + j) for i in (0, 1) for j in (0, 1)] if fine[r, c] else [(0, r, c)])])
    cu = np.concatenate([[0], np.cumsum([len(t) for t in tok])]).astype(np.int32)

    def fine_pass(first, frames, room):
        sub = synth.replace(cfg, B=frames)
        enc = K.Encoder(sub, w, max_tokens_total=room)
        desc = torch.from_numpy(O.pack_tok_desc(np.asarray(sum(tok[first:first + frames], [])))).cuda()
        offs = torch.from_numpy(cu[first:first + frames + 1] - cu[first]).cuda()
        y = torch.empty((int(offs[-1]), cfg.d), device="cuda")
        full = torch.full((room, cfg.d), float("nan"), device="cuda")
        enc.fine_encode(enc.upload_images(images[first:first + frames]), frames, desc, offs, None, full)
        enc.sync_status()
        y.copy_(full[:y.shape[0]])
        enc.close()
        return y

    many = fine_pass(0, 3, 20480)
    assert torch.isfinite(many).all()
    for f in range(3):
        assert torch.equal(fine_pass(f, 1, 884), many[cu[f]:cu[f + 1]]), f
    ref = np.asarray(O.fine_encode(images, np.asarray(sum(tok, [])), cu, cfg.patch, w, cfg.heads))
    assert float(np.abs(many.cpu().numpy() - ref).max() / np.abs(ref).max()) <= 2e-2
