"""The kernels for few rows (widths 384 and 768, encoder and decoder): a frame's result is the same
bit for bit whether it is encoded or decoded alone, where they run, or in a batch large enough for
the others; at row counts around the edges of their tiles of 32 and 64 rows.  Alone the result is
also held against the oracle."""
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


# cells of a frame, frames of the batch: 384 leaves the kernels behind 3,840 rows, or has no layer kernel (hidden widths past
# 2,048) and leaves them behind some 1,500 (first feed-forward matrix) to 2,700 rows, 768 behind 320 to 2,700 rows
@pytest.mark.parametrize("d, heads, ffn, cells, frames", [
    (384, 6, 1536, (1, 31), 60), (384, 6, 768, (5, 13), 40), (384, 6, 384, (29, 31), 3),
    (768, 12, 3072, (3, 11), 60), (768, 12, 1536, (5, 13), 64), (768, 12, 3072, (29, 31), 8),
    (384, 6, 768, (5, 13), 64), (384, 6, 1536, (29, 31), 5), (768, 12, 3072, (5, 13), 11), (768, 12, 3072, (5, 13), 40),
    (384, 6, 2304, (3, 11), 64), (384, 6, 2304, (5, 13), 64), (384, 6, 2688, (29, 31), 4), (384, 6, 2688, (19, 37), 8)])
def test_encoder_alone_and_in_a_batch(d, heads, ffn, cells, frames):
    import torch

    cfg = synth.Config("few", frames, 8 * cells[0], 8 * cells[1], (8,), d, heads, 2, ffn, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 11)
    rng = np.random.default_rng(3)
    images = synth.bf16_round(rng.normal(0.5, 0.25, (frames, 3, cfg.H, cfg.W)).astype(np.float32))
    many = _coarse(cfg, w, images)
    for f in (0, frames - 1):
        one = _coarse(synth.replace(cfg, B=1), w, images[f:f + 1])[0]
        assert torch.isfinite(one).all()
        assert torch.equal(one, many[f]), f
    ref = np.asarray(O.coarse_encode(images[f:f + 1], cfg.patch, w, cfg.heads)[-1]).reshape(-1, d)
    err = float(np.abs(one.cpu().numpy() - ref).max() / np.abs(ref).max())
    print("few rows against the oracle:", err, flush=True)
    assert err <= BAR


# (the last: 64 frames take the attention's items of 256 queries, one frame those of 128)
@pytest.mark.parametrize("d, heads, ffn, queries",
                         [(384, 6, 1536, 1), (384, 6, 384, 65), (768, 12, 1536, 97), (768, 12, 1536, 155), (384, 6, 2304, 97),
                          (384, 6, 2688, 703)])
def test_decoder_alone_and_in_a_batch(d, heads, ffn, queries):
    import torch
    from paper_2505_23317_amd import cfdetr as K

    frames = 64
    cfg = synth.Config("few_dec", frames, 256, 256, (32, 16), d, heads, 1, ffn, "bf16", box_rule="poisson",
                       box_lambda=2.0, side_lo=8, side_hi=40)
    enc = K.Encoder(cfg, synth.make_weights(cfg, 7))
    enc.attach_decoder(synth.make_decoder_weights(cfg, 3, n_queries=queries, layers=2))
    tokens = 37
    gen = torch.Generator().manual_seed(5)
    mem = torch.randn((frames * tokens, d), generator=gen).cuda()
    cu = torch.arange(frames + 1, dtype=torch.int32).cuda() * tokens
    many = torch.empty((frames, queries, 5), device="cuda")
    enc.decode(mem, cu, frames, many)
    one = torch.empty((1, queries, 5), device="cuda")
    for f in (0, frames - 1):
        enc.decode(mem[f * tokens:(f + 1) * tokens].clone(), cu[:2].clone(), 1, one)
        enc.sync_status()
        assert torch.isfinite(one).all()
        assert torch.equal(one[0], many[f]), f
    enc.close()


# Attention to tokens of several tiles of 64 keys, the last one ragged, by items of 256 queries (64 frames) and of 128
@pytest.mark.parametrize("d, heads, queries, tokens", [(768, 12, 155, 411), (256, 4, 449, 330)])
def test_decoder_over_several_key_tiles(d, heads, queries, tokens):
    import torch
    from paper_2505_23317_amd import cfdetr as K

    frames = 64
    cfg = synth.Config("few_dec", frames, 352, 352, (32, 16), d, heads, 1, 512, "bf16", box_rule="poisson",
                       box_lambda=2.0, side_lo=8, side_hi=40)
    assert frames * queries * heads > 3500 * 32 >= queries * heads
    enc = K.Encoder(cfg, synth.make_weights(cfg, 7))
    dw = synth.make_decoder_weights(cfg, 3, n_queries=queries, layers=1)
    for k in ("w_cls", "w_box3"):   # logits of a few units
        dw[k] = synth.bf16_round((dw[k] * (4.0 / np.sqrt(d))).astype(np.float32))
    for k in ("w_box1", "w_box2"):
        dw[k] = synth.bf16_round((dw[k] * np.sqrt(256.0 / d)).astype(np.float32))
    enc.attach_decoder(dw)
    mem = torch.randn((frames * tokens, d), generator=torch.Generator().manual_seed(5)).cuda()
    cu = torch.arange(frames + 1, dtype=torch.int32).cuda() * tokens
    many = torch.empty((frames, queries, 5), device="cuda")
    enc.decode(mem, cu, frames, many)
    one = torch.empty((1, queries, 5), device="cuda")
    for f in (0, frames - 1):
        enc.decode(mem[f * tokens:(f + 1) * tokens].clone(), cu[:2].clone(), 1, one)
        enc.sync_status()
        assert torch.isfinite(one).all()
        assert torch.equal(one[0], many[f]), f
    enc.close()
    ref = np.asarray(O.decode(mem[-tokens:].cpu().numpy(), np.array([0, tokens], np.int32), dw, heads))
    assert float(np.abs(one.cpu().numpy() - ref.reshape(1, queries, 5)).max() / np.abs(ref).max()) <= BAR
