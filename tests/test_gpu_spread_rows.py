"""Width 384: layers spread over the chip (up to 15 rows a CU, 3,840 rows on 256 CUs; workgroups of 32 rows, then of 64
in the second feed-forward matrix) and one kernel a layer beyond give a frame the same bits.  Decoders of
widths 256 and 384 on the same kernels: a frame's queries alone and in a batch."""
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


# one frame: 32 rows, 899, 1,279; then rows in the range of 64 a workgroup, the last spread count and the first fused one
@pytest.mark.parametrize("ffn, cells, batches", [
    (1536, (4, 8), (2, 60)), (1536, (29, 31), (3, 4, 5)), (768, (1, 1279), (2, 3, 4)), (384, (1, 1280), (3, 4))])
def test_spread_and_fused_layers(ffn, cells, batches):
    import torch

    frames = max(batches)
    cfg = synth.Config("spread", frames, 8 * cells[0], 8 * cells[1], (8,), 384, 6, 2, ffn, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 31)
    images = synth.bf16_round(np.random.default_rng(8).normal(0.5, 0.25, (frames, 3, cfg.H, cfg.W)).astype(np.float32))
    one = _coarse(synth.replace(cfg, B=1), w, images[:1])[0]
    ref = np.asarray(O.coarse_encode(images[:1], cfg.patch, w, cfg.heads)[-1]).reshape(-1, cfg.d)
    assert float(np.abs(one.cpu().numpy() - ref).max() / np.abs(ref).max()) <= BAR
    for n in batches:
        many = _coarse(synth.replace(cfg, B=n), w, images[:n])
        assert torch.isfinite(many).all() and torch.equal(many[0], one), n


# 64 frames x 33, 97, 65 and 129 queries: one tile of 32 rows and a row up to some 8,000 rows
@pytest.mark.parametrize("d, heads, ffn, queries",
                         [(256, 8, 256, 33), (256, 8, 1024, 97), (384, 6, 640, 65), (384, 6, 1536, 129)])
def test_decoders_alone_and_in_a_batch(d, heads, ffn, queries):
    import torch
    from paper_2505_23317_amd import cfdetr as K

    frames, tokens = 64, 37
    cfg = synth.Config("spread_dec", frames, 256, 256, (32, 16), d, heads, 1, ffn, "bf16", box_rule="poisson",
                       box_lambda=2.0, side_lo=8, side_hi=40)
    enc = K.Encoder(cfg, synth.make_weights(cfg, 7))
    dw = synth.make_decoder_weights(cfg, 3, n_queries=queries, layers=2)
    for k in ("w_cls", "w_box3"):   # logits of a few units: the logistic values are not all 0 and 1
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
    ref = np.asarray(O.decode(mem[-tokens:].cpu().numpy(), np.array([0, tokens], np.int32), dw, heads))
    err = float(np.abs(one.cpu().numpy() - ref.reshape(1, queries, 5)).max() / np.abs(ref).max())
    print("decoder against the oracle:", err, flush=True)
    assert err <= BAR
    enc.close()


# weights asked for during attention (up to 16 rows a CU: 4,096 rows on 256 CUs): spread (2 x 1,024), the fused form
# (4 x 1,024, the last count) and without (5 x 1,024), for both head widths
@pytest.mark.parametrize("heads, ffn", [(6, 384), (12, 768)])
def test_weights_asked_for_during_attention(heads, ffn):
    import torch

    cfg = synth.Config("ahead", 5, 8 * 32, 8 * 32, (8,), 384, heads, 3, ffn, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 17)
    images = synth.bf16_round(np.random.default_rng(9).normal(0.5, 0.25, (5, 3, cfg.H, cfg.W)).astype(np.float32))
    many = _coarse(cfg, w, images)
    ref = np.asarray(O.coarse_encode(images[:1], cfg.patch, w, cfg.heads)[-1]).reshape(-1, cfg.d)
    assert float(np.abs(many[0].cpu().numpy() - ref).max() / np.abs(ref).max()) <= BAR
    for n in (2, 4):
        few = _coarse(synth.replace(cfg, B=n), w, images[:n])
        assert torch.equal(few, many[:n]), n
