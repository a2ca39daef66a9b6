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


def _mixed_model(frames, heads, seed):
    """Frames whose patches have one of eight colours (s, z, w), |s, z, w| = 1, that the embedding lays
    along three directions, and weights with q = s and k = z: the base-2 logit of query i for key j is
    600 s_i z_j.  z is -0.3 or -0.8.  s = +-0.02 keeps the sums in range (logits up to 10); s = 0.55 takes
    all logits below -90 and s = -0.55 the largest to 260, so those queries are computed again; which key
    group wins goes by the sign of s.  Of the blocks of 32 queries one in three has some such lanes, every
    ninth a single one, the others none; a wavefront of 64 queries has two blocks."""
    cfg = synth.Config("mixed", frames, 232, 248, (8,), 128, heads, 1, 128, "bf16", box_rule="poisson")
    rng = np.random.default_rng(seed)
    n, d, dh = cfg.n_cells(0), cfg.d, cfg.d_head
    i = np.arange(n)
    again = ((i // 32) % 3 == 0) & (rng.random(n) < 0.4)
    again[(i // 32) % 9 == 6] = False
    again[i[(i // 32) % 9 == 6][17::32]] = True
    s = np.where(again, 0.55, 0.02) * rng.choice([-1.0, 1.0], n)
    z = rng.choice([-0.3, -0.8], n)
    colour = np.stack([s, z, np.sqrt(1.0 - s * s - z * z)])
    patches = colour.reshape(3, *cfg.grid(0))
    images = np.broadcast_to(np.kron(patches, np.ones((1, 8, 8))), (frames, 3, cfg.H, cfg.W))
    w = {k: np.zeros_like(v) for k, v in synth.make_weights(cfg, seed).items()}
    for k in ("ln1_g", "ln2_g", "lnf_g"):
        w[k] += 1.0
    r = np.linalg.qr(np.concatenate([np.ones((d, 1)), rng.standard_normal((d, 3))], 1))[0][:, 1:]
    scale = 1000.0 * np.sqrt(d)     # the position's share of a token: a thousandth
    w["w_embed0"] = synth.bf16_round(np.repeat(scale / 64.0 * r, 64, axis=1).astype(np.float32))
    # LayerNorm makes a token sqrt(d) (s, z, w) along the directions
    beta = np.sqrt(600.0 / (d * 1.4426950408889634 * np.sqrt(dh)))
    w["w_qkv"][0, :d] = synth.bf16_round(np.tile(beta * r[:, 0], (d, 1)).astype(np.float32))
    w["w_qkv"][0, d:2 * d] = synth.bf16_round(np.tile(beta * r[:, 1], (d, 1)).astype(np.float32))
    w["w_qkv"][0, 2 * d:] = synth.bf16_round((rng.standard_normal((d, d)) / np.sqrt(d)).astype(np.float32))
    w["w_o"][0] = synth.bf16_round((1000.0 * rng.standard_normal((d, d)) / np.sqrt(d)).astype(np.float32))
    return cfg, w, synth.bf16_round(images.astype(np.float32)), again


@pytest.mark.parametrize("heads, frames", [(2, 1), (4, 1), (2, FRAMES)])
def test_some_lanes_of_a_wavefront_are_computed_again(heads, frames):
    import torch
    from paper_2505_23317_amd import cfdetr as K

    cfg, w, images, again = _mixed_model(frames, heads, 17)
    assert 0.05 < again.mean() < 0.3 and (again.reshape(-1)[:896].reshape(-1, 32).sum(1) == 1).any()
    # the sums the kernel would have, from the oracle's own numbers
    x = O.embed_frame(images[0], np.asarray([(0, r, c) for r in range(29) for c in range(31)]), cfg.patch, w)
    qkv = O.layer_norm(x, w["ln1_g"][0], w["ln1_b"][0]) @ w["w_qkv"][0].astype(np.float64).T
    dh, d = cfg.d_head, cfg.d
    logits = 1.4426950408889634 / np.sqrt(dh) * (qkv[:, :dh] @ qkv[:, d:d + dh].T)
    top = logits.max(axis=1) + np.log2((logits > logits.max(axis=1, keepdims=True) - 30.0).sum(axis=1))
    assert ((np.abs(top) > 80.0) == again).all() and (top[again] < -64.0).any() and (top[again] > 100.0).any()
    ref = np.asarray(O.coarse_encode(images[:1], cfg.patch, w, cfg.heads)[-1]).reshape(-1, d)

    enc = K.Encoder(cfg, w)
    out = enc.alloc_outputs(frames)
    enc.coarse_encode(enc.upload_images(images), frames, out["x0_cache"], out["y_coarse"])
    enc.sync_status()
    y = out["y_coarse"].reshape(frames, -1, d)
    got = y[0].cpu().numpy()
    # the result tells the two groups of keys apart
    plus = ref[(~again)][0]
    assert np.abs(ref - plus).max() / np.abs(ref).max() > 10 * BAR
    err = np.abs(got - ref).max(axis=1) / np.abs(ref).max()
    print(f"lanes computed again, {heads} heads, {frames} frames: {err[again].max():.2e}, the others {err[~again].max():.2e}",
          flush=True)
    assert err.max() <= BAR
    for f in range(1, frames):
        assert torch.equal(y[f], y[0]), f
    enc.close()
