"""The contraction with packed weights (64, 96 or 128 rows by 256 columns a tile): a frame's tokens are
the same bit for bit alone, where the kernels for few rows run, and in a batch, whose rows end inside, one
before and one behind a tile, in workgroups with one tile and with several.  The last frame is also
held against the oracle: two layers of bf16 products, the bar of the kernels for few rows."""
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


# 705 rows = 11 x 64 + 1, 2,686 = 28 x 96 - 2 = 42 x 64 - 2, 4,609 = 36 x 128 + 1 = 48 x 96 + 1 = 72 x 64 + 1; 12,276 and
# 17,081 with several tiles a workgroup and a last one that is partly empty
@pytest.mark.parametrize("ffn, cells, frames", [
    (3072, (3, 47), 5), (3072, (17, 79), 2), (1536, (1, 419), 11), (3072, (31, 33), 12), (768, (29, 31), 19)])
def test_rows_alone_and_in_a_batch(ffn, cells, frames):
    import torch

    d = 768
    cfg = synth.Config("packed", frames, 8 * cells[0], 8 * cells[1], (8,), d, 12, 2, ffn, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 11)
    rng = np.random.default_rng(3)
    images = synth.bf16_round(rng.normal(0.5, 0.25, (frames, 3, cfg.H, cfg.W)).astype(np.float32))
    many = _coarse(cfg, w, images)
    assert torch.isfinite(many).all()
    for f in (0, frames - 1):
        one = _coarse(synth.replace(cfg, B=1), w, images[f:f + 1])[0]
        assert torch.equal(one, many[f]), f
    ref = np.asarray(O.coarse_encode(images[f:f + 1], cfg.patch, w, cfg.heads)[-1]).reshape(-1, d)
    err = float(np.abs(one.cpu().numpy() - ref).max() / np.abs(ref).max())
    print("packed tiles against the oracle:", err, flush=True)
    assert err <= BAR
