"""The LayerNorm launches of widths without a layer kernel are wavefronts for 8,192 rows on 256 CUs, and a wavefront goes on
to further ones: a frame's rows have the same bits alone (one row a wavefront at most) and among 8,150 to 24,650 rows, at the
first and the last row of one, two and three turns."""
import numpy as np
import pytest

from paper_2505_23317_amd import synth

pytestmark = pytest.mark.gpu


# 48, 192 and 256 groups of four columns for 64 lanes; frames of 163, 132 and 493 cells: 8,150 and 8,313 rows, 8,316, 24,650
@pytest.mark.parametrize("d, heads, cells, batches", [(192, 3, (1, 163), (50, 51)), (768, 12, (4, 33), (63,)),
                                                      (1024, 16, (17, 29), (50,))])
def test_rows_of_all_turns(d, heads, cells, batches):
    import torch
    from paper_2505_23317_amd import cfdetr as K

    frames = max(batches)
    cfg = synth.Config("norm", frames, 8 * cells[0], 8 * cells[1], (8,), d, heads, 1, 128, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 5)
    images = synth.bf16_round(np.random.default_rng(d).normal(0.5, 0.25, (frames, 3, cfg.H, cfg.W)).astype(np.float32))
    many, one = K.Encoder(cfg, w), K.Encoder(synth.replace(cfg, B=1), w)
    img, out, o1 = many.upload_images(images), many.alloc_outputs(frames), one.alloc_outputs(1)
    n = cells[0] * cells[1]
    for b in batches:
        many.coarse_encode(img, b, out["x0_cache"], out["y_coarse"])
        many.sync_status()
        assert torch.isfinite(out["y_coarse"][:b * n]).all()
        for f in (0, b // 3, 2 * b // 3, b - 1):
            one.coarse_encode(img[f:f + 1], 1, o1["x0_cache"], o1["y_coarse"])
            assert torch.equal(o1["y_coarse"], out["y_coarse"][f * n:(f + 1) * n]), (b, f)
    one.sync_status()
    many.close()
    one.close()
