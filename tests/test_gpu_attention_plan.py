"""The attention's work list cuts the items of the sequences of as many tiles into eight runs, one for each XCD, and
deals what does not divide by eight in turn: with 1, 3 or 4 heads and one to three items a head all
remainders occur, with fewer items than XCDs and with more.  64 frames are 128 sequences, two wavefronts
of them.  Queues of 32 entries and fewer, and of more, whose first 32 are turned round.  An item that were missing or done for another sequence would show in its frame's rows: every
frame has the same bits as alone."""
import numpy as np
import pytest

from paper_2505_23317_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames, d, heads", [(64, 64, 1), (64, 128, 4), (5, 192, 3), (33, 192, 3)])
def test_every_item_of_mixed_lengths(frames, d, heads):
    import torch
    from paper_2505_23317_amd import cfdetr as K

    cfg = synth.Config("plan", frames, 128, 192, (16, 8), d, heads, 2, 128, "bf16", box_rule="poisson")
    w = synth.make_weights(cfg, 4)
    rng = np.random.default_rng(frames + d)
    images = synth.bf16_round(rng.normal(0.5, 0.25, (frames, 3, cfg.H, cfg.W)).astype(np.float32))
    # frame f: a box of f % 13 columns of coarse cells, so 96 to 384 tokens
    boxes = [[0, 0, 16 * (f % 13), 128] for f in range(frames)]
    enc, one = K.Encoder(cfg, w), K.Encoder(synth.replace(cfg, B=1), w)
    b, t, o = enc.upload_boxes(boxes, [1] * frames, np.arange(frames + 1))
    out, o1 = enc.alloc_outputs(frames), one.alloc_outputs(1)
    img = enc.upload_images(images)
    enc.multilevel_batch(img, frames, b, t, o, out)
    enc.sync_status()
    cu = out["cu_seqlens"].tolist()
    assert [cu[f + 1] - cu[f] for f in range(frames)] == [96 + 24 * (f % 13) for f in range(frames)]
    for f in range(frames):
        one.multilevel_batch(img[f:f + 1], 1, b[f:f + 1], t[f:f + 1], o[:2], o1)
        n = cu[f + 1] - cu[f]
        assert torch.equal(o1["y_mixed"][:n], out["y_mixed"][cu[f]:cu[f + 1]]), f
        assert torch.equal(o1["y_coarse"], out["y_coarse"][96 * f:96 * (f + 1)]), f
    one.sync_status()
    assert torch.isfinite(out["y_mixed"][:cu[-1]]).all()
    enc.close()
    one.close()
