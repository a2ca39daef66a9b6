"""GPU parity: the HIP library (through its C ABI) against the fp64 CPU oracle.

Bars: token tables, offsets and counts bit-exact; activations within
max|gpu - ref| / max|ref| <= 2e-2 with bf16 contractions and <= 1e-4 in the
all-fp32 check mode.
"""
import os
import sys

import numpy as np
import pytest

from oracle import cfdetr_oracle as O
from paper_2505_23317_amd import synth

pytestmark = pytest.mark.gpu

TOL = {"bf16": 2e-2, "fp32": 1e-4}
GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden")


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def rel_err(g, r):
    """The bar's metric: largest absolute deviation over the largest reference magnitude."""
    return float(np.abs(np.asarray(g, np.float64) - r).max() / np.abs(r).max())


def rms_err(g, r):
    """Root-mean-square deviation over the root-mean-square of the reference (reported beside
    the bar's metric: it cannot be satisfied by a few large reference values)."""
    g, r = np.asarray(g, np.float64), np.asarray(r, np.float64)
    return float(np.sqrt(((g - r) ** 2).mean() / (r ** 2).mean()))


@pytest.fixture(scope="module")
def K():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2505_23317_amd import cfdetr
    cfdetr.load_library()
    return cfdetr


def gpu_multilevel(K, cfg, wl, act, max_tokens=None):
    import torch
    enc = K.Encoder(cfg, wl["weights"], act_dtype=act, max_tokens_total=max_tokens)
    img = enc.upload_images(wl["images"])
    b, t, o = enc.upload_boxes(wl["boxes"], wl["tier"], wl["box_offsets"])
    out = enc.alloc_outputs(cfg.B)
    enc.multilevel_batch(img, cfg.B, b, t, o, out)
    enc.sync_status()
    torch.cuda.synchronize()
    res = {k: v.cpu().numpy() for k, v in out.items()}
    enc.close()
    return res


def oracle_multilevel(cfg, wl):
    yc, ym, tok, cu, counts = O.multilevel_batch(wl["images"], wl["boxes"], wl["tier"],
                                                 wl["box_offsets"], cfg.patch, wl["weights"],
                                                 cfg.heads)
    return {"y_coarse": yc, "y_mixed": ym, "tok_desc": O.pack_tok_desc(tok),
            "cu_seqlens": cu, "level_counts": counts}


def check_all(got, ref, act, label):
    T = int(ref["cu_seqlens"][-1])
    np.testing.assert_array_equal(got["cu_seqlens"], ref["cu_seqlens"])
    np.testing.assert_array_equal(got["level_counts"], ref["level_counts"])
    np.testing.assert_array_equal(got["tok_desc"][:T], ref["tok_desc"])
    ec = rel_err(got["y_coarse"], ref["y_coarse"])
    em = rel_err(got["y_mixed"][:T], ref["y_mixed"])
    _say(f"[parity] {label} {act}: T={T} coarse {ec:.2e} mixed {em:.2e} (bar {TOL[act]:.0e}); "
         f"rms-relative coarse {rms_err(got['y_coarse'], ref['y_coarse']):.2e} "
         f"mixed {rms_err(got['y_mixed'][:T], ref['y_mixed']):.2e}")
    assert np.isfinite(got["y_mixed"][:T]).all()
    assert ec <= TOL[act], (label, act, ec)
    assert em <= TOL[act], (label, act, em)
    # rows past the token total stay as the caller left them (zero-filled here)
    assert not got["y_mixed"][T:].any()


# ------------------------------------------------------------------ selection
@pytest.mark.parametrize("cfg_id", [1, 2, 3, 4, 5])
def test_selection_is_bit_exact_on_every_config(K, cfg_id):
    import torch
    cfg = synth.config(cfg_id)
    _say(f"[case] selection cfg{cfg_id}")
    images, boxes, tier, offs, _ = synth.make_frames(synth.replace(cfg, H=cfg.H, W=cfg.W), cfg_id)
    w = synth.make_weights(synth.replace(cfg, layers=1), 1)
    enc = K.Encoder(synth.replace(cfg, layers=1), w)
    b, t, o = enc.upload_boxes(boxes, tier, offs)
    out = enc.alloc_outputs(cfg.B)
    enc.select_fine(b, t, o, cfg.B, out["tok_desc"], out["cu_seqlens"], out["level_counts"])
    enc.sync_status()
    tok, cu, counts = O.select_fine(boxes, tier, offs, cfg.B, cfg.H, cfg.W, cfg.patch)
    T = int(cu[-1])
    np.testing.assert_array_equal(out["cu_seqlens"].cpu().numpy(), cu)
    np.testing.assert_array_equal(out["level_counts"].cpu().numpy(), counts)
    np.testing.assert_array_equal(out["tok_desc"].cpu().numpy()[:T], O.pack_tok_desc(tok))
    # a second call on the same context starts from clean counters
    enc.select_fine(b, t, o, cfg.B, out["tok_desc"], out["cu_seqlens"], None)
    enc.sync_status()
    np.testing.assert_array_equal(out["cu_seqlens"].cpu().numpy(), cu)
    enc.close()


def test_selection_edge_cases(K):
    cfg = synth.Config("edge", 4, 128, 192, (64, 32, 16), 64, 2, 1, 128, "f32")
    w = synth.make_weights(cfg, 2)
    enc = K.Encoder(cfg, w)
    # frame 0: no box; 1: everything at finest; 2: clipped / empty / outside boxes and
    # a mid-tier box; 3: tier above the finest level acts as finest
    boxes = np.asarray([[0, 0, 192, 128],
                        [-50, -50, 1, 1], [40, 40, 40, 90], [500, 0, 600, 50], [100, 70, 130, 100],
                        [191, 127, 4000, 4000],
                        [10, 10, 20, 20]], np.int32)
    tier = np.asarray([2, 2, 2, 2, 1, 2, 9], np.uint8)
    offs = np.asarray([0, 0, 1, 6, 7], np.int32)
    b, t, o = enc.upload_boxes(boxes, tier, offs)
    out = enc.alloc_outputs(cfg.B)
    enc.select_fine(b, t, o, cfg.B, out["tok_desc"], out["cu_seqlens"], out["level_counts"])
    enc.sync_status()
    tok, cu, counts = O.select_fine(boxes, np.minimum(tier, 2), offs, cfg.B, cfg.H, cfg.W, cfg.patch)
    np.testing.assert_array_equal(out["cu_seqlens"].cpu().numpy(), cu)
    np.testing.assert_array_equal(out["level_counts"].cpu().numpy(), counts)
    np.testing.assert_array_equal(out["tok_desc"].cpu().numpy()[:cu[-1]], O.pack_tok_desc(tok))
    assert counts[0].tolist() == [6, 0, 0] and counts[1].tolist() == [0, 0, 96]
    enc.close()


# frames, most boxes of a frame: the lanes that share a box go from eight to one with the number of
# boxes to a thread's share (1024 threads over the frames), which these pass on both sides of
@pytest.mark.parametrize("frames, most", [(1, 600), (5, 100), (12, 130), (33, 45), (64, 20), (64, 37), (64, 300)])
def test_selection_of_many_boxes(K, frames, most):
    cfg = synth.Config("many", frames, 256, 320, (32, 16, 8), 64, 2, 1, 128, "f32")
    rng = np.random.default_rng(most)
    boxes, tier, offs = [], [], [0]
    for f in range(frames):
        n = 0 if f == 3 else most if f == frames // 2 else int(rng.integers(0, most + 1))
        # most boxes are a few pixels, so that cells stay whole; some are wide, outside, or empty
        side = rng.choice([1, 6, 12, 200], n, p=[0.6, 0.3, 0.09, 0.01])
        x0, y0 = rng.integers(-20, cfg.W + 20, n), rng.integers(-20, cfg.H + 20, n)
        boxes.append(np.stack([x0, y0, x0 + rng.integers(0, side + 1), y0 + rng.integers(0, side + 1)], 1))
        tier.append(rng.choice([0, 1, 2, 7], n, p=[0.3, 0.4, 0.2, 0.1]))
        offs.append(offs[-1] + n)
    boxes = np.concatenate(boxes).astype(np.int32).reshape(-1, 4)
    tier, offs = np.concatenate(tier).astype(np.uint8), np.asarray(offs, np.int32)
    _say(f"[case] selection of {offs[-1]} boxes in {frames} frames")
    enc = K.Encoder(cfg, synth.make_weights(cfg, 4))
    b, t, o = enc.upload_boxes(boxes, tier, offs)
    out = enc.alloc_outputs(frames)
    tok, cu, counts = O.select_fine(boxes, np.minimum(tier, 2), offs, frames, cfg.H, cfg.W, cfg.patch)
    assert (counts.sum(axis=0) > 0).all()
    for _ in range(2):
        enc.select_fine(b, t, o, frames, out["tok_desc"], out["cu_seqlens"], out["level_counts"])
        enc.sync_status()
        np.testing.assert_array_equal(out["cu_seqlens"].cpu().numpy(), cu)
        np.testing.assert_array_equal(out["level_counts"].cpu().numpy(), counts)
        np.testing.assert_array_equal(out["tok_desc"].cpu().numpy()[:cu[-1]], O.pack_tok_desc(tok))
    enc.close()


# one frame has nearly all boxes: its own threads paint them, with as few lanes a box as its own number asks for
@pytest.mark.parametrize("frames, most", [(12, 200), (33, 513), (64, 512)])
def test_selection_with_one_full_frame(K, frames, most):
    cfg = synth.Config("full", frames, 256, 320, (32, 16, 8), 64, 2, 1, 128, "f32")
    rng = np.random.default_rng(most)
    boxes, tier, offs = [], [], [0]
    for f in range(frames):
        n = most if f == frames - 2 else f % 3
        side = rng.choice([1, 6, 12], n, p=[0.6, 0.3, 0.1])
        x0, y0 = rng.integers(0, cfg.W, n), rng.integers(0, cfg.H, n)
        boxes.append(np.stack([x0, y0, x0 + rng.integers(0, side + 1), y0 + rng.integers(0, side + 1)], 1))
        tier.append(rng.choice([0, 1, 2], n, p=[0.3, 0.5, 0.2]))
        offs.append(offs[-1] + n)
    boxes = np.concatenate(boxes).astype(np.int32).reshape(-1, 4)
    tier, offs = np.concatenate(tier).astype(np.uint8), np.asarray(offs, np.int32)
    _say(f"[case] selection, {most} of {offs[-1]} boxes in one of {frames} frames")
    enc = K.Encoder(cfg, synth.make_weights(cfg, 4))
    b, t, o = enc.upload_boxes(boxes, tier, offs)
    out = enc.alloc_outputs(frames)
    tok, cu, counts = O.select_fine(boxes, tier, offs, frames, cfg.H, cfg.W, cfg.patch)
    enc.select_fine(b, t, o, frames, out["tok_desc"], out["cu_seqlens"], out["level_counts"])
    enc.sync_status()
    np.testing.assert_array_equal(out["cu_seqlens"].cpu().numpy(), cu)
    np.testing.assert_array_equal(out["level_counts"].cpu().numpy(), counts)
    np.testing.assert_array_equal(out["tok_desc"].cpu().numpy()[:cu[-1]], O.pack_tok_desc(tok))
    enc.close()


def test_selection_with_changing_batch_size_on_one_context(K):
    # flags raised by a call with many frames must not leak into later, smaller or larger calls
    cfg = synth.Config("varb", 4, 128, 128, (64, 32, 16), 64, 2, 1, 128, "f32")
    enc = K.Encoder(cfg, synth.make_weights(cfg, 4))
    rng = np.random.default_rng(5)
    for B in (4, 2, 4, 1, 3, 4):
        boxes, tier, offs = [], [], [0]
        for _ in range(B):
            for _ in range(int(rng.integers(0, 4))):
                x0, y0 = int(rng.integers(0, 100)), int(rng.integers(0, 100))
                boxes.append((x0, y0, x0 + int(rng.integers(1, 60)), y0 + int(rng.integers(1, 60))))
                tier.append(int(rng.integers(0, 3)))
            offs.append(len(boxes))
        boxes = np.asarray(boxes, np.int32).reshape(-1, 4)
        tier, offs = np.asarray(tier, np.uint8), np.asarray(offs, np.int32)
        b, t, o = enc.upload_boxes(boxes, tier, offs)
        out = enc.alloc_outputs(B)
        enc.select_fine(b, t, o, B, out["tok_desc"], out["cu_seqlens"], out["level_counts"])
        enc.sync_status()
        tok, cu, counts = O.select_fine(boxes, tier, offs, B, cfg.H, cfg.W, cfg.patch)
        np.testing.assert_array_equal(out["cu_seqlens"].cpu().numpy(), cu)
        np.testing.assert_array_equal(out["level_counts"].cpu().numpy(), counts)
        np.testing.assert_array_equal(out["tok_desc"].cpu().numpy()[:cu[-1]], O.pack_tok_desc(tok))
    enc.close()


def test_selection_overflow_is_reported_not_truncated(K):
    cfg = synth.Config("ovf", 2, 128, 128, (32, 16), 64, 2, 1, 128, "f32")
    enc = K.Encoder(cfg, synth.make_weights(cfg, 3), max_tokens_total=40)
    boxes = np.asarray([[0, 0, 128, 128]], np.int32)      # frame 1 alone needs 64 tokens
    b, t, o = enc.upload_boxes(boxes, np.asarray([1], np.uint8), np.asarray([0, 0, 1], np.int32))
    out = enc.alloc_outputs(cfg.B)
    out["tok_desc"].fill_(-7)
    enc.select_fine(b, t, o, cfg.B, out["tok_desc"], out["cu_seqlens"], out["level_counts"])
    with pytest.raises(K.CfdetrError) as ei:
        enc.sync_status()
    assert ei.value.status == K.CFDETR_ECAPACITY
    assert out["cu_seqlens"].cpu().tolist() == [0, 0, 0]
    assert (out["tok_desc"].cpu().numpy() == -7).all()
    enc.sync_status()                                       # flag is cleared once reported
    # the context keeps working afterwards
    b, t, o = enc.upload_boxes(np.zeros((0, 4)), np.zeros(0), np.asarray([0, 0, 0], np.int32))
    enc.select_fine(b, t, o, cfg.B, out["tok_desc"], out["cu_seqlens"], out["level_counts"])
    enc.sync_status()
    assert out["cu_seqlens"].cpu().tolist() == [0, 16, 32]
    enc.close()


def test_host_side_argument_errors(K):
    import torch
    cfg = synth.config(1)
    wl = synth.make_workload(1)
    enc = K.Encoder(cfg, wl["weights"])
    img = enc.upload_images(wl["images"])
    out = enc.alloc_outputs(1)
    with pytest.raises(K.CfdetrError) as ei:
        enc.coarse_encode(img, 2, out["x0_cache"], out["y_coarse"])
    assert ei.value.status == K.CFDETR_ECAPACITY
    with pytest.raises(K.CfdetrError) as ei:
        enc.coarse_encode(img, 0, out["x0_cache"], out["y_coarse"])
    assert ei.value.status == K.CFDETR_EINVAL
    with pytest.raises(K.CfdetrError) as ei:
        K.cfdetr_coarse_encode(enc.ctx, img.data_ptr(), 1, None, out["y_coarse"].data_ptr() + 4, 0)
    assert ei.value.status == K.CFDETR_EINVAL
    with pytest.raises(K.CfdetrError) as ei:
        K.cfdetr_fine_encode(enc.ctx, img.data_ptr(), 1, None, out["cu_seqlens"].data_ptr(), None,
                             out["y_mixed"].data_ptr(), 0)
    assert ei.value.status == K.CFDETR_EINVAL
    assert "null" in K.cfdetr_last_error(enc.ctx)
    assert K.cfdetr_workspace_bytes(enc.ctx) > 0
    enc.close()


# ------------------------------------------------------------------ whole path
@pytest.mark.parametrize("act", ["fp32", "bf16"])
@pytest.mark.parametrize("seed", [1, 2, 5])
def test_cfg1_tiny_frame(K, act, seed):
    cfg = synth.config(1)
    _say(f"[case] cfg1 seed {seed} {act}")
    wl = synth.make_workload(cfg, seed=seed)
    check_all(gpu_multilevel(K, cfg, wl, act), oracle_multilevel(cfg, wl), act, f"cfg1/s{seed}")


@pytest.mark.parametrize("act", ["fp32", "bf16"])
@pytest.mark.parametrize("cfg_id", [2, 3])
def test_cfg2_cfg3_full_size(K, act, cfg_id):
    cfg = synth.config(cfg_id)
    _say(f"[case] cfg{cfg_id} {act}")
    wl = synth.make_workload(cfg_id)
    check_all(gpu_multilevel(K, cfg, wl, act), oracle_multilevel(cfg, wl), act, f"cfg{cfg_id}")


REDUCED = {
    # head width 64, d=384: the shape family of the high-resolution config, ragged lengths
    "cfg4_reduced": synth.Config("cfg4r", 3, 512, 384, (32, 16), 384, 6, 2, 1536, "bf16",
                                 frac_lo=0.0, frac_hi=1.0, box_rule="fraction"),
    # three levels, d=768, 12 heads
    "cfg5_reduced": synth.Config("cfg5r", 3, 256, 384, (64, 32, 16), 768, 12, 2, 3072, "bf16",
                                 box_rule="tiered", box_lambda=3.0, side_lo=16, side_hi=96),
}


LIMITS = {
    # the largest batch the library takes: 64 small frames
    "max_batch": synth.Config("b64", 64, 64, 96, (16, 8), 64, 2, 1, 128, "bf16",
                              box_rule="poisson", box_lambda=2.0, side_lo=8, side_hi=40),
    # the widest model: d = 1024 with 32 heads of 32, one 8x8 patch level pair
    "max_width_32_heads": synth.Config("d1024h32", 2, 64, 64, (16, 8), 1024, 32, 1, 128, "bf16",
                                       box_rule="poisson", box_lambda=2.0, side_lo=8, side_hi=40),
    # heads of 64 at the widest model, single level (no refinement possible)
    "one_level_16_heads": synth.Config("d1024h16", 2, 64, 96, (16,), 1024, 16, 2, 64, "bf16",
                                       box_rule="poisson", box_lambda=2.0, side_lo=8, side_hi=40),
}


@pytest.mark.parametrize("act", ["fp32", "bf16"])
@pytest.mark.parametrize("name", sorted(LIMITS))
def test_limits_of_the_configuration(K, act, name):
    cfg = LIMITS[name]
    _say(f"[case] {name} {act}")
    wl = synth.make_workload(cfg, seed=29)
    check_all(gpu_multilevel(K, cfg, wl, act), oracle_multilevel(cfg, wl), act, name)


# Width 256 in bf16 runs everything of a layer after attention, and the next layer's
# q/k/v projection, in one kernel that walks the hidden width in chunks of 128 (at most
# 2048): its smallest and largest hidden widths, one layer (no projection behind it) and
# several, heads of 64, and row counts that leave the last 32-row workgroup ragged.
TAIL_SHAPES = {
    "one_chunk_one_layer": synth.Config("t128", 2, 128, 160, (32, 16), 256, 8, 1, 128, "bf16",
                                        box_rule="poisson", box_lambda=2.0, side_lo=8, side_hi=60),
    "widest_hidden": synth.Config("t2048", 3, 160, 224, (32, 16), 256, 4, 3, 2048, "bf16",
                                  box_rule="poisson", box_lambda=3.0, side_lo=8, side_hi=60),
    "five_layers": synth.Config("t5", 5, 96, 224, (32, 16), 256, 8, 5, 384, "bf16",
                                box_rule="poisson", box_lambda=2.0, side_lo=8, side_hi=60),
}


@pytest.mark.parametrize("name", sorted(TAIL_SHAPES))
def test_fused_layer_tail_shapes(K, name):
    cfg = TAIL_SHAPES[name]
    _say(f"[case] tail {name}")
    wl = synth.make_workload(cfg, seed=61)
    ref = oracle_multilevel(cfg, wl)
    assert (int(ref["cu_seqlens"][-1]) + cfg.B * cfg.n_cells(0)) % 32 != 0      # ragged last block
    check_all(gpu_multilevel(K, cfg, wl, "bf16"), ref, "bf16", name)
    sharp = synth.make_workload(cfg, seed=62, sharp=True)
    check_all(gpu_multilevel(K, cfg, sharp, "bf16"), oracle_multilevel(cfg, sharp), "bf16",
              name + " sharp")


@pytest.mark.parametrize("act", ["fp32", "bf16"])
@pytest.mark.parametrize("name", sorted(REDUCED))
def test_reduced_large_shapes(K, act, name):
    cfg = REDUCED[name]
    _say(f"[case] {name} {act}")
    wl = synth.make_workload(cfg, seed=17)
    ref = oracle_multilevel(cfg, wl)
    lens = np.diff(ref["cu_seqlens"])
    assert len(set(lens.tolist())) > 1 and (lens % 64 != 0).any()     # ragged tails
    check_all(gpu_multilevel(K, cfg, wl, act), ref, act, name)


@pytest.mark.parametrize("act", ["fp32", "bf16"])
def test_sharp_attention_weights(K, act):
    # random N(0,0.02) weights give nearly uniform attention; this set has logits of a
    # few units so that scale, mask and max-subtraction mistakes would show
    cfg = synth.replace(synth.config(3), B=3, layers=2)
    _say(f"[case] sharp {act}")
    wl = synth.make_workload(cfg, seed=23, sharp=True)
    check_all(gpu_multilevel(K, cfg, wl, act), oracle_multilevel(cfg, wl), act, "sharp")


@pytest.mark.parametrize("act", ["bf16", "fp32"])
@pytest.mark.parametrize("cfg_id", [4, 5])
def test_full_size_against_stored_oracle_rows(K, cfg_id, act):
    """The two largest configurations at full size, in the launch shapes the benchmark times,
    against rows the oracle computed (tests/golden/make_golden.py): one row of every block of
    32 rows of the merged run, both sides of every multiple of 64 rows (every edge of a row
    tile of 64, 128, 192 or 256 rows) and both ends of every sequence."""
    path = os.path.join(GOLDEN, f"cfg{cfg_id}_oracle.npz")
    ref = np.load(path)
    cfg = synth.config(cfg_id)
    _say(f"[case] cfg{cfg_id} full size {act} vs stored oracle rows")
    wl = synth.make_workload(cfg_id)
    got = gpu_multilevel(K, cfg, wl, act)
    T = int(ref["cu_seqlens"][-1])
    np.testing.assert_array_equal(got["cu_seqlens"], ref["cu_seqlens"])
    np.testing.assert_array_equal(got["level_counts"], ref["level_counts"])
    np.testing.assert_array_equal(got["tok_desc"][:T], ref["tok_desc"])
    rc, rm = ref["rows_coarse"], ref["rows_mixed"]
    n_coarse = got["y_coarse"].shape[0]
    merged = np.concatenate([rc, n_coarse + rm])
    assert len(np.unique(merged // 32)) == (n_coarse + T + 31) // 32      # every 32-row block
    edges = np.arange(64, n_coarse + T, 64)
    assert np.isin(edges, merged).all() and np.isin(edges - 1, merged).all()
    dc = got["y_coarse"][rc].astype(np.float64) - ref["y_coarse"]
    dm = got["y_mixed"][rm].astype(np.float64) - ref["y_mixed"]
    ec = np.abs(dc).max() / ref["max_abs_coarse"]
    em = np.abs(dm).max() / ref["max_abs_mixed"]
    rms_c = np.sqrt((dc ** 2).mean() / (ref["y_coarse"].astype(np.float64) ** 2).mean())
    rms_m = np.sqrt((dm ** 2).mean() / (ref["y_mixed"].astype(np.float64) ** 2).mean())
    _say(f"[parity] cfg{cfg_id} full {act}: T={T} rows {len(rc)} + {len(rm)}: coarse {ec:.2e} "
         f"mixed {em:.2e} (bar {TOL[act]:.0e}); rms-relative coarse {rms_c:.2e} mixed {rms_m:.2e}")
    assert np.isfinite(got["y_mixed"][:T]).all() and np.isfinite(got["y_coarse"]).all()
    assert ec <= TOL[act] and em <= TOL[act]


# ------------------------------------------------------------------ invariants on the GPU
def _calls_separately(K, cfg, wl, act, use_cache=True, boxes=None):
    import torch
    enc = K.Encoder(cfg, wl["weights"], act_dtype=act)
    img = enc.upload_images(wl["images"])
    bx = wl if boxes is None else boxes
    b, t, o = enc.upload_boxes(bx["boxes"], bx["tier"], bx["box_offsets"])
    out = enc.alloc_outputs(cfg.B)
    enc.coarse_encode(img, cfg.B, out["x0_cache"], out["y_coarse"])
    enc.select_fine(b, t, o, cfg.B, out["tok_desc"], out["cu_seqlens"], out["level_counts"])
    enc.fine_encode(img, cfg.B, out["tok_desc"], out["cu_seqlens"],
                    out["x0_cache"] if use_cache else None, out["y_mixed"])
    enc.sync_status()
    res = {k: v.cpu().numpy() for k, v in out.items()}
    enc.close()
    return res


@pytest.mark.parametrize("act", ["fp32", "bf16"])
def test_one_call_equals_three_calls_and_cache_equals_recompute(K, act):
    cfg = synth.replace(synth.config(3), B=3, layers=2)
    wl = synth.make_workload(cfg, seed=31)
    one = gpu_multilevel(K, cfg, wl, act)
    three = _calls_separately(K, cfg, wl, act, use_cache=True)
    fresh = _calls_separately(K, cfg, wl, act, use_cache=False)
    T = int(one["cu_seqlens"][-1])
    for k in ("y_coarse", "tok_desc", "cu_seqlens", "level_counts"):
        np.testing.assert_array_equal(one[k], three[k])
    np.testing.assert_array_equal(one["y_mixed"][:T], three["y_mixed"][:T])
    # same kernel, same arithmetic order for a coarse token whether cached or re-embedded
    np.testing.assert_array_equal(three["y_mixed"][:T], fresh["y_mixed"][:T])
    x0_ref, _ = O.coarse_encode(wl["images"], cfg.patch, wl["weights"], cfg.heads)
    assert rel_err(three["x0_cache"], x0_ref) <= TOL[act]


def test_no_roi_gives_the_coarse_result(K):
    cfg = synth.replace(synth.config(3), B=2, layers=2)
    wl = synth.make_workload(cfg, seed=37)
    none = {"boxes": np.zeros((0, 4), np.int32), "tier": np.zeros(0, np.uint8),
            "box_offsets": np.zeros(cfg.B + 1, np.int32)}
    got = _calls_separately(K, cfg, wl, "bf16", boxes=none)
    n0 = cfg.n_cells(0)
    assert got["cu_seqlens"].tolist() == [0, n0, 2 * n0]
    # the mixed pass over coarse-only token sets runs the same kernels on the same rows
    np.testing.assert_array_equal(got["y_mixed"][:2 * n0], got["y_coarse"])


@pytest.mark.parametrize("cfg_id", [3, 4])
def test_batched_equals_frame_by_frame(K, cfg_id):
    """A frame's result does not depend on its batch, bit for bit.  At cfg 4's size the batch
    and the single frames also get different contraction tiles (192 x 128 and 128 x 128 against
    smaller ones), which must not show either."""
    cfg = synth.replace(synth.config(cfg_id), B=3 if cfg_id == 3 else 4, layers=2)
    wl = synth.make_workload(cfg, seed=41, sharp=True)
    _say(f"[case] batched vs frame by frame, {cfg.name} with {cfg.B} frames, 2 layers")
    full = gpu_multilevel(K, cfg, wl, "bf16")
    cu = full["cu_seqlens"]
    n0 = cfg.n_cells(0)
    for i in range(cfg.B):
        lo, hi = wl["box_offsets"][i], wl["box_offsets"][i + 1]
        one_cfg = synth.replace(cfg, B=1)
        one = dict(wl, images=wl["images"][i:i + 1], boxes=wl["boxes"][lo:hi],
                   tier=wl["tier"][lo:hi], box_offsets=np.asarray([0, hi - lo], np.int32))
        got = gpu_multilevel(K, one_cfg, one, "bf16")
        np.testing.assert_array_equal(got["y_mixed"][:cu[i + 1] - cu[i]],
                                      full["y_mixed"][cu[i]:cu[i + 1]])
        np.testing.assert_array_equal(got["y_coarse"], full["y_coarse"][i * n0:(i + 1) * n0])


def test_two_runs_are_bit_identical(K):
    cfg = synth.replace(synth.config(3), layers=2)
    wl = synth.make_workload(cfg, seed=43)
    a = gpu_multilevel(K, cfg, wl, "bf16")
    b = gpu_multilevel(K, cfg, wl, "bf16")
    for k in a:
        np.testing.assert_array_equal(a[k], b[k])


def test_a_second_run_on_one_context_is_bit_identical(K):
    """The contraction kernels choose their tiles from the row count of the context's previous
    run of the same kind (the first run only has the capacity): the choice must not show in the
    results.  cfg5's shape (width 768) with enough rows for the large tile to be in play."""
    import torch
    cfg = synth.replace(synth.config(5), B=8, layers=1)
    wl = synth.make_workload(cfg, seed=44)
    enc = K.Encoder(cfg, wl["weights"], act_dtype="bf16")
    img = enc.upload_images(wl["images"])
    b, t, o = enc.upload_boxes(wl["boxes"], wl["tier"], wl["box_offsets"])
    runs = []
    for _ in range(3):
        out = enc.alloc_outputs(cfg.B)
        enc.multilevel_batch(img, cfg.B, b, t, o, out)
        enc.sync_status()
        torch.cuda.synchronize()
        runs.append({k: v.cpu().numpy() for k, v in out.items()})
    enc.close()
    T = int(runs[0]["cu_seqlens"][-1])
    _say(f"[case] three runs on one context, {T} mixed tokens + {cfg.B} coarse grids")
    assert T + cfg.B * (cfg.H // cfg.patch[0]) * (cfg.W // cfg.patch[0]) >= 8192
    for r in runs[1:]:
        np.testing.assert_array_equal(r["cu_seqlens"], runs[0]["cu_seqlens"])
        np.testing.assert_array_equal(r["y_coarse"], runs[0]["y_coarse"])
        np.testing.assert_array_equal(r["y_mixed"][:T], runs[0]["y_mixed"][:T])


def test_profile_interface_counts_launches(K):
    cfg = synth.replace(synth.config(2), layers=2)
    wl = synth.make_workload(cfg, seed=47)
    enc = K.Encoder(cfg, wl["weights"])
    img = enc.upload_images(wl["images"])
    b, t, o = enc.upload_boxes(wl["boxes"], wl["tier"], wl["box_offsets"])
    out = enc.alloc_outputs(cfg.B)
    K.cfdetr_profile_begin(enc.ctx)
    enc.multilevel_batch(img, cfg.B, b, t, o, out)
    prof = K.cfdetr_profile_end(enc.ctx)
    # the coarse grids and the mixed sets go through the layers as ONE varlen batch
    assert prof["attention"]["launches"] == cfg.layers
    # d_model 256: everything of a layer after attention is one kernel (counted as ffn2),
    # which also applies the LayerNorm that follows and the next layer's q/k/v projection;
    # the very first LayerNorm and projection are one launch (counted as qkv)
    assert cfg.d == 256 and prof["layernorm"]["launches"] == 0
    assert prof["ffn2"]["launches"] == cfg.layers
    assert prof["out_proj"]["launches"] == 0 and prof["ffn1"]["launches"] == 0
    assert prof["qkv"]["launches"] == 1
    # the selection kernel of a merged run also makes the attention plan
    assert prof["plan"]["launches"] == 0
    assert prof["select"]["launches"] == 1 and prof["gather"]["launches"] == 1
    assert prof["embed"]["launches"] == 2
    assert all(v["ms"] >= 0 for v in prof.values())
    enc.close()


# ------------------------------------------------------------------ offsets from the caller
def test_fine_encode_rejects_offsets_beyond_the_capacity(K):
    """cfdetr_fine_encode takes its offsets from the caller: a total above max_tokens_total, or
    a negative length, must be reported by cfdetr_sync_status and must leave y untouched."""
    import torch
    cfg = synth.replace(synth.config(3), B=2, H=128, W=128, layers=1)
    wl = synth.make_workload(cfg, seed=51)
    for act in ("bf16", "fp32"):
        enc = K.Encoder(cfg, wl["weights"], act_dtype=act, max_tokens_total=100)
        img = enc.upload_images(wl["images"])
        out = enc.alloc_outputs(cfg.B)
        out["tok_desc"].zero_()                      # every entry a valid coarse cell
        for bad in ([0, 60, 130], [0, 70, 60], [0, -5, 40]):
            _say(f"[case] fine_encode with offsets {bad} on a context of 100 tokens, {act}")
            out["y_mixed"].fill_(-7.0)
            out["cu_seqlens"].copy_(torch.tensor(bad, dtype=torch.int32))
            enc.fine_encode(img, cfg.B, out["tok_desc"], out["cu_seqlens"], None, out["y_mixed"])
            with pytest.raises(K.CfdetrError) as ei:
                enc.sync_status()
            assert ei.value.status == K.CFDETR_ECAPACITY
            assert (out["y_mixed"].cpu().numpy() == -7.0).all()
        # the context keeps working: a total that just fits
        out["cu_seqlens"].copy_(torch.tensor([0, 60, 100], dtype=torch.int32))
        enc.fine_encode(img, cfg.B, out["tok_desc"], out["cu_seqlens"], None, out["y_mixed"])
        enc.sync_status()
        y = out["y_mixed"].cpu().numpy()
        assert np.isfinite(y).all() and (y != -7.0).all()
        enc.close()


@pytest.mark.parametrize("act", ["fp32", "bf16"])
def test_easy_frames_skip_the_fine_stage(K, act):
    """Sec. III-B, A1: a frame found easy after the coarse stage has no fine stage.  With the
    difficulty flags the selection gives such a frame no token and the fine pass computes
    nothing for it; the other frames come out as without the flags."""
    import torch
    cfg = synth.replace(synth.config(3), B=4, H=320, W=320, layers=2)
    wl = synth.make_workload(cfg, seed=53)
    for hard in ([1, 0, 1, 0], [0, 1, 1, 1], [0, 0, 0, 0]):
        _say(f"[case] easy-frame skip, hard = {hard}, {act}")
        tok, cu, counts = O.select_fine(wl["boxes"], wl["tier"], wl["box_offsets"], cfg.B, cfg.H,
                                        cfg.W, cfg.patch, hard=np.asarray(hard))
        ref = O.fine_encode(wl["images"], tok, cu, cfg.patch, wl["weights"], cfg.heads)
        enc = K.Encoder(cfg, wl["weights"], act_dtype=act)
        img = enc.upload_images(wl["images"])
        b, t, o = enc.upload_boxes(wl["boxes"], wl["tier"], wl["box_offsets"])
        out = enc.alloc_outputs(cfg.B)
        out["y_mixed"].fill_(-7.0)
        h = torch.tensor(hard, dtype=torch.int32, device="cuda")
        enc.coarse_encode(img, cfg.B, out["x0_cache"], out["y_coarse"])
        enc.select_fine_hard(b, t, o, h, cfg.B, out["tok_desc"], out["cu_seqlens"],
                             out["level_counts"])
        enc.fine_encode(img, cfg.B, out["tok_desc"], out["cu_seqlens"], out["x0_cache"],
                        out["y_mixed"])
        enc.sync_status()
        T = int(cu[-1])
        np.testing.assert_array_equal(out["cu_seqlens"].cpu().numpy(), cu)
        np.testing.assert_array_equal(out["level_counts"].cpu().numpy(), counts)
        np.testing.assert_array_equal(out["tok_desc"].cpu().numpy()[:T], O.pack_tok_desc(tok))
        y = out["y_mixed"].cpu().numpy()
        assert (y[T:] == -7.0).all()
        if T:
            e = rel_err(y[:T], ref)
            _say(f"[parity] easy-frame skip {hard} {act}: T={T} mixed {e:.2e} rms {rms_err(y[:T], ref):.2e}")
            assert e <= TOL[act]
        enc.close()


def test_a_run_with_non_finite_values_does_not_poison_later_runs(K):
    """The feature-major copy of V pads every sequence to a multiple of 64 positions, and the
    padding moves with the sequence lengths.  Whatever a run leaves there (here: NaN from a
    frame of NaN pixels) must not reach a later run on the same context."""
    import torch
    cfg = synth.replace(synth.config(3), B=3, H=320, W=320, layers=2)
    wl = synth.make_workload(cfg, seed=57)
    clean = gpu_multilevel(K, cfg, wl, "bf16")
    enc = K.Encoder(cfg, wl["weights"], act_dtype="bf16")
    b, t, o = enc.upload_boxes(wl["boxes"], wl["tier"], wl["box_offsets"])
    # run 1: NaN frames, every cell refined (the longest sequences the context takes)
    bad_img = enc.upload_images(np.full_like(wl["images"], np.nan))
    everything = np.tile(np.asarray([[0, 0, cfg.W, cfg.H]], np.int32), (cfg.B, 1))
    ab, at, ao = enc.upload_boxes(everything, np.ones(cfg.B, np.uint8), np.arange(cfg.B + 1))
    out = enc.alloc_outputs(cfg.B)
    enc.multilevel_batch(bad_img, cfg.B, ab, at, ao, out)
    enc.sync_status()
    assert not np.isfinite(out["y_mixed"].cpu().numpy()).any()
    # run 2: the clean workload on the same context
    img = enc.upload_images(wl["images"])
    out = enc.alloc_outputs(cfg.B)
    enc.multilevel_batch(img, cfg.B, b, t, o, out)
    enc.sync_status()
    T = int(clean["cu_seqlens"][-1])
    assert (np.diff(clean["cu_seqlens"]) % 64 != 0).any()
    np.testing.assert_array_equal(out["y_mixed"].cpu().numpy()[:T], clean["y_mixed"][:T])
    np.testing.assert_array_equal(out["y_coarse"].cpu().numpy(), clean["y_coarse"])
    enc.close()
