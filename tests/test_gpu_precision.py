"""What the kernels hold in fp32 between their bf16 operands.  The weights are chosen so that no
operand is rounded (attention that averages equal values, hidden units that the activation passes
through), which leaves the rounding of the fp32 sums alone; the reference is float64."""
import numpy as np
import pytest

from paper_2505_23317_amd import synth

pytestmark = pytest.mark.gpu

# 899 tokens a frame: one frame goes where few rows go (width 384: the spread kernels), the others
# to workgroups of 32, 64 and 96 rows
FORMS = [(256, 1), (256, 10), (256, 19), (384, 1), (384, 4), (384, 10), (384, 19)]


def _weights(cfg, seed):
    """Every matrix and bias zero but what follows: values v for all tokens (queries and keys are zero,
    so attention returns v), hidden units h between 8 and 16 (the activation returns them)."""
    rng = np.random.default_rng(seed)
    w = {k: np.zeros_like(a) for k, a in synth.make_weights(cfg, seed).items()}
    for k in ("ln1_g", "ln2_g", "lnf_g"):
        w[k] += 1.0
    w["b_qkv"][0, 2 * cfg.d:] = v = synth.bf16_round(rng.uniform(-2.0, 2.0, cfg.d).astype(np.float32))
    w["b_ff1"][0] = h = synth.bf16_round(rng.uniform(8.0, 15.9, cfg.ffn).astype(np.float32))
    return w, v.astype(np.float64), h.astype(np.float64), rng


def _coarse(cfg, w):
    """(embedded tokens, result) of black frames"""
    import torch
    from paper_2505_23317_amd import cfdetr as K
    enc = K.Encoder(cfg, w)
    out = enc.alloc_outputs(cfg.B)
    img = enc.upload_images(np.zeros((cfg.B, 3, cfg.H, cfg.W), np.float32))
    enc.coarse_encode(img, cfg.B, out["x0_cache"], out["y_coarse"])
    enc.sync_status()
    torch.cuda.synchronize()
    x0, y = (out[k].cpu().numpy().astype(np.float64) for k in ("x0_cache", "y_coarse"))
    enc.close()
    return x0, y


@pytest.mark.parametrize("ratio", [1.0, 30.0, 1000.0])
@pytest.mark.parametrize("d, frames", FORMS)
def test_products_are_not_rounded_at_the_residuals_magnitude(d, frames, ratio):
    """Residual rows of the size of what the two products of a layer add to them, and of 30 and 1000
    times that.  A product that is summed by itself and added once leaves half a unit at the residual's
    magnitude at most (3e-8 root mean square of it for both), its own sum's rounding, which is as much
    where the two are of a size, and that of LayerNorm's few operations: 1.3e-7 is above their sum.
    Summed on top of the residual a product leaves a rounding for each of its 16 to 96 steps."""
    cfg = synth.Config("sums", frames, 232, 248, (8,), d, 8 if d == 256 else 6, 1, 4 * d, "bf16", box_rule="poisson")
    w, v, h, rng = _weights(cfg, 3)
    w["b_embed0"] += rng.normal(0.0, ratio, d).astype(np.float32)
    w["w_o"][0] = synth.bf16_round(rng.normal(0.0, 0.9 / np.sqrt(d), (d, d)).astype(np.float32))
    w["w_ff2"][0] = synth.bf16_round(rng.normal(0.0, 0.08 / np.sqrt(cfg.ffn), (d, cfg.ffn)).astype(np.float32))
    w["b_o"][0] = rng.normal(0.0, 0.1, d)
    w["b_ff2"][0] = rng.normal(0.0, 0.1, d)
    x0, y = _coarse(cfg, w)
    x1 = x0 + (w["w_o"][0].astype(np.float64) @ v + w["b_o"][0].astype(np.float64))
    x2 = x1 + (w["w_ff2"][0].astype(np.float64) @ h + w["b_ff2"][0].astype(np.float64))
    assert 0.5 < np.std(x1 - x0) < 2.0 and 0.5 < np.std(x2 - x1) < 2.0 and 0.7 * ratio < np.std(x0) < 2.0 * ratio
    c = x2 - x2.mean(axis=1, keepdims=True)
    ref = c / np.sqrt((c * c).mean(axis=1, keepdims=True) + 1e-5)
    rms = float(np.sqrt(((y - ref) ** 2).mean()))
    print(f"residual {ratio} times the products, width {d}, {frames} frames: {rms:.2e}", flush=True)
    assert rms <= 1.3e-7


@pytest.mark.parametrize("d, frames", FORMS + [(768, 1), (768, 10)])
def test_rows_of_equal_values_normalise_to_the_offsets(d, frames):
    """Every column 3 * 2^29 (the bias is added to tokens too small to change it; sums and mean of such
    rows are exact): x - mean is 0, and the result is LayerNorm's offset to the bit.  With x / sigma and
    mean / sigma rounded apart it is off by what a float leaves of 5e11, and so it is with a mean that
    is rounded."""
    cfg = synth.Config("equal", frames, 232, 248, (8,), d, 8 if d == 256 else d // 64, 1, 4 * d, "bf16", box_rule="poisson")
    w, _, _, rng = _weights(cfg, 5)
    w["b_qkv"][:] = 0.0
    w["b_ff1"][:] = 0.0
    w["b_o"][0] = 3.0 * 2.0 ** 29
    w["lnf_b"][:] = rng.normal(0.0, 1.0, d)
    x0, y = _coarse(cfg, w)
    assert np.abs(x0).max() < 64.0
    assert (y == w["lnf_b"].astype(np.float64)).all()


# Probabilities p, a head each, and its value v: attention over equal keys gives v bf16(p) / p, and p
# is chosen so that this lies 1e-5 of itself below or above a boundary between two bf16 numbers.  Of
# 6,400 equal probabilities a sum that runs over one pair after the other is off by 2.3e-5 (-2.3e-5 for
# the first, 2.2e-5 for the second) and lands on the other side; tile by tile it is off by less than 1e-6.
EDGES = [(1.203125, 1.5, 1.50390625, -1), (1.28125, 1.75, 1.75390625, 1)]   # bf16(p), v, boundary, side


def _edge_probability(edge):
    P, v, boundary, side = edge
    return v * P / (boundary * (1.0 + side * 1e-5))


def _summed(p, keys, pairs):
    """Relative error of a lane's sum of half the keys in fp32, `pairs` pairs at a time."""
    pair, total = np.float32(p) + np.float32(p), np.float32(0.0)
    for _ in range(keys // (4 * pairs)):
        part = np.float32(0.0)
        for _ in range(pairs):
            part = np.float32(part + pair)
        total = np.float32(total + part)
    return float(total) / (keys / 2 * float(np.float32(p))) - 1.0


@pytest.mark.parametrize("heads, frames", [(2, 1), (2, 9), (4, 1)])
def test_probabilities_are_summed_tile_by_tile(heads, frames):
    """6,400 keys a frame; items of 128 queries, of 256 (nine frames) and heads of 32."""
    d, keys = 128, 6400
    for edge in EDGES:
        p = _edge_probability(edge)
        assert synth.bf16_round(np.array([p], np.float32))[0] == edge[0]
        assert np.sign(_summed(p, keys, 1)) == edge[3] and abs(_summed(p, keys, 1)) > 1.8e-5
        assert abs(_summed(p, keys, 16)) < 1e-6
    cfg = synth.Config("tiles", frames, 640, 640, (8,), d, heads, 1, 64, "bf16", box_rule="poisson")
    assert cfg.n_cells(0) == keys and (frames == 1 or frames * keys * heads > 3500 * 32)
    w, _, _, _ = _weights(cfg, 9)
    w["b_ff1"][:] = 0.0
    dh = cfg.d_head
    out = np.zeros(d)
    for h in range(heads):
        edge = EDGES[h % 2]
        rest = np.float32(np.log2(_edge_probability(edge)))   # in three parts, so that no bf16 rounds it
        for k in range(3):
            part = synth.bf16_round(np.array([rest], np.float32))[0]
            w["b_qkv"][0, h * dh + k] = part * np.sqrt(dh) / 1.4426950408889634
            rest = np.float32(rest - part)
        assert rest == 0.0
        w["b_qkv"][0, d + h * dh:d + h * dh + 3] = 1.0
        w["b_qkv"][0, 2 * d + h * dh:2 * d + (h + 1) * dh] = edge[1]
        exact = edge[1] * edge[0] / _edge_probability(edge)
        out[h * dh:(h + 1) * dh] = synth.bf16_round(np.array([exact], np.float32))[0]
    w["w_o"][0] = np.eye(d)
    x0, y = _coarse(cfg, w)
    c = x0 + out - (x0 + out).mean(axis=1, keepdims=True)
    ref = c / np.sqrt((c * c).mean(axis=1, keepdims=True) + 1e-5)
    # a bf16 step of one head's output moves its columns by 4e-3 and more; fp32 leaves 1e-6
    assert np.abs(y - ref).max() < 1e-4
