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


# widths 64 and 128 are one kernel at every row count, width 768 has its kernels for few rows and for more
@pytest.mark.parametrize("ratio", [1.0, 30.0, 1000.0])
@pytest.mark.parametrize("d, frames", FORMS + [(64, 1), (64, 10), (128, 1), (128, 10), (768, 1), (768, 10)])
def test_products_of_two_layers_are_not_rounded_at_the_residuals_magnitude(d, frames, ratio):
    """As above over two layers, so that residual rows also go on from one layer to the next.  Four products are
    added: twice the variance of the errors, 1.3e-7 sqrt(2) = 1.8e-7; at width 768, whose sums have twice the steps of width
    384, the products' own rounding, which is all of it where the two are of a size, has twice the variance again: 2.6e-7.
    Sums on top of the residual (2.6e-7 and more a layer at width 256) are at 3.7e-7 and more."""
    cfg = synth.Config("sums", frames, 232, 248, (8,), d, d // 32 if d <= 256 else d // 64, 2, 4 * d, "bf16", box_rule="poisson")
    w, _, _, rng = _weights(cfg, 3)
    w["b_embed0"] += rng.normal(0.0, ratio, d).astype(np.float32)
    x0 = x = None
    steps = []
    for l in range(2):
        w["b_qkv"][l, 2 * d:] = v = synth.bf16_round(rng.uniform(-2.0, 2.0, d).astype(np.float32))
        w["b_ff1"][l] = h = synth.bf16_round(rng.uniform(8.0, 15.9, cfg.ffn).astype(np.float32))
        w["w_o"][l] = synth.bf16_round(rng.normal(0.0, 0.9 / np.sqrt(d), (d, d)).astype(np.float32))
        w["w_ff2"][l] = synth.bf16_round(rng.normal(0.0, 0.08 / np.sqrt(cfg.ffn), (d, cfg.ffn)).astype(np.float32))
        w["b_o"][l] = rng.normal(0.0, 0.1, d)
        w["b_ff2"][l] = rng.normal(0.0, 0.1, d)
        steps += [w["w_o"][l].astype(np.float64) @ v.astype(np.float64) + w["b_o"][l],
                  w["w_ff2"][l].astype(np.float64) @ h.astype(np.float64) + w["b_ff2"][l]]
    x0, y = _coarse(cfg, w)
    assert all(0.5 < np.std(step) < 2.0 for step in steps) and 0.6 * ratio < np.std(x0) < 2.0 * ratio
    x = x0 + sum(steps)
    c = x - x.mean(axis=1, keepdims=True)
    ref = c / np.sqrt((c * c).mean(axis=1, keepdims=True) + 1e-5)
    rms = float(np.sqrt(((y - ref) ** 2).mean()))
    print(f"two layers, residual {ratio} times the products, width {d}, {frames} frames: {rms:.2e}", flush=True)
    assert rms <= (2.6e-7 if d == 768 else 1.8e-7)


# 1,024 queries of one to four frames: spread over the chip and, at width 384, one kernel a layer
@pytest.mark.parametrize("d, heads, frames", [(128, 4, 1), (256, 8, 1), (256, 8, 4), (384, 6, 1), (384, 6, 4), (768, 12, 1),
                                              (768, 12, 4)])
def test_products_of_the_decoder_are_not_rounded_at_the_residuals_magnitude(d, heads, frames):
    """Queries of C = 49,152 plus values of a few units, two layers of three products each: the last LayerNorm takes C
    off, and its bf16 rows show what was lost beside it.  The bar is what one rounding to a float for each addition to the
    rows leaves, and the rounding to bf16, worked out here, and half of that again for LayerNorm in fp32 (the mean comes from
    sums of up to d values of C).  Summed on top of C, the 48 (width 128) to 288 steps of a layer's products would be rounded
    there one by one: three times that and more."""
    import torch
    from paper_2505_23317_amd import cfdetr as K

    Q, C, layers, rng = 1024, 49152.0, 2, np.random.default_rng(13)
    cfg = synth.Config("dec_sums", frames, 64, 64, (16,), d, heads, 1, 4 * d, "bf16", box_rule="poisson")
    dw = {k: np.zeros_like(a) for k, a in synth.make_decoder_weights(cfg, 3, n_queries=Q, layers=layers).items()}
    for k in ("ln1_g", "ln2_g", "ln3_g", "lnf_g"):
        dw[k] += 1.0
    x = C + np.round(rng.normal(0.0, 1.0, (Q, d)) * 256.0) / 256.0      # exact in fp32
    dw["query_embed"] = x.astype(np.float32)
    assert (dw["query_embed"].astype(np.float64) == x).all()
    rounded = dw["query_embed"]
    for l in range(layers):
        for b, o in (("b_qkv", "o"), ("b_kv", "o2")):
            v = synth.bf16_round(rng.uniform(-2.0, 2.0, d).astype(np.float32))
            dw[b][l, -d:] = v
            dw["w_" + o][l] = synth.bf16_round(rng.normal(0.0, 0.9 / np.sqrt(d), (d, d)).astype(np.float32))
            dw["b_" + o][l] = rng.normal(0.0, 0.1, d)
            step = dw["w_" + o][l].astype(np.float64) @ v.astype(np.float64) + dw["b_" + o][l]
            x, rounded = x + step, rounded + step.astype(np.float32)
        dw["b_ff1"][l] = h = synth.bf16_round(rng.uniform(8.0, 15.9, cfg.ffn).astype(np.float32))
        dw["w_ff2"][l] = synth.bf16_round(rng.normal(0.0, 0.08 / np.sqrt(cfg.ffn), (d, cfg.ffn)).astype(np.float32))
        dw["b_ff2"][l] = rng.normal(0.0, 0.1, d)
        step = dw["w_ff2"][l].astype(np.float64) @ h.astype(np.float64) + dw["b_ff2"][l]
        x, rounded = x + step, rounded + step.astype(np.float32)

    def normed(rows):
        c = rows - rows.mean(axis=1, keepdims=True)
        return c / np.sqrt((c * c).mean(axis=1, keepdims=True) + 1e-5)

    assert rounded.dtype == np.float32
    z, z_once = normed(x), synth.bf16_round(normed(rounded.astype(np.float64)).astype(np.float32)).astype(np.float64)
    # logits that are values of z: the confidence one column, the box four columns where they are positive
    for k in ("w_box1", "w_box2"):
        dw[k][:] = np.eye(d)
    mem = torch.randn((frames * 16, d), generator=torch.Generator().manual_seed(5)).cuda()
    cu = torch.arange(frames + 1, dtype=torch.int32).cuda() * 16
    out = torch.empty((frames, Q, 5), device="cuda")
    errors, once = [], []
    for columns in rng.permutation(d)[:30].reshape(6, 5):
        for k in ("w_cls", "w_box3"):
            dw[k][:] = 0.0
        dw["w_cls"][0, columns[4]] = 1.0
        dw["w_box3"][range(4), columns[:4]] = 1.0
        enc = K.Encoder(cfg, synth.make_weights(cfg, 1))
        enc.attach_decoder(dw)
        enc.decode(mem, cu, frames, out)
        enc.sync_status()
        got = out.cpu().numpy().astype(np.float64)
        enc.close()
        want = np.broadcast_to(z[:, columns], got.shape)
        use = (want > 0.05) & (want < 4.0)
        use[..., 4] |= (want[..., 4] > -4.0) & (want[..., 4] < -0.05)
        assert use.sum() > 1024 * frames
        errors.append((np.log(got[use] / (1.0 - got[use])) - want[use]) ** 2)
        once.append((np.broadcast_to(z_once[:, columns], got.shape)[use] - want[use]) ** 2)
    rms, bar = (float(np.sqrt(np.concatenate(e).mean())) for e in (errors, once))
    print(f"decoder of width {d}, {frames} frames: {rms:.2e}, one rounding an addition {bar:.2e}", flush=True)
    assert rms <= 1.5 * bar


@pytest.mark.parametrize("d", [64, 128])
def test_deviation_of_a_row_at_narrow_widths(d):
    """1/sigma of the rows, as the factor by which a whole row is off (its elements' own roundings average out).  The
    reciprocal root and as many roundings of the squares' sum as layernorm4_kernel has; that leaves 3.79e-8 (width 64) and
    3.52e-8 (128) root mean square of these rows, and the bar is a twentieth above.  A lane's sixteen squares one after the
    other and one rounding more at the sum's magnitude leave 4.29e-8 and 3.90e-8."""
    import torch
    from paper_2505_23317_amd import cfdetr as K

    cfg = synth.Config("rows", 16, 232, 248, (8,), d, d // 32, 1, 128, "bf16", box_rule="poisson")
    w, _, _, rng = _weights(cfg, 7)
    w["b_qkv"][:] = 0.0
    w["b_ff1"][:] = 0.0
    w["b_embed0"] += rng.normal(0.0, 1.0, d).astype(np.float32)
    w["w_embed0"][:] = synth.bf16_round(rng.normal(0.0, 0.1, w["w_embed0"].shape).astype(np.float32))
    enc = K.Encoder(cfg, w)
    out = enc.alloc_outputs(cfg.B)
    img = enc.upload_images(synth.bf16_round(rng.normal(0.5, 0.5, (cfg.B, 3, cfg.H, cfg.W)).astype(np.float32)))
    enc.coarse_encode(img, cfg.B, out["x0_cache"], out["y_coarse"])
    enc.sync_status()
    x0, y = (out[k].cpu().numpy().astype(np.float64) for k in ("x0_cache", "y_coarse"))
    enc.close()
    c = x0 - x0.mean(axis=1, keepdims=True)
    ref = c / np.sqrt((c * c).mean(axis=1, keepdims=True) + 1e-5)
    rms = float(np.sqrt((((y * ref).sum(axis=1) / (ref * ref).sum(axis=1) - 1.0) ** 2).mean()))
    print(f"deviation of rows of width {d}: {rms:.3e}", flush=True)
    assert rms <= (4.0e-8 if d == 64 else 3.7e-8)
