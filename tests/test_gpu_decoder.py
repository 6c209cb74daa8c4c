"""map_decoder_layer on the GPU against the decoder-layer oracle (float64),
on the same bf16 inputs and weights.

Bar.  The layer stores bf16 intermediates (the two RMSNorm outputs, q, k and
v, the attention output, the block residual, the SwiGLU product, and gate and
up where their product runs on the register-staged kernel) and its output, each
rounded to 2^-9 relative; the products sum them in float32.  The layer's update Y - X must match the oracle's in the
relative Frobenius norm to 3e-2, and Y itself (dominated by the residual X)
to 1e-2; the cosine between the updates must exceed 0.999.  Cases: ragged
packed sequences at a small width (two heads), one sequence of the pruned
LLaVA-NeXT length (160 kept + 64 question tokens) at the 7B shape, and the
layer-0 input map_prune_assemble writes for a two-image batch.
"""
import numpy as np
import pytest
import torch

import oracle
from workloads import bf16_bits_to_f32, f32_to_bf16_bits

from gpu_util import announce, device

pytestmark = pytest.mark.gpu


def _weights(d, ff, seed, std=0.02):
    rng = np.random.default_rng(seed)
    shapes = {"attn_norm": (d,), "w_qkv": (3 * d, d), "w_o": (d, d), "ffn_norm": (d,), "w_gate_up": (2 * ff, d),
              "w_down": (d, ff)}
    out = {}
    for k, s in shapes.items():
        x = (1.0 + 0.1 * rng.standard_normal(s)) if "norm" in k else std * rng.standard_normal(s)
        out[k] = f32_to_bf16_bits(x.astype(np.float32))
    return out


def _dev(bits, dev):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to(dev).view(torch.bfloat16)


def _run_and_check(X_bits, pos, seq_off, wb, n_heads, tag):
    import paper_2608_06411_amd as mp
    dev = device()
    d = X_bits.shape[1]
    w = mp.DecoderWeights(**{k: _dev(v, dev) for k, v in wb.items()}, n_heads=n_heads)
    Y = mp.map_decoder_layer(w, _dev(X_bits, dev), torch.from_numpy(np.asarray(pos, np.int32)).to(dev), seq_off)
    torch.cuda.synchronize()
    got = bf16_bits_to_f32(Y.view(torch.int16).cpu().numpy().view(np.uint16)).astype(np.float64)
    X = bf16_bits_to_f32(X_bits).astype(np.float64)
    want = oracle.decoder_layer(X, pos, seq_off, {k: bf16_bits_to_f32(v) for k, v in wb.items()}, n_heads)
    du, dw = got - X, want - X
    err_u = np.linalg.norm(du - dw) / np.linalg.norm(dw)
    err_y = np.linalg.norm(got - want) / np.linalg.norm(want)
    cos = float(np.sum(du * dw) / (np.linalg.norm(du) * np.linalg.norm(dw)))
    print(f"[decoder {tag}] update err {err_u:.2e}, output err {err_y:.2e}, cosine {cos:.6f}", flush=True)
    assert err_u <= 3e-2 and err_y <= 1e-2 and cos >= 0.999, (err_u, err_y, cos)
    return got


def test_decoder_small_ragged_sequences():
    d, H, ff = 256, 2, 512
    announce("decoder small ragged")
    rng = np.random.default_rng(3)
    seq_off = [0, 37, 140, 141, 300]          # one single-token sequence; blocks of 64 with tails
    R = seq_off[-1]
    X = f32_to_bf16_bits(rng.standard_normal((R, d)).astype(np.float32))
    pos = np.concatenate([np.sort(rng.choice(3000, seq_off[b + 1] - seq_off[b], replace=False))
                          for b in range(len(seq_off) - 1)]).astype(np.int32)
    _run_and_check(X, pos, seq_off, _weights(d, ff, 5, std=0.05), H, "small")


def test_decoder_7b_shape_pruned_length():
    """d 4096, 32 heads x 128, SwiGLU 11008: one sequence of 224 rows (the
    LLaVA-NeXT image pruned to 160 tokens, then a 64-token question)."""
    d, H, ff = 4096, 32, 11008
    announce("decoder 7B shape, 224 rows")
    rng = np.random.default_rng(4)
    X = f32_to_bf16_bits(rng.standard_normal((224, d)).astype(np.float32))
    pos = np.concatenate([np.sort(rng.choice(2880, 160, replace=False)), 2880 + np.arange(64)]).astype(np.int32)
    _run_and_check(X, pos, [0, 224], _weights(d, ff, 6), H, "7B 224")


def test_decoder_long_sequences_large_tiles():
    """Two sequences of 2944 and 1500 rows at d 1024 (8 heads), SwiGLU 2816:
    every product runs on tiles of 256 columns, cut into tiles of several
    heights (4444 rows: a ragged last tile row)."""
    d, H, ff = 1024, 8, 2816
    announce("decoder long sequences, 4444 rows at d 1024")
    rng = np.random.default_rng(8)
    seq_off = [0, 2944, 4444]
    X = f32_to_bf16_bits(rng.standard_normal((seq_off[-1], d)).astype(np.float32))
    pos = np.concatenate([np.arange(2944), np.arange(1500) * 2]).astype(np.int32)
    _run_and_check(X, pos, seq_off, _weights(d, ff, 9, std=0.03), H, "long")


def test_decoder_on_the_pruned_layer0_input():
    """map_prune_assemble's output for two images is the layer's input: the
    sequences are each image's kept rows then its question rows."""
    import paper_2608_06411_amd as mp
    from workloads import PredictorShape, get_config, make_inputs
    from gpu_util import dev_inputs
    cfg = get_config("sweep", B=2, N=600, M=(16, 40), K=64, K0=32, pred=PredictorShape(D=512, D_h=128, d_p=64))
    announce("decoder on map_prune_assemble's output")
    x = make_inputs(cfg)
    dev = device()
    di = dev_inputs(x, dev)
    f = mp.map_prune_assemble(di["w"], di["V"], di["pos_v"], di["T"], di["pos_t"], x["t_off"], cfg.K, cfg.K0, cfg.tau)
    torch.cuda.synchronize()
    seq_off = [b * cfg.K + int(x["t_off"][b]) for b in range(cfg.B + 1)]
    X_bits = f["X"].view(torch.int16).cpu().numpy().view(np.uint16)
    _run_and_check(X_bits, f["pos_x"].cpu().numpy(), seq_off, _weights(512, 768, 7, std=0.04), 4, "layer-0 input")


@pytest.mark.parametrize("lens", [
    [1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 200],        # 64 query rows per workgroup
    [500, 129, 128, 127, 1, 65, 64, 33, 32, 31] + [97] * 54,  # enough of them for 128 rows each
])
def test_decoder_attention_block_edges(lens):
    """Sequences that end at and beside the edges of the attention's query
    rows (32 per wave) and key blocks (64), every row of the update held to
    the update's bar (a row lost or wrongly masked moves its own update by
    far more)."""
    d, H, ff = 256, 2, 256
    announce(f"decoder attention edges, {len(lens)} sequences")
    rng = np.random.default_rng(len(lens))
    seq_off = [0] + [int(v) for v in np.cumsum(lens)]
    R = seq_off[-1]
    X = f32_to_bf16_bits(rng.standard_normal((R, d)).astype(np.float32))
    pos = np.concatenate([np.sort(rng.choice(3000, n, replace=False)) for n in lens]).astype(np.int32)
    wb = _weights(d, ff, 11, std=0.06)
    got = _run_and_check(X, pos, seq_off, wb, H, "attention edges")
    x = bf16_bits_to_f32(X).astype(np.float64)
    want = oracle.decoder_layer(x, pos, seq_off, {k: bf16_bits_to_f32(v) for k, v in wb.items()}, H)
    row = np.linalg.norm(got - want, axis=1) / np.linalg.norm(want - x, axis=1)
    assert row.max() <= 3e-2, (int(row.argmax()), float(row.max()))


@pytest.mark.parametrize("lens", [
    [500, 500, 409],            # products of 128-row tiles only, and of 192-row tiles with a last one of 65 rows
    [512] * 5 + [451],          # 192-row tiles whose last one reaches into its lower half (131 rows)
    [512] * 5 + [384],          # 256-row tiles, then 128 rows more; 192-row tiles, then 64 rows more
    [512] * 9 + [392],          # 192-row tiles for the first rounds, 128-row tiles for the rest
])
def test_decoder_tile_heights(lens):
    """Row counts whose products are cut into tiles of 256, 192 and 128 rows,
    every row of the update held to the update's bar."""
    d, H, ff = 1024, 8, 2816
    announce(f"decoder tile heights, {sum(lens)} rows")
    rng = np.random.default_rng(sum(lens))
    seq_off = [0] + [int(v) for v in np.cumsum(lens)]
    X = f32_to_bf16_bits(rng.standard_normal((seq_off[-1], d)).astype(np.float32))
    pos = np.concatenate([np.arange(n) for n in lens]).astype(np.int32)
    wb = _weights(d, ff, 12, std=0.03)
    got = _run_and_check(X, pos, seq_off, wb, H, "tile heights")
    x = bf16_bits_to_f32(X).astype(np.float64)
    want = oracle.decoder_layer(x, pos, seq_off, {k: bf16_bits_to_f32(v) for k, v in wb.items()}, H)
    row = np.linalg.norm(got - want, axis=1) / np.linalg.norm(want - x, axis=1)
    assert row.max() <= 3e-2, (int(row.argmax()), float(row.max()))


def test_decoder_weights_off_alignment():
    """Gate and up weights two bytes off a 16-byte boundary: the product by
    the register-staged kernel and its separate SwiGLU."""
    import paper_2608_06411_amd as mp
    dev = device()
    d, H, ff = 256, 2, 512
    announce("decoder, gate and up weights off alignment")
    rng = np.random.default_rng(13)
    seq_off = [0, 70, 133]
    x = _dev(f32_to_bf16_bits(rng.standard_normal((133, d)).astype(np.float32)), dev)
    pos = torch.arange(133, dtype=torch.int32, device=dev)
    wt = {k: _dev(v, dev) for k, v in _weights(d, ff, 14, std=0.05).items()}
    want = mp.map_decoder_layer(mp.DecoderWeights(**wt, n_heads=H), x, pos, seq_off)
    flat = torch.empty(2 * ff * d + 1, dtype=torch.bfloat16, device=dev)
    flat[1:] = wt["w_gate_up"].reshape(-1)
    wt["w_gate_up"] = flat[1:].view(2 * ff, d)
    got = mp.map_decoder_layer(mp.DecoderWeights(**wt, n_heads=H), x, pos, seq_off)
    du, dw = (got - x).double(), (want - x).double()
    assert float((du - dw).norm() / dw.norm()) <= 1e-2  # two bf16 roundings more (2^-9 each) in one path


@pytest.mark.parametrize("name", ["w_qkv", "w_o", "w_gate_up", "w_down"])
@pytest.mark.parametrize("rows", [[70, 63], [4400]])  # the products by w_o and w_down split over K; whole
def test_decoder_each_weight_off_alignment(name, rows):
    """Any one of the weights two bytes off a 16-byte boundary."""
    import paper_2608_06411_amd as mp
    dev = device()
    d, H, ff = 512, 4, 768
    announce(f"decoder, {name} off alignment, {sum(rows)} rows")
    rng = np.random.default_rng(15)
    seq_off = [0] + [int(v) for v in np.cumsum(rows)]
    x = _dev(f32_to_bf16_bits(rng.standard_normal((seq_off[-1], d)).astype(np.float32)), dev)
    pos = torch.arange(seq_off[-1], dtype=torch.int32, device=dev)
    wt = {k: _dev(v, dev) for k, v in _weights(d, ff, 16, std=0.05).items()}
    want = mp.map_decoder_layer(mp.DecoderWeights(**wt, n_heads=H), x, pos, seq_off)
    flat = torch.empty(wt[name].numel() + 1, dtype=torch.bfloat16, device=dev)
    flat[1:] = wt[name].reshape(-1)
    wt[name] = flat[1:].view(wt[name].shape)
    got = mp.map_decoder_layer(mp.DecoderWeights(**wt, n_heads=H), x, pos, seq_off)
    du, dw = (got - x).double(), (want - x).double()
    assert float((du - dw).norm() / dw.norm()) <= 1e-2  # the other kernel's sums may round a bf16 intermediate (2^-9) the other way


@pytest.mark.parametrize("lens", [[200], [129] * 60 + [600]])  # 64 and 128 query rows per workgroup
def test_decoder_attention_scores_past_float32(lens):
    """Keys whose scores are below float32's range (-1e50: -inf in the products)
    fill a sequence's first key block for the rows after it: they weigh
    nothing, and the rows' update meets the update's bar."""
    d, H, ff = 256, 2, 256
    announce(f"decoder attention, scores past float32, {len(lens)} sequences")
    rng = np.random.default_rng(17)
    seq_off = [0] + [int(v) for v in np.cumsum(lens)]
    place = np.concatenate([np.arange(n) for n in lens])
    x = rng.standard_normal((seq_off[-1], d)).astype(np.float32)
    x[:, 0] = np.where(place < 64, 2.0, 0.0)   # the far keys ...
    x[:, 1] = np.where(place < 64, 0.0, 2.0)   # ... and the queries that see them so
    X = f32_to_bf16_bits(x)
    wb = _weights(d, ff, 18, std=0.05)
    w = bf16_bits_to_f32(wb["w_qkv"])
    w[63] = w[d + 63] = 0.0                     # head 0's slowest pair: angles of at most 0.05
    w[127] = w[d + 127] = 0.0
    w[63, 1], w[d + 63, 0] = 1e25, -1e25
    wb["w_qkv"] = f32_to_bf16_bits(w)
    pos = (place % 400).astype(np.int32)
    got = _run_and_check(X, pos, seq_off, wb, H, "scores past float32")
    assert np.isfinite(got).all()


def test_decoder_rounds_to_nearest_even():
    """The bf16 rounding of float32 sums, read out value by value: one row whose
    RMSNorm is exactly 1 makes v[j] the sum of three weights that add up to a
    chosen float32 (its bits in three pieces, every partial sum exact); the row
    attends to itself only, W_o is the identity and the FFN zero, and the row
    itself (2^-60) vanishes beside v.  Values: ties on either side of even, the
    floats beside them, carries into the exponent, both signs, many exponents."""
    import paper_2608_06411_amd as mp
    dev = device()
    d, ff = 2048, 256
    announce("decoder, rounding to bf16")
    rng = np.random.default_rng(19)
    low = np.array([0x0000, 0x0001, 0x7fff, 0x8000, 0x8001, 0xffff, 0x4000, 0xc000], np.uint32)
    top = rng.integers(0, 0x80, d // 8).astype(np.uint32)
    top[:4] = [0x7f, 0x7e, 0x00, 0x01]
    exp = rng.integers(127 - 30, 127 + 30, d // 8).astype(np.uint32)
    sign = rng.integers(0, 2, d // 8).astype(np.uint32)
    bits = ((sign << 31) | (exp << 23) | (top << 16))[:, None] | low[None, :]
    val = bits.reshape(-1).astype(np.uint32).view(np.float32)

    def head(x):  # the leading eight bits, as a float32 that bf16 holds exactly
        return (x.view(np.uint32) & 0xffff0000).view(np.float32)

    w_v = np.zeros((d, d), np.float32)
    rest = val.copy()
    for col in (3, 700, 1900):
        piece = head(rest)
        w_v[:, col] = piece
        rest = rest - piece
    assert not rest.any()
    w_qkv = np.concatenate([np.zeros((2 * d, d), np.float32), w_v])
    wt = {"attn_norm": np.ones(d), "ffn_norm": np.ones(d), "w_qkv": w_qkv, "w_o": np.eye(d), "w_gate_up": np.zeros((2 * ff, d)),
          "w_down": np.zeros((d, ff))}
    wt = {k: torch.from_numpy(np.asarray(v, np.float32)).to(dev).to(torch.bfloat16) for k, v in wt.items()}
    x = torch.full((1, d), 2.0 ** -60, dtype=torch.bfloat16, device=dev)
    y = mp.map_decoder_layer(mp.DecoderWeights(**wt, n_heads=d // 128, eps=0.0), x, torch.zeros(1, dtype=torch.int32, device=dev),
                             [0, 1])
    u = val.view(np.uint32).astype(np.uint64)
    want = ((u + 0x7fff + ((u >> 16) & 1)) >> 16).astype(np.uint16)  # round to nearest, ties to even
    np.testing.assert_array_equal(y.view(torch.int16).cpu().numpy().view(np.uint16)[0], want)
