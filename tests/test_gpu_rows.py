"""Passes of the GEMMs over the stacked operand (streaming to 64 rows, tiles
above) against the float64 oracle, at the edges of their row tiles, on shapes whose
tile counts leave remainders in every unit size and fewer k-steps than waves,
and at the 7B widths that take the large units."""
import numpy as np
import pytest

from paper_2608_10362_amd import binding, synth
from tests.gpu_util import i32, install_context, kv_to_device, log, torch_cuda
from tests.test_gpu_int4 import _int4_case
from tests.test_gpu_model import _bf16_case, test_bf16_prefill_in_large_chunks as _prefill_case

pytestmark = pytest.mark.gpu

# 20 Q|K|V tiles, 12 residual tiles, 22 gate / up pairs, 31 head tiles; K of 192 (6 k-steps) and 352 (11)
ODD = synth.ModelShape(2, 192, 6, 2, 32, 352, 496)
# K of 576 (18 k-steps) and 1184 (37): waves of a block with different numbers of batches, odd and even, fewer than the
# two a wave holds and more; 275 LM-head units of four tiles, more than one round of the CUs
UNEVEN = synth.ModelShape(2, 576, 18, 6, 32, 1184, 17600)
# float32-accuracy products (2^-17 per product) behind keys and values stored in bf16: single values one
# bf16 unit apart (2^-8) move the logits by 1e-5 to 5e-5 of their norm
REL = 2e-4


def _rows_case(shape, n_layers, lengths, g, seed):
    got, ref, _ = _bf16_case(shape, n_layers, lengths, g, seed=seed, return_logits=True)
    rel = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    log(f"rows {len(lengths) * (g + 1)}: relative error {rel:.3g}")
    assert rel < REL


@pytest.mark.parametrize("B,g", [(17, 0), (4, 7), (11, 2), (6, 7), (7, 6), (8, 7)])
def test_odd_shape_rows(B, g):
    _rows_case(ODD, 2, [1 + (37 * b) % 90 for b in range(B)], g, seed=B)


@pytest.mark.parametrize("B,g", [(1, 0), (1, 7), (3, 2), (4, 3), (5, 3), (5, 7), (7, 7)])
def test_uneven_k_rows(B, g):
    _rows_case(UNEVEN, 1, [1 + (37 * b) % 90 for b in range(B)], g, seed=B)


@pytest.mark.parametrize("shape,B,g", [(UNEVEN, 3, 3), (UNEVEN, 5, 2), (synth.LLAMA_1B, 3, 2), (synth.LLAMA_1B, 2, 7)])
def test_rows_equal_their_sequences_alone(shape, B, g):
    """9 to 16 rows (two fragments of x per k-step) against each sequence in a
    pass of its own (at most 8 rows, one fragment): the same logits bit for bit.
    Contexts of one 32-key sub-chunk, so the attention is cut the same way."""
    torch = torch_cuda()
    lengths = [7 + 5 * b for b in range(B)]
    dw = binding.DeviceWeights(shape, synth.make_weights(shape, n_layers=1))
    ctx = synth.make_kv_context(shape, 1, lengths, seed=70)
    pend = synth.make_prompt(1, shape.vocab, batch=B, seed=71)[:, 0]
    drafts = synth.make_prompt(g, shape.vocab, batch=B, seed=72)

    def verify(seqs):
        n = len(seqs)
        m = binding.Model(dw, 1, max_rows=n * (g + 1), max_ctx=64)
        kv = binding.KVCache(m, n, 64)
        install_context(kv, [[ctx[0][b] for b in seqs]], [lengths[b] for b in seqs], 1, shape.dtype)
        kv.set_state([lengths[b] for b in seqs], [[0, int(pend[b])] for b in seqs], [1] * n)
        logits = torch.empty((n, g + 1, shape.vocab), dtype=torch.float32, device="cuda")
        binding.specdec_verify(m, kv, g, i32(drafts[seqs]), g, logits)
        assert kv.read_state()["status"] == 0
        return logits.cpu().numpy()

    block = verify(list(range(B)))
    for b in range(B):
        assert np.array_equal(verify([b])[0], block[b]), b


@pytest.mark.parametrize("shape,rows,limit", [(synth.LLAMA_1B, 24, 15.5), (synth.LLAMA_1B, 64, 17),
                                              (synth.LLAMA_7B, 24, 22), (synth.LLAMA_7B, 64, 21), (synth.LLAMA_7B, 120, 25)])
def test_first_layer_keys_and_values_round_as_in_64_bits(shape, rows, limit):
    """Keys and values of one prefilled layer against their 64-bit values rounded
    to bf16: only a value within the float32 sums' error of a tie may differ.
    `limit` per 1e5 values lies halfway between what hi and lo products summed
    apart give (11.7, 15.3, 19.6, 17.5, 21.3) and what they give in one
    accumulator (19.3, 18.8, 24.7, 24.0, 29.5); the sums have a fixed order."""
    torch = torch_cuda()
    G, hd, differ, total = shape.n_kv_heads, shape.head_dim, 0, 0
    W = synth.make_weights(shape, n_layers=1)
    gain = 1.0 + 0.1 * np.random.default_rng(79).standard_normal(shape.d_model, dtype=np.float32)
    W["layers"][0]["attn_norm"] = synth.f32_to_bf16_bits(gain)  # (x = embedding times gain: a lo part that is not 0)
    dw = binding.DeviceWeights(shape, W)
    up = lambda bits: kv_to_device(np.asarray(bits), "bf16").double()  # noqa: E731
    lw = {k: up(W["layers"][0][k]) for k in ("attn_norm", "wk", "wv")}
    m = binding.Model(dw, 1, max_rows=rows, max_ctx=1024)
    n = max(rows, -(-400000 // (2 * G * hd)) // rows * rows)  # (whole passes; at least 400000 values)
    half, pos = hd // 2, torch.arange(rows, dtype=torch.float64, device="cuda")
    inv = shape.rope_base ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / hd)
    c, s = torch.cos(pos[:, None] * inv)[:, None], torch.sin(pos[:, None] * inv)[:, None]
    for i in range(n // rows):
        kv = binding.KVCache(m, 1, 1024)
        tok = synth.make_prompt(rows + 1, shape.vocab, batch=1, seed=80 + i)
        binding.specdec_prefill(m, kv, i32(tok))
        x = up(np.asarray(W["embed"])[tok[0, :rows]])
        x = x / torch.sqrt((x * x).mean(-1, keepdim=True) + shape.rms_eps) * lw["attn_norm"]
        k, v = ((x @ lw[w].t()).reshape(rows, G, hd) for w in ("wk", "wv"))
        k = torch.cat([k[..., :half] * c - k[..., half:] * s, k[..., half:] * c + k[..., :half] * s], -1)
        for got, ref in zip(kv.read_context(0, 0, 0, rows), (k, v)):
            differ += int((got != ref.float().to(torch.bfloat16)).sum())
            total += ref.numel()
    log(f"rows {rows}: {differ} of {total} values differ, {1e5 * differ / total:.1f} per 1e5")
    assert differ <= limit * total / 1e5


# (the tile kernel: more than 64 rows, row tiles of 96, 128 and 256 with remainders, launches of 1024 rows)
@pytest.mark.parametrize("B,g", [(13, 4), (16, 4), (12, 7), (97, 0), (16, 7), (43, 2), (50, 5), (75, 7), (130, 7)])
def test_odd_shape_tile_rows(B, g):
    _rows_case(ODD, 2, [1 + (37 * b) % 90 for b in range(B)], g, seed=B)


@pytest.mark.parametrize("B,g", [(3, 5), (8, 4), (8, 6), (16, 3), (9, 7), (16, 6), (32, 7), (56, 8)])
def test_7b_width_rows(B, g):
    _rows_case(synth.LLAMA_7B, 1, [40 + 13 * b for b in range(B)], g, seed=B)


# (INT4 groups of 128 columns: 192 and 352 leave a partial group, and a split or a wave without one)
@pytest.mark.parametrize("B,g", [(17, 0), (4, 7), (11, 2), (6, 7), (7, 6), (8, 7)])
def test_int4_odd_shape_rows(B, g):
    _int4_case(ODD, 2, [1 + (37 * b) % 90 for b in range(B)], g, seed=B)


@pytest.mark.parametrize("B,g", [(3, 5), (8, 4), (16, 3)])
def test_int4_7b_width_rows(B, g):
    _int4_case(synth.LLAMA_7B, 1, [40 + 13 * b for b in range(B)], g, seed=B)


# The long-context attention (more 32-key sub-chunks times (sequence, kv head, 16-query tile) units than 12 per CU): 32-dim
# heads with one and with two query tiles per unit, more sequences than a wave has lanes, few units over many blocks (one
# sequence: 2 units of 1600 sub-chunks, 62 parts) and units that end at, before and after a block's border
@pytest.mark.parametrize("B,g,lo,hi", [(130, 3, 340, 460), (97, 7, 300, 420), (70, 0, 700, 1100), (1, 4, 51100, 51100),
                                       (3, 7, 8000, 11000)])
def test_odd_shape_long_contexts(B, g, lo, hi):
    lengths = [lo + (hi - lo) * ((7 * b + 3) % B) // max(B - 1, 1) for b in range(B)]
    n_mt, cus = -(-(g + 1) * 3 // 16), torch_cuda().cuda.get_device_properties(0).multi_processor_count
    assert -(-(max(lengths) + g + 1) // 32) * B * 2 * n_mt > 12 * cus  # (the rule of the dispatch)
    _rows_case(ODD, 1, lengths, g, seed=B)


def test_long_contexts_with_an_invalid_last_row():
    """A drafted token out of range in the last row of some sequences: their keys
    are counted by the pass's bound then.  The status says so; all other rows
    keep their logits (another cut into blocks: to float32 rounding)."""
    torch = torch_cuda()
    B, g, bad = 130, 3, (0, 63, 64, 101, 129)
    lengths = [340 + (37 * b) % 120 for b in range(B)]
    cap = 512
    dw = binding.DeviceWeights(ODD, synth.make_weights(ODD, n_layers=1))
    m = binding.Model(dw, 1, max_rows=B * (g + 1), max_ctx=cap)
    kv = binding.KVCache(m, B, cap)
    install_context(kv, synth.make_kv_context(ODD, 1, lengths, seed=73), lengths, 1, ODD.dtype)
    pend = synth.make_prompt(1, ODD.vocab, batch=B, seed=74)[:, 0]
    drafts = synth.make_prompt(g, ODD.vocab, batch=B, seed=75).copy()
    out, status = [], []
    for invalid in (False, True):
        if invalid:
            drafts[list(bad), g - 1] = ODD.vocab
        kv.set_state(lengths, np.stack([np.zeros(B, np.int32), pend], 1), np.ones(B, np.int32))
        logits = torch.empty((B, g + 1, ODD.vocab), dtype=torch.float32, device="cuda")
        binding.specdec_verify(m, kv, g, i32(drafts), g, logits)
        out.append(logits.cpu().numpy())
        status.append(kv.read_state()["status"])
    assert status == [0, -7]
    keep = np.ones((B, g + 1), bool)
    keep[list(bad), g] = False
    rel = float(np.linalg.norm(out[1][keep] - out[0][keep]) / np.linalg.norm(out[0][keep]))
    log(f"invalid last rows: relative difference of the others {rel:.3g}")
    assert rel < REL


# (one pass of 1500 rows, two launches of the tile kernel; the shared-K/V attention with 32-dim heads, 3 query heads per
# kv head: 900 query rows in 15 blocks of 64, the last of them ragged; then ragged chunks of it)
@pytest.mark.parametrize("B,rows,n", [(5, 1500, 301), (7, 1470, 380)])
def test_odd_shape_prefill(monkeypatch, B, rows, n):
    monkeypatch.setattr(synth, "ODD", ODD, raising=False)
    _prefill_case("ODD", B, rows, n)
