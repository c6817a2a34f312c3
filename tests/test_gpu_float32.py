"""GPU parity of the float32 kernel family at the edges of its tiles: 32-query tiles and blocks of eight of them, keys in
more than one LDS portion, head dimensions around the 8- and 32-channel groups, contraction lengths around the chunks
of 32, rows that are no multiple of four elements, LayerNorm rows in and beyond registers.

Tolerance: max-abs 1e-4, the benchmark definition's for float32 (measured: below 2e-6).  The bfloat16 cases run the
same kernels on bfloat16 storage (shapes the bfloat16 matrix-core family does not take, or a token pointer that is not
16-byte aligned): max-abs 2e-2, relative L2 1e-2.
"""
import numpy as np
import pytest
import torch

import paper_2203_00854_amd as P
from oracle import evoformer_attention as O
from paper_2203_00854_amd import inputs as I
from helpers import f64_inputs, max_abs, patchy_mask, poison_masked_tokens, rel_l2, small_spec

pytestmark = pytest.mark.gpu
ROW, COL, TS, TE = I.MODE_ROW, I.MODE_COL, I.MODE_TRI_START, I.MODE_TRI_END

SHAPES = [   # mode, n_a, n_b, c, c_z, heads, d, mask, chunk
    (ROW, 1, 1, 1, 1, 1, 1, "none", 0), (ROW, 3, 31, 32, 8, 2, 8, "tail:3", 0), (ROW, 2, 32, 36, 12, 3, 16, "none", 0),
    (ROW, 5, 33, 64, 20, 2, 32, "random:0.7", 2), (COL, 65, 3, 30, 0, 2, 24, "random:0.8", 2), (TS, 66, 66, 31, 0, 3, 5, "outer:0.9", 0),
    (TE, 40, 40, 48, 0, 2, 33, "outer:0.8", 7), (COL, 289, 2, 64, 0, 2, 32, "tail:30", 0), (ROW, 2, 257, 32, 16, 2, 128, "tail:20", 0),
    (COL, 530, 3, 300, 0, 2, 64, "random:0.9", 0), (ROW, 9, 70, 520, 264, 9, 8, "none", 4), (ROW, 100, 130, 128, 64, 8, 16, "tail:2", 0),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mode,n_a,n_b,c,c_z,heads,d,mask,chunk", SHAPES)
def test_edges(dtype, mode, n_a, n_b, c, c_z, heads, d, mask, chunk):
    spec = small_spec(mode, n_a, n_b, c, heads, d, c_z=c_z, dtype=dtype, mask=mask, chunk_rows=chunk)
    case = I.make_case(spec)
    desc, w, x, z, m = P.to_device(case, "cuda:0")
    if P.ff_attention_path(desc) != "generic":        # (the bfloat16 matrix-core family wants 16-byte aligned pointers)
        x = torch.cat([x.new_zeros(4), x.flatten()])[4:].view_as(x)
    ws = torch.full((P.ff_attention_workspace_bytes(desc, chunk),), 0xFF, dtype=torch.uint8, device="cuda:0")   # NaN patterns
    if chunk:
        got = P.ff_attention_chunked(desc, w, x, z, m, chunk_rows=chunk, ws=ws)
    else:
        got = P.ff_gated_attention(desc, w, x, z, m, ws=ws)
    torch.cuda.synchronize()
    assert P.ff_attention_last_path() == "generic"
    xf, zf, mf, wf = f64_inputs(case)
    ref = O.gated_attention(mode, xf, zf, mf, wf, heads, spec.ln_eps)
    g = got.float().cpu().numpy().astype(np.float64)
    ma, rl = max_abs(g, ref), rel_l2(g, ref)
    print(f"{spec.name}: max_abs={ma:.3e} rel_l2={rl:.3e}", flush=True)
    assert np.isfinite(g).all()
    if dtype == "f32":
        assert ma <= 1e-4
    else:
        assert ma <= 2e-2 and rl <= 1e-2


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mode,n_a,n_b,c,heads,d", [(ROW, 13, 70, 32, 2, 12), (COL, 290, 7, 30, 2, 40), (ROW, 6, 5, 20, 1, 5), (TE, 75, 75, 36, 2, 20)])
def test_content_of_masked_tokens_is_irrelevant(dtype, mode, n_a, n_b, c, heads, d):
    """NaN and infinities in masked tokens, whole tiles of keys and single ones: a masked key has weight exactly 0, so every other
    token's result is that of a finite token there."""
    case = I.make_case(small_spec(mode, n_a, n_b, c, heads, d, c_z=12, dtype=dtype))
    if mode == TE:
        keep = patchy_mask(4, n_a)[3]
        mask = np.outer(keep, keep)
    else:
        mask = patchy_mask(n_a, n_b) if mode == ROW else patchy_mask(n_b, n_a).T
    bad = poison_masked_tokens(case, mask)
    xf, zf, mf, wf = f64_inputs(case)
    ref = O.gated_attention(mode, xf, zf, mf, wf, heads, case.spec.ln_eps)
    case.x = bad
    desc, w, x, z, m = P.to_device(case, "cuda:0")
    got = P.ff_gated_attention(desc, w, x, z, m).float().cpu().numpy().astype(np.float64)
    assert P.ff_attention_last_path() == "generic"
    live = case.mask != 0
    assert np.isfinite(got[live]).all()
    assert max_abs(got[live], ref[live]) <= (1e-4 if dtype == "f32" else 2e-2)


@pytest.mark.parametrize("mode,n_a,n_b,c,c_z,heads,d,limit", [
    (ROW, 8, 32, 32, 16, 4, 8, 2.30e-7), (ROW, 16, 200, 64, 32, 4, 16, 2.65e-7), (ROW, 40, 155, 256, 128, 8, 32, 4.85e-7),
    (TE, 96, 96, 256, 0, 8, 32, 4.92e-7), (TS, 120, 120, 32, 0, 4, 8, 2.42e-7)])
def test_rounding_of_the_float32_sums(mode, n_a, n_b, c, c_z, heads, d, limit):
    """Relative error against float64.  limit: that of vector multiply-adds, a chain per output and the keys of a query spread over 64
    lanes (measured with such kernels on these inputs); one chain per output on the matrix instruction, with the bias
    as its starting value and all keys in a row, has 2.56, 3.48, 5.61, 5.61 and 2.97e-7."""
    spec = small_spec(mode, n_a, n_b, c, heads, d, c_z=c_z, dtype="f32")
    case = I.make_case(spec)
    desc, w, x, z, m = P.to_device(case, "cuda:0")
    got = P.ff_gated_attention(desc, w, x, z, m).cpu().numpy().astype(np.float64)
    assert P.ff_attention_last_path() == "generic"
    xf, zf, mf, wf = f64_inputs(case)
    rl = rel_l2(got, O.gated_attention(mode, xf, zf, mf, wf, heads, spec.ln_eps))
    print(f"{spec.name}: rel_l2={rl:.3e}", flush=True)
    assert rl <= limit


@pytest.mark.parametrize("mode,n_a,n_b,c,c_z,heads,d,limit", [
    (ROW, 8, 32, 32, 16, 4, 8, 1.81e-7), (ROW, 16, 200, 64, 32, 4, 16, 1.91e-7), (ROW, 40, 155, 256, 128, 8, 32, 2.53e-7), (TE, 96, 96, 256, 0, 8, 32, 2.60e-7),
    (TS, 120, 120, 32, 0, 4, 8, 1.90e-7), (COL, 70, 20, 128, 0, 4, 32, 1.90e-7), (ROW, 4, 601, 64, 32, 4, 16, 1.76e-7), (TS, 60, 60, 36, 0, 3, 20, 2.16e-7),
    (COL, 150, 9, 300, 0, 2, 64, 2.02e-7), (ROW, 6, 90, 30, 16, 2, 128, 2.13e-7), (TE, 40, 40, 512, 0, 8, 32, 3.15e-7), (ROW, 2, 1030, 32, 16, 4, 8, 1.75e-7),
    (COL, 33, 300, 261, 0, 3, 40, 2.39e-7), (ROW, 100, 130, 128, 64, 8, 16, 2.30e-7)])
def test_rounding_of_the_split_sums(mode, n_a, n_b, c, c_z, heads, d, limit):
    """Relative error against float64 of the sums of bfloat16 planes.  limit: 1.08 times the measured one, for another order of the sums; the float32
    matrix instruction in two sums per output has 2.15, 2.33, 3.82, 3.90, 2.22, 3.02, 2.15, 2.61, 3.39, 3.34, 5.06, 1.89, 3.91 and 3.16e-7 on these
    inputs, so that a loss of any of the six products of planes or a return to that instruction's error shows."""
    spec = small_spec(mode, n_a, n_b, c, heads, d, c_z=c_z, dtype="f32")
    case = I.make_case(spec)
    desc, w, x, z, m = P.to_device(case, "cuda:0")
    got = P.ff_gated_attention(desc, w, x, z, m).cpu().numpy().astype(np.float64)
    assert P.ff_attention_last_path() == "generic"
    xf, zf, mf, wf = f64_inputs(case)
    rl = rel_l2(got, O.gated_attention(mode, xf, zf, mf, wf, heads, spec.ln_eps))
    print(f"{spec.name}: rel_l2={rl:.3e}", flush=True)
    assert rl <= limit


def intervals(desc, w, x, z, m, chunk=0):
    """How often the launch timer saw the family in one call."""
    P.ff_profile_enable(True)
    if chunk:
        P.ff_attention_chunked(desc, w, x, z, m, chunk_rows=chunk)
    else:
        P.ff_gated_attention(desc, w, x, z, m)
    torch.cuda.synchronize()
    n = P.ff_profile_collect()["generic family"][1]
    P.ff_profile_enable(False)
    return n


# The form of the projections: statistics and weights in the blocks themselves (one), weights split ahead (planes) or per block (blocks)
ONE, PLANES, BLOCKS = "one", "planes", "blocks"


def projections(mode, n_a, n_b, c, heads, d, chunk):
    """The form that an unchunked call (chunk = 0) or chunks of so many batch rows take, of aligned float32 tensors and 256 compute units."""
    rows, length = (n_a, n_b) if mode in (ROW, TS) else (n_b, n_a)
    tokens, feat = min(chunk or rows, rows) * length, 4 * heads * d
    blocks, tri = -(-tokens // 64) * -(-feat // 64), mode in (TS, TE)
    if blocks <= 1024 and (mode == COL or length ** 2 <= 40 * 32 * 256):
        if c <= 256 or (tri and heads >= 2 and 2 * blocks <= (5 if heads > 2 else 2) * 256 and tokens * blocks <= 64 * 256 ** 2):
            return ONE
    return PLANES if c % 32 == 0 and 6 * (-(-feat // 128) * 128) * c <= tokens * heads * d * 4 else BLOCKS


@pytest.mark.parametrize("mode,n_a,n_b,c,heads,d,chunk,forms", [      # forms: unchunked, chunks of `chunk`, chunks of one row
    (ROW, 12, 33, 64, 2, 32, 0, (ONE, ONE, ONE)), (ROW, 11, 33, 64, 2, 32, 0, (ONE, ONE, ONE)),
    (ROW, 24, 45, 32, 3, 16, 5, (ONE, ONE, ONE)), (COL, 37, 40, 96, 1, 40, 13, (ONE, ONE, ONE)),
    (TS, 200, 200, 160, 2, 64, 0, (PLANES, PLANES, ONE)), (TE, 90, 90, 32, 5, 8, 90, (ONE, ONE, ONE)), (ROW, 640, 129, 32, 4, 8, 0, (PLANES, PLANES, ONE)),
    (ROW, 3, 572, 30, 2, 8, 2, (ONE, ONE, ONE)), (ROW, 3, 573, 32, 2, 12, 2, (PLANES, PLANES, PLANES)), (ROW, 50, 70, 300, 1, 8, 0, (BLOCKS, BLOCKS, BLOCKS)),
    (ROW, 3, 600, 128, 4, 32, 2, (PLANES, PLANES, BLOCKS)),              # 128 channels: 768 tokens hold the planes
    (COL, 10, 84, 288, 2, 16, 2, (BLOCKS, BLOCKS, BLOCKS)), (COL, 10, 200, 288, 2, 16, 173, (PLANES, PLANES, BLOCKS)),      # 1728 tokens
    (COL, 60, 100, 1024, 16, 32, 11, (BLOCKS, BLOCKS, BLOCKS)),          # blocks of 128 features, weights split by each
    (ROW, 640, 129, 36, 4, 8, 64, (BLOCKS, ONE, ONE)), (ROW, 640, 129, 33, 4, 8, 64, (BLOCKS, ONE, ONE)),                   # rows of whole pieces, and not
    (COL, 33, 30, 260, 3, 8, 4, (BLOCKS, BLOCKS, BLOCKS)), (COL, 33, 30, 261, 3, 8, 4, (BLOCKS, BLOCKS, BLOCKS)), (TS, 104, 104, 288, 4, 8, 40, (ONE, ONE, ONE))])
def test_weights_split_ahead_and_chunks(mode, n_a, n_b, c, heads, d, chunk, forms):
    """Statistics in the projections' launch or ahead of it, weights split once per chunk where the chunk has tokens enough or else by every block, blocks
    of 64 and 128 features: every form against float64, and all of them bit for bit the same."""
    assert forms == tuple(projections(mode, n_a, n_b, c, heads, d, k) for k in (0, chunk, 1))
    case = I.make_case(small_spec(mode, n_a, n_b, c, heads, d, c_z=16, dtype="f32", mask="none"))
    desc, w, x, z, m = P.to_device(case, "cuda:0")
    got = P.ff_gated_attention(desc, w, x, z, m)
    assert P.ff_attention_last_path() == "generic"
    assert (intervals(desc, w, x, z, m) == 1) == (forms[0] == ONE)
    for rows in {1, chunk} - {0}:
        assert torch.equal(P.ff_attention_chunked(desc, w, x, z, m, chunk_rows=rows), got)
    # an address that is no multiple of sixteen takes the form of rows of no whole pieces, which splits per block
    odd = torch.cat([x.new_zeros(1), x.flatten()])[1:].view_as(x)
    assert torch.equal(P.ff_gated_attention(desc, w, odd, z, m), got)
    if n_a * n_b <= 20000:
        xf, zf, mf, wf = f64_inputs(case)
        ref = O.gated_attention(mode, xf, zf, mf, wf, heads, case.spec.ln_eps)
        assert rel_l2(got.cpu().numpy().astype(np.float64), ref) <= 5e-7      # (above the largest limit of the sums' rounding)


def test_large_and_small_magnitudes():
    """Scales far from one pass through the splitting as they do through float32: LayerNorm takes the scale of x away, that of w_v and w_o remains."""
    case = I.make_case(small_spec(ROW, 9, 40, 64, 2, 32, c_z=16, dtype="f32", mask="none"))
    desc, w, x, z, m = P.to_device(case, "cuda:0")
    w = dict(w, b_o=torch.zeros_like(w["b_o"]))
    base = P.ff_gated_attention(desc, w, x, z, m).clone()
    for s in (2.0 ** 60, 2.0 ** -60):
        big = P.ff_gated_attention(desc, dict(w, w_v=w["w_v"] * s, w_o=w["w_o"] * 2.0 ** -20), x, z, m)
        assert torch.equal(big, base * (s * 2.0 ** -20))


def same_values(got, ref, tol):
    """got against a float64 reference that holds infinities and NaN: those in the same places, the rest within tol of the largest."""
    with np.errstate(invalid="ignore"):
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        assert np.array_equal(np.isinf(got), np.isinf(ref))
        assert np.array_equal(np.sign(got[np.isinf(ref)]), np.sign(ref[np.isinf(ref)]))
    fin = np.isfinite(ref)
    if fin.any():
        assert max_abs(got[fin], ref[fin]) <= tol * max(1.0, np.abs(ref[fin]).max())


# one launch for statistics and projections; 64 and 128 features per block; split ahead and per block; head dims of every kernel;
# the last tile of tokens, features, keys and channels partly filled
INF_SHAPES = [(ROW, 3, 45, 64, 2, 8, 0), (COL, 70, 5, 36, 3, 12, 2), (ROW, 90, 130, 96, 3, 32, 0), (TS, 100, 100, 260, 4, 24, 0), (TE, 66, 66, 33, 1, 64, 0),
              (ROW, 4, 601, 64, 3, 16, 1), (ROW, 5, 170, 40, 2, 128, 2), (ROW, 61, 136, 32, 8, 32, 7), (COL, 8, 4100, 256, 1, 8, 1000)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("where", ["w_g", "w_v", "w_o"])
@pytest.mark.parametrize("mode,n_a,n_b,c,heads,d,chunk", INF_SHAPES)
def test_infinite_weights(dtype, where, mode, n_a, n_b, c, heads, d, chunk):
    """An infinity in a weight does what it does to float32 products and sums: a gate of exactly 0 or 1, an infinite value channel, infinite
    outputs of the sign of their product, NaN only where an infinity meets a zero or its opposite.  (Channel 0 is positive in every normalised token, so
    that an infinite weight there gives one sign.)"""
    case = I.make_case(small_spec(mode, n_a, n_b, c, heads, d, c_z=16, dtype=dtype, mask="none"))
    hd = heads * d
    w = {k: v.copy() for k, v in case.widened_weights().items()}
    w["ln_b"][0] = 24.0
    if where == "w_g":
        w["w_g"][0, 0], w["w_g"][hd - 1, 0] = -np.inf, np.inf
    elif where == "w_v":
        w["w_v"][hd // 2, 0] = np.inf
    else:
        w["w_v"][hd - 1, 0] = 1.0               # (its context is far from zero: the sign of the infinity is certain)
        w["w_o"][c - 1, hd - 1] = -np.inf
    case.weights = {k: I.to_storage(v.astype(np.float32), dtype) for k, v in w.items()}
    desc, dw, x, z, m = P.to_device(case, "cuda:0")
    if P.ff_attention_path(desc) != "generic":
        x = torch.cat([x.new_zeros(4), x.flatten()])[4:].view_as(x)
    got = P.ff_gated_attention(desc, dw, x, z, m)
    assert P.ff_attention_last_path() == "generic"
    if chunk:
        assert torch.equal(P.ff_attention_chunked(desc, dw, x, z, m, chunk_rows=chunk).nan_to_num(5.0), got.nan_to_num(5.0))
    xf, zf, mf, wf = f64_inputs(case)
    with np.errstate(all="ignore"):
        ref = O.gated_attention(mode, xf, zf, mf, wf, heads, case.spec.ln_eps)
    same_values(got.float().cpu().numpy().astype(np.float64), ref, 1e-4 if dtype == "f32" else 2e-2)


@pytest.mark.parametrize("where", ["w_v", "w_o", "score", "masked"])
@pytest.mark.parametrize("mode,n_a,n_b,c,heads,d,chunk", INF_SHAPES)
def test_top_of_the_float32_range(where, mode, n_a, n_b, c, heads, d, chunk):
    """Finite values up to the largest float32: weights, products of huge and tiny factors, a key whose score is -infinity in float32 (weight
    exactly 0), and infinities and the like in masked tokens next to them."""
    case = I.make_case(small_spec(mode, n_a, n_b, c, heads, d, c_z=16, dtype="f32", mask="none"))
    hd, top = heads * d, np.finfo(np.float32).max
    w = {k: v.copy() for k, v in case.weights.items()}
    x = case.x.copy()
    w["b_o"][:] = 0
    if where == "w_o":
        w["w_v"] *= np.float32(2.0 ** -70)
        w["w_o"][:] = np.sign(w["w_o"]) * top * np.linspace(0.99, 1.0, c, dtype=np.float32)[:, None]
    elif where == "score":
        # token 1 of every batch row has nothing but channel 0, zero elsewhere: its key overflows to infinity, its product with every
        # query, negative there, to -infinity (-700 or less in float64)
        x[:, :, 0] = 0
        tok = x[:, 1] if mode in (ROW, TS) else x[1]
        tok[:] = 0
        tok[:, 0] = 1000.0
        w["ln_g"][:], w["ln_b"][:] = 1, 0
        w["ln_b"][1] = -8.0
        w["w_k"][::d] = 0
        w["w_k"][::d, 0] = top / np.sqrt(c - 1.0) * 1.01
        w["w_q"][::d] = 0
        w["w_q"][::d, 1] = 2.0 ** -118
    else:
        w["ln_g"] *= np.float32(2.0 ** -80)
        w["ln_b"] *= np.float32(2.0 ** -80)
        for k in ("w_q", "w_k", "w_g") + (("w_b",) if mode in (TS, TE) else ()):
            w[k] *= np.float32(2.0 ** 80)
        w["w_v"][:] = np.sign(w["w_v"]) * top * np.linspace(0.99, 1.0, hd, dtype=np.float32)[:, None]
        w["w_o"] *= np.float32(2.0 ** -48)
    case.weights, case.x = w, x
    bad = x
    if where == "masked":
        bad = poison_masked_tokens(case, np.random.default_rng(3).random((n_a, n_b)) < 0.7)
        if mode in (TS, TE):           # (a masked token is an entry of the pair bias of all rows: finite there)
            bad = case.x
    xf, zf, mf, wf = f64_inputs(case)
    case.x = bad
    desc, dw, dx, z, m = P.to_device(case, "cuda:0")
    got = P.ff_gated_attention(desc, dw, dx, z, m)
    if chunk:
        assert torch.equal(P.ff_attention_chunked(desc, dw, dx, z, m, chunk_rows=chunk).nan_to_num(5.0), got.nan_to_num(5.0))
    got = got.cpu().numpy().astype(np.float64)
    ref = O.gated_attention(mode, xf, zf, mf, wf, heads, case.spec.ln_eps)
    if where == "masked":
        got, ref = got[mf != 0], ref[mf != 0]
    assert np.isfinite(got).all()
    # (scores of up to a hundred carry errors of 100 x 2^-23 where they are that large)
    assert rel_l2(got, ref) <= (3e-5 if where == "score" else 2e-6)


def test_gate_is_divided_exactly():
    """sigmoid(t) = 1 / (1 + exp(-t)) for t in [0, 8]: with the division rounded correctly its relative error is 3.80e-8 (root mean square of 20480
    values, good to 0.3 %), with the reciprocal instruction in its place 3.89e-8.  (One token, value 1 in every channel, the output
    projection the identity.)"""
    n = 512
    case = I.make_case(small_spec(COL, 1, 1, n, 16, 32, dtype="f32", mask="none"))
    for v in case.weights.values():
        v[...] = 0
    case.weights["ln_b"][:], case.weights["w_v"][:, 0], case.weights["w_o"][:] = 1, 1, np.eye(n)
    desc, w, x, z, m = P.to_device(case, "cuda:0")
    rng, sq = np.random.default_rng(0), []
    for _ in range(40):
        t = rng.uniform(0, 8, n).astype(np.float32)
        got = P.ff_gated_attention(desc, dict(w, b_g=torch.from_numpy(t).cuda()), x, z, m).cpu().numpy()[0, 0].astype(np.float64)
        sq.append((got * (1 + np.exp(-t.astype(np.float64))) - 1) ** 2)
    rms = float(np.sqrt(np.mean(sq)))
    print(f"relative error of a gate: {rms:.3e}", flush=True)
    assert rms <= 3.87e-8


@pytest.mark.parametrize("where", ["values", "tokens", "scores"])
@pytest.mark.parametrize("mode,n_a,n_b,c,heads,d,chunk", INF_SHAPES)
def test_bottom_of_the_float32_range(where, mode, n_a, n_b, c, heads, d, chunk):
    """Operands around 2^-120 against others around 2^120 lose no bits: the result is as accurate as without the factors (float32 products
    have 2.4e-7 to 2.9e-7 with and without; planes without the bits below 2^-133 have 4e-5 to 4e-4)."""
    case = I.make_case(small_spec(mode, n_a, n_b, c, heads, d, c_z=16, dtype="f32", mask="none"))
    w, f = case.weights, np.float32(2.0 ** 118)
    if where == "values":
        w["w_v"] /= f
        w["w_o"] *= f
    elif where == "tokens":
        for k in ("ln_g", "ln_b"):
            w[k] /= f
        for k in ("w_q", "w_k", "w_v", "w_g") + (("w_b",) if mode in (TS, TE) else ()):
            w[k] *= f
    else:
        w["w_q"] /= f
        w["w_k"] *= f
    desc, dw, x, z, m = P.to_device(case, "cuda:0")
    got = P.ff_gated_attention(desc, dw, x, z, m)
    if chunk:
        assert torch.equal(P.ff_attention_chunked(desc, dw, x, z, m, chunk_rows=chunk), got)
    xf, zf, mf, wf = f64_inputs(case)
    rl = rel_l2(got.cpu().numpy().astype(np.float64), O.gated_attention(mode, xf, zf, mf, wf, heads, case.spec.ln_eps))
    print(f"{case.spec.name} {where}: rel_l2={rl:.3e}", flush=True)
    assert rl <= 5e-7


@pytest.mark.parametrize("exponent", [-90, -112, -120, -127, -131])
@pytest.mark.parametrize("n_a,n_b,c,heads,d,dead", [(3, 45, 64, 2, 8, 0), (40, 200, 96, 3, 32, 0), (2, 70, 36, 1, 128, 0), (7, 90, 30, 2, 20, 11)])
def test_small_softmax_weights(n_a, n_b, c, heads, d, dead, exponent):
    """One key with a weight of 2^exponent of the others' and a value so large that both count alike in the context: weights below the normal range
    of float32, and ones whose lower planes are below that of bfloat16.  (The score's own rounding is |exponent| 2^-24, a weight of 2^-131 has 18 bits.)"""
    case = I.make_case(small_spec(ROW, n_a, n_b, c, heads, d, c_z=16, dtype="f32", mask="none"))
    half, w = c // 2, case.weights
    rng = np.random.default_rng(1)
    x = np.zeros_like(case.x)
    x[:, :, 2:half] = rng.integers(1, 9, (n_a, n_b, half - 2)) / 8
    x[:, :, half:] = -x[:, :, :half]                # means are exactly zero
    x[:, 1] = 0
    x[:, 1, 0], x[:, 1, half] = 1, -1               # the only live token with channel 0
    if dead:
        case.mask = np.ones((n_a, n_b), np.float32)
        x[:, n_b - dead:], case.mask[:, n_b - dead:] = x[:, 1:2], 0
    case.x = x
    w["ln_g"][:], w["ln_b"][:] = 1, 0
    w["ln_b"][1] = 8                                # channel 1 is 8 in every token
    w["b_o"][:] = w["w_b"][:] = w["w_q"][:] = w["w_k"][:] = 0
    w["w_q"][::d, 1] = 1
    w["w_k"][::d, 0] = exponent * np.log(2.0) * np.sqrt(d) / 8 / np.sqrt(half)
    w["w_v"][:, :2] = 0
    w["w_v"] *= np.float32(2.0 ** -34)
    w["w_v"][:, 0] = 2.0 ** (-34 - exponent)
    w["w_o"] *= np.float32(2.0 ** 34)
    desc, dw, dx, z, m = P.to_device(case, "cuda:0")
    got = P.ff_gated_attention(desc, dw, dx, z, m).cpu().numpy().astype(np.float64)
    xf, zf, mf, wf = f64_inputs(case)
    rl = rel_l2(got, O.gated_attention(ROW, xf, zf, mf, wf, heads, case.spec.ln_eps))
    print(f"weight 2^{exponent}: rel_l2={rl:.3e}", flush=True)
    assert rl <= 2e-5


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mode,n_a,n_b,c,heads,d,chunk,n", [(ROW, 8, 32, 36, 4, 8, 0, 1), (ROW, 8, 32, 36, 4, 8, 3, 3), (COL, 20, 9, 40, 1, 24, 4, 3),
                                                            (TS, 300, 300, 96, 3, 40, 0, 2), (ROW, 3, 573, 36, 2, 12, 2, 3)])
def test_launch_timer_counts_what_was_launched(dtype, mode, n_a, n_b, c, heads, d, chunk, n):
    """An interval per chunk, and one ahead of them only where something is launched there: small calls form the token statistics and the pair
    bias in the projections' launch."""
    case = I.make_case(small_spec(mode, n_a, n_b, c, heads, d, c_z=16, dtype=dtype))
    assert intervals(*P.to_device(case, "cuda:0"), chunk=chunk) == n


@pytest.mark.parametrize("dtype,mode,n_a,n_b,c,heads,d,n", [
    ("f32", COL, 40, 9, 256, 2, 8, 1), ("f32", COL, 40, 9, 260, 2, 8, 2), ("bf16", COL, 40, 9, 260, 2, 8, 2), ("f32", ROW, 7, 40, 260, 2, 8, 2),
    ("bf16", ROW, 7, 40, 260, 2, 8, 1), ("bf16", ROW, 7, 40, 261, 2, 8, 2), ("bf16", TS, 20, 20, 261, 2, 8, 1), ("f32", TE, 30, 30, 260, 3, 8, 1),
    ("f32", TS, 90, 90, 261, 4, 8, 1), ("f32", TS, 90, 90, 260, 4, 24, 2), ("f32", TS, 41, 41, 260, 9, 40, 1),
    ("f32", TS, 48, 48, 260, 9, 40, 2), ("f32", TE, 30, 30, 260, 2, 8, 1), ("f32", TE, 38, 38, 260, 2, 96, 2),
    ("f32", TE, 30, 30, 260, 1, 8, 2), ("f32", TE, 104, 104, 260, 4, 8, 1), ("f32", TE, 109, 109, 260, 4, 8, 2), ("bf16", TS, 66, 66, 261, 8, 20, 1),
    ("bf16", TS, 70, 70, 261, 8, 20, 2)])
def test_long_rows_have_a_launch_for_their_statistics(dtype, mode, n_a, n_b, c, heads, d, n):
    """Rows of more than 256 channels, which every block of 64 features would read two more times: a launch of their own, but where the pair
    bias is worth hiding behind the projections.  Both ways against float64."""
    case = I.make_case(small_spec(mode, n_a, n_b, c, heads, d, c_z=16, dtype=dtype))
    desc, w, x, z, m = P.to_device(case, "cuda:0")
    if P.ff_attention_path(desc) != "generic":
        x = torch.cat([x.new_zeros(4), x.flatten()])[4:].view_as(x)
    assert intervals(desc, w, x, z, m) == n
    got = P.ff_gated_attention(desc, w, x, z, m).float().cpu().numpy().astype(np.float64)
    xf, zf, mf, wf = f64_inputs(case)
    rl = rel_l2(got, O.gated_attention(mode, xf, zf, mf, wf, heads, case.spec.ln_eps))
    assert rl <= (5e-7 if dtype == "f32" else 1e-2)
