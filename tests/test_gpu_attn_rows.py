"""GPU parity of k_attn_rows (attention outside the sequences of k_proj_attn) against the float64 oracle.

Sizes at its edges: one key, remainders of 32 keys, of four query tiles per block and of the two / four batch rows of a
wavefront, more than eight row blocks, a last ring slot of every index; masks that empty whole key tiles or rows; logits
far outside the range in which a softmax needs no reference.
"""
import numpy as np
import pytest
import torch

import paper_2203_00854_amd as P
from oracle import evoformer_attention as O
from paper_2203_00854_amd import inputs as I
from helpers import small_spec, f64_inputs, max_abs, patchy_mask, poison_masked_tokens, rel_l2

pytestmark = pytest.mark.gpu

ROW, COL, TS, TE = I.MODE_ROW, I.MODE_COL, I.MODE_TRI_START, I.MODE_TRI_END
DEV = "cuda:0"


def run(case, chunk=0):
    desc, w, x, z, mask = P.to_device(case, DEV)
    ws = torch.full((P.ff_attention_workspace_bytes(desc, chunk),), 0xFF, dtype=torch.uint8, device=DEV)      # (NaN patterns)
    out = P.ff_attention_chunked(desc, w, x, z, mask, chunk_rows=chunk, ws=ws) if chunk else P.ff_gated_attention(desc, w, x, z, mask, ws=ws)
    torch.cuda.synchronize()
    assert P.ff_attention_last_path() == "mfma_bf16"
    return out.float().cpu().numpy().astype(np.float64)


def check(case, got, what):
    x, z, m, w = f64_inputs(case)
    ref = O.gated_attention(case.spec.mode, x, z, m, w, case.spec.heads, case.spec.ln_eps)
    ma, rl = max_abs(got, ref), rel_l2(got, ref)
    print(f"{what}: max_abs={ma:.3e} rel_l2={rl:.3e}", flush=True)
    assert np.isfinite(got).all() and ma <= 2e-2 and rl <= 1e-2, (what, ma, rl)


@pytest.mark.parametrize("mode,n_a,n_b,c,H,c_z,mask,chunk", [
    (ROW, 3, 1, 64, 2, 16, "none", 0),
    (ROW, 5, 31, 32, 1, 16, "tail:3", 0),
    (ROW, 2, 65, 96, 3, 16, "random:0.7", 0),
    (ROW, 150, 97, 64, 8, 32, "tail:40", 0),                 # many row blocks; the last key tiles hold no valid key
    (ROW, 40, 300, 256, 8, 32, "random:0.9", 0),
    (ROW, 3, 513, 64, 2, 16, "tail:1", 0),
    (COL, 128, 5, 64, 2, 0, "none", 0),
    (COL, 290, 45, 256, 8, 0, "tail:30", 0),
    (TS, 127, 127, 128, 4, 0, "outer:0.9", 50),
    (TE, 257, 257, 64, 2, 0, "none", 0),
    (TS, 275, 275, 128, 4, 0, "outer:0.95", 0),
])
@pytest.mark.parametrize("d", [8, 16, 32])
def test_shapes(mode, n_a, n_b, c, H, c_z, mask, chunk, d):
    H = H if H * d % 32 == 0 else 32 // d
    case = I.make_case(small_spec(mode, n_a, n_b, c, H, d, c_z=c_z, dtype="bf16", mask=mask))
    check(case, run(case, chunk), case.spec.name)


@pytest.mark.parametrize("mode,n_a,n_b,mask,chunk", [
    (COL, 1, 7, "none", 0), (COL, 32, 9, "tail:3", 0), (COL, 33, 6, "random:0.6", 0), (COL, 64, 301, "tail:40", 0), (COL, 63, 5, "none", 2),
    (ROW, 7, 64, "random:0.8", 0), (ROW, 6, 33, "tail:1", 0), (TS, 64, 64, "outer:0.9", 15), (TE, 50, 50, "none", 0)])
@pytest.mark.parametrize("d", [8, 16, 32])
def test_one_or_two_query_tiles(mode, n_a, n_b, mask, chunk, d):
    """Up to 64 positions: blocks of two wavefronts, a ring of two steps."""
    case = I.make_case(small_spec(mode, n_a, n_b, 64, 4, d, c_z=16, dtype="bf16", mask=mask))
    check(case, run(case, chunk), case.spec.name)


@pytest.mark.parametrize("n_a,n_b,d", [(3, 70, 32), (300, 260, 32), (5, 150, 8), (300, 100, 16), (7, 200, 32)])
def test_logits_far_from_zero(n_a, n_b, d):
    """The softmax runs without a reference while the denominator stays inside [2^-60, 2^96].  An offset of the pair bias moves all
    logits of a head by the same amount (which the softmax removes): heads at about -140, +140, -50 and +50 log2 units, the
    first two outside that range; one batch row is fully masked.  (200 positions at d = 32: k_proj_attn, which does the same.)"""
    case = I.make_case(small_spec(ROW, n_a, n_b, 64, 4, d, c_z=16, dtype="bf16", mask="random:0.8"))
    case.mask[1, :] = 0.0
    case.weights["lnz_b"] = I.to_storage(np.full(16, 4.0), "bf16")
    wb = I.widen(case.weights["w_b"]).astype(np.float64)
    for h, shift in enumerate((-97.0, 97.0, -35.0, 35.0)):
        wb[h] += shift / 64.0
    case.weights["w_b"] = I.to_storage(wb, "bf16")
    check(case, run(case), f"{n_a} x {n_b}, d {d}")


@pytest.mark.parametrize("n_a,n_b,d,live", [(6, 160, 8, 64), (6, 160, 16, 96), (5, 128, 32, 32), (9, 320, 32, 288), (4, 256, 32, 192)])
def test_content_of_masked_tail_tiles_is_irrelevant(n_a, n_b, d, live):
    """NaN tokens in the last key tiles of 32, which hold no valid key in any row, and in a whole masked row: the other tokens'
    results are those of finite tokens there, bit for bit."""
    case = I.make_case(small_spec(ROW, n_a, n_b, 64, 4, d, c_z=16, dtype="bf16"))
    case.mask = np.ones((n_a, n_b), np.float32)
    case.mask[:, live:] = 0.0
    case.mask[3, :] = 0.0
    desc, w, x, z, mask = P.to_device(case, DEV)
    a = P.ff_gated_attention(desc, w, x, z, mask)
    x2 = x.clone()
    x2[mask == 0] = float("nan")
    b = P.ff_gated_attention(desc, w, x2, z, mask)
    torch.cuda.synchronize()
    assert P.ff_attention_last_path() == "mfma_bf16"
    assert torch.isfinite(a).all() and torch.equal(a[mask != 0], b[mask != 0])


@pytest.mark.parametrize("mode,n_a,n_b,d", [(ROW, 14, 160, 8), (ROW, 14, 160, 16), (ROW, 14, 100, 32), (ROW, 300, 260, 32), (COL, 330, 9, 8), (ROW, 9, 160, 32),
                                            (COL, 250, 13, 32), (TS, 300, 300, 32), (TE, 140, 140, 32), (TS, 90, 90, 16)])
def test_content_of_masked_tokens_is_irrelevant(mode, n_a, n_b, d):
    """NaN and infinities in masked tokens where the batch rows of a wavefront have their valid keys in different tiles: lead, gap,
    tail and single keys (129 .. 256 positions at d = 32: k_proj_attn)."""
    case = I.make_case(small_spec(mode, n_a, n_b, 64, 4, d, c_z=16, dtype="bf16"))
    if mode in (TS, TE):
        keep = patchy_mask(4, n_a)[3]
        keep[32:64] = 0.0
        mask = np.outer(keep, keep)
    else:
        mask = patchy_mask(n_a, n_b) if mode == ROW else patchy_mask(n_b, n_a).T
    bad = poison_masked_tokens(case, mask)
    x, z, m, w = f64_inputs(case)
    ref = O.gated_attention(mode, x, z, m, w, 4, case.spec.ln_eps)
    case.x = bad
    live = case.mask != 0
    got = run(case)[live]
    assert np.isfinite(got).all()
    assert max_abs(got, ref[live]) <= 2e-2 and rel_l2(got, ref[live]) <= 1e-2


@pytest.mark.parametrize("n_a,n_b,d", [(6, 70, 32), (5, 150, 8), (9, 100, 16), (7, 200, 32)])
def test_values_that_overflow_unnormalised_sums(n_a, n_b, d):
    """Weights up to 2^85 or so, which pass as they are, times values of about 2^60: the sum over the keys leaves float32 although
    the weighted mean does not."""
    case = I.make_case(small_spec(ROW, n_a, n_b, 64, 4, d, c_z=16, dtype="bf16", mask="random:0.8"))
    case.weights["lnz_b"] = I.to_storage(np.full(16, 4.0), "bf16")
    wb = I.widen(case.weights["w_b"]).astype(np.float64)
    for h, shift in enumerate((50.0, 45.0, -30.0, 0.0)):
        wb[h] += shift / 64.0
    case.weights["w_b"] = I.to_storage(wb, "bf16")
    case.weights["w_v"] = I.to_storage(I.widen(case.weights["w_v"]).astype(np.float64) * 2.0 ** 60, "bf16")
    got = run(case) * 2.0 ** -60
    x, z, m, w = f64_inputs(case)
    ref = O.gated_attention(ROW, x, z, m, w, 4, case.spec.ln_eps) * 2.0 ** -60
    assert np.isfinite(got).all()
    assert max_abs(got, ref) <= 2e-2 and rel_l2(got, ref) <= 1e-2
