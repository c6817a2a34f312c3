"""GPU parity of the projection and output GEMM (k_gemm) around the attention, through the module, against the float64 oracle.

Sizes at its edges: more token tiles than a launch holds wavefronts (each takes a second one), batch rows that are no whole tiles,
channels that do not fill the contraction (96 of 128, 160 of 256), feature tiles that pass through the ring of weight halves or
all fit, shares of feature tiles with a short last one; with the residual added in place the tokens of a repeated tile must be added once.
Tolerance as in the other parity tests; the residual form adds half an ulp of the sum, 2^-8 |ref|.
"""
import numpy as np
import pytest
import torch

import paper_2203_00854_amd as P
from oracle import evoformer_attention as O
from paper_2203_00854_amd import inputs as I
from helpers import small_spec, f64_inputs, max_abs, rel_l2

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("mode,n_a,n_b,c,H,d,c_z,mask", [
    (I.MODE_COL, 30, 4200, 128, 4, 32, 0, "tail:3"),          # whole weights, 4200 token tiles of 4096 wavefronts
    (I.MODE_COL, 33, 2100, 96, 4, 8, 0, "none"),               # two tiles per batch row, the second almost empty
    (I.MODE_ROW, 20, 300, 160, 8, 32, 32, "tail:20"),         # 32 feature tiles through the ring
    (I.MODE_ROW, 90, 129, 256, 8, 16, 16, "random:0.9"),
    (I.MODE_TRI_START, 65, 65, 128, 4, 32, 0, "none"),        # the pair-bias tile as a share of its own
    (I.MODE_TRI_END, 290, 290, 64, 2, 16, 0, "outer:0.9"),
    (I.MODE_COL, 30, 2200, 128, 8, 32, 0, "tail:3"),          # 32 feature tiles at 128 channels, many tokens: all in one block would not fit LDS
    (I.MODE_TRI_START, 290, 290, 96, 16, 16, 0, "none"),      # 33 of them with the pair-bias tile
])
@pytest.mark.parametrize("residual", [False, True])
def test_shapes(mode, n_a, n_b, c, H, d, c_z, mask, residual):
    check(mode, n_a, n_b, c, H, d, c_z, mask, residual)


@pytest.mark.parametrize("mode,n_a,n_b,c,H,d,c_z,mask", [
    (I.MODE_COL, 5, 70, 96, 12, 8, 0, "none"),                # two of 128 channels' steps missing in both contractions, heads of 8 channels
    (I.MODE_ROW, 7, 40, 160, 10, 16, 32, "tail:7"),           # six of sixteen, heads of 16
    (I.MODE_ROW, 9, 33, 224, 7, 32, 32, "random:0.8"),        # two of sixteen, heads of 32
    (I.MODE_TRI_END, 37, 37, 32, 1, 32, 0, "none"),           # two steps, one tile of each kind
])
@pytest.mark.parametrize("residual", [False, True])
def test_contraction_lengths(mode, n_a, n_b, c, H, d, c_z, mask, residual):
    """Channels and head channels that leave steps of the contraction empty, at each head dim (the step to the next operand differs)."""
    check(mode, n_a, n_b, c, H, d, c_z, mask, residual)


@pytest.mark.parametrize("mode,n_a,n_b,c,H,d,c_z,mask", [
    (I.MODE_ROW, 8, 48, 256, 8, 32, 32, "tail:3"),            # shares of one tile; two blocks along the tokens on eight XCDs
    (I.MODE_TRI_START, 43, 43, 128, 4, 32, 0, "outer:0.9"),   # seventeen tiles, the last share the pair bias alone
    (I.MODE_COL, 100, 100, 256, 8, 32, 0, "tail:9"),          # five shares of seven tiles: they begin inside q, k, v and gate
    (I.MODE_ROW, 3, 500, 256, 8, 16, 16, "none"),             # a token block that is mostly empty
    (I.MODE_COL, 40, 830, 256, 8, 32, 0, "none"),             # more token tiles than resident wavefronts, in shares
])
@pytest.mark.parametrize("residual", [False, True])
def test_shares(mode, n_a, n_b, c, H, d, c_z, mask, residual):
    """How the feature tiles are shared out over blocks, and the blocks over the XCDs."""
    check(mode, n_a, n_b, c, H, d, c_z, mask, residual)


def check(mode, n_a, n_b, c, H, d, c_z, mask, residual):
    case = I.make_case(small_spec(mode, n_a, n_b, c, H, d, c_z=c_z, dtype="bf16", mask=mask))
    desc, w, x, z, m = P.to_device(case, DEV)
    ws = torch.full((P.ff_attention_workspace_bytes(desc, 0),), 0xFF, dtype=torch.uint8, device=DEV)      # (NaN patterns)
    if residual:
        got = P.ff_gated_attention_residual(desc, w, x, z, m, out=x, ws=ws)
    else:
        got = P.ff_gated_attention(desc, w, x, z, m, ws=ws)
    torch.cuda.synchronize()
    assert P.ff_attention_last_path() == "mfma_bf16"
    got = got.float().cpu().numpy().astype(np.float64)
    fx, fz, fm, fw = f64_inputs(case)
    ref = O.gated_attention(mode, fx, fz, fm, fw, case.spec.heads, case.spec.ln_eps)
    if residual:
        ref = ref + fx
    ma, rl = max_abs(got, ref), rel_l2(got, ref)
    print(f"{case.spec.name} residual={residual}: max_abs={ma:.3e} rel_l2={rl:.3e}", flush=True)
    assert np.isfinite(got).all()
    assert np.all(np.abs(got - ref) <= 2e-2 + (2.0 ** -8 * np.abs(ref) if residual else 0.0)), ma
    assert rl <= 1e-2, rl
