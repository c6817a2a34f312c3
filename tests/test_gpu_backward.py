"""GPU parity of the backward pass of the fused attention core (ff_attention_core_backward through the C ABI)
against the float64 oracle, element by element on the same seeded inputs.

Tolerance, per gradient tensor: relative L2 1e-2, and per element 2e-2 * scale + 2^-8 |ref| with scale the
tensor's root mean square (at least 1): gradients are sums of up to L (for dbias: rows x 1) products whose
size depends on dout, so the absolute bound of the forward modules (2e-2 for outputs of order one) is taken
relative to that scale, and the second term is the rounding of a large element itself (half a bfloat16 ulp
of the result, or of the summands of the bias gradient, is up to 2^-8 of the value).  The library rounds P, dS,
dctx and the results to bfloat16; logsumexp, delta and accumulators are float32.  Measured: relative L2 3e-3.
The bias gradient gets twice the absolute part: where one key takes nearly all the weight, dS = P (dP - delta) is
the difference of two numbers of size |dctx . v| (about 5 here) that agree to first order, so the 2^-9 relative
rounding of the bfloat16 operands dctx and v survives in absolute terms (up to 2.5e-2 on the 256-row case) however
small the result is, and the sum over the rows keeps the largest of them; every bfloat16 implementation of this
backward pass has that term.
"""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2203_00854_amd as P
from oracle import attention_core_backward as O
from paper_2203_00854_amd import binding as B
from paper_2203_00854_amd import inputs as I
from helpers import max_abs, rel_l2

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
NAMES = ("dq", "dk", "dv", "dg", "dbias")


def f64(case):
    t = {k: (I.widen(v) if v.dtype == np.uint16 else v).astype(np.float64) for k, v in case.tensors.items()}
    return t


def run(case):
    desc, t, mask = P.core_to_device(case, DEV)
    out = P.ff_attention_core_backward(desc, t["q"], t["k"], t["v"], t["g"], t.get("bias"), mask, t["do"])
    torch.cuda.synchronize()
    return out


def check_all(case, got, ref, what):
    for name, gt, rf in zip(NAMES, got, ref):
        if rf is None:
            assert gt is None
            continue
        g = gt.float().cpu().numpy().astype(np.float64)
        scale = max(1.0, float(np.sqrt((rf ** 2).mean())))
        ma, rl = max_abs(g, rf), rel_l2(g, rf)
        print(f"{what} {name}: max_abs={ma:.3e} (scale {scale:.2f}) rel_l2={rl:.3e}", flush=True)
        assert np.isfinite(g).all(), (what, name)
        absolute = (4e-2 if name == "dbias" else 2e-2) * scale
        assert np.all(np.abs(g - rf) <= absolute + 2.0 ** -8 * np.abs(rf)), (what, name, ma, scale)
        assert rl <= 1e-2, (what, name, rl)


def oracle(case):
    t = f64(case)
    return O.attention_core_backward(t["q"], t["k"], t["v"], t["g"], t.get("bias"), case.mask, t["do"])


SHAPES = [   # rows, heads, length, head_dim, bias, mask: ragged around the 32-wide tiles
    (1, 1, 1, 8, True, "none"), (2, 3, 31, 16, True, "random:0.7"), (3, 2, 33, 32, True, "tail:5"),
    (2, 2, 64, 32, False, "random:0.8"), (5, 4, 97, 8, True, "random:0.9"), (2, 8, 130, 32, True, "tail:20"),
    (3, 1, 200, 16, False, "none"), (9, 2, 70, 32, True, "random:0.5"),
    (26, 2, 64, 16, True, "random:0.8"),       # three uneven row chunks of the bias gradient (9, 9, 8 rows)
]


@pytest.mark.parametrize("rows,heads,length,d,bias,mask", SHAPES)
def test_ragged_shapes(rows, heads, length, d, bias, mask):
    spec = I.CoreSpec(f"t_core_{rows}_{heads}_{length}_{d}_{int(bias)}_{mask}", rows, heads, length, d, bias, mask)
    case = I.make_core_case(spec)
    check_all(case, run(case), oracle(case), spec.name)


@pytest.mark.parametrize("rows,heads,length,d,bias,mask", [
    (2, 2, 32, 32, True, "tail:3"),                                                   # one wavefront
    (2, 1, 257, 8, True, "random:0.8"), (1, 2, 320, 16, False, "tail:40"), (2, 1, 479, 32, True, "random:0.7"),
    (1, 2, 512, 32, True, "tail:33"),                                                # the longest that one block takes whole
    (1, 1, 513, 32, True, "random:0.9"), (1, 1, 540, 16, False, "tail:9"),          # the kernels for longer sequences
])
def test_lengths_around_the_limits_of_a_block(rows, heads, length, d, bias, mask):
    """Up to 512 positions a block holds a whole (row, head), a wavefront per 32 positions; beyond, three kernels pass tiles."""
    spec = I.CoreSpec(f"t_core_limits_{rows}_{heads}_{length}_{d}_{int(bias)}_{mask}", rows, heads, length, d, bias, mask)
    case = I.make_core_case(spec)
    check_all(case, run(case), oracle(case), spec.name)


@pytest.mark.parametrize("d", [8, 16, 32])
@pytest.mark.parametrize("bias", [True, False])
@pytest.mark.parametrize("rows,heads,length,mask", [(2, 2, 416, "random:0.8"), (3, 1, 430, "tail:17"), (1, 2, 544, "none"), (1, 1, 530, "random:0.7")])
def test_kernels_that_pass_tiles(rows, heads, length, mask, bias, d):
    """Few (row, head)s of long sequences, and sequences longer than a block holds: whole tiles and a ragged last one, at every head dim."""
    spec = I.CoreSpec(f"t_core_tiles_{rows}_{heads}_{length}_{d}_{int(bias)}_{mask}", rows, heads, length, d, bias, mask)
    case = I.make_core_case(spec)
    check_all(case, run(case), oracle(case), spec.name)


@pytest.mark.parametrize("rows,heads,length,d,bias,mask", [
    (26, 4, 512, 32, True, "random:0.9"), (25, 4, 470, 16, False, "tail:21"), (33, 4, 449, 8, True, "none"), (86, 4, 290, 16, False, "random:0.9")])
def test_blocks_that_hold_a_row(rows, heads, length, d, bias, mask):
    """As many (row, head)s as one block each takes, of lengths that leave a block alone on its compute unit."""
    spec = I.CoreSpec(f"t_core_rows_{rows}_{heads}_{length}_{d}_{int(bias)}_{mask}", rows, heads, length, d, bias, mask)
    case = I.make_core_case(spec)
    check_all(case, run(case), oracle(case), spec.name)


@pytest.mark.parametrize("rows,heads,length,bias,d,whole", [
    (1, 4, 320, True, 32, True), (1, 4, 384, False, 32, False), (16, 4, 384, False, 32, True), (16, 4, 416, True, 16, False), (16, 4, 512, False, 8, False),
    (32, 4, 512, False, 32, True), (33, 8, 512, False, 8, False), (33, 8, 512, True, 8, True), (33, 8, 384, False, 32, True), (37, 8, 512, False, 32, True),
    (40, 8, 512, False, 8, False), (42, 8, 512, False, 8, True), (42, 8, 384, False, 16, False), (43, 8, 384, False, 16, True),
    (2, 4, 128, True, 32, True), (64, 8, 520, True, 32, False)])
def test_which_kernels_take_a_call(rows, heads, length, bias, d, whole):
    """A block per (row, head) leaves an MI355X of 256 compute units idle where there are few of them, and needs a second round where there
    are just more than units: there the kernels that pass tiles are the faster ones."""
    q = torch.zeros((rows, heads, length, d), dtype=torch.bfloat16, device=DEV)
    b = torch.zeros((heads, length, length), device=DEV) if bias else None
    P.ff_profile_enable(True)
    P.ff_attention_core_backward(P.CoreDesc(P.FF_BF16, rows, heads, length, d), q, q, q, q, b, None, q)
    kinds = set(P.ff_profile_collect())
    P.ff_profile_enable(False)
    assert ("k_bwd_rows" in kinds) == whole, kinds
    assert ("k_bwd_dq" in kinds) != whole, kinds


@pytest.mark.parametrize("rows,length,expected", [
    (128, 64, {"k_bwd_prepare": 1, "k_bwd_rows": 1, "k_bwd_dbias": 1, "k_bwd_dbias_reduce": 1}),
    (1, 513, {"k_bwd_prepare": 1, "k_bwd_stats": 1, "k_bwd_dq": 1, "k_bwd_dkv": 1, "k_bwd_dbias": 1})])
def test_launch_timer_kinds(rows, length, expected):
    """Every kernel has a kind of its own: the rate of one that contracts must not be taken over launches that do not."""
    q = torch.zeros((rows, 2, length, 16), dtype=torch.bfloat16, device=DEV)
    P.ff_profile_enable(True)
    P.ff_attention_core_backward(P.CoreDesc(P.FF_BF16, rows, 2, length, 16), q, q, q, q, torch.zeros((2, length, length), device=DEV), None, q)
    kinds = {k: n for k, (_, n) in P.ff_profile_collect().items()}
    P.ff_profile_enable(False)
    assert kinds == expected


@pytest.mark.parametrize("rows,heads,length,d", [(4, 2, 100, 8), (3, 2, 255, 32), (26, 4, 500, 16), (2, 2, 420, 32), (1, 1, 515, 8)])
def test_masked_keys_with_a_far_larger_bias(rows, heads, length, d):
    """The bias of the keys that are attended to lies 300 below that of the masked ones: weights of masked keys that a kernel forms and
    drops are infinite (2^433), and times a zero or negative dP - delta NaN or -infinity."""
    case = I.make_core_case(I.CoreSpec(f"t_core_shift_{rows}_{heads}_{length}_{d}", rows, heads, length, d, True, "tail:37"))
    live = length - 37
    case.tensors["bias"][:, :, :live] -= np.float32(300.0)
    got = run(case)
    check_all(case, got, oracle(case), case.spec.name)
    for name, g in zip(NAMES, got):
        masked = g[..., live:] if name == "dbias" else g[:, :, live:]
        if name in ("dk", "dv", "dbias"):
            assert not masked.any(), name


@pytest.mark.parametrize("d", [8, 16, 32])
@pytest.mark.parametrize("bias", [True, False])
@pytest.mark.parametrize("rows,heads,length", [(5, 2, 71, ), (16, 8, 128), (2, 2, 416), (1, 2, 545), (1, 1, 576)])
def test_content_of_masked_keys_reaches_nothing(rows, heads, length, bias, d):
    """NaN and infinities in k and v of masked keys give the very gradients that zeros there give, in both paths."""
    case = I.make_core_case(I.CoreSpec(f"t_core_poison_{rows}_{heads}_{length}_{d}_{int(bias)}", rows, heads, length, d, bias, "random:0.8"))
    desc, t, mask = P.core_to_device(case, DEV)
    dead = (mask == 0)[:, None, :].expand(rows, heads, length)
    got = []
    for value in (0.0, float("nan"), float("inf")):
        k, v = t["k"].clone(), t["v"].clone()
        k[dead] = value
        v[dead] = -value
        got.append(P.ff_attention_core_backward(desc, t["q"], k, v, t["g"], t.get("bias"), mask, t["do"]))
    torch.cuda.synchronize()
    for name, a, b, c in zip(NAMES, *got):
        if a is None:
            continue
        assert torch.isfinite(a).all(), name
        assert torch.equal(a, b) and torch.equal(a, c), name


def test_fully_masked_rows_have_zero_gradients():
    spec = I.CoreSpec("t_core_dead", 4, 2, 50, 32, True, "random:0.8")
    case = I.make_core_case(spec)
    case.mask[2, :] = 0.0
    got = run(case)
    for t in got[:4]:
        assert torch.count_nonzero(t[2]).item() == 0
    check_all(case, got, oracle(case), "dead row")


def test_workspace_content_does_not_reach_the_bias_gradient():
    """81 rows: the rounded-up share of nine rows leaves one of the ten row chunks without rows.  Its partial sums are
    never written, so they must not be added; the workspace holds NaN patterns here."""
    case = I.make_core_case(I.CoreSpec("t_core_chunks", 81, 1, 32, 8, True, "random:0.8"))
    desc, t, mask = P.core_to_device(case, DEV)
    ws = torch.full((P.ff_attention_core_backward_workspace_bytes(desc),), 0xFF, dtype=torch.uint8, device=DEV)
    got = P.ff_attention_core_backward(desc, t["q"], t["k"], t["v"], t["g"], t["bias"], mask, t["do"], ws=ws)
    check_all(case, got, oracle(case), "dirty workspace")


@pytest.mark.parametrize("name", ["core_row_256", "core_tri_256"])
def test_paper_shapes(name):
    """The attention cores of the initial-training shapes: MSA row attention (128 x 8 x 256 x 32 with pair bias)
    and triangle attention (256 x 4 x 256 x 32)."""
    case = I.make_core_case(name)
    check_all(case, run(case), oracle(case), name)


def test_bad_arguments_are_status_codes():
    d = P.CoreDesc(P.FF_F32, 2, 2, 16, 8)
    assert P.lib().ff_attention_core_backward_workspace_bytes(C.byref(d)) == 0
    d = P.CoreDesc(P.FF_BF16, 2, 2, 16, 24)
    assert P.lib().ff_attention_core_backward_workspace_bytes(C.byref(d)) == 0
    d = P.CoreDesc(P.FF_BF16, 2, 2, 16, 8)
    need = P.lib().ff_attention_core_backward_workspace_bytes(C.byref(d))
    assert need > 0 and need % 256 == 0
    a = [0x10000 * (n + 1) for n in range(12)]
    call = lambda bias, dbias, ws_bytes: P.lib().ff_attention_core_backward(
        C.byref(d), a[0], a[1], a[2], a[3], bias, None, a[4], a[5], a[6], a[7], a[8], dbias, 0x1000000, ws_bytes, None)
    assert call(None, a[9], need) == B.FF_EINVAL            # dbias without bias
    assert call(a[9], a[10], need - 1) == B.FF_EWORKSPACE
