"""Timing cases of the framework: what a user of libff has it do, one pass per public entry point.

listed() names twelve passes from the smallest call to the largest, draw() gives further ones of the same ranges.
Shapes are those of inputs.py and bench.py (initial-training crop 128 x 256, fine-tuning 512 x 384, extra MSA of
1024 .. 5120 sequences, long-sequence inference at 2048 residues in chunks of 64 rows) and lengths between them, as
proteins have any length.  Inputs follow inputs.py: activations N(0, 1), weights N(0, 1 / fan_in), gate biases 1,
masks that pad a tail or drop residues.  Output and workspace buffers are the caller's, as in bench.py.
"""
import math

import torch

import paper_2203_00854_amd as P

MODES = {"row": P.FF_MSA_ROW, "col": P.FF_MSA_COL, "tri_start": P.FF_TRI_START, "tri_end": P.FF_TRI_END}


# --------------------------------------------------------------------------------------------------- the cases
def _attn(name, mode, dtype, n_a, n_b, c, c_z, heads, d, mask="none", residual=False, chunk=0):
    return {"name": name, "kind": "attention", "mode": mode, "dtype": dtype, "n_a": n_a, "n_b": n_b, "c": c, "c_z": c_z,
            "heads": heads, "d": d, "mask": mask, "residual": residual, "chunk": chunk}


def _trimul(name, n, incoming, residual, masked, c=128):
    return {"name": name, "kind": "trimul", "n": n, "c": c, "incoming": incoming, "residual": residual, "masked": masked}


def _global(name, n_seq, n_res, pad):
    return {"name": name, "kind": "global", "n_seq": n_seq, "n_res": n_res, "pad": pad}


def _core(name, rows, heads, length, d, bias, masked):
    return {"name": name, "kind": "core_backward", "rows": rows, "heads": heads, "length": length, "d": d, "bias": bias,
            "masked": masked}


def _norm(name, rows, c, dtype):
    return {"name": name, "kind": "layernorm", "rows": rows, "c": c, "dtype": dtype}


def listed():
    return [
        # the smallest call of the benchmark: one float32 module on a toy crop, where launches and host time count
        _attn("row_f32_8x32", "row", "f32", 8, 32, 32, 16, 4, 8, "tail"),
        # float32 inference of a short protein with a shallow alignment (length no multiple of a tile)
        _attn("row_f32_64x155", "row", "f32", 64, 155, 256, 128, 8, 32, "tail"),
        # MSA row attention with pair bias of the initial-training crop: the default workload of bench.py
        _attn("row_bf16_128x256", "row", "bf16", 128, 256, 256, 128, 8, 32, "tail"),
        # triangle attention of the same crop, residues missing at random
        _attn("tri_start_bf16_256", "tri_start", "bf16", 256, 256, 128, 0, 4, 32, "outer"),
        # triangle attention of a protein of any length, with the residual update that closes it in the block
        _attn("tri_end_bf16_333_residual", "tri_end", "bf16", 333, 333, 128, 0, 4, 32, "outer", residual=True),
        # long-sequence inference in chunks of 64 rows: the largest call
        _attn("tri_start_bf16_2048_chunk64", "tri_start", "bf16", 2048, 2048, 128, 0, 4, 32, "none", chunk=64),
        # column attention of the extra-MSA stack
        _attn("col_bf16_1024x384", "col", "bf16", 1024, 384, 64, 0, 8, 8, "tail"),
        # triangular multiplicative update of the initial-training crop, outgoing edges
        _trimul("trimul_out_256", 256, False, False, True),
        # the same for incoming edges at a longer, odd length, as a residual update
        _trimul("trimul_in_701_residual", 701, True, True, True),
        # global column attention of the extra-MSA stack
        _global("global_1024x384", 1024, 384, 102),
        # backward of the attention core at the row-attention shape of the training crop
        _core("core_backward_128x8x256x32", 128, 8, 256, 32, True, True),
        # LayerNorm of the fine-tuning crop's MSA representation
        _norm("layernorm_bf16_512x384x256", 512 * 384, 256, "bf16"),
    ]


def _log_size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["f32", "row", "tri", "tri", "col", "col_extra", "trimul", "trimul", "global", "core", "core", "norm"])
    if what == "f32":
        c, c_z, heads, d = rng.choice([(32, 16, 4, 8), (64, 32, 4, 16), (256, 128, 8, 32)])
        mode = rng.choice(["row", "col", "tri_start", "tri_end"])
        n = _log_size(rng, 16, 256)
        n_a = n if mode.startswith("tri") else _log_size(rng, 4, 128)
        case = _attn("", mode, "f32", n_a, n, c, c_z if mode == "row" else 0, heads, d, rng.choice(["tail", "none"]),
                     residual=rng.random() < 0.3)
    elif what == "row":
        case = _attn("", "row", "bf16", _log_size(rng, 8, 512), _log_size(rng, 48, 512), 256, 128, 8, 32,
                     rng.choice(["tail", "none"]), residual=rng.random() < 0.4)
    elif what == "tri":
        n = _log_size(rng, 48, 1536)
        case = _attn("", rng.choice(["tri_start", "tri_end"]), "bf16", n, n, 128, 0, 4, 32, rng.choice(["outer", "none"]),
                     residual=rng.random() < 0.4, chunk=64 if n >= 1024 else 0)
    elif what == "col":
        case = _attn("", "col", "bf16", _log_size(rng, 64, 512), _log_size(rng, 48, 384), 256, 0, 8, 32,
                     rng.choice(["tail", "none"]), residual=rng.random() < 0.4)
    elif what == "col_extra":
        case = _attn("", "col", "bf16", _log_size(rng, 128, 4096), _log_size(rng, 48, 384), 64, 0, 8, 8, "tail",
                     residual=rng.random() < 0.4)
    elif what == "trimul":
        case = _trimul("", _log_size(rng, 48, 1024), rng.random() < 0.5, rng.random() < 0.5, rng.random() < 0.5,
                       rng.choice([64, 128, 128]))
    elif what == "global":
        n_seq = _log_size(rng, 64, 5120)
        case = _global("", n_seq, _log_size(rng, 48, 384), rng.choice([0, n_seq // 10]))
    elif what == "core":
        case = _core("", _log_size(rng, 16, 256), rng.choice([4, 8]), _log_size(rng, 32, 512), rng.choice([8, 16, 32, 32]),
                     rng.random() < 0.7, rng.random() < 0.7)
    else:
        case = _norm("", _log_size(rng, 1000, 2000000), rng.choice([64, 128, 256]), rng.choice(["bf16", "f32"]))
    del case["name"]
    return case


# --------------------------------------------------------------------------------------------------- inputs
def _generator(seed):
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    return g


def _normal(g, shape, dtype, scale=1.0, shift=0.0):
    return (torch.randn(shape, generator=g, device="cuda:0") * scale + shift).to(dtype)


def _dtype(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.bfloat16


def _workspace(n):
    # (zeroed once, so that a pass can depend on nothing but its inputs)
    return torch.zeros(n, dtype=torch.uint8, device="cuda:0")


def _prepare_attention(case, g):
    dt, c, cz, hd = _dtype(case), case["c"], case["c_z"], case["heads"] * case["d"]
    x = _normal(g, (case["n_a"], case["n_b"], c), dt)
    z = _normal(g, (case["n_b"], case["n_b"], cz), dt) if case["mode"] == "row" else None
    w = {"ln_g": _normal(g, (c,), dt, 0.1, 1.0), "ln_b": _normal(g, (c,), dt, 0.1)}
    if case["mode"] == "row":
        w.update(lnz_g=_normal(g, (cz,), dt, 0.1, 1.0), lnz_b=_normal(g, (cz,), dt, 0.1),
                 w_b=_normal(g, (case["heads"], cz), dt, cz ** -0.5))
    elif case["mode"] != "col":
        w["w_b"] = _normal(g, (case["heads"], c), dt, c ** -0.5)
    for k in ("w_q", "w_k", "w_v", "w_g"):
        w[k] = _normal(g, (hd, c), dt, c ** -0.5)
    w.update(b_g=torch.ones(hd, dtype=dt, device="cuda:0"), w_o=_normal(g, (c, hd), dt, hd ** -0.5), b_o=_normal(g, (c,), dt, 0.1))
    mask = None
    if case["mask"] == "tail":           # the last positions of the attended axis are padding
        mask = torch.ones(case["n_a"], case["n_b"], device="cuda:0")
        if case["mode"] == "col":
            mask[case["n_a"] - (case["n_a"] + 9) // 10:, :] = 0
        else:
            mask[:, case["n_b"] - (case["n_b"] + 15) // 16:] = 0
    elif case["mask"] == "outer":        # residues missing at random
        r = (torch.rand(case["n_a"], generator=g, device="cuda:0") < 0.95).float()
        mask = torch.outer(r, r).contiguous()
    desc = P.make_desc(MODES[case["mode"]], x, case["heads"], case["d"], cz)
    ws = _workspace(P.ff_attention_workspace_bytes(desc, case["chunk"]))
    return {"desc": desc, "w": w, "x": x, "z": z, "mask": mask, "out": torch.empty_like(x), "ws": ws}


def _prepare_trimul(case, g):
    n, c, dt = case["n"], case["c"], torch.bfloat16
    w = {}
    for side in ("a", "b"):
        w["w_%sp" % side], w["b_%sp" % side] = _normal(g, (c, c), dt, c ** -0.5), _normal(g, (c,), dt, 0.1)
        w["w_%sg" % side], w["b_%sg" % side] = _normal(g, (c, c), dt, c ** -0.5), torch.ones(c, dtype=dt, device="cuda:0")
    w["w_g"], w["b_g"] = _normal(g, (c, c), dt, c ** -0.5), torch.ones(c, dtype=dt, device="cuda:0")
    w["w_o"], w["b_o"] = _normal(g, (c, c), dt, c ** -0.5), _normal(g, (c,), dt, 0.1)
    for k in ("ln", "lno"):
        w[k + "_g"], w[k + "_b"] = _normal(g, (c,), dt, 0.1, 1.0), _normal(g, (c,), dt, 0.1)
    z = _normal(g, (n, n, c), dt)
    mask = None
    if case["masked"]:
        r = (torch.rand(n, generator=g, device="cuda:0") < 0.95).float()
        mask = torch.outer(r, r).contiguous()
    desc = P.TriMulDesc(P.FF_BF16, 1 if case["incoming"] else 0, n, c, c, 1e-5)
    ws = _workspace(P.ff_triangle_multiplication_workspace_bytes(desc))
    return {"desc": desc, "w": w, "z": z, "mask": mask, "out": torch.empty_like(z), "ws": ws}


def _prepare_global(case, g):
    c, heads, d, dt = 64, 8, 8, torch.bfloat16
    hd = heads * d
    m = _normal(g, (case["n_seq"], case["n_res"], c), dt)
    w = {"ln_g": _normal(g, (c,), dt, 0.1, 1.0), "ln_b": _normal(g, (c,), dt, 0.1), "w_q": _normal(g, (hd, c), dt, c ** -0.5),
         "w_k": _normal(g, (d, c), dt, c ** -0.5), "w_v": _normal(g, (d, c), dt, c ** -0.5),
         "w_g": _normal(g, (hd, c), dt, c ** -0.5), "b_g": torch.ones(hd, dtype=dt, device="cuda:0"),
         "w_o": _normal(g, (c, hd), dt, hd ** -0.5), "b_o": _normal(g, (c,), dt, 0.1)}
    mask = None
    if case["pad"]:
        mask = torch.ones(case["n_seq"], case["n_res"], device="cuda:0")
        mask[case["n_seq"] - case["pad"]:, :] = 0
    desc = P.GlobalDesc(P.FF_BF16, case["n_seq"], case["n_res"], c, heads, d, 1e-5)
    ws = _workspace(P.ff_global_column_attention_workspace_bytes(desc))
    return {"desc": desc, "w": w, "m": m, "mask": mask, "out": torch.empty_like(m), "ws": ws}


def _prepare_core(case, g):
    shape, dt = (case["rows"], case["heads"], case["length"], case["d"]), torch.bfloat16
    t = {k: _normal(g, shape, dt) for k in ("q", "k", "v", "dout")}
    t["g"] = torch.sigmoid(torch.randn(shape, generator=g, device="cuda:0") + 1.0).to(dt)
    t["bias"] = _normal(g, (case["heads"], case["length"], case["length"]), torch.float32) if case["bias"] else None
    t["mask"] = None
    if case["masked"]:
        t["mask"] = torch.ones(case["rows"], case["length"], device="cuda:0")
        t["mask"][:, case["length"] - case["length"] // 16:] = 0
    t["desc"] = P.CoreDesc(P.FF_BF16, *shape)
    t["ws"] = _workspace(P.ff_attention_core_backward_workspace_bytes(t["desc"]))
    return t


def _prepare_norm(case, g):
    dt = _dtype(case)
    x = _normal(g, (case["rows"], case["c"]), dt, 1.5, 0.3)
    return {"x": x, "gamma": _normal(g, (case["c"],), dt, 0.1, 1.0), "beta": _normal(g, (case["c"],), dt, 0.1), "out": torch.empty_like(x)}


def prepare(case, seed):
    make = {"attention": _prepare_attention, "trimul": _prepare_trimul, "global": _prepare_global, "core_backward": _prepare_core,
            "layernorm": _prepare_norm}[case["kind"]]
    state = make(case, _generator(seed))
    state["case"] = case
    return state


# --------------------------------------------------------------------------------------------------- one pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "attention":
        if case["residual"]:
            return P.ff_gated_attention_residual(s["desc"], s["w"], s["x"], s["z"], s["mask"], chunk_rows=case["chunk"], out=s["out"],
                                                 ws=s["ws"])
        if case["chunk"]:
            return P.ff_attention_chunked(s["desc"], s["w"], s["x"], s["z"], s["mask"], chunk_rows=case["chunk"], out=s["out"], ws=s["ws"])
        return P.ff_gated_attention(s["desc"], s["w"], s["x"], s["z"], s["mask"], out=s["out"], ws=s["ws"])
    if kind == "trimul":
        return P.ff_triangle_multiplication(s["desc"], s["w"], s["z"], s["mask"], residual=case["residual"], out=s["out"], ws=s["ws"])
    if kind == "global":
        return P.ff_global_column_attention(s["desc"], s["w"], s["m"], s["mask"], out=s["out"], ws=s["ws"])
    if kind == "core_backward":
        grads = P.ff_attention_core_backward(s["desc"], s["q"], s["k"], s["v"], s["g"], s["bias"], s["mask"], s["dout"], ws=s["ws"])
        return [t for t in grads if t is not None]
    return P.ff_layernorm(s["x"], s["gamma"], s["beta"], out=s["out"])


# --------------------------------------------------------------------------------------------------- floors and tolerances
def work(case):
    kind = case["kind"]
    if kind == "attention":
        e = 4 if case["dtype"] == "f32" else 2
        row_like = case["mode"] in ("row", "tri_start")
        rows, length = (case["n_a"], case["n_b"]) if row_like else (case["n_b"], case["n_a"])
        tokens, c, cz, h, hd = rows * length, case["c"], case["c_z"], case["heads"], case["heads"] * case["d"]
        flops = 2 * tokens * c * 4 * hd + 4 * rows * h * length * length * case["d"] + 2 * tokens * hd * c
        nbytes = 2 * tokens * c * e + (4 * hd * c + hd * c) * e
        if case["mode"] == "row":
            flops += 2 * length * length * cz * h
            nbytes += length * length * cz * e
        elif case["mode"] != "col":
            flops += 2 * length * length * c * h
        if case["mask"] != "none":
            nbytes += tokens * 4
        return {"bytes": nbytes, "flops": flops}
    if kind == "trimul":
        n, c = case["n"], case["c"]
        return {"bytes": 2 * n * n * c * 2 + (n * n * 4 if case["masked"] else 0) + 6 * c * c * 2,
                "flops": 2 * n * n * c * 6 * c + 2 * n * n * n * c}
    if kind == "global":
        tokens, c, hd, d = case["n_seq"] * case["n_res"], 64, 64, 8
        return {"bytes": 2 * tokens * c * 2 + (tokens * 4 if case["pad"] else 0) + 3 * hd * c * 2,
                "flops": 2 * tokens * c * (2 * hd + 2 * d) + 4 * tokens * hd}
    if kind == "core_backward":
        n = case["rows"] * case["heads"] * case["length"]
        pairs = n * case["length"]
        # logits, context, dP, dv, dq and dk: the forward quantities are recomputed because nothing else was saved
        return {"bytes": 9 * n * case["d"] * 2 + (2 * case["heads"] * case["length"] ** 2 * 4 if case["bias"] else 0)
                + (case["rows"] * case["length"] * 4 if case["masked"] else 0), "flops": 12 * pairs * case["d"]}
    n = case["rows"] * case["c"]
    return {"bytes": 2 * n * (4 if case["dtype"] == "f32" else 2), "flops": 8 * n}


def tolerance(case):
    # About four times the relative error seen against the same module in float64 (1.7e-3 where only the rounding of the
    # result to bfloat16 shows, 2e-3 to 4.2e-3 where rounded operands precede it, 5e-7 in float32).
    if case.get("dtype") == "f32":
        return {"rel": 2e-6}
    if case["kind"] == "layernorm":
        return {"rel": 7e-3}
    if case.get("residual"):
        return {"rel": 1.2e-2 if case["kind"] == "trimul" else 7e-3}
    return {"rel": {"global": 8e-3, "core_backward": 1.2e-2}.get(case["kind"], 1.6e-2)}
