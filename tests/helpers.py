"""Helpers shared by the tests: small seeded cases and error measures."""
import numpy as np

from paper_2203_00854_amd import inputs as I


def small_spec(mode, n_a, n_b, c, heads, d, c_z=0, dtype="f32", mask="none", name=None, chunk_rows=0):
    if mode == I.MODE_ROW and c_z == 0:
        c_z = 8
    if mode != I.MODE_ROW:
        c_z = 0
    name = name or f"t_{I.MODE_NAMES[mode]}_{dtype}_{n_a}x{n_b}x{c}_h{heads}d{d}_{mask}"
    return I.CaseSpec(name, mode, dtype, n_a, n_b, c, c_z, heads, d, mask, chunk_rows=chunk_rows)


def f64_inputs(case):
    """(x, z, mask, weights) as float64 arrays holding exactly the stored values."""
    x = case.widened("x").astype(np.float64)
    z = None if case.z is None else case.widened("z").astype(np.float64)
    w = {k: v.astype(np.float64) for k, v in case.widened_weights().items()}
    return x, z, case.mask, w


def max_abs(a, b):
    return float(np.max(np.abs(np.asarray(a, np.float64) - np.asarray(b, np.float64))))


def rel_l2(a, b):
    a = np.asarray(a, np.float64)
    b = np.asarray(b, np.float64)
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def patchy_mask(rows, length, seed=7):
    """[rows, length] masks whose rows differ in where they have no valid key: a long tail, a long lead, a gap of whole tiles of
    32, single keys at random, none at all, all but one key."""
    rng = np.random.default_rng(seed)
    m = np.ones((rows, length), np.float32)
    for r in range(rows):
        kind = r % 6
        if kind == 0:
            m[r, min(33, length - 1):] = 0.0
        elif kind == 1:
            m[r, :max(length - 40, 0)] = 0.0
        elif kind == 2:
            m[r, 31:min(97, length - 1)] = 0.0
        elif kind == 3:
            m[r] = rng.random(length) < 0.7
        elif kind == 5:
            m[r] = 0.0
        if not m[r].any() or kind == 5:
            m[r, length // 2] = 1.0
    return m


def poison_masked_tokens(case, mask):
    """Sets the case's mask ([n_a, n_b]) and puts zeros into its masked tokens; returns x with NaN and infinities there instead
    (storage type of the case)."""
    case.mask = np.ascontiguousarray(mask, np.float32)
    dead = case.mask == 0
    case.x = case.x.copy()
    case.x[dead] = 0
    bad = case.x.copy()
    n = int(dead.sum())
    v = np.resize(np.array([np.nan, np.inf, -np.inf], np.float32), n)[:, None] * np.ones(case.x.shape[2], np.float32)
    bad[dead] = I.to_storage(v, case.spec.dtype)
    return bad
