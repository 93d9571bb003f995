"""CPU checks of what the kernels read of a layer's radial functions, decoded
from the arrays that model creation uploads (mpip_radial_operands), against the
oracle's radial MLP a(d) and the weights: the directions are orthonormal, the
tables hold the functions turn^T a(d) and their derivatives, the weights are
turn^T W3 of the paths (FP32 form) or of the edge frame's coefficients (BF16
form) to the parts they are held in, and weights whose radial functions are
steep keep all hidden units."""
import numpy as np
import pytest

import workloads as W
from oracle.weights import parse_weights
from test_gpu_radial import steep
from test_radial_table import _oracle_a


U = 2.0 ** -8   # unit roundoff of BF16


def _lib():
    import paper_2509_21694_amd as M
    return M


def _paths(layer, L):
    return [(a, b, c) for a in ([0] if layer == 1 else range(L + 1)) for b in range(L + 1) for c in range(L + 1)
            if (a + b + c) % 2 == 0 and abs(a - b) <= c <= a + b]


def columns(hp, lay, layer, prec, last):
    """W3 of the columns, [hidden][columns]."""
    M, L, C = _lib(), hp.l_max, hp.channels
    paths = _paths(layer, L)
    W3 = np.asarray(lay["W3"], dtype=np.float64).reshape(hp.radial_hidden, len(paths), C)
    live = [p for p in range(len(paths)) if not last or paths[p][2] == 0]
    if prec == "fp32":
        return W3[:, live].reshape(hp.radial_hidden, -1)
    out = []
    for a in range(1 if layer == 1 else L + 1):
        for c in range(1 if last else L + 1):
            for am in range(1 if L == 1 else min(a, c) + 1):
                t = 0.0
                for p in live:
                    if paths[p][0] == a and paths[p][2] == c:
                        b = paths[p][1]
                        t = t + np.sqrt(2 * b + 1) * M.coupling_tensor(a, b, c)[a + am, b, c + am] * W3[:, p]
                out.append(t + np.zeros((hp.radial_hidden, C)))
    return np.stack(out, axis=1).reshape(hp.radial_hidden, -1)


def functions(table, d, rc):
    """b(d) and db/dd of a table."""
    n = table.shape[0]
    t = d / rc * n
    k = np.minimum(t.astype(int), n - 1)
    tau = (t - k)[:, None]
    c = table[k].astype(np.float64)
    return (c[..., 0] + tau * (c[..., 1] + tau * (c[..., 2] + tau * c[..., 3])),
            (c[..., 1] + tau * (2 * c[..., 2] + 3 * tau * c[..., 3])) * n / rc)


def _case(scale, layer, hp=None):
    hp = hp or W.HParams(n_species=3, n_layers=3, l_max=2, channels=64)
    blob = steep(W.make_weights(hp, 21), hp, scale)
    return hp, blob, parse_weights(blob, hp)["layers"][layer - 1]


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("layer,kind", [(1, 0), (1, 1), (1, 2), (2, 0), (3, 1)])
@pytest.mark.parametrize("scale", [1.0, 1.5, 4.0])
def test_tables_and_weights(prec, layer, kind, scale):
    M = _lib()
    hp, blob, lay = _case(scale, layer)
    direc, turn, table, wts = M.radial_operands(hp, blob, layer, prec, kind)
    n = turn.shape[1]
    if scale == 4.0 or (kind == 2 and prec == "fp32"):
        assert not direc
    if not direc:
        assert scale > 1.0 or kind == 2
        assert n == hp.radial_hidden and np.array_equal(turn, np.eye(n))
    else:
        assert n == (32 if kind == 2 else 24 if prec == "bf16" else 48)
        assert np.abs(turn.T @ turn - np.eye(n)).max() < 1e-12
    # distances from 0.1 A, off the knots (tau between 0 and 1)
    d = 0.1 + (hp.r_cut - 0.1) * (np.arange(4000) + 0.37) / 4000
    a, da = _oracle_a(d, lay, hp)
    b, db = functions(table, d, hp.r_cut)
    scale_a, scale_d = np.abs(a @ turn).max(), np.abs(da @ turn).max()
    if prec == "bf16":
        # a line from the knot before, at most h |db| away, BF16 value and increment (each to U), off by h^2/8 |b''|,
        # its slope by h/2 |b''|; |b''| over an interval from da/dd at the sample and h to either side, twice that for
        # its change
        h = hp.r_cut / table.shape[0]
        curve = 2 * np.maximum(np.abs(_oracle_a(d + h, lay, hp)[1] - da), np.abs(_oracle_a(d - h, lay, hp)[1] - da)) / h
        b2 = curve if not direc else np.repeat(np.linalg.norm(curve, axis=1)[:, None], n, axis=1)
        assert np.all(np.abs(b - a @ turn) <= U * (1 + U) * (np.abs(a @ turn) + 2 * h * np.abs(da @ turn)) + h * h * b2)
        assert np.all(np.abs(db - da @ turn) <= U * np.abs(da @ turn) + (1 + U) * h / 2 * b2)
    else:                # interpolated to 1e-8 and 1e-7 of the maxima, FP32 coefficients (2^-24 each, four of them)
        assert np.abs(b - a @ turn).max() <= (1e-8 + 2.0 ** -22) * scale_a
        assert np.abs(db - da @ turn).max() <= (1e-7 + 2.0 ** -22) * scale_d
    if kind == 2:
        assert wts.size == 0
        return
    ref = turn.T @ columns(hp, lay, layer, prec, kind == 1)
    assert wts.shape == ref.shape
    if prec == "fp32":
        # three BF16 parts; of directions 16 .. 31 two, of 32 .. 47 one (and one rounding to FP32)
        tol = np.full(n, U ** 3 + 2.0 ** -24)
        if direc:
            tol[16:32], tol[32:] = U ** 2 + 2.0 ** -24, U
        assert np.all(np.abs(wts - ref) <= tol[:, None] * np.abs(ref) + 1e-30)
    else:
        # W3 takes one of the two neighbouring BF16 values (2 U at most), is turned, and rounded again
        size = np.linalg.norm(columns(hp, lay, layer, prec, kind == 1), axis=0)
        assert np.all(np.linalg.norm(wts - ref, axis=0) <= (2 * U + U * (1 + 2 * U)) * size)


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
@pytest.mark.parametrize("scale", [1.0, 1.25, 1.5, 2.0])
@pytest.mark.parametrize("layer,kind", [(1, 2), (2, 0), (3, 1)])
def test_directions_hold_at_every_distance(prec, layer, kind, scale):
    """What the directions leave out of a(d) and da/dd is small beside a(d) and da/dd at the same distance, from 0.1 A
    to one per cent below the cutoff (where a(d) is 1e-5 of its largest): 2^-9 and 2^-8 of them in the BF16 form (of
    the first layer's 32: 2^-10 and 2^-9), 2^-22 and 2^-20 in the FP32 form, there with what the directions that
    have one (from the 32nd on) or two BF16 parts (from the 16th) lose, half a unit roundoff U of a part on average.
    To that the rounding of the table.  Distances at which the tables are exact but for that: the FP32 form's knots,
    the middles of the BF16 form's intervals (the increment is h b' to h^2 / 24 of the third derivative, below
    2^-12 b' here)."""
    M = _lib()
    hp, blob, lay = _case(scale, layer)
    direc, turn, table, _ = M.radial_operands(hp, blob, layer, prec, kind)
    if not direc:
        assert scale > 1.0 or (kind == 2 and prec == "fp32")
        return
    n = table.shape[0]
    d = (np.arange(n // 50 + 1, int(0.99 * n), max(1, n // 1500)) + (0.5 if prec == "bf16" else 0.0)) * hp.r_cut / n
    a, da = _oracle_a(d, lay, hp)
    b, db = functions(table, d, hp.r_cut)
    rest, drest = (2.0 ** -10, 2.0 ** -9) if kind == 2 else (2.0 ** -9, 2.0 ** -8)
    lose, rnd = 0.0, U
    if prec == "fp32":
        rest, drest, lose, rnd = 2.0 ** -22, 2.0 ** -20, U / 2, 2.0 ** -23
    for got, ref, most in ((b, a, rest + rnd), (db, da, drest + rnd + (2.0 ** -12 if prec == "bf16" else 0.0))):
        parts = lose * np.linalg.norm(got[:, 32:], axis=1) + lose * U * np.linalg.norm(got[:, 16:32], axis=1)
        off = np.hypot(np.linalg.norm(ref - got @ turn.T, axis=1), parts) / np.linalg.norm(ref, axis=1)
        print(prec, layer, kind, scale, "worst", off.max(), "at", d[off.argmax()], "bound", most)
        assert off.max() <= most


@pytest.mark.parametrize("layer,kind,m", [(1, 2, 32), (2, 0, 8), (3, 1, 8)])
def test_no_function_carries_the_rounding(layer, kind, m):
    """BF16 form: a function that is most of a(d) would round as a whole, with one sign for all edges of a distance.
    The direction that is most of it (the leading singular vector of the samples the directions come from, each
    relative to its size) has the same share 1/m of each of m functions."""
    M = _lib()
    hp, blob, lay = _case(1.0, layer)
    direc, turn, _, _ = M.radial_operands(hp, blob, layer, "bf16", kind)
    assert direc
    a, da = _oracle_a(hp.r_cut * (np.arange(512) + 0.5) / 512, lay, hp)
    rows = np.concatenate([x / np.linalg.norm(x, axis=1, keepdims=True) for x in (a, da)])
    lead = np.linalg.svd(rows, full_matrices=False)[2][0]
    share = (turn.T @ lead) ** 2
    assert np.abs(share[:m] - 1.0 / m).max() < 1e-9
    assert m == len(share) or share[m:].max() < 1e-18


def test_rejects_bad_arguments():
    M = _lib()
    hp, blob, _ = _case(1.0, 1)
    for layer, kind in ((0, 0), (4, 0), (1, 3), (1, -1), (2, 2)):
        with pytest.raises(M.MpipError):
            M.radial_operands(hp, blob, layer, "bf16", kind)
    with pytest.raises(M.MpipError):
        M.radial_operands(hp, blob[:-1], 1, "bf16", 0)
