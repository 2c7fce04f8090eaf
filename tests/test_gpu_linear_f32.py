"""The fp32 LoRA-adapted linear step at the sizes where its tiles can go wrong: every kernel and tile shape (fragments straight from
memory, tiles of 64, operands in bf16 parts, wide rows; test_linear_plan.py holds which size takes which), row lengths that are no
multiple of four floats, ragged rows, columns, ranks and contractions, an update in place, values of every scale, values that are not
finite or not normal.  Reference: fp64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2401_11504_amd import api  # noqa: E402

LR = 5e-5


def tol(*dims):
    """A chain of K fp32 products strays by about sqrt(K) 2^-24 of its 2-norm, K the longest contraction (16 more for the few
    roundings around it); doubled for the low-rank chain.  (Where eight waves share a contraction, or the matrix instruction rounds once per
    eight elements, there are fewer roundings.)"""
    return 2 * (max(dims) + 16) ** 0.5 * 2.0 ** -24


CASES = [
    # T, d_in, d_out, r; the low-rank products are direct-16x16 throughout
    (1, 1, 1, 1), (33, 100, 101, 4), (5, 64, 3, 32), (31, 129, 66, 33), (65, 1030, 259, 16), (8200, 65, 40, 64),      # direct-16x16
    (300, 777, 1003, 7),                                                                                              # direct-32x32
    (512, 768, 768, 8), (592, 741, 2895, 8), (621, 1264, 686, 24), (8192, 63, 4096, 3),                               # 64x64
    (515, 1023, 1030, 64), (700, 1200, 1111, 37), (130, 4096, 16400, 5),                                              # split-128x128
    (1027, 4096, 2050, 64), (1400, 2049, 4101, 48),                                                                   # split-256x128
]


def make(T, din, dout, r):
    g = torch.Generator().manual_seed(T * 7 + din)
    n = lambda std, *size: torch.randn(*size, generator=g) * std
    return [n(1.0, T, din), n(0.02, dout, din), n(0.02, r, din), n(0.01, dout, r), n(1.0, T, dout)]


def reference(ins, s):
    X, W, A, B, dY = (t.double() for t in ins)
    H, dH = X @ A.T, s * dY @ B
    return {"Y": X @ W.T + s * H @ B.T, "dX": dY @ W + dH @ A, "dA": dH.T @ X, "dB": s * dY.T @ H}


def step(ins, s, outs, A_new, B_new):
    api.tl_linear_step(*ins, s, LR, 0.9, 0.999, 1e-8, 0.01, True, *outs, A_new, B_new)


@pytest.mark.parametrize("T,din,dout,r", CASES)
def test_linear_step(T, din, dout, r):
    ins, s = make(T, din, dout, r), 1.5
    dev = [t.cuda() for t in ins]
    shapes = dict(Y=(T, dout), dX=(T, din), dA=(r, din), dB=(dout, r))
    # what lies behind an output's last element stays as it is
    flat = {k: torch.full((a * b + 64,), 3.0, device="cuda") for k, (a, b) in shapes.items()}
    outs = [flat[k][:a * b].view(a, b) for k, (a, b) in shapes.items()]
    new = [torch.empty_like(dev[2]), torch.empty_like(dev[3])]
    step(dev, s, outs, *new)
    ref = reference(ins, s)
    for (k, (a, b)), o in zip(shapes.items(), outs):
        err = (o.cpu().double() - ref[k]).norm() / ref[k].norm()
        assert err < tol(T, din, dout), (k, err)
        assert bool((flat[k][a * b:] == 3.0).all()), k
    for p, gname, p1 in ((ins[2], "dA", new[0]), (ins[3], "dB", new[1])):
        gr = outs[2 if gname == "dA" else 3].cpu().double()
        want = p.double() * (1 - LR * 0.01) - LR * gr / (gr.abs() + 1e-8)       # first AdamW step, from the gradient handed out
        # p itself is rounded to fp32 (|p| < 0.1: 4e-9), the step of size LR to a few ulp
        assert (p1.cpu().double() - want).abs().max() < 8e-9 + LR * 1e-6, gname

    # the same in place: the factors are updated where they are
    dev2 = [t.cuda() for t in ins]
    outs2 = [torch.empty_like(o) for o in outs]
    step(dev2, s, outs2, dev2[2], dev2[3])
    for k, o, o2 in zip(shapes, outs, outs2):
        err = (o2.cpu().double() - ref[k]).norm() / ref[k].norm()
        assert err < tol(T, din, dout), (k, err)
    for p, g2, p1 in ((ins[2], outs2[2], dev2[2]), (ins[3], outs2[3], dev2[3])):
        gr = g2.cpu().double()
        want = p.double() * (1 - LR * 0.01) - LR * gr / (gr.abs() + 1e-8)
        assert (p1.cpu().double() - want).abs().max() < 8e-9 + LR * 1e-6


# Rows of more than 2^22 floats, whose offsets within a tile exceed 32 bits; the in-place update takes one launch per product.
@pytest.mark.parametrize("T,din,dout,r", [(2, (1 << 22) + 3, 3, 2), (3, 5, (1 << 22) + 1, 4), (70, (1 << 22) + 6, 2, 1)])
@pytest.mark.parametrize("in_place", [False, True])
def test_wide_rows(T, din, dout, r, in_place):
    ins, s = make(T, din, dout, r), 1.5
    dev = [t.cuda() for t in ins]
    outs = [torch.empty(*size, device="cuda") for size in ((T, dout), (T, din), (r, din), (dout, r))]
    new = dev[2:4] if in_place else [torch.empty_like(dev[2]), torch.empty_like(dev[3])]
    step(dev, s, outs, *new)
    ref = reference(ins, s)
    for k, o in zip(("Y", "dX", "dA", "dB"), outs):
        err = (o.cpu().double() - ref[k]).norm() / ref[k].norm()
        assert err < tol(T, din, dout), (k, err)
    for p, gr, p1 in ((ins[2], outs[2], new[0]), (ins[3], outs[3], new[1])):
        gr = gr.cpu().double()
        want = p.double() * (1 - LR * 0.01) - LR * gr / (gr.abs() + 1e-8)
        assert (p1.cpu().double() - want).abs().max() < 8e-9 + LR * 1e-6


# An infinite or undefined operand shows where it is a factor and nowhere else: not in the rows, columns and contractions that
# a ragged tile reads beside it.
@pytest.mark.parametrize("T,din,dout,r", [(33, 101, 67, 5), (515, 1023, 1030, 6)])
@pytest.mark.parametrize("which,at", [(0, (5, -1)), (0, (-1, 0)), (1, (2, -1)), (1, (-1, 0)), (2, (0, -1)), (3, (-1, -1)), (4, (7, 0))])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_non_finite_operands(T, din, dout, r, which, at, value):
    ins, s = make(T, din, dout, r), 1.5
    ins[which][at] = value
    dev = [t.cuda() for t in ins]
    outs = [torch.empty(*size, device="cuda") for size in ((T, dout), (T, din), (r, din), (dout, r))]
    step(dev, s, outs, torch.empty_like(dev[2]), torch.empty_like(dev[3]))
    ref = reference(ins, s)
    for k, o in zip(("Y", "dX", "dA", "dB"), outs):
        o, fine = o.cpu().double(), torch.isfinite(ref[k])
        assert torch.equal(torch.isfinite(o), fine), k
        if fine.any():
            assert (o - ref[k])[fine].norm() < tol(T, din, dout) * ref[k][fine].norm(), k


def test_subnormal_products_and_sums():
    T, din, dout, r = 33, 64, 70, 4
    ins = make(T, din, dout, r)
    ins[0] *= 1e-21                       # X W^T and H = X A^T are of the order of 1e-42
    ins[1] *= 1e-20
    ins[2] *= 1e-20
    dev = [t.cuda() for t in ins]
    outs = [torch.empty(*size, device="cuda") for size in ((T, dout), (T, din), (r, din), (dout, r))]
    step(dev, 1.0, outs, torch.empty_like(dev[2]), torch.empty_like(dev[3]))
    ref = reference([t.cpu() for t in dev], 1.0)
    assert 1e-43 < ref["Y"].abs().max() < 1e-38
    # every sum is rounded to a multiple of 2^-149: 64 of them and the low-rank chain's 4 (behind a product with B < 1)
    assert (outs[0].cpu().double() - ref["Y"]).abs().max() < 69 * 2.0 ** -149


# Operands cut into bf16 parts: ragged rows, columns and contractions of both tiles (256x128: the first; 128x128: the others), and
# what the parts do not hold (infinities) or hold by a scale (values below 2^-110) in the first and the last tile of a contraction, in
# either half of a tile's rows, and in the low-rank factors.
SPLIT = [(1029, 2050, 2049, 64), (701, 2500, 2501, 33), (257, 4095, 4100, 7), (1400, 1030, 1100, 1)]


@pytest.mark.parametrize("T,din,dout,r", SPLIT)
def test_split_operands(T, din, dout, r):
    ins, s = make(T, din, dout, r), 1.5
    dev = [t.cuda() for t in ins]
    outs = [torch.empty(*size, device="cuda") for size in ((T, dout), (T, din), (r, din), (dout, r))]
    step(dev, s, outs, torch.empty_like(dev[2]), torch.empty_like(dev[3]))
    ref = reference(ins, s)
    for k, o in zip(("Y", "dX", "dA", "dB"), outs):
        assert (o.cpu().double() - ref[k]).norm() < tol(T, din, dout) * ref[k].norm(), k


@pytest.mark.parametrize("T,din,dout,r", SPLIT[:2])
@pytest.mark.parametrize("which,at", [(0, (5, -1)), (0, (-1, 0)), (0, (200, 40)), (1, (2, -1)), (1, (-1, 0)), (2, (0, -1)), (3, (-1, -1)), (4, (7, 0))])
@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_split_operands_not_finite(T, din, dout, r, which, at, value):
    ins, s = make(T, din, dout, r), 1.5
    ins[which][at] = value
    dev = [t.cuda() for t in ins]
    outs = [torch.empty(*size, device="cuda") for size in ((T, dout), (T, din), (r, din), (dout, r))]
    step(dev, s, outs, torch.empty_like(dev[2]), torch.empty_like(dev[3]))
    ref = reference(dev, s)                      # (on the GPU, in fp64)
    for k, o in zip(("Y", "dX", "dA", "dB"), outs):
        fine = torch.isfinite(ref[k])
        assert torch.equal(torch.isfinite(o), fine), k
        assert torch.equal(torch.isnan(o), torch.isnan(ref[k])), k
        assert torch.equal(o[~fine & ~torch.isnan(o)].double(), ref[k][~fine & ~torch.isnan(o)]), k
        if fine.any():
            assert (o.double() - ref[k])[fine].norm() < tol(T, din, dout) * ref[k][fine].norm(), k


@pytest.mark.parametrize("T,din,dout,r", SPLIT[:2])
@pytest.mark.parametrize("rows", [slice(0, None), slice(100, 101), slice(-1, None)])
def test_split_operands_tiny(T, din, dout, r, rows):
    """Rows of X of the order of 2^-116, which bf16 parts without a scale would hold to 17 bits: their outputs (2^-116 too) are as precise as the others."""
    ins, s = make(T, din, dout, r), 1.5
    ins[0][rows] *= 2.0 ** -116
    dev = [t.cuda() for t in ins]
    outs = [torch.empty(*size, device="cuda") for size in ((T, dout), (T, din), (r, din), (dout, r))]
    step(dev, s, outs, torch.empty_like(dev[2]), torch.empty_like(dev[3]))
    ref = reference(ins, s)
    # each of the K sums of an entry may also be off by half of 2^-149, far below a row of 2^-116
    assert (outs[0].cpu().double() - ref["Y"])[rows].norm() < tol(T, din, dout) * ref["Y"][rows].norm()
    assert (outs[0].cpu().double() - ref["Y"]).norm() < tol(T, din, dout) * ref["Y"].norm()


# Operands far from 1 and too small for the parts, zeros, rows and columns far below the largest magnitude (an outlier puts every other
# element there), in products of two long contractions and of a long and a short one.  Every row
# and every column of the outputs is held to the tolerance by itself (twice, for the fewer entries it has).
def _scale(ins, what):
    X, W, A, B, dY = ins
    if what == "large": X *= 2.0 ** 90; W *= 2.0 ** -95; B *= 2.0 ** -90; dY *= 2.0 ** 60
    elif what == "beyond": W *= 2.0 ** -104; B *= 2.0 ** -100; dY *= 2.0 ** 40
    elif what == "zero rows": X[3:400] = 0; W[:, 5:90] = 0; W[7] = 0; B[7] = 0; dY[-200:] = 0
    elif what == "rows": X[100] *= 2.0 ** -12; X[-1] *= 2.0 ** -30; dY[257] *= 2.0 ** -20
    elif what == "columns": W[:, 9] *= 2.0 ** -16; A[:, 9] *= 2.0 ** -16; W[-1] *= 2.0 ** -25; B[-1] *= 2.0 ** -25
    elif what == "outlier": X[300, 11] = 3.0e4; dY[2, 2] = -7.0e5
    elif what == "all zero": X *= 0


@pytest.mark.parametrize("T,din,dout,r", [(1029, 2050, 2049, 64), (701, 2500, 2501, 33), (1400, 31, 4100, 3), (1400, 4100, 63, 3)])
@pytest.mark.parametrize("what", ["", "large", "beyond", "zero rows", "rows", "columns", "outlier", "all zero"])
def test_split_operands_scales(T, din, dout, r, what):
    ins, s = make(T, din, dout, r), 1.5
    _scale(ins, what)
    dev = [t.cuda() for t in ins]
    outs = [torch.empty(*size, device="cuda") for size in ((T, dout), (T, din), (r, din), (dout, r))]
    step(dev, s, outs, torch.empty_like(dev[2]), torch.empty_like(dev[3]))
    X, W, A, B, dY = (t.double() for t in dev)
    for k, o, main, low in (("Y", outs[0], X @ W.T, s * (X @ A.T) @ B.T), ("dX", outs[1], dY @ W, s * (dY @ B) @ A)):
        err = o.double() - (main + low)
        for dim in (0, 1):
            # each term strays by the tolerance of its own norm; the two may cancel (beside an outlier they do, in a few entries)
            bound = tol(T, din, dout) * (main.norm(dim=dim) + low.norm(dim=dim))
            assert bool((err.norm(dim=dim) <= 2 * bound).all()), (k, dim)


# Fragments straight from memory: both tiles (DIRECT32: 32x32 for the main products; the others 16x16, but for the one of 1157 tokens, which is split),
# sides one off a multiple of the tile, contractions shorter than one piece of sixteen elements, one off it, and of fewer pieces than there are waves.
DIRECT16 = [(17, 15, 33, 1), (16, 128, 16, 16), (31, 129, 47, 17), (48, 127, 2000, 5), (2, 3000, 1, 2), (1382, 182, 120, 33), (1400, 16, 96, 15)]
DIRECT32 = [(631, 389, 961, 4), (301, 1001, 999, 17), (129, 2047, 2050, 15), (1001, 129, 1100, 31)]


@pytest.mark.parametrize("T,din,dout,r", DIRECT16 + DIRECT32 + [(1157, 377, 486, 64)])
def test_direct_fragments(T, din, dout, r):
    ins, s = make(T, din, dout, r), 1.5
    dev = [t.cuda() for t in ins]
    shapes = ((T, dout), (T, din), (r, din), (dout, r))
    flat = [torch.full((a * b + 64,), 3.0, device="cuda") for a, b in shapes]
    outs = [f[:a * b].view(a, b) for f, (a, b) in zip(flat, shapes)]
    step(dev, s, outs, torch.empty_like(dev[2]), torch.empty_like(dev[3]))
    ref = reference(ins, s)
    for k, o, f in zip(("Y", "dX", "dA", "dB"), outs, flat):
        assert (o.cpu().double() - ref[k]).norm() < tol(T, din, dout) * ref[k].norm(), k
        assert bool((f[o.numel():] == 3.0).all()), k


# Operands whose scale varies along the contraction: what is small in X (dY) meets what is not small in W, and may be all that an output
# is made of.  `e`: binary orders between the two scales.  "blocks": W is block-diagonal, so that half of the outputs see the small half of
# X only; "period": the same with every fourth element large; "balanced": W is small where X is large.  The factors are zero (balanced: small)
# where X is large, so that the low-rank term has the outputs' scale.
@pytest.mark.parametrize("T,din,dout,r", SPLIT[:2])
@pytest.mark.parametrize("pattern", ["blocks", "period", "balanced"])
@pytest.mark.parametrize("e", [14, 20, 28, 36])
def test_scale_varies_along_the_contraction(T, din, dout, r, pattern, e):
    ins, s = make(T, din, dout, r), 1.5
    X, W, A, B, dY = ins
    big_in, big_out = ((torch.arange(n) % 4 == 0) if pattern == "period" else (torch.arange(n) < n // 2) for n in (din, dout))
    X[:, big_in] *= 2.0 ** e
    dY[:, big_out] *= 2.0 ** e
    if pattern == "balanced":
        for t in (W, A):
            t[:, big_in] *= 2.0 ** -e
        for t in (W, B):
            t[big_out] *= 2.0 ** -e
    else:
        W[big_out[:, None] != big_in[None, :]] = 0
        A[:, big_in] = 0
        B[big_out] = 0
    dev = [t.cuda() for t in ins]
    outs = [torch.empty(*size, device="cuda") for size in ((T, dout), (T, din), (r, din), (dout, r))]
    step(dev, s, outs, torch.empty_like(dev[2]), torch.empty_like(dev[3]))
    X, W, A, B, dY = (t.double() for t in dev)
    for k, o, main, low in (("Y", outs[0], X @ W.T, s * (X @ A.T) @ B.T), ("dX", outs[1], dY @ W, s * (dY @ B) @ A)):
        err = (o.double() - (main + low)).norm(dim=0)          # (of each column: its outputs have one scale)
        bound = 2 * tol(T, din, dout) * (main.norm(dim=0) + low.norm(dim=0))
        assert bool((err <= bound).all()), (k, (err / bound).max())


# Operands of one sign: what a sum leaves out does not cancel.  Random mantissas, and ones whose bits are all set; the low-rank term is
# far larger than any one product.  Roundings stay at random: the walk of a chain without the doubling of `tol`.
@pytest.mark.parametrize("T,din,dout,r", [(512, 1024, 1536, 16)] + SPLIT[:2])
@pytest.mark.parametrize("values", ["random", "all bits set"])
def test_operands_of_one_sign(T, din, dout, r, values):
    ins = [t.abs() + 0.1 if values == "random" else torch.full_like(t, 2 - 2.0 ** -23) for t in make(T, din, dout, r)]
    s = 1.5
    dev = [t.cuda() for t in ins]
    outs = [torch.empty(*size, device="cuda") for size in ((T, dout), (T, din), (r, din), (dout, r))]
    step(dev, s, outs, torch.empty_like(dev[2]), torch.empty_like(dev[3]))
    ref = reference(dev, s)
    for k, o in zip(("Y", "dX", "dA", "dB"), outs):
        err = ((o.double() - ref[k]).norm() / ref[k].norm()).item()
        assert err < tol(T, din, dout) / 2, (k, err)


# Values far below the others of a tile, down to fp32's smallest: they change no output but their own, and cost none its route.
@pytest.mark.parametrize("T,din,dout,r", SPLIT[:2])
@pytest.mark.parametrize("value", [1.2345678e-36, 1.1754944e-38, 9.2e-41, 1.4e-45])
def test_a_tiny_value_changes_no_other_output(T, din, dout, r, value):
    ins, s = make(T, din, dout, r), 1.5
    got = []
    for v in (0.0, value):
        ins[0][5, -1] = ins[4][7, 0] = v
        dev = [t.cuda() for t in ins]
        outs = [torch.empty(*size, device="cuda") for size in ((T, dout), (T, din), (r, din), (dout, r))]
        step(dev, s, outs, torch.empty_like(dev[2]), torch.empty_like(dev[3]))
        got.append(outs)
    assert torch.equal(torch.cat([got[0][0][:5], got[0][0][6:]]), torch.cat([got[1][0][:5], got[1][0][6:]]))
    assert torch.equal(torch.cat([got[0][1][:7], got[0][1][8:]]), torch.cat([got[1][1][:7], got[1][1][8:]]))


# Operands and sums beyond what the scaled parts and their accumulators hold, all of them or a few rows, and scales of the low-rank term that would move that.
@pytest.mark.parametrize("T,din,dout,r", SPLIT[:2])
@pytest.mark.parametrize("what", ["operands", "one operand", "sums", "one sum", "small s", "large s"])
def test_split_operands_beyond_the_scaled_parts(T, din, dout, r, what):
    ins, s = make(T, din, dout, r), 1.5
    X, W, A, B, dY = ins
    if what == "operands": X *= 2.0 ** 108; W *= 2.0 ** -100; A *= 2.0 ** -100; dY *= 2.0 ** -10
    elif what == "one operand": X[9, 3] = 2.0 ** 106; W[:, 3] *= 2.0 ** -90; A[:, 3] *= 2.0 ** -100
    elif what == "sums": X *= 2.0 ** 50; W *= 2.0 ** 40; B *= 2.0 ** 40
    elif what == "one sum": X[9] *= 2.0 ** 90; dY[3] *= 2.0 ** 90
    elif what == "small s": s = 2.0 ** -40; A *= 2.0 ** 30; B *= 2.0 ** 12
    elif what == "large s": s = 2.0 ** 40; A *= 2.0 ** -35
    dev = [t.cuda() for t in ins]
    outs = [torch.empty(*size, device="cuda") for size in ((T, dout), (T, din), (r, din), (dout, r))]
    step(dev, s, outs, torch.empty_like(dev[2]), torch.empty_like(dev[3]))
    X, W, A, B, dY = (t.double() for t in dev)
    for k, o, main, low in (("Y", outs[0], X @ W.T, s * (X @ A.T) @ B.T), ("dX", outs[1], dY @ W, s * (dY @ B) @ A)):
        err = (o.double() - (main + low)).norm(dim=1)
        assert bool((err <= 2 * tol(T, din, dout) * (main.norm(dim=1) + low.norm(dim=1))).all()), k


# Short contractions (in place, where each product is a launch of its own: Y where d_in is the short side, dX where d_out is), the first two too
# short for the split kernel, the others of one or two of its tiles: no further from fp64 than a chain of fused multiply-adds in fp32, which is
# emulated (but for the chain that leads to H or dH, of 4100 elements at most beside a term of a hundredth of the result: 1 %).
SHORT = [(1400, 8, 4100, 3), (8192, 4100, 8, 3), (1400, 32, 4100, 1), (1400, 33, 4100, 3), (1400, 63, 4100, 8), (8192, 4100, 32, 3), (1400, 4100, 63, 3)]


@pytest.mark.parametrize("T,din,dout,r", SHORT)
def test_short_contractions(T, din, dout, r):
    ins, s = make(T, din, dout, r), 1.5
    dev = [t.cuda() for t in ins]
    ref = reference(dev, s)
    X, W, A, B, dY = (t.clone() for t in dev)
    outs = [torch.empty(*size, device="cuda") for size in ((T, dout), (T, din), (r, din), (dout, r))]
    step(dev, s, outs, dev[2], dev[3])

    def chain(a, b):      # (a product of two floats is exact in fp64)
        c = torch.zeros(a.shape[0], b.shape[1], device="cuda")
        for k in range(a.shape[1]):
            c = (c.double() + a[:, k:k + 1].double() * b[k:k + 1].double()).float()
        return c

    k, o = ("Y", outs[0]) if din < dout else ("dX", outs[1])
    want = chain(X, W.T) + s * chain((X.double() @ A.double().T).float(), B.T) if k == "Y" else chain(dY, W) + chain((s * dY.double() @ B.double()).float(), A)
    err, err_chain = ((t.double() - ref[k]).norm().item() for t in (o, want))
    assert err <= 1.01 * err_chain, err / err_chain


# A contraction of which a few large products are almost all (a gradient that is a softmax): a chain rounds a few times at the size of the result and
# the parts some four times each.  A few roundings of at most 2^-24 each, at random: 2 * 2^-24 (a chain 1.0 to 1.1 of them).
@pytest.mark.parametrize("T,din,dout,r", SPLIT[:2])
def test_a_few_large_products(T, din, dout, r):
    ins, s = make(T, din, dout, r), 1.5
    ins[4] = torch.softmax(ins[4] * 25, -1)
    ins[0] = torch.softmax(ins[0] * 25, -1)
    dev = [t.cuda() for t in ins]
    outs = [torch.empty(*size, device="cuda") for size in ((T, dout), (T, din), (r, din), (dout, r))]
    step(dev, s, outs, torch.empty_like(dev[2]), torch.empty_like(dev[3]))
    ref = reference(dev, s)
    for k, o in zip(("Y", "dX"), outs):
        err = ((o.double() - ref[k]).norm() / ref[k].norm()).item()
        assert err < 2 * 2.0 ** -24, (k, err)
