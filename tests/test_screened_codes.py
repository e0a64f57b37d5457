"""The screened float path of the fused attention kernels: codes from binary32
values, with every decision that rounding could have changed detected and
taken again exactly.  On the CPU the formulas themselves (I-Exp over every
input; the code is right wherever the screen does not call it undecided, and
exact ties are always undecided); on the GPU, kernels on rows built to sit on
the thresholds."""
import numpy as np
import pytest

import workloads as W

# Largest relative error of a lane's binary32 tree sum of depth 3.
TREE = 3.01 * 2.0 ** -24
ZONE = 16


def _consts(orc, s, n):
    k = orc.iexp_constants(s, n)
    d, qb, qc = -k.q_ln2, int(k.q_b), int(k.q_c)
    pre = 0
    while (d << pre) <= 512:
        pre += 1
    return k, dict(d=d, qb=qb, qc=qc, n=n, pre=pre, magic=(1 << 32) // (d << pre))


@pytest.mark.parametrize("s", [0.5, 0.05, 2.0 ** -8, 2.0 ** -10, 0.00042])
@pytest.mark.parametrize("n", [1, 8, 20, 30])
def test_screen_iexp_every_input(orc, s, n):
    """-z = floor(a / d) by the signed 24-bit multiply-high of a = d - 1 - u,
    the float 2^23 + (a + z d) built as an integer, one add and one fma."""
    k, f = _consts(orc, s, n)
    assert f["qb"] ** 2 + f["qc"] < 2 ** 24 and f["magic"] < 2 ** 23
    u = np.arange(n * f["d"] + 4, dtype=np.int64)
    a = np.maximum(f["d"] - 1 - u, f["d"] - 1 - n * f["d"])
    assert np.all(np.abs(a << f["pre"]) < 2 ** 23)
    nz = ((a << f["pre"]) * f["magic"]) >> 32
    bits = nz * -f["d"] + a + 0x4B000000
    w = bits.astype(np.uint32).view(np.float32) + np.float32(f["qb"] - f["d"] + 1 - 2 ** 23)
    ql = (w.astype(np.float64) ** 2 + f["qc"]).astype(np.float32)     # the fma is exact
    e = ((nz << 23) + ql.view(np.int32)).astype(np.int32).view(np.float32)
    ref = np.array([orc.iexp(-int(x), k)[0] for x in u], dtype=np.float64)
    assert np.array_equal(e.astype(np.float64) * 2.0 ** n, ref)


def _screen(e, S, top, e0, exact):
    """(codes, undecided) of e and the row sums S (2^-n scaled, float64); e0 the
    row maximum's e, exact the row sum without error (which decides 2S < 3 e0)."""
    T = min(top, 62) + 1
    xs = (S * (4 / 3 * (1 + 6 * 2.0 ** -24) * 2.0 ** -T)).astype(np.float32)
    c = np.float32(float.fromhex("0x1.555556p-1") * 2.0 ** -T)
    tau = np.float32(0.75 * e0 if exact < 1.5 * e0 else np.inf)
    # binary64 holds e c exactly and the sum to 2^-53: rounding it to binary32
    # is the fma's result or a neighbour within the stated bound
    y = (e.astype(np.float64) * np.float64(c) + xs.astype(np.float64)).astype(np.float32)
    y = np.where(e > tau, xs, y)
    b = np.maximum(e.view(np.int32).astype(np.int64) - y.view(np.int32).astype(np.int64), 0)
    return min(top, 62) - (b >> 23), (b & (2 ** 23 - 1)) >= 2 ** 23 - ZONE


@pytest.mark.parametrize("top", [3, 15, 255])
def test_screen_decides_only_what_rounding_cannot_change(top):
    """Keys e placed on and around every threshold 2S = c_k e (c_1 = 3, c_k =
    3 2^(k-1) - 1) and at random, with S off by up to the tree's error: where
    the screen decides, its code is that of the exact S."""
    rng = np.random.default_rng(top)
    caught = 0
    for trial in range(40):
        e0 = int(rng.integers(2 ** 20, 2 ** 22))
        S = int(rng.integers(e0, 200 * e0)) << 20
        if trial % 4 == 3:      # 2S = 3 e0 and beside it
            S = (3 * e0 << 19) + int(rng.integers(-3, 4))
        es = []
        for k in range(1, 45):
            ck = 3 if k == 1 else 3 * 2 ** (k - 1) - 1
            t = (2 * S) // ck
            sh = max(t.bit_length() - 22, 0)
            es += [((t >> sh) + j) << sh for j in range(-3, 4)]
        es += [int(x) << int(y) for x, y in zip(rng.integers(2 ** 20, 2 ** 22, 200),
                                                rng.integers(0, 21, 200))]
        es = sorted({x for x in es if 0 < x <= e0 << 20 and x <= S})
        r = [(2 * S + x) // (2 * x) for x in es]
        # I-Log2 of the rounded quotient, floor(log2(4 r / 3)), cut at top
        ref = np.array([min(((4 * q) // 3).bit_length() - 1, top) for q in r])
        e = np.array([x * 2.0 ** -20 for x in es]).astype(np.float32)
        for err in (-TREE, 0.0, TREE):
            Sf = np.full(e.shape, S * 2.0 ** -20 * (1 + err))
            code, und = _screen(e, Sf, top, e0, S * 2.0 ** -20)
            # only the row maximum can be above 2S / 3
            ok = ~und & ((np.array(es) * 3 <= 2 * S) | (e == np.float32(e0)))
            assert np.array_equal(code[ok], ref[ok])
            caught += int(und.sum())
    assert caught > 0


def test_screen_exact_ties_are_undecided():
    """2S = c_k e exactly: undecided whatever the error of S."""
    for k in range(2, 16):
        ck = 3 * 2 ** (k - 1) - 1
        for m in (2 ** 21 + 2, 2942328, 3 * 2 ** 20):
            for err in (-TREE, 0.0, TREE):
                code, und = _screen(np.array([m], dtype=np.float32),
                                    np.array([m * ck / 2 * (1 + err)]), 15, 2.0 * m, m * ck / 2)
                assert und[0]


def test_screen_ties_of_the_maximum_are_decided():
    """2S = 3 e0 and sums beside it: code 1 or 0 by the exact sum, never by a
    whole row left undecided (rows of 577 keys took 13 us more for it)."""
    for e0 in (2 ** 21 + 2, 2942328, 3 * 2 ** 20):
        for unit in (0, 1, 5, 2 ** 10):
            for sign in (-1, 1):
                S = 1.5 * e0 + sign * unit * 2.0 ** -20
                far = e0 * 2.0 ** -12      # a key of the rest of the row
                code, und = _screen(np.array([e0, far], dtype=np.float32), np.full(2, S), 15, e0, S)
                assert not und[1]
                if S >= 1.5 * e0:
                    assert code[0] == 1 and not und[0]
                else:
                    assert code[0] == 0 or und[0]


# ---------------------------------------------------------------------------
# GPU
# ---------------------------------------------------------------------------

def _tie_logits(rng, G, Lq, Lk, d):
    """Rows whose I-Exp values are the maximum's times powers of two (logits
    multiples of d = |q_ln2|), a few keys near the maximum and the rest far
    below: row sums such as 5/2 or 11/2 of a key, or 3/2 of the maximum, fall
    on the thresholds exactly or to within the clamped keys' sum."""
    z = rng.integers(10, 40, size=(G, Lq, Lk))
    near = rng.integers(0, min(Lk, 7) + 1, size=(G, Lq))
    for g in range(G):
        for i in range(Lq):
            j = rng.choice(Lk, size=near[g, i], replace=False)
            z[g, i, j] = rng.integers(0, 4, size=j.size)
    z[:, ::5] = np.where(z[:, ::5] < 10, z[:, ::5], 100)   # nothing between
    return (-z * d + rng.integers(-50, 50, size=(G, Lq, 1))).astype(np.int32)


@pytest.fixture(scope="module")
def fq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_13824_amd as fq
    return fq


SHAPES = [(1024, 17, 5, 32), (700, 33, 49, 32), (520, 49, 130, 64), (512, 70, 197, 64),
          (512, 50, 224, 64), (24, 60, 197, 64), (6, 40, 400, 64), (3, 50, 577, 48)]


@pytest.mark.gpu
@pytest.mark.parametrize("G,Lq,Lk,d", SHAPES)
@pytest.mark.parametrize("n", [20, 4])
def test_rows_on_the_thresholds(fq, orc, G, Lq, Lk, d, n):
    """The fused head, the stored codes (4 and 8 bits) and the attention from Q
    and K (Q zero, so that its logits are the bias) on such rows (rows of more
    than a few keys come near the thresholds only: the keys far below add up;
    test_rows_on_exact_thresholds has them on the thresholds)."""
    import torch
    print("CASE screened ties", G, Lq, Lk, d, n, flush=True)
    rng = np.random.default_rng(G + Lk + n)
    s = 2.0 ** -10
    lg = _tie_logits(rng, G, Lq, Lk, -orc.iexp_constants(s, n).q_ln2)
    v = rng.integers(-128, 128, size=(G, Lk, d)).astype(np.int8)
    dl, dv = torch.from_numpy(lg).cuda(), torch.from_numpy(v).cuda()
    ref = orc.lis_attention_head(lg, v, s, exp_n=n, zp_v=5)
    assert np.array_equal(fq.lis_attention_head(dl, dv, s, exp_n=n, zp_v=5).cpu().numpy(), ref)
    for bits in (4, 8):
        got = fq.lis_softmax_log4(dl, s, bits=bits, exp_n=n).cpu().numpy()
        assert np.array_equal(got, orc.lis_softmax_log4(lg, s, bits=bits, exp_n=n))
    q = torch.zeros((G, Lq, 32), dtype=torch.int8, device="cuda")
    k = torch.zeros((G, Lk, 32), dtype=torch.int8, device="cuda")
    got = fq.lis_attention_qk(q, k, dv, s, exp_n=n, zp_v=5, bias=dl).cpu().numpy()
    assert np.array_equal(got, ref)


def _exact_tie_logits(rng, G, Lq, Lk, d, top):
    """Rows of logits -z d, z <= 20, whose I-Exp values are the maximum's times
    2^-z, with 2S = c_k e for a key e (c_1 = 3, c_k = 3 2^(k-1) - 1, k <= top):
    the sum as powers of two, split until there are Lk of them.  In one row of
    three a key of the smallest value is moved by up to two logits."""
    n = 20
    out = np.empty((G, Lq, Lk), dtype=np.int32)
    for row in out.reshape(-1, Lk):
        while True:
            k = int(rng.integers(1, min(top, 12) + 1))
            zj = 0 if k == 1 else int(rng.integers(max(k - 4, 0), k))
            M = 3 << (n - 1) if k == 1 else (3 * 2 ** (k - 1) - 1) << (n - zj - 1)
            z = [0] if zj == 0 else [0, zj]
            rest = M - sum(1 << (n - a) for a in z)
            if rest < 0:
                continue
            extra = [0] * (rest >> n) + [n - b for b in range(n) if rest >> b & 1]
            if len(z) + len(extra) <= Lk:
                break
        while len(z) + len(extra) < Lk:
            open_ = [i for i, a in enumerate(extra) if a < n]
            i = open_[int(rng.integers(len(open_)))]
            extra[i] += 1
            extra.append(extra[i])
        v = -np.array(z + extra, dtype=np.int64) * d
        if rng.integers(3) == 0:
            v[np.argmin(v)] += int(rng.integers(-2, 3))
        row[:] = rng.permutation(v) + int(rng.integers(-50, 50))
    return out


def _undecided_rows(orc, lg, s, n, top):
    """Rows with a key that the screen leaves open, or 2S within rounding of 3 e0."""
    k = orc.iexp_constants(s, n)
    u, inv = np.unique(lg.max(-1, keepdims=True).astype(np.int64) - lg, return_inverse=True)
    e = np.array([orc.iexp(-int(x), k)[0] for x in u], dtype=np.float64)[inv].reshape(lg.shape)
    e *= 2.0 ** -n
    count = 0
    for row in e.reshape(-1, lg.shape[-1]):
        _, und = _screen(row.astype(np.float32), np.full(row.shape, row.sum()), top, row.max(),
                         row.sum())
        count += bool(und.any() or abs(row.sum() / row.max() - 1.5) < 2.0 ** -20)
    return count


@pytest.mark.gpu
@pytest.mark.parametrize("s,bits", [(2.0 ** -8, 4), (2.0 ** -8, 3), (2.0 ** -10, 4), (2.0 ** -10, 3),
                                    (0.05, 4)])
@pytest.mark.parametrize("Lk", [12, 16, 33, 96, 120, 150, 176, 197, 224, 230, 288, 400, 448, 461, 577, 640])
def test_rows_on_exact_thresholds(fq, orc, plan, s, bits, Lk):
    """Every row on a threshold or beside one, at scales with the I-Exp pre-shift
    (above 1.3e-3) and without, codes cut at 7, 15 and 255, rows of each kernel,
    Q and K of both widths."""
    import torch
    G, Lq, d = 5, 24, (64, 32)[Lk % 2]
    print("CASE exact thresholds", s, bits, Lk, flush=True)
    rng = np.random.default_rng(Lk + bits)
    lg = _exact_tie_logits(rng, G, Lq, Lk, -orc.iexp_constants(s, 20).q_ln2, 2 ** bits - 1)
    assert _undecided_rows(orc, lg, s, 20, 2 ** bits - 1) > G * Lq // 2
    assert plan.head(G, Lq, Lk, d, s=s, bits=bits).kernel == "unit"
    v = rng.integers(-128, 128, size=(G, Lk, d)).astype(np.int8)
    dl, dv = torch.from_numpy(lg).cuda(), torch.from_numpy(v).cuda()
    ref = orc.lis_attention_head(lg, v, s, bits=bits, zp_v=5)
    got = fq.lis_attention_head(dl, dv, s, bits=bits, zp_v=5).cpu().numpy()
    assert np.array_equal(got, ref)
    for b in (bits, 8):
        assert plan.codes(G, Lq, Lk, s=s, bits=b).kernel == "unit"
        got = fq.lis_softmax_log4(dl, s, bits=b).cpu().numpy()
        assert np.array_equal(got, orc.lis_softmax_log4(lg, s, bits=b))
    for dk in (32, 64):
        q = torch.zeros((G, Lq, dk), dtype=torch.int8, device="cuda")
        k = torch.zeros((G, Lk, dk), dtype=torch.int8, device="cuda")
        got = fq.lis_attention_qk(q, k, dv, s, bits=bits, zp_v=5, bias=dl).cpu().numpy()
        assert np.array_equal(got, ref)
