"""Units divided over several workgroups (few units, many query rows), the long
rows of the unit kernels, and the requantization on both sides of its 32-bit
shift, against the oracle bit for bit."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

S = 2.0 ** -10


@pytest.fixture(scope="module")
def fq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2111_13824_amd as fq
    return fq


def dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


def host(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


# G, Lq, Lk, d, Hb: one workgroup to one a tile; last tiles of 1 and 15 rows;
# first and last chunk counts of each kernel family (7 | 8, 14 | 15, 20) with
# last chunks of 1, 16, 17 and 32 keys; d that takes the byte-wise V loads
HEADS = [(1, 300, 225, 64, 0), (5, 257, 256, 32, 5), (150, 143, 240, 64, 3), (2, 129, 448, 48, 0),
         (260, 33, 449, 64, 2), (3, 200, 480, 20, 3), (2, 145, 640, 64, 0), (300, 31, 577, 32, 0),
         (90, 113, 33, 64, 4), (700, 65, 49, 32, 7)]


@pytest.mark.parametrize("G,Lq,Lk,d,Hb", HEADS)
def test_divided_heads(fq, orc, G, Lq, Lk, d, Hb):
    print("CASE divided head", G, Lq, Lk, d, Hb, flush=True)
    a = W.attn_inputs(G, Lq, Lk, d, seed=G + Lk, heads=max(Hb, 1), sigma=(1.0, 3.0, 6.0),
                      bias=Hb > 0, v_lo=-128, v_hi=127)
    got = host(fq.lis_attention_head(dev(a["logits"]), dev(a["v"]), S, zp_v=-3,
                                     bias=dev(a["bias"]) if Hb else None))
    assert np.array_equal(got, orc.lis_attention_head(a["logits"], a["v"], S, zp_v=-3,
                                                      bias=a["bias"]))


@pytest.mark.parametrize("G,Lq,Lk,bits", [(300, 130, 225, 8), (40, 300, 448, 4), (260, 33, 449, 8),
                                          (30, 200, 640, 8), (200, 40, 577, 3)])
def test_long_code_rows(fq, orc, G, Lq, Lk, bits):
    """Dense code rows of more than 224 keys, guard bytes on both sides."""
    import torch
    print("CASE long codes", G, Lq, Lk, bits, flush=True)
    a = W.attn_inputs(G, Lq, Lk, 1, seed=G + Lk, heads=3, sigma=(1.0, 3.0, 9.0))
    nb = Lk if bits > 4 else (Lk + 1) // 2
    buf = torch.full((G * Lq * nb + 70,), 0xA5, dtype=torch.uint8, device="cuda:0")
    codes = buf[3:3 + G * Lq * nb].view(G, Lq, nb)
    fq.lis_softmax_log4(dev(a["logits"]), S, bits=bits, codes=codes)
    assert np.array_equal(host(codes), orc.lis_softmax_log4(a["logits"], S, bits=bits))
    edge = host(buf)
    assert np.all(edge[:3] == 0xA5) and np.all(edge[3 + G * Lq * nb:] == 0xA5)


@pytest.mark.parametrize("G,Lq,Lk,d,bits", [(1, 300, 130, 64, 8), (3, 205, 197, 32, 8),
                                            (2, 129, 1024, 64, 6), (5, 70, 65, 48, 5),
                                            (2, 200, 100, 64, 4), (600, 33, 40, 16, 8)])
def test_divided_products(fq, orc, G, Lq, Lk, d, bits):
    """The product with units divided over workgroups; codes above W (the
    floor path) in some tiles only; extreme V, whose range sums are largest."""
    print("CASE divided product", G, Lq, Lk, d, bits, flush=True)
    rng = np.random.default_rng(G * Lk + d + bits)
    top = min(2 ** bits - 1, 44)
    codes = rng.integers(0, top + 1, size=(G, Lq, Lk))
    codes[0, :20] = rng.integers(0, 7, size=(20, Lk))      # every P large
    v = rng.choice([-128, 127], size=(G, Lk, d)).astype(np.int8)

    def store(c):
        if bits >= 5:
            return c.astype(np.uint8)
        packed = np.zeros((G, Lq, (Lk + 1) // 2), dtype=np.uint8)
        packed |= c[..., 0::2].astype(np.uint8)
        packed[..., :Lk // 2] |= (c[..., 1::2] << 4).astype(np.uint8)
        return packed
    over = codes.copy()
    if bits >= 6:
        over[0, 67 % Lq, Lk - 1] = 2 ** bits - 1
        over[G - 1, Lq - 1, 0] = 45
    for c in (codes, over):
        pk = store(c)
        got = host(fq.lis_attn_v_shift_wide(dev(pk), dev(v), Lk, zp_v=9, bits=bits))
        assert np.array_equal(got, orc.lis_attn_v_shift_wide(pk, v, zp_v=9, bits=bits, Lk=Lk))
    if bits <= 4:
        pk = store(codes)
        got = host(fq.lis_attn_v_shift(dev(pk), dev(v), Lk, zp_v=9, bits=bits))
        assert np.array_equal(got, orc.lis_attn_v_shift(pk, v, zp_v=9, bits=bits, Lk=Lk))


@pytest.mark.parametrize("G,Lq,Lk,dk,s", [(1, 300, 225, 64, S), (20, 143, 577, 32, S),
                                          (3, 129, 640, 64, S), (2, 200, 300, 64, 2e-4),
                                          (150, 197, 197, 32, 2.0 ** -8), (40, 65, 449, 64, 0.02)])
def test_divided_qk(fq, orc, G, Lq, Lk, dk, s):
    print("CASE divided qk", G, Lq, Lk, dk, s, flush=True)
    x = W.qk_inputs(G, Lq, Lk, dk, dk, seed=G + Lk, sigma=19.6, zp_q=5, zp_k=-9, heads=2, bias=True)
    got = host(fq.lis_attention_qk(dev(x["q"]), dev(x["k"]), dev(x["v"]), s, 5, -9, zp_v=4,
                                   bias=dev(x["bias"])))
    assert np.array_equal(got, orc.lis_attention_qk(x["q"], x["k"], x["v"], s, 5, -9, zp_v=4,
                                                    bias=x["bias"]))


@pytest.mark.parametrize("M", [0.6, 0.5, 0.49999997, 0.25, 2.0 ** -31, 1.5 * 2.0 ** -32, 3.0])
def test_requant_both_shifts(fq, orc, M):
    """N1 = 31 and 32 around M = 1/2, the deepest shifts, and M above 1."""
    print("CASE requant shift", M, flush=True)
    rng = np.random.default_rng(7)
    q = rng.integers(-2 ** 31, 2 ** 31, size=40001).astype(np.int32)
    near = np.rint(rng.uniform(-140, 140, size=20000) / M)
    q[:40000:2] = np.clip(near, -2 ** 31, 2 ** 31 - 1).astype(np.int64).astype(np.int32)
    q[-5:] = [0, 1, -1, 2 ** 31 - 1, -2 ** 31]
    for zp, bits in ((0, 8), (-128, 8), (3, 4)):
        got = host(fq.requant_dyadic_int8(dev(q), M, 1.0, zp, bits))
        assert np.array_equal(got, orc.requant_dyadic_int8(q, M, 1.0, zp, bits))
