"""Every instance of the Log-Int-Softmax unit kernel, against the oracle bit for
bit: chunk counts, half and full last chunks, V^T widths, wavefronts a
workgroup, wavefronts that walk several tiles of a unit.  Each test asks the
launch selection which kernel its sizes reach, so that a change of the selection
cannot leave an instance without a test."""
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


def _head(fq, orc, G, Lq, Lk, d, Hb, bits=4):
    print("CASE unit head", G, Lq, Lk, d, Hb, bits, flush=True)
    a = W.attn_inputs(G, Lq, Lk, d, seed=G + Lk + d, heads=max(Hb, 1), sigma=(1.0, 3.0, 6.0),
                      bias=Hb > 0, v_lo=-128, v_hi=127)
    got = host(fq.lis_attention_head(dev(a["logits"]), dev(a["v"]), S, zp_v=3, bits=bits,
                                     bias=dev(a["bias"]) if Hb else None))
    assert np.array_equal(got, orc.lis_attention_head(a["logits"], a["v"], S, zp_v=3, bits=bits,
                                                      bias=a["bias"]))


# Last chunks: the first and the last key count of the half and of the full form.
TAILS = ((True, 1), (True, 16), (False, 17), (False, 32))
# d of each V^T width: 16-byte V rows; V in pieces; scalar output stores
DIMS = {2: (32, 20, 17), 4: (64, 48, 33)}


@pytest.mark.parametrize("nc", range(1, 21))
def test_fused_instances(fq, orc, plan, nc):
    """Few units, at most one tile a wavefront; last tiles of 1 to 11 rows."""
    sizes = ((1, 11), (2, 33), (4, 97)) if nc <= 4 else ((4 if nc <= 10 else 8, 33),)
    n = 0
    for waves, Lq in sizes:
        for half, tail in TAILS:
            for dt, dims in DIMS.items():
                G, Lk, d, Hb = 2, 32 * (nc - 1) + tail, dims[n % 3], (0, 2)[n % 2]
                p = plan.head(G, Lq, Lk, d, Hb=Hb)
                assert (p.kernel, p.nc, p.dt, p.half, p.waves) == ("unit", nc, dt, half, waves)
                _head(fq, orc, G, Lq, Lk, d, Hb, bits=(4, 3)[n % 5 == 4])
                n += 1


# G, Lq, Lk, d, Hb: wavefronts walk several tiles, and prefetch the next one, in
# whole units and in units divided over several workgroups; last tiles of one
# row among them (the one-row path of rows of up to two chunks)
WALKS = [(1600, 49, 20, 64, 0), (1600, 64, 70, 32, 4), (3100, 33, 40, 17, 0), (800, 81, 100, 48, 5),
         (300, 305, 33, 64, 0), (300, 300, 64, 32, 3), (260, 209, 180, 64, 2), (300, 150, 224, 64, 0),
         (400, 81, 257, 64, 0), (300, 97, 320, 64, 0), (130, 145, 370, 64, 2), (100, 300, 430, 64, 0),
         (130, 145, 500, 32, 0), (130, 145, 640, 64, 2)]


@pytest.mark.parametrize("G,Lq,Lk,d,Hb", WALKS)
def test_fused_walks(fq, orc, plan, G, Lq, Lk, d, Hb):
    p = plan.head(G, Lq, Lk, d, Hb=Hb)
    tiles = -(-Lq // 16)
    assert p.kernel == "unit" and tiles > p.waves * p.split
    _head(fq, orc, G, Lq, Lk, d, Hb)


def test_walks_include_divided_units(plan):
    """Short and long rows whose units are divided and whose wavefronts still
    walk several tiles."""
    split = [p.nc for p in (plan.head(*w[:4], Hb=w[4]) for w in WALKS) if p.split > 1]
    assert min(split) <= 2 and 8 <= max(split)


def _codes(fq, orc, G, Lq, Lk, bits, pad, shift):
    import torch
    print("CASE unit codes", G, Lq, Lk, bits, pad, shift, flush=True)
    a = W.attn_inputs(G, Lq, Lk, 1, seed=3 * G + Lk + bits, heads=G, sigma=(1.0, 3.0, 9.0))
    nb = (Lk if bits > 4 else (Lk + 1) // 2) + pad
    n = G * Lq * nb
    buf = torch.full((n + shift + 70,), 0xA5, dtype=torch.uint8, device="cuda:0")
    fq.lis_softmax_log4(dev(a["logits"]), S, bits=bits, codes=buf[shift:shift + n].view(G, Lq, nb))
    edge = host(buf)
    got = edge[shift:shift + n].reshape(G, Lq, nb)
    assert np.array_equal(got[..., :nb - pad], orc.lis_softmax_log4(a["logits"], S, bits=bits))
    assert np.all(got[..., nb - pad:] == 0xA5)
    assert np.all(edge[:shift] == 0xA5) and np.all(edge[shift + n:] == 0xA5)


@pytest.mark.parametrize("nc", range(1, 21))
def test_stored_code_instances(fq, orc, plan, nc):
    """Dense rows at every offset from a dword boundary, and padded rows (unit
    kernel up to 224 keys, tile kernel beyond); guard bytes around the codes."""
    for n, (half, tail) in enumerate(TAILS):
        Lk = 32 * (nc - 1) + tail
        for bits in (4, 8, 3, 6)[n % 2::2]:
            p = plan.codes(3, 21, Lk, bits=bits)
            assert p.kernel == "unit" and p.gathered > 0 and (p.nc, p.half) == (nc, half)
            _codes(fq, orc, 3, 21, Lk, bits, 0, n)
        p = plan.codes(3, 21, Lk, bits=4, pad=2)
        assert p.kernel == ("unit" if nc <= 7 else "tile") and p.gathered == 0
        _codes(fq, orc, 3, 21, Lk, 4, 2, 1)


@pytest.mark.parametrize("nc", range(1, 10))
def test_stored_codes_tile_kernel(fq, orc, plan, nc):
    """Sizes whose codes the tile kernel stores from its registers."""
    Lk = 32 * nc - 13
    assert plan.codes(65, 62, Lk).kernel == "tile"
    _codes(fq, orc, 65, 62, Lk, 4, 0, 1)
    if nc <= 2:
        assert plan.codes(65, 62, Lk, bits=8).kernel == "tile"
        _codes(fq, orc, 65, 62, Lk, 8, 0, 3)
