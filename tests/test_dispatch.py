"""Launch selection of the Log-Int-Softmax kernels, on the CPU: the kernel, the
wavefronts and the workgroups that calls of every size reach."""
import pytest

LIMIT = 2 ** 32         # work-items of a launch


def threads(p):
    """Work-items along the launch's first dimension (unit kernel: units)."""
    return p.blocks // p.split * 64 * p.waves


# Few rows a unit and many units (up to about 3000): four wavefronts a unit, of
# which one had a tile, took 2048 units of 1 x 64 from 4.0 to 8.8 us and 2900 of
# 16 x 16 from 4.9 to 9.8.
@pytest.mark.parametrize("G", [1, 48, 700, 1024, 1500, 2048, 2900, 3072, 6000])
@pytest.mark.parametrize("Lq,Lk", [(1, 5), (16, 16), (17, 17), (1, 64), (9, 64), (16, 64), (33, 33),
                                   (49, 49), (49, 100), (64, 128)])
def test_fused_short_units_have_no_idle_wavefronts(plan, G, Lq, Lk):
    tiles = -(-Lq // 16)
    p = plan.head(G, Lq, Lk, 64)
    assert p.kernel == "unit"
    assert p.waves <= tiles and p.split <= -(-tiles // p.waves)


def test_fused_float_rows_take_the_unit_kernel(plan):
    """Rows of up to 640 keys on the float path, d <= 64, at every size."""
    for G in (1, 3, 24, 96, 256, 300, 520, 768, 2000, 10000):
        for L in (1, 32, 33, 197, 224, 225, 257, 288, 289, 320, 321, 577, 640):
            assert plan.head(G, L, L, 64).kernel == "unit"
    assert plan.head(3, 641, 641, 64).kernel == "stream"
    assert plan.head(3, 197, 197, 65).kernel == "stream"
    assert plan.head(3, 197, 197, 64, codes_out=True).kernel == "stream"
    # the integer path; a plane too large for the unit kernel's offsets
    assert plan.head(3, 197, 197, 64, s=2.0 ** -12).kernel == "tile"
    assert plan.head(3, 289, 289, 64, s=2.0 ** -12).kernel == "stream"
    assert plan.head(1, 2 ** 29 // 197 + 1, 197, 64).kernel == "tile"


def test_fused_short_rows_fill_the_last_pass(plan):
    """A few units more than the CUs (or a multiple of them) ran a whole second
    pass: 300 units of 288 x 288 38.6 us undivided and 33.5 divided, 520 of 257 x
    257 with a bias 84 and 70.  Even loads are not divided: 768 units of 257 x
    257 56 us undivided and 73 divided."""
    assert plan.head(300, 288, 288, 64).split > 1
    assert plan.head(520, 257, 257, 48, Hb=3).split > 1
    assert plan.head(768, 257, 257, 64).split == 1
    assert plan.head(48, 197, 197, 64).split == 4       # one tile a wavefront
    assert plan.head(768, 197, 197, 64).split == 1
    assert plan.head(6144, 49, 49, 32).split == 1
    # no division leaves a wavefront without a tile
    for G in (1, 100, 200, 300, 400):
        for L in (65, 145, 197, 257, 400, 577):
            p = plan.head(G, L, L, 64)
            tiles = -(-L // 16)
            assert (p.split - 1) * p.waves < tiles


def test_fused_rows_of_320_keys_are_divided_evenly(plan):
    """Rows of 257 to 320 keys, fewer units than CUs: as many workgroups as fill
    the slots could leave some CUs with one more than the others (200 units of 288
    x 288 29.1 us with two a unit, 27.7 with five; 180 of 300 x 300 with a bias
    29.9 and 26.1).  More units, and two workgroups a unit are the better ones
    again (240 of 257 x 257 24.3 us, 28.1 with five)."""
    assert plan.head(200, 288, 288, 64).split == 5
    assert plan.head(180, 300, 300, 32, Hb=3).split == 5
    assert plan.head(160, 257, 257, 64).split == 3
    assert plan.head(240, 257, 257, 64).split == 2
    assert plan.head(60, 320, 320, 64).split == 5


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("Lq,Lk", [(1, 225), (16, 577), (33, 577), (100, 400), (325, 325), (400, 400),
                                   (577, 577), (640, 640), (49, 49), (197, 197)])
def test_stored_codes_have_no_idle_wavefronts(plan, Lq, Lk, bits):
    """A tile a wavefront, none without one: eight wavefronts a workgroup took
    3000 units of 16 x 577 from 49 to 138 us, four-tile walks 300 of 400 x 400
    from 54 to 77."""
    tiles = -(-Lq // 16)
    for G in (1, 144, 300, 520, 1000, 3000):
        p = plan.codes(G, Lq, Lk, bits=bits)
        if p.kernel == "tile":
            assert Lk <= 288 and Lk % 32 and Lq > 8
            assert 256 < G * tiles <= (2816 if Lk <= 64 and tiles >= 4 else 1024 if bits == 4 else 0)
        else:
            assert p.kernel == "unit" and p.waves == 1 and p.split == tiles
            assert p.gathered >= 16 * (Lk if bits > 4 else (Lk + 1) // 2)


def test_stored_codes_kernels(plan):
    """Rows with padding: the unit kernel up to 224 keys; the integer path and
    longer rows as before."""
    assert plan.codes(1500, 49, 49, pad=1).kernel == "unit"
    assert plan.codes(1500, 49, 49, pad=1).gathered == 0
    assert plan.codes(700, 49, 225, pad=1).kernel == "tile"
    assert plan.codes(700, 49, 49, s=2.0 ** -12).kernel == "tile"
    assert plan.codes(3, 641, 641).kernel == "stream"


def test_launches_stay_within_the_grid(plan):
    """Calls of many units stay below 2^32 work-items, and as many units are
    accepted as one 256-thread workgroup a unit allows."""
    for G in (2 ** 22, 2 ** 23, 2 ** 24 - 1):
        for Lk in (1, 33, 197, 225, 288, 320):
            assert threads(plan.head(G, 1, Lk, 16)) < LIMIT
    for Lk in (321, 640):
        assert threads(plan.head(2 ** 23 - 1, 1, Lk, 16)) < LIMIT
    # (units, parts): each dimension of the grid by itself
    for G, Lq in ((2 ** 23, 1), (2 ** 24 - 1, 16), (2 ** 24, 64), (3, 2 ** 22)):
        for Lk in (1, 64):
            for bits in (4, 8):
                p = plan.codes(G, Lq, Lk, bits=bits)
                assert p.kernel == "unit" and G * 64 * p.waves < LIMIT and p.split <= 65535
    # rows of more than 320 keys: eight wavefronts a unit refused 2^23 units
    for G in (2 ** 23, 2 ** 24 - 1):
        for Lk in (321, 640):
            for bits in (4, 8):
                p = plan.codes(G, 1, Lk, bits=bits)
                assert G * 64 * p.waves < LIMIT
