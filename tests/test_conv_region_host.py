"""The input region that the matrix-core convolution keeps in LDS.

The library sizes the region by a bound over all tiles (bnn_testing_conv_region, no GPU) and the kernel derives each
tile's rows and every column's offset from its first and last pixel.  The kernel's half is modelled here; for random
geometries no tile may need more rows than the library's bound, and every word that a column reads must lie inside its
plane of the region, on the row of its own image, and every plane inside the region's bytes.  (The kernel itself is
compared with the oracle on the GPU.)"""
import ctypes
import random

import pytest

from paper_1911_04477_amd import binding as B


def region(*args):
    """bnn_testing_conv_region -> (rows, pixels per row, bytes between planes, bytes), or None / ValueError."""
    out = (ctypes.c_int64 * 4)()
    got = B.lib().bnn_testing_conv_region(*args, out)
    if got < 0:
        raise ValueError(args)
    return tuple(out) if got else None


def check_geometry(N, C, H, W, kH, kW, sH, sW, pH, pW, pool, bn):
    r = region(N, C, H, W, kH, kW, sH, sW, pH, pW, 2 if pool else 0, bn)
    if r is None:
        return False
    bound, Wp, plane, nbytes = r
    words = (C + 63) // 64
    # a row of an odd number of words reads its missing one from a plane of zeros
    assert plane * (words + (kH * kW * words) % 2) <= nbytes <= 100 * 1024
    OH, OW = (H + 2 * pH - kH) // sH + 1, (W + 2 * pW - kW) // sW + 1
    us = 2 if pool else 1  # output rows per unit
    units, ustep, uspan = OH // us, us * sH, (us - 1) * sH + kH
    full = (units - 1) * ustep + uspan

    def pixel(c):
        if not pool:
            t = c // OW
            return t // OH, t % OH, c % OW
        j, w = c & 3, c >> 2  # window-major
        t = w // (OW // 2)
        return t // (OH // 2), 2 * (t % (OH // 2)) + (j >> 1), 2 * (w % (OW // 2)) + (j & 1)

    P = N * OH * OW
    for n0 in range(0, P, bn):
        last = min(n0 + bn, P) - 1
        i0, oh0, _ = pixel(n0)
        i1, oh1, _ = pixel(last)
        u0, u1 = oh0 // us, oh1 // us
        rows0 = ((u1 if i0 == i1 else units - 1) - u0) * ustep + uspan
        rows = rows0 if i0 == i1 else rows0 + (i1 - i0 - 1) * full + u1 * ustep + uspan
        assert rows <= bound
        for c in range(n0, last + 1, max(1, (last - n0) // 9)):
            img, oh, ow = pixel(c)
            r = oh * sH - u0 * ustep if img == i0 else rows0 + (img - i0 - 1) * full + oh * sH
            for kh in (0, kH - 1):
                q = r + kh
                assert 0 <= q < rows
                if q >= rows0:
                    k = (q - rows0) // full
                    assert (i0 + 1 + k, q - rows0 - k * full - pH) == (img, oh * sH - pH + kh)
                else:
                    assert (i0, u0 * ustep - pH + q) == (img, oh * sH - pH + kh)
            assert ow * sW + kW <= Wp
            assert ((r + kH - 1) * Wp + ow * sW + kW) * 8 <= plane
    return True


@pytest.mark.parametrize("seed", range(6))
def test_region_bound_covers_every_tile(seed):
    rng = random.Random(seed)
    seen = 0
    while seen < 150:
        H, W, kH = rng.randint(1, 40), rng.randint(1, 40), rng.choice([1, 2, 3, 5, 7])
        kW, sH, sW = rng.choice([kH, 1, 3]), rng.choice([1, 1, 2, 3]), rng.choice([1, 1, 2, 3])
        pH, pW = rng.choice([0, kH // 2, 1, 3]), rng.choice([0, kW // 2, 1])
        if H + 2 * pH < kH or W + 2 * pW < kW:
            continue
        OH, OW = (H + 2 * pH - kH) // sH + 1, (W + 2 * pW - kW) // sW + 1
        pool = OH % 2 == 0 and OW % 2 == 0 and rng.random() < 0.6
        C = rng.choice([1, 64, 65, 128, 300])
        seen += check_geometry(rng.randint(1, 9), C, H, W, kH, kW, sH, sW, pH, pW, pool, rng.choice([128, 256]))


def test_rows_beyond_the_pitch_are_gathered():
    """Input rows of 4 GiB and more, of which one output column's taps read three pixels: the region would be small,
    but the pitch that the copy into it steps by is a 32-bit number of bytes."""
    for H, W, C, taken in ((3, 1 << 29, 1, False), (3, 1 << 29, 5, False), (2, (1 << 30) - 1, 4, False),
                           (3, (1 << 29) - 1, 1, True), (2, (1 << 29) - 1, 8, True)):
        assert (region(1, C, H, W, H, 3, 1, 1 << 30, 0, 0, 0, 256) is not None) == taken, (H, W, C)


def test_what_the_convolution_refuses_is_refused():
    for args in ((1, 64, 3, 3, 3, 3, 1, 1, 0, 0, 2, 128),    # one output pixel, pooled
                 (1, 64, 5, 6, 3, 3, 1, 1, 0, 0, 2, 128),    # three output rows, pooled
                 (1, 64, 2, 2, 3, 3, 1, 1, 0, 0, 0, 128),    # no output
                 (0, 64, 4, 4, 3, 3, 1, 1, 0, 0, 0, 128), (1, 64, 4, 4, 3, 3, 1, 1, 0, 0, 1, 128),
                 (1, 64, 4, 4, 3, 3, 1, 1, 0, 0, 0, 0)):
        with pytest.raises(ValueError):
            region(*args)


@pytest.mark.parametrize("N,C,H,W,D,k,packed,want", [
    (7, 64, 32, 32, 64, 3, 1, 1), (8, 64, 32, 32, 64, 3, 1, 2),        # one word: t = 1.75, 2
    (10, 64, 32, 16, 128, 3, 0, 1), (11, 64, 32, 16, 128, 3, 0, 2),    # maps: 2.5, 2.75
    (12, 65, 32, 32, 64, 3, 1, 1), (13, 65, 32, 32, 64, 3, 1, 2),      # two words: 3, 3.25
    (16, 128, 32, 32, 64, 3, 0, 1), (17, 128, 32, 32, 64, 3, 0, 2),    # maps: 4, 4.25
    (48, 129, 32, 32, 64, 3, 1, 1), (49, 192, 32, 32, 64, 3, 0, 2),    # three words: u = 0.75, 0.766
    (64, 256, 32, 32, 64, 3, 1, 1), (65, 256, 32, 32, 64, 3, 1, 2), (128, 256, 32, 32, 64, 3, 0, 2),  # four: 1, 1.016, 2
    (129, 256, 32, 32, 64, 3, 0, 1), (192, 256, 32, 32, 64, 3, 1, 1), (193, 256, 32, 32, 64, 3, 1, 2),  # 2.016, 3, 3.016
    (250, 128, 7, 7, 128, 3, 1, 1), (168, 128, 7, 8, 128, 3, 1, 2),    # small maps: t = 6, 4.6
    (1, 256, 1, 1, 1, 1, 1, 2), (1, 257, 32, 32, 64, 1, 1, 0), (200, 64, 32, 32, 64, 5, 1, 0)])
def test_conv_word_rule_lines(N, C, H, W, D, k, packed, want):
    """Both sides of every line of the rule for the kernel whose taps go straight to the matrix cores, on 256 compute units."""
    assert B.lib().bnn_testing_conv_word(N, C, H, W, D, k, k, 1, 1, k // 2, k // 2, 0, packed, 256) == want


@pytest.mark.parametrize("N,C,H,W,D,want", [
    (128, 192, 32, 32, 64, 2), (129, 192, 32, 32, 64, 1), (192, 129, 32, 32, 64, 1), (193, 129, 32, 32, 64, 2),  # three words: 1, 1.5
    (77, 256, 8, 30, 435, 1), (256, 256, 32, 32, 64, 2), (257, 256, 32, 32, 64, 1),  # four: 259 workgroups; two a unit ...
    (288, 256, 32, 32, 64, 1), (289, 256, 32, 32, 64, 2)])                           # ... and an eighth of a third
def test_conv_word_rule_lines_of_maps(N, C, H, W, D, want):
    """Maps of a few more workgroups of 512 pixels than one or two a unit: those left over last as long as all others."""
    assert B.lib().bnn_testing_conv_word(N, C, H, W, D, 3, 3, 1, 1, 1, 1, 0, 0, 256) == want


@pytest.mark.parametrize("N,C,H,W,D,k,s,outputs,want", [
    (64, 64, 15, 8, 64, 3, 1, 1, 1), (64, 64, 15, 8, 65, 3, 1, 1, 2),            # signs of one word: t = 1.875, 2.8
    (8, 64, 32, 16, 192, 3, 1, 0, 2), (8, 64, 32, 16, 193, 3, 1, 0, 1), (9, 64, 32, 16, 256, 3, 1, 0, 2),      # a map: 3, 3.5, 4.5
    (16, 64, 32, 16, 128, 3, 1, 2, 2), (12, 64, 32, 16, 128, 3, 1, 2, 1), (13, 64, 32, 16, 128, 3, 1, 2, 2),   # both: 4, 3, 3.25
    (48, 64, 32, 16, 32, 3, 1, 2, 2), (24, 64, 32, 16, 33, 3, 1, 2, 1),          # to 32 and 33 channels: 3
    (8, 64, 32, 16, 256, 3, 1, 2, 1), (9, 64, 32, 16, 256, 3, 1, 2, 2),          # to 256 channels: 4, 4.5
    (217, 192, 32, 32, 64, 3, 1, 2, 2), (218, 192, 32, 32, 64, 3, 1, 2, 1), (218, 192, 32, 32, 64, 3, 1, 0, 2),  # 1.7 workgroups a unit
    (218, 256, 32, 32, 64, 3, 1, 2, 1), (161, 256, 44, 10, 301, 3, 1, 2, 2),      # four; pieces of lines
    (1, 256, 31, 10, 64, 1, 2, 0, 2), (1, 256, 21, 31, 64, 1, 2, 0, 1), (1, 256, 21, 31, 32, 1, 2, 0, 2),      # 1 x 1: 160 pixels, 176
    (64, 256, 31, 15, 64, 1, 2, 0, 1), (65, 256, 31, 15, 64, 1, 2, 0, 2),        # four words: t = 2
    (25, 128, 31, 15, 128, 1, 2, 0, 2), (14, 128, 31, 15, 128, 1, 2, 0, 1), (15, 128, 31, 15, 128, 1, 2, 0, 2),  # two: 1.6, 0.9, 0.94
    (20, 128, 31, 15, 129, 1, 2, 0, 1), (21, 128, 31, 15, 129, 1, 2, 0, 2),      # to 129 channels: 1.56, 1.64
    (1, 256, 17, 9, 63, 1, 2, 0, 1), (1, 256, 17, 9, 64, 1, 2, 0, 2),            # 45 pixels: not to part of a tile's channels
    (64, 128, 11, 15, 256, 1, 2, 0, 1), (65, 128, 11, 15, 256, 1, 2, 0, 2),      # 48 pixels to 256 channels: 3
    (1, 64, 21, 31, 64, 1, 2, 0, 2), (1, 256, 21, 31, 64, 1, 2, 1, 2)])          # one word, signs
def test_conv_word_rule_lines_of_outputs(N, C, H, W, D, k, s, outputs, want):
    """Signs (1), a map (0) and both maps (2), few and many channels: both sides of every line between them."""
    assert B.lib().bnn_testing_conv_word(N, C, H, W, D, k, k, s, s, k // 2, k // 2, 0, outputs, 256) == want


@pytest.mark.parametrize("N,C,H,W,D,want", [
    (163, 256, 19, 36, 435, 0), (163, 256, 19, 36, 512, 0), (387, 256, 37, 20, 60, 0), (223, 192, 58, 10, 57, 0),  # rows computed for nothing
    (48, 256, 46, 18, 56, 1), (163, 256, 32, 8, 435, 1), (4, 128, 18, 12, 65, 1)])  # few rows; whole lines; small calls
def test_conv_word_map_stores(N, C, H, W, D, want):
    """Pieces of lines are stored past the caches only where the rule says that it does not matter."""
    assert B.lib().bnn_testing_conv_word_nontemporal(N, C, H, W, D, 3, 3, 1, 1, 1, 1) == want


def test_conv_word_offsets_fit_32_bits():
    """64 columns span at most 63 / (OH OW) + 2 images; their bytes are a 32-bit offset in the kernel."""
    f = lambda N, H, s: B.lib().bnn_testing_conv_word(N, 1, H, H, 64, 3, 3, s, s, 1, 1, 0, 1, 256)
    assert f(70, 2100, 2100) > 0 and f(70, 2900, 2900) == 0  # one output pixel an image: 65 images
    assert f(2, 16300, 5) > 0 and f(2, 16400, 5) == 0        # two images and a bit


@pytest.mark.parametrize("N,H,W,D,want", [
    (32, 32, 32, 128, 0), (33, 32, 32, 128, 2), (128, 32, 32, 32, 0), (129, 32, 32, 32, 2),  # q = 8, 8.25; 8, 8.06
    (108, 32, 32, 128, 2), (109, 32, 32, 128, 3),                                               # 27, 27.25: one round of eight waves
    (128, 32, 32, 128, 3), (129, 32, 32, 128, 4), (257, 32, 32, 128, 3), (640, 32, 32, 128, 3),  # one, two, three, five
    (641, 32, 32, 128, 4), (769, 32, 32, 128, 4), (64, 32, 32, 250, 3), (128, 32, 32, 200, 4)])  # six, seven; 256 channels
def test_first_sign_forms(N, H, W, D, want):
    """Both sides of every line between the forms of the first layer's signs, on 256 compute units."""
    assert B.lib().bnn_testing_first_sign(N, H, W, D, 1, 1, 1, 1, 256) == want


def test_first_sign_forms_of_very_large_images():
    """64 pixels that span 4 GiB are left to the chains: four channel groups a workgroup as soon as there is work for them, so that no
    channel count is refused that a launch has room for."""
    form = lambda N, H, D, s: B.lib().bnn_testing_first_sign(N, H, H, D, s, s, 0, 0, 256)
    assert form(60, 2300, 98336, 2300) >= 2 and form(60, 2400, 98304, 2400) == 0 and form(60, 2400, 98336, 2400) == 0
    assert form(60, 2400, 196608, 2400) == 0 and form(60, 2400, 196609, 2400) == 1 and form(1, 2400, 2200000, 2400) == 1
    assert form(1, 13300, 64, 1) >= 2 and form(1, 13400, 64, 1) == 1


def image(N, C, H, W, D, kH, kW, sH, sW, pH, pW, shape=-1, pixel=0):
    """bnn_testing_conv_image on 256 compute units -> (shape, first row, last row, rows with room)."""
    out = (ctypes.c_int64 * 3)()
    r = B.lib().bnn_testing_conv_image(N, C, H, W, D, kH, kW, sH, sW, pH, pW, 256, shape, pixel, out)
    return (r, *out)


def test_image_tiles_have_room_for_the_rows_they_read():
    """Every tile of random small convolutions: the rows between its first and its last tap (outside the image: the nearest
    row) are among those that it encodes, these fit the launch's LDS, and the tiles together encode the whole image."""
    rng = random.Random(7)
    tiles = 0
    while tiles < 3000:
        N, H, W = rng.choice([1, 2, 3, 7]), rng.randint(1, 14), rng.randint(1, 14)
        kH, kW, sH, sW, pH, pW = (rng.randint(a, b) for a, b in ((1, 6), (1, 6), (1, 7), (1, 7), (0, 7), (0, 7)))
        if H + 2 * pH < kH or W + 2 * pW < kW:
            continue
        OH, OW = (H + 2 * pH - kH) // sH + 1, (W + 2 * pW - kW) // sW + 1
        done = -1
        for n0 in range(0, N * OH * OW, 32):
            shape, r0, r1, most = image(N, 64, H, W, 40, kH, kW, sH, sW, pH, pW, shape=1, pixel=n0)
            assert shape == 1 and 0 <= r0 <= r1 < N * H and r1 - r0 + 1 <= most and r0 <= done + 1
            done, tiles = max(done, r1), tiles + 1
            for q in range(n0, min(N * OH * OW, n0 + 32)):
                n, oh = q // (OH * OW), q // OW % OH
                first, last = (n * H + min(max(oh * sH - pH + k, 0), H - 1) for k in (0, kH - 1))
                assert r0 <= first and last <= r1
        assert done == N * H - 1


@pytest.mark.parametrize("case,want", [
    ((16, 128, 16, 16, 64, 3, 1), 1), ((17, 128, 16, 16, 64, 3, 1), 0),   # t = 1, 1.06
    ((32, 128, 16, 16, 64, 3, 1), 0), ((33, 128, 16, 16, 64, 3, 1), -1),  # 2, 2.06: b = 32
    ((48, 96, 16, 16, 64, 3, 1), 0), ((48, 97, 16, 16, 64, 3, 1), -1),    # t = 3: b = 24, 24.25
    ((49, 96, 16, 16, 64, 3, 1), -1),                                     # t = 3.06
    ((1, 213, 32, 64, 32, 3, 1), 1), ((1, 214, 32, 64, 32, 3, 1), -1),    # t up to 1: b = 159.75, 160.5
    ((32, 256, 16, 20, 32, 3, 1), -1), ((32, 256, 16, 16, 33, 3, 1), 0),  # above: b = 80 (of five rows, 100), 64
    ((1, 8129, 1, 1, 8, 3, 1), -1)])                                      # more channels than the encode takes
def test_image_rule_lines(case, want):
    """Both sides of every line of the rule for convolutions in one launch, on 256 compute units."""
    N, C, H, W, D, k, s = case
    assert image(N, C, H, W, D, k, k, s, s, k // 2, k // 2)[0] == want
