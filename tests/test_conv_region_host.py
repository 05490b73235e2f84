"""The input region that the matrix-core convolution keeps in LDS, modelled on the CPU.

The host sizes the region by a bound over all tiles (halo_region in gemm_fp4.hip) and the kernel derives each tile's
rows and every column's offset from its first and last pixel.  The model states both and checks, for random
geometries, that no tile needs more rows than the bound and that every tap a column reads lies inside the region on
the row of its own image."""
import ctypes
import random

import pytest

from paper_1911_04477_amd import binding as B


def cells_touched(length, cell):
    if length % cell == 0:
        return length // cell
    if cell % length == 0:
        return 1
    return (length - 2) // cell + 2


def check_geometry(N, H, W, kH, kW, sH, sW, pH, pW, pool, bn):
    OH, OW = (H + 2 * pH - kH) // sH + 1, (W + 2 * pW - kW) // sW + 1
    us = 2 if pool else 1  # output rows per unit
    Wp, units, ustep, uspan = (OW - 1) * sW + kW, OH // us, us * sH, (us - 1) * sH + kH
    full = (units - 1) * ustep + uspan
    ucols = us * us * (OW // us)
    nu = cells_touched(bn, ucols)
    ni = min(nu, cells_touched(bn, ucols * units))
    bound = max((nu - 1) * ustep + uspan, (nu - ni) * ustep + ni * uspan)

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
            assert (r + kH - 1) * Wp + ow * sW + kW - 1 < rows * Wp


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
        check_geometry(rng.randint(1, 9), H, W, kH, kW, sH, sW, pH, pW, pool, rng.choice([64, 128, 256]))
        seen += 1


def test_rows_beyond_the_pitch_are_gathered():
    """Input rows of 4 GiB and more, of which one output column's taps read three pixels: the region would be small,
    but the pitch that the copy into it steps by is a 32-bit number of bytes."""
    out = (ctypes.c_int64 * 4)()
    region = B.lib().bnn_testing_conv_region
    for H, W, C, taken in ((3, 1 << 29, 1, 0), (3, 1 << 29, 5, 0), (2, (1 << 30) - 1, 4, 0), (3, (1 << 29) - 1, 1, 1),
                           (2, (1 << 29) - 1, 8, 1)):
        assert region(1, C, H, W, H, 3, 1, 1 << 30, 0, 0, 0, 256, out) == taken, (H, W, C)
