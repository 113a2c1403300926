"""Default tiles of the fused z pass on both sides of the rules that depend on a
call's size. The tile follows from the bytes of the kernel spectrum, whose rows
are padded to whole tiles (no device work)."""
import pytest

from paper_1804_01830_amd import binding as B

E_Z, TILT, OBLIQUE = (0.0, 0.0, 1.0), (0.6, 0.0, 0.8), (0.0, 0.6, 0.8)


def tile(n, lines, precision, batch, periodic=False):
    d = B.make_desc(n, (1.0, 1.0, 2.0), 1.0, 0.3, (E_Z, TILT, OBLIQUE)[:lines], precision=precision, batch=batch,
                    periodic=(periodic, periodic))
    px, py, pz = B.padded_lengths(n, (periodic, periodic))
    rows = (py // 2 + 1 if lines < 3 else py) * (pz // 2 + 1 if lines == 1 else pz)
    columns = (B.footprint(d)[0] - 2048 * 2 * precision // 8) / (rows * 18 * lines * precision // 8)
    assert columns == int(columns)
    fit = [t for t in (1, 2, 4, 8, 16, 32, 64) if -(-(px // 2 + 1) // t) * t == columns]
    assert len(fit) == 1
    return fit[0]


@pytest.mark.parametrize("n,periodic,expected", [((128, 128, 32), False, 4), ((256, 64, 32), False, 4),
                                                 ((64, 64, 32), False, 4), ((128, 256, 32), False, 8),
                                                 ((256, 256, 32), True, 8), ((400, 60, 30), False, 8),
                                                 ((256, 256, 32), False, 8)])
def test_two_realisations_of_three_channels_at_length_64(n, periodic, expected):
    assert tile(n, 1, 32, 2, periodic) == expected


@pytest.mark.parametrize("n,batch,periodic,expected", [((128, 128, 32), 6, False, 16), ((128, 128, 30), 8, False, 16),
                                                       ((128, 128, 32), 5, False, 8), ((128, 128, 28), 8, False, 8),
                                                       ((100, 75, 20), 8, False, 8), ((64, 64, 32), 8, False, 8),
                                                       ((128, 128, 32), 8, True, 8)])
def test_six_to_eleven_realisations_of_three_channels_at_length_64(n, batch, periodic, expected):
    assert tile(n, 1, 32, batch, periodic) == expected


@pytest.mark.parametrize("n,batch,expected", [((128, 128, 16), 12, 16), ((256, 256, 16), 6, 16), ((256, 256, 16), 5, 4),
                                              ((64, 64, 16), 12, 4), ((128, 128, 32), 12, 8), ((128, 128, 32), 11, 4),
                                              ((100, 75, 20), 12, 4)])
def test_double_precision_batches_of_nine_channels(n, batch, expected):
    assert tile(n, 3, 64, batch) == expected
