"""The bytes that the server counts for a shape's spectrum are those of the plan
that holds it, whose tiles are those of one realisation (no device work)."""
import pytest

from paper_1804_01830_amd import binding as B
from paper_1804_01830_amd.serving import GpuExecutor, ShapeKey

LINES = ((0.0, 0.0, 1.0), (0.6, 0.0, 0.8), (0.0, 0.6, 0.8))


@pytest.mark.parametrize("n,lines,precision", [((16, 9, 32), 3, 32), ((16, 9, 64), 1, 32), ((20, 9, 3), 1, 64),
                                               ((9, 9, 16), 2, 64)])
@pytest.mark.parametrize("batch", [2, 4, 16])
def test_footprint_of_a_shape(n, lines, precision, batch):
    ex = GpuExecutor.__new__(GpuExecutor)
    ex.B = B
    key = ShapeKey(n=n, d=(1.0, 1.0, 2.0), mu=1.0, nu=0.3, lines=LINES[:lines], precision=precision)
    cells, elem = key.cells, precision // 8
    one, many = (B.footprint(B.make_desc(n, key.d, key.mu, key.nu, key.lines, precision=precision, batch=b))
                 for b in (1, batch))
    shape, slot = ex.footprint(key, batch)
    assert shape == one[0] + one[1]
    assert slot == many[1] + batch * (key.channels + 6) * cells * elem
