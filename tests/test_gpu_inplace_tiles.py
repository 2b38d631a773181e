"""The in-place move's tiles against the oracle's in-place rebuild: moved rows
just short of, at and past one, two and four tiles of every slice width that
the size rule takes (a slice's columns dividing the workgroup's threads or
leaving some over, a row in one slice or in several)."""
import pytest

from test_gpu_inplace import E, _run  # noqa: F401

pytestmark = pytest.mark.gpu

# 256 walks and more: one slice per row; 8 walks: the narrowest slices
MANY = dict(L=16, lengths=[90, 140, 200, 300, 333, 131, 400, 260])
FEW = dict(L=2, lengths=[700, 333])


@pytest.mark.parametrize("H,d,K,shape", [
    (8, 128, 63, MANY), (8, 128, 64, MANY), (8, 128, 65, MANY), (8, 128, 129, MANY),
    (8, 128, 255, FEW), (8, 128, 257, FEW), (8, 128, 600, FEW),
    (6, 128, 81, MANY), (5, 128, 97, MANY), (3, 128, 200, MANY), (7, 128, 300, FEW),
    (6, 128, 300, FEW), (3, 128, 640, FEW), (1, 128, 513, FEW), (1, 64, 650, FEW),
    (1, 64, 200, MANY), (16, 128, 33, MANY), (8, 256, 150, FEW)],
    ids=lambda v: str(v) if isinstance(v, int) else ("many" if v is MANY else "few"))
@pytest.mark.parametrize("page", [16, 5])
def test_tiles(E, H, d, K, shape, page):  # noqa: F811
    print(f"in-place tiles H {H} d {d} K {K} page {page} L {shape['L']}", flush=True)
    _run(E, f"tiles{H}.{d}.{K}.{page}", K=K, H=H, d=d, page=page, **shape)
