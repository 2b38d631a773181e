"""The in-place move's tiles against the oracle's in-place rebuild: slices of
every kind that the size rule takes (a slice's columns dividing the workgroup's
threads or leaving some over, a row in one slice or in several), and numbers of
moved rows just short of, at and past one, two, four and nine tiles, with and
without page remapping."""
import numpy as np
import pytest

import oracle as O
import synth
from harness import dev, host, remap_expected
from test_gpu_inplace import E, _expected, _run  # noqa: F401

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


def _slice_cols(planes, row_vec):
    """Columns of the slices that the library cuts a row into."""
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    fits = [s for s in range(1, row_vec + 1) if row_vec % s == 0 and row_vec // s % 8 == 0]

    def fill(s):
        return planes * s / (-(-planes * s // cus) * cus)

    for s in fits:
        if planes * s <= cus and fill(s) >= 0.6:
            return row_vec // s
    cols = 128 if row_vec > 128 else 32
    narrow = planes > cus and (row_vec > 128 or planes < 4 * cus)
    if narrow and row_vec % cols == 0 and fill(row_vec // cols) >= 0.9:
        return cols
    best = 0
    for s in fits:
        if best == 0 or fill(s) > fill(best):
            best = s
        if fill(best) >= 0.9:
            break
    return row_vec // best


def _call(E, H, d, L, page, keeps, lengths, remap):  # noqa: F811
    import torch
    g = synth.rng(77 * H + d + L)
    B, K = len(keeps), max(k.size for k in keeps)
    cfg = E.default_cfg(batch=B, n_layers=L, n_kv_heads=H, head_dim=d, page_size=page, budget=K)
    pt, used = synth.page_tables(np.asarray(lengths), page, g)
    pool = synth.random_bits16(g, (L, 2, used + 3, page, H * d))
    keep_idx = np.full((B, K), -3, np.int32)
    for b, k in enumerate(keeps):
        keep_idx[b, :k.size] = k
    n_keep = np.array([k.size for k in keeps], np.int32)
    if remap:
        want, want_pt = remap_expected(pool, pt, keeps, page)
    else:
        want, want_pt = _expected(pool, pt, keeps, lengths), pt
    pool_d, pt_d = dev(pool), dev(pt)
    status = torch.zeros(B, dtype=torch.int32, device="cuda")
    n = E.compact_workspace_bytes(cfg)
    ws = torch.full((n,), 0x7F, dtype=torch.uint8, device="cuda")
    call = E.epikv_compact_remap if remap else E.epikv_compact_inplace
    call(cfg, E.pool_of(pool_d.view(L, 2, used + 3, page, H, d)), pt_d, pt.shape[1],
         dev(keep_idx), dev(n_keep), seq_status=status, workspace=ws, workspace_bytes_=n)
    torch.cuda.synchronize()
    assert int(status.count_nonzero()) == 0
    assert np.array_equal(host(pt_d), want_pt)
    assert np.array_equal(host(pool_d), want)


@pytest.mark.parametrize("H,d,L,page,cols", [
    (8, 128, 16, 16, 128), (5, 128, 16, 16, 80), (7, 128, 16, 5, 112), (3, 64, 16, 16, 24),
    (1, 64, 16, 16, 8), (8, 256, 16, 5, 256),              # whole rows
    (8, 128, 4, 5, 32), (5, 128, 4, 16, 16), (3, 128, 4, 5, 16), (11, 64, 1, 16, 8),
    (8, 128, 24, 16, 32), (8, 256, 40, 16, 128)])          # cut; more than one round of walks
def test_moved_rows_around_tiles(E, H, d, L, page, cols):  # noqa: F811
    """Position 0 is dropped, so every kept row moves."""
    assert _slice_cols(2 * L * 6, H * d // 8) == cols
    T = 1024 // cols * 8
    moved = [T - 1, T, T + 1, 2 * T, 4 * T + 1, 9 * T]
    print(f"in-place tiles H {H} d {d} L {L} page {page}: {cols} columns, T {T}", flush=True)
    g = synth.rng(T + cols)
    lengths = [m + 1 + int(g.integers(0, m // 4 + 2)) for m in moved]
    keeps = [np.sort(g.choice(n - 1, m, replace=False)) + 1 for m, n in zip(moved, lengths)]
    _call(E, H, d, L, page, keeps, lengths, remap=False)


@pytest.mark.parametrize("H,d,L", [(8, 128, 32), (5, 128, 32)])
def test_remapped_tiles(E, H, d, L):  # noqa: F811
    """Released pages among the destinations of many tiles: in every ten pages
    sixteen rows of the first six are dropped, so that the rows of those pages
    move and the last four change places."""
    page, B = 16, 3
    T = 1024 // _slice_cols(2 * L * B, H * d // 8) * 8
    g = synth.rng(31 * H)
    keeps, lengths = [], []
    for b in range(B):
        mask = np.ones(160 * (9 + b) + 7 * b, bool)
        for a in range(0, mask.size - 160, 160):
            mask[a + g.choice(96, 16, replace=False)] = False
        keeps.append(np.nonzero(mask)[0])
        lengths.append(mask.size)
    tiles = []
    for k in keeps:
        pairs = len(O.remap_pairs(k, page))
        tiles.append((k.size - O.first_hole(k) - pairs * page) / T)
        assert pairs >= 24
    print(f"remapped tiles H {H} d {d}: T {T}, tiles {tiles}", flush=True)
    assert min(tiles) >= 6
    _call(E, H, d, L, page, keeps, lengths, remap=True)
