"""The out-of-place gather over row lengths: whole KiB, the narrow rows that
share a workgroup (128, 256, 512 bytes) and every other length."""
import numpy as np
import pytest

import oracle as O
import synth
from harness import dev, gather_logical, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_26472_amd import epikv
    epikv.lib()
    return epikv


@pytest.mark.parametrize("page,K", [(16, 64), (3, 50), (1, 33)])
@pytest.mark.parametrize("H,d", [(1, 64), (1, 128), (2, 64), (4, 64), (3, 64), (5, 64),
                                 (3, 128), (6, 128), (7, 256), (8, 128), (8, 256)])
def test_compact_row_lengths(E, H, d, page, K):
    """Rows of 128 to 4096 bytes, B * slots not a multiple of the rows per
    workgroup among them (pages of 3 tokens and of 1), a sequence shorter
    than the budget and one that is refused: the oracle's bytes, and nothing
    past them."""
    import torch
    print(f"compact rows H={H} d={d} page={page} K={K}", flush=True)
    g = synth.rng(1700 + 10 * H + d + page)
    L = 2
    Ns = np.array([K + 37, K - 20, K + 5])
    keeps = [np.sort(g.choice(n, K, replace=False)) if n > K else np.arange(n) for n in Ns]
    keeps[2] = None                                    # refused: untouched
    B = len(Ns)
    src_pt, n_src = synth.page_tables(Ns, page, g)
    dpp = (K + page - 1) // page
    dst_pt, n_dst = synth.page_tables(np.full(B, K), page, g, n_pages_total=B * dpp + 3)
    pool = synth.random_bits16(g, (L, 2, n_src, page, H * d))
    keep = np.full((B, K), -1, dtype=np.int32)
    n_keep = np.full(B, -1, dtype=np.int32)
    for b, k in enumerate(keeps):
        if k is not None:
            keep[b, :k.size] = k
            n_keep[b] = k.size
    sent = 0x5A5A
    dst_t = torch.full((L, 2, n_dst, page, H * d), sent, dtype=torch.int16, device="cuda")
    src_t = dev(pool)
    cfg = E.default_cfg(batch=B, n_layers=L, n_kv_heads=H, head_dim=d, budget=K, page_size=page)
    n = E.compact_workspace_bytes(cfg)
    ws = torch.full((n,), 0x7F, dtype=torch.uint8, device="cuda")
    status = torch.zeros(B, dtype=torch.int32, device="cuda")
    E.epikv_compact(cfg, E.pool_of(src_t.view(L, 2, n_src, page, H, d)), dev(src_pt),
                    src_pt.shape[1], E.pool_of(dst_t.view(L, 2, n_dst, page, H, d)), dev(dst_pt),
                    dst_pt.shape[1], dev(keep), dev(n_keep), seq_status=status, workspace=ws,
                    workspace_bytes_=n)
    torch.cuda.synchronize()
    assert np.all(host(status) == 0)
    got = host(dst_t)
    exp = np.full_like(got, sent)
    for b, k in enumerate(keeps):
        if k is None:
            continue
        rows = gather_logical(pool, src_pt[b], int(Ns[b]))
        j = np.arange(k.size)
        exp[:, :, dst_pt[b, j // page], j % page] = \
            O.compact_rows(rows.transpose(2, 0, 1, 3), k).transpose(1, 2, 0, 3)
    assert np.array_equal(got, exp)
