"""Calls whose launches have more workgroups than one grid dimension takes
(2^32 threads): nearly all of their sequences have nothing to do, a few at the
ends and in the middle are compared with the same sequences in a small call."""
import pytest

pytestmark = pytest.mark.gpu

B = 65535
DIM = 1 << 22          # workgroups of 1024 threads that come to 2^32 threads


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_26472_amd import epikv
    epikv.lib()
    return epikv


@pytest.mark.parametrize("remap", [False, True])
def test_in_place_walks(E, remap):
    """33 layers of 65,535 sequences: 4.3 million walks, each a workgroup."""
    import torch
    L, K, page = 33, 2, 2
    assert 2 * L * B > DIM
    live = [0, 1, B // 2, B - 2, B - 1]
    print(f"in-place walks {2 * L * B} remap {remap}", flush=True)
    cfg = E.default_cfg(batch=B, n_layers=L, n_kv_heads=1, head_dim=64, page_size=page, budget=K)
    pool = torch.randint(-2 ** 15, 2 ** 15, (L, 2, len(live), page, 1, 64), dtype=torch.int16,
                         device="cuda")
    want = pool.clone()
    want[:, :, :, 0] = pool[:, :, :, 1]                  # slot 0 receives row 1
    pt = torch.zeros(B, 1, dtype=torch.int32, device="cuda")
    keep = torch.zeros(B, K, dtype=torch.int32, device="cuda")
    n_keep = torch.zeros(B, dtype=torch.int32, device="cuda")
    for i, b in enumerate(live):
        pt[b, 0], keep[b, 0], n_keep[b] = i, 1, 1
    table = pt.clone()
    scores = torch.arange(2 * B, dtype=torch.float32, device="cuda").view(B, 2)
    moved = scores.clone()
    moved[live, 0] = scores[live, 1]
    status = torch.zeros(B, dtype=torch.int32, device="cuda")
    n = E.compact_workspace_bytes(cfg)
    ws = torch.full((n,), 0x7F, dtype=torch.uint8, device="cuda")
    call = E.epikv_compact_remap if remap else E.epikv_compact_inplace
    call(cfg, E.pool_of(pool), pt, 1, keep, n_keep, scores=scores, ld_s=2, seq_status=status,
         workspace=ws, workspace_bytes_=n)
    torch.cuda.synchronize()
    assert torch.equal(pool, want)
    assert torch.equal(scores, moved)
    assert torch.equal(pt, table) and int(status.count_nonzero()) == 0
