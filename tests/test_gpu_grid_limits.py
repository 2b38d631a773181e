"""Calls whose launches have more workgroups than one grid dimension takes
(2^32 threads): nearly all of their sequences have nothing to do, a few at the
ends and in the middle are compared with the same sequences in a small call."""
import numpy as np
import pytest

from harness import host

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


@pytest.mark.parametrize("recent", [4160, 64])
def test_step_smoothing_tiles(E, recent):
    """A step of 65,535 sequences with chunks of 4160 tokens: 4.3 million
    smoothing tiles, beside the resolve stage (the chunk inside the recency
    window) or ahead of the selection."""
    import torch
    C, D, K, page, H, d = 4160, 8, 4200, 16, 1, 64
    assert (C + 63) // 64 * B > DIM
    live = [0, B // 2, B - 1]
    lengths = [C + 17, C + 40, C]
    print(f"step smoothing tiles {(C + 63) // 64 * B} recent {recent}", flush=True)
    torch.manual_seed(5)
    per, ld_s = (K + page - 1) // page, K + 24
    tables = torch.randperm(len(live) * per, device="cuda").to(torch.int32).view(-1, per)
    src = torch.randint(-2 ** 15, 2 ** 15, (1, 2, len(live) * per, page, H, d), dtype=torch.int16,
                        device="cuda")
    rows = torch.randn(len(live), C, D, device="cuda").to(torch.bfloat16)
    old = torch.randn(len(live), ld_s, device="cuda")

    def step(batch, at):
        cfg = E.default_cfg(batch=batch, hidden=D, n_layers=1, n_kv_heads=H, head_dim=d,
                            page_size=page, n_band_a=1, n_band_b=0, budget=K, recent=recent)
        assert E.check_cfg(cfg) == 0
        hid = torch.zeros(batch, C, D, dtype=torch.bfloat16, device="cuda")
        pt = torch.zeros(batch, per, dtype=torch.int32, device="cuda")
        n_cached = torch.zeros(batch, dtype=torch.int32, device="cuda")
        scores = torch.zeros(batch, ld_s, device="cuda")
        hid[at], pt[at], scores[at] = rows, tables, old
        n_cached[at] = torch.tensor(lengths, dtype=torch.int32, device="cuda")
        dst = torch.zeros_like(src)
        new_scores = torch.full((batch, ld_s), -9.0, device="cuda")
        keep = torch.full((batch, K), -5, dtype=torch.int32, device="cuda")
        n_keep = torch.zeros(batch, dtype=torch.int32, device="cuda")
        status = torch.zeros(batch, dtype=torch.int32, device="cuda")
        st = [torch.zeros(E.state_bytes(cfg), dtype=torch.uint8, device="cuda") for _ in range(2)]
        n = E.workspace_bytes(cfg, C)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        io = E.make_step_io(C, [hid], D, C * D, n_cached, torch.zeros_like(n_cached),
                            E.pool_of(src), pt, per, E.pool_of(dst), pt, per, scores, ld_s, st[0],
                            st[1], keep, n_keep, status, ws, n, dst_scores=new_scores)
        E.epikv_evict_step(cfg, io)
        torch.cuda.synchronize()
        sec = E.state_sections(cfg, st[1])
        assert int((n_keep >= 0).sum()) == len(live)
        return [host(t) for t in (dst, scores[at], new_scores[at], keep[at], n_keep[at],
                                  status[at], sec["n_tok"][at], sec["ring"][at])]

    for got, ref in zip(step(B, live), step(len(live), list(range(len(live))))):
        assert np.array_equal(got, ref)
