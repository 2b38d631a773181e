"""The eviction step's merged launches (select + score + page order, then
smoothing + resolve; or smoothing + reduction + scratch clearing, then select
+ page order) against its stages called one by one, bit for bit."""
import numpy as np
import pytest

import synth
from harness import dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_26472_amd import epikv
    epikv.lib()
    return epikv


# lengths: longer than K, at K, shorter, exactly the chunk, too short for it
RAGGED = [700, 256, 200, None, 1]


@pytest.mark.parametrize("smoothing", ["z", "mean", "raw", "ema"])
@pytest.mark.parametrize("C,page,order,bad", [
    (64, 16, "scattered", False), (1, 3, "scattered", True), (33, 16, "rising", True),
    (64, 1, "scattered", False)])
def test_step_equals_its_stages(E, smoothing, C, page, order, bad):
    """Sequences of every kind (longer than the budget, at it, shorter, as
    long as the chunk, shorter than it: refused), one whose prefix leaves no
    room (refused), and, with `bad`, tables that hold ids out of range for a
    page in the middle and for the page of the chunk's tail."""
    _compare(E, smoothing, C, page, order, bad, RAGGED, 256)


@pytest.mark.parametrize("smoothing", ["z", "ema"])
def test_many_sequences(E, smoothing):
    """Two smoothing tiles for each of 140 sequences (EMA: both with one
    workgroup), several score units per workgroup, budgets of 512."""
    _compare(E, smoothing, 100, 16, "scattered", False, [600, 512, 130, 513] * 35, 512)


@pytest.mark.parametrize("signal,smoothing,C,window,H", [
    ("lagkv", "mean", 64, 64, 8), ("lagkv", "mean", 65, 256, 1), ("lagkv", "z", 130, 1, 2),
    ("kv_key", "mean", 63, 64, 8), ("kv_val", "raw", 1, 2, 1), ("lagkv_key", "mean", 100, 64, 8),
    ("lagkv", "ema", 130, 64, 8)])
def test_kv_step_equals_its_stages(E, signal, smoothing, C, window, H):
    """KV-vector signals: the smoothing workgroups add up the planes of their
    tile and the window before it; rows split between workgroups (ranges
    combined in the same launch) and not; rows of scores long enough that the
    selection is split (its scratch cleared in that launch)."""
    _compare(E, smoothing, C, 16, "scattered", False, [1500, 700, C, 1300], 600, signal, window, H)


@pytest.mark.parametrize("C,D,lengths", [
    (200, 64, [1500, 700, 200, 1300]),       # longer than the recency window
    (64, 4104, [1500, 700, 64, 1300]),       # rows wider than the merged scorer takes
    (200, 64, [700, 650, 601]),              # the selection is not split
    (0, 64, [1500, 700, 10, 1300])])         # nothing to score
def test_unfused_step_equals_its_stages(E, C, D, lengths):
    _compare(E, "z", C, 16, "scattered", False, lengths, 600, D=D)


@pytest.mark.parametrize("signal,C,lengths,K", [
    ("hs", 0, [1500, 700, 10, 1300], 600),          # nothing to score
    ("hs", 120, [1500, 700, 120, 1300], 100),       # a chunk longer than the budget
    ("lagkv", 120, [300, 250, 120, 299], 100)])     # the same; the selection is not split
def test_counts_updated_in_place(E, signal, C, lengths, K):
    """One buffer as n_cached and n_keep: the page order, which needs the
    counts, must not run beside the selection that rewrites them."""
    _compare(E, "mean", C, 16, "scattered", False, lengths, K, signal, counts_in_place=True)


def _compare(E, smoothing, C, page, order, bad, lengths, K, signal="hs", window=64, H=1, D=64,
             counts_in_place=False):
    import torch
    print(f"merged step {signal} {smoothing} C={C} page={page} {order} bad={bad}", flush=True)
    g = synth.rng(2100 + C + page)
    lengths = np.array([C if n is None else n for n in lengths] + [K + 50])
    B, L, d, na, nb = lengths.size, 1 if signal == "hs" else 3, 64, 3, 2
    kv = signal != "hs"
    ld_s = int(lengths.max())
    cfg = E.default_cfg(batch=B, hidden=D, n_layers=L, n_kv_heads=H, head_dim=d, page_size=page,
                        n_band_a=na, n_band_b=nb, budget=K, window=window,
                        signal=getattr(E, "SIGNAL_" + signal.upper()),
                        smoothing=getattr(E, "SMOOTH_" + smoothing.upper()))
    src_pt, n_src = synth.page_tables(lengths, page, g)
    if order == "rising":
        dst_pt, n_dst = synth.contiguous_page_tables(np.full(B, K), page, first=1)
    else:
        dst_pt, n_dst = synth.page_tables(np.full(B, K), page, g)
    if bad:
        src_pt[0, (lengths[0] - 1) // page] = n_src          # the chunk's last page
        dst_pt[1, 3] = -1
        dst_pt[2, (lengths[2] - 1) // page] = n_dst + 5      # the last kept row's page
    shape = (L, 2, n_src, page, H * d)
    pool = dev(synth.kv_rows(g, shape) if kv else synth.random_bits16(g, shape))
    hid = dev(synth.f32_to_bf16_bits(
        g.standard_normal((na + nb, B, max(C, 1), D)).astype(np.float32)))
    sc = g.standard_normal((B, ld_s)).astype(np.float32)
    st_in = torch.zeros(E.state_bytes(cfg), dtype=torch.uint8, device="cuda")
    sec = E.state_sections(cfg, st_in)
    n_tok = np.maximum(lengths - C, 0).astype(np.int32)
    sec["n_tok"].copy_(dev(n_tok))
    sec["ring"].copy_(dev((20 + g.standard_normal(tuple(sec["ring"].shape))).astype(np.float32)))
    sec["ema"].copy_(dev((20 + g.standard_normal(tuple(sec["ema"].shape))).astype(np.float32)))
    if "range" in sec:
        sec["range"].copy_(torch.randn(sec["range"].shape, device="cuda"))
        sec["range"][1] += 6.0
        sec["n_tok"][1] = 0                                  # a fresh stream among the others
    n_cached = dev(lengths.astype(np.int32))
    prefix = np.zeros(B, np.int32)
    prefix[-1] = K
    n_prefix = dev(prefix)
    pos = dev(np.tile(np.arange(ld_s, dtype=np.int32), (B, 1)))
    hidden = [hid[l] for l in range(na + nb)]

    def outputs():
        return dict(dst=torch.full((L, 2, n_dst, page, H * d), 77, dtype=torch.int16,
                                   device="cuda"),
                    scores=dev(sc), dsc=torch.full((B, ld_s), -9.0, device="cuda"),
                    dpos=torch.full((B, ld_s), -9, dtype=torch.int32, device="cuda"),
                    keep=torch.full((B, K), -5, dtype=torch.int32, device="cuda"),
                    nk=torch.zeros(B, dtype=torch.int32, device="cuda"),
                    status=torch.zeros(B, dtype=torch.int32, device="cuda"),
                    st_out=torch.zeros_like(st_in))

    src = E.pool_of(pool.view(L, 2, n_src, page, H, d))
    spt, dpt = dev(src_pt), dev(dst_pt)
    a, s = outputs(), outputs()
    n = E.workspace_bytes(cfg, C)
    ws = torch.full((n,), 0x7F, dtype=torch.uint8, device="cuda")
    if counts_in_place:
        a["nk"].copy_(n_cached)
    io = E.make_step_io(C, hidden, D, C * D, a["nk"] if counts_in_place else n_cached, n_prefix,
                        src, spt, src_pt.shape[1],
                        E.pool_of(a["dst"].view(L, 2, n_dst, page, H, d)), dpt, dst_pt.shape[1],
                        a["scores"], ld_s, st_in, a["st_out"], a["keep"], a["nk"], a["status"],
                        ws, n, dst_scores=a["dsc"], src_pos=pos, dst_pos=a["dpos"])
    E.epikv_evict_step(cfg, io)
    sig = torch.zeros((1 if kv else na + nb, B, max(C, 1)), device="cuda")
    sws = torch.full((n,), 0x7F, dtype=torch.uint8, device="cuda")
    if kv:
        E.epikv_score(cfg, C, pool=src, page_table=spt, ld_pt=src_pt.shape[1], n_cached=n_cached,
                      state_in=st_in, state_out=s["st_out"], sig=sig, workspace=sws,
                      workspace_bytes_=n)
    elif C:
        E.epikv_score(cfg, C, hidden, D, C * D, state_in=st_in, state_out=s["st_out"], sig=sig)
    if C:
        E.epikv_zscore(cfg, C, sig, n_cached, st_in, s["st_out"], s["scores"], ld_s)
    E.epikv_select(cfg, s["scores"], ld_s, n_cached, n_prefix, s["keep"], s["nk"], s["status"])
    # (the step refuses a sequence shorter than its chunk; select alone does not)
    short = torch.from_numpy(lengths < C).cuda()
    s["nk"][short] = -1
    s["status"][short] = E.SEQ_RANGE
    s["keep"][short] = -5
    m = E.compact_workspace_bytes(cfg)
    cws = torch.full((m,), 0x7F, dtype=torch.uint8, device="cuda")
    E.epikv_compact(cfg, src, spt, src_pt.shape[1],
                    E.pool_of(s["dst"].view(L, 2, n_dst, page, H, d)), dpt, dst_pt.shape[1],
                    s["keep"], s["nk"], s["scores"], s["dsc"], pos, s["dpos"], ld_s, s["status"],
                    cws, m)
    torch.cuda.synchronize()
    for k in a:
        assert np.array_equal(host(a[k]), host(s[k])), k
    status = host(a["status"])
    assert status[-1] == E.SEQ_BUDGET
    if bad:
        assert list(status[:3]) == [E.SEQ_RANGE] * 3
