"""A Lag-KV stream's first chunk, large enough that its range is found by a
launch of its own (128 MiB of rows, split between workgroups)."""
import numpy as np
import pytest

import synth
import test_gpu_kernels as K
from harness import dev, host

pytestmark = pytest.mark.gpu
E = K.E


@pytest.mark.parametrize("signal,H,d,L,C,B,page,nan", [
    ("lagkv", 8, 128, 32, 1024, 1, 16, False),      # two row segments, whole shares
    ("lagkv", 8, 128, 32, 1031, 1, 16, True),       # a NaN key; a short last share
    ("lagkv", 2, 128, 64, 1040, 2, 3, False),        # narrow rows, two shares
    ("lagkv_key", 16, 128, 33, 1030, 1, 64, False),  # one tensor, four row segments
])
def test_large_first_chunk_matches_oracle(E, signal, H, d, L, C, B, page, nan):
    planes = (2 if signal == "lagkv" else 1) * L
    assert planes * B * C * H * d * 2 >= 128 << 20
    K._run_kv(E, signal, C, nan=nan, H=H, d=d, L=L, B=B, page=page)


def test_fresh_and_carried_sequences_in_one_call(E):
    """One fresh and one carried sequence share the call: each gets the
    bits that it gets alone, where the call is below the size and a first
    chunk is one workgroup's."""
    import torch
    g = synth.rng(1812)
    B, C, L, H, d, page = 2, 1030, 16, 8, 128, 16
    assert 2 * L * B * C * H * d * 2 >= 128 << 20 > 2 * L * C * H * d * 2
    Ns = np.array([C, C + 21])
    pt, n_pages = synth.page_tables(Ns, page, g)
    pool = dev(synth.kv_rows(g, (L, 2, n_pages, page, H * d))).view(L, 2, n_pages, page, H, d)

    def cfg_of(n):
        return E.default_cfg(batch=n, n_layers=L, n_kv_heads=H, head_dim=d, page_size=page,
                             signal=E.SIGNAL_LAGKV, smoothing=E.SMOOTH_MEAN)

    rng = torch.randn(2, B, L, 2, H, d, device="cuda")
    rng[0] -= 5.0
    rng[1] += 5.0
    n_tok = np.array([0, 21], dtype=np.int32)

    def score(seqs):
        cfg = cfg_of(len(seqs))
        st = [torch.zeros(E.state_bytes(cfg), dtype=torch.uint8, device="cuda") for _ in range(2)]
        sec = E.state_sections(cfg, st[0])
        sec["n_tok"].copy_(dev(n_tok[seqs]))
        sec["range"].copy_(rng[:, seqs])
        n = E.workspace_bytes(cfg, C)
        ws = torch.full((n,), 0x7F, dtype=torch.uint8, device="cuda")
        sig = torch.zeros(1, len(seqs), C, device="cuda")
        E.epikv_score(cfg, C, pool=E.pool_of(pool), page_table=dev(pt[seqs]), ld_pt=pt.shape[1],
                      n_cached=dev(Ns[seqs].astype(np.int32)), state_in=st[0], state_out=st[1],
                      sig=sig, workspace=ws, workspace_bytes_=n)
        torch.cuda.synchronize()
        return host(sig)[0], host(E.state_sections(cfg, st[1])["range"])

    both = score([0, 1])
    for b in range(B):
        alone = score([b])
        assert np.array_equal(both[0][b], alone[0][0])
        assert np.array_equal(both[1][:, b], alone[1][:, 0])
