"""Hidden-state scoring of rows wider than 4096: segments of 32 tokens, or
shorter ones where the call would leave compute units idle."""
import pytest

from harness import POSITIVE, TOL, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2606_26472_amd import epikv
    epikv.lib()
    return epikv


@pytest.mark.parametrize("D", [4104, 5120, 8192, 16384])
@pytest.mark.parametrize("C", [70, 3])
def test_any_segment_length_gives_the_same_bits(E, D, C):
    """24 sequences in one call (segments of 32), 5 of them (16), and each of
    two alone (4): the same bits, and those of 64-bit sums within the
    tolerance; one sequence of the three is fresh."""
    import torch
    print(f"score wide D={D} C={C}", flush=True)
    torch.manual_seed(D + C)
    B, na, nb = 24, 7, 8
    n = na + nb
    hid = [torch.randn(B, C, D, device="cuda").to(torch.bfloat16) for _ in range(n)]
    before = torch.randn(B, n, D, device="cuda").to(torch.bfloat16)
    n_tok = torch.full((B,), 9, dtype=torch.int32, device="cuda")
    n_tok[1] = 0

    def score(lo, hi):
        b = hi - lo
        cfg = E.default_cfg(batch=b, hidden=D, n_band_a=na, n_band_b=nb)
        st = [torch.zeros(E.state_bytes(cfg), dtype=torch.uint8, device="cuda") for _ in range(2)]
        sec = E.state_sections(cfg, st[0])
        sec["n_tok"].copy_(n_tok[lo:hi])
        sec["h_prev"].copy_(before[lo:hi].view(torch.int16))
        sig = torch.full((n, b, C), -7.0, device="cuda")
        E.epikv_score(cfg, C, [h[lo:hi] for h in hid], D, C * D, state_in=st[0], state_out=st[1],
                      sig=sig)
        torch.cuda.synchronize()
        return host(sig), host(E.state_sections(cfg, st[1])["h_prev"])

    whole, last = score(0, B)
    for lo, hi in ((0, 5), (0, 1), (1, 2)):
        part, part_last = score(lo, hi)
        assert (part == whole[:, lo:hi]).all()
        assert (part_last == last[lo:hi]).all()
    for l in range(n):
        h = hid[l].double()
        prev = torch.cat([before[:, l:l + 1].double(), h[:, :-1]], 1)
        ref = (h - prev).square().sum(-1).sqrt()
        ref[1, 0] = 0.0
        assert rel_err(whole[l], host(ref), POSITIVE) <= TOL
        assert (last[:, l] == host(hid[l][:, -1].view(torch.int16))).all()
