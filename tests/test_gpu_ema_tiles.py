"""EMA smoothing of long chunks: a workgroup finds the average carried into
its tiles from the samples before them."""
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


@pytest.mark.parametrize("signal,na,nb,B,C,alpha,carried,bad", [
    ("hs", 7, 8, 2, 64, 0.9, True, None),
    ("hs", 7, 8, 2, 129, 0.9, False, None),            # two tiles before the last
    ("hs", 7, 8, 2, 64 * 5 + 1, 0.9, True, None),      # one group of four tiles, less one
    ("hs", 7, 8, 3, 64 * 18, 0.9, False, None),        # a whole round of loads, one tile more
    ("hs", 9, 9, 5, 64 * 70 + 3, 0.999, True, None),   # several tiles each; two rows a wavefront
    ("hs", 2, 0, 1, 20011, 0.9, False, None),
    ("hs", 2, 2, 2, 1000, 1.0, True, None),
    ("hs", 2, 2, 2, 1000, 0.0, False, None),
    ("hs", 2, 2, 2, 1000, 0.9, True, np.inf),
    ("hs", 2, 2, 2, 1000, 0.9, True, np.nan),
    ("kv_key", 7, 8, 3, 64 * 21 + 63, 0.9, False, None),
])
def test_one_call_gives_the_bits_of_64_token_calls(E, signal, na, nb, B, C, alpha, carried, bad):
    """One call over the chunk against calls of at most 64 tokens, a tile
    each (checked against the oracle elsewhere), with the state handed on."""
    import torch
    print(f"ema {signal} B={B} C={C} alpha={alpha} carried={carried} bad={bad}", flush=True)
    g = synth.rng(1901)
    cfg = E.default_cfg(batch=B, n_band_a=na, n_band_b=nb, hidden=64, ema_alpha=alpha,
                        signal=E.SIGNAL_HS if signal == "hs" else E.SIGNAL_KV_KEY,
                        smoothing=E.SMOOTH_EMA)
    n_sig = E.n_sig(cfg)
    x = (90.0 * np.exp(0.5 * g.standard_normal((n_sig, B, C)))).astype(np.float32)
    if bad is not None:
        x[0, 0, 70] = bad
    start = 500 if carried else 0
    ld = start + C

    def fresh_state():
        st = [torch.zeros(E.state_bytes(cfg), dtype=torch.uint8, device="cuda") for _ in range(2)]
        sec = E.state_sections(cfg, st[0])
        if carried:
            sec["n_tok"].fill_(start)
            sec["ring"].copy_(dev(ring))
            sec["ema"].copy_(dev(ema))
        return st

    ring = (90.0 + g.standard_normal((B, n_sig, 63))).astype(np.float32)
    ema = (90.0 + g.standard_normal((B, n_sig))).astype(np.float32)

    def run(pieces):
        st = fresh_state()
        scores = torch.zeros(B, ld, device="cuda")
        smooth, done = [], 0
        for n in pieces:
            sig = dev(x[:, :, done:done + n])
            done += n
            out = torch.full((n_sig, B, n), -7.0, device="cuda")
            n_cached = torch.full((B,), start + done, dtype=torch.int32, device="cuda")
            E.epikv_zscore(cfg, n, sig, n_cached, st[0], st[1], scores, ld, smoothed=out)
            torch.cuda.synchronize()
            smooth.append(host(out))
            st.reverse()
        sec = E.state_sections(cfg, st[0])
        return (host(scores), np.concatenate(smooth, 2), host(sec["ring"]), host(sec["ema"]),
                host(sec["n_tok"]))

    whole = run([C])
    parts = run([64] * (C // 64) + ([C % 64] if C % 64 else []))
    for name, a, b in zip(("scores", "smoothed", "ring", "ema", "n_tok"), whole, parts):
        assert np.array_equal(a, b, equal_nan=True), name
