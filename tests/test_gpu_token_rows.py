"""The fused per-token scorer at the edges of its row pipeline and of the
window statistics: rows that end inside a wavefront's last 16-byte columns,
chunks of one row, of fewer rows than are kept in flight, around that many and
of the most a call takes, more band rows than a workgroup has wavefronts,
windows around 64 and of one sample.  Bit for bit the two separate calls, and
the oracle's float64 scores."""
import numpy as np
import pytest

import synth
from harness import NEAR_ZERO, TOL, rel_err
from test_gpu_online import E, _oracle_stream, _score_stream  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,na,nb,window,mode", [
    (8, 1, 0, 64, "mean"), (504, 2, 1, 64, "z"), (520, 7, 8, 63, "z"), (1016, 1, 1, 65, "mean"),
    (2048, 16, 16, 64, "z"), (2056, 9, 8, 256, "z"), (3080, 2, 2, 1, "raw"), (4096, 7, 8, 64, "z"),
    (4096, 3, 2, 2, "mean")])
def test_token_rows(E, D, na, nb, window, mode):  # noqa: F811
    chunks = [1, 1, 2, 3, 4, 5, 6, 7, 8, 9, 1, 17, 64, 1, 64, 2]
    print(f"token rows D {D} bands {na}+{nb} window {window} {mode}", flush=True)
    g = np.random.default_rng(D + window)
    T = sum(chunks)
    scale = np.exp(g.normal(0.0, 0.5, size=(na + nb, 1, T, 1)))
    hid = synth.f32_to_bf16_bits(
        (g.standard_normal((na + nb, 2, T, D)) * scale).astype(np.float32))
    smode = {"z": E.SMOOTH_Z, "mean": E.SMOOTH_MEAN, "raw": E.SMOOTH_RAW}[mode]
    cfg = E.default_cfg(batch=2, hidden=D, n_band_a=na, n_band_b=nb, smoothing=smode,
                        window=window)
    assert E.check_cfg(cfg) == 0
    two = _score_stream(E, cfg, hid, chunks)
    fused = _score_stream(E, cfg, hid, chunks, fused=True)
    assert fused[0].tobytes() == two[0].tobytes()
    assert fused[1].tobytes() == two[1].tobytes()
    ref = _oracle_stream(hid, na, nb, mode, window)
    assert rel_err(fused[0], ref, NEAR_ZERO) <= TOL
