"""The fused per-token scorer at the edges of its walks over a chunk's rows and
of the window statistics: rows that end inside a wavefront's last 16-byte
columns, chunks of one row, of so few that they go row by row, around the
number that is pipelined and of the most a call takes, more sequences than the
widest rows are pipelined for, more band rows than a workgroup has wavefronts,
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
    _rows(E, D, na, nb, window, mode, 2, [1, 1, 2, 3, 4, 5, 6, 7, 8, 9, 1, 17, 64, 1, 64, 2])


@pytest.mark.parametrize("D,B", [(2048, 65), (2056, 64), (2056, 65), (4096, 66)])
def test_token_rows_of_many_sequences(E, D, B):  # noqa: F811
    _rows(E, D, 1, 1, 64, "z", B, [1, 8, 9, 10, 2, 64])


def _rows(E, D, na, nb, window, mode, B, chunks):  # noqa: F811
    print(f"token rows D {D} B {B} bands {na}+{nb} window {window} {mode}", flush=True)
    g = np.random.default_rng(D + window)
    T = sum(chunks)
    scale = np.exp(g.normal(0.0, 0.5, size=(na + nb, 1, T, 1)))
    hid = synth.f32_to_bf16_bits(
        (g.standard_normal((na + nb, B, T, D)) * scale).astype(np.float32))
    smode = {"z": E.SMOOTH_Z, "mean": E.SMOOTH_MEAN, "raw": E.SMOOTH_RAW}[mode]
    cfg = E.default_cfg(batch=B, hidden=D, n_band_a=na, n_band_b=nb, smoothing=smode,
                        window=window)
    assert E.check_cfg(cfg) == 0
    two = _score_stream(E, cfg, hid, chunks)
    fused = _score_stream(E, cfg, hid, chunks, fused=True)
    assert fused[0].tobytes() == two[0].tobytes()
    assert fused[1].tobytes() == two[1].tobytes()
    ref = _oracle_stream(hid, na, nb, mode, window)
    assert rel_err(fused[0], ref, NEAR_ZERO) <= TOL
