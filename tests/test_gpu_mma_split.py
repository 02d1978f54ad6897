"""The matrix-core sweep whose workgroups split every row's steps over four waves (16-bit, int8): rows of
fewer steps than waves (some waves have none), of uneven shares and with a ragged last step, over
several row groups with a ragged last one, several matrices in one call and the outputs' bounds."""
import numpy as np
import pytest

import oracle
import synth
from synth import workloads as wl
from gpu_util import needs_gpu, rel_l2
from test_gpu_mma import TOL, host_matrix, run_mma

pytestmark = [pytest.mark.gpu, needs_gpu]

STEP = {wl.F16: 64, wl.BF16: 64, wl.I8: 128}      # weights of a 128-byte step


@pytest.mark.parametrize("fmt", [wl.F16, wl.BF16, wl.I8])
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 7, 9])
@pytest.mark.parametrize("ragged", [0, 16], ids=["whole", "ragged"])
def test_split_steps(fmt, steps, ragged):
    M, T, K = 150, 5, steps * STEP[fmt] + ragged
    W, S = host_matrix(fmt, M, K, seed=31)
    X = synth.normal16((T + 1, K), wl.X_SIGMA, wl.BF16 if fmt == wl.BF16 else wl.F16, seed=31, stream=631)
    y = run_mma(fmt, W, S, X, M, K, T, y_rows=M + 3)
    assert np.isnan(y[:, M:]).all() and np.isnan(y[T:]).all()
    ora = oracle.get()
    for t in range(T):
        want = ora.gemv(dict(fmt=fmt, w=W, s=S), X[t]) if fmt == wl.I8 else ora.gemv16(W, X[t], fmt)
        assert rel_l2(y[t, :M], want) <= TOL, (fmt, K, t)
