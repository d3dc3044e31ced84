"""Relocation at the edges of its blocks (64 items a wave, 1024 a block, rows in
steps of 8), with everything, nothing and all but one dead, and draws at both
ends of the range: against the oracle, as in test_gpu_mcmc (draws and copies
bit for bit, the opacity and scale rule to float rounding)."""

import numpy as np
import pytest

from test_gpu_mcmc import _compare, _relocate, _state, gs  # noqa: F401  (the fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("deg", [0, 1, 3])
@pytest.mark.parametrize("N", [4, 63, 64, 65, 1023, 1024, 1025, 5000])
def test_relocate_at_block_edges(gs, N, deg):
    rng = np.random.default_rng(N + deg)
    g, m1, m2 = _state(rng, N, deg, 0.4)
    u = rng.uniform(size=N).astype(np.float32)
    u[:: 7] = 0.0
    u[1:: 7] = np.float32(1.0) - np.float32(2.0) ** -24
    _compare(g, m1, m2, u, deg, _relocate(gs, g, m1, m2, u, deg))


@pytest.mark.parametrize("N", [1, 2, 700, 3000])
@pytest.mark.parametrize("case", ["none dead", "all dead", "one live"])
def test_relocate_extremes(gs, N, case):
    rng = np.random.default_rng(N)
    g, m1, m2 = _state(rng, N, 1, 0.0)
    g["opacity_logit"][:] = 1.0 if case == "none dead" else -9.0
    if case == "one live":
        g["opacity_logit"][N // 2] = 0.5
    u = rng.uniform(size=N).astype(np.float32)
    n, _ = _compare(g, m1, m2, u, 1, _relocate(gs, g, m1, m2, u, 1))
    assert n == (N - 1 if case == "one live" else 0)
