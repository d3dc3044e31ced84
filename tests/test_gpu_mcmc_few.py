"""Relocation with few dead: the moments are cleared by the list of the dead below
one in a hundred, by the words of what moved from there on (in steps of 65536
items), to the same result; against the oracle as in test_gpu_mcmc."""

import numpy as np
import pytest

from test_gpu_mcmc import _compare, _relocate, _state, gs  # noqa: F401  (the fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [900, 70_000])
@pytest.mark.parametrize("per_mille", [0, 1, 9.98, 10, 10.02, 80])
def test_relocate_few(gs, N, per_mille):  # noqa: F811
    rng = np.random.default_rng(int(N + 100 * per_mille))
    g, m1, m2 = _state(rng, N, 1, 0.0)
    dead = 3 + rng.permutation(N - 3)[:int(np.ceil(N * per_mille / 1000.0))]
    g["opacity_logit"] = np.maximum(g["opacity_logit"], np.float32(-4.0))
    g["opacity_logit"][dead] = -9.0
    u = rng.uniform(size=N).astype(np.float32)
    n, _ = _compare(g, m1, m2, u, 1, _relocate(gs, g, m1, m2, u, 1))
    assert n == len(dead)
