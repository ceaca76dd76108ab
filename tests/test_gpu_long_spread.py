"""The scan of a long system by one workgroup at the edges of its blocks: 64
chunks per wave, up to 8 waves, several rounds of 8, one wave from 257 systems
on.  A chain of affine maps scanned in blocks and step by step rounds
differently by a few units in the last place of the chunk-boundary states, and
the matrices' kappa is below 100: 1e-12 covers both against the oracle."""
import numpy as np
import pytest

from tests.gpu_util import dev, fp64_tol, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,cyclic", [("tri", False), ("tri", True), ("penta", False), ("penta", True)])
@pytest.mark.parametrize("full,tail,m", [(128, 1, 3), (129, 32, 2), (511, 5, 1), (512, 32, 2), (513, 2, 1),
                                         (1025, 31, 1), (70, 32, 256), (70, 32, 257)])
def test_block_edges(oracle, tuning, kind, cyclic, full, tail, m):
    from paper_2107_05395_amd import Factor, inputs
    n = 32 * full + tail
    bands = (inputs.random_dominant_tri if kind == "tri" else inputs.random_dominant_penta)(n, 3)
    f = (Factor.tri if kind == "tri" else Factor.penta)(*bands, cyclic=cyclic)
    rhs = inputs.uniform_batch(n, m, 4)
    tuning.set("max_chunk", 32)
    for spread in (1, 0):
        tuning.set("long_spread", spread)
        x = host(f.solve(dev(rhs)))
        r = [rhs[i] - sum(b[i] * x[(i + q - len(bands) // 2) % n] for q, b in enumerate(bands)
                          if cyclic or 0 <= i + q - len(bands) // 2 < n) for i in range(n)]
        size = max(np.max(np.abs(b)) for b in bands) * np.max(np.abs(x)) + np.max(np.abs(rhs))
        assert np.max(np.abs(r)) < fp64_tol() * size, spread
        if spread:
            first = x
    assert rel_err(first, x) < fp64_tol()
