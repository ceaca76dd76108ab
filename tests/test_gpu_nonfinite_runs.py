"""Systems share waves, lanes' broadcasts and exchange areas: one that is not
finite (the batch's last, whose column the lanes past the batch repeat, and one
inside) leaves every other system's bits alone.  And the forced step's weights,
formed without a division, at states whose differences' fourth powers are near
the overflow end."""
import numpy as np
import pytest

from tests.gpu_util import dev, fp64_tol, host, rel_err

pytestmark = pytest.mark.gpu

# one chunk per wave by rows, through the scalar cache, ragged; 16 chunks in
# split groups; one wave for several systems
SIZES = [512, 256, 200, 1024, 1000]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_other_systems_keep_their_bits(n, bad):
    from paper_2107_05395_amd import Factor, inputs
    m = 5000
    c = inputs.uniform_batch(n, m, seed=n, lo=-0.1, hi=0.1)
    d = c.copy()
    d[n // 2, m - 1] = d[3, 77] = bad
    keep = np.ones(m, dtype=bool)
    keep[[77, m - 1]] = False
    (tb, tw), (pb, pw) = inputs.cn_diffusion_problem(n, 0.8), inputs.cn_hyperdiffusion_problem(n, 0.8)
    tri, penta = Factor.tri(*tb, cyclic=True), Factor.penta(*pb, cyclic=True)
    plain = Factor.penta(*inputs.random_dominant_penta(n, n))
    length = 2 * np.pi
    dx = length / n
    ch = Factor.cahn_hilliard(n, length, 0.01, 0.1 * dx)
    v, f0, k = dev(np.where(np.arange(m) % 2, 0.5, -0.7)), dev(np.ones(m)), dev(np.ones(m))
    calls = {
        "solve": lambda x: plain.solve(x),
        "periodic solve": lambda x: penta.solve(x),
        "refined solve": lambda x: tri.solve(x, precision="f32r"),
        "refined FP32 solve": lambda x: tri.solve(x.float(), precision="f32rhs"),
        "adjoint": lambda x: plain.adjoint(x),
        "tri steps": lambda x: tri.cn_step(x, tw, steps=3),
        "penta states": lambda x: penta.cn_trajectory(x, pw, 2),
        "steps": lambda x: ch.ch_step(x, ch.alpha, steps=2),
        "forced steps": lambda x: ch.ch_forced_step(x, 0.1 * dx, dx, v, f0, k, steps=2),
    }
    for name, call in calls.items():
        want, got = host(call(dev(c))), host(call(dev(d)))
        assert np.isfinite(want).all(), name
        assert np.array_equal(got[..., keep], want[..., keep]), name
        assert not np.isfinite(got[..., ~keep]).all(), name


@pytest.mark.parametrize("n", [512, 256, 100, 1000])
@pytest.mark.parametrize("scale", [1e30, 1e50, 1e70])
def test_forced_step_of_large_states(oracle, n, scale):
    from paper_2107_05395_amd import Factor, inputs
    m, length, gamma = 70, 2 * np.pi, 0.01
    dx = length / n
    dt = 0.1 * dx
    f = Factor.cahn_hilliard(n, length, gamma, dt)
    c0 = inputs.uniform_batch(n, m, 11) * scale
    v = np.where(np.arange(m) % 2 == 0, 0.5, -0.7)
    zero, k = np.zeros(m), np.ones(m)
    got = host(f.ch_forced_step(dev(c0), dt, dx, dev(v), dev(zero), dev(k), steps=1))
    ref = oracle.ch_forced_step(c0, f.sigma, f.alpha, dt * v / dx, zero, k * dx, steps=1)
    assert np.isfinite(ref).all() and np.isfinite(got).all()
    assert rel_err(got / scale ** 3, ref / scale ** 3) <= fp64_tol(1.0 + 16.0 * f.sigma, 1)
