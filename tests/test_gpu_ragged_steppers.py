"""Fused steppers with one chunk per wave where no power-of-two number of
chunks tiles n: the wave count and the last wave's rows at their edges (a last
chunk of 1, 2 or 3 rows, so that rows n-1 .. n-3 lie in two waves; one whose
periodic ghost rows reach past its padding; chunks that tile n), against the
oracle and against the kernel with one wave per group of systems."""
import ctypes

import numpy as np
import pytest

from paper_2107_05395_amd import _lib, inputs
from tests.gpu_util import dev, fp64_tol, host, lbar_tol, rel_err

EDGES = [(32, n) for n in (33, 34, 35, 61, 62, 63, 95, 96, 97, 224, 225, 255)] + \
        [(64, n) for n in (40, 63, 65, 66, 67, 126, 127, 192, 257, 320, 449, 450, 451, 509, 510, 511)]


def test_plans_hold_every_row_once():
    """Every stepper plan covers n rows, with no empty chunk where each wave
    has its own."""
    L = _lib.lib()
    for n in list(range(5, 600)) + [1000, 1024]:
        h = ctypes.c_void_p()
        bands = [np.ascontiguousarray(b) for b in inputs.ch_penta_bands(n, 0.3)]
        assert L.bb_factor_shared_penta_cyclic(*(_lib.dptr(a) for a in bands), n, ctypes.byref(h)) == 0
        for m in (1, 100, 3000, 5000, 20000, 1 << 17):
            o = [ctypes.c_int32() for _ in range(4)]
            assert L.bb_plan(h, m, 1, 0, *(ctypes.byref(x) for x in o)) == 0
            chunk, lanes, waves, scalar = (x.value for x in o)
            assert chunk * lanes >= n, (n, m)
            if scalar:
                assert waves == lanes <= 8 and (lanes - 1) * chunk < n, (n, m)
        L.bb_factor_destroy(h)


def _both(tuning, chunk, call):
    """The call's results with one chunk per wave and with one wave per group."""
    tuning.set("max_chunk", chunk)
    ours = call()
    tuning.set("waves_per_system", 1)
    general = call()
    tuning.reset()
    return ours, general


@pytest.mark.gpu
@pytest.mark.parametrize("chunk,n", EDGES)
def test_ragged_crank_nicolson(oracle, tuning, chunk, n):
    from paper_2107_05395_amd import Factor
    m, steps, real = 70, 3, -(-n // chunk)   # two groups of 64 systems, the second with six
    for kind, cyclic in (("tri", True), ("tri", False), ("penta", True), ("penta", False)):
        bands, w = (inputs.cn_diffusion_problem if kind == "tri" else
                    inputs.cn_hyperdiffusion_problem)(n, 0.7)
        if not cyclic:
            bands = (inputs.random_dominant_tri if kind == "tri" else inputs.random_dominant_penta)(n, n)
            w = tuple(inputs.rng(n + 1).uniform(-1, 1, len(bands)))
        f = (Factor.tri if kind == "tri" else Factor.penta)(*bands, cyclic=cyclic)
        c0 = inputs.uniform_batch(n, m, seed=n)
        ref = oracle.cn_step(bands, w, c0, steps=steps, cyclic=cyclic)
        for got in _both(tuning, chunk, lambda: host(f.cn_step(dev(c0), w, steps=steps))):
            assert rel_err(got, ref) < fp64_tol(), (kind, cyclic)   # kappa below 50
        tuning.set("max_chunk", chunk)
        assert f.plan(m, stepper=True) == dict(chunk=chunk, lanes=real, waves=real, scalar=True)
        states = f.cn_trajectory(dev(c0), w, steps)
        assert np.array_equal(host(states[-1]), host(f.cn_step(dev(c0), w, steps=steps)))
        lam = host(f.adjoint_trajectory(dev(c0), 1)[0])
        assert rel_err(lam, host(f.adjoint(dev(c0)))) < fp64_tol()
        tuning.reset()


@pytest.mark.gpu
@pytest.mark.parametrize("chunk,n", EDGES)
def test_ragged_cahn_hilliard(oracle, tuning, chunk, n):
    from paper_2107_05395_amd import Factor
    m, steps, length = 70, 4, 2 * np.pi
    dx = length / n
    f = Factor.cahn_hilliard(n, length, 0.01, 0.1 * dx)
    sigma, alpha = oracle.ch_coefficients(0.01, dx, 0.1 * dx)
    g = inputs.rng(n)
    v, f0 = g.uniform(-1, 1, m), g.uniform(0, 2, m)
    k = g.integers(1, 4, m).astype(np.float64)
    c0 = inputs.uniform_batch(n, m, seed=n + 1, lo=-0.5, hi=0.5)
    tol = fp64_tol(1.0 + 16.0 * sigma, steps)   # of the scale of the start, see lbar_tol
    lref, ref = oracle.ch_coarsening(c0, sigma, alpha, steps, 2)
    fref = oracle.ch_forced_step(c0, sigma, alpha, *oracle.ch_forced_parameters(0.1 * dx, dx, v, f0, k),
                                 steps=steps)
    t, kw = dev(c0), dict(dt=0.1 * dx, dx=dx, v=dev(v), f0=dev(f0), k=dev(k))
    for got in _both(tuning, chunk, lambda: host(f.ch_forced_step(t, steps=steps, **kw))):
        assert np.max(np.abs(got - fref)) < tol * np.max(np.abs(fref))
    for out, lbar in _both(tuning, chunk, lambda: f.ch_step_stats(t, f.alpha, steps=steps, every=2)):
        assert np.max(np.abs(host(out) - ref)) < tol * np.max(np.abs(c0))
        assert np.max(np.abs(host(lbar) - lref) / (lref - 1.0)) < lbar_tol(1.0 + 16.0 * sigma, steps, c0, lref)
