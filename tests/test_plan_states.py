"""Host logic of the decomposition (no GPU): the steppers that store every
state (trajectories, one step a call; bb_plan what = 3) and those that keep it
on chip (what = 1) where their rules differ and where they agree, and the wave
counts of ragged systems."""
import ctypes

import numpy as np
import pytest

from paper_2107_05395_amd import _lib, inputs


def plan(kind, n, m, what):
    L = _lib.lib()
    h = ctypes.c_void_p()
    bands = (inputs.cn_diffusion_problem if kind == "tri" else inputs.cn_hyperdiffusion_problem)(n, 1.0)[0]
    arrs = [np.ascontiguousarray(b, dtype=np.float64) for b in bands]
    assert getattr(L, "bb_factor_shared_%s_cyclic" % kind)(*(_lib.dptr(a) for a in arrs), n, ctypes.byref(h)) == 0
    out = [ctypes.c_int32() for _ in range(4)]
    assert L.bb_plan(h, m, what, 0, *(ctypes.byref(o) for o in out)) == 0
    L.bb_factor_destroy(h)
    return tuple(o.value for o in out)


# (kind, n, m) -> (chunk, lanes, waves, scalar) on chip, with the states stored
CASES = [
    ("tri", 1024, 1 << 16, (64, 16, 4, 0), (64, 16, 8, 0)),
    ("tri", 1024, 4096, (64, 16, 4, 0), (64, 16, 8, 0)),
    ("tri", 1024, 4095, (32, 32, 8, 0), (32, 32, 8, 0)),   # small batch: 32-row chunks
    ("penta", 1024, 1 << 16, (64, 16, 8, 0), (64, 16, 8, 0)),
    ("tri", 2048, 1 << 16, (64, 32, 8, 0), (64, 32, 8, 0)),
    ("tri", 512, 1 << 17, (64, 8, 8, 1), (64, 8, 8, 1)),
    # ragged: one chunk per wave up to 8 chunks
    ("penta", 500, 5000, (64, 8, 8, 1), (64, 8, 8, 1)),
    ("penta", 300, 1 << 16, (64, 5, 5, 1), (64, 5, 5, 1)),
    ("tri", 200, 1 << 13, (32, 7, 7, 1), (32, 7, 7, 1)),
    ("tri", 40, 1 << 17, (64, 1, 1, 1), (64, 1, 1, 1)),
    ("tri", 1000, 1 << 16, (64, 16, 1, 0), (64, 16, 1, 0)),
]


@pytest.mark.parametrize("kind,n,m,on_chip,stored", CASES)
def test_stepper_plans(kind, n, m, on_chip, stored):
    assert plan(kind, n, m, 1) == on_chip
    assert plan(kind, n, m, 3) == stored


def test_python_plan_with_states():
    from paper_2107_05395_amd import Factor
    f = Factor.tri(*inputs.diffusion_tri_bands(1024, 1.0))
    assert f.plan(1 << 16, stepper=True)["waves"] == 4
    assert f.plan(1 << 16, stepper=True, states=True)["waves"] == 8
