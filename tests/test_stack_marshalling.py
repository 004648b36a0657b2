"""Stack arrays built one by one (few stacks) and through NumPy (many) hold what the dicts hold."""
import ctypes

import numpy as np
import pytest

import paper_2502_03170_amd as rw


@pytest.mark.parametrize("n", [0, 1, 3, 4, 5, 40])
def test_make_stacks_holds_the_values(n):
    rng = np.random.default_rng(n)
    kinds = [None, (), [1, 2.5, np.float32(0.1)], rng.normal(size=22), rng.normal(size=5).astype(np.float32),
             np.arange(3), rng.normal(size=44)[::2], np.float64(2.0) * np.ones(36)]
    stacks = [dict(t_s=3 * i, z_offset=np.float32(0.1 * i), zernike=kinds[i % len(kinds)]) for i in range(n)]
    for i in range(0, n, 2):
        stacks[i].update(x0=-1.5 * i, y0=np.float64(i))
    arr, keep = rw.make_stacks(stacks)
    assert isinstance(arr, ctypes.Array) and arr._type_ is rw.Stack and len(arr) == n
    for a, s in zip(arr, stacks):
        assert (a.t_s_nm, a.x0_nm, a.y0_nm, a.z_offset_nm) == tuple(
            float(s.get(k, 0.0)) for k in ("t_s", "x0", "y0", "z_offset"))
        c = [] if s["zernike"] is None else [float(v) for v in s["zernike"]]
        assert a.n_zernike == len(c) and [a.zernike_waves[q] for q in range(len(c))] == c
        assert not a.phase_map


@pytest.mark.parametrize("n", [1, 6])
@pytest.mark.parametrize("bad", [dict(x0=None), dict(zernike=[1j]), dict(zernike=np.zeros((2, 3)))])
def test_make_stacks_refuses(n, bad):
    with pytest.raises(TypeError):
        rw.make_stacks([dict()] * (n - 1) + [bad])
