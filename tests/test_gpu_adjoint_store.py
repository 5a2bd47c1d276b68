"""Where the adjoint keeps its recorded window: lent memory, an allocation of
its own, the last segment kept from the record or run again.  Every way must
give the same gradient.  The forward run is bit-reproducible, so the reverse
sweeps differ only in the order of FP64 atomic sums: a few hundred terms of
one sign pattern per particle and step, bounded here by 1e-11 of the largest
component."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KSTEPS = 7


def _sim(W, H):
    dims = (33, 26, 21)           # no multiple of any block
    sc = W.random_small_scene(17, dims, 4, size_range=(1.8, 2.8), gap=1.5,
                              speed=0.01, spin=0.004)
    p = W.Params(nx=dims[0], ny=dims[1], nz=dims[2], tau=0.7,
                 gravity=(1e-5, 0.0, -2e-4), balance=1, young=0.4, u_k=3e-4,
                 max_pairs=64, tile_capacity=16)
    g = H.Simulation(p, sc)
    g.init_equilibrium(u=(0.002, 0.001, 0.0))
    return g


def _close(a, b):
    for k in a:
        scale = np.abs(b[k]).max()
        assert scale > 0 and np.abs(a[k] - b[k]).max() <= 1e-11 * scale, k


@pytest.mark.parametrize("every", [1, 3, 7, 50])
def test_window_stores_agree(W, H, every):
    print("adjoint store, checkpoints every", every, flush=True)
    seed = np.random.default_rng(5).normal(size=(4, 3))
    a = _sim(W, H)
    a.adjoint_record(KSTEPS, every)          # lent memory
    assert a.adj_mem is not None
    end = a.populations()
    first = a.adjoint_gradient(seed)
    assert np.array_equal(a.populations(), end)
    _close(a.adjoint_gradient(seed), first)  # the last segment run again

    b = _sim(W, H)                           # allocated by the library
    b._check(b.L.hlbm_adjoint_record(b.h, KSTEPS, every))
    assert np.array_equal(b.populations(), end)
    b.step(3)                                # the window outlives further steps
    _close(b.adjoint_gradient(seed), first)
    assert np.array_equal(b.populations(), end)

    c = _sim(W, H)                           # lent memory that is too small
    mem = c.torch.empty(4096, dtype=c.torch.uint8, device=c.device)
    c._check(c.L.hlbm_bind_adjoint(c.h, ctypes.c_void_p(mem.data_ptr()), 4096))
    c._check(c.L.hlbm_adjoint_record(c.h, KSTEPS, every))
    _close(c.adjoint_gradient(seed), first)
    for g in (a, b, c):
        g.close()
