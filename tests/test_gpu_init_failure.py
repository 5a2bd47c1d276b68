"""A particle set that does not fit the device: the call reports it, the
context then has no particles (nothing of the earlier set, whose memory is
gone, and nothing of the new one), and the next set starts afresh."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

E_STATE = -6


def _init(H, g, X, size):
    n = len(X)
    a = [np.full(n, size), np.full(n, 2.0), np.ascontiguousarray(X, np.float64),
         np.tile([1.0, 0.0, 0.0, 0.0], (n, 1)), np.zeros((n, 3)), np.zeros((n, 3))]
    shape = np.zeros(n, np.int32)
    return g.L.hlbm_init_particles(g.h, n, H._ip(shape), *[H._dp(v) for v in a])


def test_particles_that_do_not_fit(W, H):
    print("particle set that does not fit", flush=True)
    dims = (128, 128, 128)
    sc = W.random_small_scene(4, dims, 3, size_range=(3.0, 4.0), gap=2.0)
    p = W.Params(nx=dims[0], ny=dims[1], nz=dims[2], tau=0.7, young=0.4, u_k=3e-4,
                 max_pairs=64, tile_capacity=16)
    g = H.Simulation(p, sc)
    g.init_equilibrium()
    # 10^6 spheres of radius 58: 8000 lattice blocks each, 48 bytes per
    # particle and block, 384 GB of partial sums
    n = 1_000_000
    total = g.torch.cuda.get_device_properties(g.device).total_memory
    assert 8000 * 48 * n > total
    assert _init(H, g, np.full((n, 3), 64.0), 58.0) != 0
    buf = np.zeros(3 * n)
    # (each checked before the next: the later ones would run on the freed set)
    for call in (lambda: g.L.hlbm_read_particles(g.h, H._dp(buf), None, None, None),
                 lambda: g.L.hlbm_read_forces(g.h, H._dp(buf), None, None, None),
                 lambda: g.L.hlbm_step(g.h, 0),
                 lambda: g.L.hlbm_init_fluid_equilibrium(g.h, 1.0, H._dp(np.zeros(3)))):
        assert call() == E_STATE
    # a set that fits: as in a new simulation
    assert _init(H, g, sc.X, 3.5) == 0
    g.np = sc.n
    g.init_equilibrium()
    g.step(2)
    f = g.populations()
    sc.shape[:], sc.size[:], sc.density[:] = W.SPHERE, 3.5, 2.0
    sc.q[:], sc.U[:], sc.omega[:] = [1.0, 0.0, 0.0, 0.0], 0.0, 0.0
    o = H.Simulation(p, sc)
    o.init_equilibrium()
    o.step(2)
    assert np.array_equal(f, o.populations())
    assert all(np.array_equal(g.particles()[k], v) for k, v in o.particles().items())
    g.close()
    o.close()
