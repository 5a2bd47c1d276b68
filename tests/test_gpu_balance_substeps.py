"""The balance controller's sums with contact sub-steps: taken along by the
first sub-step of the next step of a call, or by launches of their own after
the last one, and in graphs of one and of several steps.  The same functions
run either way: the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("n_sub", [1, 2, 3])
def test_balance_sums_with_sub_steps(W, H, n_sub, prec):
    print("balance sums: sub-steps", n_sub, "precision", prec, flush=True)
    dims = (70, 21, 18)
    sc = W.random_small_scene(3, dims, 8, size_range=(1.6, 2.6), gap=-0.4, speed=0.01)
    p = W.Params(nx=dims[0], ny=dims[1], nz=dims[2], tau=0.7, gravity=(0.0, 0.0, -2e-4),
                 balance=2, young=0.4, u_k=3e-4, max_pairs=256, tile_capacity=16,
                 precision=prec, n_sub=n_sub)
    out = []
    for calls, graph in (([67], False), ([1] * 67, False), ([5, 62], False), ([67], True),
                         ([1] * 3 + [64], True)):
        g = H.Simulation(p, sc, graph=graph)
        g.init_equilibrium()
        for n in calls:
            g.step(n)
        out.append((g.populations(), g.fluid_acceleration(), g.particles(), g.forces(),
                    g.counters()))
        g.close()
    f, a, q, F, k = out[0]
    assert np.abs(a).max() > 0
    for o in out[1:]:
        assert np.array_equal(o[0], f) and np.array_equal(o[1], a) and o[4] == k
        assert all(np.array_equal(o[2][m], q[m]) for m in q)
        assert all(np.array_equal(o[3][m], F[m]) for m in F)
