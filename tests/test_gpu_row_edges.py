"""The lattice pass takes the owners of a node's neighbours along x from the
neighbouring lanes of its wavefront and, at the ends of a 64-node row segment,
from separate loads: particles across x = 0 and across x = 64, on rows that
end inside a segment, with it, and one node after it.  The momentum exchange
must come out as in the FP64 oracle, within the tolerances of the parity tests
(1e-11 FP64, 1e-4 FP32, 1e-2 binary16 of the larger of the force and a
reference force after a few steps): a missed or doubled link changes a force
by whole per cents."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FTOL = {0: 1e-11, 1: 1e-4, 2: 1e-2}


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("nx,pz", [(13, 1), (63, 0), (64, 1), (65, 1), (66, 0), (128, 1)])
def test_row_ends(O, W, H, nx, pz, prec):
    print("row ends: nx", nx, "periodic z", pz, "precision", prec, flush=True)
    dims = (nx, 17, 14)
    rng = np.random.default_rng(nx)
    xs = [0.3, (nx if nx < 40 else 63.6) - 5.2, 63.6] if nx >= 40 else [0.3]
    n = len(xs)
    sc = W.Scene(np.array([W.SPHERE, W.CUBE, W.SPHERE][:n], np.int32),
                 np.array([2.3, 3.1, 2.1][:n]), np.array([1.5, 2.0, 1.2][:n]),
                 np.array([[x % nx, 7.4 + 0.3 * i, 6.6 - 0.2 * i] for i, x in enumerate(xs)]),
                 np.tile([1.0, 0.0, 0.0, 0.0], (n, 1)), 0.01 * rng.normal(size=(n, 3)),
                 0.004 * rng.normal(size=(n, 3)))
    p = W.Params(nx=dims[0], ny=dims[1], nz=dims[2], periodic_z=pz, tau=0.7,
                 gravity=(0.0, 0.0, -2e-4), balance=pz, young=0.4, u_k=3e-4,
                 max_pairs=64, tile_capacity=16, precision=prec)
    f0 = W.perturbed_populations(nx, dims, O.feq(1.0, [0.004, -0.002, 0.001]), amp=0.01)
    o, g = O.OracleSim(p, sc), H.Simulation(p, sc)
    o.set_populations(f0)
    g.set_populations(f0)
    Fref = 2e-4 * 0.5 * (4 / 3 * math.pi * 1.6 ** 3)
    for _ in range(3):
        o.step(1)
        g.step(1)
        if prec == 0:
            assert np.array_equal(g.fields()["owner"], o.fields()["owner"])
        fo, fg = o.forces()["Fh"], g.forces()["Fh"]
        err = (np.abs(fg - fo) / np.maximum(np.abs(fo), Fref)).max()
        print(f"  force error {err:.2e}", flush=True)
        assert err <= FTOL[prec]
