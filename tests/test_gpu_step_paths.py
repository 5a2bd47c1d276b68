"""Branches of a step and of the read-outs at the sizes where they change.

* Contact treatment: face and integration samples fill rounds of 128, so sample
  counts below, at and above a round (n_c from 1 to 32), for particle pairs and
  walls, against the FP64 oracle.  Counts exactly; the means and forces differ
  by the order of FP64 sums of at most 32^3 terms: 32^3 x 1.1e-16 = 4e-12,
  bounded by 1e-11.
* Detection: bands narrower than the screen's error, and wider than the
  detection reach, on lattices that end inside a tile; owners and pairs exactly.
* Balance sums inside the next step's launches or in launches of their own, and
  graphs: the same bits.
* Field read-outs of several chunks with a remainder: against the populations,
  sums of 19 terms of about 1/3 (1e-14).
"""
import numpy as np
import pytest

from test_gpu_parity import compare_contacts

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pz", [0, 1])
@pytest.mark.parametrize("n_c", [1, 3, 7, 8, 9, 12, 32])
def test_treatment_sample_rounds(O, W, H, n_c, pz):
    print("treatment: n_c", n_c, "periodic z", pz, flush=True)
    dims = (26, 21, 23)
    sc = W.random_small_scene(12, dims, 8, periodic_z=pz, size_range=(1.6, 3.0), gap=-0.8,
                              speed=0.01, spin=0.004)
    p = W.Params(nx=dims[0], ny=dims[1], nz=dims[2], periodic_z=pz, tau=0.7, young=0.4,
                 u_k=3e-4, max_pairs=256, tile_capacity=16, n_c=n_c)
    o, g = O.OracleSim(p, sc), H.Simulation(p, sc)
    o.init_equilibrium()
    g.init_equilibrium()
    o.step(1)
    g.step(1)
    assert len(o.contacts()) > 0
    compare_contacts(o.contacts(), g.contacts(), 1e-11)
    fo, fg = o.forces()["Fc"], g.forces()["Fc"]
    assert np.abs(fg - fo).max() <= 1e-11 * max(np.abs(fo).max(), 1e-300)


@pytest.mark.parametrize("dims,n", [((13, 17, 14), 1), ((30, 22, 18), 6)])
@pytest.mark.parametrize("eps_b", [1e-3, 0.5, 3.0])
def test_detection_bands(O, W, H, dims, n, eps_b):
    print("detection: eps_b", eps_b, dims, flush=True)
    sc = W.random_small_scene(5, dims, n, size_range=(1.5, 2.2), gap=-0.6)
    p = W.Params(nx=dims[0], ny=dims[1], nz=dims[2], tau=0.7, young=0.4, u_k=3e-4,
                 max_pairs=256, tile_capacity=32, eps_b=eps_b)
    o, g = O.OracleSim(p, sc), H.Simulation(p, sc)
    o.init_equilibrium()
    g.init_equilibrium()
    assert np.array_equal(g.fields()["owner"], o.fields()["owner"])
    assert (g.counters()["pairs"], g.counters()["cells"]) == o.counters()


@pytest.mark.parametrize("prec", [0, 1, 2])
def test_balance_paths_agree(W, H, prec):
    print("balance paths, precision", prec, flush=True)
    dims = (70, 21, 18)
    sc = W.random_small_scene(3, dims, 8, size_range=(1.6, 2.6), gap=-0.4, speed=0.01)
    p = W.Params(nx=dims[0], ny=dims[1], nz=dims[2], tau=0.7, gravity=(0.0, 0.0, -2e-4),
                 balance=2, young=0.4, u_k=3e-4, max_pairs=256, tile_capacity=16,
                 precision=prec)
    out = []
    for calls, graph in (([66], False), ([1] * 66, False), ([66], True), ([1, 64, 1], True)):
        g = H.Simulation(p, sc, graph=graph)
        g.init_equilibrium()
        for n in calls:
            g.step(n)
        out.append((g.populations(), g.particles(), g.fluid_acceleration()))
    for f, q, a in out[1:]:
        assert np.array_equal(f, out[0][0]) and np.array_equal(a, out[0][2])
        assert all(np.array_equal(q[k], out[0][1][k]) for k in q)


@pytest.mark.parametrize("dims", [(67, 41, 29), (128, 64, 8), (33, 9, 7)])
def test_field_read_outs(O, W, H, dims):
    print("field read-outs", dims, flush=True)
    p = W.Params(nx=dims[0], ny=dims[1], nz=dims[2], tau=0.7, young=0.4, u_k=3e-4,
                 max_pairs=8, tile_capacity=4)
    g = H.Simulation(p, W.Scene.empty())
    f0 = W.perturbed_populations(2, dims, O.feq(1.0, [0.004, -0.002, 0.001]), amp=0.01)
    g.set_populations(f0)
    o = O.OracleSim(p, W.Scene.empty())
    o.set_populations(f0)
    full, ref = g.fields(), o.fields()
    for k in ("rho", "u", "owner"):
        assert full[k].shape == ref[k].shape
        assert np.abs(full[k] - ref[k]).max() <= 1e-14, k
    for k in ("rho", "u", "owner"):                # one output alone
        only = g.fields(rho=k == "rho", u=k == "u", owner=k == "owner")
        assert np.array_equal(only[k], full[k]), k
