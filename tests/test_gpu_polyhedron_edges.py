"""A polyhedron's distance at points nearest to an edge or a vertex: the
search evaluates only the edges that the point lies beyond.  Plates, needles,
sharp tetrahedra and random hulls with a coupling band reaching 1.75 cells
out; the coupling weight of every node against the FP64 oracle.  Both take the
same distance with other roundings: at most some 20 units in the last place of
lengths up to 10 (4e-14), times the ramp's slope (below 0.5): 1e-13."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _body(W, name):
    if name == "plate":
        return W.polyhedron_cuboid(0.3, 2.0, 2.2)
    if name == "needle":
        return W.polyhedron_cuboid(0.5, 0.6, 3.0)
    if name == "tetrahedron":
        return W.polyhedron_tetrahedron(2.4)
    return W.polyhedron_random(np.random.default_rng(int(name)), 12)


@pytest.mark.parametrize("name", ["plate", "needle", "tetrahedron", "3", "8", "21"])
def test_distance_beyond_edges(O, W, H, name):
    print("polyhedron edges:", name, flush=True)
    dims = (27, 25, 22)
    P = _body(W, name)
    O.define_polyhedron(0, P.vertices, P.faces)
    rc = O.polyhedron_info(0, len(P.vertices))[2]
    rng = np.random.default_rng(11)
    q = rng.normal(size=(2, 4))
    sc = W.Scene(np.full(2, W.POLY0, np.int32), np.full(2, 4.5 / rc), np.full(2, 1.5),
                 np.array([[7.3, 6.1, 5.7], [20.4, 17.2, 15.9]]),
                 q / np.linalg.norm(q, axis=1)[:, None], np.zeros((2, 3)), np.zeros((2, 3)))
    p = W.Params(nx=dims[0], ny=dims[1], nz=dims[2], tau=0.7, young=0.4, u_k=3e-4,
                 max_pairs=64, tile_capacity=16, eps_b=3.5)
    o, g = O.OracleSim(p, sc), H.Simulation(p, sc, polyhedra={0: P})
    o.init_equilibrium()
    g.init_equilibrium()
    fo = o.fields()
    assert np.array_equal(g.fields()["owner"], fo["owner"])
    B = g.coupling()["B"]
    assert ((B > 0) & (B < 1)).sum() > 100
    assert np.abs(B - fo["B"]).max() <= 1e-13
