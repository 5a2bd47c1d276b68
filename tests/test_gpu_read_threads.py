"""Read-outs of one simulation from several threads: each call returns the
state it asked for, whatever the other threads read meanwhile (the state does
not change, so every read-out has to give the same values)."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_read_outs_from_several_threads(W, H):
    print("read-outs from several threads", flush=True)
    dims = (40, 36, 32)
    sc = W.random_small_scene(8, dims, 12, size_range=(1.8, 3.0), gap=-0.5, speed=0.01,
                              spin=0.004)
    p = W.Params(nx=dims[0], ny=dims[1], nz=dims[2], tau=0.7, gravity=(0.0, 0.0, -1e-4),
                 young=0.4, u_k=3e-4, max_pairs=256, tile_capacity=16)
    g = H.Simulation(p, sc)
    g.init_equilibrium()
    g.step(3)
    calls = dict(particles=g.particles, forces=g.forces, fields=g.fields,
                 populations=lambda: dict(f=g.populations()))
    want = {name: call() for name, call in calls.items()}
    wrong = []

    def read(name, n):
        for _ in range(n):
            got = calls[name]()
            if not all(np.array_equal(got[k], want[name][k]) for k in want[name]):
                wrong.append(name)

    threads = [threading.Thread(target=read, args=a)
               for a in (("particles", 200), ("forces", 200), ("particles", 200),
                         ("fields", 20), ("populations", 20))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, {name: wrong.count(name) for name in set(wrong)}
    g.close()
