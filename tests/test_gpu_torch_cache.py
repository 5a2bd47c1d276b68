"""The library allocates beside torch's allocator, which keeps the blocks of
closed simulations (populations, adjoint windows) for later use: where the
library finds no memory, they are given back first."""
import gc

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GB = 1 << 30


def test_simulation_beside_unused_torch_blocks(W, H):
    import torch
    print("simulation beside unused torch blocks", flush=True)
    gc.collect()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info(0)[0]
    block = torch.empty(free - 6 * GB, dtype=torch.uint8, device="cuda:0")
    del block                     # unused from here on, but torch's
    assert torch.cuda.mem_get_info(0)[0] < 8 * GB
    # two pair tables of 2^25 slots, about 7 GB each
    sc = W.random_small_scene(3, (26, 22, 20), 4, size_range=(1.8, 2.8), gap=0.5)
    p = W.Params(nx=26, ny=22, nz=20, tau=0.7, young=0.4, u_k=3e-4, max_pairs=1 << 24,
                 tile_capacity=16)
    g = H.Simulation(p, sc)
    g.init_equilibrium()
    g.step(2)
    g.sync()
    g.close()
    del g
    # and the particles' blocks: 200 000 spheres of radius 25 in a box of 64^3
    # list up to 944 lattice blocks of 48 bytes each, 9 GB
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info(0)[0]
    block = torch.empty(free - 3 * GB, dtype=torch.uint8, device="cuda:0")
    del block
    n = 200_000
    sc = W.Scene(np.zeros(n, np.int32), np.full(n, 25.0), np.full(n, 2.0), np.full((n, 3), 32.0),
                 np.tile([1.0, 0.0, 0.0, 0.0], (n, 1)), np.zeros((n, 3)), np.zeros((n, 3)))
    p = W.Params(nx=64, ny=64, nz=64, tau=0.7, young=0.4, u_k=3e-4, max_pairs=64,
                 tile_capacity=16)
    H.Simulation(p, sc).close()
    torch.cuda.empty_cache()
