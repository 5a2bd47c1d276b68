"""Device memory of the adjoint's window: what a record holds until its
gradient, where the gradient's store stands, what a refused record leaves as
it was, what a larger window needs beside the one it replaces, and what may be
lent."""
import ctypes
import gc

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

E_ARG = -1
MB = 1 << 20


def _sim(W, H, dims=(64, 64, 64), **kw):
    # (nothing left of earlier simulations, whose unused blocks could serve here)
    import torch
    gc.collect()
    torch.cuda.empty_cache()
    sc = W.random_small_scene(17, dims, 4, size_range=(1.8, 2.8), gap=1.5, speed=0.01,
                              spin=0.004)
    p = W.Params(nx=dims[0], ny=dims[1], nz=dims[2], tau=0.7, gravity=(1e-5, 0.0, -2e-4),
                 balance=1, young=0.4, u_k=3e-4, max_pairs=64, tile_capacity=16).replace(**kw)
    g = H.Simulation(p, sc)
    g.init_equilibrium()
    g.sync()
    return g


def _free(g):
    """Device memory that nothing holds (torch's unused blocks given back)."""
    g.torch.cuda.synchronize()
    g.torch.cuda.empty_cache()
    return g.torch.cuda.mem_get_info(g.device)[0]


def test_record_holds_snapshots_only(W, H):
    """The population fields of the reverse sweep are the gradient's: a program
    that records many windows before its first gradient holds the snapshots
    alone (a start and an end state here: two fields of 40 MB and their
    tables, against 43 fields in the sweep)."""
    print("adjoint memory: record", flush=True)
    g = _sim(W, H)
    field = 19 * 8 * 64 ** 3
    seed = np.random.default_rng(5).normal(size=(4, 3))
    free = _free(g)
    g.adjoint_record(40, 40)
    held = free - _free(g)
    assert 2 * field <= held <= 2 * field + 64 * MB
    r = g.adjoint_gradient(seed)
    # the window stays, for another gradient of it
    assert free - _free(g) <= held + 43 * field + 64 * MB
    again = g.adjoint_gradient(seed)
    for k in r:
        assert np.abs(r[k]).max() > 0
        assert np.abs(again[k] - r[k]).max() <= 1e-11 * np.abs(r[k]).max(), k
    g.close()


@pytest.mark.parametrize("every", [3, 7])
def test_stores_lent_and_allocated_agree(W, H, every):
    """Where the store of a gradient stands: in one block with the snapshots, in
    a block of its own lent before the record (which then leaves the last
    segment there) or after it, in an allocation.  The reverse sweeps differ
    only in the order of FP64 atomic sums (1e-11 of the largest component, a few
    hundred terms of one sign pattern per particle and step)."""
    print("adjoint memory: stores, checkpoints every", every, flush=True)
    seed = np.random.default_rng(5).normal(size=(4, 3))
    size = ctypes.c_size_t
    first = None

    def gradient(g):
        out = dict(s=np.zeros(4), theta0=np.zeros((4, 3)), q0=np.zeros((4, 4)),
                   X0=np.zeros((4, 3)), U0=np.zeros((4, 3)), omega0=np.zeros((4, 3)))
        assert g.L.hlbm_adjoint_gradient(g.h, H._dp(seed), *[H._dp(v) for v in out.values()]) == 0
        return out

    for how in ("binding", "whole", "before", "after", "allocated", "one call", "its own"):
        g = _sim(W, H, dims=(33, 26, 21))
        L, snapshots, store, both = g.L, size(), size(), size()
        assert L.hlbm_adjoint_parts(g.h, 7, every, ctypes.byref(snapshots), ctypes.byref(store)) == 0
        assert L.hlbm_adjoint_bytes(g.h, 7, every, ctypes.byref(both)) == 0
        assert both.value == snapshots.value + store.value
        n = {"whole": both.value, "before": store.value, "after": store.value}.get(how, 0)
        mem = g.torch.empty(max(n, 1), dtype=g.torch.uint8, device=g.device)
        at = ctypes.c_void_p(mem.data_ptr())
        if how == "whole":
            assert L.hlbm_bind_adjoint(g.h, at, n) == 0
        if how == "before":
            assert L.hlbm_bind_adjoint_store(g.h, at, n) == 0
        if how == "binding":
            g.adjoint_record(7, every)
        elif how not in ("one call", "its own"):
            assert L.hlbm_adjoint_record(g.h, 7, every) == 0
        if how == "after":
            assert L.hlbm_bind_adjoint_store(g.h, at, n) == 0
        if how in ("one call", "its own"):           # record and gradient in one
            if how == "one call":
                s, q0 = g.adjoint(7, every, seed)
            else:
                s, q0 = np.zeros(4), np.zeros((4, 4))
                assert L.hlbm_adjoint(g.h, 7, every, H._dp(seed), H._dp(s), H._dp(q0)) == 0
            r = gradient(g)                          # the window is still there
            assert np.abs(s - r["s"]).max() <= 1e-11 * np.abs(s).max()
            assert np.abs(q0 - r["q0"]).max() <= 1e-11 * np.abs(q0).max()
        else:
            r = g.adjoint_gradient(seed) if how == "binding" else gradient(g)
        end = g.populations()
        if how == "before":                          # the lent block goes away
            assert L.hlbm_bind_adjoint_store(g.h, None, 0) == 0
            mem.fill_(255)
        again = g.adjoint_gradient(seed) if how == "binding" else gradient(g)
        assert np.array_equal(g.populations(), end)
        first = first or r
        for k in first:
            scale = np.abs(first[k]).max()
            assert scale > 0
            for other in (r, again):
                assert np.abs(other[k] - first[k]).max() <= 1e-11 * scale, (how, k)
        g.close()


@pytest.mark.parametrize("kw", [dict(precision=1), dict(periodic_z=0), dict(n_sub=2),
                                dict(balance=2)])
def test_refused_window_takes_no_memory(W, H, kw):
    """A window of a configuration that the adjoint does not support."""
    print("adjoint memory: refused", kw, flush=True)
    g = _sim(W, H, **kw)
    free = _free(g)
    for call in (lambda: g.adjoint_record(40, 40),
                 lambda: g.adjoint(40, 40, np.zeros((4, 3)))):
        with pytest.raises(H.HlbmError) as e:
            call()
        assert e.value.code == E_ARG
        assert free - _free(g) <= 4 * MB
    size = ctypes.c_size_t()
    assert g.L.hlbm_adjoint_bytes(g.h, 40, 40, ctypes.byref(size)) == E_ARG
    g.close()


def test_refused_record_keeps_the_window(W, H):
    """A record refused because a timing window is open leaves the recorded
    window to its gradient."""
    print("adjoint memory: window kept", flush=True)
    g = _sim(W, H, dims=(33, 26, 21))
    seed = np.random.default_rng(5).normal(size=(4, 3))
    g.adjoint_record(4, 2)
    r = g.adjoint_gradient(seed)
    g.timing_begin(4)
    with pytest.raises(H.HlbmError):
        g.adjoint_record(8, 1)
    g.timing_end()
    again = g.adjoint_gradient(seed)
    for k in r:
        assert np.abs(again[k] - r[k]).max() <= 1e-11 * np.abs(r[k]).max(), k
    g.close()


def test_larger_window_replaces_the_smaller(W, H):
    """The memory of the earlier window goes back before a larger one is taken:
    the two never stand side by side, and none stays without a window."""
    print("adjoint memory: larger window", flush=True)
    g = _sim(W, H)
    field = 19 * 8 * 64 ** 3
    cuda = g.torch.cuda
    g.adjoint_record(8, 1)                    # nine snapshots
    _free(g)
    cuda.reset_peak_memory_stats(g.device)
    base = cuda.memory_allocated(g.device) - g.adj_mem.numel()
    g.adjoint_record(10, 1)                   # eleven
    assert cuda.max_memory_allocated(g.device) - base <= 11 * field + 64 * MB
    # and a smaller one does not keep the larger block
    g.adjoint_record(2, 1)
    assert cuda.memory_allocated(g.device) - base <= 3 * field + 64 * MB
    # a restored state drops the window, and its memory with it
    g.set_state(g.get_state())
    assert cuda.memory_allocated(g.device) - base <= MB
    g.close()


def test_lent_memory_has_to_be_aligned(W, H):
    """Aligned for FP64 accesses: else refused; at 8 bytes past a larger
    alignment the same gradient (to the order of its FP64 atomic sums)."""
    print("adjoint memory: alignment", flush=True)
    seed = np.random.default_rng(5).normal(size=(4, 3))
    size = ctypes.c_size_t()
    r = []
    for off in (0, 8):
        g = _sim(W, H, dims=(33, 26, 21))
        assert g.L.hlbm_adjoint_bytes(g.h, 7, 3, ctypes.byref(size)) == 0
        n = size.value
        mem = g.torch.empty(n + 256, dtype=g.torch.uint8, device=g.device)
        for bind in (g.L.hlbm_bind_adjoint_store, g.L.hlbm_bind_adjoint):
            for odd in (1, 4):
                assert bind(g.h, ctypes.c_void_p(mem.data_ptr() + odd), n) == E_ARG
            assert bind(g.h, None, 0) == 0
        assert g.L.hlbm_bind_adjoint(g.h, ctypes.c_void_p(mem.data_ptr() + off), n) == 0
        assert g.L.hlbm_adjoint_record(g.h, 7, 3) == 0
        r.append(g.adjoint_gradient(seed))
        g.close()
    for k in r[0]:
        assert np.abs(r[1][k] - r[0][k]).max() <= 1e-11 * np.abs(r[0][k]).max(), k
