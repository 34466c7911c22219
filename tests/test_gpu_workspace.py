"""Workspace of the library's calls: taken from PyTorch's caching allocator, given
back when a call ends, bounded where the library keeps it itself."""
import ctypes
import gc

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hub():
    import torch
    import paper_1307_7542_amd as h
    h.lib()
    torch.cuda.set_device(0)
    return h


@pytest.fixture
def allocator(hub):
    """Sets another allocator for one test."""
    keep = []

    def use(alloc, release, idle, trim):
        f = (ctypes.CFUNCTYPE(ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int32, ctypes.c_void_p)(alloc),
             ctypes.CFUNCTYPE(None, ctypes.c_void_p)(release),
             ctypes.CFUNCTYPE(ctypes.c_size_t, ctypes.c_int32)(idle), ctypes.CFUNCTYPE(None)(trim))
        keep.append(f)
        assert hub.lib().hub_set_allocator(*f) == 0

    yield use
    assert hub.lib().hub_set_allocator(hub._ws_alloc, hub._ws_release, hub._ws_idle,
                                         hub._ws_trim) == 0


MB = 1 << 20


def _free(torch):
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def test_memory_comes_back_to_the_program(hub):
    """After a solve PyTorch can have the memory again while the sector lives, but
    for what the library may keep."""
    import torch
    s = hub.Sector(W.ring(12, U=4.0, n_up=6, n_dn=6))   # 6.8 MB a vector, about 100 of them kept
    s.ground_state(want_vector=False)                   # tuned, code loaded
    before = _free(torch)
    gs = s.ground_state()
    assert gs.info["iters"] * 8 * s.dim > 400 * MB
    del gs
    assert before - _free(torch) <= 256 * MB
    s.close()


def test_energy_gradients_reuse_the_memory(hub):
    """A loop of energies with gradients, each with a sector of its own, takes its
    Lanczos vectors from PyTorch's pool and asks the driver for nothing new."""
    import torch
    from paper_1307_7542_amd import autograd
    m = W.ring(12, U=4.0, n_up=6, n_dn=6)

    def call():
        t, u, e = (torch.tensor(v, dtype=torch.float64, requires_grad=True) for v in (m.t, m.U, m.eps))
        autograd.ground_energy(t, u, e, n_sites=m.n_sites, bonds=m.bonds, n_up=6, n_dn=6).backward()
        return t.grad

    first = call()
    call()
    torch.cuda.reset_peak_memory_stats()
    asked = torch.cuda.memory_stats()["num_device_alloc"]
    held = torch.cuda.memory_allocated()
    for _ in range(6):
        assert torch.equal(call(), first)
    assert torch.cuda.memory_stats()["num_device_alloc"] == asked
    assert torch.cuda.memory_allocated() == held
    assert torch.cuda.max_memory_allocated() - held > 64 * 8 * 924 * 924   # the kept vectors are in its books


def test_idle_blocks_are_bounded_and_given_back(hub):
    import torch
    for M, n in ((8, 4), (10, 5), (11, 5), (12, 6), (13, 6)):
        with hub.Sector(W.ring(M, U=4.0, n_up=n, n_dn=n)) as s:
            s.ground_state(max_iter=40, allow_not_converged=True)
            s.ground_state(dtype=hub.F32, reorth=1, max_iter=40, allow_not_converged=True)
    before = torch.cuda.mem_get_info()[0]
    n = hub.workspace_trim()
    assert 0 < n <= 256 * MB
    assert hub.workspace_trim() == 0
    assert torch.cuda.mem_get_info()[0] - before >= n // 2   # (the driver hands out whole pages)


def test_blocks_move_between_streams(hub):
    """Blocks of a solve on one stream serve the next one on another."""
    import torch
    s = hub.Sector(W.ring(12, U=4.0, n_up=6, n_dn=6))
    a = s.ground_state()
    st = torch.cuda.Stream()
    st.wait_stream(torch.cuda.current_stream())
    for _ in range(3):
        with torch.cuda.stream(st):
            b = s.ground_state()
        st.synchronize()
        c = s.ground_state()
        assert a.e0 == b.e0 == c.e0 and torch.equal(a.psi, b.psi) and torch.equal(a.psi, c.psi)
    s.close()


def test_refused_blocks(hub, allocator):
    """An allocator that refuses the blocks of kept vectors leaves a solve without
    them, not without a result; what a solve needs it then takes from the driver, and
    trim is called before a solve is found too large."""
    import torch
    s = hub.Sector(W.ring(12, U=4.0, n_up=6, n_dn=6))
    big = hub.Sector(W.ring(14, U=4.0, n_up=7, n_dn=7))  # 94 MB a vector
    want, bigwant = s.ground_state(), big.ground_state(max_iter=30, allow_not_converged=True)
    calls = {"alloc": 0, "trim": 0, "idle": 0}

    def alloc(size, device, stream):
        calls["alloc"] += 1
        return torch.cuda.caching_allocator_alloc(size, device, stream or 0) if size < 64 * MB else None

    def trim():
        calls["trim"] += 1

    allocator(alloc, torch.cuda.caching_allocator_delete, lambda d: calls["idle"], trim)
    got = s.ground_state()
    assert calls["alloc"] > 0 and got.info["iters"] == want.info["iters"] and got.e0 == want.e0
    # both sum m terms of at most |psi| in FP64, in the same order
    assert float((got.psi - want.psi).abs().max()) <= 4 * got.info["iters"] * 2.0 ** -53
    got = big.ground_state(max_iter=30, allow_not_converged=True)
    assert got.e0 == bigwant.e0 and float((got.psi - bigwant.psi).abs().max()) <= 4 * 30 * 2.0 ** -53
    # 9.4 TB of vectors: refused; the allocator trims only where that would be enough
    for idle, trims in ((0, 0), (1 << 44, 1)):
        calls["idle"], calls["trim"] = idle, 0
        with pytest.raises(hub.HubError) as e:
            big.ground_state(reorth=1, max_iter=100000)
        assert e.value.status == 3 and calls["trim"] == trims
    s.close()
    big.close()


def test_batch_blocks_outlive_its_stream(hub):
    """A batched solve works on a stream of its own; its blocks return to PyTorch's
    pool for the caller's stream and serve the next solve."""
    import torch
    secs = [hub.Sector(W.ring(12, U=1.0 + p, n_up=6, n_dn=6)) for p in range(6)]   # 41 MB a vector
    b = hub.Batch(secs)
    e0, _, psi, _ = b.ground_state(want_vector=True)
    b.ground_state(want_vector=True)
    asked = torch.cuda.memory_stats()["num_device_alloc"]
    for _ in range(4):
        e1, _, psi1, _ = b.ground_state(want_vector=True)
        assert np.array_equal(e0, e1) and torch.equal(psi, psi1)
    assert torch.cuda.memory_stats()["num_device_alloc"] == asked
    b.close()
    for s in secs:
        s.close()


def test_solves_in_threads_share_the_pool(hub):
    """Solves in several threads, each on a stream of its own, beside the program's
    own allocations."""
    import threading
    import torch
    secs = [hub.Sector(W.ring(12, U=2.0 + p, n_up=6, n_dn=6)) for p in range(4)]
    want = [s.ground_state() for s in secs]
    torch.cuda.synchronize()
    bad = []

    def work(p):
        try:
            torch.cuda.set_device(0)
            with torch.cuda.stream(torch.cuda.Stream()):
                for i in range(3):
                    junk = torch.full((secs[p].dim * (1 + i),), float("nan"), dtype=torch.float64, device="cuda")
                    got = secs[p].ground_state()
                    del junk
                    torch.cuda.current_stream().synchronize()
                    if got.e0 != want[p].e0 or not torch.equal(got.psi, want[p].psi):
                        bad.append((p, i))
        except Exception as e:  # reported below, in the main thread
            bad.append((p, repr(e)))

    threads = [threading.Thread(target=work, args=(p,)) for p in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    for s in secs:
        s.close()


def test_limits_of_pytorch_do_not_bind_the_library(hub):
    """A program that keeps PyTorch to a small part of the device can still solve what
    the device holds: three vectors of 94 MB beside a limit of 300 MB."""
    import torch
    _free(torch)
    total = torch.cuda.mem_get_info()[1]
    s = hub.Sector(W.ring(14, U=4.0, n_up=7, n_dn=7))
    want = s.ground_state(want_vector=False, max_iter=30, allow_not_converged=True)
    _free(torch)
    try:
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + 300 * MB) / total)
        got = s.ground_state(max_iter=30, allow_not_converged=True)
        assert got.e0 == want.e0
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    s.close()
