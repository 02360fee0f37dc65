"""The pool of idle scratch: what stays in it, how much, and who gets it back."""
import gc

import numpy as np
import pytest

from test_gpu_operator import say
from tinygeo import tiny_geometry

pytestmark = pytest.mark.gpu
GIB = 1 << 30


def free_bytes():
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def large_geometry():
    """About 3.3M data rows: the blocks of a rank-256 rSVD (288 vectors) are 3.8 GB each."""
    return tiny_geometry(seed=330, rays=(20000, 3000, 2800), n_r=16, n_phi=24, n_frames=128)


def test_idle_scratch_is_bounded_and_given_back_on_request(gpu_lib):
    rtt = gpu_lib
    G = rtt.Geometry(large_geometry())
    rtt.scratch_trim()
    before = free_bytes()
    rtt.rsvd(G, k=256, p=32, q=0)      # Y and Y2 alone are 7.6 GB; the pool keeps what fits its bound
    held = before - free_bytes()
    say("case idle scratch", held)
    assert GIB < held <= 8 * GIB
    assert rtt.scratch_trim() >= held - (64 << 20)
    assert rtt.scratch_trim() == 0
    assert before - free_bytes() <= 64 << 20
    # a block that does not fit beside what is idle sends the longest idle ones away
    for k in (64, 128, 192, 224, 256):
        rtt.rsvd(G, k=k, p=32, q=0)
        assert before - free_bytes() <= 8 * GIB, k
    rtt.scratch_trim()


def test_idle_scratch_returns_with_the_last_handle(gpu_lib):
    rtt = gpu_lib
    gc.collect()
    alive = [o for o in gc.get_objects() if type(o) is rtt.Geometry and getattr(o, "_h", None) is not None]
    if alive:
        pytest.skip("%d handles of other tests are alive" % len(alive))
    G, H = rtt.Geometry(large_geometry()), rtt.Geometry(tiny_geometry(seed=331))
    rtt.scratch_trim()
    before = free_bytes()
    rtt.rsvd(G, k=64, p=32, q=0)
    held = before - free_bytes()
    H.free()
    assert held > GIB and before - free_bytes() >= held - (64 << 20)   # G is alive
    G.free()
    say("case last handle", held)
    assert free_bytes() >= before
    assert rtt.scratch_trim() == 0


def fill_device(leave):
    """Tensors that leave about `leave` bytes of the device free."""
    import torch
    kept = []
    for piece in (8 * GIB, GIB, 64 << 20):
        while torch.cuda.mem_get_info()[0] > leave + piece:
            kept.append(torch.empty(piece, dtype=torch.uint8, device="cuda"))
    return kept


@pytest.mark.parametrize("what", ["geometry", "synthesis"])
def test_a_handle_that_needs_the_idle_memory_gets_it(gpu_lib, what):
    """Drivers freed their scratch on return before it was pooled: what fitted beside them then must fit now."""
    rtt = gpu_lib
    G = rtt.Geometry(large_geometry())
    S = rtt.Geometry(tiny_geometry(seed=332, n_r=64, n_phi=64, n_frames=240))
    big = tiny_geometry(seed=333, rays=(3000000,), n_r=64, n_phi=64, n_frames=1)     # about 1 GB of tables
    rtt.scratch_trim()
    rtt.rsvd(G, k=256, p=32, q=0)
    kept = fill_device(384 << 20)
    say("case full device", what, len(kept), S.n_cols)
    try:
        if what == "geometry":
            made = rtt.Geometry(big)
            assert made.table_bytes > (384 << 20) + (64 << 20)
        else:
            made = rtt.Synthesis(S, n_radial=8, m_max=4, n_temporal=8)                # 576 columns of Q, 2.4 GB
        made.free()
    finally:
        del kept
        rtt.scratch_trim()
        free_bytes()       # torch's cache goes back to the device too


def test_scratch_that_a_handle_outgrows_is_not_handed_to_other_calls(gpu_lib):
    """A graph captured from a call on the handle still names the old buffers: no other driver may get them."""
    import torch
    rtt = gpu_lib
    geo = tiny_geometry(seed=334, rays=(900, 90, 60), n_r=12, n_phi=16, n_frames=64)
    G = rtt.Geometry(geo)
    sv = rtt.rsvd(G, k=48, p=16, q=0, seed=1)
    M = rtt.Mixer(G, "total_flux")
    S = rtt.Synthesis(G, n_radial=4, m_max=3, n_temporal=8)
    calls = {
        "ridge": lambda n: rtt.ridge_solve(G, torch.ones((n, G.n_rows), device="cuda"), 1.0, maxit=2, async_mode=True),
        "tsvd": lambda n: rtt.tsvd_solve(G, sv, torch.ones((n, G.n_rows), device="cuda"), t=40),
        "mixer": lambda n: rtt.mix_apply(M, torch.ones((n, G.n_rows), device="cuda")),
        "synthesis": lambda n: S.project(torch.ones((n, G.n_cols), device="cuda")),
    }
    for name, call in calls.items():
        call(3)
        rtt.scratch_trim()
        call(40)
        call(90)
        torch.cuda.synchronize()
        say("case outgrown", name)
        assert rtt.scratch_trim() == 0, name


@pytest.mark.parametrize("rays,blocks", [((300, 40, 20), 3), ((4000, 400, 300), 4)])
def test_ridge_keeps_a_second_share_of_the_adjoint_only_where_it_uses_it(gpu_lib, rays, blocks):
    """Scratch of a solve: the residual, the direction and A^T A p, a data block, and a second share of A^T A p
    where the adjoint goes by base cells (from 4.5 rays a cell on)."""
    import torch
    rtt = gpu_lib
    geo = tiny_geometry(seed=335, rays=rays, n_r=16, n_phi=24, n_frames=64)
    G = rtt.Geometry(geo)
    nrhs = 512
    Y = torch.ones((nrhs, G.n_rows), device="cuda")
    rtt.scratch_trim()
    rtt.ridge_solve(G, Y, 1.0, maxit=1, raise_on_noconv=False)
    used = rtt.scratch_trim()
    say("case ridge scratch", used, 4 * nrhs * G.n_cols)
    assert blocks * 4 * nrhs * G.n_cols <= used - 4 * nrhs * G.n_rows < (blocks + 0.5) * 4 * nrhs * G.n_cols
