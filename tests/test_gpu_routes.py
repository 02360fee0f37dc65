"""Calls at the sizes where the choice of kernels of an unpinned handle turns: a vector alone and inside a
block, one launch and one launch per geometry, aligned and unaligned data, finite and not.

Equal means equal bits (the same additions in the same order); the oracle checks use the tolerance of the
other operator tests.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from test_gpu_operator import TOL, rel, say, to_dev
from tinygeo import tiny_geometry

pytestmark = pytest.mark.gpu


def hats(geo, n):
    geo.grid = dataclasses.replace(geo.grid, n_hat=n)
    return geo


def same(a, b):
    import torch
    return bool(torch.equal(torch.isnan(a), torch.isnan(b))) and bool(torch.equal(torch.nan_to_num(a, nan=0.5), torch.nan_to_num(b, nan=0.5)))


@pytest.mark.parametrize("dt_obs", [4.0, 2.0])
def test_non_finite_sample_reaches_the_same_nodes_alone_and_in_a_block(gpu_lib, dt_obs):
    """150 vectors on 64 x 64 cells take row pairs, a few take single rows, 12 geometries take either in one
    launch; 16 x 12 cells take the base cells."""
    import torch
    rtt = gpu_lib
    sparse = tiny_geometry(seed=301, rays=(4000, 300, 200), n_r=64, n_phi=64, n_frames=32, dt_obs=dt_obs)
    dense = tiny_geometry(seed=302, rays=(4000, 300, 200), n_r=12, n_phi=16, n_frames=32, dt_obs=dt_obs)
    for name, geos in (("pairs", sparse), ("cells", dense), ("batch", [sparse] * 4 + [dense] * 2)):
        G = rtt.Geometry(geos)
        for bad in (float("nan"), float("inf"), -float("inf")):
            say("case non-finite", name, dt_obs, bad)
            Y, X = torch.randn((150, G.n_rows), device="cuda"), torch.rand((150, G.n_cols), device="cuda")
            Y[:, 1000 * 32 + 7] = bad
            X[:, G.n_cols // 2 + 3] = bad
            y, x = rtt.op_apply(G, X), rtt.op_apply_adjoint(G, Y)
            assert 0 < int((~torch.isfinite(x[0])).sum()) <= 4 * 3   # four corners, at most three hats
            for nv in (1, 2, 9):
                assert same(rtt.op_apply_adjoint(G, Y[:nv].contiguous()), x[:nv]), (name, bad, nv)
                assert same(rtt.op_apply(G, X[:nv].contiguous()), y[:nv]), (name, bad, nv)


@pytest.mark.parametrize("rays", [(300, 40), (900, 90), (4000, 400)])
@pytest.mark.parametrize("frames", [60, 256])
def test_half_step_adjoint_gives_the_same_bits_at_any_alignment(gpu_lib, rays, frames):
    import torch
    rtt = gpu_lib
    geo = tiny_geometry(seed=303, rays=rays, n_r=6, n_phi=9, n_frames=frames, dt_obs=2.0)
    G = rtt.Geometry(geo)
    say("case alignment", rays, frames, rtt.variant_names(True)[G.members[0]["adjoint_variant"]])
    Y = to_dev(np.random.default_rng(7).standard_normal((5, G.n_rows)))
    x = rtt.op_apply_adjoint(G, Y)
    assert rel(x.cpu().numpy(), oracle.adjoint(geo, Y.double().cpu().numpy())) <= TOL
    buf = torch.full((5 * G.n_rows + 8,), float("nan"), device="cuda")
    for pad in (1, 2, 3):
        off = buf[pad:pad + 5 * G.n_rows].view(5, G.n_rows)
        off.copy_(Y)
        assert torch.equal(rtt.op_apply_adjoint(G, off), x), pad
        assert torch.equal(rtt.op_apply_adjoint(G, off[:1]), x[:1]), pad
        buf.fill_(float("nan"))


@pytest.mark.parametrize("dt_obs", [4.0, 2.0])
@pytest.mark.parametrize("n_hat,frames,rays", [(128, (96, 97, 134), 900), (170, (150, 192, 301), 900), (200, (134, 192, 150), 12000)])
def test_forward_gives_the_same_bits_by_every_lean_route(gpu_lib, dt_obs, n_hat, frames, rays):
    """The variants that an unpinned handle chooses from, alone and in one launch, at any start of the block."""
    import torch
    rtt = gpu_lib
    geos = [hats(tiny_geometry(seed=305 + i, rays=(rays, rays // 8, 80), n_r=6, n_phi=9, n_frames=f, dt_obs=dt_obs), n_hat)
            for i, f in enumerate(frames)]
    G = rtt.Geometry(geos)
    X = to_dev(np.random.default_rng(8).random((5, G.n_cols)))
    y = rtt.op_apply(G, X)
    for geo, m in zip(geos, G.members):
        cs, rs = slice(m["col_offset"], m["col_offset"] + m["n_cols"]), slice(m["row_offset"], m["row_offset"] + m["n_rows"])
        assert rel(y[0, rs].cpu().numpy(), oracle.forward(geo, X[0, cs].double().cpu().numpy())) <= TOL
    buf = torch.empty((5 * G.n_rows + 8,), device="cuda")
    names = ["lean4", "lean8", "lean4r"] + (["lean4q"] if n_hat % 4 == 0 else []) + (["abs4", "abs8", "abs4r"] if n_hat <= 128 else [])
    for name in [None] + names:
        if name:
            G.set_variant(apply=rtt.variant_names(False).index(name))
        for mode in (0, 1, 2):
            G.set_batch_mode(mode, mode)
            for pad in (0, 1, 2):
                say("case forward bits", dt_obs, n_hat, name, mode, pad)
                for nv in (1, 5):
                    out = buf[pad:pad + nv * G.n_rows].view(nv, G.n_rows)
                    rtt.op_apply(G, X[:nv], y=out)
                    assert torch.equal(out, y[:nv]), (name, mode, pad, nv)


def test_host_cost_of_a_call_grows_with_the_members_not_their_square(gpu_lib):
    """4096 members, the most a handle takes.  Linear host work is well below a millisecond; a pass over all
    members for each of them was 16."""
    import time
    rtt = gpu_lib
    G = rtt.Geometry([tiny_geometry(seed=306, rays=(6, 3), n_r=4, n_phi=6)] * 4096)
    best = 1.0
    for _ in range(5):
        t0 = time.perf_counter()
        assert G.launches[1] == 4096 // 16
        best = min(best, time.perf_counter() - t0)
    say("case host cost", best)
    assert best < 3e-3


def kernel_nodes(fn):
    """Kernels that one call launches, counted in a captured graph."""
    import ctypes
    import torch
    fn()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        fn()
    n = ctypes.c_size_t()
    hip = ctypes.CDLL("libamdhip64.so")
    hip.hipGraphGetNodes.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.POINTER(ctypes.c_size_t)]
    assert hip.hipGraphGetNodes(graph.raw_cuda_graph(), None, ctypes.byref(n)) == 0
    return n.value


def launches_and_bits(rtt, geos, nvecs, default):
    """Launches of A at every mode against `default` (those of a handle whose mode was never set), the bits of
    each against the first, and the oracle's values."""
    import torch
    G = rtt.Geometry(geos)
    X = to_dev(np.random.default_rng(9).random((max(nvecs), G.n_cols)))
    Y = torch.empty((max(nvecs), G.n_rows), device="cuda")
    y = rtt.op_apply(G, X)
    for geo, m in zip(geos, G.members):
        cs, rs = slice(m["col_offset"], m["col_offset"] + m["n_cols"]), slice(m["row_offset"], m["row_offset"] + m["n_rows"])
        assert rel(y[0, rs].cpu().numpy(), oracle.forward(geo, X[0, cs].double().cpu().numpy())) <= TOL
    for mode in (None, 0, 1, 2):
        if mode is not None:
            G.set_batch_mode(apply=mode)
        for nv in nvecs:
            want = default if mode is None else len(geos) if mode == 0 else (len(geos) + 15) // 16
            n = kernel_nodes(lambda: rtt.op_apply(G, X[:nv], y=Y[:nv]))
            say("case launches", len(geos), mode, nv, n)
            assert n == want, (mode, nv)
            assert torch.equal(Y[:nv], y[:nv]), (mode, nv)


def test_small_geometries_go_in_one_launch_at_any_number_of_vectors(gpu_lib):
    geos = [tiny_geometry(seed=310 + i, rays=(90 + 30 * i, 12, 8), n_r=6, n_phi=9, n_frames=32 + 3 * i) for i in range(3)]
    launches_and_bits(gpu_lib, [geos[i % 3] for i in range(18)], (1, 2, 3, 9), 2)


@pytest.mark.parametrize("dt_obs", [4.0, 2.0])
def test_geometries_of_few_and_of_many_hats_share_a_launch(gpu_lib, dt_obs):
    geos = [hats(tiny_geometry(seed=313 + i, rays=(90, 12, 8), n_r=6, n_phi=9, n_frames=f, dt_obs=dt_obs), n)
            for i, (f, n) in enumerate(((40, 60), (151, 170), (134, 128), (192, 129)))]
    launches_and_bits(gpu_lib, geos, (1, 3), 1)


def test_a_launch_mode_that_was_set_holds_for_large_geometries(gpu_lib):
    """8 vectors of about 8 MB a geometry go by one launch a geometry unless the caller asked for one."""
    geos = [hats(tiny_geometry(seed=317 + i, rays=(12000, 1500, 1000), n_r=16, n_phi=24, n_frames=134 + i), 100) for i in range(2)]
    launches_and_bits(gpu_lib, geos, (8,), 2)


@pytest.mark.parametrize("name,geos,blocks", [
    # one geometry, row sweep: one, two (2 .. 7), four vectors a wave on 64 rows (8 .. 31), row pairs from 8192 waves (128)
    ("sweep", lambda: [tiny_geometry(seed=320, rays=(3000, 300, 200), n_r=64, n_phi=64, n_frames=33)], (1, 2, 7, 8, 31, 32, 127, 129)),
    ("sweep half steps", lambda: [tiny_geometry(seed=321, rays=(3000, 300, 200), n_r=64, n_phi=64, n_frames=34, dt_obs=2.0)], (1, 2, 8, 32, 129)),
    # half steps, more than 128 hats: records in row order up to 128 MiB of coefficients (60 vectors of 2.2 MB)
    ("columns", lambda: [hats(tiny_geometry(seed=322, rays=(900, 90, 60), n_r=64, n_phi=64, n_frames=40, dt_obs=2.0), 136)], (1, 59, 60, 61)),
    # several in one launch: row pairs from 2048 waves of short members (16 vectors), from 4096 of longer ones (31)
    ("short members", lambda: [tiny_geometry(seed=323 + i, rays=(3000, 300, 200), n_r=32, n_phi=64, n_frames=33 + i) for i in range(4)], (1, 2, 15, 16, 17)),
    ("longer members", lambda: [tiny_geometry(seed=327 + i, rays=(9000, 300, 200), n_r=32, n_phi=64, n_frames=33 + i) for i in range(4)], (1, 29, 30, 31, 32, 33)),
])
def test_blocks_on_both_sides_of_each_line_of_the_choice(gpu_lib, name, geos, blocks):
    import torch
    rtt = gpu_lib
    geos = geos()
    G = rtt.Geometry(geos)
    nv = max(blocks) + 1
    gen = torch.Generator("cuda").manual_seed(11)
    X, Y = torch.rand((nv, G.n_cols), device="cuda", generator=gen), torch.randn((nv, G.n_rows), device="cuda", generator=gen)
    y, x = rtt.op_apply(G, X), rtt.op_apply_adjoint(G, Y)
    for geo, m in zip(geos, G.members):
        cs, rs = slice(m["col_offset"], m["col_offset"] + m["n_cols"]), slice(m["row_offset"], m["row_offset"] + m["n_rows"])
        assert rel(y[-1, rs].cpu().numpy(), oracle.forward(geo, X[-1, cs].double().cpu().numpy())) <= TOL
        assert rel(x[-1, cs].cpu().numpy(), oracle.adjoint(geo, Y[-1, rs].double().cpu().numpy())) <= TOL
    for n in blocks:
        say("case lines", name, n)
        assert torch.equal(rtt.op_apply(G, X[:n]), y[:n]), n
        assert torch.equal(rtt.op_apply_adjoint(G, Y[:n]), x[:n]), n


@pytest.mark.parametrize("n_hat", [8191, 8192, 8193])
@pytest.mark.parametrize("late", [False, True])
def test_age_windows_at_the_most_hats_they_take(gpu_lib, n_hat, late):
    """8192 FP64 hats fill the 64 KB of LDS of a table's workgroup; one more goes by probes.  FP32 weights and
    fractions enter a square, as in the other test of the windows: 2e-6 of the order's largest energy."""
    rtt = gpu_lib
    geo = hats(tiny_geometry(seed=331, rays=(50, 20), n_r=3, n_phi=4, n_frames=9), n_hat)
    if late:   # the frames' origins at the other end of the hats
        geo.grid = dataclasses.replace(geo.grid, s0=geo.grid.s0 - 4.0 * (n_hat - 12))
    G = rtt.Geometry(geo)
    ages = np.linspace(-8.0, 70.0, 9)
    say("case age hats", n_hat, late)
    E = rtt.age_information(G, ages, h=3.0)
    Y = oracle.forward(geo, oracle.age_probes(geo.grid, ages, 3.0)).reshape(9, -1)
    at = 0
    for n, m in enumerate(geo.maps):
        end = at + m.n_rays * 9
        want = np.einsum("ar,ar->a", Y[:, at:end], Y[:, at:end])
        assert np.max(want) > 0 and np.max(np.abs(E[:, 0, n] - want)) <= 2e-6 * np.max(want), n
        at = end
