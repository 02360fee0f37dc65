"""The base-cell adjoint at the edges of its tiles, and the choice of kernels for unpinned handles.

Tolerance: relative L2 error <= 1e-5 against the FP64 oracle on the same FP32 inputs (sums of at most
about 1500 FP32 terms here: sqrt(1500) 2^-24, a few times).
"""
import numpy as np
import pytest

import oracle
from test_gpu_operator import TOL, rel, say, to_dev
from tinygeo import tiny_geometry

pytestmark = pytest.mark.gpu

# rays a cell below 20, up to 80 and above choose 1, 2 and 4 waves per cell (7 or 15, 3, 3 columns per
# workgroup); hats 62 .. 64, 126 .. 128, 190 .. 192 and 255, 256 sit at the edges of 1 to 4 slots with and
# without halo lanes; the last row of an odd n_r has no rays of its own
CELLS = {
    "one_wave_ragged": dict(rays=(500, 90, 60), n_r=6, n_phi=15, n_frames=70),
    "one_wave_7_columns": dict(rays=(300,), n_r=5, n_phi=7, n_frames=58),
    "two_rows_8_columns": dict(rays=(100, 20), n_r=2, n_phi=8, n_frames=33),
    "one_column": dict(rays=(40, 10), n_r=5, n_phi=1, n_frames=17),
    "two_waves": dict(rays=(900, 200, 150), n_r=5, n_phi=10, n_frames=123),
    "four_waves": dict(rays=(900, 200, 150), n_r=3, n_phi=4, n_frames=60),
    "empty_cells": dict(rays=(30,), n_r=9, n_phi=12, n_frames=64),
    "half_steps": dict(rays=(700, 80, 60), n_r=6, n_phi=9, n_frames=90, dt_obs=2.0),
    "half_steps_two_waves": dict(rays=(900, 90), n_r=4, n_phi=9, n_frames=256, dt_obs=2.0),
    "half_steps_odd_rows": dict(rays=(300, 40), n_r=5, n_phi=8, n_frames=61, dt_obs=2.0),
}
HATS = [62, 63, 64, 126, 127, 128, 190, 191, 192, 255, 256]


def check_cells(rtt, geo, seed):
    import torch
    G = rtt.Geometry(geo)
    G.set_variant(adjoint=rtt.variant_names(True).index("visitc"))
    Y = to_dev(np.random.default_rng(seed).standard_normal((3, geo.n_rows)))
    X = rtt.op_apply_adjoint(G, Y, x=torch.full((3, G.n_cols), 7.0, device="cuda"))
    ref = oracle.adjoint(geo, Y.double().cpu().numpy())
    assert rel(X.cpu().numpy(), ref) <= TOL
    for b in range(3):   # one vector per wave gives the bits of two per wave
        assert torch.equal(X[b], rtt.op_apply_adjoint(G, Y[b].contiguous()))
    m = rtt.op_apply_adjoint(G, Y, order_mask=1).cpu().numpy()
    assert rel(m, oracle.adjoint(geo, Y.double().cpu().numpy(), order_mask=1)) <= TOL


@pytest.mark.parametrize("name", list(CELLS))
def test_base_cell_adjoint_matches_oracle(gpu_lib, name):
    say("case cells", name)
    check_cells(gpu_lib, tiny_geometry(seed=201, **CELLS[name]), 1)


@pytest.mark.parametrize("dt_obs", [4.0, 2.0])
@pytest.mark.parametrize("hats", HATS)
def test_base_cell_adjoint_at_the_edges_of_its_hat_slots(gpu_lib, hats, dt_obs):
    from synth import Grid
    import dataclasses
    geo = tiny_geometry(seed=202, rays=(60, 20), n_r=4, n_phi=6, n_frames=hats - 8, dt_obs=dt_obs)
    geo.grid = dataclasses.replace(geo.grid, n_hat=hats)   # the first or last frames may lie outside the hats
    assert isinstance(geo.grid, Grid)
    say("case cells hats", hats, dt_obs)
    check_cells(gpu_lib, geo, 2)


@pytest.mark.parametrize("rays,frames,n_hat", [((30, 8, 4), 40, 60), ((300, 60, 50), 134, 128), ((200, 30, 20), 150, 165),
                                               ((40, 9, 6), 192, 210)])
def test_unpinned_handle_gives_a_vector_the_same_bits_alone_and_in_a_block(gpu_lib, rays, frames, n_hat):
    import dataclasses
    import torch
    rtt = gpu_lib
    geo = tiny_geometry(seed=203, rays=rays, n_r=6, n_phi=9, n_frames=frames)
    geo.grid = dataclasses.replace(geo.grid, n_hat=n_hat)
    say("case unpinned", rays, frames, n_hat)
    G = rtt.Geometry(geo)
    rng = np.random.default_rng(3)
    X, Y = to_dev(rng.random((9, G.n_cols))), to_dev(rng.standard_normal((9, G.n_rows)))
    y, x = rtt.op_apply(G, X), rtt.op_apply_adjoint(G, Y)
    assert rel(y.cpu().numpy(), oracle.forward(geo, X.double().cpu().numpy())) <= TOL
    assert rel(x.cpu().numpy(), oracle.adjoint(geo, Y.double().cpu().numpy())) <= TOL
    for nv in (1, 2, 3, 8):
        assert torch.equal(rtt.op_apply(G, X[:nv]), y[:nv]), nv
        assert torch.equal(rtt.op_apply_adjoint(G, Y[:nv]), x[:nv]), nv


def test_unpinned_batch_gives_the_same_bits_in_every_launch_mode_and_block(gpu_lib):
    import torch
    rtt = gpu_lib
    geos = [tiny_geometry(seed=210 + i, rays=(90 + 200 * i, 12, 8), n_r=6, n_phi=9, n_frames=f)
            for i, f in enumerate((40, 134, 64, 151))]
    import dataclasses
    for g in geos:
        g.grid = dataclasses.replace(g.grid, n_hat=100, s0=-64.0)
    G = rtt.Geometry(geos)
    say("case unpinned batch", [g.n_rays for g in geos])
    rng = np.random.default_rng(4)
    X, Y = to_dev(rng.random((9, G.n_cols))), to_dev(rng.standard_normal((9, G.n_rows)))
    y, x = rtt.op_apply(G, X), rtt.op_apply_adjoint(G, Y)
    for geo, m in zip(geos, G.members):
        cs = slice(m["col_offset"], m["col_offset"] + m["n_cols"])
        rs = slice(m["row_offset"], m["row_offset"] + m["n_rows"])
        assert rel(y[:, rs].cpu().numpy(), oracle.forward(geo, X[:, cs].double().cpu().numpy())) <= TOL
        assert rel(x[:, cs].cpu().numpy(), oracle.adjoint(geo, Y[:, rs].double().cpu().numpy())) <= TOL
    for mode in (0, 1, 2):
        G.set_batch_mode(mode, mode)
        for nv in (1, 2, 3, 9):
            assert torch.equal(rtt.op_apply(G, X[:nv].contiguous()), y[:nv]), (mode, nv)
            assert torch.equal(rtt.op_apply_adjoint(G, Y[:nv].contiguous()), x[:nv]), (mode, nv)


@pytest.mark.parametrize("frames", [1, 2, 3, 4, 5, 7, 63, 125, 126, 127, 128, 129, 131, 259])
def test_forward_of_absolute_hats_at_every_row_length(gpu_lib, frames):
    """Four frames a store at any row start: rows shorter than a store, ragged ends, one and two more passes,
    and nothing written beside the block."""
    import dataclasses
    import torch
    rtt = gpu_lib
    say("case row length", frames)
    geo = tiny_geometry(seed=204, rays=(37, 6), n_r=4, n_phi=6, n_frames=frames)
    geo.grid = dataclasses.replace(geo.grid, n_hat=min(geo.grid.n_hat, 128))   # later frames lie outside the hats
    G = rtt.Geometry(geo)
    G.set_variant(apply=rtt.variant_names(False).index("abs4"))
    X = to_dev(np.random.default_rng(5).standard_normal((2, G.n_cols)))
    ref = oracle.forward(geo, X.double().cpu().numpy())
    for pad in (0, 1, 2, 3):   # every phase of the block's start
        buf = torch.full((2 * G.n_rows + 16,), 7.0, device="cuda")
        out = buf[4 + pad:4 + pad + 2 * G.n_rows].view(2, G.n_rows)
        rtt.op_apply(G, X, y=out)
        assert rel(out.cpu().numpy(), ref) <= TOL
        assert bool((buf[:4 + pad] == 7.0).all()) and bool((buf[4 + pad + 2 * G.n_rows:] == 7.0).all())


@pytest.mark.parametrize("name", ["one_wave_ragged", "one_wave_7_columns", "two_rows_8_columns", "one_column",
                                  "four_waves", "empty_cells", "half_steps", "half_steps_odd_rows"])
def test_ridge_by_shares_of_the_cell_rows_matches_oracle(gpu_lib, name):
    """The solver's one-launch adjoint (even and odd cell rows apart) on a handle pinned to the base cells,
    and the two launches of a handle with another kernel, after the same iterations.  lambda = |A|^2: a
    condition of 2, so three iterations carry the FP32 errors of six products, within TOL."""
    rtt = gpu_lib
    say("case ridge shares", name)
    geo = tiny_geometry(seed=203, **CELLS[name])
    rng = np.random.default_rng(4)
    v = rng.standard_normal(geo.grid.n_cols)
    for _ in range(8):
        v = oracle.adjoint(geo, oracle.forward(geo, v / np.linalg.norm(v)))
    lam = float(np.float32(np.linalg.norm(v)))
    Y = to_dev(rng.standard_normal((3, geo.n_rows)))
    y = Y.double().cpu().numpy()
    for mask in (0, 1):
        for kernel in ("visitc", "visitd"):
            G = rtt.Geometry(geo)
            G.set_variant(adjoint=rtt.variant_names(True).index(kernel))
            X, _ = rtt.ridge_solve(G, Y, lam, tol=1e-12, maxit=3, async_mode=True, order_mask=mask)
            for b in range(3):
                want = three_iterations(geo, y[b], lam, mask or None)
                assert rel(X[b].cpu().numpy(), want) <= TOL, (kernel, mask, b)


def three_iterations(geo, y, lam, mask):
    A = lambda x: oracle.forward(geo, x, order_mask=mask)  # noqa: E731
    At = lambda q: oracle.adjoint(geo, q, order_mask=mask)  # noqa: E731
    r = At(y)
    x, p, rr = np.zeros_like(r), r.copy(), r @ r
    for _ in range(3):
        Ap = At(A(p)) + lam * p
        a = rr / (p @ Ap)
        x, r = x + a * p, r - a * Ap
        new = r @ r
        p, rr = r + new / rr * p, new
    return x
