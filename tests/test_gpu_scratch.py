"""Scratch kept between calls: what a call leaves in a block must not reach the next one."""
import gc
import threading

import numpy as np
import pytest

import oracle
from test_gpu_operator import say, to_dev
from tinygeo import tiny_geometry

pytestmark = pytest.mark.gpu


def poison(rtt, n_floats=1 << 22):
    """A driver call whose scratch is full of NaN when it is given back."""
    import torch
    geo = tiny_geometry(seed=230, rays=(400, 60, 50), n_r=6, n_phi=9, n_frames=64)
    G = rtt.Geometry(geo)
    Y = torch.full((max(1, n_floats // geo.n_rows), geo.n_rows), float("nan"), device="cuda")
    rtt.ridge_solve(G, Y, 1e-3, maxit=2, raise_on_noconv=False)
    om = torch.full((64, G.n_cols), float("nan"), device="cuda")
    rtt.rsvd(G, k=32, p=32, q=1, omega=om)


def test_masked_lanczos_on_reused_scratch_matches_oracle(gpu_lib):
    rtt = gpu_lib
    geo = tiny_geometry(seed=231, rays=(300, 50, 40), n_r=6, n_phi=9, n_frames=32)
    G = rtt.Geometry(geo)
    om = np.random.default_rng(5).standard_normal((32, G.n_cols)).astype(np.float32)
    say("case masked lanczos", G.n_rows, G.n_cols)
    for mask in (0b001, 0b110, 0):
        poison(rtt)
        s, _, _ = oracle.block_lanczos(geo, om.astype(np.float64), 4, order_mask=mask or None)
        sv = rtt.rsvd(G, k=16, method="lanczos", block=32, steps=4, omega=to_dev(om), order_mask=mask)
        # singular values to 1e-4 relative, as for the other spectral drivers
        assert np.max(np.abs(sv.sigma - s[:16]) / s[:16]) <= 1e-4, mask


def test_drivers_on_two_threads_and_streams_keep_their_scratch_apart(gpu_lib):
    import torch
    rtt = gpu_lib
    geos = [tiny_geometry(seed=232 + i, rays=(300, 50, 40), n_r=6, n_phi=9, n_frames=32) for i in range(2)]
    Gs = [rtt.Geometry(g) for g in geos]
    om = [to_dev(np.random.default_rng(6 + i).standard_normal((48, Gs[i].n_cols))) for i in range(2)]
    ages = 4.0 * np.arange(20)
    want = [(rtt.rsvd(Gs[i], k=32, p=16, q=1, omega=om[i]).sigma, rtt.age_information(Gs[i], ages)) for i in range(2)]
    torch.cuda.synchronize()
    bad = []

    def work(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(6):
                a = rtt.rsvd(Gs[i], k=32, p=16, q=1, omega=om[i]).sigma
                b = rtt.age_information(Gs[i], ages)
                if not (np.array_equal(a, want[i][0]) and np.array_equal(b, want[i][1])):
                    bad.append(i)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    say("case two threads")
    assert not bad


def test_scratch_is_bounded_and_returned_with_the_last_handle(gpu_lib):
    import torch
    rtt = gpu_lib
    gc.collect()
    torch.cuda.empty_cache()
    geo = tiny_geometry(seed=235, rays=(3000, 500, 400), n_r=16, n_phi=24, n_frames=128)
    before = torch.cuda.mem_get_info()[0]
    G = rtt.Geometry(geo)
    rtt.age_information(G, 4.0 * np.arange(200))   # about 0.5 GB of probes and responses
    held = before - torch.cuda.mem_get_info()[0]
    say("case returned scratch", held)
    assert held < (9 << 30)
    G.free()
    gc.collect()
    torch.cuda.empty_cache()
    # other tests' handles may be alive still: then the idle blocks stay, within their bound
    assert before - torch.cuda.mem_get_info()[0] <= max(held, 0)
