"""Walks of the marching kernels that differ by one slice, and the empty site
set that pads an odd number of sets for pairs."""
import numpy as np
import pytest
import torch

import oracle
from paper_1210_8018_amd.api import GaugeFixer
from paper_1210_8018_amd.inputs import random_links

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(36, 18, 24, 54), (36, 18, 12, 54), (27, 18, 18, 27), (48, 24, 9, 18), (32, 16, 16, 27)])
@pytest.mark.parametrize("kw", [dict(), dict(fft_prec=1, link_prec=1), dict(reunit_every=2)])
def test_planned_walks_equal_single_slices(monkeypatch, dims, kw):
    """The planned walks against one slice per walk and one site set per block:
    links bit for bit, F and theta to the rounding of their sums; the first
    measurement against the oracle."""
    U = random_links(dims, 0.3, 71)
    out = []
    for env in ({}, {"GF_TCHUNK": "1", "GF_PAIR": "0"}):
        for k, v in env.items():
            monkeypatch.setenv(k, v)
        Ud = torch.from_numpy(U).to("cuda")
        fx = GaugeFixer(Ud, fft_schedule=2, **kw)
        first = fx.functional()
        F, th = fx.step(5)
        fx.close()
        out.append((first, F, th, Ud))
    Fr, thr = oracle.measure(dims, U)
    assert abs(out[0][0][0] - Fr) < 1e-13 and abs(out[0][0][1] - thr) < 1e-12 * thr
    assert torch.equal(out[0][3], out[1][3])
    assert abs(out[0][1] - out[1][1]) <= 1e-15 * abs(out[1][1]) and abs(out[0][2] - out[1][2]) <= 1e-14 * out[1][2]


@pytest.mark.parametrize("dims", [(8, 8, 6, 4), (16, 16, 16, 32), (9, 6, 4, 27), (48, 16, 8, 8)])
@pytest.mark.parametrize("kw", [dict(fft_prec=1), dict(), dict(fft_prec=1, reunit_every=2)])
def test_binary32_links_in_and_out_of_a_call(dims, kw):
    """Binary32 storage: updates that read the caller's links and write them
    back equal those of a call that copies them in and out, bit for bit, in
    one call and in calls of one update."""
    U = random_links(dims, 0.3, 72)
    U = U * np.exp(1e-3j)  # not special unitary to rounding: rows 0 and 1 alone count
    a, b, c = (torch.from_numpy(U).to("cuda") for _ in range(3))
    kw = dict(kw, link_prec=1, fft_schedule=3, refine_theta=1e-20)
    fa, fb, fc = (GaugeFixer(u, **kw) for u in (a, b, c))
    Fa = fa.step(4)
    it, F, th = fb.fix_until(1e-20, 4, allow_maxiter=True)
    for _ in range(4):
        Fc = fc.step(1)
    assert it == 4 and torch.equal(a, b) and torch.equal(a, c)
    assert Fa == (F, th) and abs(Fa[0] - Fc[0]) < 1e-6


@pytest.mark.parametrize("dims", [(12, 12, 18, 64), (12, 9, 6, 256), (18, 18, 18, 48)])
@pytest.mark.parametrize("kw", [dict(), dict(fft_prec=1, link_prec=1), dict(reunit_every=2)])
def test_few_site_sets_with_an_empty_one(monkeypatch, dims, kw):
    """11, 3 and 23 site sets, padded to pairs."""
    test_planned_walks_equal_single_slices(monkeypatch, dims, kw)
