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
