"""Calls that go on where an earlier one stopped: the same values, bit for
bit, as one uninterrupted call, wherever the earlier one stopped within the
updates it had launched, and whatever stage calls lie in between."""
from functools import lru_cache

import numpy as np
import pytest
import torch

from paper_1210_8018_amd.api import BatchGaugeFixer, GaugeFixer
from paper_1210_8018_amd.inputs import random_links

pytestmark = pytest.mark.gpu

N = 12  # updates: the call's first, a whole chunk of 8 and part of another
# (x, y) planes of every pass that carries the reduction of the update before:
# register groups, registers throughout with 256 and 192 work-items per
# work-group, and the LDS-staged pass (an extent above 64)
DIMS = [(8, 8, 8, 8), (6, 4, 9, 4), (24, 24, 4, 6), (32, 32, 4, 4), (48, 48, 3, 4), (72, 4, 4, 6)]
KINDS = [dict(), dict(fft_prec=1), dict(fft_prec=1, link_prec=1, refine_theta=1e-30), dict(reunit_every=3)]


@lru_cache(maxsize=1)
def large_links(dims):
    return random_links(dims, 0.25, 503)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("sched", [1, 2, 3])
@pytest.mark.parametrize("kw", KINDS)
@pytest.mark.parametrize("dims", DIMS)
def test_fix_until_goes_on_after_any_stop(dims, kw, sched):
    """A first call stopped by its cap or by its bound on theta after k
    updates, then a second one (a step after it where k is even)."""
    U = random_links(dims, 0.25, 501)
    kw = dict(kw, fft_schedule=sched)
    whole = dev(U)
    fx = GaugeFixer(whole, **kw)
    fx.fix_until(1e-28, N, allow_maxiter=True)
    F, T = fx.history()
    fx.close()
    assert len(T) == N + 1
    for k in range(1, N):
        for stop in ("cap", "theta"):
            links = dev(U)
            fx = GaugeFixer(links, **kw)
            if stop == "cap":
                it, _, _ = fx.fix_until(1e-28, k, allow_maxiter=True)
            elif min(T[:k]) > T[k]:
                it, _, _ = fx.fix_until(T[k], N, allow_maxiter=True)
            else:
                continue
            assert it == k
            if k % 2:
                fx.fix_until(1e-28, N - k, allow_maxiter=True)
            else:
                fx.step(N - k)
            assert fx.history() == (F, T), (k, stop)
            assert torch.equal(links, whole), (k, stop)
            fx.close()


@pytest.mark.parametrize("sched", [1, 2, 3])
@pytest.mark.parametrize("dims,prec", [((32, 32, 32, 24), 0), ((24, 36, 24, 36), 0), ((72, 48, 16, 16), 0),
                                       ((32, 32, 48, 32), 1), ((72, 48, 24, 24), 1)])
def test_large_lattices_go_on(dims, prec, sched):
    """Lattices transformed in two sets of fields, not three."""
    kw = dict(fft_prec=prec, fft_schedule=sched)
    whole, links = dev(large_links(dims)), dev(large_links(dims))
    fx = GaugeFixer(whole, **kw)
    fx.fix_until(-1.0, N, allow_maxiter=True)
    fa = GaugeFixer(links, **kw)
    for n in (3, 2, N - 5):
        fa.fix_until(-1.0, n, allow_maxiter=True)
    assert fa.history() == fx.history() and torch.equal(links, whole)


@pytest.mark.parametrize("sched", [1, 2, 3])
@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (24, 24, 4, 6), (72, 4, 4, 6)])
def test_separate_update_and_divergence_go_on(monkeypatch, dims, sched):
    monkeypatch.setenv("GF_NOFUSE", "1")
    for kw in (dict(), dict(fft_prec=1)):
        test_fix_until_goes_on_after_any_stop(dims, kw, sched)


@pytest.mark.parametrize("sched", [1, 2, 3])
@pytest.mark.parametrize("prec", [0, 1])
def test_stage_calls_leave_the_next_update_as_it_was(prec, sched):
    """gauge() measures Delta as functional() does; an update after either is the same."""
    dims = (8, 8, 8, 8)
    U = random_links(dims, 0.25, 502)
    kw = dict(fft_prec=prec, fft_schedule=sched)
    a, b = dev(U), dev(U)
    fa, fb = GaugeFixer(a, **kw), GaugeFixer(b, **kw)
    for n in (1, 3):
        fa.functional()
        fa.step(n)
        fb.gauge()
        fb.plaquette()
        fb.fft(torch.zeros((2, a.numel() // 36), dtype=torch.complex64 if prec else torch.complex128, device="cuda"), -1)
        fb.step(n)
    assert fa.history() == fb.history() and torch.equal(a, b)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("sched", [2, 3])
def test_batch_goes_on(prec, sched):
    """Members that stop at different updates of the first call, against one
    uninterrupted call of a context each (F and theta to the rounding of sums
    over other walks)."""
    members = [((8, 8, 8, 8), 0.3, 511), ((24, 24, 4, 6), 0.05, 512), ((12, 8, 6, 4), 0.2, 513), ((16, 16, 8, 8), 0.02, 514)]
    kw = dict(fft_prec=prec, fft_schedule=sched)
    links = [random_links(d, e, s) for d, e, s in members]
    bl, sl = [dev(u) for u in links], [dev(u) for u in links]
    bx, fx = BatchGaugeFixer(bl, **kw), [GaugeFixer(u, **kw) for u in sl]
    first = bx.fix_until(1e-7, 400)[0]
    second = bx.fix_until(1e-12, 400)[0]
    for k, f in enumerate(fx):
        it, _, _ = f.fix_until(1e-12, 400)
        assert it == first[k] + second[k]
        assert torch.equal(bl[k], sl[k])
        (Fb, Tb), (Fs, Ts) = bx.history(k), f.history()
        assert np.max(np.abs(np.subtract(Fb, Fs))) <= 1e-15 and np.max(np.abs(np.divide(Tb, Ts) - 1)) <= 1e-12


@pytest.mark.parametrize("chunk", [1, 254, 255, 256])
def test_history_of_any_chunk_length(chunk):
    """As many (F, theta) as updates, the same for every chunk length that is
    taken (256: the length of the device's history ring)."""
    U = random_links((4, 4, 4, 4), 0.3, 521)
    out = []
    for n in (8, chunk):
        fx = GaugeFixer(dev(U), chunk=n, fft_schedule=3)
        fx.fix_until(-1.0, 600, allow_maxiter=True)
        fx.step(514)
        out.append(fx.history())
    assert len(out[0][0]) == 1 + 600 + 514 and out[0] == out[1]
