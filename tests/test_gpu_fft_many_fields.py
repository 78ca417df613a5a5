"""gf_fft of so many fields that one launch of a pass over all of them would
have 2^32 work-items or more."""
import numpy as np
import pytest
import torch

import oracle
from paper_1210_8018_amd.api import GaugeFixer
from paper_1210_8018_amd.inputs import random_links

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 8191, 8192, 33000])
def test_many_fields(n):
    """64 x 64 x 2 x 2: 512 work-groups of 256 per field in the (z, t) pass, so
    32768 fields are 2^32 work-items (8.7 GB of fields). Every field is the same
    one times a phase of its own; bound as for a few fields, 1e-13 of the largest."""
    dims = (64, 64, 2, 2)
    V = int(np.prod(dims))
    fx = GaugeFixer(torch.from_numpy(random_links(dims, 0.3, 1)).to("cuda"), fft_schedule=3)
    rng = np.random.default_rng(43)
    f = rng.standard_normal(V) + 1j * rng.standard_normal(V)
    ref = torch.from_numpy(oracle.fft4d(dims, f, -1)).to("cuda")
    phase = torch.polar(torch.ones(n, dtype=torch.float64), 0.001 * torch.arange(n, dtype=torch.float64)).to("cuda")
    got = fx.fft(torch.outer(phase, torch.from_numpy(f).to("cuda")), -1)
    top = float(ref.abs().max())
    for a in range(0, n, 4096):
        assert float((got[a:a + 4096] - torch.outer(phase[a:a + 4096], ref)).abs().max()) < 1e-13 * top, a
