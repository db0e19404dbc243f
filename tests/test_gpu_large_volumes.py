"""Gradients on lattices whose launches pass 2^32 work-items, which HIP does not take in one grid dimension: fields that are
the same at every site (N_c = 1, periodic), so that every site's gradient is the one of a small lattice, and a site left
out or visited twice shows."""
import gc

import numpy as np
import pytest
import torch

from paper_2112_14640_amd import dirac
from tests.gpu_helpers import DEV

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _free():
    yield
    gc.collect()
    torch.cuda.empty_cache()


def _everywhere(dims, block):
    """The values of one site on every site of the lattice."""
    b = torch.from_numpy(block).to(DEV)
    out = torch.empty(dims[::-1] + b.shape, dtype=b.dtype, device=DEV)
    return out.copy_(b.expand(out.shape))


def _cg(rng, shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def _same_on_every_site(big, small):
    worst = max(float((t - small).abs().max()) for t in big)  # one t slice at a time
    assert worst <= 1e-13 * float(small.abs().max()), worst


def test_links_backward_past_2_32_work_items():
    """64 N_c threads per site: 4.33e9 at 64^3 x 258 (43 GB of gW)."""
    rng = np.random.default_rng(700)
    v = np.exp(1j * rng.uniform(0, 2 * np.pi, (4, 1, 1)))
    gw = _cg(rng, (40, 1, 1))
    small, big = (dirac.brillouin_links_backward(_everywhere(d, v), _everywhere(d, gw))
                  for d in ((4, 4, 4, 4), (64, 64, 64, 258)))
    _same_on_every_site(big, small[0, 0, 0, 0])


@pytest.mark.parametrize("nv", [3, 1])
def test_brillouin_force_past_2_32_work_items(nv):
    """128 threads per site from three right-hand sides on: 4.36e9 at 64^3 x 130 (22 GB of gradient)."""
    rng = np.random.default_rng(701)
    psi, chi = _cg(rng, (1, 4, nv)), _cg(rng, (1, 4, nv))
    w = np.ones((40, 1, 1), dtype=complex)
    small, big = (dirac.force("brillouin", _everywhere(d, w), _everywhere(d, psi), _everywhere(d, chi),
                              antiperiodic_t=False) for d in ((4, 4, 4, 4), (64, 64, 64, 130)))
    _same_on_every_site(big, small[0, 0, 0, 0])
