"""Lattices past a 32-bit limit: launches of 2^32 work-items, which HIP does not take in one grid dimension, and rows of
4 GiB.  The fields are the same at every site (periodic), so that every site's result is the one of a small lattice, and
a site left out, visited twice or read from elsewhere shows."""
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


def _same_on_every_site(big, small, tol=1e-13):
    worst = max(float((t - small).abs().max()) for t in big)  # one t slice at a time
    assert worst <= tol * float(small.abs().max()), worst


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


def test_brillouin_row_of_4_gib_of_links():
    """A lattice row whose links pass the 32-bit byte offsets of the row kernel (34 GB of W; a prime extent, so that only
    overlapping segments could cut it)."""
    rng = np.random.default_rng(702)
    w, u = _cg(rng, (40, 3, 3)), _cg(rng, (3, 4, 4))
    # (the bar of the FP64 applies: the two lattices take different kernels)
    small, big = (dirac.apply("brillouin", _everywhere(d, w), _everywhere(d, u), 0.1, antiperiodic_t=False)
                  for d in ((5, 2, 2, 2), (745673, 2, 2, 2)))
    _same_on_every_site(big, small[0, 0, 0, 0], 1e-12)
