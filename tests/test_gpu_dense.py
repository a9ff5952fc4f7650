"""The dense FP64 building blocks at the edges of their tiles and blocks: the
two tile shapes of the complex GEMM, the register-resident pivot-block inverse
of eps^-1 and the Cholesky blocks of Diag, against NumPy."""
import numpy as np
import pytest
import torch

import paper_2509_23018_amd as gw
from gpu_helpers import device, rel_fro

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


def _crand(rng, *shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def _to(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(device())


# pivot blocks of 64: one row of them, a full one, one past, the last of 1 and
# of 63, and (past 512) a second level
@pytest.mark.parametrize("n", [1, 16, 17, 63, 64, 65, 127, 513, 575])
def test_epsinv_pivot_blocks(n):
    rng = np.random.default_rng(n)
    x = _crand(rng, 2, n, 2 * n)
    chi = -(x @ x.conj().swapaxes(1, 2)) / (2 * n)   # I - v chi: eigenvalues in about [1, 6]
    v = rng.uniform(0.1, 2.0, n)
    got = gw.gw_epsinv(_to(chi), _to(v)).cpu().numpy()
    want = np.linalg.inv(np.eye(n)[None] - v[None, :, None] * chi)
    # condition times unit roundoff, n steps of elimination
    cond = max(np.linalg.cond(w) for w in want)
    for w in range(2):
        assert rel_fro(got[w], want[w]) < 8 * EPS * cond * np.sqrt(n + 1)
