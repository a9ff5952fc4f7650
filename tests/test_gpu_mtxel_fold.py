"""gw_mtxel at the edges of its stage z and y kernels: line lengths around the
8-pair blocks of folded lines, class counts around the groups of 4 and past the
16 that are folded, windows of one sign, ragged band tiles, and tables that
leave room for a ring of two slabs only."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_23018_amd as gw
from gpu_helpers import FP64_TOL, device, rel_fro
from workloads import gen

pytestmark = pytest.mark.gpu


def _axis(n, classes, sign):
    """Frequencies of `classes` classes min(k, n - k): the class numbers 0, 1, ...
    with one sign or both."""
    ks = set()
    for a in range(classes):
        if sign >= 0:
            ks.add(a)
        if sign <= 0:
            ks.add(-a)
    lo = -(n // 2)
    return sorted({(k - lo) % n + lo for k in ks})


@pytest.mark.parametrize("n2,n3,c2,c3,sign,nv,nc", [
    (1, 1, 1, 1, 0, 1, 1),        # one point on both axes
    (2, 1, 2, 1, 0, 1, 2),        # the Nyquist class alone
    (15, 16, 3, 4, 0, 2, 9),      # 8 pairs, odd (the centre halved) and even
    (17, 18, 4, 5, 0, 4, 8),      # 9 pairs: one past a block
    (7, 33, 4, 8, 0, 5, 17),      # one partial block; ragged tiles
    (32, 31, 8, 9, 0, 3, 5),      # third group of k3 classes
    (31, 24, 9, 12, 1, 1, 11),    # k >= 0 only
    (26, 25, 13, 13, -1, 4, 3),   # k <= 0 only
    (30, 31, 16, 16, 0, 2, 5),    # the last folded box (Nyquist class of 30: 15)
    (34, 34, 16, 17, 0, 2, 3),    # k3 past it
    (34, 34, 17, 16, 0, 2, 3),    # k2 past it
    (200, 198, 6, 5, 0, 1, 9),    # a ring of two slabs
])
def test_mtxel_line_edges(n2, n3, c2, c3, sign, nv, nc):
    n = (3, n2, n3)
    g = np.array([(a, b, c) for a in (-1, 0, 1) for b in _axis(n2, c2, sign)
                  for c in _axis(n3, c3, sign)], dtype=np.int32)
    p = gen.make_problem(n, nv, nc, gvec=g, seed=n2 + 7 * n3)
    dev = [torch.from_numpy(np.ascontiguousarray(a)).to(device()) for a in (p.psi_v, p.psi_c)]
    m = gw.gw_mtxel(*dev, g, n, p.volume).cpu().numpy()
    ref = oracle.mtxel(p.psi_v, p.psi_c, g, n, p.volume)
    assert m.shape == ref.shape
    assert rel_fro(m, ref) < FP64_TOL
    assert np.max(np.abs(m - ref)) < FP64_TOL * np.max(np.abs(ref))
