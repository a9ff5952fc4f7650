"""The FP64 contraction at the edges of its 16-pair stages and of its tiles,
on both tile shapes and in the batched kernel, and the adjoint's product at the
edges of its stages, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_23018_amd as gw
from gpu_helpers import FP64_TOL, device, rel_fro, run_chi0, to_dev
from workloads import gen

pytestmark = pytest.mark.gpu


# pairs: no whole stage, one, one and a remainder, two, three with a remainder
# of 1 and 15, and enough for the pipelined loop; r2 = 6 gives 81 G: one tile
# and a ragged one
@pytest.mark.parametrize("nc", [1, 15, 16, 17, 32, 33, 47, 48, 49, 63, 95, 130])
@pytest.mark.parametrize("flags", [0, gw.GW_FLAG_FP64_TILE128], ids=["tile64", "tile128"])
def test_pair_stage_edges(nc, flags):
    p = gen.make_problem((10, 10, 10), 1, nc, r2=6, z=(0.0, 0.4j, 0.3 + 0.02j), seed=nc,
                         orthonormalize=False)
    want = oracle.chi0(p.psi_v, p.psi_c, p.e_v, p.e_c, p.gvec, p.z, p.n, p.volume)
    assert rel_fro(run_chi0(p, flags=flags), want) < FP64_TOL
    two = gw.gw_chi0([to_dev(p), to_dev(p)], flags=flags)   # the batched kernel
    for chi in two:
        assert rel_fro(chi.cpu().numpy(), want) < FP64_TOL
    assert np.array_equal(two[0].cpu().numpy(), two[1].cpu().numpy())


# G counts around the 16-G stages of the adjoint's g_M product on real Delta and
# around its pipelined pairs of stages (four whole stages and more); pair counts
# around its 32-pair tiles
@pytest.mark.parametrize("ng,nc", [(1, 1), (15, 3), (16, 31), (17, 32), (33, 33), (64, 5), (65, 64),
                                   (80, 7), (95, 2), (112, 9)])
def test_adjoint_product_stage_edges(ng, nc):
    g = gen.gsphere(12)[1:ng + 1]      # not G = 0, where orthonormal bands give M = 0
    p = gen.make_problem((8, 9, 10), 1, nc, gvec=g, z=(0.0, 0.3j), seed=ng, pair_chunk=1000)
    rng = np.random.default_rng(ng)
    w = rng.standard_normal((2, ng, ng)) + 1j * rng.standard_normal((2, ng, ng))
    got = gw.gw_chi0_backward(to_dev(p), torch.from_numpy(w).to(device()), pair_chunk=1000)
    ref = oracle.chi0_backward(p.psi_v, p.psi_c, p.e_v, p.e_c, p.gvec, p.z, p.n, p.volume, w,
                               spin=p.spin, pair_chunk=1000)
    for a, b in zip(got, ref):
        assert rel_fro(a.cpu().numpy(), b) < FP64_TOL
