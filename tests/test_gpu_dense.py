"""The dense FP64 building blocks at the edges of their tiles and blocks: the
two tile shapes of the complex GEMM, the register-resident pivot-block inverse
of eps^-1, the Cholesky blocks of Diag and the GPP kernel's row tiles and band
batches, against NumPy and the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2509_23018_amd as gw
from gpu_helpers import FP64_TOL, device, rel_fro
from workloads import gen

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


def _crand(rng, *shape):
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def _to(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(device())


# k around the 16-deep stages (none, one, an odd and an even count, each with
# and without a partial last one); m, n off and on the tile edges.  The batch
# puts the same products on 64 x 32 tiles (from 1,024 of them on) and alone on
# 32 x 32 tiles.
@pytest.mark.parametrize("m,n,k", [(64, 32, 16), (65, 33, 1), (63, 31, 15), (33, 65, 17),
                                   (1, 70, 32), (70, 1, 33), (40, 40, 48), (96, 64, 63),
                                   (64, 64, 64), (31, 97, 95), (129, 33, 97)])
def test_zgemm_tile_shapes_agree(m, n, k):
    rng = np.random.default_rng(m + 100 * n + k)
    batch = -(-1024 // (-(-m // 64) * -(-n // 32)))
    a, b = _crand(rng, batch, m, k), _crand(rng, batch, k, n)
    many = gw.gw_zgemm("N", "N", _to(a), _to(b)).cpu().numpy()
    one = gw.gw_zgemm("N", "N", _to(a[-1]), _to(b[-1])).cpu().numpy()
    assert np.array_equal(many[-1], one)      # a tile does not change the order of a sum
    # k products and as many sums of rounded three-product terms per entry
    assert rel_fro(many, a @ b) < 8 * EPS * np.sqrt(k + 1)
    for op in ("T", "C"):
        ta = _to(np.swapaxes(a if op == "T" else a.conj(), 1, 2))
        tb = _to(np.swapaxes(b if op == "T" else b.conj(), 1, 2))
        assert np.array_equal(gw.gw_zgemm(op, op, ta, tb).cpu().numpy(), many)


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


# Cholesky blocks of 64 on nb = n_eig + guard columns: below, at and past one
# and two blocks; rank: of the matrix (below nb: directions are lost)
@pytest.mark.parametrize("n_eig,guard,rank", [(40, 23, 200), (40, 24, 200), (41, 24, 200),
                                              (100, 28, 200), (100, 29, 200), (30, 40, 50)])
def test_diag_cholesky_blocks(n_eig, guard, rank):
    ng = 200
    rng = np.random.default_rng(n_eig + guard)
    q = np.linalg.qr(_crand(rng, ng, ng))[0]
    ev = np.zeros(ng)
    ev[:rank] = 0.95 ** np.arange(rank)              # -chi, decreasing
    chi = -(q * ev) @ q.conj().T
    chi = 0.5 * (chi + chi.conj().T)
    basis, w, info = gw.gw_subspace_basis(_to(chi), n_eig, guard=guard, max_iter=200)
    basis, w = basis.cpu().numpy(), w.cpu().numpy()
    # the default tol bounds each kept pair's residual by 1e-10 of the Gershgorin bound
    res = 1e-10 * info["bound"]
    assert info["residual"] <= 1e-10
    assert np.abs(w + ev[:n_eig]).max() < res
    assert np.abs(basis.conj().T @ basis - np.eye(n_eig)).max() < 1e-13
    assert np.linalg.norm(chi @ basis - basis * w, axis=0).max() < 1.01 * res


# ns on the four row-tile heights and past them; ng without a whole 16-row
# stage, with one, two, an odd number of them, and remainders; more bands than a
# launch holds (64).  An exact-size workspace holds one band per launch.
@pytest.mark.parametrize("nb,ns,ng,ne", [(3, 1, 1, 2), (2, 16, 15, 3), (2, 17, 16, 1),
                                         (3, 32, 33, 2), (2, 33, 48, 2), (2, 48, 65, 3),
                                         (2, 49, 79, 2), (2, 64, 112, 1), (2, 65, 130, 2),
                                         (67, 5, 40, 2)])
def test_gpp_tiles_and_bands(nb, ns, ng, ne):
    inp = gen.gpp_inputs(nb, ns, ng, ne, seed=nb + ns + ng)
    want = oracle.gpp_sigma_offdiag(inp["m"], inp["e_n"], inp["occupied"], inp["energies"],
                                    inp["omega2"], inp["wtilde"], inp["v"])
    d = {k: _to(inp[k]) for k in ("m", "omega2", "wtilde", "v")}
    args = (d["m"], inp["e_n"], inp["occupied"], inp["energies"], d["omega2"], d["wtilde"], d["v"])
    assert rel_fro(gw.gw_gpp_sigma(*args).cpu().numpy(), want) < FP64_TOL
    need = int(gw.lib().gw_gpp_sigma_workspace_bytes(ns, ng, ne))
    ws = gw.new_workspace(need + 256, device())
    ws[need:] = 7
    got = gw.gw_gpp_sigma(*args, workspace=ws[:need])
    assert rel_fro(got.cpu().numpy(), want) < FP64_TOL
    assert bool((ws[need:] == 7).all())
    with pytest.raises(gw.GWError):
        gw.gw_gpp_sigma(*args, workspace=ws[:need - 256])


# one workgroup per matrix below n = 64: no rotation, one, odd sizes (a phantom
# index), the largest; diagonal, degenerate, rank-one, graded and zero matrices
@pytest.mark.parametrize("n", [1, 2, 3, 5, 16, 31, 47, 62, 63])
def test_heev_one_workgroup(n):
    rng = np.random.default_rng(n)
    x = _crand(rng, n, n)
    u = _crand(rng, n, 1)
    g = np.logspace(0, -12, n)
    a = np.stack([x + x.conj().T, np.diag(rng.standard_normal(n)).astype(complex), np.eye(n) + 0j,
                  u @ u.conj().T, g[:, None] * (x + x.conj().T) * g[None, :],
                  np.zeros((n, n), complex)])
    w, v = (t.cpu().numpy() for t in gw.gw_heev(_to(a)))
    for i in range(len(a)):
        want = np.linalg.eigvalsh(a[i])
        scale = np.abs(want).max()
        # some ten sweeps of n - 1 steps, each within a few units of roundoff
        tol = 10 * n * EPS
        assert np.abs(w[i] - want).max() <= tol * scale
        assert np.abs(v[i].conj().T @ v[i] - np.eye(n)).max() <= tol
        assert np.abs(a[i] @ v[i] - v[i] * w[i][None, :]).max() <= tol * scale
