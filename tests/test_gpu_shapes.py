"""Sizes at which the batched kernels change shape: right-hand sides that
select workgroups of 4, 6 or 8, lattices that end inside a workgroup of the
layout conversion, and waves of the force kernel that reach past the lattice."""
import numpy as np
import pytest

import oracle as O
import synth_inputs as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import paper_1108_2473_amd as fl
    fl.lib()
    return fl


def make(F, dims, kappa=0.12, seed=51):
    U = S.random_links(dims, 0.5, seed)
    lat = F.Lattice(dims, -1)
    lat.set_gauge(U)
    lat.set_kappa(kappa)
    return lat, U


@pytest.mark.parametrize("prec,reals", [(0, 18), (1, 12), (1, 18), (2, 12), (3, 12)])
@pytest.mark.parametrize("nrhs", [9, 12, 17, 20])
def test_workgroup_shapes_change_no_result(F, prec, reals, nrhs):
    """One block and a few right-hand sides more than 8 or 16: smaller
    workgroups are chosen; the results equal those of workgroups of 8 bit for
    bit."""
    dims = (6, 4, 4, 6)
    lat, _ = make(F, dims)
    psi = S.random_spinors(dims, nrhs, 52)
    prm = F.SolverParams(inner_prec=prec, gauge_reals=reals)
    got = lat.apply_schur(psi, prm)
    lat.set_tile(prec=prec, gauge_reals=reals, rt=8)
    assert np.array_equal(got, lat.apply_schur(psi, prm))
    lat.close()


# Vh = 8, 136 (a workgroup of 128 pairs and 8 more), 128 and 384
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (2, 2, 2, 34), (4, 4, 4, 4), (4, 4, 6, 8)])
def test_layout_conversion_round_trip(F, dims):
    """With a vanishing hopping parameter D is the identity up to kappa: the
    conversions to and from the checkerboard layout return every value."""
    lat, U = make(F, dims, kappa=0.11)
    psi = S.random_spinors(dims, 3, 53)
    got = lat.apply_D(psi)
    want = O.apply_D(U, psi, dims, -1, 0.11)
    assert np.abs(got - want).max() <= 1e-13 * np.abs(want).max()
    lat.set_kappa(1e-300)
    assert np.array_equal(lat.apply_D(psi), psi)
    lat.close()


@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (6, 4, 2, 6), (4, 2, 6, 4)])
def test_gradient_ragged(F, dims):
    """Vh = 8, 144 and 96: partial waves, directions of extent 2, several
    insertions."""
    lat, U = make(F, dims, kappa=0.13)
    Vs = dims[0] * dims[1] * dims[2]
    rng = np.random.Generator(np.random.PCG64(54))
    w = np.zeros((3, 1, Vs), complex)
    w[:, 0, :3] = rng.standard_normal((3, 3)) + 1j * rng.standard_normal((3, 3))
    t = dims[3] - 1
    dU, dk = lat.loops_grad([t], [0, 15, 4], w, F.SolverParams(tol=1e-12))
    dUo, dko = O.loops_grad(U, dims, -1, 0.13, [t], [0, 15, 4], w, tol=1e-14)
    assert np.abs(dU - dUo).max() <= 1e-9 * np.abs(dUo).max()
    assert abs(dk - dko) <= 1e-9 * abs(dko)
    lat.close()


@pytest.mark.parametrize("prec,reals", [(1, 12), (1, 18), (3, 12)])
@pytest.mark.parametrize("solver", [0, 1])
def test_small_grid_truncated_bits(F, prec, reals, solver):
    """Truncated solves in the low precisions: alone on a small grid (scalar
    steps inside the vector kernels, 16-bit hops with a wave per direction) and
    in a batch beyond both limits (3072 and 1024 tiles) the results are equal
    bit for bit."""
    dims = (4, 4, 4, 6)  # 192 sites: three blocks
    lat, _ = make(F, dims)
    n = 1400
    few = S.random_spinors(dims, 4, 55)  # 4: fewer use another FP64 hop around the iteration
    b = np.ascontiguousarray(np.broadcast_to(few, (n // 4,) + few.shape)).reshape((n,) + few.shape[1:])
    prm = F.SolverParams(inner_prec=prec, gauge_reals=reals, truncated=True, max_iter=7, solver=solver)
    big, _ = lat.solve(b, prm, check=False)
    small, _ = lat.solve(few, prm, check=False)
    assert np.array_equal(big[:4], small)
    assert np.array_equal(big[-4:], small)
    lat.close()


@pytest.mark.parametrize("prec", [0, 1, 3])
@pytest.mark.parametrize("solver", [0, 1])
@pytest.mark.parametrize("dims,nrhs", [((2, 2, 2, 2), 1), ((6, 4, 2, 6), 3), ((8, 8, 8, 28), 2), ((8, 8, 8, 28), 3),
                                       ((4, 4, 4, 6), 341), ((4, 4, 4, 6), 342)])
def test_small_grid_solves(F, prec, solver, dims, nrhs):
    """On both sides of the limits of the hop with a wave per direction (FP64 330
    tiles: 224 and 336; 16-bit 1024: 1023 and 1026; FP32 up to 3 right-hand
    sides) and down to one partly filled site block: the residual recomputed
    with the operator meets the tolerance (rounding of the recomputation:
    1e-14)."""
    lat, U = make(F, dims, kappa=0.13)
    b = S.random_spinors(dims, nrhs, 56)
    tol = 1e-10
    x, info = lat.solve(b, F.SolverParams(inner_prec=prec, solver=solver, tol=tol))
    assert all(q["converged"] for q in info)
    r = (b - lat.apply_D(x)).reshape(nrhs, -1)
    rel = np.linalg.norm(r, axis=1) / np.linalg.norm(b.reshape(nrhs, -1), axis=1)
    assert rel.max() <= tol + 1e-14
    want = O.apply_D(U, x[-1:], dims, -1, 0.13)
    assert np.linalg.norm(b[-1:] - want) <= (tol + 1e-14) * np.linalg.norm(b[-1:])
    lat.close()
