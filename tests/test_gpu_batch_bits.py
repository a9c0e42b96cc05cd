"""A right-hand side's result does not depend on the right-hand sides beside it,
in no bit: the kernels that a batch's size selects (a wave per direction or
shared links, scalar steps in launches of their own or inside the vector
kernels, one pass or one hop per parity) form the same sums."""
import ctypes

import numpy as np
import pytest

import synth_inputs as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    import paper_1108_2473_amd as fl
    fl.lib()
    return fl


def make(F, dims):
    lat = F.Lattice(dims, -1)
    lat.set_gauge(S.random_links(dims, 0.5, 71))
    lat.set_kappa(0.13)
    return lat


# 192 sites a parity (three blocks): 3 right-hand sides 9 tiles, 342 beyond the
# 1024 tiles of the hop with a wave per direction, 1100 beyond the 3072 of the
# folded scalar steps; 64 blocks: 3 and 12 right-hand sides
@pytest.mark.parametrize("prec,reals", [(0, 18), (1, 12), (1, 18), (2, 12), (3, 12)])
@pytest.mark.parametrize("solver", [0, 1])
@pytest.mark.parametrize("truncated", [False, True])
@pytest.mark.parametrize("dims,counts", [((4, 4, 4, 6), (1, 2, 3, 342, 1100)), ((8, 8, 8, 16), (1, 2, 3, 12))])
def test_solution_independent_of_batch(F, prec, reals, solver, truncated, dims, counts):
    """The same system n times: CGNR's host checks follow the fastest system
    of a batch, so batches of equal systems are checked at the same iterations."""
    lat = make(F, dims)
    b = S.random_spinors(dims, 1, 72)
    kw = dict(inner_prec=prec, gauge_reals=reals, solver=solver)
    kw.update(dict(truncated=True, max_iter=7) if truncated else dict(tol=1e-9))
    want = None
    for n in counts:
        bn = np.ascontiguousarray(np.broadcast_to(b, (n,) + b.shape[1:]))
        x, _ = lat.solve(bn, F.SolverParams(**kw), check=False)
        want = x[0].copy() if want is None else want
        for k in (0, n // 2, n - 1):
            assert np.array_equal(x[k], want), (n, k)
    lat.close()


# host and device fields, up to and beyond 256 blocks of the one-pass kernels,
# and the even/odd route (result over the input) in every shape of its hop
@pytest.mark.parametrize("dims", [(4, 4, 4, 6), (6, 4, 2, 6), (8, 8, 8, 16)])
@pytest.mark.parametrize("dagger", [False, True])
def test_operator_same_on_every_route(F, dims, dagger):
    import torch
    lat = make(F, dims)
    psi = S.random_spinors(dims, 90, 73) if dims[3] == 6 else S.random_spinors(dims, 12, 73)
    x = torch.from_numpy(psi).cuda()
    want = lat.apply_D(x, dagger=dagger).cpu().numpy()
    assert np.array_equal(lat.apply_D(psi, dagger=dagger), want)
    for n in (1, 2, 3, 4, 12):
        assert np.array_equal(lat.apply_D(x[:n].clone(), dagger=dagger).cpu().numpy(), want[:n]), n
        for rt, lds in ((0, -1), (1, 0), (1, 1), (2, 1), (4, 2), (4, 4), (8, 4)):
            lat.set_tile(prec=0, gauge_reals=18, rt=rt, lds=lds)
            y = x[:n].clone()
            st = F.lib().fl_apply_D(lat._h, ctypes.c_void_p(y.data_ptr()), ctypes.c_void_p(y.data_ptr()), n, int(dagger),
                                    F.FL_DEVICE)
            assert st == 0
            assert np.array_equal(y.cpu().numpy(), want[:n]), (n, rt, lds)
    lat.close()


def test_staged_16bit_links_are_unbiased(F):
    """The packed 16-bit hop works with links at half scale.  Every odd entry is
    a tie there; rounded up instead of to even, the entries of rows 0 and 1 are
    1/4 unit too large on average and the operator shifts coherently.  The
    mean difference from the kernel that reads the links at full scale is
    projected on that shift.  Its coefficient is 1 for rounding up; unbiased
    errors (rms 0.35 units, 24 of them a hop) average over 2048 sites to about
    0.02 of it, so 0.1 separates the two."""
    import oracle as O
    dims, kappa = (8, 8, 8, 8), 0.2
    U = S.random_links(dims, 0.3, 74)
    V = U.shape[1]
    lat = F.Lattice(dims, -1)
    lat.set_gauge(U)
    lat.set_kappa(kappa)
    prm = F.SolverParams(inner_prec=3, gauge_reals=12)
    x = np.arange(V)
    even = sum(x // int(np.prod(dims[:m])) % dims[m] for m in range(4)) % 2 == 0
    psi = np.zeros((1, V, 4, 3), complex)
    psi[0, even] = 1.0
    out = {}
    for lds in (0, 4):
        lat.set_tile(prec=3, gauge_reals=12, rt=8, lds=lds)
        out[lds] = lat.apply_schur(psi, prm)[0]
    lat.close()

    def schur(links):  # psi - kappa^2 H H psi, with H = (1 - D) / kappa
        h = (psi - O.apply_D(links, psi, dims, -1, kappa).reshape(psi.shape)) / kappa
        hh = (h - O.apply_D(links, h, dims, -1, kappa).reshape(psi.shape)) / kappa
        return (psi - kappa ** 2 * hh)[0]

    up = U.copy()
    up[:, :, :2] += 0.25 * (1 + 1j) / 16383.5
    shift = (schur(up) - schur(U))[even].mean(axis=0)
    got = (out[4] - out[0])[even].mean(axis=0)
    assert abs(np.vdot(shift, got)) <= 0.1 * np.vdot(shift, shift).real


@pytest.mark.parametrize("nrhs", [9, 12, 17, 20])
def test_16bit_workgroups_of_four(F, nrhs):
    """The workgroups of 4 right-hand sides that the 16-bit hop takes for these
    counts, the last one partly filled (lds=4 keeps the built-in workgroup and
    turns the wave per direction off), against workgroups of 8 and a wave per
    direction."""
    dims = (6, 4, 4, 6)
    lat = make(F, dims)
    psi = S.random_spinors(dims, nrhs, 75)
    prm = F.SolverParams(inner_prec=3, gauge_reals=12)
    split = lat.apply_schur(psi, prm)
    lat.set_tile(prec=3, gauge_reals=12, lds=4)
    four = lat.apply_schur(psi, prm)
    lat.set_tile(prec=3, gauge_reals=12, rt=8)
    eight = lat.apply_schur(psi, prm)
    lat.close()
    assert np.array_equal(four, split)
    assert np.array_equal(four, eight)


def test_noalloc_scratch_is_reused(F):
    """Result over the input: the work fields in the fixed scratch array, which
    the second, smaller call finds as the first left them."""
    import torch
    dims = (8, 8, 8, 16)
    lat = make(F, dims)
    for nrhs, seed in ((16, 76), (3, 77)):
        psi = torch.from_numpy(S.random_spinors(dims, nrhs, seed)).cuda()
        want = lat.apply_D(psi)
        lat.apply_D_noalloc(psi, psi)
        torch.cuda.synchronize()
        assert torch.equal(psi, want)
    lat.close()
