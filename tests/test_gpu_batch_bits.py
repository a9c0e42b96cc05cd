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
