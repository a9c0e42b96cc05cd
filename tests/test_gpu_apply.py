"""The Wilson-Dirac operator on canonical fields in one pass: block and sheet
remainders, both kernels, and the even/odd route that calls with overlapping
fields take, against the oracle.  Tolerance: a component of D psi sums 8
directions of 3 complex products (2 after projection): at most 100 roundings of
1.1e-16, relative to the largest component 1e-14."""
import ctypes

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


# V = 16 and 288 (partial last blocks); sheets of 4 timeslices with 2 over and 8
# blocks a slice with 1 over; up to and beyond 256 blocks; 1, 4 and 5 right-hand
# sides (a workgroup holds 4)
@pytest.mark.parametrize("dims,nrhs", [((2, 2, 2, 2), 1), ((6, 4, 2, 6), 5), ((4, 4, 4, 4), 70), ((6, 4, 2, 6), 52),
                                       ((8, 8, 4, 6), 16), ((8, 12, 6, 6), 5), ((4, 2, 6, 4), 90)])
@pytest.mark.parametrize("bc,dagger", [(-1, False), (1, True), (-1, True)])
def test_apply_D_both_routes(F, dims, nrhs, bc, dagger):
    import torch
    U = S.random_links(dims, 0.7, 61)
    lat = F.Lattice(dims, bc)
    lat.set_gauge(U)
    lat.set_kappa(0.13)
    psi = S.random_spinors(dims, nrhs, 62)
    want = O.apply_D(U, psi, dims, bc, 0.13, dagger=dagger).reshape(psi.shape)
    bound = 1e-14 * np.abs(want).max()
    assert np.abs(lat.apply_D(psi, dagger=dagger) - want).max() <= bound
    x = torch.from_numpy(psi).cuda()
    assert np.abs(lat.apply_D(x, dagger=dagger).cpu().numpy() - want).max() <= bound
    # the result over the input: the even/odd route
    st = F.lib().fl_apply_D(lat._h, ctypes.c_void_p(x.data_ptr()), ctypes.c_void_p(x.data_ptr()), nrhs, int(dagger),
                            F.FL_DEVICE)
    assert st == 0
    assert np.abs(x.cpu().numpy() - want).max() <= bound
    x = torch.from_numpy(psi).cuda()
    lat.apply_D_noalloc(x, x, dagger=dagger)
    assert np.abs(x.cpu().numpy() - want).max() <= bound
    lat.close()
