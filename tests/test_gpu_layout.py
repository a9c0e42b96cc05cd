"""The conversions between canonical and checkerboard fields: lattices that end
inside a workgroup of 128 site pairs, the field stride of the smearing, and
fields that begin at any 8-byte boundary.  Callers reach them through the
even/odd route of the operator (result over the input) and through smearing."""
import ctypes

import numpy as np
import pytest

import oracle as O
import synth_inputs as S

pytestmark = pytest.mark.gpu

# Vh = 8, 136 (128 pairs and 8 more), 128 and 384
DIMS = [(2, 2, 2, 2), (2, 2, 2, 34), (4, 4, 4, 4), (4, 4, 6, 8)]


@pytest.fixture(scope="module")
def F():
    import paper_1108_2473_amd as fl
    fl.lib()
    return fl


def make(F, dims, kappa):
    U = S.random_links(dims, 0.5, 91)
    lat = F.Lattice(dims, -1)
    lat.set_gauge(U)
    lat.set_kappa(kappa)
    return lat, U


def apply_at(F, lat, src, dst, nrhs):
    """fl_apply_D on device addresses."""
    return F.lib().fl_apply_D(lat._h, ctypes.c_void_p(src), ctypes.c_void_p(dst), nrhs, 0, F.FL_DEVICE)


@pytest.mark.parametrize("dims", DIMS)
def test_round_trip_returns_every_value(F, dims):
    import torch
    lat, _ = make(F, dims, 1e-300)
    psi = S.random_spinors(dims, 3, 92)
    x = torch.from_numpy(psi).cuda()
    assert apply_at(F, lat, x.data_ptr(), x.data_ptr(), 3) == 0
    assert np.array_equal(x.cpu().numpy(), psi)
    x = torch.from_numpy(psi).cuda()
    lat.smear(x, alpha=0.0, n=1, norm=1.0)
    assert np.array_equal(x.cpu().numpy(), psi)
    lat.close()


@pytest.mark.parametrize("dims", DIMS)
def test_sites_land_where_they_belong(F, dims):
    """Against the oracle (a round trip would not see sites exchanged in both
    directions).  Tolerance: at most 100 roundings of 1.1e-16 a component of D,
    relative to the largest; a smearing step has fewer."""
    import torch
    lat, U = make(F, dims, 0.11)
    psi = S.random_spinors(dims, 3, 93)
    x = torch.from_numpy(psi).cuda()
    assert apply_at(F, lat, x.data_ptr(), x.data_ptr(), 3) == 0
    want = O.apply_D(U, psi, dims, -1, 0.11).reshape(psi.shape)
    assert np.abs(x.cpu().numpy() - want).max() <= 1e-14 * np.abs(want).max()
    want = O.smear(U, psi, dims, 1.5, 1, 1.0)
    assert np.abs(lat.smear(psi, 1.5, 1, 1.0) - want).max() <= 1e-14 * np.abs(want).max()
    lat.close()


@pytest.mark.parametrize("dims,nrhs", [((2, 2, 2, 34), 3), ((4, 4, 4, 4), 70)])
def test_fields_at_8_byte_boundaries(F, dims, nrhs):
    """Both kernels of the one-pass route, the even/odd route and smearing on
    fields one double behind a 16-byte boundary: the same bits."""
    import torch
    lat, _ = make(F, dims, 0.11)
    psi = S.random_spinors(dims, nrhs, 94)
    flat = torch.from_numpy(psi.view(np.float64).reshape(-1)).cuda()
    want = lat.apply_D(psi)
    x, y = (torch.zeros(flat.numel() + 1, dtype=torch.float64, device="cuda") for _ in range(2))
    x[1:] = flat
    assert x[1:].data_ptr() % 16 == 8
    got = lambda t: t[1:].cpu().numpy().view(np.complex128).reshape(psi.shape)
    assert apply_at(F, lat, x[1:].data_ptr(), y[1:].data_ptr(), nrhs) == 0
    assert np.array_equal(got(y), want)
    assert apply_at(F, lat, x[1:].data_ptr(), x[1:].data_ptr(), nrhs) == 0
    assert np.array_equal(got(x), want)
    want = lat.smear(psi, 1.5, 3, 2.0)
    x[1:] = flat
    assert F.lib().fl_smear(lat._h, ctypes.c_void_p(x[1:].data_ptr()), nrhs, 1.5, 3, 2.0, F.FL_DEVICE) == 0
    assert np.array_equal(got(x), want)
    lat.close()
