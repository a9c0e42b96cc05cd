"""GPU parity of the momentum projection and the disconnected two-point
function (Sec. III, Eq. all_dis_corr) against the oracle, on random loops and
on loops the library computes, at 4^3x8, 8^3x16 and 16^3x32."""
import numpy as np
import pytest

import oracle as O
import synth_inputs as S

pytestmark = pytest.mark.gpu

GAMMAS = [0, 15, 1, 2, 4, 8]
MOM = [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1), (-1, 0, 0), (1, 1, 0), (1, -1, 1), (2, 0, -1)]


@pytest.fixture(scope="module")
def F():
    import paper_1108_2473_amd as fl
    fl.lib()
    return fl


def _rand(shape, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


@pytest.mark.parametrize("dims", [(4, 4, 4, 8), (8, 8, 8, 16), (16, 16, 16, 32), (6, 4, 2, 4)])
def test_projection_and_correlator_random(F, dims):
    Vs, T = dims[0] * dims[1] * dims[2], dims[3]
    lat = F.Lattice(dims, -1)
    L1, L2 = _rand((6, T, Vs), 11), _rand((6, T, Vs), 12)
    neg = [(-a, -b, -c) for a, b, c in MOM]
    P1, P2 = lat.momentum_project(L1, MOM), lat.momentum_project(L2, neg)
    W1, W2 = O.momentum_project(L1, dims, MOM), O.momentum_project(L2, dims, neg)
    scale = np.sqrt(Vs)  # size of a sum of Vs unit-variance terms
    assert np.abs(P1 - W1).max() <= 1e-12 * scale
    assert np.abs(P2 - W2).max() <= 1e-12 * scale
    pairs = [(0, 0), (1, 1), (0, 1), (2, 5)]
    D = lat.disconnected_corr(P1, P2, pairs)
    Dw = O.disconnected_correlator(W1, W2, Vs, pairs)
    assert np.abs(D - Dw).max() <= 1e-12 * np.abs(Dw).max()
    lat.close()


@pytest.mark.parametrize("ng", [1, 3, 4, 5, 16])
def test_projection_gamma_counts(F, ng):
    """The projection handles the Gamma matrices in groups of four per
    workgroup: one, a partial group, exactly one group, a group and one more,
    and the maximum of sixteen, on a lattice with unequal spatial extents."""
    dims = (6, 4, 8, 4)
    Vs, T = 6 * 4 * 8, 4
    lat = F.Lattice(dims, -1)
    L = _rand((ng, T, Vs), 20 + ng)
    P = lat.momentum_project(L, MOM)
    assert P.shape == (ng, len(MOM), T)
    assert np.abs(P - O.momentum_project(L, dims, MOM)).max() <= 1e-12 * np.sqrt(Vs)
    lat.close()


@pytest.mark.parametrize("dims,nmom", [((18, 16, 4, 2), 3), ((2, 2, 4, 2), 5), ((6, 10, 2, 4), 65), ((16, 16, 2, 2), 131)])
def test_projection_planes_and_many_momenta(F, dims, nmom):
    """Planes larger than a workgroup, of one site per thread, dividing it and
    not; more momenta and pairs than one launch takes; integer momenta beyond
    the lattice's extents on either side."""
    Vs, T = dims[0] * dims[1] * dims[2], dims[3]
    mom = [((7 * k) % 41 - 20, (5 * k) % 37 - 18, (3 * k) % 31 - 15) for k in range(nmom)]
    lat = F.Lattice(dims, -1)
    L = _rand((2, T, Vs), 15)
    P = lat.momentum_project(L, mom)
    W = O.momentum_project(L, dims, mom)
    assert np.abs(P - W).max() <= 1e-12 * np.sqrt(Vs)
    pairs = [(k % 2, (k // 2) % 2) for k in range(nmom)]
    D = lat.disconnected_corr(P, P, pairs)
    Dw = O.disconnected_correlator(W, W, Vs, pairs)
    assert np.abs(D - Dw).max() <= 1e-12 * np.abs(Dw).max()
    lat.close()


def test_device_arrays_and_argument_checks(F):
    import torch
    dims = (4, 4, 4, 8)
    lat = F.Lattice(dims, -1)
    L = _rand((2, 8, 64), 13)
    Pd = lat.momentum_project(torch.from_numpy(L).cuda(), MOM)
    assert Pd.is_cuda
    assert np.abs(Pd.cpu().numpy() - O.momentum_project(L, dims, MOM)).max() <= 1e-12 * 8
    with pytest.raises(F.FloopError):
        lat.disconnected_corr(Pd, Pd, [(0, 2)])  # Gamma index out of range
    lat.close()
    # spatial extents beyond the projection's phase tables (Lx + Ly + Lz <= 1024)
    wide = F.Lattice((1022, 2, 2, 2), -1)
    with pytest.raises(F.FloopError):
        wide.momentum_project(_rand((1, 2, 1022 * 4), 14), MOM)
    wide.close()


def test_exact_loop_correlator_4x4x4x8(F):
    """Exact loops computed by the library on every timeslice of a 4^3x8
    lattice (eps 0.3, kappa 0.10), projected at zero and unit momenta and
    correlated, against the oracle's own exact loops put through the oracle's
    projection and correlator."""
    W = S.WORKLOADS["exact_4x4x4x4"]
    dims = (4, 4, 4, 8)
    U = S.random_links(dims, W["eps"], W["link_seed"])
    lat = F.Lattice(dims, -1)
    lat.set_gauge(U)
    lat.set_kappa(W["kappa"])
    L = lat.loops_exact(list(range(8)), GAMMAS, F.SolverParams(tol=1e-12))
    Lo = O.loops_exact(U, dims, -1, W["kappa"], list(range(8)), GAMMAS, tol=1e-14)
    mom = [(0, 0, 0), (1, 0, 0), (0, 0, 1)]
    neg = [(-a, -b, -c) for a, b, c in mom]
    D = lat.disconnected_corr(lat.momentum_project(L, mom), lat.momentum_project(L, neg), [(1, 1), (0, 0)])
    Dw = O.disconnected_correlator(O.momentum_project(Lo, dims, mom), O.momentum_project(Lo, dims, neg), 64,
                                   [(1, 1), (0, 0)])
    assert np.abs(D - Dw).max() <= 1e-9 * np.abs(Dw).max()
    # gamma_5 loops are real for exact loops, so the g5-g5 zero-momentum correlator is real
    assert np.abs(D[0, 0].imag).max() <= 1e-9 * np.abs(D[0, 0]).max()
    lat.close()


@pytest.mark.parametrize("dims", [(1020, 2, 2, 2), (2, 1020, 2, 2), (2, 2, 1020, 2), (512, 510, 2, 2)])
def test_projection_largest_extents(F, dims):
    """Lx + Ly + Lz = 1024: phase tables of 64 KB for the four momenta of a workgroup."""
    Vs, T = dims[0] * dims[1] * dims[2], dims[3]
    mom = [(0, 0, 0), (1, -1, 1), (511, 3, -2), (-509, 1, 0), (7, 513, 1)]
    mom += [(3 * k, k, 5 * k) for k in range(255)]  # enough for workgroups of four momenta
    lat = F.Lattice(dims, -1)
    L = _rand((2, T, Vs), 16)
    P = lat.momentum_project(L, mom)
    lat.close()
    # the oracle takes the phases' arguments as they are, with an error that grows
    # with n x: the same momenta within half the extents
    red = [tuple((n + e // 2) % e - e // 2 for n, e in zip(k, dims)) for k in mom]
    W = O.momentum_project(L, dims, red)
    assert np.abs(P - W).max() <= 1e-12 * np.sqrt(Vs)


@pytest.mark.parametrize("nmom", [5, 300])
def test_projection_rounds_once_per_site(F, nmom):
    """Accuracy of a thread's sum over 480 sites along z: no worse than a plain FP64
    evaluation in the same order, which rounds each site's term once into the
    sum.  Two roundings per site would be 2 ** 0.5 = 1.41 times as far off; 1.2
    separates them."""
    dims, mom = (16, 16, 480, 2), [(0, 0, 1), (1, 0, 3), (-3, 5, 7), (2, 7, -100), (1, -1, 1)]
    Vs, T = dims[0] * dims[1] * dims[2], dims[3]
    L = _rand((3, T, Vs), 17)
    lat = F.Lattice(dims, -1)
    P = lat.momentum_project(L, mom + [(0, 0, k) for k in range(nmom - len(mom))])
    lat.close()
    ld = np.longdouble
    two_pi = 2 * ld("3.14159265358979323846264338327950288")
    f = L.reshape(3, T, dims[2], dims[1], dims[0])
    err = np.zeros(2)
    for k, n in enumerate(mom):
        ph = []
        for mu in range(3):
            a = two_pi * ((n[mu] * np.arange(dims[mu])) % dims[mu]).astype(ld) / dims[mu]
            ph.append(np.cos(a) + 1j * np.sin(a))
        exact = f.astype(np.clongdouble)
        for p in ph:
            exact = (exact * p).sum(-1)
        x, y, z = (p.astype(np.complex128) for p in ph)
        xy = x[None, :] * y[:, None]
        acc = np.zeros(f.shape[:2] + xy.shape, complex)
        for i in range(dims[2]):
            acc += f[:, :, i] * (xy * z[i])
        err += [(np.abs(v.astype(np.clongdouble) - exact) ** 2).sum().astype(float)
                for v in (P[:, k], acc.reshape(acc.shape[:2] + (-1,)).sum(-1))]
    assert err[0] <= 1.2 ** 2 * err[1]


@pytest.mark.parametrize("dims", [(18, 16, 4, 40), (2, 2, 4, 40), (6, 10, 2, 40), (16, 16, 2, 40), (4, 4, 6, 40)])
@pytest.mark.parametrize("ng,nmom", [(1, 1), (1, 12), (1, 13), (3, 66), (5, 6), (5, 7), (16, 14)])
def test_projection_momenta_per_workgroup(F, dims, ng, nmom):
    """Both sides of the 512 workgroups up to which each momentum has its own,
    and remainders of the groups of four momenta and of up to four Gammas, on
    planes of one and of several columns a thread; odd and even numbers of
    sites a thread."""
    Vs, T = dims[0] * dims[1] * dims[2], dims[3]
    mom = [((7 * k) % 41 - 20, (5 * k) % 37 - 18, (3 * k) % 31 - 15) for k in range(nmom)]
    lat = F.Lattice(dims, -1)
    L = _rand((ng, T, Vs), 18)
    P = lat.momentum_project(L, mom)
    W = O.momentum_project(L, dims, mom)
    lat.close()
    assert np.abs(P - W).max() <= 1e-12 * np.sqrt(Vs)
