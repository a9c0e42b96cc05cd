// fl_corr.hip -- momentum-projected loops and the disconnected two-point
// function built from them (Sec. III, Eq. all_dis_corr):
//
//   Lp_G(p, t) = sum_x exp(+i p.x) L_G(x, t),  p = 2 pi (n_x/Lx, n_y/Ly, n_z/Lz)
//   D_AB(p, t) = (1/V_s)(1/T) sum_ti Lp_A(p, ti + t) Lp_B(-p, ti)
//
// The phase of site x for the integer vector n is the product of the three
// per-axis factors exp(2 pi i r_mu / L_mu), r_mu = (n_mu x_mu) mod L_mu,
// each evaluated once per workgroup by sincospi on the exactly reduced
// argument 2 r_mu / L_mu and kept in LDS (two complex products per site
// instead of a sine and cosine).  Sums run in FP64 in a fixed order (a
// thread's columns along z, then a wave's lanes by pairwise exchanges, then the
// four waves), so results do not depend on the launch.
#include <algorithm>
#include <cstring>
#include <type_traits>

#include "fl_host.h"

namespace {

constexpr int MAXG = 16;    // Gamma matrices per call
constexpr int BLK = 256;
constexpr int MAXAX = 1024;  // Lx + Ly + Lz: the per-axis phase tables in LDS (16 KB a momentum)
constexpr int MOMS = 4;      // momenta per workgroup of the projection (of more than one)
constexpr int MCH = 64;      // momenta, or Gamma pairs, per launch: they travel as kernel arguments

struct MomArgs {
    const double2 *L;  // [ngamma][nt][Vs]
    double2 *Lp;       // [ngamma][nmom][nt]
    int ngamma, nt, nmom, Lx, Ly, Lz, P, Vs;  // P = Lx Ly
    int k0, nk;             // momenta k0 .. k0 + nk - 1 of the call
    unsigned short mom[MCH][4];  // reduced to 0 .. L_mu - 1
};

// real and imaginary part of the product of a phase and a value
__device__ __forceinline__ double phase_re(double2 p, double2 l) { return fma(p.x, l.x, -(p.y * l.y)); }
__device__ __forceinline__ double phase_im(double2 p, double2 l) { return fma(p.x, l.y, p.y * l.x); }

// one workgroup per (timeslice, MB momenta, group of GB Gammas), in
// XCD-contiguous order with the Gamma group innermost, then the momenta: each
// XCD takes a run of timeslices, so a timeslice's loops (ngamma x V_s values)
// come from HBM once and then from that XCD's L2, once for every MB momenta.
// A thread walks along z with the phases of z and applies the phase of (x, y)
// to the column's sum.  Loads past the last Gamma or momentum repeat it; its
// sum is not stored.  The sums of a
// thread's GB x MB values over the wave halve the number of values per lane at
// every exchange: 32 doubles take 32 exchanges instead of 192.  Bound by
// instruction issue and the start of its short workgroups: 16^3x32 with 6
// Gammas and 33 momenta 37 us a call with its wait (58 with one momentum a
// workgroup, which drew 13 TB/s from L2).
// ONE: planes of up to BLK sites, one column a thread.
template <int GB, int MB, bool ONE>
__global__ __launch_bounds__(BLK) void k_momproj(MomArgs a)
{
    constexpr int NV = 2 * MB * 4;   // values of a lane, Gammas padded to 4 for the exchanges
    extern __shared__ double2 ph[];  // [MB][Lx + Ly + Lz]: exp(2 pi i n_mu x_mu / L_mu), the three axes in a row
    const int ngr = (a.ngamma + GB - 1) / GB, nkg = (a.nk + MB - 1) / MB;
    const int tile = xcd_tile(blockIdx.x, gridDim.x, 0);
    const int g0 = (tile % ngr) * GB, k0 = ((tile / ngr) % nkg) * MB, t = tile / (ngr * nkg);
    const int nL = a.Lx + a.Ly + a.Lz;
    for (int q = threadIdx.x; q < MB * nL; q += BLK) {
        const int m = q / nL, i = q - m * nL;
        const int mu = i < a.Lx ? 0 : (i < a.Lx + a.Ly ? 1 : 2);
        const int L = mu == 0 ? a.Lx : (mu == 1 ? a.Ly : a.Lz);
        const int x = i - (mu == 0 ? 0 : (mu == 1 ? a.Lx : a.Lx + a.Ly));
        const unsigned r = ((unsigned)a.mom[min(k0 + m, a.nk - 1)][mu] * (unsigned)x) % (unsigned)L;
        double sn, cs;
        sincospi(2.0 * (double)r / (double)L, &sn, &cs);
        ph[q] = make_double2(cs, sn);
    }
    __syncthreads();
    const double2 *src[GB];
#pragma unroll
    for (int j = 0; j < GB; ++j) src[j] = a.L + ((size_t)min(g0 + j, a.ngamma - 1) * a.nt + t) * a.Vs;
    double v[NV];  // [m][j][re, im]
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = 0.0;
    // planes of up to BLK sites: BLK / P threads share a column
    const int nz = a.P >= BLK ? 1 : BLK / a.P;
    const int z0 = a.P >= BLK ? 0 : (int)threadIdx.x / a.P;
    const double2 *pz = ph + a.Lx + a.Ly;
    if (z0 < nz)
        for (int xy = (int)threadIdx.x - z0 * a.P; xy < a.P; xy += BLK) {
            double own[ONE ? 1 : NV];
            double *u = ONE ? v : own;  // the column's sums with the phases of z
#pragma unroll
            for (int k = 0; k < (ONE ? 0 : NV); ++k) u[k] = 0.0;
            // two sites at a time, their terms added up first: one rounding in
            // two sites has the size of the sum
            int z = z0;
#pragma unroll 2
            for (; z + nz < a.Lz; z += 2 * nz) {
                double2 l[2][GB];
#pragma unroll
                for (int j = 0; j < GB; ++j) {
                    l[0][j] = src[j][z * a.P + xy];
                    l[1][j] = src[j][(z + nz) * a.P + xy];
                }
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    const double2 p = pz[m * nL + z], q = pz[m * nL + z + nz];
#pragma unroll
                    for (int j = 0; j < GB; ++j) {
                        double *w = u + 2 * (m * 4 + j);
                        w[0] += fma(q.x, l[1][j].x, fma(-q.y, l[1][j].y, phase_re(p, l[0][j])));
                        w[1] += fma(q.x, l[1][j].y, fma(q.y, l[1][j].x, phase_im(p, l[0][j])));
                    }
                }
            }
            if (z < a.Lz)
#pragma unroll
                for (int j = 0; j < GB; ++j) {
                    const double2 l = src[j][z * a.P + xy];
#pragma unroll
                    for (int m = 0; m < MB; ++m) {
                        const double2 p = pz[m * nL + z];
                        u[2 * (m * 4 + j)] += phase_re(p, l);
                        u[2 * (m * 4 + j) + 1] += phase_im(p, l);
                    }
                }
            const int y = xy / a.Lx, x = xy - y * a.Lx;
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                const double2 px = ph[m * nL + x], py = ph[m * nL + a.Lx + y];
                const double2 p = make_double2(phase_re(px, py), phase_im(px, py));
#pragma unroll
                for (int j = 0; j < GB; ++j) {
                    double *w = v + 2 * (m * 4 + j);
                    const double2 c = make_double2(u[2 * (m * 4 + j)], u[2 * (m * 4 + j) + 1]);
                    w[0] = (ONE ? 0.0 : w[0]) + phase_re(p, c);
                    w[1] = (ONE ? 0.0 : w[1]) + phase_im(p, c);
                }
            }
        }
    // lane l ends with the wave's sum of value (l >> 1) % NV
    const int lane = threadIdx.x % FL_WAVE, wave = threadIdx.x / FL_WAVE;
#pragma unroll
    for (int n = NV / 2; n >= 1; n /= 2) {
        const bool up = (lane & (2 * n)) != 0;
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const double mine = up ? v[k + n] : v[k], other = up ? v[k] : v[k + n];
            v[k] = mine + __shfl_xor(other, 2 * n, FL_WAVE);
        }
    }
#pragma unroll
    for (int n = FL_WAVE / 2; n > NV; n /= 2) v[0] += __shfl_xor(v[0], n, FL_WAVE);
    v[0] += __shfl_xor(v[0], 1, FL_WAVE);
    __shared__ double red[BLK / FL_WAVE][NV];
    if ((lane & 1) == 0 && (lane >> 1) < NV) red[wave][lane >> 1] = v[0];
    __syncthreads();
    // one store instruction, one value a lane, which ends the kernel
    if ((int)threadIdx.x >= NV / 2) return;
    const int m = threadIdx.x / 4, j = threadIdx.x % 4;
    static_assert(BLK == 4 * FL_WAVE, "four waves");
    const int n = 2 * threadIdx.x;
    const double2 o = make_double2((red[0][n] + red[1][n]) + (red[2][n] + red[3][n]),
                                   (red[0][n + 1] + red[1][n + 1]) + (red[2][n + 1] + red[3][n + 1]));
    if (k0 + m < a.nk && j < GB && g0 + j < a.ngamma)
        a.Lp[((size_t)(g0 + j) * a.nmom + a.k0 + k0 + m) * a.nt + t] = o;
}

struct CorrArgs {
    const double2 *Lp1, *Lp2;  // [ngamma][nmom][T]
    double2 *D;                // [npair][nmom][T], from the launch's first pair
    int nmom, T, npair;        // npair: pairs of this launch
    double norm;  // 1 / (V_s T)
    int pairs[MCH][2];
};

// one thread per (pair, momentum, separation), summing the source times in order
__global__ __launch_bounds__(BLK) void k_dcorr(CorrArgs a)
{
    const long long id = blockIdx.x * (long long)BLK + threadIdx.x;
    if (id >= (long long)a.npair * a.nmom * a.T) return;
    const int t = (int)(id % a.T), k = (int)((id / a.T) % a.nmom), j = (int)(id / ((long long)a.T * a.nmom));
    const double2 *f = a.Lp1 + ((size_t)a.pairs[j][0] * a.nmom + k) * a.T;
    const double2 *h = a.Lp2 + ((size_t)a.pairs[j][1] * a.nmom + k) * a.T;
    double re = 0.0, im = 0.0;
    int tf = t;  // (ti + t) mod T
#pragma unroll 8
    for (int ti = 0; ti < a.T; ++ti) {
        const double2 u = f[tf], v = h[ti];
        tf = tf + 1 == a.T ? 0 : tf + 1;
        re += u.x * v.x - u.y * v.y;
        im += u.x * v.y + u.y * v.x;
    }
    a.D[id] = make_double2(re * a.norm, im * a.norm);
}

unsigned blocks(long long n) { return (unsigned)((n + BLK - 1) / BLK); }

}  // namespace

bool momproj_fits(const int L4[4]) { return L4[0] + L4[1] + L4[2] <= MAXAX; }

void launch_momproj(const double2 *L, double2 *Lp, const int *mom, int ngamma, int nt, int nmom, const int L4[4],
                    hipStream_t s)
{
    MomArgs a;
    a.L = L;
    a.Lp = Lp;
    a.ngamma = ngamma;
    a.nt = nt;
    a.nmom = nmom;
    a.Lx = L4[0];
    a.Ly = L4[1];
    a.Lz = L4[2];
    a.P = L4[0] * L4[1];
    a.Vs = a.P * L4[2];
    // Gammas per workgroup: as few groups of at most 4 as cover them, evenly
    const int ngr = (ngamma + 3) / 4, gb = (ngamma + ngr - 1) / ngr;
    // up to 512 workgroups (two per CU) a momentum has one to itself: four in one
    // would leave CUs idle and, below four, compute repeats.  Calls with four and
    // with one: 24^3x16, 16 Gammas, 2 momenta 52.7 and 39.3 us, 16^3x32, 6 Gammas,
    // 5 momenta 29.0 and 27.0; above, 16^3x32, 6 Gammas, 33 momenta 37 and 58
    const int mb = (long long)nt * ngr * nmom <= 512 ? 1 : MOMS;
    const size_t shm = (size_t)mb * (L4[0] + L4[1] + L4[2]) * sizeof(double2);
    for (a.k0 = 0; a.k0 < nmom; a.k0 += MCH) {
        a.nk = std::min(MCH, nmom - a.k0);
        for (int k = 0; k < a.nk; ++k)
            for (int mu = 0; mu < 3; ++mu) {
                const int r = mom[3 * (size_t)(a.k0 + k) + mu] % L4[mu];
                a.mom[k][mu] = (unsigned short)(r < 0 ? r + L4[mu] : r);
            }
        const dim3 grid((unsigned)(nt * ((a.nk + mb - 1) / mb) * ngr)), block(BLK);
        auto momenta = [&](auto n, auto m) {
            constexpr int GB = decltype(n)::value, MB = decltype(m)::value;
            if (a.P <= BLK)
                hipLaunchKernelGGL((k_momproj<GB, MB, true>), grid, block, shm, s, a);
            else
                hipLaunchKernelGGL((k_momproj<GB, MB, false>), grid, block, shm, s, a);
        };
        auto launch = [&](auto n) {
            if (mb == 1)
                momenta(n, std::integral_constant<int, 1>());
            else
                momenta(n, std::integral_constant<int, MOMS>());
        };
        switch (gb) {
        case 1: launch(std::integral_constant<int, 1>()); break;
        case 2: launch(std::integral_constant<int, 2>()); break;
        case 3: launch(std::integral_constant<int, 3>()); break;
        default: launch(std::integral_constant<int, 4>()); break;
        }
    }
}

fl_status fl_momentum_project(fl_ctx *c, const double *L, int ngamma, int nt, const int *mom, int nmom, double *Lp,
                              fl_where where)
{
    if (!c) return set_err(nullptr, FL_ERR_ARG, "ctx is NULL");
    if (ngamma < 1 || ngamma > MAXG || nt < 1 || nmom < 1 || !L || !Lp || !mom)
        return set_err(c, FL_ERR_ARG, "need 1..16 Gammas, nt >= 1, nmom >= 1 and non-NULL arrays");
    if (!momproj_fits(c->L)) return set_err(c, FL_ERR_ARG, "momentum projection needs Lx + Ly + Lz <= 1024");
    if (where != FL_HOST && where != FL_DEVICE) return set_err(c, FL_ERR_ARG, "bad `where`");
    hipSetDevice(c->device);
    const int Vs = c->L[0] * c->L[1] * c->L[2];
    const size_t nin = (size_t)ngamma * nt * Vs * sizeof(double2), nout = (size_t)ngamma * nmom * nt * sizeof(double2);
    fl_status e;
    const double2 *din = (const double2 *)L;
    double2 *dout = (double2 *)Lp;
    if (where == FL_HOST) {
        double2 *bi = (double2 *)ws_get(c, WS_CORR_A, nin), *bo = (double2 *)ws_get(c, WS_CORR_OUT, nout);
        if (!bi || !bo) return set_err(c, FL_ERR_NOMEM, "device allocation failed");
        if ((e = hip_check(c, hipMemcpyAsync(bi, L, nin, hipMemcpyHostToDevice, c->stream), "upload loops"))) return e;
        din = bi;
        dout = bo;
    }
    launch_momproj(din, dout, mom, ngamma, nt, nmom, c->L, c->stream);
    if ((e = hip_check(c, hipGetLastError(), "momentum projection"))) return e;
    if (where == FL_HOST &&
        (e = hip_check(c, hipMemcpyAsync(Lp, dout, nout, hipMemcpyDeviceToHost, c->stream), "download")))
        return e;
    return hip_check(c, hipStreamSynchronize(c->stream), "momentum projection");
}

fl_status fl_disconnected_corr(fl_ctx *c, const double *Lp1, const double *Lp2, int ngamma, int nmom,
                               const int *pairs, int npair, double *D, fl_where where)
{
    if (!c) return set_err(nullptr, FL_ERR_ARG, "ctx is NULL");
    if (ngamma < 1 || nmom < 1 || npair < 1 || !Lp1 || !Lp2 || !pairs || !D)
        return set_err(c, FL_ERR_ARG, "need ngamma, nmom, npair >= 1 and non-NULL arrays");
    for (int j = 0; j < 2 * npair; ++j)
        if (pairs[j] < 0 || pairs[j] >= ngamma) return set_err(c, FL_ERR_ARG, "pair index outside 0..ngamma-1");
    if (where != FL_HOST && where != FL_DEVICE) return set_err(c, FL_ERR_ARG, "bad `where`");
    hipSetDevice(c->device);
    const int T = c->L[3], Vs = c->L[0] * c->L[1] * c->L[2];
    const size_t nin = (size_t)ngamma * nmom * T * sizeof(double2), nout = (size_t)npair * nmom * T * sizeof(double2);
    fl_status e;
    const double2 *a1 = (const double2 *)Lp1, *a2 = (const double2 *)Lp2;
    double2 *o = (double2 *)D;
    if (where == FL_HOST) {
        double2 *b1 = (double2 *)ws_get(c, WS_CORR_A, nin), *b2 = (double2 *)ws_get(c, WS_CORR_B, nin);
        double2 *bo = (double2 *)ws_get(c, WS_CORR_OUT, nout);
        if (!b1 || !b2 || !bo) return set_err(c, FL_ERR_NOMEM, "device allocation failed");
        if ((e = hip_check(c, hipMemcpyAsync(b1, Lp1, nin, hipMemcpyHostToDevice, c->stream), "upload")) ||
            (e = hip_check(c, hipMemcpyAsync(b2, Lp2, nin, hipMemcpyHostToDevice, c->stream), "upload")))
            return e;
        a1 = b1;
        a2 = b2;
        o = bo;
    }
    CorrArgs a;
    a.Lp1 = a1;
    a.Lp2 = a2;
    a.nmom = nmom;
    a.T = T;
    a.norm = 1.0 / ((double)Vs * T);
    for (int j0 = 0; j0 < npair; j0 += MCH) {
        a.npair = std::min(MCH, npair - j0);
        a.D = o + (size_t)j0 * nmom * T;
        std::memcpy(a.pairs, pairs + 2 * (size_t)j0, sizeof(int) * 2 * a.npair);
        hipLaunchKernelGGL(k_dcorr, dim3(blocks((long long)a.npair * nmom * T)), dim3(BLK), 0, c->stream, a);
    }
    if ((e = hip_check(c, hipGetLastError(), "disconnected correlator"))) return e;
    if (where == FL_HOST &&
        (e = hip_check(c, hipMemcpyAsync(D, o, nout, hipMemcpyDeviceToHost, c->stream), "download")))
        return e;
    return hip_check(c, hipStreamSynchronize(c->stream), "disconnected correlator");
}
