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
// instead of a sine and cosine).  Sums run in FP64 in a fixed order
// (per-thread partial sums over a strided site range, then a fixed tree in
// LDS), so results do not depend on the launch.
#include <algorithm>
#include <cstring>

#include "fl_host.h"

namespace {

constexpr int MAXG = 16;    // Gamma matrices per call
constexpr int BLK = 256;
constexpr int MAXAX = 1024;  // Lx + Ly + Lz: the per-axis phase tables in LDS (16 KB a momentum)
constexpr int MB = 4;        // momenta per workgroup of the projection
constexpr int MCH = 64;      // momenta, or Gamma pairs, per launch: they travel as kernel arguments

struct MomArgs {
    const double2 *L;  // [ngamma][nt][Vs]
    double2 *Lp;       // [ngamma][nmom][nt]
    int ngamma, nt, nmom, Lx, Ly, Lz, P, Vs;  // P = Lx Ly
    int k0, nk;             // momenta k0 .. k0 + nk - 1 of the call
    unsigned short mom[MCH][4];  // reduced to 0 .. L_mu - 1
};

// one workgroup per (timeslice, MB momenta, group of GB Gammas), in
// XCD-contiguous order with the Gamma group innermost, then the momenta: each
// XCD takes a run of timeslices, so a timeslice's loops (ngamma x V_s values)
// come from HBM once and then from that XCD's L2, once for every MB momenta.
// A thread keeps one (x, y) and its phase and walks along z.  Loads past the
// last Gamma or momentum repeat it; its sum is not stored.  The sums of a
// thread's GB x MB values over the wave halve the number of values per lane at
// every exchange: 32 doubles take 32 exchanges instead of 192.  Bound by
// instruction issue and the start of its short workgroups: 16^3x32 with 6
// Gammas and 33 momenta 15.7 us (31.5 us with one momentum a workgroup, which
// drew 13 TB/s from L2; 21.7 us with three table reads a site).
template <int GB>
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
    if (z0 < nz)
        for (int xy = (int)threadIdx.x - z0 * a.P; xy < a.P; xy += BLK) {
            const int y = xy / a.Lx, x = xy - y * a.Lx;
            double2 pxy[MB];
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                const double2 px = ph[m * nL + x], py = ph[m * nL + a.Lx + y];
                pxy[m] = make_double2(px.x * py.x - px.y * py.y, px.x * py.y + px.y * py.x);
            }
            const double2 *pz = ph + a.Lx + a.Ly;
#pragma unroll 4
            for (int z = z0; z < a.Lz; z += nz) {
                double2 l[GB];
#pragma unroll
                for (int j = 0; j < GB; ++j) l[j] = src[j][z * a.P + xy];
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    const double2 q = pz[m * nL + z];
                    const double cs = pxy[m].x * q.x - pxy[m].y * q.y, sn = pxy[m].x * q.y + pxy[m].y * q.x;
#pragma unroll
                    for (int j = 0; j < GB; ++j) {
                        double *w = v + 2 * (m * 4 + j);
                        w[0] = fma(cs, l[j].x, fma(-sn, l[j].y, w[0]));
                        w[1] = fma(cs, l[j].y, fma(sn, l[j].x, w[1]));
                    }
                }
            }
        }
    // lane l ends with the wave's sum of value l >> 1
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
    v[0] += __shfl_xor(v[0], 1, FL_WAVE);
    __shared__ double red[BLK / FL_WAVE][NV];
    if ((lane & 1) == 0) red[wave][lane >> 1] = v[0];
    __syncthreads();
    // one store instruction, one value a lane, which ends the kernel
    if ((int)threadIdx.x >= NV / 2) return;
    const int m = threadIdx.x / 4, j = threadIdx.x % 4;
    double2 o = make_double2(0.0, 0.0);
#pragma unroll
    for (int w = 0; w < BLK / FL_WAVE; ++w) {
        o.x += red[w][2 * threadIdx.x];
        o.y += red[w][2 * threadIdx.x + 1];
    }
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
    const size_t shm = (size_t)MB * (L4[0] + L4[1] + L4[2]) * sizeof(double2);
    // Gammas per workgroup: as few groups of at most 4 as cover them, evenly
    const int ngr = (ngamma + 3) / 4, gb = (ngamma + ngr - 1) / ngr;
    for (a.k0 = 0; a.k0 < nmom; a.k0 += MCH) {
        a.nk = std::min(MCH, nmom - a.k0);
        for (int k = 0; k < a.nk; ++k)
            for (int mu = 0; mu < 3; ++mu) {
                const int r = mom[3 * (size_t)(a.k0 + k) + mu] % L4[mu];
                a.mom[k][mu] = (unsigned short)(r < 0 ? r + L4[mu] : r);
            }
        const dim3 grid((unsigned)(nt * ((a.nk + MB - 1) / MB) * ngr)), block(BLK);
        switch (gb) {
        case 1: hipLaunchKernelGGL(k_momproj<1>, grid, block, shm, s, a); break;
        case 2: hipLaunchKernelGGL(k_momproj<2>, grid, block, shm, s, a); break;
        case 3: hipLaunchKernelGGL(k_momproj<3>, grid, block, shm, s, a); break;
        default: hipLaunchKernelGGL(k_momproj<4>, grid, block, shm, s, a); break;
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
