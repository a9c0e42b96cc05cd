// fl_apply.hip -- the Wilson-Dirac operator on FP64 fields in the caller's
// layout: one pass from the canonical input to the canonical output.
//
// The even/odd route to the same result converts the input, applies one hop
// per parity and converts back: four launches and three times the traffic of
// the two fields (16^3x32, 12 right-hand sides: 534 us; here 291, with the
// whole call's 302 MB read and 302 MB written once at 5.6 TB/s 110).  Here a
// wave computes 64 consecutive sites of one right-hand side, both parities.
// What bounds it is the traffic behind L2: neighbours in t, and the FP64 links
// once for every 4 right-hand sides.
#include <type_traits>

#include "fl_host.h"
#include "fl_stencil.h"

namespace {

constexpr int FA_RT = 4;   // right-hand sides (waves) per workgroup
constexpr int FA_ST = 13;  // 16-byte words per site in LDS, odd against bank conflicts

struct FullSite {
    int par, cb;       // parity and checkerboard index
    int nb[8];         // lexicographic neighbours, forward and backward of each direction
    bool tlast, tfirst;
};

__device__ __forceinline__ FullSite full_site(const LatGeom &g, int i)
{
    FullSite s;
    const Coord c = cb_coords(g, 0, i >> 1);
    const int X = g.L[0], Y = g.L[1], Z = g.L[2], x = i - c.rest * X;
    s.par = (x + c.y + c.z + c.t) & 1;
    s.cb = i >> 1;
    s.nb[0] = x + 1 == X ? i + 1 - X : i + 1;
    s.nb[1] = x == 0 ? i - 1 + X : i - 1;
    s.nb[2] = c.y + 1 == Y ? i + X - X * Y : i + X;
    s.nb[3] = c.y == 0 ? i - X + X * Y : i - X;
    s.nb[4] = c.z + 1 == Z ? i + X * Y - X * Y * Z : i + X * Y;
    s.nb[5] = c.z == 0 ? i - X * Y + X * Y * Z : i - X * Y;
    const int W = X * Y * Z, V = 2 * g.Vh;
    s.tlast = c.t + 1 == g.L[3];
    s.tfirst = c.t == 0;
    s.nb[6] = s.tlast ? i + W - V : i + W;
    s.nb[7] = s.tfirst ? i - W + V : i - W;
    return s;
}

// The 64 spinors of a wave's neighbours pass between memory and the lanes in
// rows: lane l holds the 16-byte words q = 64 k + l (k = 0 .. 11) of the 768,
// word q % 12 of the spinor of lane q / 12.  A row's loads are whole lines (a
// lane reading its own 192 bytes touches 64 lines per load, evicted from the
// 32 KB L1 before their next word is read: 12 right-hand sides on 16^3x32
// 435 us).  64 k = 12 * 16 (k / 3) + 64 (k % 3): three patterns.
struct Rows {
    int s[3], w[3];  // spinor and word of k = 0, 1, 2; spinor + 16 for each 3 more
    int lane;
};

__device__ __forceinline__ Rows make_rows()
{
    Rows r;
    r.lane = threadIdx.x % FL_WAVE;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        r.s[m] = (64 * m + r.lane) / 12;
        r.w[m] = 64 * m + r.lane - 12 * r.s[m];
    }
    return r;
}

__device__ __forceinline__ void rows_load(const Buf &in, const Rows &r, int site, v4f v[12])
{
    const int off = site * 192;
#pragma unroll
    for (int k = 0; k < 12; ++k)
        v[k] = buf_ld16(in, __shfl(off, r.s[k % 3] + 16 * (k / 3), FL_WAVE) + 16 * r.w[k % 3], 0);
}

__device__ __forceinline__ void rows_put(v4f *sh, const Rows &r, const v4f v[12])
{
#pragma unroll
    for (int k = 0; k < 12; ++k) sh[(r.s[k % 3] + 16 * (k / 3)) * FA_ST + r.w[k % 3]] = v[k];
    wave_sync();
}

// link of direction slot D
template <int D>
__device__ __forceinline__ void full_link(const Buf &gauge, const LatGeom &g, const FullSite &s, double2 v[9])
{
    typedef LinkF64R18 LK;
    const int lp = (D & 1) ? 1 - s.par : s.par;
    const int voff = (((D & 1) ? s.nb[D] >> 1 : s.cb) + lp * LK::NC * g.Vh) * LK::ESZ;
#pragma unroll
    for (int c = 0; c < LK::NC; ++c) v[c] = LK::buf_get(gauge, voff, ((D >> 1) * 2 * LK::NC + c) * g.Vh * LK::ESZ);
}

template <int D, bool DAG>
__device__ __forceinline__ void full_hop(const Buf &in, const Buf &gauge, const LatGeom &g, const FullSite &s,
                                         const Rows &r, v4f *sh, v4f row[12], cx<double> acc[12])
{
    constexpr int MU = D >> 1;
    constexpr int SGN = (D & 1) ? (DAG ? -1 : 1) : (DAG ? 1 : -1);
    cx<double> psi[12], h[6], w[6], U[3][3];
    double2 lv[9];
    rows_put(sh, r, row);
    if constexpr (D < 7) rows_load(in, r, s.nb[D + 1], row);
    full_link<D>(gauge, g, s, lv);
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const double2 d = v4f_to_d2(sh[r.lane * FA_ST + k]);
        psi[k] = cx<double>{d.x, d.y};
    }
    wave_sync();
    LinkF64R18::unpack(lv, U);
    project<MU, SGN>(psi, h);
    if constexpr (D & 1)
        link_adj_mul(U, h, w);
    else
        link_mul(U, h, w);
    double f = 1.0;
    if constexpr (D == 6) f = s.tlast ? (double)g.bc_t : 1.0;
    if constexpr (D == 7) f = s.tfirst ? (double)g.bc_t : 1.0;
    accumulate_scaled<MU, SGN>(acc, w, f);
}

// psi - kappa acc of a wave's sites, in rows
__device__ __forceinline__ void store_canon(const Buf &in, const Rows &r, double *out, int i0, int V, double kappa,
                                            const cx<double> acc[12], v4f *sh)
{
    v4f v[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = buf_ld16(in, i0 * 192 + (k * FL_WAVE + r.lane) * 16, 0);
#pragma unroll
    for (int k = 0; k < 12; ++k) sh[r.lane * FA_ST + k] = d2_to_v4f(double2{acc[k].re, acc[k].im});
    wave_sync();
#pragma unroll
    for (int k = 0; k < 12; ++k) {
        const double2 d = v4f_to_d2(sh[(r.s[k % 3] + 16 * (k / 3)) * FA_ST + r.w[k % 3]]), p = v4f_to_d2(v[k]);
        v[k] = d2_to_v4f(double2{fma(-kappa, d.x, p.x), fma(-kappa, d.y, p.y)});
    }
    v4f *dst = (v4f *)out + (size_t)i0 * 12;
    if (i0 + FL_WAVE <= V) {
        v4f *p[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) p[k] = dst + k * FL_WAVE + r.lane;
        store_fence_begin();
#pragma unroll
        for (int k = 0; k < 12; ++k) __builtin_nontemporal_store(v[k], p[k]);
        store_drain();
    } else {
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            const int q = k * FL_WAVE + r.lane;
            if (q < 12 * (V - i0)) dst[q] = v[k];
            store_drain();  // the lattice's last, partial block: one store at a time
        }
    }
}

// The order of the 64-site blocks: sheets of FA_TB timeslices by FA_CH blocks, so
// that the blocks in flight on an XCD (about 64) share their z and t
// neighbours in its L2; right-hand sides inside, sharing the links.  Lattices
// whose timeslice is no multiple of 64 sites go block by block.  16^3x32: 4
// right-hand sides 120 -> 104 us, 12 321 -> 291, 24 610 -> 569; sheets of 2 x 32
// blocks 308, 8 x 8 290, 16 x 4 333 (12 right-hand sides).
constexpr int FA_TB = 4, FA_CH = 8;
__device__ __forceinline__ int plane_block(const LatGeom &g, int b, int nblk)
{
    const int T = g.L[3], S = nblk / T;
    if (S * T != nblk || S * FL_WAVE * T != 2 * g.Vh) return b;
    const int tb = b / (FA_TB * S), tn = min(FA_TB, T - FA_TB * tb), r = b - tb * FA_TB * S;
    const int c = r / (FA_CH * tn), cn = min(FA_CH, S - c * FA_CH), r2 = r - c * FA_CH * tn, t = r2 / cn;
    return (FA_TB * tb + t) * S + c * FA_CH + r2 - t * cn;
}

template <bool DAG>
__global__ __launch_bounds__(FL_WAVE *FA_RT, 2) void k_apply_full(const double *in, double *out, const void *links,
                                                                  LatGeom g, int nrhs, int RT, int nblk, double kappa)
{
    __shared__ v4f shm[FA_RT][FL_WAVE * FA_ST];
    const int tile = xcd_tile(blockIdx.x, gridDim.x, 0), nrb = (nrhs + RT - 1) / RT;
    const int q = tile / nrb, rb = tile - q * nrb, i0 = plane_block(g, q, nblk) * FL_WAVE;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / FL_WAVE), rhs = rb * RT + wave;
    if (rhs >= nrhs) return;
    const int V = 2 * g.Vh, i = min(i0 + (int)(threadIdx.x % FL_WAVE), V - 1);
    const FullSite s = full_site(g, i);
    const Rows r = make_rows();
    const Buf b = make_buf(in + (size_t)rhs * V * 24, (unsigned)V * 192u);
    const Buf gauge = make_buf(links, 8u * LinkF64R18::BYTES * (unsigned)g.Vh);
    v4f *sh = shm[wave], row[12];
    rows_load(b, r, s.nb[0], row);
    cx<double> acc[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = cx<double>{0.0, 0.0};
    full_hop<0, DAG>(b, gauge, g, s, r, sh, row, acc);
    full_hop<1, DAG>(b, gauge, g, s, r, sh, row, acc);
    full_hop<2, DAG>(b, gauge, g, s, r, sh, row, acc);
    full_hop<3, DAG>(b, gauge, g, s, r, sh, row, acc);
    full_hop<4, DAG>(b, gauge, g, s, r, sh, row, acc);
    full_hop<5, DAG>(b, gauge, g, s, r, sh, row, acc);
    full_hop<6, DAG>(b, gauge, g, s, r, sh, row, acc);
    full_hop<7, DAG>(b, gauge, g, s, r, sh, row, acc);
    store_canon(b, r, out + (size_t)rhs * V * 24, i0, V, kappa, acc, sh);
}

// Few blocks: a wave per direction, as in the hop of small grids; a wave's
// chain of eight neighbour loads becomes one.
template <bool DAG>
__global__ __launch_bounds__(8 * FL_WAVE) void k_apply_split(const double *in, double *out, const void *links,
                                                            LatGeom g, int nblk, double kappa)
{
    __shared__ v4f shm[8 * 6 * FL_WAVE + 32];  // the products, then the result's FL_WAVE * FA_ST words
    const int rhs = blockIdx.x / nblk, i0 = (blockIdx.x - rhs * nblk) * FL_WAVE;
    const int d = __builtin_amdgcn_readfirstlane(threadIdx.x / FL_WAVE), lane = threadIdx.x % FL_WAVE;
    const int V = 2 * g.Vh, i = min(i0 + lane, V - 1);
    const FullSite s = full_site(g, i);
    const Buf b = make_buf(in + (size_t)rhs * V * 24, (unsigned)V * 192u);
    const Buf gauge = make_buf(links, 8u * LinkF64R18::BYTES * (unsigned)g.Vh);
    auto product = [&](auto dd) {
        constexpr int D = decltype(dd)::value, MU = D >> 1;
        constexpr int SGN = (D & 1) ? (DAG ? -1 : 1) : (DAG ? 1 : -1);
        cx<double> psi[12], h[6], w[6], U[3][3];
        double2 lv[9];
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            const double2 q = v4f_to_d2(buf_ld16(b, s.nb[D] * 192, 16 * k));
            psi[k] = cx<double>{q.x, q.y};
        }
        full_link<D>(gauge, g, s, lv);
        LinkF64R18::unpack(lv, U);
        project<MU, SGN>(psi, h);
        if constexpr (D & 1)
            link_adj_mul(U, h, w);
        else
            link_mul(U, h, w);
#pragma unroll
        for (int k = 0; k < 6; ++k) shm[(D * 6 + k) * FL_WAVE + lane] = d2_to_v4f(double2{w[k].re, w[k].im});
    };
    switch (d) {
    case 0: product(std::integral_constant<int, 0>()); break;
    case 1: product(std::integral_constant<int, 1>()); break;
    case 2: product(std::integral_constant<int, 2>()); break;
    case 3: product(std::integral_constant<int, 3>()); break;
    case 4: product(std::integral_constant<int, 4>()); break;
    case 5: product(std::integral_constant<int, 5>()); break;
    case 6: product(std::integral_constant<int, 6>()); break;
    default: product(std::integral_constant<int, 7>()); break;
    }
    __syncthreads();
    if (d != 0) return;
    cx<double> acc[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = cx<double>{0.0, 0.0};
    auto add = [&](auto dd) {
        constexpr int D = decltype(dd)::value;
        constexpr int SGN = (D & 1) ? (DAG ? -1 : 1) : (DAG ? 1 : -1);
        cx<double> w[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            const double2 q = v4f_to_d2(shm[(D * 6 + k) * FL_WAVE + lane]);
            w[k] = cx<double>{q.x, q.y};
        }
        double f = 1.0;
        if (D == 6) f = s.tlast ? (double)g.bc_t : 1.0;
        if (D == 7) f = s.tfirst ? (double)g.bc_t : 1.0;
        accumulate_scaled<(D >> 1), SGN>(acc, w, f);
    };
    add(std::integral_constant<int, 0>());
    add(std::integral_constant<int, 1>());
    add(std::integral_constant<int, 2>());
    add(std::integral_constant<int, 3>());
    add(std::integral_constant<int, 4>());
    add(std::integral_constant<int, 5>());
    add(std::integral_constant<int, 6>());
    add(std::integral_constant<int, 7>());
    wave_sync();
    store_canon(b, make_rows(), out + (size_t)rhs * V * 24, i0, V, kappa, acc, shm);
}

}  // namespace

// A wave per direction while there are no more blocks than CUs: 8^3x16, one
// right-hand side (128 blocks), 30.0 -> 27.7 us per call, 4^4 29.8 -> 27.7;
// 10x6x14x18, two (474 blocks), 31.2 -> 33.9
static constexpr int FA_SPLIT = 256;

void launch_apply_full(const double *in, double *out, const void *links, const LatGeom &g, int nrhs, double kappa,
                       bool dag, hipStream_t s)
{
    if (!nrhs) return;
    const int nblk = (2 * g.Vh + FL_WAVE - 1) / FL_WAVE, RT = nrhs < FA_RT ? nrhs : FA_RT;
    if ((long long)nblk * nrhs <= FA_SPLIT) {
        const dim3 grid((unsigned)nblk * nrhs), block(8 * FL_WAVE);
        if (dag)
            hipLaunchKernelGGL(k_apply_split<true>, grid, block, 0, s, in, out, links, g, nblk, kappa);
        else
            hipLaunchKernelGGL(k_apply_split<false>, grid, block, 0, s, in, out, links, g, nblk, kappa);
        return;
    }
    const dim3 grid((unsigned)nblk * ((nrhs + RT - 1) / RT)), block(FL_WAVE * RT);
    if (dag)
        hipLaunchKernelGGL(k_apply_full<true>, grid, block, 0, s, in, out, links, g, nrhs, RT, nblk, kappa);
    else
        hipLaunchKernelGGL(k_apply_full<false>, grid, block, 0, s, in, out, links, g, nrhs, RT, nblk, kappa);
}
