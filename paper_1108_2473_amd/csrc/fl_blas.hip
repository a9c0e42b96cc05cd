// fl_blas.hip -- vector updates, reductions and per-system scalar steps of
// the batched Krylov solvers.
//
// BiCGStab (van der Vorst 1992) is run independently for every right-hand
// side of a batch (no block method: the low-precision map of each source
// must not depend on the rest of the batch).  The iteration is split into
//   v = Dhat p (+ <r0, v>)      -> alpha = rho / <r0, v>
//   s = r - alpha v
//   t = Dhat s (+ <t, s>, |t|^2) -> omega = <t, s> / |t|^2
//   x += alpha p + omega s, r = s - omega t (+ <r0, r>, |r|^2)
//                               -> beta = (rho'/rho)(alpha/omega)
//   p = r + beta (p - omega v)
// with the operator launches in fl_dslash.hip carrying the reductions in
// their epilogue.  Reductions are two-stage and deterministic: each
// wavefront writes one partial per 64-site block, and the partials of a system
// are summed in a fixed order by one workgroup (k_scal) or, on small grids, by
// every wave that needs the sum (FoldedStep), with the same bits.
#include "fl_host.h"

namespace {

// per-wave buffer view of right-hand side `rhs` of a field stored as
// SpinorFmt<S> (one resource per field, built in scalar registers)
template <typename S>
__device__ __forceinline__ Buf fbuf(const void *base, const LatGeom &g, int rhs)
{
    return spinor_buf<S>(base, g.Vh, rhs);
}

// a result that the next kernel reads as neighbours (p, s): kept in the caches
// (FP32, 16^3x32, 12 right-hand sides: solve 79.0 -> 77.9 ms)
template <typename S>
__device__ __forceinline__ void store_next(const Buf &b, int Vh, int i, cx<typename SpinorFmt<S>::R> s[12])
{
    SpinorFmt<S>::template store<0>(b, Vh, i, s);
}

template <typename R>
__device__ __forceinline__ cx<R> cpx_of(const double *v)
{
    return cx<R>{(R)v[0], (R)v[1]};
}

// ---------------------------------------------------------------------------
// per-system scalar steps: the partials of a slot are summed in a fixed order,
// then the recurrence advances
// ---------------------------------------------------------------------------

// a b + c d with the rounding written down: the scalar steps have the same bits
// in a launch of their own and inside a vector kernel
__device__ __forceinline__ double dot2(double a, double b, double c, double d) { return fma(a, b, c * d); }

// one step of a system's scalar recurrence on a local copy of its state
template <int STEP>
__device__ __forceinline__ void scal_step(int stamp, int carried_r, const double P[6], SysState &s, int &act)
{
    switch (STEP) {
    case SC_ALPHA: {
        double den = dot2(P[0], P[0], P[1], P[1]);
        if (!(den > 0) || !finite_d(den)) {
            s.flags |= ST_BREAK;
            act = 0;
            break;
        }
        // alpha = rho / r0v
        s.alpha[0] = dot2(s.rho[0], P[0], s.rho[1], P[1]) / den;
        s.alpha[1] = dot2(s.rho[1], P[0], -s.rho[0], P[1]) / den;
        break;
    }
    case SC_OMEGA: {
        double tt = P[2];
        if (tt > 0 && finite_d(tt)) {
            s.omega[0] = P[0] / tt;
            s.omega[1] = P[1] / tt;
        } else if (tt == 0) {
            s.omega[0] = s.omega[1] = 0;
        } else {
            s.flags |= ST_BREAK;
            act = 0;
        }
        break;
    }
    case SC_BETA: {
        // slots of their own: the kernel that forms r may still be reading the
        // omega step's sums (slots 0 to 2)
        double rho_n[2] = {P[3], P[4]};
        double rr = P[5];
        s.iter += 1;
        if (!finite_d(rr) || !finite_d(rho_n[0]) || !finite_d(rho_n[1])) {
            s.flags |= ST_BREAK;
            act = 0;
            break;
        }
        s.rr = rr;
        if (rr > s.rmax2) s.rmax2 = rr;
        if (rr < s.delta2 * s.rmax2) s.flags |= ST_WANT_UPD;
        if (rr <= s.stop2) {
            s.flags |= ST_CONV_ITER;
            act = 0;
        } else if (s.iter >= s.max_iter) {
            s.flags |= ST_MAXIT;
            act = 0;
        }
        double om2 = dot2(s.omega[0], s.omega[0], s.omega[1], s.omega[1]);
        double rh2 = dot2(s.rho[0], s.rho[0], s.rho[1], s.rho[1]);
        if (act && (!(om2 > 0) || !(rh2 > 0))) {
            s.flags |= ST_BREAK;
            act = 0;
        }
        if (om2 > 0 && rh2 > 0) {
            // beta = (rho_n / rho) * (alpha / omega)
            double q[2] = {dot2(rho_n[0], s.rho[0], rho_n[1], s.rho[1]) / rh2,
                           dot2(rho_n[1], s.rho[0], -rho_n[0], s.rho[1]) / rh2};
            double w[2] = {dot2(s.alpha[0], s.omega[0], s.alpha[1], s.omega[1]) / om2,
                           dot2(s.alpha[1], s.omega[0], -s.alpha[0], s.omega[1]) / om2};
            s.beta[0] = dot2(q[0], w[0], -q[1], w[1]);
            s.beta[1] = dot2(q[0], w[1], q[1], w[0]);
        }
        s.rho[0] = rho_n[0];
        s.rho[1] = rho_n[1];
        break;
    }
    case SC_RESET:
        s.tr2 = P[2];
        s.rho[0] = P[3];
        s.rho[1] = P[4];
        s.rr = P[5];
        s.rmax2 = P[5];
        s.flags &= ~(ST_CONV_ITER | ST_WANT_UPD);
        break;
    case SC_INIT:
        s.rho[0] = P[3];
        s.rho[1] = P[4];
        s.rr = P[5];
        s.rmax2 = P[5];
        s.flags = 0;
        s.alpha[0] = s.omega[0] = 1;
        s.alpha[1] = s.omega[1] = 0;
        s.beta[0] = s.beta[1] = 0;
        if (P[5] <= s.stop2) {
            s.flags |= ST_CONV_ITER;
            act = 0;
        } else {
            act = 1;
        }
        break;
    case SC_CG_INIT:  // slot 2: |z|^2 with z = Dhat^+ r; slot 5: |r|^2
        s.zz = P[2];
        s.rr = P[5];
        s.beta[0] = s.beta[1] = 0;
        s.flags &= ST_MAXIT;
        if (P[5] <= s.stop2 || !(P[2] > 0)) {
            s.flags |= ST_CONV_ITER;
            act = 0;
        } else {
            act = 1;
        }
        break;
    case SC_CG_ALPHA:  // slot 2: |q|^2 with q = Dhat p
        if (!(P[2] > 0) || !finite_d(P[2])) {
            s.flags |= ST_BREAK;
            act = 0;
        } else {
            s.alpha[0] = s.zz / P[2];
        }
        break;
    case SC_CG_BETA: {  // slot 3: |z'|^2 of the updated z = Dhat^+ r (slot 2 may still be read
                        // for alpha while z is formed); slot 5: |r|^2 if carried
        // Without a carried r: |r - alpha q|^2 = |r|^2 - 2 alpha Re<q, r>
        // + alpha^2 |q|^2 with <q, r> = <p, Dhat^+ r> = <p, z> = |z|^2 (CG;
        // restored at every residual replacement) and alpha = |z|^2 / |q|^2.
        // The recurrence holds to the rounding of the low-precision operator
        // relative to |r|^2 at the last replacement, so below 1e-6 of that
        // value it is no longer trusted: it still asks for a replacement
        // (far below the delta trigger) but claims no convergence
        double zn = P[3], rr = carried_r ? P[5] : fma(-s.alpha[0], s.zz, s.rr);
        const bool trusted = carried_r || rr > 1e-6 * s.rmax2;
        s.xstamp = stamp;  // r moved by alpha q in this iteration: x moves by alpha p
        s.iter += 1;
        s.rr = rr;
        if (!finite_d(zn) || !finite_d(rr)) {
            s.flags |= ST_BREAK;
            act = 0;
            break;
        }
        s.beta[0] = zn / s.zz;
        s.zz = zn;
        if (rr > s.rmax2) s.rmax2 = rr;
        if (rr < s.delta2 * s.rmax2 || !trusted) s.flags |= ST_WANT_UPD;
        if (trusted && rr <= s.stop2) {
            s.flags |= ST_CONV_ITER;
            act = 0;
        } else if (s.iter >= s.max_iter) {
            s.flags |= ST_MAXIT;
            act = 0;
        }
        break;
    }
    case SC_CG_REZ: {  // after a residual replacement that keeps p: slot 2 |z|^2, z = Dhat^+ r;
                       // slots 0, 1 <z, p>; slot 5 |r|^2
        // CG's step length alpha = |z|^2 / |Dhat p|^2 assumes <z, p> = |z|^2,
        // which holds for the iteration's own z but not for the replaced one;
        // p += c z with c = (|z|^2 - <z, p>) / |z|^2 restores it
        s.zz = P[2];
        s.rr = P[5];
        s.rmax2 = P[5];
        s.flags &= ~(ST_CONV_ITER | ST_WANT_UPD);
        const double zz = P[2] > 0 ? P[2] : 1.0;
        s.beta[0] = (P[2] - P[0]) / zz;
        s.beta[1] = -P[1] / zz;
        if (!(P[2] > 0) || !finite_d(P[2])) {
            s.flags |= ST_BREAK;
            act = 0;
        }
        break;
    }
    default: break;
    }
}

// the partial-sum slots each scalar step reads (bit k: slot k)
constexpr int scal_slots(int step)
{
    switch (step) {
    case SC_ALPHA: return 0x03;     // <r0, v>
    case SC_OMEGA: return 0x07;     // <t, s>, |t|^2
    case SC_BETA: return 0x38;      // <r0, r>, |r|^2
    case SC_RESET: return 0x3c;     // |rh|^2, <r0, r>, |r|^2
    case SC_INIT: return 0x38;      // <r0, r>, |r|^2
    case SC_CG_INIT: return 0x24;   // |z|^2, |r|^2
    case SC_CG_ALPHA: return 0x04;  // |q|^2
    case SC_CG_BETA: return 0x28;   // |z|^2, |r|^2 (if carried)
    case SC_CG_REZ: return 0x27;    // <z, p>, |z|^2, |r|^2
    default: return 0x3f;
    }
}

// The scalar step of one system by every wave that needs its result.  All that
// it reads is loaded together: one after the other the sums, the state and the
// flag took 13000 cycles of the wave (three round trips behind L2, where other
// XCDs left them).
template <int STEP>
struct FoldedStep {
    static constexpr int SLOTS = scal_slots(STEP);
    double v[6][4];        // the first 256 partial sums of each slot, 64 apart
    unsigned long long w;  // word `lane` of the state
    int was;               // the active flag

    __device__ __forceinline__ void fetch(const BlasArgs &a, int sys, int nsb)
    {
        const int lane = threadIdx.x % FL_WAVE;
#pragma unroll
        for (int slot = 0; slot < 6; ++slot)
            if ((SLOTS >> slot) & 1) {
                const double *q = a.partial + pidx(slot, a.nsys, sys, a.B.nsb_max, 0);
#pragma unroll
                for (int k = 0; k < 4; ++k) v[slot][k] = q[min(lane + 64 * k, nsb - 1)];
            }
        constexpr int NW = (int)(sizeof(SysState) / 8);
        w = ((const unsigned long long *)(a.st + sys))[min(lane, NW - 1)];
        int z = 0;
        asm volatile("" : "+v"(z));  // a vector load, in flight with the others
        was = a.active[sys + z];
    }

    __device__ __forceinline__ void run(const BlasArgs &a, int sys, int nsb, SysState &s, int &act)
    {
        double P[6];
#pragma unroll
        for (int slot = 0; slot < 6; ++slot)
            P[slot] = (SLOTS >> slot) & 1 ? slot_sum(v[slot], a.partial, slot, a.nsys, sys, a.B.nsb_max, nsb) : 0.0;
        was = __builtin_amdgcn_readfirstlane(was);
        s = state();
        act = 1;
        scal_step<STEP>(a.stamp, a.carried_r, P, s, act);
        // not to be contracted into the vector arithmetic
        asm volatile("" : "+v"(s.alpha[0]), "+v"(s.alpha[1]), "+v"(s.omega[0]), "+v"(s.omega[1]), "+v"(s.beta[0]), "+v"(s.beta[1]));
    }

    __device__ __forceinline__ SysState state() const
    {
        constexpr int NW = (int)(sizeof(SysState) / 8);
        unsigned u[2 * NW];
#pragma unroll
        for (int k = 0; k < NW; ++k) {
            u[2 * k] = __builtin_amdgcn_readlane((unsigned)w, k);
            u[2 * k + 1] = __builtin_amdgcn_readlane((unsigned)(w >> 32), k);
        }
        SysState s;
        __builtin_memcpy(&s, u, sizeof(s));
        return s;
    }
};

// the state of one system as one store instruction of 8-byte words, one per
// lane, through this wave's copy in LDS
__device__ __forceinline__ void store_state(SysState *dst, const SysState &s, SysState *sh)
{
    constexpr int NW = (int)(sizeof(SysState) / 8);
    const int lane = threadIdx.x % FL_WAVE;
    if (lane == 0) *sh = s;
    wave_sync();
    if (lane < NW) {
        unsigned long long w;
        __builtin_memcpy(&w, (const char *)sh + 8 * lane, 8);
        ((unsigned long long *)dst)[lane] = w;
    }
    store_drain();
}

__device__ __forceinline__ void store_flag(int *dst, int v)
{
    if (threadIdx.x % FL_WAVE == 0) *dst = v;
    store_drain();
}

// S: storage format of the iteration vectors, arithmetic in SpinorFmt<S>::R
// LARGE: OP_CG_PX on fields beyond the caches.
template <typename S, int OP, bool FOLD = false, bool LARGE = false>
__global__ __launch_bounds__(FOLD || sizeof(typename SpinorFmt<S>::R) == 8 ? 512 : 1024) void k_blas(BlasArgs a)
{
    typedef typename SpinorFmt<S>::R R;
    TileInfo T = tile_info(a.B);
    if (!T.valid_rhs) return;
    const LatGeom &g = a.B.lat[T.lat];
    const int l = T.lat, i = FOLD ? min(T.site, g.Vh - 1) : T.site, Vh = g.Vh;
    const int rhs = __builtin_amdgcn_readfirstlane(T.rhs);
    typedef SpinorFmt<S> F;
    typedef SpinorFmt<double> F64;
    SysState fs;   // FOLD: this system's state after the scalar step
    int fact = 1;  // FOLD: still active after it
    // FOLD: a small grid's launch takes as long as one wave's chain of loads,
    // so everything a wave may need is loaded at once, the vectors before the
    // scalar step, and the step is recorded behind the vectors (whole
    // solves on 10x6x14x18, 7 right-hand sides: 16-bit CGNR 5.62 -> 4.93 ms,
    // FP64 BiCGStab 3.76 -> 3.35)
    // (five FP64 fields don't fit the registers)
    constexpr int FIELDS = !FOLD ? 0
                         : OP == OP_BICG_XR ? (sizeof(R) == 8 ? 0 : 0x2f)
                         : OP == OP_BICG_S || OP == OP_CG_R ? 0x3 : 0x7;
    cx<R> fv[FOLD ? 6 : 1][12];
    // fields that the next kernels don't read, loaded so that the others stay
    // cached: BiCGStab's r of s, x, s, t, r0 of the x and r update, v of p
    // (16^3x32, FP32, 12 right-hand sides: solve 81.8 -> 79.0 ms, FP64, 8: 21.9 ->
    // 21.1); CGNR's z and x
    // where they are too large for the cache anyway (LARGE)
    constexpr unsigned ONCE = OP == OP_BICG_S ? 0x1 : OP == OP_BICG_XR ? 0x2d : OP == OP_BICG_P ? 0x4
                            : OP == OP_CG_PX && LARGE ? 0x6 : 0;
    auto load = [&](int k, cx<R> v[12]) {
        if constexpr (FIELDS != 0) {
#pragma unroll
            for (int c = 0; c < 12; ++c) v[c] = fv[k][c];
        } else if ((ONCE >> k) & 1) {
            load_once<S, R>(fbuf<S>(a.f[k][l], g, rhs), Vh, i, v);
        } else {
            F::load(fbuf<S>(a.f[k][l], g, rhs), Vh, i, v);
        }
    };
    constexpr int STEP = OP == OP_BICG_S ? SC_ALPHA : OP == OP_BICG_XR ? SC_OMEGA : OP == OP_BICG_P ? SC_BETA
                       : OP == OP_CG_R ? SC_CG_ALPHA : SC_CG_BETA;
    constexpr bool BETA = STEP == SC_BETA || STEP == SC_CG_BETA;
    __shared__ SysState shs[FOLD ? 8 : 1];  // a copy per wave
    // what the first wave of a system records
    auto record = [&](bool was_active) {
        if (T.sb != 0) return;
        SysState *sh = shs + threadIdx.x / FL_WAVE;
        if (BETA) {
            store_state(a.st_out + T.sys, fs, sh);
            store_flag(a.act_out + T.sys, fact);
        } else if (was_active) {
            // only what no other wave of this launch reads: alpha or
            // omega, the flags, and the active flag of a breakdown
            double *dst = STEP == SC_OMEGA ? a.st[T.sys].omega : a.st[T.sys].alpha;
            const double *v = STEP == SC_OMEGA ? fs.omega : fs.alpha;
            const int lane = threadIdx.x % FL_WAVE;
            const double w = lane == 0 ? v[0] : v[1];
            if (lane < 2) dst[lane] = w;
            store_drain();
            if (!fact) {
                store_flag(&a.st[T.sys].flags, fs.flags);
                store_flag(a.active + T.sys, 0);
            }
        }
    };
    if constexpr (FOLD) {
        FoldedStep<STEP> step;
        step.fetch(a, T.sys, g.nsb);
#pragma unroll
        for (int k = 0; k < 6; ++k)
            if ((FIELDS >> k) & 1) F::load(fbuf<S>(a.f[k][l], g, rhs), Vh, i, fv[k]);
        step.run(a, T.sys, g.nsb, fs, fact);
        // the loads are not moved behind the branch
#pragma unroll
        for (int k = 0; k < 6; ++k)
            if ((FIELDS >> k) & 1)
#pragma unroll
                for (int c = 0; c < 12; ++c) asm volatile("" : "+v"(fv[k][c].re), "+v"(fv[k][c].im));
        if (!step.was) {
            // a wave that finds the flag taken back by the first one in this
            // launch (alpha, omega) stops like it
            fs = step.state();
            fact = 0;
            record(false);
            return;
        }
        if (!fact && OP != OP_CG_PX) {
            record(true);
            return;
        }
    } else if (OP == OP_CG_PX) {
        // a system that stopped in this iteration still owes its x update
        if (!a.mask[T.sys] && a.st[T.sys].xstamp != a.stamp) return;
    } else if (a.mask && !a.mask[T.sys]) {
        return;
    }
    const SysState &cur = FOLD ? fs : a.st[T.sys];
    R q0 = 0, q1 = 0, q2 = 0;
    if (T.valid_site) {
        if (OP == OP_BICG_S) {
            const SysState &st = cur;
            cx<R> al = cpx_of<R>(st.alpha);
            cx<R> r[12], v[12];
            load(0, r);
            load(1, v);
#pragma unroll
            for (int k = 0; k < 12; ++k) r[k] = cmsub(r[k], al, v[k]);
            store_next<S>(fbuf<S>(a.f[2][l], g, rhs), Vh, i, r);
        } else if (OP == OP_BICG_XR) {
            const SysState &st = cur;
            cx<R> al = cpx_of<R>(st.alpha), om = cpx_of<R>(st.omega);
            cx<R> x[12], p[12], s[12], t[12], r0[12];
            load(0, x);
            load(1, p);
            load(2, s);
            load(3, t);
            load(5, r0);
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                x[k] = cmad(cmad(x[k], al, p[k]), om, s[k]);
                s[k] = cmsub(s[k], om, t[k]);  // new r
            }
            store_result<S>(fbuf<S>(a.f[0][l], g, rhs), Vh, i, x);
            store_result<S>(fbuf<S>(a.f[4][l], g, rhs), Vh, i, s);  // reductions of the stored values
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                cx<R> d = cjmul(r0[k], s[k]);
                q0 += d.re;
                q1 += d.im;
                q2 += s[k].re * s[k].re + s[k].im * s[k].im;
            }
        } else if (OP == OP_BICG_P) {
            const SysState &st = cur;
            cx<R> be = cpx_of<R>(st.beta), om = cpx_of<R>(st.omega);
            cx<R> p[12], r[12], v[12];
            load(0, p);
            load(1, r);
            load(2, v);
#pragma unroll
            for (int k = 0; k < 12; ++k) p[k] = cmad(r[k], be, cmsub(p[k], om, v[k]));
            store_next<S>(fbuf<S>(a.f[0][l], g, rhs), Vh, i, p);
        } else if (OP == OP_HI_TO_LO) {
            cx<double> h[12];
            cx<R> lo[12], r0[12];
            F64::load(fbuf<double>(a.f[1][l], g, rhs), Vh, i, h);
#pragma unroll
            for (int k = 0; k < 12; ++k) lo[k] = cx<R>{(R)h[k].re, (R)h[k].im};
            store_result<S>(fbuf<S>(a.f[0][l], g, rhs), Vh, i, lo);
            if (a.flag) {
                store_result<S>(fbuf<S>(a.f[2][l], g, rhs), Vh, i, lo);
                store_result<S>(fbuf<S>(a.f[3][l], g, rhs), Vh, i, lo);
                cx<R> z[12];
#pragma unroll
                for (int k = 0; k < 12; ++k) z[k] = cx<R>{(R)0, (R)0};
                store_result<S>(fbuf<S>(a.f[4][l], g, rhs), Vh, i, z);
#pragma unroll
                for (int k = 0; k < 12; ++k) r0[k] = lo[k];
            } else {
                F::load(fbuf<S>(a.f[2][l], g, rhs), Vh, i, r0);
            }
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                cx<R> d = cjmul(r0[k], lo[k]);
                q0 += d.re;
                q1 += d.im;
                q2 += lo[k].re * lo[k].re + lo[k].im * lo[k].im;
            }
        } else if (OP == OP_ACC_HI) {
            cx<double> h[12];
            cx<R> lo[12];
            F64::load(fbuf<double>(a.f[0][l], g, rhs), Vh, i, h);
            F::load(fbuf<S>(a.f[1][l], g, rhs), Vh, i, lo);
#pragma unroll
            for (int k = 0; k < 12; ++k) h[k] = h[k] + cx<double>{(double)lo[k].re, (double)lo[k].im};
            store_result<double>(fbuf<double>(a.f[0][l], g, rhs), Vh, i, h);
            if (a.flag) {
#pragma unroll
                for (int k = 0; k < 12; ++k) lo[k] = cx<R>{(R)0, (R)0};
                store_result<S>(fbuf<S>(a.f[1][l], g, rhs), Vh, i, lo);
            }
        } else if (OP == OP_SUB_HI) {
            cx<double> u[12], w[12];
            F64::load(fbuf<double>(a.f[1][l], g, rhs), Vh, i, u);
            F64::load(fbuf<double>(a.f[2][l], g, rhs), Vh, i, w);
#pragma unroll
            for (int k = 0; k < 12; ++k) u[k] = u[k] - w[k];
            store_result<double>(fbuf<double>(a.f[0][l], g, rhs), Vh, i, u);
        } else if (OP == OP_NORM) {
            cx<R> f[12];
            F::load(fbuf<S>(a.f[0][l], g, rhs), Vh, i, f);
#pragma unroll
            for (int k = 0; k < 12; ++k) q2 += f[k].re * f[k].re + f[k].im * f[k].im;
        } else if (OP == OP_ZERO) {
            cx<R> z[12];
#pragma unroll
            for (int k = 0; k < 12; ++k) z[k] = cx<R>{(R)0, (R)0};
            store_result<S>(fbuf<S>(a.f[0][l], g, rhs), Vh, i, z);
        } else if (OP == OP_DOT) {
            cx<R> u[12], w[12];
            F::load(fbuf<S>(a.f[0][l], g, rhs), Vh, i, u);
            F::load(fbuf<S>(a.f[1][l], g, rhs), Vh, i, w);
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                cx<R> d = cjmul(u[k], w[k]);
                q0 += d.re;
                q1 += d.im;
            }
        } else if (OP == OP_CG_FIXP) {
            const cx<R> c = {(R)a.st[T.sys].beta[0], (R)a.st[T.sys].beta[1]};
            cx<R> p[12], z[12];
            F::load(fbuf<S>(a.f[0][l], g, rhs), Vh, i, p);
            F::load(fbuf<S>(a.f[1][l], g, rhs), Vh, i, z);
#pragma unroll
            for (int k = 0; k < 12; ++k) p[k] = cmad(p[k], c, z[k]);
            store_result<S>(fbuf<S>(a.f[0][l], g, rhs), Vh, i, p);
        } else if (OP == OP_CG_R) {
            const R al = (R)cur.alpha[0];
            cx<R> r[12], q[12];
            load(0, r);
            load(1, q);
#pragma unroll
            for (int k = 0; k < 12; ++k) r[k] = cx<R>{fma(-al, q[k].re, r[k].re), fma(-al, q[k].im, r[k].im)};
            store_result<S>(fbuf<S>(a.f[0][l], g, rhs), Vh, i, r);
#pragma unroll
            for (int k = 0; k < 12; ++k) q2 += r[k].re * r[k].re + r[k].im * r[k].im;
        } else if (OP == OP_CG_P) {
            const R be = (R)a.st[T.sys].beta[0];
            cx<R> p[12], z[12];
            F::load(fbuf<S>(a.f[0][l], g, rhs), Vh, i, p);
            F::load(fbuf<S>(a.f[1][l], g, rhs), Vh, i, z);
#pragma unroll
            for (int k = 0; k < 12; ++k) p[k] = cx<R>{fma(be, p[k].re, z[k].re), fma(be, p[k].im, z[k].im)};
            store_result<S>(fbuf<S>(a.f[0][l], g, rhs), Vh, i, p);
        } else if (OP == OP_CG_PX) {
            // wave-uniform: one wave is one system
            const SysState &st = cur;
            const bool xu = FOLD || st.xstamp == a.stamp, pu = FOLD ? fact != 0 : a.mask[T.sys] != 0;
            cx<R> p[12];
            load(0, p);
            if (xu) {
                const R al = (R)st.alpha[0];
                cx<R> x[12];
                load(2, x);
#pragma unroll
                for (int k = 0; k < 12; ++k) x[k] = cx<R>{fma(al, p[k].re, x[k].re), fma(al, p[k].im, x[k].im)};
                store_result<S>(fbuf<S>(a.f[2][l], g, rhs), Vh, i, x);
            }
            if (pu) {
                const R be = (R)st.beta[0];
                cx<R> z[12];
                load(1, z);
#pragma unroll
                for (int k = 0; k < 12; ++k) p[k] = cx<R>{fma(be, p[k].re, z[k].re), fma(be, p[k].im, z[k].im)};
                store_next<S>(fbuf<S>(a.f[0][l], g, rhs), Vh, i, p);
            }
        }
    }
    if constexpr (FOLD) record(true);
    if (OP == OP_BICG_XR || OP == OP_HI_TO_LO || OP == OP_NORM || OP == OP_CG_R || OP == OP_DOT) {
        double s0 = wave_sum((double)q0), s1 = wave_sum((double)q1), s2 = wave_sum((double)q2);
        constexpr int which = (OP == OP_BICG_XR || OP == OP_HI_TO_LO) ? 7 : (OP == OP_DOT ? 3 : 4);
        write_partials(a.partial, a.slot0, a.nsys, T.sys, a.B.nsb_max, T.sb, s0, s1, s2, which);
    }
}

template <typename S>
void dispatch(const BlasArgs &a, dim3 grid, dim3 block, hipStream_t s)
{
    if (a.fold) {
        switch (a.op) {
        case OP_BICG_S: hipLaunchKernelGGL((k_blas<S, OP_BICG_S, true>), grid, block, 0, s, a); break;
        case OP_BICG_XR: hipLaunchKernelGGL((k_blas<S, OP_BICG_XR, true>), grid, block, 0, s, a); break;
        case OP_BICG_P: hipLaunchKernelGGL((k_blas<S, OP_BICG_P, true>), grid, block, 0, s, a); break;
        case OP_CG_R: hipLaunchKernelGGL((k_blas<S, OP_CG_R, true>), grid, block, 0, s, a); break;
        case OP_CG_PX: hipLaunchKernelGGL((k_blas<S, OP_CG_PX, true>), grid, block, 0, s, a); break;
        default: launch_unsupported("vector operation with a scalar step"); break;
        }
        return;
    }
    // OP_CG_PX: its three fields against the 256 MB of the Infinity Cache.  z and
    // x non-temporally: 490 MB (16-bit, 8^3x16, 768 right-hand sides) 814 -> 795
    // ms a timeslice, 450 MB (FP32, 16^3x32, 24) 56.8 -> 55.7 ms; 143 MB (FP32,
    // 12^3x24, 24) 18.0 -> 18.3, 245 MB (16-bit, 16^3x32, 24) 42.8 -> 43.0
    size_t px = 0;
    for (int l = 0; l < a.B.nlat; ++l) px += 3 * (size_t)SpinorFmt<S>::SITE_BYTES * a.B.lat[l].Vh * a.B.lat[l].nrhs;
    const bool large = px > (size_t)256 << 20;
    switch (a.op) {
    case OP_BICG_S: hipLaunchKernelGGL((k_blas<S, OP_BICG_S>), grid, block, 0, s, a); break;
    case OP_BICG_XR: hipLaunchKernelGGL((k_blas<S, OP_BICG_XR>), grid, block, 0, s, a); break;
    case OP_BICG_P: hipLaunchKernelGGL((k_blas<S, OP_BICG_P>), grid, block, 0, s, a); break;
    case OP_HI_TO_LO: hipLaunchKernelGGL((k_blas<S, OP_HI_TO_LO>), grid, block, 0, s, a); break;
    case OP_ACC_HI: hipLaunchKernelGGL((k_blas<S, OP_ACC_HI>), grid, block, 0, s, a); break;
    case OP_SUB_HI: hipLaunchKernelGGL((k_blas<S, OP_SUB_HI>), grid, block, 0, s, a); break;
    case OP_NORM: hipLaunchKernelGGL((k_blas<S, OP_NORM>), grid, block, 0, s, a); break;
    case OP_ZERO: hipLaunchKernelGGL((k_blas<S, OP_ZERO>), grid, block, 0, s, a); break;
    case OP_CG_R: hipLaunchKernelGGL((k_blas<S, OP_CG_R>), grid, block, 0, s, a); break;
    case OP_CG_P: hipLaunchKernelGGL((k_blas<S, OP_CG_P>), grid, block, 0, s, a); break;
    case OP_CG_PX:
        if (large)
            hipLaunchKernelGGL((k_blas<S, OP_CG_PX, false, true>), grid, block, 0, s, a);
        else
            hipLaunchKernelGGL((k_blas<S, OP_CG_PX>), grid, block, 0, s, a);
        break;
    case OP_DOT: hipLaunchKernelGGL((k_blas<S, OP_DOT>), grid, block, 0, s, a); break;
    case OP_CG_FIXP: hipLaunchKernelGGL((k_blas<S, OP_CG_FIXP>), grid, block, 0, s, a); break;
    default: launch_unsupported("vector operation"); break;
    }
}

// Bound by the latency of its loads: the state is fetched beside the
// partial sums, the loads of up to 1024 site blocks are issued before the
// first is added, and the tree takes one barrier (four threads' sums per
// lane, then shuffles) -- the same order of additions as a halving tree over
// 256 threads.  8.5 -> 4.8 us a launch with 1024 site blocks and 12 systems,
// 4.5 -> 2.6 us with 64 site blocks and one.
template <int STEP>
__global__ __launch_bounds__(256) void k_scal(ScalArgs a)
{
    const int sys = blockIdx.x;
    const int act0 = a.active[sys];
    if (a.mask ? !a.mask[sys] : !act0) return;
    int l = 0;
    for (int k = 1; k < FL_MAXLAT; ++k)
        if (k < a.B.nlat && sys >= a.B.lat[k].sys0) l = k;
    const int nsb = a.B.lat[l].nsb, nb = a.B.nsb_max;
    constexpr int used = scal_slots(STEP);  // only the slots this step reads
    __shared__ double red[6][256];
    __shared__ SysState snew;
    constexpr int NW = (int)(sizeof(SysState) / 8);
    static_assert(sizeof(SysState) % 8 == 0, "SysState is written in 8-byte words");
    // the old state waits in the shared copy
    if ((int)threadIdx.x < NW)
        ((unsigned long long *)&snew)[threadIdx.x] = ((const unsigned long long *)(a.st + sys))[threadIdx.x];
    double acc[6];
#pragma unroll
    for (int slot = 0; slot < 6; ++slot) acc[slot] = 0.0;
    for (int sb = threadIdx.x; sb < nsb; sb += 1024) {
        double v[6][4];
#pragma unroll
        for (int slot = 0; slot < 6; ++slot)
            if ((used >> slot) & 1)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const int q = min(sb + 256 * k, nsb - 1);
                    v[slot][k] = a.partial[pidx(slot, a.nsys, sys, nb, q)];
                }
#pragma unroll
        for (int slot = 0; slot < 6; ++slot)
            if ((used >> slot) & 1)
#pragma unroll
                for (int k = 0; k < 4; ++k) acc[slot] += sb + 256 * k < nsb ? v[slot][k] : 0.0;
    }
#pragma unroll
    for (int slot = 0; slot < 6; ++slot)
        if ((used >> slot) & 1) red[slot][threadIdx.x] = acc[slot];
    __syncthreads();
    if (threadIdx.x >= FL_WAVE) return;
    double P[6];
#pragma unroll
    for (int slot = 0; slot < 6; ++slot) {
        P[slot] = 0.0;
        if (!((used >> slot) & 1)) continue;
        const double *q = red[slot] + threadIdx.x;
        P[slot] = wave_sum((q[0] + q[128]) + (q[64] + q[192]));
    }
    if (threadIdx.x == 0) {
        SysState s = snew;
        int act = act0;
        scal_step<STEP>(a.stamp, a.carried_r, P, s, act);
        snew = s;
        if (act != act0) a.active[sys] = act;
    }
    // the flag store completes before the state is written as one store
    // instruction of 8-byte words, one per lane, which ends the kernel
    wave_sync();
    store_drain();
    if ((int)threadIdx.x < NW)
        ((unsigned long long *)(a.st + sys))[threadIdx.x] = ((const unsigned long long *)&snew)[threadIdx.x];
}

}  // namespace

void launch_blas(VecFormat vf, const BlasArgs &a, hipStream_t s)
{
    if (a.B.ntiles == 0) return;
    dim3 grid(a.B.ntiles), block(FL_WAVE * a.B.RT);
    if (vf == VEC_F64)
        dispatch<double>(a, grid, block, s);
    else if (vf == VEC_F32)
        dispatch<float>(a, grid, block, s);
    else
        dispatch<H16>(a, grid, block, s);
}

void launch_scalars(const ScalArgs &a, hipStream_t s)
{
    if (a.nsys == 0) return;
    const dim3 grid(a.nsys), block(256);
    switch (a.step) {
    case SC_ALPHA: hipLaunchKernelGGL(k_scal<SC_ALPHA>, grid, block, 0, s, a); break;
    case SC_OMEGA: hipLaunchKernelGGL(k_scal<SC_OMEGA>, grid, block, 0, s, a); break;
    case SC_BETA: hipLaunchKernelGGL(k_scal<SC_BETA>, grid, block, 0, s, a); break;
    case SC_RESET: hipLaunchKernelGGL(k_scal<SC_RESET>, grid, block, 0, s, a); break;
    case SC_INIT: hipLaunchKernelGGL(k_scal<SC_INIT>, grid, block, 0, s, a); break;
    case SC_CG_INIT: hipLaunchKernelGGL(k_scal<SC_CG_INIT>, grid, block, 0, s, a); break;
    case SC_CG_ALPHA: hipLaunchKernelGGL(k_scal<SC_CG_ALPHA>, grid, block, 0, s, a); break;
    case SC_CG_BETA: hipLaunchKernelGGL(k_scal<SC_CG_BETA>, grid, block, 0, s, a); break;
    case SC_CG_REZ: hipLaunchKernelGGL(k_scal<SC_CG_REZ>, grid, block, 0, s, a); break;
    default: launch_unsupported("scalar step"); break;
    }
}
