// one_cu.h -- what the kernels share that solve one instance of a batch with
// a workgroup that holds it on a CU (closed.hip, general.hip), in most of them
// one of 1024 threads with the CU to itself: reductions, the instance's ranges
// and state, the check.
#pragma once

#include <math.h>

#include <type_traits>

#include "device_math.h"
#include "pdhcg_internal.h"

namespace pdhcg {

constexpr int REG_MAX = ONE_CU_MAX;   // variables, rows, threads
constexpr int REG_T = 16;                   // entries of a row of A' in registers (longer rows: the rest from memory)

// ---- reductions -----------------------------------------------------------------

// One step of a wavefront reduction in the lane crossbar (DPP): a lane takes
// the value of the lane that CTRL names, lanes without a source take `ident`.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_from(double v, double ident)
{
    const long long b = __double_as_longlong(v), e = __double_as_longlong(ident);
    const int lo = __builtin_amdgcn_update_dpp((int)(e & 0xffffffffll), (int)(b & 0xffffffffll), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(e >> 32), (int)(b >> 32), CTRL, ROWS, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// reduction over the 64 lanes, the result in scalar registers: shifts by 1,
// 2, 4 and 8 inside each row of 16 lanes, then lane 15 of a row into the
// next row and lane 31 into the upper half; lane 63 holds the whole.  A
// 64-lane shuffle of a double would take two LDS round trips per step.
__device__ __forceinline__ double wave_reduce(int kind, double v)
{
    const double id = rid(kind);
    v = rcomb(kind, v, dpp_from<0x111, 0xf>(v, id));
    v = rcomb(kind, v, dpp_from<0x112, 0xf>(v, id));
    v = rcomb(kind, v, dpp_from<0x114, 0xf>(v, id));
    v = rcomb(kind, v, dpp_from<0x118, 0xf>(v, id));
    v = rcomb(kind, v, dpp_from<0x142, 0xa>(v, id));
    v = rcomb(kind, v, dpp_from<0x143, 0xc>(v, id));
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), 63);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Sum (bit j of MAXM clear) or maximum (set) of NR values over the workgroup
// of T threads, in a fixed order, in every thread.  The caller puts a barrier
// between two reductions' uses of `lds` (any barrier after this returns).
constexpr int RED_SLOTS = 8;
template <int T, int NR, unsigned MAXM>
__device__ __forceinline__ void wg_sum(double (&v)[NR], double* lds)
{
    static_assert(NR <= RED_SLOTS, "the buffer holds RED_SLOTS slots");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        v[j] = wave_reduce(((MAXM >> j) & 1u) ? R_MAX : R_SUM, v[j]);
        if (lane == 0) lds[wave * NR + j] = v[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NR; ++j) {
        double r = lds[j];
        for (int w = 1; w < T / 64; ++w) r = rcomb(((MAXM >> j) & 1u) ? R_MAX : R_SUM, r, lds[w * NR + j]);
        v[j] = uniform(r);
    }
}

// Sum of squares of the threads' values (v of the first len threads) in the
// order of a workgroup of 256 threads (batch.hip's norm kernel and default
// shape), in every thread: the weight's update and the norms, from which all
// step sizes come, keep their bits, so that no operand's FP32 rounding turns.
// buf: a double per thread.  Two barriers and one more before buf is used again.
__device__ __forceinline__ double sumsq_256(double v, int len, double* buf, double* lds)
{
    buf[threadIdx.x] = v;
    __syncthreads();
    if (threadIdx.x < 256) {
        double a = 0.0;
        for (int i = threadIdx.x; i < len; i += 256) a = __builtin_fma(buf[i], buf[i], a);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) a += __shfl_xor(a, off);
        if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = a;
    }
    __syncthreads();
    double r = lds[0];
    for (int w = 1; w < 4; ++w) r += lds[w];
    return uniform(r);
}

// ---- a workgroup's rows in LDS -----------------------------------------------------

// entries of the longest row of the wave (uniform)
__device__ __forceinline__ int wave_longest(int len)
{
    int most = 0;
    while (__ballot(len > most) != 0ull) ++most;
    return uniform_int(most);
}

// the wave's share of the places [first, total): `base` and how many entries
// of each of its 64 rows fit; the waves' shares follow each other up to `end`
struct Share {
    int base, wide, end;
};
template <int T>
__device__ __forceinline__ Share share(int want, int first, int total, int* widths)
{
    const int wave = uniform_int(threadIdx.x >> 6);
    if ((threadIdx.x & 63) == 0) widths[wave] = want;
    __syncthreads();
    int base = first, end = first;
    for (int w = 0; w < T / 64; ++w) {
        if (w == wave) base = end;
        end += 64 * widths[w];
    }
    Share p;
    p.base = uniform_int(base < total ? base : total);
    p.end = uniform_int(end < total ? end : total);
    const int fit = (total - p.base) / 64;
    p.wide = uniform_int(want < fit ? want : fit);
    __syncthreads();
    return p;
}

// ---- one instance ---------------------------------------------------------------

// its ranges and per-instance values (the same in every thread)
struct ClosedInst {
    int v0, n, r0, m, unb;
    double eta, omega0, cmax, bscale, gammaq;
};

__device__ __forceinline__ ClosedInst closed_instance(const BatchDev& B, int b)
{
    ClosedInst in;
    in.v0 = uniform_int(B.voff[b]);
    in.n = uniform_int(B.voff[b + 1]) - in.v0;
    in.r0 = uniform_int(B.roff[b]);
    in.m = uniform_int(B.roff[b + 1]) - in.r0;
    in.unb = uniform_int(B.unb[b]);
    in.eta = uniform(B.eta[b]);
    in.omega0 = uniform(B.omega0[b]);
    in.cmax = uniform(B.cmax[b]);
    in.bscale = uniform(B.bscale[b]);
    in.gammaq = uniform(B.gammaq[b]);
    return in;
}

// the scalars of its solve, in LDS: one thread writes, all read
struct ClosedState {
    long long k, t, restarts;
    double omega, tau, sigma, it;
    double R_start, R_prev, pid_int, pid_prev;
    int R_prev_valid, status;
    double ndx2, ndy2, ytil_max, ptil_sum, ptil_abs, d_max, cd;
    double rp, rd, rg, pobj, dobj;
};

// column of entry q relative to the instance's first (first)
__device__ __forceinline__ int local_col(const unsigned short* c16, const int* c32, int q, int first)
{
    return c16 ? (int)c16[q] : c32[q] - first;
}

// entries [a, e) of a row times one operand, and times two
__device__ __forceinline__ double csr_dot(int a, int e, const unsigned short* c16, const int* c32, int first,
                                          const double* val, const double* x)
{
    double s = 0.0;
#pragma unroll 4
    for (int q = a; q < e; ++q) s += val[q] * x[local_col(c16, c32, q, first)];
    return s;
}
__device__ __forceinline__ void csr_dot2(int a, int e, const unsigned short* c16, const int* c32, int first,
                                         const double* val, const double* x, const double* z, double& sx, double& sz)
{
    double s = 0.0, r = 0.0;
#pragma unroll 4
    for (int q = a; q < e; ++q) {
        const double v = val[q];
        const int j = local_col(c16, c32, q, first);
        s += v * x[j];
        r += v * z[j];
    }
    sx = s;
    sz = r;
}

// the kernel's arguments, as they lie in its segment
struct ClosedArgs {
    BatchDev B;
    BatchParams P;
};

// The check at (x_T, y_T) = (B.xt, B.yt): KKT pieces and certificate pieces
// (Sections 4, 5), the stop test and the restart rule with the PID weight
// (Section 3.2); leaves A'y_T in B.aty and, in mixed precision, A x_T in
// B.axref.  Returns 1 when the round restarts; s->status != 0 ends the solve.
// A call, not inlined: it runs once in check_every iterations, and inlined it
// takes registers from the iteration, whose matrix rows are then spilled and
// reloaded in every step (5.4 us instead of 3.7 on a 748-variable instance).
// It reads the kernel's arguments from their segment.
// GEN: Q is not diagonal.  T: threads.
template <bool F32, bool GEN, int T>
__device__ __attribute__((noinline)) int one_cu_check(unsigned long long args, int b, double* red, ClosedState* s)
{
    const unsigned lo = (unsigned)uniform_int((int)(args & 0xffffffffull)), hi = (unsigned)uniform_int((int)(args >> 32));
    const ClosedArgs* ka =
        (const ClosedArgs*)(const __attribute__((address_space(4))) ClosedArgs*)(((unsigned long long)hi << 32) | lo);
    const BatchDev& B = ka->B;
    const BatchParams& P = ka->P;
    const ClosedInst in = closed_instance(B, uniform_int(b));
    const int tid = threadIdx.x, v0 = in.v0, r0 = in.r0, unb = in.unb;
    const bool xon = tid < in.n, yon = tid < in.m;
    const double *xt = B.xt + v0, *yt = B.yt + r0, *ytil = B.ytil + r0, *d = B.d + v0;
    const long long k = s->k, t = s->t;
    const bool later = k > 0;
    const int vi = v0 + tid, ri = r0 + tid;
    // A'y_T, A'ytil: maxima of |A'y| and of the violation, the sums of p
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    double aty = 0.0, l = 0.0, u = 0.0;
    if (xon) {
        l = B.lv[vi];
        u = B.uv[vi];
        const int qa = B.trp[vi], qe = B.trp[vi + 1];
        if (later) {
            double wv;
            csr_dot2(qa, qe, B.tcol16, B.tcol, r0, B.tval, yt, ytil, aty, wv);
            const double wh = projR(wv, l, u);
            a[1] = fabs(wv - wh);
            a[2] = supp(-wh, l, u);
            a[3] = supp_abs(-wh, l, u);
        } else {
            aty = csr_dot(qa, qe, B.tcol16, B.tcol, r0, B.tval, yt);
        }
        B.aty[vi] = aty;
        a[0] = fabs(aty);
    }
    __syncthreads();
    wg_sum<T, 4, 3u>(a, red);
    // A x_T, A d: violation (max), p(y), violation of A d (max)
    double c[3] = {0.0, 0.0, 0.0};
    if (yon) {
        const int qa = B.arp[ri], qe = B.arp[ri + 1];
        const double lc = B.lc[ri], uc = B.uc[ri], yj = yt[tid];
        double ax, ad = 0.0;
        if (later && unb) csr_dot2(qa, qe, B.acol16, B.acol, v0, B.aval, xt, d, ax, ad);
        else ax = csr_dot(qa, qe, B.acol16, B.acol, v0, B.aval, xt);
        if constexpr (F32) B.axref[ri] = ax;
        c[0] = fabs(ax - clampd(ax, lc, uc));
        c[1] = supp(yj, lc, uc);
        if (later && unb) c[2] = fabs(ad - projRec(ad, lc, uc));
    }
    __syncthreads();
    wg_sum<T, 3, 5u>(c, red);
    // Q x_T, Q d and the reduced cost: maxima 0, 1, 5 and 6, the rest sums
    double e[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (xon) {
        const double xi = xt[tid], ci = B.c[vi];
        double qx, qv = 0.0;
        if constexpr (GEN) {
            const int qa = B.qrp[vi], qe = B.qrp[vi + 1];
            if (later && unb) csr_dot2(qa, qe, B.qcol16, B.qcol, v0, B.qval, xt, d, qx, qv);
            else qx = csr_dot(qa, qe, B.qcol16, B.qcol, v0, B.qval, xt);
        } else {
            const double qd = B.qd[vi];
            qx = qd * xi;
            if (later && unb) qv = qd * d[tid];
        }
        const double r = qx + ci + aty;
        const double rh = projR(r, l, u);
        e[0] = fabs(r - rh);
        e[1] = fabs(qx);
        e[2] = xi * qx;
        e[3] = ci * xi;
        e[4] = supp(-rh, l, u);
        e[5] = fabs(xi - clampd(xi - r, l, u));
        e[6] = fabs(qv);
    }
    __syncthreads();
    wg_sum<T, 7, (1u << 0) | (1u << 1) | (1u << 5) | (1u << 6)>(e, red);

    const double rp = c[0] / in.bscale;
    double sd = e[1] > a[0] ? e[1] : a[0];
    sd = sd > in.cmax ? sd : in.cmax;
    const double rd = e[0] / (1.0 + sd);
    const double pobj = 0.5 * e[2] + e[3];
    const double dneg = 0.5 * e[2] + e[4] + c[1];
    const double den = fabs(pobj) > fabs(dneg) ? fabs(pobj) : fabs(dneg);
    const double rg = fabs(e[2] + e[3] + e[4] + c[1]) / (1.0 + den);
    double worst = rp > rd ? rp : rd;
    worst = worst > rg ? worst : rg;
    bool pinf = false, dinf = false;
    if (later && s->ytil_max > 0.0 && isfinite(s->ytil_max)) {
        const double val = a[2] + s->ptil_sum;
        const double imp = val < 0.0 ? -val : 0.0;
        pinf = imp > 1e-9 * (a[3] + s->ptil_abs) && a[1] <= P.eps_inf * imp;
    }
    if (later && unb && s->d_max > 0.0 && isfinite(s->d_max) && s->cd / s->d_max < -P.tol) {
        const double v1 = c[2] / s->d_max, v2 = e[6] / s->d_max / in.gammaq;
        dinf = (v1 > v2 ? v1 : v2) <= P.eps_inf;
    }
    int status = 0, restart = 0;
    double R = 0.0, omega = s->omega, mx = 0.0, my = 0.0;
    if (!isfinite(worst) || worst != worst) status = 5;
    else if (worst <= P.tol) status = 1;
    else if (pinf) status = 2;
    else if (dinf) status = 3;
    else if (k >= P.max_iter) status = 4;
    else {
        R = sqrt(omega * s->ndx2 + s->ndy2 / omega);
        restart = R <= P.rs_suff * s->R_start || (s->R_prev_valid && R <= P.rs_nec * s->R_start && R > s->R_prev) ||
                  (double)t >= P.rs_art * (double)k;
    }
    if (uniform_int(restart)) {
        double* buf = red + RED_SLOTS * (T / 64);   // the first operand's space
        __syncthreads();
        mx = sqrt(sumsq_256(xon ? xt[tid] - B.xa[vi] : 0.0, in.n, buf, red));
        __syncthreads();
        my = sqrt(sumsq_256(yon ? yt[tid] - B.ya[ri] : 0.0, in.m, buf, red));
        __syncthreads();
        buf[tid] = 0.0;                          // (its zero entries)
    }
    __syncthreads();   // every thread has read *s
    if (tid == 0) {
        s->rp = rp; s->rd = rd; s->rg = rg;
        s->pobj = pobj; s->dobj = -dneg;
        s->status = status;
        if (status == 0) {
            s->R_prev = R;
            s->R_prev_valid = 1;
        }
        if (restart) {
            if (mx > 1e-10 && my > 1e-10 && isfinite(mx) && isfinite(my)) {
                const double so = sqrt(omega);
                const double err = log(so * mx / (my / so));
                s->pid_int += err;
                double lw = log(omega) - (P.kp * err + P.ki * s->pid_int + P.kd * (err - s->pid_prev));
                const double wlo = log(in.omega0) - 10.0, whi = log(in.omega0) + 10.0;
                lw = lw < wlo ? wlo : (lw > whi ? whi : lw);
                omega = exp(lw);
                s->omega = omega;
                s->pid_prev = err;
            }
            s->tau = in.eta / omega;
            s->sigma = in.eta * omega;
            s->it = 1.0 / s->tau;
            s->R_prev_valid = 0;
            s->restarts += 1;
        }
    }
    __syncthreads();
    return restart;
}

// a / b with r = 1 / b (correctly rounded) at hand: the quotient estimate
// corrected by its exact remainder, which rounds as the division does, at 3
// operations instead of a divide's dozen.  Where that is not finite (an
// infinite operand, overflow) the division itself decides.
__device__ __forceinline__ double div_by(double a, double b, double r)
{
    const double q = a * r;
    const double c = __builtin_fma(__builtin_fma(-q, b, a), r, q);
    return isfinite(c) ? c : a / b;
}

// workgroups of a launch: `per` to a CU at most
inline int one_cu_grid(int count, int per = 1)
{
    static const int cus = [] {
        int dev = 0, c = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && c > 0)
            return c;
        return 256;
    }();
    return count < per * cus ? count : per * cus;
}

}  // namespace pdhcg
