// closed.hip -- batched instances with a diagonal Q that one CU can hold.
//
// An instance of at most REG_MAX variables and rows is solved by a workgroup
// of 1024 threads that has a CU to itself: one variable and one row per
// thread.  The thread's row of A' and its iterates stay in registers, A in
// LDS (entry k of 64 consecutive rows side by side), so an iteration touches
// no memory: two products with LDS gathers, two barriers.  The general
// batched kernel (batch.hip) reads both matrices in every iteration, from the
// memory-side cache once a batch's matrices exceed the L2s: 49 us per
// iteration of a 748-variable MPC instance with four workgroups of 256
// threads on a CU, where this kernel takes 3 to 4.  16 waves rather than 4:
// with one wave on a SIMD the same work took 8 us, bound by instruction
// fetch.  Each product sums a row with one thread in row order, as the
// general kernel does.
#include <math.h>

#include <type_traits>

#include "device_math.h"
#include "pdhcg_internal.h"

namespace pdhcg {

constexpr int REG_MAX = BATCH_CLOSED_MAX;   // variables, rows, threads
constexpr int WAVES = REG_MAX / 64;
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

// Sum (bit j of MAXM clear) or maximum (set) of NR values over the
// workgroup, in a fixed order, in every thread.  The caller puts a barrier
// between two reductions' uses of `lds` (any barrier after this returns).
constexpr int RED_SLOTS = 8;
template <int NR, unsigned MAXM>
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
        for (int w = 1; w < WAVES; ++w) r = rcomb(((MAXM >> j) & 1u) ? R_MAX : R_SUM, r, lds[w * NR + j]);
        v[j] = uniform(r);
    }
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
template <bool F32>
__device__ __attribute__((noinline)) int closed_check(unsigned long long args, int b, double* red, ClosedState* s)
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
    wg_sum<4, 3u>(a, red);
    // A x_T, A d: violation (max), p(y), movement, violation of A d (max)
    double c[4] = {0.0, 0.0, 0.0, 0.0};
    if (yon) {
        const int qa = B.arp[ri], qe = B.arp[ri + 1];
        const double lc = B.lc[ri], uc = B.uc[ri], yj = yt[tid];
        double ax, ad = 0.0;
        if (later && unb) csr_dot2(qa, qe, B.acol16, B.acol, v0, B.aval, xt, d, ax, ad);
        else ax = csr_dot(qa, qe, B.acol16, B.acol, v0, B.aval, xt);
        if constexpr (F32) B.axref[ri] = ax;
        c[0] = fabs(ax - clampd(ax, lc, uc));
        c[1] = supp(yj, lc, uc);
        const double dv = yj - B.ya[ri];
        c[2] = dv * dv;
        if (later && unb) c[3] = fabs(ad - projRec(ad, lc, uc));
    }
    __syncthreads();
    wg_sum<4, 9u>(c, red);
    // Q x_T, Q d and the reduced cost: maxima 0, 1, 5 and 7, the rest sums
    double e[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (xon) {
        const double xi = xt[tid], qd = B.qd[vi], ci = B.c[vi];
        const double qx = qd * xi;
        const double r = qx + ci + aty;
        const double rh = projR(r, l, u);
        e[0] = fabs(r - rh);
        e[1] = fabs(qx);
        e[2] = xi * qx;
        e[3] = ci * xi;
        e[4] = supp(-rh, l, u);
        e[5] = fabs(xi - clampd(xi - r, l, u));
        const double dv = xi - B.xa[vi];
        e[6] = dv * dv;
        if (later && unb) e[7] = fabs(qd * d[tid]);
    }
    __syncthreads();
    wg_sum<8, (1u << 0) | (1u << 1) | (1u << 5) | (1u << 7)>(e, red);

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
        const double v1 = c[3] / s->d_max, v2 = e[7] / s->d_max / in.gammaq;
        dinf = (v1 > v2 ? v1 : v2) <= P.eps_inf;
    }
    int status = 0, restart = 0;
    double R = 0.0, omega = s->omega;
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
            const double mx = sqrt(e[6]), my = sqrt(c[2]);
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

// ---- LDS of a workgroup: the CU's 160 KB, in doubles -----------------------------

constexpr int LDS_ALL = 160 * 1024 / 8;
constexpr int LDS_RED = RED_SLOTS * WAVES;                                // wg_sum's buffer
constexpr int LDS_OP = REG_MAX + 2;                                       // an operand and its zero entry
// each thread's cost, box and anchor; mixed precision (T = float): and the
// reference point and its products
template <class T>
constexpr int lds_own() { return (sizeof(T) == 4 ? 8 : 4) * REG_MAX; }
constexpr int LDS_STATE = (int)((sizeof(ClosedState) + 7) / 8);
constexpr int LDS_MISC = 16;                                              // instance taken; widths of the waves' rows
constexpr int LDS_FIXED = LDS_RED + 2 * LDS_OP + LDS_STATE + LDS_MISC;

// places of A (a value and a 16-bit operand offset each) in what is left
template <class T>
constexpr int mat_places() { return (int)((LDS_ALL - LDS_FIXED - lds_own<T>()) * 8 / (sizeof(T) + 2)) & ~63; }

// entries of the longest row of the wave (uniform)
__device__ __forceinline__ int wave_longest(int len)
{
    int most = 0;
    while (__ballot(len > most) != 0ull) ++most;
    return uniform_int(most);
}

// A wave's rows of A in LDS: `wide` entries of each of its 64 rows from place
// `base` on, entry after entry.  The waves' places follow each other; where
// the space ends, the rest of the rows' entries is read from memory.
struct WaveMat {
    int base, wide;
};
template <class T>
__device__ __forceinline__ WaveMat place_rows(int most, int* widths)
{
    const int wave = uniform_int(threadIdx.x >> 6);
    if ((threadIdx.x & 63) == 0) widths[wave] = most;
    __syncthreads();
    int base = 0;
    for (int w = 0; w < wave; ++w) base += 64 * widths[w];
    WaveMat p;
    p.base = uniform_int(base < mat_places<T>() ? base : mat_places<T>());
    const int fit = (mat_places<T>() - p.base) / 64;
    p.wide = uniform_int(most < fit ? most : fit);
    __syncthreads();
    return p;
}

// Loads the first CAP entries of the thread's row (a, len) into registers:
// values, and offsets in bytes into the operand.  A missing entry is 0 times
// the operand's entry `zero`, a zero, so a wave's rows need no masks.
template <class T, int CAP>
__device__ __forceinline__ void load_row(int a, int len, const T* val, const unsigned short* c16, const int* c32, int first,
                                         int zero, T (&v)[CAP], unsigned (&o)[CAP])
{
#pragma unroll
    for (int k = 0; k < CAP; ++k) {
        v[k] = T(0);
        o[k] = (unsigned)(zero * (int)sizeof(T));
        if (k < len) {
            v[k] = val[a + k];
            o[k] = (unsigned)(local_col(c16, c32, a + k, first) * (int)sizeof(T));
        }
    }
}

// the same for a wave's rows of A in LDS
template <class T>
__device__ __forceinline__ void load_mat(WaveMat p, int a, int len, const T* val, const unsigned short* c16, const int* c32,
                                         int first, int zero, T* lv, unsigned short* lo)
{
    const int at = p.base + (threadIdx.x & 63);
    for (int k = 0; k < p.wide; ++k) {
        T v = T(0);
        int j = zero;
        if (k < len) {
            v = val[a + k];
            j = local_col(c16, c32, a + k, first);
        }
        lv[at + 64 * k] = v;
        lo[at + 64 * k] = (unsigned short)(j * (int)sizeof(T));
    }
}

template <class T>
__device__ __forceinline__ T at_offset(const T* x, unsigned bytes)
{
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(x) + bytes);
}

// row of A' in registers times the operand x, in row order; `most`: entries
// of the wave's longest row
template <class T, int CAP>
__device__ __forceinline__ T dot_row(const T (&v)[CAP], const unsigned (&o)[CAP], int most, int a, int len, const T* val,
                                     const unsigned short* c16, const int* c32, int first, const T* x)
{
    T s = T(0);
#pragma unroll
    for (int k = 0; k < CAP; k += 4) {
        if (k < most) {
            T g[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) g[q] = at_offset(x, o[k + q]);
#pragma unroll
            for (int q = 0; q < 4; ++q) s += v[k + q] * g[q];
        }
    }
    if (most > CAP)
        for (int k = CAP; k < len; ++k) s += val[a + k] * x[local_col(c16, c32, a + k, first)];
    return s;
}

// row of A in LDS times the operand x, in row order
template <class T>
__device__ __forceinline__ T dot_mat(WaveMat p, int most, const T* lv, const unsigned short* lo, int a, int len,
                                     const T* val, const unsigned short* c16, const int* c32, int first, const T* x)
{
    const int at = p.base + (threadIdx.x & 63);
    T s = T(0);
    int k = 0;
    for (; k + 4 <= p.wide; k += 4) {
        T v[4], g[4];
        unsigned o[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) { o[q] = lo[at + 64 * (k + q)]; v[q] = lv[at + 64 * (k + q)]; }
#pragma unroll
        for (int q = 0; q < 4; ++q) g[q] = at_offset(x, o[q]);
#pragma unroll
        for (int q = 0; q < 4; ++q) s += v[q] * g[q];
    }
    for (; k < p.wide; ++k) s += lv[at + 64 * k] * at_offset(x, lo[at + 64 * k]);
    if (most > p.wide)
        for (int q = p.wide; q < len; ++q) s += val[a + q] * x[local_col(c16, c32, a + q, first)];
    return s;
}

// ---- the solve -------------------------------------------------------------------

template <bool F32>
__global__ __launch_bounds__(REG_MAX) void k_closed_solve(BatchDev B, BatchParams P)
{
    typedef typename std::conditional<F32, float, double>::type T;
    __shared__ double sh[LDS_ALL];
    double* red = sh;
    T* sx = reinterpret_cast<T*>(sh + LDS_RED);                // x_bar (mixed: minus x_ref)
    T* sy = reinterpret_cast<T*>(sh + LDS_RED + LDS_OP);       // y (mixed: minus y_ref)
    ClosedState* s = reinterpret_cast<ClosedState*>(sh + LDS_RED + 2 * LDS_OP);
    int* misc = reinterpret_cast<int*>(sh + LDS_RED + 2 * LDS_OP + LDS_STATE);   // [0] instance, [16..31] widths
    double* own = sh + LDS_FIXED + threadIdx.x;
    T* lav = reinterpret_cast<T*>(sh + LDS_FIXED + lds_own<T>());
    unsigned short* lao = reinterpret_cast<unsigned short*>(lav + mat_places<T>());
    const int tid = threadIdx.x;
    const T *aval, *tval;
    if constexpr (F32) { aval = B.aval32; tval = B.tval32; }
    else { aval = B.aval; tval = B.tval; }

    for (;;) {
        if (tid == 0) misc[0] = atomicAdd(B.queue + 1, 1);
        __syncthreads();
        const int at = uniform_int(misc[0]);
        if (at >= B.closed_count) return;
        const int b = uniform_int(B.closed_list[at]);
        const unsigned long long t_start = wall_clock64();
        const ClosedInst in = closed_instance(B, b);
        const int v0 = in.v0, r0 = in.r0, n = in.n, m = in.m, unb = in.unb;
        const bool xon = tid < n, yon = tid < m;
        const int vi = v0 + (xon ? tid : 0), ri = r0 + (yon ? tid : 0);
        const int ta = xon ? B.trp[vi] : 0, tl = xon ? B.trp[vi + 1] - ta : 0;
        const int aa = yon ? B.arp[ri] : 0, al = yon ? B.arp[ri + 1] - aa : 0;
        const int tmost = wave_longest(tl), amost = wave_longest(al);
        const WaveMat wm = place_rows<T>(amost, misc + 16);
        load_mat<T>(wm, aa, al, aval, B.acol16, B.acol, v0, n, lav, lao);
        double x = 0.0, y = 0.0;
        if (xon) {
            x = clampd(0.0, B.lv[vi], B.uv[vi]);
            B.xa[vi] = x;
            B.xt[vi] = x;
        }
        if (yon) {
            B.ya[ri] = 0.0;
            B.yt[ri] = 0.0;
        }
        for (int i = tid; i < 2 * LDS_OP; i += REG_MAX) sh[LDS_RED + i] = 0.0;
        if (tid == 0) {
            ClosedState z = {};
            z.omega = in.omega0;
            z.tau = in.eta / z.omega;
            z.sigma = in.eta * z.omega;
            z.it = 1.0 / z.tau;
            *s = z;
        }
        __syncthreads();

        long long k = 0, t = 0;   // iterations, and those of the round
        bool seen = false;        // a check has run (mixed precision: the reference point is its point)
        int status = 0;
        for (;;) {
            if ((k > 0 || P.max_iter == 0) && (k % P.check_every == 0 || k >= P.max_iter)) {
                if (tid == 0) { s->k = k; s->t = t; }
                __syncthreads();
                const int restart = uniform_int(
                    closed_check<F32>((unsigned long long)__builtin_amdgcn_kernarg_segment_ptr(), b, red, s));
                status = uniform_int(s->status);
                if (status) break;
                seen = true;
                if (restart) {
                    t = 0;
                    if (xon) { x = B.xt[vi]; B.xa[vi] = x; }
                    if (yon) { y = B.yt[ri]; B.ya[ri] = y; }
                }
                if (yon) {
                    if constexpr (F32) sy[tid] = (float)(y - B.yt[ri]);
                    else sy[tid] = y;
                }
                __syncthreads();
            }
            if (k >= P.max_iter) { status = 4; break; }
            // The iterations to the next check (in pieces of at most 2^30).
            // What they hold in registers is loaded here, not before the loop
            // over the checks: live across a check it would be spilled.  Step
            // sizes change only at a check: the divisors' reciprocals.
            double ya = 0.0, lc = 0.0, uc = 0.0, qd = 1.0;
            if (xon) {
                qd = B.qd[vi];
                own[0] = B.c[vi];
                own[REG_MAX] = B.lv[vi];
                own[2 * REG_MAX] = B.uv[vi];
                own[3 * REG_MAX] = B.xa[vi];
                if constexpr (F32) {
                    own[4 * REG_MAX] = seen ? B.aty[vi] : 0.0;
                    own[5 * REG_MAX] = seen ? B.xt[vi] : 0.0;
                }
            }
            if (yon) {
                lc = B.lc[ri];
                uc = B.uc[ri];
                ya = B.ya[ri];
                if constexpr (F32) {
                    own[6 * REG_MAX] = seen ? B.axref[ri] : 0.0;
                    own[7 * REG_MAX] = seen ? B.yt[ri] : 0.0;
                }
            }
            T tv[REG_T];
            unsigned to[REG_T];
            load_row<T, REG_T>(ta, tl, tval, B.tcol16, B.tcol, r0, m, tv, to);
            const double it = uniform(s->it), sigma = uniform(s->sigma), rsig = 1.0 / sigma;
            const double den = qd + it, rden = 1.0 / den;
            long long left = P.check_every - k % P.check_every;
            left = left < P.max_iter - k ? left : P.max_iter - k;
            const int steps = uniform_int((int)(left < (1ll << 30) ? left : (1ll << 30)));
            const bool last = (k + steps) % P.check_every == 0 || k + steps >= P.max_iter;   // a check follows
            const double th1 = 1.0 + P.theta, th = P.theta;
            const int halpern = P.use_halpern;
            double td = (double)t;
            for (int r = 0; r < steps; ++r) {
                const bool store = last && r + 1 == steps;
                const bool opens = r == 0 && t == 0;
                const double w = (td + 1.0) / (td + 2.0), wa = 1.0 / (td + 2.0);
                td += 1.0;
                double dx = 0.0, dy = 0.0;
                // primal step (Section 2.2), x_bar, and the Halpern average of x
                if (tmost > 0 || xon) {
                    const T p = dot_row<T, REG_T>(tv, to, tmost, ta, tl, tval, B.tcol16, B.tcol, r0, sy);
                    double sd = (double)p;
                    if constexpr (F32) sd = own[4 * REG_MAX] + sd;
                    const double c = own[0], l = own[REG_MAX], u = own[2 * REG_MAX], xa = own[3 * REG_MAX];
                    const double v = clampd(div_by(x * it - c - sd, den, rden), l, u);
                    const double xb = 2.0 * v - x;
                    dx = v - x;
                    if (xon) {
                        if constexpr (F32) sx[tid] = (float)(xb - own[5 * REG_MAX]);
                        else sx[tid] = xb;
                        if (store) B.xt[vi] = v;   // read only by the check that follows
                        x = halpern ? w * (th1 * v - th * x) + wa * xa : v;
                    }
                }
                __syncthreads();
                // dual step and the Halpern average of y
                if (amost > 0 || yon) {
                    const T p = dot_mat<T>(wm, amost, lav, lao, aa, al, aval, B.acol16, B.acol, v0, sx);
                    double sd = (double)p;
                    if constexpr (F32) sd = own[6 * REG_MAX] + sd;
                    const double v = div_by(y, sigma, rsig) + sd;
                    const double yt = sigma * (v - clampd(v, lc, uc));
                    dy = yt - y;
                    if (yon) {
                        y = halpern ? w * (th1 * yt - th * y) + wa * ya : yt;
                        if constexpr (F32) sy[tid] = (float)(y - own[7 * REG_MAX]);
                        else sy[tid] = y;
                        if (store) B.yt[ri] = yt;
                    }
                }
                // movements and certificate pieces, only where something reads
                // them: the round's first step, and the step before a check
                if (store || opens) {
                    double a[7] = {0, 0, 0, 0, 0, 0, 0};
                    if (xon) {
                        a[0] = dx * dx;
                        if (store && unb) {
                            const double di = projRec(dx, own[REG_MAX], own[2 * REG_MAX]);
                            B.d[vi] = di;
                            a[5] = fabs(di);
                            a[6] = own[0] * di;
                        }
                    }
                    if (yon) {
                        a[1] = dy * dy;
                        if (store) {
                            const double yy = projY(dy, lc, uc);
                            B.ytil[ri] = yy;
                            a[2] = fabs(yy);
                            a[3] = supp(yy, lc, uc);
                            a[4] = supp_abs(yy, lc, uc);
                        }
                    }
                    __syncthreads();
                    wg_sum<7, (1u << 2) | (1u << 5)>(a, red);   // its barrier also publishes sy
                    if (tid == 0) {
                        s->ndx2 = a[0];
                        s->ndy2 = a[1];
                        if (store) {
                            s->ytil_max = a[2]; s->ptil_sum = a[3]; s->ptil_abs = a[4];
                            s->d_max = unb ? a[5] : 0.0;
                            s->cd = unb ? a[6] : 0.0;
                        }
                        if (opens) s->R_start = sqrt(s->omega * a[0] + a[1] / s->omega);
                    }
                } else {
                    __syncthreads();
                }
            }
            k += steps;
            t += steps;
        }
        if (tid == 0) {
            BatchOut o;
            o.status = status;
            o.pad = 0;
            o.iterations = k;
            o.restarts = s->restarts;
            o.inner_iterations = 0;
            o.r_primal = s->rp; o.r_dual = s->rd; o.r_gap = s->rg;
            o.pobj = s->pobj; o.dobj = s->dobj; o.omega = s->omega;
            o.ytil_max = s->ytil_max; o.d_max = s->d_max;
            o.t_start = t_start;
            o.t_end = wall_clock64();
            B.out[b] = o;
        }
        __syncthreads();
    }
}

// ---- ||A_b||_2 by power iteration on A_b'A_b --------------------------------------
//
// The same residency for the norm of an instance: its row of A' in
// registers, A in LDS, two products and three barriers per iteration (the
// general kernel re-reads both matrices: 7.8 ms for a batch of 8 MPC
// instances, about half of a whole solve from host arrays).
__global__ __launch_bounds__(REG_MAX) void k_closed_norm(BatchDev B, double tol, long long max_iter, double* out)
{
    __shared__ double sh[LDS_ALL];
    double* red = sh;
    double* sv = sh + LDS_RED;                 // v, and its zero entry
    double* sw = sh + LDS_RED + LDS_OP;        // w = A v
    int* misc = reinterpret_cast<int*>(sh + LDS_RED + 2 * LDS_OP + LDS_STATE);
    double* lav = sh + LDS_FIXED;
    unsigned short* lao = reinterpret_cast<unsigned short*>(lav + mat_places<double>());
    const int tid = threadIdx.x;
    for (;;) {
        if (tid == 0) misc[0] = atomicAdd(B.queue + 1, 1);
        __syncthreads();
        const int at = uniform_int(misc[0]);
        if (at >= B.closed_count) return;
        const int b = uniform_int(B.closed_list[at]);
        const int v0 = uniform_int(B.voff[b]), n = uniform_int(B.voff[b + 1]) - v0;
        const int r0 = uniform_int(B.roff[b]), m = uniform_int(B.roff[b + 1]) - r0;
        const bool xon = tid < n, yon = tid < m;
        const int ta = xon ? B.trp[v0 + tid] : 0, tl = xon ? B.trp[v0 + tid + 1] - ta : 0;
        const int aa = yon ? B.arp[r0 + tid] : 0, al = yon ? B.arp[r0 + tid + 1] - aa : 0;
        const int tmost = wave_longest(tl), amost = wave_longest(al);
        const WaveMat wm = place_rows<double>(amost, misc + 16);
        load_mat<double>(wm, aa, al, B.aval, B.acol16, B.acol, v0, n, lav, lao);
        for (int i = tid; i < 2 * LDS_OP; i += REG_MAX) sh[LDS_RED + i] = 0.0;
        double tv[REG_T];
        unsigned to[REG_T];
        load_row<double, REG_T>(ta, tl, B.tval, B.tcol16, B.tcol, r0, m, tv, to);
        // start vector: SplitMix64 of the local index (seed 0), in [-1, 1)
        double v = 0.0;
        if (xon) {
            unsigned long long z = (static_cast<unsigned long long>(tid) + 1ull) * 0x9E3779B97F4A7C15ull;
            z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
            z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
            z ^= z >> 31;
            v = 2.0 * ((double)(z >> 11) * (1.0 / 9007199254740992.0)) - 1.0;
        }
        double acc[1] = {v * v};
        __syncthreads();
        wg_sum<1, 0u>(acc, red);
        if (xon) sv[tid] = v / sqrt(acc[0]);
        __syncthreads();
        double sig = 0.0, prev = 0.0;
        for (long long i = 1; i <= max_iter; ++i) {
            double w = 0.0;
            if (amost > 0) w = dot_mat<double>(wm, amost, lav, lao, aa, al, B.aval, B.acol16, B.acol, v0, sv);
            if (yon) sw[tid] = w;
            acc[0] = yon ? w * w : 0.0;
            wg_sum<1, 0u>(acc, red);   // its barrier also publishes w
            sig = sqrt(acc[0]);
            if (uniform_int(sig == 0.0)) break;
            double u = 0.0;
            if (tmost > 0) u = dot_row<double, REG_T>(tv, to, tmost, ta, tl, B.tval, B.tcol16, B.tcol, r0, sw);
            acc[0] = xon ? u * u : 0.0;
            __syncthreads();
            wg_sum<1, 0u>(acc, red);
            const double nu = sqrt(acc[0]);
            if (uniform_int(nu == 0.0)) break;
            if (xon) sv[tid] = u / nu;
            __syncthreads();
            if (uniform_int(fabs(sig - prev) <= tol * sig)) break;
            prev = sig;
        }
        if (tid == 0) out[b] = sig;
        __syncthreads();
    }
}

// ---- launches ----------------------------------------------------------------------

static int closed_grid(int count)
{
    static const int cus = [] {
        int dev = 0, c = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && c > 0)
            return c;
        return 256;
    }();
    return count < cus ? count : cus;
}

hipError_t launch_closed_solve(const BatchDev& B, const BatchParams& P, hipStream_t s)
{
    if (B.closed_count < 1) return hipSuccess;
    const int grid = closed_grid(B.closed_count);
    if (B.aval32) k_closed_solve<true><<<grid, REG_MAX, 0, s>>>(B, P);
    else k_closed_solve<false><<<grid, REG_MAX, 0, s>>>(B, P);
    return hipGetLastError();
}

hipError_t launch_closed_norm(const BatchDev& B, double tol, long long max_iter, double* out, hipStream_t s)
{
    if (B.closed_count < 1) return hipSuccess;
    k_closed_norm<<<closed_grid(B.closed_count), REG_MAX, 0, s>>>(B, tol, max_iter, out);
    return hipGetLastError();
}

}  // namespace pdhcg
