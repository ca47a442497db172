// general.hip -- batched instances with a non-diagonal Q that one CU can hold.
//
// An instance of at most 1024 variables and rows is solved by a workgroup of
// 1024 threads that has a CU to itself, one variable and one row per thread.
// The iteration is the general batched kernel's (batch.hip), with the
// thread's row of Q and the inner solve's vectors in registers and A in LDS:
// an inner step is LDS gathers and four barriers, where the general kernel
// read Q and six vectors from memory in every step (about 30 us a step).
//
// The variables are dealt to the threads by the length of their row of Q,
// longest first: a wave's product takes as long as its longest row, so in
// index order most of its lanes would wait (random QPs: 11 entries a row on
// average, the longest of 64 rows about 25).  A thread sums its row in row
// order, as the general kernel does.
//
// FP64 only: the other order of the reductions moves results by 1e-15, but
// in mixed precision the last bit of a sum can turn the FP32 rounding of an
// operand, which moves them by 1e-8.
#include <math.h>

#include "device_math.h"
#include "one_cu.h"
#include "pdhcg_internal.h"

namespace pdhcg {

constexpr int REG_Q = 16;            // entries of a row of Q in registers
constexpr int REST_Q = 4096;         // places in LDS for the longer rows' other entries
constexpr int LDS_ALL = 160 * 1024 / 8;
constexpr int OP = REG_MAX + 2;      // an operand and its zero entry
// LDS in doubles: reductions, three operands, state, the deal of the variables
constexpr int AT_RED = 0;
constexpr int AT_OPS = AT_RED + RED_SLOTS * WAVES;        // (the check uses the first operand's space)
constexpr int AT_STEP = AT_OPS + 3 * OP;                  // two buffers of the step's reductions
constexpr int AT_STATE = AT_STEP + 2 * 4 * WAVES;
constexpr int AT_MISC = AT_STATE + (int)((sizeof(ClosedState) + 7) / 8);
constexpr int AT_DEAL = AT_MISC + 16;                     // place of a variable, variable of a place (16 bits each)
constexpr int AT_REST = AT_DEAL + 2 * REG_MAX / 4;
constexpr int AT_A = AT_REST + REST_Q + REST_Q / 4;
constexpr int A_PLACES = ((LDS_ALL - AT_A) * 8 / 10) & ~63;

// four values over the workgroup, in every thread: sums, but the last a
// minimum where MIN3.  One barrier; every wave reads the 16 waves' values in
// one load and finishes the reduction in its lane crossbar.
template <bool MIN3>
__device__ __forceinline__ void step_sum(double (&v)[4], double* lds)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[j] = wave_reduce(MIN3 && j == 3 ? R_MIN : R_SUM, v[j]);
        if (lane == 0) lds[j * WAVES + wave] = v[j];
    }
    __syncthreads();
    static_assert(WAVES == 16, "a value's partials fill a row of 16 lanes");
    double r = lds[lane];
    const bool mn = MIN3 && lane >= 48;
    const double id = mn ? INFINITY : 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double o = q == 0   ? dpp_from<0x111, 0xf>(r, id)
                         : q == 1 ? dpp_from<0x112, 0xf>(r, id)
                         : q == 2 ? dpp_from<0x114, 0xf>(r, id)
                                  : dpp_from<0x118, 0xf>(r, id);
        r = mn ? rcomb(R_MIN, r, o) : r + o;
    }
    const long long b = __double_as_longlong(r);
    const int lo = (int)(b & 0xffffffffll), hi = (int)(b >> 32);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int l = __builtin_amdgcn_readlane(lo, 16 * j + 15), h = __builtin_amdgcn_readlane(hi, 16 * j + 15);
        v[j] = __longlong_as_double(((long long)h << 32) | (long long)(unsigned)l);
    }
}

// entries of the longest row of the wave (uniform)
__device__ __forceinline__ int longest(int len)
{
    int most = 0;
    while (__ballot(len > most) != 0ull) ++most;
    return uniform_int(most);
}

// the wave's share of `total` places: `base` and how many entries of each of
// its 64 rows fit; the waves' shares follow each other
struct Share {
    int base, wide;
};
__device__ __forceinline__ Share share(int want, int total, int* widths)
{
    const int wave = uniform_int(threadIdx.x >> 6);
    if ((threadIdx.x & 63) == 0) widths[wave] = want;
    __syncthreads();
    int base = 0;
    for (int w = 0; w < wave; ++w) base += 64 * widths[w];
    Share p;
    p.base = uniform_int(base < total ? base : total);
    const int fit = (total - p.base) / 64;
    p.wide = uniform_int(want < fit ? want : fit);
    __syncthreads();
    return p;
}

// entries [from, from + wide) of the thread's row to the wave's places;
// deal: place of a column; a missing entry is 0 times the operand's zero
__device__ __forceinline__ void fill(Share p, int a, int len, int from, const double* val, const unsigned short* c16,
                                     const int* c32, int first, const unsigned short* deal, int zero, double* lv,
                                     unsigned short* lo)
{
    const int at = p.base + (threadIdx.x & 63);
    for (int k = 0; k < p.wide; ++k) {
        double v = 0.0;
        int j = zero;
        if (from + k < len) {
            v = val[a + from + k];
            j = deal[local_col(c16, c32, a + from + k, first)];
        }
        lv[at + 64 * k] = v;
        lo[at + 64 * k] = (unsigned short)j;
    }
}

__global__ __launch_bounds__(REG_MAX) void k_general_solve(BatchDev B, BatchParams P)
{
    __shared__ double sh[LDS_ALL];
    double* red = sh + AT_RED;
    double* redh = sh + AT_STEP;
    double* redu = redh + 4 * WAVES;
    double* sp = sh + AT_OPS;              // direction; x_bar
    double* sxt = sh + AT_OPS + OP;        // x_T
    double* sy = sh + AT_OPS + 2 * OP;     // y
    ClosedState* s = reinterpret_cast<ClosedState*>(sh + AT_STATE);
    int* misc = reinterpret_cast<int*>(sh + AT_MISC);       // [0] instance, [16..31] widths
    unsigned short* place = reinterpret_cast<unsigned short*>(sh + AT_DEAL);
    unsigned short* var = place + REG_MAX;
    double* lqv = sh + AT_REST;
    unsigned short* lqo = reinterpret_cast<unsigned short*>(lqv + REST_Q);
    double* lav = sh + AT_A;
    unsigned short* lao = reinterpret_cast<unsigned short*>(lav + A_PLACES);
    const int tid = threadIdx.x;

    for (;;) {
        if (tid == 0) misc[0] = atomicAdd(B.queue + 2, 1);
        __syncthreads();
        const int at = uniform_int(misc[0]);
        if (at >= B.general_count) return;
        const int b = uniform_int(B.general_list[at]);
        const unsigned long long t_start = wall_clock64();
        const ClosedInst in = closed_instance(B, b);
        const int v0 = in.v0, r0 = in.r0, n = in.n, m = in.m, unb = in.unb;
        const double normq = uniform(B.normq[b]);
        const bool xon = tid < n, yon = tid < m;
        // the deal: rows of Q by length, ties in index order
        {
            int* lens = reinterpret_cast<int*>(sh + AT_OPS);
            lens[tid] = xon ? B.qrp[v0 + tid + 1] - B.qrp[v0 + tid] : -1;
            __syncthreads();
            const int mine = lens[tid];
            int r = 0;
            for (int j = 0; j < n; ++j) {
                const int o = lens[j];
                r += (o > mine || (o == mine && j < tid)) ? 1 : 0;
            }
            if (xon) {
                place[tid] = (unsigned short)r;
                var[r] = (unsigned short)tid;
            }
            __syncthreads();
        }
        const int vi = v0 + (xon ? (int)var[tid] : 0), ri = r0 + (yon ? tid : 0);
        const int qa = xon ? B.qrp[vi] : 0, ql = xon ? B.qrp[vi + 1] - qa : 0;
        const int ta = xon ? B.trp[vi] : 0, tl = xon ? B.trp[vi + 1] - ta : 0;
        const int aa = yon ? B.arp[ri] : 0, al = yon ? B.arp[ri + 1] - aa : 0;
        const int qmost = longest(ql), amost = longest(al);
        const Share qs = share(qmost > REG_Q ? qmost - REG_Q : 0, REST_Q, misc + 16);
        const Share as = share(amost, A_PLACES, misc + 16);
        fill(qs, qa, ql, REG_Q, B.qval, B.qcol16, B.qcol, v0, place, n, lqv, lqo);
        fill(as, aa, al, 0, B.aval, B.acol16, B.acol, v0, place, n, lav, lao);
        for (int i = tid; i < 3 * OP; i += REG_MAX) sh[AT_OPS + i] = 0.0;
        __syncthreads();
        double x = 0.0, y = 0.0, xt = 0.0;
        if (xon) {
            x = clampd(0.0, B.lv[vi], B.uv[vi]);
            xt = x;
            B.xa[vi] = x;
            B.xt[vi] = x;
            sxt[tid] = x;
        }
        if (yon) {
            B.ya[ri] = 0.0;
            B.yt[ri] = 0.0;
        }
        if (tid == 0) {
            ClosedState z = {};
            z.omega = in.omega0;
            z.tau = in.eta / z.omega;
            z.sigma = in.eta * z.omega;
            z.it = 1.0 / z.tau;
            *s = z;
        }
        __syncthreads();

        double eps = INFINITY;
        long long k = 0, t = 0, inner_total = 0;
        int status = 0;
        for (;;) {
            if ((k > 0 || P.max_iter == 0) && (k % P.check_every == 0 || k >= P.max_iter)) {
                if (tid == 0) { s->k = k; s->t = t; }
                __syncthreads();
                const int restart = uniform_int(
                    one_cu_check<false, true>((unsigned long long)__builtin_amdgcn_kernarg_segment_ptr(), b, red, s));
                status = uniform_int(s->status);
                if (status) break;
                if (restart) {
                    t = 0;
                    if (xon) { x = B.xt[vi]; B.xa[vi] = x; }
                    if (yon) { y = B.yt[ri]; B.ya[ri] = y; }
                }
                if (yon) sy[tid] = y;
                __syncthreads();
            }
            if (k >= P.max_iter) { status = 4; break; }
            // The iterations to the next check (in pieces of at most 2^30);
            // the row of Q and the box are loaded here, not before the loop
            // over the checks: live across a check they would be spilled.
            double qv[REG_Q];
            unsigned qo[REG_Q / 2];   // places, two to a word
#pragma unroll
            for (int q = 0; q < REG_Q; ++q) {
                const bool have = q < ql;
                qv[q] = have ? B.qval[qa + q] : 0.0;
                const unsigned j = have ? place[local_col(B.qcol16, B.qcol, qa + q, v0)] : (unsigned)n;
                qo[q / 2] = q % 2 ? qo[q / 2] | (j << 16) : j;
            }
            const double l = xon ? B.lv[vi] : -INFINITY, u = xon ? B.uv[vi] : INFINITY;
            // row of Q times an operand in LDS, in row order
            auto qdot = [&](const double* op) __attribute__((always_inline)) {
                double r = 0.0;
#pragma unroll
                for (int q = 0; q < REG_Q; q += 4) {
                    if (q < qmost) {
                        double g[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) g[e] = op[(qo[(q + e) / 2] >> (16 * (e & 1))) & 0xffffu];
#pragma unroll
                        for (int e = 0; e < 4; ++e) r += qv[q + e] * g[e];
                    }
                }
                if (qmost > REG_Q) {
                    const int f = qs.base + (tid & 63);
                    int w = 0;
                    for (; w + 4 <= qs.wide; w += 4) {
                        double v[4], g[4];
                        unsigned o[4];
#pragma unroll
                        for (int e = 0; e < 4; ++e) { o[e] = lqo[f + 64 * (w + e)]; v[e] = lqv[f + 64 * (w + e)]; }
#pragma unroll
                        for (int e = 0; e < 4; ++e) g[e] = op[o[e]];
#pragma unroll
                        for (int e = 0; e < 4; ++e) r += v[e] * g[e];
                    }
                    for (; w < qs.wide; ++w) r += lqv[f + 64 * w] * op[lqo[f + 64 * w]];
                    for (int q = REG_Q + qs.wide; q < ql; ++q)
                        r += B.qval[qa + q] * op[place[local_col(B.qcol16, B.qcol, qa + q, v0)]];
                }
                return r;
            };
            const double it = uniform(s->it), sigma = uniform(s->sigma), tau = uniform(s->tau), omega = uniform(s->omega);
            const double abar = P.abar_scale / (normq + it);
            const double gamma2 = P.mprgp_gamma * P.mprgp_gamma;
            long long left = P.check_every - k % P.check_every;
            left = left < P.max_iter - k ? left : P.max_iter - k;
            const int steps = uniform_int((int)(left < (1ll << 30) ? left : (1ll << 30)));
            const bool last = (k + steps) % P.check_every == 0 || k + steps >= P.max_iter;   // a check follows
            for (int r = 0; r < steps; ++r) {
                const bool store = last && r + 1 == steps;
                // right-hand side, and the gradient at x_T with a product with Q
                double rhs = 0.0, g = 0.0, p = 0.0, hp = 0.0;
                double st[4] = {0.0, 0.0, 0.0, 0.0};   // ||g^P||^2, ||beta||^2, phit'phi
                {
                    double aty = 0.0;
#pragma unroll 4
                    for (int q = 0; q < tl; ++q) aty += B.tval[ta + q] * sy[local_col(B.tcol16, B.tcol, ta + q, r0)];
                    const double qx = qdot(sxt);
                    if (xon) {
                        rhs = x * it - B.c[vi] - aty;
                        g = qx + it * xt - rhs;
                        const Split f = split(xt, g, l, u, abar);
                        st[0] = f.phi * f.phi + f.beta * f.beta;
                        st[1] = f.beta * f.beta;
                        st[2] = f.phit * f.phi;
                    }
                }
                step_sum<false>(st, redu);
                if (isinf(eps) && P.eps_fixed <= 0.0) eps = uniform(fmax(P.gamma_inner * sqrt(st[0]), P.eps_min));
                const double eps_use = P.eps_fixed > 0.0 ? P.eps_fixed : eps;
                long long inner = 0;
                double gam = 0.0;
                int done = uniform_int(sqrt(st[0]) <= eps_use || P.max_inner <= 0);
                int mode = uniform_int(st[1] <= gamma2 * st[2] ? DIR_PHI : DIR_BETA);
                while (!done) {
                    if (xon) {
                        const Split f = split(xt, g, l, u, abar);
                        p = mode == DIR_BETA ? f.beta : (mode == DIR_PHI ? f.phi : f.phi - gam * p);
                        sp[tid] = p;
                    }
                    __syncthreads();
                    double hs[4] = {0.0, 0.0, 0.0, INFINITY};   // p'Hp, g'p, -, feasible step
                    const double qp = qdot(sp);
                    if (xon) {
                        hp = qp + it * p;
                        hs[0] = p * hp;
                        hs[1] = g * p;
                        if (p > 0.0 && isfinite(l)) hs[3] = (xt - l) / p;
                        else if (p < 0.0 && isfinite(u)) hs[3] = (xt - u) / p;
                    }
                    step_sum<true>(hs, redh);
                    if (uniform_int(!(hs[0] > 0.0))) break;
                    const double af = hs[3] < 0.0 ? 0.0 : hs[3];
                    const double acg = hs[1] / hs[0];
                    int kind;
                    double alpha;
                    if (mode == DIR_BETA) { kind = STEP_PROP; alpha = acg < af ? acg : af; }
                    else if (acg <= af) { kind = STEP_CG; alpha = acg; }
                    else { kind = STEP_EXPAND; alpha = af; }
                    kind = uniform_int(kind);
                    alpha = uniform(alpha);
                    double us[4] = {0.0, 0.0, 0.0, 0.0};   // the same three and phi'Hp
                    if (xon) {
                        xt = clampd(xt - alpha * p, l, u);
                        g = g - alpha * hp;
                        const Split f = split(xt, g, l, u, abar);
                        if (kind == STEP_EXPAND) {
                            xt = clampd(xt - abar * f.phi, l, u);
                            sxt[tid] = xt;
                        } else {
                            us[0] = f.phi * f.phi + f.beta * f.beta;
                            us[1] = f.beta * f.beta;
                            us[2] = f.phit * f.phi;
                            us[3] = f.phi * hp;
                        }
                    }
                    ++inner;
                    if (kind == STEP_EXPAND) {
                        __syncthreads();
                        const double qx = qdot(sxt);
                        if (xon) {
                            g = qx + it * xt - rhs;
                            const Split f = split(xt, g, l, u, abar);
                            us[0] = f.phi * f.phi + f.beta * f.beta;
                            us[1] = f.beta * f.beta;
                            us[2] = f.phit * f.phi;
                        }
                    }
                    step_sum<false>(us, redu);
                    if (kind == STEP_CG) gam = uniform(us[3] / hs[0]);
                    done = uniform_int(sqrt(us[0]) <= eps_use || inner >= P.max_inner);
                    const bool prop = us[1] <= gamma2 * us[2];
                    mode = uniform_int(!prop ? DIR_BETA : (kind == STEP_CG ? DIR_CONJ : DIR_PHI));
                }
                inner_total += inner;
                // x_bar
                if (xon) {
                    sxt[tid] = xt;
                    sp[tid] = 2.0 * xt - x;
                }
                __syncthreads();
                // dual step and the Halpern averages of y and x
                const double w = (double)(t + 1) / (double)(t + 2), wa = 1.0 / (double)(t + 2);
                const double th = P.theta;
                double dy = 0.0, dx = 0.0, lc = 0.0, uc = 0.0;
                if (amost > 0 || yon) {
                    const int f = as.base + (tid & 63);
                    double ax = 0.0;
#pragma unroll 4
                    for (int q = 0; q < as.wide; ++q) ax += lav[f + 64 * q] * sp[lao[f + 64 * q]];
                    for (int q = as.wide; q < al; ++q) ax += B.aval[aa + q] * sp[place[local_col(B.acol16, B.acol, aa + q, v0)]];
                    if (yon) {
                        lc = B.lc[ri];
                        uc = B.uc[ri];
                        const double v = y / sigma + ax;
                        const double yt = sigma * (v - clampd(v, lc, uc));
                        dy = yt - y;
                        y = P.use_halpern ? w * ((1.0 + th) * yt - th * y) + wa * B.ya[ri] : yt;
                        sy[tid] = y;
                        if (store) B.yt[ri] = yt;   // read only by the check that follows
                    }
                }
                if (xon) {
                    dx = xt - x;
                    x = P.use_halpern ? w * ((1.0 + th) * xt - th * x) + wa * B.xa[vi] : xt;
                    if (store) B.xt[vi] = xt;
                }
                double mv[4] = {dx * dx, dy * dy, 0.0, 0.0};
                step_sum<false>(mv, redh);   // its barrier also publishes y
                if (P.eps_fixed <= 0.0)
                    eps = uniform(fmin(eps, fmax(P.gamma_inner * omega * sqrt(mv[0]) / tau, P.eps_min)));
                if (store) {   // the certificate pieces
                    double a[5] = {0, 0, 0, 0, 0};
                    if (yon) {
                        const double yy = projY(dy, lc, uc);
                        B.ytil[ri] = yy;
                        a[0] = fabs(yy);
                        a[1] = supp(yy, lc, uc);
                        a[2] = supp_abs(yy, lc, uc);
                    }
                    if (xon && unb) {
                        const double di = projRec(dx, l, u);
                        B.d[vi] = di;
                        a[3] = fabs(di);
                        a[4] = B.c[vi] * di;
                    }
                    wg_sum<5, 1u | (1u << 3)>(a, red);
                    if (tid == 0) {
                        s->ytil_max = a[0]; s->ptil_sum = a[1]; s->ptil_abs = a[2];
                        s->d_max = a[3];
                        s->cd = a[4];
                    }
                }
                if (tid == 0) {
                    s->ndx2 = mv[0];
                    s->ndy2 = mv[1];
                    if (t == 0) s->R_start = sqrt(omega * mv[0] + mv[1] / omega);
                }
                ++t;
            }
            k += steps;
        }
        if (tid == 0) {
            BatchOut o;
            o.status = status;
            o.pad = 0;
            o.iterations = k;
            o.restarts = s->restarts;
            o.inner_iterations = inner_total;
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

hipError_t launch_general_solve(const BatchDev& B, const BatchParams& P, hipStream_t s)
{
    if (B.general_count < 1) return hipSuccess;
    const int grid = one_cu_grid(B.general_count);
    k_general_solve<<<grid, REG_MAX, 0, s>>>(B, P);
    return hipGetLastError();
}

}  // namespace pdhcg
