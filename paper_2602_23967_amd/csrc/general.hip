// general.hip -- batched instances with a non-diagonal Q that one CU can hold.
//
// An instance of at most 1024 variables and rows is solved by a workgroup of
// 1024 threads that has a CU to itself, one variable and one row per thread.
// The iteration is the general batched kernel's (batch.hip), with the
// thread's row of Q and the inner solve's vectors in registers and A in LDS:
// an inner step is LDS gathers and three barriers, where the general kernel
// read Q and six vectors from memory in every step.  24 random QPs of 200 to
// 1000 variables, 320 iterations: 76 ms there, 19.4 here, 4.6 to 5.5 us an
// inner step with its share of the outer one.  What is left is bound by
// instruction issue: 16 waves of some 700 instructions a step.
//
// An instance of at most 256 variables and rows takes a workgroup of 256
// threads and a quarter of the CU's LDS, so that four share the CU: most of
// 1024 threads would only take part in the barriers and the sums, and a batch
// that fills the chip was slower than in the general kernel, which kept four
// instances on a CU (128 iterations of 1024 random QPs, general kernel, 1024
// threads and 256: 128 variables 6.2, 8.1 and 2.4 ms, 256 9.6, 8.7 and 3.0;
// 48 of them 4.4, 2.1 and 1.6, 4.8, 2.3 and 1.8).  Both sizes of workgroup
// make the same results to the bit: the waves that only the larger one has
// add zeros at the end of every sum.
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

constexpr int REG_Q = ONE_CU_REG_Q;     // entries of a row of Q in registers
// A workgroup of T threads and its share of the CU's 160 KB of LDS, in
// doubles: reductions, three operands, state, the deal of the variables, and
// places (a value and a 16-bit operand index each) for what the registers do
// not hold of Q and, after it, A
template <int T>
struct Cu {
    static constexpr int WAVES = T / 64;
    static constexpr int ALL = 160 * 1024 / 8 / (REG_MAX / T);
    static constexpr int OP = T + 2;                               // an operand and its zero entry
    static constexpr int AT_OPS = RED_SLOTS * WAVES;               // (the check uses the first operand's space)
    static constexpr int AT_STEP = AT_OPS + 3 * OP;                // two buffers of the step's reductions
    static constexpr int AT_STATE = AT_STEP + 2 * 16 * WAVES;
    static constexpr int AT_MISC = AT_STATE + (int)((sizeof(ClosedState) + 7) / 8);
    static constexpr int AT_DEAL = AT_MISC + 16;                   // place of a variable, variable of a place (16 bits each)
    static constexpr int AT_MAT = AT_DEAL + 2 * T / 4;
    static constexpr int PLACES = ((ALL - AT_MAT) * 8 / 10) & ~63;
};
static_assert(ONE_CU_REST_Q <= Cu<REG_MAX>::PLACES && ONE_CU_SMALL_Q <= Cu<ONE_CU_SMALL>::PLACES, "Q has to fit");

// v of the lane `CTRL` names, lanes without a source 0
template <int CTRL>
__device__ __forceinline__ double row_from(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
// sum over a row of 16 lanes, in its lane 15
__device__ __forceinline__ double row_sum(double v)
{
    v += row_from<0x111>(v);
    v += row_from<0x112>(v);
    v += row_from<0x114>(v);
    return v + row_from<0x118>(v);
}
__device__ __forceinline__ double lesser(double a, double b) { return b < a ? b : a; }
__device__ __forceinline__ double row_min(double v)
{
    v = lesser(v, dpp_from<0x111, 0xf>(v, INFINITY));
    v = lesser(v, dpp_from<0x112, 0xf>(v, INFINITY));
    v = lesser(v, dpp_from<0x114, 0xf>(v, INFINITY));
    return lesser(v, dpp_from<0x118, 0xf>(v, INFINITY));
}

// Four values over the workgroup, in every thread: sums, but the last a
// minimum where MIN3.  One barrier.  The kernel is bound by instruction
// issue (4 waves on a SIMD), so a wave reduces no further than its rows of
// 16 lanes; then every wave reads all rows' partials, 16 lanes for each
// value.  live: the wave has a variable (otherwise its values are the
// identities).
template <int T, bool MIN3>
__device__ __forceinline__ void step_sum(double (&v)[4], bool live, double* lds)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int WAVES = T / 64, PER = WAVES / 4;   // partials that a lane reads
    static_assert(PER == 1 || PER == 4, "a value's partials are shared by 16 lanes");
    if (live) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = MIN3 && j == 3 ? row_min(v[j]) : (MIN3 && j == 2 ? 0.0 : row_sum(v[j]));
    }
    if ((lane & 15) == 15) {
#pragma unroll
        for (int j = 0; j < 4; ++j) lds[(j * WAVES + wave) * 4 + (lane >> 4)] = v[j];
    }
    __syncthreads();
    const double* q = lds + PER * lane;
    double sum = q[0], least = q[0];
    if constexpr (PER == 4) {
        sum = (q[0] + q[1]) + (q[2] + q[3]);
        least = lesser(lesser(q[0], q[1]), lesser(q[2], q[3]));
    }
    double r = row_sum(sum);
    if constexpr (MIN3) {
        const double mn = row_min(least);
        r = lane >= 48 ? mn : r;
    }
    const long long b = __double_as_longlong(r);
    const int lo = (int)(b & 0xffffffffll), hi = (int)(b >> 32);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int l = __builtin_amdgcn_readlane(lo, 16 * j + 15), h = __builtin_amdgcn_readlane(hi, 16 * j + 15);
        v[j] = __longlong_as_double(((long long)h << 32) | (long long)(unsigned)l);
    }
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

// the thread's row of Q: REG_Q entries in registers (places of their columns
// two to a word), the others in its wave's share of the LDS
struct RowQ {
    double v[REG_Q];
    unsigned o[REG_Q / 2];
    int most;            // entries of the wave's longest row
    int base, wide;
    const double* lv;
    const unsigned short* lo;

    __device__ __forceinline__ void load(int a, int len, const double* val, const unsigned short* c16, const int* c32,
                                         int first, const unsigned short* deal, int zero)
    {
#pragma unroll
        for (int q = 0; q < REG_Q; ++q) {
            const bool have = q < len;
            v[q] = have ? val[a + q] : 0.0;
            const unsigned j = have ? deal[local_col(c16, c32, a + q, first)] : (unsigned)zero;
            o[q / 2] = q % 2 ? o[q / 2] | (j << 16) : j;
        }
    }
    // times an operand in LDS, in row order
    __device__ __forceinline__ double dot(const double* op) const
    {
        double r = 0.0;
#pragma unroll
        for (int q = 0; q < REG_Q; q += 4) {
            if (q < most) {
                double g[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) g[e] = op[(o[(q + e) / 2] >> (16 * (e & 1))) & 0xffffu];
#pragma unroll
                for (int e = 0; e < 4; ++e) r += v[q + e] * g[e];
            }
        }
        if (wide > 0) {
            const int f = base + (threadIdx.x & 63);
            int w = 0;
            for (; w + 4 <= wide; w += 4) {
                double x[4], g[4];
                unsigned c[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) { c[e] = lo[f + 64 * (w + e)]; x[e] = lv[f + 64 * (w + e)]; }
#pragma unroll
                for (int e = 0; e < 4; ++e) g[e] = op[c[e]];
#pragma unroll
                for (int e = 0; e < 4; ++e) r += x[e] * g[e];
            }
            for (; w < wide; ++w) r += lv[f + 64 * w] * op[lo[f + 64 * w]];
        }
        return r;
    }
};

// The boxed CG inner solve (MPRGP) of the subproblem with right-hand side
// rhs from x_T = xt with gradient g; st: ||g^P||^2, ||beta||^2 and phit'phi
// there, left as they are at the end.  live: the wave has a variable.
struct Inner {
    double it, abar, gamma2, eps;
    long long max_inner;
    long long steps = 0, products = 0;
};
template <int T>
__device__ __forceinline__ void inner_solve(Inner& s, const RowQ& Q, bool on, bool live, double l, double u, double rhs,
                                            double& xt, double& g, double (&st)[4], double* sp, double* sxt, double* redh,
                                            double* redu)
{
    const int tid = threadIdx.x;
    double p = 0.0, hp = 0.0, gam = 0.0;
    int done = uniform_int(sqrt(st[0]) <= s.eps || s.max_inner <= 0);
    int mode = uniform_int(st[1] <= s.gamma2 * st[2] ? DIR_PHI : DIR_BETA);
    while (!done) {
        if (on) {
            const Split f = split(xt, g, l, u, s.abar);
            p = mode == DIR_BETA ? f.beta : (mode == DIR_PHI ? f.phi : f.phi - gam * p);
            sp[tid] = p;
        }
        __syncthreads();
        double hs[4] = {0.0, 0.0, 0.0, INFINITY};   // p'Hp, g'p, -, feasible step
        if (live) {
            const double qp = Q.dot(sp);
            if (on) {
                hp = qp + s.it * p;
                hs[0] = p * hp;
                hs[1] = g * p;
                if (p > 0.0 && isfinite(l)) hs[3] = (xt - l) / p;
                else if (p < 0.0 && isfinite(u)) hs[3] = (xt - u) / p;
            }
        }
        ++s.products;
        step_sum<T, true>(hs, live, redh);
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
        if (on) {
            xt = clampd(xt - alpha * p, l, u);
            g = g - alpha * hp;
            const Split f = split(xt, g, l, u, s.abar);
            if (kind == STEP_EXPAND) {
                xt = clampd(xt - s.abar * f.phi, l, u);
                sxt[tid] = xt;
            } else {
                us[0] = f.phi * f.phi + f.beta * f.beta;
                us[1] = f.beta * f.beta;
                us[2] = f.phit * f.phi;
                us[3] = f.phi * hp;
            }
        }
        ++s.steps;
        if (kind == STEP_EXPAND) {
            __syncthreads();
            ++s.products;
            if (live) {
                const double qx = Q.dot(sxt);
                if (on) {
                    g = qx + s.it * xt - rhs;
                    const Split f = split(xt, g, l, u, s.abar);
                    us[0] = f.phi * f.phi + f.beta * f.beta;
                    us[1] = f.beta * f.beta;
                    us[2] = f.phit * f.phi;
                }
            }
        }
        step_sum<T, false>(us, live, redu);
        if (kind == STEP_CG) gam = uniform(us[3] / hs[0]);
        st[0] = us[0];
        done = uniform_int(sqrt(us[0]) <= s.eps || s.steps >= s.max_inner);
        const bool prop = us[1] <= s.gamma2 * us[2];
        mode = uniform_int(!prop ? DIR_BETA : (kind == STEP_CG ? DIR_CONJ : DIR_PHI));
    }
}

// the deal of the variables to the threads: rows of Q by length, ties in
// index order
__device__ __forceinline__ void deal_rows(int n, const int* rp, int* lens, unsigned short* place, unsigned short* var)
{
    const int tid = threadIdx.x;
    lens[tid] = tid < n ? rp[tid + 1] - rp[tid] : -1;
    __syncthreads();
    const int mine = lens[tid];
    int r = 0;
    for (int j = 0; j < n; ++j) {
        const int o = lens[j];
        r += (o > mine || (o == mine && j < tid)) ? 1 : 0;
    }
    if (tid < n) {
        place[tid] = (unsigned short)r;
        var[r] = (unsigned short)tid;
    }
    __syncthreads();
}

template <int T>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(4))) void k_general_solve(BatchDev B, BatchParams P)
{
    typedef Cu<T> L;
    __shared__ double sh[L::ALL];
    double* red = sh;
    double* redh = sh + L::AT_STEP;
    double* redu = redh + 16 * L::WAVES;
    double* sp = sh + L::AT_OPS;              // direction; x_bar
    double* sxt = sh + L::AT_OPS + L::OP;     // x_T
    double* sy = sh + L::AT_OPS + 2 * L::OP;  // y
    ClosedState* s = reinterpret_cast<ClosedState*>(sh + L::AT_STATE);
    int* misc = reinterpret_cast<int*>(sh + L::AT_MISC);       // [0] instance, [16..31] widths
    unsigned short* place = reinterpret_cast<unsigned short*>(sh + L::AT_DEAL);
    unsigned short* var = place + T;
    double* lv = sh + L::AT_MAT;
    unsigned short* lo = reinterpret_cast<unsigned short*>(lv + L::PLACES);
    const int tid = threadIdx.x;

    const int count = T == REG_MAX ? B.general_count : B.small_count;
    const int* list = T == REG_MAX ? B.general_list : B.small_list;

    for (;;) {
        if (tid == 0) misc[0] = atomicAdd(B.queue + (T == REG_MAX ? 2 : 3), 1);
        __syncthreads();
        const int at = uniform_int(misc[0]);
        if (at >= count) return;
        const int b = uniform_int(list[at]);
        const unsigned long long t_start = wall_clock64();
        const ClosedInst in = closed_instance(B, b);
        const int v0 = in.v0, r0 = in.r0, n = in.n, m = in.m, unb = in.unb;
        const double normq = uniform(B.normq[b]);
        const bool xon = tid < n, yon = tid < m;
        deal_rows(n, B.qrp + v0, reinterpret_cast<int*>(sh + L::AT_OPS), place, var);
        const int vi = v0 + (xon ? (int)var[tid] : 0), ri = r0 + (yon ? tid : 0);
        const int qa = xon ? B.qrp[vi] : 0, ql = xon ? B.qrp[vi + 1] - qa : 0;
        const int ta = xon ? B.trp[vi] : 0, tl = xon ? B.trp[vi + 1] - ta : 0;
        const int aa = yon ? B.arp[ri] : 0, al = yon ? B.arp[ri + 1] - aa : 0;
        const int qmost = wave_longest(ql), amost = wave_longest(al);
        const bool live = uniform_int(tid & ~63) < n, any = uniform_int(tid & ~63) < (n > m ? n : m);
        RowQ Q;
        Q.most = qmost;
        const Share qs = share<T>(qmost > REG_Q ? qmost - REG_Q : 0, 0, L::PLACES, misc + 16);
        const Share as = share<T>(amost, qs.end, L::PLACES, misc + 16);
        Q.base = qs.base;
        Q.wide = qs.wide;
        Q.lv = lv;
        Q.lo = lo;
        fill(qs, qa, ql, REG_Q, B.qval, B.qcol16, B.qcol, v0, place, n, lv, lo);
        fill(as, aa, al, 0, B.aval, B.acol16, B.acol, v0, place, n, lv, lo);
        for (int i = tid; i < 3 * L::OP; i += T) sh[L::AT_OPS + i] = 0.0;
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
                    one_cu_check<false, true, T>((unsigned long long)__builtin_amdgcn_kernarg_segment_ptr(), b, red, s));
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
            Q.load(qa, ql, B.qval, B.qcol16, B.qcol, v0, place, n);
            const double l = xon ? B.lv[vi] : -INFINITY, u = xon ? B.uv[vi] : INFINITY;
            const double it = uniform(s->it), sigma = uniform(s->sigma), tau = uniform(s->tau), omega = uniform(s->omega);
            Inner cg;
            cg.it = it;
            cg.abar = P.abar_scale / (normq + it);
            cg.gamma2 = P.mprgp_gamma * P.mprgp_gamma;
            cg.max_inner = P.max_inner;
            long long left = P.check_every - k % P.check_every;
            left = left < P.max_iter - k ? left : P.max_iter - k;
            const int steps = uniform_int((int)(left < (1ll << 30) ? left : (1ll << 30)));
            const bool last = (k + steps) % P.check_every == 0 || k + steps >= P.max_iter;   // a check follows
            for (int r = 0; r < steps; ++r) {
                const bool store = last && r + 1 == steps;
                // right-hand side, and the gradient at x_T with a product with Q
                double rhs = 0.0, g = 0.0;
                double st[4] = {0.0, 0.0, 0.0, 0.0};   // ||g^P||^2, ||beta||^2, phit'phi
                {
                    double aty = 0.0;
#pragma unroll 4
                    for (int q = 0; q < tl; ++q) aty += B.tval[ta + q] * sy[local_col(B.tcol16, B.tcol, ta + q, r0)];
                    const double qx = Q.dot(sxt);
                    if (xon) {
                        rhs = x * it - B.c[vi] - aty;
                        g = qx + it * xt - rhs;
                        const Split f = split(xt, g, l, u, cg.abar);
                        st[0] = f.phi * f.phi + f.beta * f.beta;
                        st[1] = f.beta * f.beta;
                        st[2] = f.phit * f.phi;
                    }
                }
                step_sum<T, false>(st, live, redu);
                if (isinf(eps) && P.eps_fixed <= 0.0) eps = uniform(fmax(P.gamma_inner * sqrt(st[0]), P.eps_min));
                cg.eps = P.eps_fixed > 0.0 ? P.eps_fixed : eps;
                cg.steps = 0;
                inner_solve<T>(cg, Q, xon, live, l, u, rhs, xt, g, st, sp, sxt, redh, redu);
                inner_total += cg.steps;
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
                    for (int q = 0; q < as.wide; ++q) ax += lv[f + 64 * q] * sp[lo[f + 64 * q]];
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
                step_sum<T, false>(mv, any, redh);   // its barrier also publishes y
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
                    wg_sum<T, 5, 1u | (1u << 3)>(a, red);
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

// ---- one problem on one CU --------------------------------------------------------
//
// The same for a single problem: whole iterations up to the next check, as
// coop.hip's kernel makes them with a group of workgroups (the gradient
// updated from the previous subproblem's), whose rounds cost 5 us each: the
// random QP with n = 1000, instance 0, to 1e-6 (17,990 inner steps) takes 98 ms
// here, 5.5 us a step, and 0.50 s launch by launch; there a step took 10.9 us.
__global__ __launch_bounds__(REG_MAX) void k_single_solve(DevState S, CoopRun R)
{
    constexpr int T = REG_MAX;
    typedef Cu<T> L;
    __shared__ double sh[L::ALL];
    double* red = sh;
    double* redh = sh + L::AT_STEP;
    double* redu = redh + 16 * L::WAVES;
    double* sp = sh + L::AT_OPS;              // direction; x_bar
    double* sxt = sh + L::AT_OPS + L::OP;     // x_T
    double* sy = sh + L::AT_OPS + 2 * L::OP;  // y
    int* misc = reinterpret_cast<int*>(sh + L::AT_MISC);       // [0] instance, [16..31] widths
    unsigned short* place = reinterpret_cast<unsigned short*>(sh + L::AT_DEAL);
    unsigned short* var = place + T;
    double* lv = sh + L::AT_MAT;
    unsigned short* lo = reinterpret_cast<unsigned short*>(lv + L::PLACES);
    const int tid = threadIdx.x, n = S.n, m = S.m;
    const bool xon = tid < n, yon = tid < m;
    const bool live = uniform_int(tid & ~63) < n, any = uniform_int(tid & ~63) < (n > m ? n : m);
    deal_rows(n, S.Q.rowptr, reinterpret_cast<int*>(sh + L::AT_OPS), place, var);
    const int vi = xon ? (int)var[tid] : 0, ri = yon ? tid : 0;
    const int qa = xon ? S.Q.rowptr[vi] : 0, ql = xon ? S.Q.rowptr[vi + 1] - qa : 0;
    const int ta = xon ? S.AT.rowptr[vi] : 0, tl = xon ? S.AT.rowptr[vi + 1] - ta : 0;
    const int aa = yon ? S.A.rowptr[ri] : 0, al = yon ? S.A.rowptr[ri + 1] - aa : 0;
    const int qmost = wave_longest(ql), amost = wave_longest(al);
    const Share qs = share<T>(qmost > REG_Q ? qmost - REG_Q : 0, 0, L::PLACES, misc + 16);
    const Share as = share<T>(amost, qs.end, L::PLACES, misc + 16);
    fill(qs, qa, ql, REG_Q, S.Q.val, nullptr, S.Q.col, 0, place, n, lv, lo);
    fill(as, aa, al, 0, S.A.val, nullptr, S.A.col, 0, place, n, lv, lo);
    RowQ Q;
    Q.most = qmost;
    Q.base = qs.base;
    Q.wide = qs.wide;
    Q.lv = lv;
    Q.lo = lo;
    Q.load(qa, ql, S.Q.val, nullptr, S.Q.col, 0, place, n);
    for (int i = tid; i < 3 * L::OP; i += T) sh[L::AT_OPS + i] = 0.0;
    __syncthreads();

    const Ctrl* c0 = S.ctrl;
    const double tau = uniform(c0->tau), sigma = uniform(c0->sigma), omega = uniform(c0->omega), th = uniform(c0->theta);
    const double gamma_inner = uniform(c0->gamma_inner), eps_min = uniform(c0->eps_min), eps_fixed = uniform(c0->eps_fixed);
    const int halpern = uniform_int(c0->use_halpern), unb = uniform_int(c0->has_unbounded_x);
    const double it = uniform(c0->inv_tau);
    Inner cg;
    cg.it = it;
    cg.abar = uniform(c0->abar);
    cg.gamma2 = uniform(c0->mprgp_gamma) * uniform(c0->mprgp_gamma);
    cg.max_inner = c0->max_inner;
    double eps = uniform(c0->eps), g_it = uniform(c0->g_inv_tau), ndx2 = uniform(c0->ndx2), ndy2 = uniform(c0->ndy2);
    double R_start = uniform(c0->R_start), res = 0.0;
    double cert[5] = {uniform(c0->ytil_max), uniform(c0->ptil_sum), uniform(c0->ptil_abs), uniform(c0->d_max), uniform(c0->cd)};
    long long inner_total = 0;

    const double l = xon ? S.lv[vi] : -INFINITY, u = xon ? S.uv[vi] : INFINITY;
    double x = xon ? S.x[vi] : 0.0, y = yon ? S.y[ri] : 0.0, xt = xon ? S.xt[vi] : 0.0;
    double rhs = xon ? S.rhs[vi] : 0.0, g = xon ? S.g[vi] : 0.0, yt = 0.0;
    if (xon) sxt[tid] = xt;
    if (yon) sy[tid] = y;
    __syncthreads();

    for (int iter = 0; iter < R.iters; ++iter) {
        const long long k = R.k + iter, t = R.t + iter;
        const bool store = !R.sub && (((k + 1) % R.check_every == 0) || (k + 1 >= R.max_iter));
        const bool exact = R.exact && iter == 0;
        // right-hand side and the gradient at the warm start
        double st[4] = {0.0, 0.0, 0.0, 0.0};
        if (live) {
            double r = rhs;
            if (!R.sub) {
                double aty = 0.0;
#pragma unroll 4
                for (int q = 0; q < tl; ++q) aty += S.AT.val[ta + q] * sy[S.AT.col[ta + q]];
                if (xon) r = x * it - S.c[vi] - aty;
            }
            double qx = 0.0;
            if (exact) qx = Q.dot(sxt);
            if (xon) {
                g = exact ? qx + it * xt - r : g + (rhs - r) + xt * (it - g_it);
                rhs = r;
                const Split f = split(xt, g, l, u, cg.abar);
                st[0] = f.phi * f.phi + f.beta * f.beta;
                st[1] = f.beta * f.beta;
                st[2] = f.phit * f.phi;
            }
        }
        step_sum<T, false>(st, live, redu);
        if (exact && isinf(eps) && eps_fixed <= 0.0) eps = uniform(fmax(gamma_inner * sqrt(st[0]), eps_min));
        g_it = it;
        cg.eps = eps_fixed > 0.0 ? eps_fixed : eps;
        cg.steps = 0;
        inner_solve<T>(cg, Q, xon, live, l, u, rhs, xt, g, st, sp, sxt, redh, redu);
        inner_total += cg.steps;
        res = sqrt(st[0]);
        if (R.sub) break;
        // x_bar
        if (xon) {
            sxt[tid] = xt;
            sp[tid] = 2.0 * xt - x;
        }
        __syncthreads();
        // dual step and the Halpern averages of y and x
        const double tt = (double)t, w = (tt + 1.0) / (tt + 2.0), wa = 1.0 / (tt + 2.0);
        double dy = 0.0, dx = 0.0, lc = 0.0, uc = 0.0;
        if (amost > 0 || yon) {
            const int f = as.base + (tid & 63);
            double ax = 0.0;
#pragma unroll 4
            for (int q = 0; q < as.wide; ++q) ax += lv[f + 64 * q] * sp[lo[f + 64 * q]];
            for (int q = as.wide; q < al; ++q) ax += S.A.val[aa + q] * sp[place[S.A.col[aa + q]]];
            if (yon) {
                lc = S.lc[ri];
                uc = S.uc[ri];
                const double v = y / sigma + ax;
                yt = sigma * (v - clampd(v, lc, uc));
                dy = yt - y;
                y = halpern ? w * ((1.0 + th) * yt - th * y) + wa * S.ya[ri] : yt;
                sy[tid] = y;
            }
        }
        if (xon) {
            dx = xt - x;
            x = halpern ? w * ((1.0 + th) * xt - th * x) + wa * S.xa[vi] : xt;
        }
        double mv[4] = {dx * dx, dy * dy, 0.0, 0.0};
        step_sum<T, false>(mv, any, redh);   // its barrier also publishes y
        ndx2 = mv[0];
        ndy2 = mv[1];
        if (eps_fixed <= 0.0) eps = uniform(fmin(eps, fmax(gamma_inner * omega * sqrt(ndx2) / tau, eps_min)));
        if (t == 0) R_start = uniform(sqrt(omega * ndx2 + ndy2 / omega));
        if (store) {   // the certificate pieces
            double a[5] = {0, 0, 0, 0, 0};
            if (yon) {
                const double yy = projY(dy, lc, uc);
                S.ytil[ri] = yy;
                a[0] = fabs(yy);
                a[1] = supp(yy, lc, uc);
                a[2] = supp_abs(yy, lc, uc);
            }
            if (xon && unb) {
                const double di = projRec(dx, l, u);
                S.dx[vi] = di;
                a[3] = fabs(di);
                a[4] = S.c[vi] * di;
            }
            wg_sum<T, 5, 1u | (1u << 3)>(a, red);
#pragma unroll
            for (int j = 0; j < 5; ++j) cert[j] = a[j];
        }
    }
    if (xon) {
        S.xt[vi] = xt;
        S.g[vi] = g;
        S.rhs[vi] = rhs;
        S.x[vi] = x;
    }
    if (yon && !R.sub) {
        S.y[ri] = y;
        S.yt[ri] = yt;
    }
    if (tid == 0) {
        Ctrl* c = S.ctrl;
        c->eps = eps;
        c->g_inv_tau = g_it;
        c->inner_it = cg.steps;
        c->inner_total += inner_total;
        c->hp_active += cg.products;
        c->res = res;
        if (!R.sub) {
            c->k = R.k + R.iters;
            c->t = R.t + R.iters;
            c->ndx2 = ndx2;
            c->ndy2 = ndy2;
            c->R_start = R_start;
            c->ytil_max = cert[0];
            c->ptil_sum = cert[1];
            c->ptil_abs = cert[2];
            c->d_max = cert[3];
            c->cd = cert[4];
        }
        post_status(S.dstat, R.iters, 0);
    }
}

hipError_t launch_single_solve(const DevState& S, const CoopRun& R, hipStream_t s)
{
    k_single_solve<<<1, REG_MAX, 0, s>>>(S, R);
    return hipGetLastError();
}

hipError_t launch_general_solve(const BatchDev& B, const BatchParams& P, hipStream_t s)
{
    if (B.general_count < 1) return hipSuccess;
    k_general_solve<REG_MAX><<<one_cu_grid(B.general_count), REG_MAX, 0, s>>>(B, P);
    return hipGetLastError();
}

int one_cu_places() { return one_cu_grid(1 << 30); }

hipError_t launch_small_solve(const BatchDev& B, const BatchParams& P, hipStream_t s)
{
    if (B.small_count < 1) return hipSuccess;
    constexpr int T = ONE_CU_SMALL;
    k_general_solve<T><<<one_cu_grid(B.small_count, REG_MAX / T), T, 0, s>>>(B, P);
    return hipGetLastError();
}

}  // namespace pdhcg
