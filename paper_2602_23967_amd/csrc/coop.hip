// coop.hip -- the iteration of a single problem with a non-diagonal Q in one
// launch: a group of workgroups runs whole outer iterations (Sections 2.1 to
// 3.3: right-hand side, boxed CG inner solve, extrapolation, dual step,
// Halpern averages) up to the next check, exchanging what they need.
//
// For problems whose products take a few microseconds the multi-launch path
// (kernels.hip) is bound by its chain of launches: five per inner step, 21 us
// at n = 1000 and 37 us at n = 20,000 of which the arithmetic is a fraction.
// Here an inner step is two rounds of the group.  In a round each workgroup
// reduces its rows, posts its partial sums in a slot and reads everyone's:
// a round costs 1.5 us for 8 workgroups, 2.7 for 128 and 4.1 for 256
// (measured), and the sums are the same in every workgroup, so each takes
// the method's decisions itself.  A solve of the random QPs, launch by launch
// for 128 iterations, and here: n = 3000 37.2 and 13.2 ms, n = 20,011 50.1
// and 24.2 ms, n = 50,000 80.6 and 38.5 ms.  What is left is the rounds'
// latency: about 5 us each with their gathers.  (general.hip takes the
// problems that one CU holds.)
//
// Exchange.  Values that other workgroups read go through agent-scope relaxed
// atomic stores and loads (performed at memory, past the XCDs' L2s, which are
// not coherent with each other); a workgroup waits for its stores to finish
// before it posts the round's slot.  A slot word is 64 bits: half a double
// and the round's number, so one load both waits for a value and reads it.
// No cache is flushed or invalidated.
//
// Progress.  The rows are cut into slices that do not depend on W; workgroup i
// of W takes slices i, i + W, ..., at least one of each matrix, so that it
// posts in every round (coop_rounds.h: why it has to).  W is how many
// workgroups had started when the first of them closed the list (all of the
// grid, or those that came within REG_WAIT_TICKS): nobody waits for a
// workgroup that has not started, so kernels of other streams cannot block the
// group, and the result does not depend on W.
//
// FP64 only.  The FP64 sums differ from the launch-by-launch path's in their
// last bits, which moves a solve's result by 1e-15; in mixed precision such a
// bit can turn the FP32 rounding of an operand, and results moved by 1e-8.
#include <math.h>

#include "coop_rounds.h"
#include "device_math.h"
#include "pdhcg_internal.h"

namespace pdhcg {

typedef unsigned long long u64;

constexpr int SPIN_MAX = 1 << 23;              // polls before a wait gives up (seconds)
constexpr long long REG_WAIT_TICKS = 200000;   // 2 ms of the 100 MHz wall clock

__device__ __forceinline__ u64 agent_load(const u64* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void agent_store(u64* p, u64 v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double peer_load(const double* p)
{
    return __longlong_as_double((long long)agent_load(reinterpret_cast<const u64*>(p)));
}
__device__ __forceinline__ void peer_store(double* p, double v)
{
    agent_store(reinterpret_cast<u64*>(p), (u64)__double_as_longlong(v));
}
// the thread's own stores have reached memory
__device__ __forceinline__ void stores_done()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
}

// kinds of a round's four values, two bits each
constexpr int kinds4(int a, int b, int c, int d) { return a | (b << 2) | (c << 4) | (d << 6); }
__device__ __forceinline__ int kind_of(int kinds, int j) { return (kinds >> (2 * j)) & 3; }

template <int T>
struct Group {
    int me, W;
    unsigned tag;       // number of the next round
    int* bad;           // LDS: a wait gave up
    double* red;        // LDS: 4 doubles per wave

    // reduces v over the workgroup and posts it in the slot of slice s
    template <int KINDS>
    __device__ __forceinline__ void post(u64* slots, int s, double (&v)[4])
    {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v[j] = rcomb(kind_of(KINDS, j), v[j], __shfl_xor(v[j], off));
        }
        stores_done();
        if (lane == 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) red[4 * wave + j] = v[j];
        }
        __syncthreads();
        if (threadIdx.x < 8) {
            const int j = threadIdx.x >> 1;
            double r = red[j];
#pragma unroll
            for (int w = 1; w < T / 64; ++w) r = rcomb(kind_of(KINDS, j), r, red[4 * w + j]);
            const u64 b = (u64)__double_as_longlong(r);
            const u64 half = (threadIdx.x & 1) ? b >> 32 : b & 0xffffffffull;
            agent_store(&slots[coop_slot(0, 0, s) + threadIdx.x], ((u64)tag << 32) | half);
        }
        __syncthreads();
    }

    // the round's sums over the slots of ns slices, in every thread
    template <int KINDS>
    __device__ __forceinline__ void wait(const u64* slots, int ns, double (&out)[4])
    {
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, j = (threadIdx.x >> 1) & 3;
        double acc = rid(kind_of(KINDS, j));
        for (int i = threadIdx.x; i < ((8 * ns + 63) & ~63); i += T) {
            u64 w = 0;
            if (i < 8 * ns) {
                int spins = 0;
                do {
                    w = agent_load(&slots[i]);
                } while ((unsigned)(w >> 32) != tag && ++spins < SPIN_MAX);
                if ((unsigned)(w >> 32) != tag) *bad = 1;
            }
            const unsigned mine = (unsigned)w, other = (unsigned)__shfl_xor((int)mine, 1);
            const unsigned lo = (threadIdx.x & 1) ? other : mine, hi = (threadIdx.x & 1) ? mine : other;
            if (i < 8 * ns) acc = rcomb(kind_of(KINDS, j), acc, __longlong_as_double((long long)(((u64)hi << 32) | lo)));
        }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int off = 32; off >= 8; off >>= 1) acc = rcomb(kind_of(KINDS, j), acc, __shfl_xor(acc, off));
        if (lane < 8 && (lane & 1) == 0) red[4 * wave + j] = acc;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            double r = red[q];
#pragma unroll
            for (int w = 1; w < T / 64; ++w) r = rcomb(kind_of(KINDS, q), r, red[4 * w + q]);
            out[q] = uniform(r);
        }
        __syncthreads();
        ++tag;
    }
};

// sum of term(i), i in [a, b), in order, four terms in flight
template <class F>
__device__ __forceinline__ double row_sum(int a, int b, F term)
{
#pragma clang fp contract(off)
    double s = 0.0;
    int i = a;
    for (; i + 4 <= b; i += 4) {
        const double t0 = term(i), t1 = term(i + 1), t2 = term(i + 2), t3 = term(i + 3);
        s += t0; s += t1; s += t2; s += t3;
    }
    for (; i < b; ++i) s += term(i);
    return s;
}

template <int T>
__global__ __launch_bounds__(T) void k_coop(DevState S, CoopDev D, CoopRun R)
{
    constexpr int EPT = COOP_EPT;
    __shared__ double prod[EPT * T];
    __shared__ double red[4 * (T / 64)];
    __shared__ int sh_me, sh_W, bad;
    const int tid = threadIdx.x;

    // ---- who takes part ----------------------------------------------------------
    if (tid == 0) {
        bad = 0;
        const int grid = (int)gridDim.x;
        const int s = __hip_atomic_fetch_add(&D.reg[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int W = 0;
        if (s == 0) {
            const long long t0 = (long long)wall_clock64();
            while (__hip_atomic_load(&D.reg[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < grid &&
                   (long long)wall_clock64() - t0 < REG_WAIT_TICKS) {
            }
            W = __hip_atomic_fetch_add(&D.reg[0], 1 << 20, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            W = W < grid ? W : grid;
            __hip_atomic_store(&D.reg[1], W, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else if (s < grid) {
            int spins = 0;
            while ((W = __hip_atomic_load(&D.reg[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == 0 && ++spins < SPIN_MAX) {
            }
        }
        sh_me = s;
        sh_W = W;
    }
    __syncthreads();
    Group<T> G;
    G.me = uniform_int(sh_me);
    G.W = uniform_int(sh_W);
    G.tag = 1;
    G.bad = &bad;
    G.red = red;
    if (G.me >= G.W) return;   // started after the list was closed
    const int NS = D.ns, NSA = D.nsa;
    const bool one = NS <= G.W;          // one slice per workgroup: its entries stay in registers
    const int iters = G.W < D.full && R.iters > 8 ? 8 : R.iters;

    // ---- the method's scalars ------------------------------------------------------
    const Ctrl* c0 = S.ctrl;
    const double it = uniform(c0->inv_tau), tau = uniform(c0->tau), sigma = uniform(c0->sigma), omega = uniform(c0->omega);
    const double abar = uniform(c0->abar), th = uniform(c0->theta), gamma2 = uniform(c0->mprgp_gamma) * uniform(c0->mprgp_gamma);
    const double gamma_inner = uniform(c0->gamma_inner), eps_min = uniform(c0->eps_min), eps_fixed = uniform(c0->eps_fixed);
    const int halpern = uniform_int(c0->use_halpern), unb = uniform_int(c0->has_unbounded_x);
    const long long max_inner = c0->max_inner;
    double eps = uniform(c0->eps), g_it = uniform(c0->g_inv_tau);
    double ndx2 = uniform(c0->ndx2), ndy2 = uniform(c0->ndy2), R_start = uniform(c0->R_start), d_max = uniform(c0->d_max),
           cd = uniform(c0->cd), ytil_max = uniform(c0->ytil_max), ptil_sum = uniform(c0->ptil_sum), ptil_abs = uniform(c0->ptil_abs);
    double res = 0.0;
    long long inner_total = 0, active = 0, inner_it = 0;

    double* const e0 = D.ex;            // phi (or beta), or x_bar
    double* const e1 = D.ex + S.n;      // the last direction, or x_T

    int cj[EPT];
    double av[EPT];
    BlkDesc qb{0, 0, 0, 0, 0, 0, 0, 0};
    int row = 0, ra = 0, rb = 0, own = 0;
    // slice s: its block, the thread's row and the block's entries
    auto enter = [&](int s) __attribute__((always_inline)) {
        qb = D.qblk[s];
        const int cnt = qb.k1 - qb.k0;
        own = tid < qb.nrows;
        row = qb.row0 + (own ? tid : 0);
        ra = own ? S.Q.rowptr[row] - qb.k0 : 0;
        rb = own ? S.Q.rowptr[row + 1] - qb.k0 : 0;
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            const int q = tid + i * T;
            const bool in = q < cnt;
            cj[i] = in ? S.Q.col[qb.k0 + q] : -1;
            av[i] = in ? S.Q.val[qb.k0 + q] : 0.0;
        }
    };
    if (one) enter(G.me);   // (there are NS >= W slices)

    // row of Q times an operand: the block's products in LDS, the thread's row
    // summed in its order; xop(j): FP64 operand
    auto product = [&](auto xop) __attribute__((always_inline)) -> double {
#pragma clang fp contract(off)
        double x[EPT];
#pragma unroll
        for (int i = 0; i < EPT; ++i) x[i] = cj[i] >= 0 ? xop(cj[i]) : 0.0;
#pragma unroll
        for (int i = 0; i < EPT; ++i)
            if (cj[i] >= 0) prod[tid + i * T] = av[i] * x[i];
        __syncthreads();
        double s = 0.0;
        if (own) s = row_sum(ra, rb, [&](int i) { return prod[i]; });
        __syncthreads();
        return s;
    };
    auto slots = [&]() { return D.slots + coop_slot(G.tag, D.nslots, 0); };   // of the next round

    for (int iter = 0; iter < iters; ++iter) {
        const long long k = R.k + iter, t = R.t + iter;
        const bool store = !R.sub && (((k + 1) % R.check_every == 0) || (k + 1 >= R.max_iter));
        const bool exact = R.exact && iter == 0;
        double v[4];

        // ---- right-hand side and gradient at the warm start ------------------------
        for (int s = G.me; s < NS; s += G.W) {
            if (!one) enter(s);
            double a[4] = {0.0, 0.0, 0.0, 0.0};
            double qx = 0.0;
            if (exact) qx = product([&](int j) { return S.xt[j]; });
            if (own) {
                const int i = row;
                const double xti = S.xt[i], l = S.lv[i], u = S.uv[i];
                double r;
                if (R.sub) {
                    r = S.rhs[i];
                } else {
                    const int qa = S.AT.rowptr[i], qe = S.AT.rowptr[i + 1];
                    const double aty = iter == 0
                        ? row_sum(qa, qe, [&](int q) { return S.AT.val[q] * S.y[S.AT.col[q]]; })
                        : row_sum(qa, qe, [&](int q) { return S.AT.val[q] * peer_load(&D.ey[S.AT.col[q]]); });
                    r = S.x[i] * it - S.c[i] - aty;
                }
                const double g = exact ? qx + it * xti - r : S.g[i] + (S.rhs[i] - r) + xti * (it - g_it);
                S.rhs[i] = r;
                S.g[i] = g;
                const Split sp = split(xti, g, l, u, abar);
                a[0] = sp.phi * sp.phi + sp.beta * sp.beta;
                a[1] = sp.beta * sp.beta;
                a[2] = sp.phit * sp.phi;
                peer_store(&e0[i], sp.phi);
            }
            G.template post<kinds4(0, 0, 0, 0)>(slots(), s, a);
        }
        G.template wait<kinds4(0, 0, 0, 0)>(slots(), NS, v);
        if (exact && isinf(eps) && eps_fixed <= 0.0) eps = uniform(fmax(gamma_inner * sqrt(v[0]), eps_min));
        g_it = it;
        inner_it = 0;
        res = sqrt(v[0]);
        const double stop = eps_fixed > 0.0 ? eps_fixed : eps;
        int done = uniform_int(res <= stop || inner_it >= max_inner);
        int mode = uniform_int(v[1] <= gamma2 * v[2] ? DIR_PHI : DIR_BETA);
        double gam = 0.0;

        // ---- the inner solve (MPRGP) -------------------------------------------------
        while (!done) {
            if (mode == DIR_BETA) {   // a direction that the slots do not hold yet
                for (int s = G.me; s < NS; s += G.W) {
                    if (!one) enter(s);
                    double a[4] = {0.0, 0.0, 0.0, 0.0};
                    if (own) peer_store(&e0[row], split(S.xt[row], S.g[row], S.lv[row], S.uv[row], abar).beta);
                    G.template post<kinds4(0, 0, 0, 0)>(slots(), s, a);
                }
                G.template wait<kinds4(0, 0, 0, 0)>(slots(), NS, v);
            }
            // H p = Q p + p / tau with p'Hp, g'p and the feasible step
            const int conj = mode == DIR_CONJ;
            ++active;
            for (int s = G.me; s < NS; s += G.W) {
                if (!one) enter(s);
                double a[4] = {0.0, 0.0, 0.0, INFINITY};
                auto dir = [&](int j) {
                    const double f = peer_load(&e0[j]);
                    return conj ? __builtin_fma(-gam, peer_load(&e1[j]), f) : f;
                };
                double h = product(dir);
                if (own) {
                    const int i = row;
                    const double l = S.lv[i], u = S.uv[i], xi = S.xt[i], gi = S.g[i];
                    const Split sp = split(xi, gi, l, u, abar);
                    const double p = mode == DIR_BETA ? sp.beta : (conj ? __builtin_fma(-gam, S.p[i], sp.phi) : sp.phi);
                    h += it * p;
                    S.p[i] = p;
                    S.hp[i] = h;
                    a[0] = p * h;
                    a[1] = gi * p;
                    if (p > 0.0 && isfinite(l)) a[3] = (xi - l) / p;
                    else if (p < 0.0 && isfinite(u)) a[3] = (xi - u) / p;
                }
                G.template post<kinds4(0, 0, 0, 2)>(slots(), s, a);
            }
            G.template wait<kinds4(0, 0, 0, 2)>(slots(), NS, v);
            if (uniform_int(!(v[0] > 0.0))) break;   // no descent direction left
            const double pHp = v[0], af = v[3] < 0.0 ? 0.0 : v[3], acg = v[1] / v[0];
            int kind;
            double alpha;
            if (mode == DIR_BETA) { kind = STEP_PROP; alpha = acg < af ? acg : af; }
            else if (acg <= af) { kind = STEP_CG; alpha = acg; }
            else { kind = STEP_EXPAND; alpha = af; }
            kind = uniform_int(kind);
            alpha = uniform(alpha);
            // the step; an expansion asks for a fresh gradient
            for (int s = G.me; s < NS; s += G.W) {
                if (!one) enter(s);
                double a[4] = {0.0, 0.0, 0.0, 0.0};
                if (own) {
                    const int i = row;
                    const double l = S.lv[i], u = S.uv[i], p = S.p[i], hp = S.hp[i];
                    double xi = clampd(S.xt[i] - alpha * p, l, u);
                    const double gi = S.g[i] - alpha * hp;
                    S.g[i] = gi;
                    const Split sp = split(xi, gi, l, u, abar);
                    if (kind == STEP_EXPAND) {
                        xi = clampd(xi - abar * sp.phi, l, u);
                        peer_store(&e1[i], xi);
                    } else {
                        a[0] = sp.phi * sp.phi + sp.beta * sp.beta;
                        a[1] = sp.beta * sp.beta;
                        a[2] = sp.phit * sp.phi;
                        a[3] = sp.phi * hp;
                        peer_store(&e0[i], sp.phi);
                        peer_store(&e1[i], p);
                    }
                    S.xt[i] = xi;
                }
                G.template post<kinds4(0, 0, 0, 0)>(slots(), s, a);
            }
            G.template wait<kinds4(0, 0, 0, 0)>(slots(), NS, v);
            ++inner_it;
            ++inner_total;
            if (kind == STEP_EXPAND) {
                ++active;
                for (int s = G.me; s < NS; s += G.W) {
                    if (!one) enter(s);
                    double a[4] = {0.0, 0.0, 0.0, 0.0};
                    const double qx = product([&](int j) { return peer_load(&e1[j]); });
                    if (own) {
                        const int i = row;
                        const double xi = S.xt[i];
                        const double gi = qx + it * xi - S.rhs[i];
                        S.g[i] = gi;
                        const Split sp = split(xi, gi, S.lv[i], S.uv[i], abar);
                        a[0] = sp.phi * sp.phi + sp.beta * sp.beta;
                        a[1] = sp.beta * sp.beta;
                        a[2] = sp.phit * sp.phi;
                        peer_store(&e0[i], sp.phi);
                    }
                    G.template post<kinds4(0, 0, 0, 0)>(slots(), s, a);
                }
                G.template wait<kinds4(0, 0, 0, 0)>(slots(), NS, v);
            } else if (kind == STEP_CG) {
                gam = uniform(v[3] / pHp);
            }
            res = sqrt(v[0]);
            done = uniform_int(res <= stop || inner_it >= max_inner);
            mode = uniform_int(!(v[1] <= gamma2 * v[2]) ? DIR_BETA : (kind == STEP_CG ? DIR_CONJ : DIR_PHI));
            if (uniform_int(bad)) break;
        }
        if (R.sub || uniform_int(bad)) break;

        // ---- x_bar and the Halpern average of x ----------------------------------------
        const double tt = (double)t, w = (tt + 1.0) / (tt + 2.0), wa = 1.0 / (tt + 2.0);
        for (int s = G.me; s < NS; s += G.W) {
            if (!one) enter(s);
            double a[4] = {0.0, 0.0, 0.0, 0.0};
            if (own) {
                const int i = row;
                const double xti = S.xt[i], xi = S.x[i];
                const double xb = 2.0 * xti - xi;
                peer_store(&e0[i], xb);
                const double dx = xti - xi;
                a[0] = dx * dx;
                S.x[i] = halpern ? w * ((1.0 + th) * xti - th * xi) + wa * S.xa[i] : xti;
                if (store && unb) {
                    const double di = projRec(dx, S.lv[i], S.uv[i]);
                    S.dx[i] = di;
                    a[1] = fabs(di);
                    a[2] = S.c[i] * di;
                }
            }
            G.template post<kinds4(0, 1, 0, 0)>(slots(), s, a);
        }
        G.template wait<kinds4(0, 1, 0, 0)>(slots(), NS, v);
        ndx2 = v[0];
        if (store) {
            d_max = unb ? v[1] : 0.0;
            cd = unb ? v[2] : 0.0;
        }
        if (eps_fixed <= 0.0) eps = uniform(fmin(eps, fmax(gamma_inner * omega * sqrt(ndx2) / tau, eps_min)));

        // ---- dual step and the Halpern average of y --------------------------------------
        for (int s = G.me; s < NSA; s += G.W) {
            const BlkDesc ab = D.ablk[s];
            const int cnt = ab.k1 - ab.k0;
            double a[4] = {0.0, 0.0, 0.0, 0.0};
            {
#pragma clang fp contract(off)
                int aj[EPT];
                double pv[EPT], xv[EPT];
#pragma unroll
                for (int i = 0; i < EPT; ++i) {
                    const int q = tid + i * T;
                    aj[i] = q < cnt ? S.A.col[ab.k0 + q] : -1;
                    pv[i] = q < cnt ? S.A.val[ab.k0 + q] : 0.0;
                }
#pragma unroll
                for (int i = 0; i < EPT; ++i) xv[i] = aj[i] >= 0 ? peer_load(&e0[aj[i]]) : 0.0;
#pragma unroll
                for (int i = 0; i < EPT; ++i)
                    if (aj[i] >= 0) prod[tid + i * T] = pv[i] * xv[i];
            }
            __syncthreads();
            if (tid < ab.nrows) {
                const int i = ab.row0 + tid;
                const int qa = S.A.rowptr[i] - ab.k0, qe = S.A.rowptr[i + 1] - ab.k0;
                const double ax = row_sum(qa, qe, [&](int q) { return prod[q]; });
                const double yi = S.y[i], l = S.lc[i], u = S.uc[i];
                const double vv = yi / sigma + ax;
                const double yti = sigma * (vv - clampd(vv, l, u));
                const double yn = halpern ? w * ((1.0 + th) * yti - th * yi) + wa * S.ya[i] : yti;
                const double dy = yti - yi;
                a[0] = dy * dy;
                S.yt[i] = yti;
                S.y[i] = yn;
                peer_store(&D.ey[i], yn);
                if (store) {
                    const double yy = projY(dy, l, u);
                    S.ytil[i] = yy;
                    a[1] = fabs(yy);
                    a[2] = supp(yy, l, u);
                    a[3] = supp_abs(yy, l, u);
                }
            }
            G.template post<kinds4(0, 1, 0, 0)>(slots(), s, a);
        }
        G.template wait<kinds4(0, 1, 0, 0)>(slots(), NSA, v);
        ndy2 = v[0];
        if (store) {
            ytil_max = v[1];
            ptil_sum = v[2];
            ptil_abs = v[3];
        }
        if (t == 0) R_start = uniform(sqrt(omega * ndx2 + ndy2 / omega));
        if (uniform_int(bad)) break;
    }

    const int failed = uniform_int(bad);
    if (G.me == 0 && tid == 0) {
        Ctrl* c = S.ctrl;
        c->eps = eps;
        c->g_inv_tau = g_it;
        c->inner_it = inner_it;
        c->inner_total += inner_total;
        c->hp_active += active;
        c->res = res;
        if (!R.sub) {
            c->k = R.k + iters;
            c->t = R.t + iters;
            c->ndx2 = ndx2;
            c->ndy2 = ndy2;
            c->R_start = R_start;
            c->d_max = d_max;
            c->cd = cd;
            c->ytil_max = ytil_max;
            c->ptil_sum = ptil_sum;
            c->ptil_abs = ptil_abs;
        }
        // iterations done; 0 (or, for a subproblem, 2) after a wait that gave up
        post_status(S.dstat, failed ? 0 : iters, failed);
    }
}

__global__ __launch_bounds__(256) void k_coop_begin(CoopDev D, long long words)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < words) D.slots[i] = 0;
    if (i < 4) D.reg[i] = 0;
}

hipError_t launch_coop(const DevState& S, const CoopDev& D, const CoopRun& R, hipStream_t s)
{
    const long long words = 16ll * D.nslots;
    k_coop_begin<<<(int)((words + 255) / 256), 256, 0, s>>>(D, words);
    const int grid = D.cap > 0 && D.cap < D.full ? D.cap : D.full;
    if (D.threads == 256) k_coop<256><<<grid, 256, 0, s>>>(S, D, R);
    else k_coop<512><<<grid, 512, 0, s>>>(S, D, R);
    return hipGetLastError();
}

}  // namespace pdhcg
