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
// threads on a CU.  4096 MPC problems in mixed precision: 83 ms there, 23
// here; a handful from host arrays to results 28 ms and 6.  16 waves rather
// than 4: with one wave on a SIMD the same work took twice as long, bound by
// instruction fetch.  Instances far smaller than the workgroup are no slower
// for it (640 iterations of 4096 of them, general kernel and here: 16
// variables 19.1 and 18.8 ms, 64 19.6 and 19.5, 256 22.4 and 20.8, in mixed
// precision 18.9 and 18.5, 19.5 and 18.6, 22.8 and 19.8; of 64 of them, 3.7
// to 4.1 and 1.1 to 1.3).
//
// The iterates are the general kernel's of 256 threads to the bit: each
// product sums a row with one thread in row order, the norms and the weight's
// update take their sums in its order, the Halpern averages its fused form.
// (In mixed precision a last bit that differs turns FP32 roundings: other
// orders moved results by 1e-10, single entries by 3e-8.)  The check's other
// sums are grouped by the workgroup, so the residuals and objectives that it
// reports, and a certificate's entries, may differ in their last bits.
#include <math.h>

#include <type_traits>

#include "device_math.h"
#include "one_cu.h"
#include "pdhcg_internal.h"

namespace pdhcg {

// ---- LDS of a workgroup: the CU's 160 KB, in doubles -----------------------------

constexpr int LDS_ALL = 160 * 1024 / 8;
constexpr int LDS_RED = RED_SLOTS * (REG_MAX / 64);                                // wg_sum's buffer
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

// Loads the first CAP entries of the thread's row (a, len) into registers:
// values, and offsets in bytes into the operand.  A missing entry is 0 times
// the operand's entry `zero`, a zero, so a wave's rows need no masks.
template <class T, int CAP>
__device__ __forceinline__ void load_row(int a, int len, const T* val, const unsigned short* c16, const int* c32, int first,
                                         int zero, T (&v)[CAP], unsigned (&o)[CAP])
{
    if constexpr (sizeof(T) == 4) {
        // Without a branch per entry (a missing one reads entry 0 and drops
        // it): the branches' merges made one 64-byte vector of v, and every
        // iteration then reloaded 256 bytes of it from scratch (4096 MPC
        // problems: 54 ms, 23 without; 1024 instances of 256 variables 9.4 and
        // 5.0, where the general kernel takes 5.9).  (The FP64 form spills
        // less with the branches.)
        int j[CAP];
        if (c16) {
#pragma unroll
            for (int k = 0; k < CAP; ++k) j[k] = c16[k < len ? a + k : 0];
        } else {
#pragma unroll
            for (int k = 0; k < CAP; ++k) j[k] = c32[k < len ? a + k : 0] - first;
        }
#pragma unroll
        for (int k = 0; k < CAP; ++k) {
            const T e = val[k < len ? a + k : 0];
            v[k] = k < len ? e : T(0);
            o[k] = (unsigned)((k < len ? j[k] : zero) * (int)sizeof(T));
        }
    } else {
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
}

// the same for a wave's rows of A in LDS
template <class T>
__device__ __forceinline__ void load_mat(Share p, int a, int len, const T* val, const unsigned short* c16, const int* c32,
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
__device__ __forceinline__ T dot_mat(Share p, int most, const T* lv, const unsigned short* lo, int a, int len,
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
        const Share wm = share<REG_MAX>(amost, 0, mat_places<T>(), misc + 16);
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
                    one_cu_check<F32, false, REG_MAX>((unsigned long long)__builtin_amdgcn_kernarg_segment_ptr(), b, red, s));
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
                        x = halpern ? __builtin_fma(w, th1 * v - th * x, wa * xa) : v;
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
                        y = halpern ? __builtin_fma(w, th1 * yt - th * y, wa * ya) : yt;
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
                    wg_sum<REG_MAX, 7, (1u << 2) | (1u << 5)>(a, red);   // its barrier also publishes sy
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
// registers, A in LDS, two products and five barriers per iteration (the
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
        const Share wm = share<REG_MAX>(amost, 0, mat_places<double>(), misc + 16);
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
        __syncthreads();
        const double nv = sqrt(sumsq_256(v, n, sv, red));
        if (xon) sv[tid] = v / nv;
        __syncthreads();
        double sig = 0.0, prev = 0.0;
        for (long long i = 1; i <= max_iter; ++i) {
            double w = 0.0;
            if (amost > 0) w = dot_mat<double>(wm, amost, lav, lao, aa, al, B.aval, B.acol16, B.acol, v0, sv);
            sig = sqrt(sumsq_256(yon ? w : 0.0, m, sw, red));   // leaves w in sw
            if (uniform_int(sig == 0.0)) break;
            double u = 0.0;
            if (tmost > 0) u = dot_row<double, REG_T>(tv, to, tmost, ta, tl, B.tval, B.tcol16, B.tcol, r0, sw);
            const double nu = sqrt(sumsq_256(xon ? u : 0.0, n, sv, red));
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

hipError_t launch_closed_solve(const BatchDev& B, const BatchParams& P, hipStream_t s)
{
    if (B.closed_count < 1) return hipSuccess;
    const int grid = one_cu_grid(B.closed_count);
    if (B.aval32) k_closed_solve<true><<<grid, REG_MAX, 0, s>>>(B, P);
    else k_closed_solve<false><<<grid, REG_MAX, 0, s>>>(B, P);
    return hipGetLastError();
}

hipError_t launch_closed_norm(const BatchDev& B, double tol, long long max_iter, double* out, hipStream_t s)
{
    if (B.closed_count < 1) return hipSuccess;
    k_closed_norm<<<one_cu_grid(B.closed_count), REG_MAX, 0, s>>>(B, tol, max_iter, out);
    return hipGetLastError();
}

}  // namespace pdhcg
