// Symmetric (Hermitian) solve of a window by tridiagonalization, split over
// three kernels so that every phase runs where it is fast:
//
//   k_trid_reduce   one workgroup: Householder reduction T = Q^* xtx Q with the
//                   matrix in registers
//   k_trid_values   one wavefront per eigenvalue: multisection of T (windows of
//                   up to 8 columns: in the third kernel)
//   k_trid_vectors  one workgroup: the r leading eigenvectors (twisted
//                   factorizations, back-transformation), V_r, the A~ of
//                   Algorithm 2 and the POD coefficients
//
// The reduction is a chain of n dependent column steps; what bounds a step is
// the latency between its two barriers, not its arithmetic: (4/3) n^3 flops
// are 9 us of one CU's FP64 rate at n = 128, where the steps of a reduction
// with the matrix in LDS or in L2 cost 5 to 38 thousand cycles each.
//
// Measured on an MI355X, one window, reduction + values + vectors, against the
// solve by one 1024-thread workgroup that they replace (matrix in LDS to
// m = 64 real, else in the workspace): m = 32, r = 10: 20 + 10 + 14 us, was 119;
// m = 64, r = 20: 50 + 18 + 25, was 294; m = 120, r = 15: 117 + 32 + 50, was
// 781 (these with the finalize); m = 256, r = 32: 619 + 63 + 203, was 3951;
// Hermitian m = 128, r = 24: 262 + 34 + 95, was 1209.  Hermitian windows of
// more than 128 columns exceed the registers and keep the one-workgroup solve.
#include <type_traits>

#include "gram_finalize.h"
#include "solve_common.h"

namespace dmd {
namespace {

typedef double v4d __attribute__((ext_vector_type(4)));

// Rows of the reduction's thread grid for windows of m columns (its instances
// in reduce_class), also the stride of the stored reflectors.
__host__ __device__ constexpr int trid_rows(int m, int cplx) {
    return m <= 32 ? 32 : m <= 64 ? 64 : (m <= 96 && !cplx) ? 96 : m <= 128 ? 128 : m <= 192 ? 192 : 256;
}
__device__ __forceinline__ int trid_padded(int n) { return 1 + (n + 6) / 8 * 8; }

// What the three kernels hand on, in the solve's workspace (SolveArgs::work).
template <typename S> struct TridWork {
    double* hdr;   // [0] columns of X (0: nothing to solve), [1] the scale of T
    double2* de;   // pairs (d_k, e_{k-1}^2) of T / scale, padded to 8 j + 1 pairs (kTridPad more than m at most)
    double* e;     // m off-diagonal entries of T / scale (e_{n-1} = 0)
    double* lam;   // m eigenvalues of T / scale, ascending
    S* tau;        // m
    S* refl;       // m columns of ldr entries: column j = reflector u_j (zero to row j and past the matrix)
    int ldr;
    __device__ explicit TridWork(const SolveArgs& a) {
        ldr = trid_rows(a.m, a.cplx);
        hdr = a.work;
        de = reinterpret_cast<double2*>(a.work + 2);
        e = a.work + 2 + 2 * (a.m + kTridPad);
        lam = e + a.m;
        tau = reinterpret_cast<S*>(lam + a.m);
        refl = tau + a.m;
    }
};

// A pointer whose uniform reads become scalar loads: for data that an earlier
// kernel wrote and this one does not.
template <typename T> using scalar_ptr = const __attribute__((address_space(4))) T*;
template <typename T> __device__ __forceinline__ scalar_ptr<T> as_scalar(const T* p) {
    return (scalar_ptr<T>)(uintptr_t)p;
}

// Barrier for data exchanged through LDS: global stores (the reflectors, read
// by a later kernel only) stay in flight.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ double fma_s(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ cplx fma_s(cplx a, cplx b, cplx c) {
    return {fma(-a.im, b.im, fma(a.re, b.re, c.re)), fma(a.im, b.re, fma(a.re, b.im, c.im))};
}
// c - (v conj(w) + u conj(x)), the rank-2 update of one entry
__device__ __forceinline__ double upd_s(double c, double v, double w, double u, double x) {
    return fma(-u, x, fma(-v, w, c));
}
__device__ __forceinline__ cplx upd_s(cplx c, cplx v, cplx w, cplx u, cplx x) {
    return {fma(-u.im, x.im, fma(-u.re, x.re, fma(-v.im, w.im, fma(-v.re, w.re, c.re)))),
            fma(u.re, x.im, fma(-u.im, x.re, fma(v.re, w.im, fma(-v.im, w.re, c.im))))};
}
__device__ __forceinline__ double re_conj_mul(double a, double b) { return a * b; }
__device__ __forceinline__ double re_conj_mul(cplx a, cplx b) { return fma(a.im, b.im, a.re * b.re); }
__device__ __forceinline__ double norm2(double a) { return a * a; }
__device__ __forceinline__ double norm2(cplx a) { return fma(a.im, a.im, a.re * a.re); }

__device__ __forceinline__ double scale_pow2(double x, int e) { return __builtin_ldexp(x, e); }
__device__ __forceinline__ cplx scale_pow2(cplx x, int e) { return {__builtin_ldexp(x.re, e), __builtin_ldexp(x.im, e)}; }

template <int CTRL> __device__ __forceinline__ cplx dpp_s(cplx x) { return {dpp_f64<CTRL>(x.re), dpp_f64<CTRL>(x.im)}; }
template <int CTRL> __device__ __forceinline__ double dpp_s(double x) { return dpp_f64<CTRL>(x); }
__device__ __forceinline__ double sel(bool c, double a, double b) { return c ? a : b; }
__device__ __forceinline__ cplx sel(bool c, cplx a, cplx b) { return {c ? a.re : b.re, c ? a.im : b.im}; }

// Sums V values over the 16 lanes of a row.  The first two levels halve the
// number of values a lane carries (it keeps those its lane bit names and
// hands the others over); the last two are sums over rotations of the row.
// Lane l then holds the sums of the values a(l) below; store(a, sum) is
// called on one lane for each a.
template <int V, typename S, typename F> __device__ __forceinline__ void row_sums(const S (&s)[V], F store) {
    constexpr int V1 = V > 1 ? (V + 1) / 2 : 1, V2 = V1 > 1 ? (V1 + 1) / 2 : 1;
    const int l = threadIdx.x & 15;
    S t[V1], u[V2];
    if constexpr (V > 1) {
        const bool b = l & 1;
#pragma unroll
        for (int i = 0; i < V1; ++i) {
            const S lo = s[i], hi = i + V1 < V ? s[i + V1 < V ? i + V1 : 0] : Scal<S>::zero();
            t[i] = sel(b, hi, lo) + dpp_s<0xB1>(sel(b, lo, hi));
        }
    } else {
        t[0] = s[0] + dpp_s<0xB1>(s[0]);
    }
    if constexpr (V1 > 1) {
        const bool b = l & 2;
#pragma unroll
        for (int i = 0; i < V2; ++i) {
            const S lo = t[i], hi = i + V2 < V1 ? t[i + V2 < V1 ? i + V2 : 0] : Scal<S>::zero();
            u[i] = sel(b, hi, lo) + dpp_s<0x4E>(sel(b, lo, hi));
        }
    } else {
        u[0] = t[0] + dpp_s<0x4E>(t[0]);
    }
#pragma unroll
    for (int i = 0; i < V2; ++i) {
        u[i] = u[i] + dpp_s<0x124>(u[i]);  // row_ror:4
        u[i] = u[i] + dpp_s<0x128>(u[i]);  // row_ror:8
    }
    // lane l < 4 V2 stores value i = l / 4 of its V2
    const int a0 = (V > 1 ? (l & 1) * V1 : 0), a1 = (V1 > 1 ? ((l >> 1) & 1) * V2 : 0);
    const bool first = (V > 1 || !(l & 1)) && (V1 > 1 || !(l & 2));
    const int i = l >> 2;
    S x = u[0];
#pragma unroll
    for (int q = 1; q < V2; ++q) x = sel(i == q, u[q], x);
    const int a = a0 + a1 + i;
    if (first && i < V2 && a1 + i < V1 && a < V) store(a, x);
}

// --------------------------------------------------------------------------
// k_trid_reduce: entry (i, j) of the matrix belongs to the thread (ri, ci) of
// a PR x 16 grid with i = PR a + ri, j = 16 b + ci, as the thread's register
// A[a][b] (both triangles, cyclic in both directions, so that the trailing
// matrix of every step is spread over all threads); for n > 192 the first NL
// column blocks, which the reduction finishes first, sit in LDS slots private
// to their thread instead.  One step, column j with x = A[j+1.., j]:
//   u = x - beta e_1, H = I - tau u u^* (u is kept unnormalized: no division
//   and no scaling of its entries), for the thread's rows and columns;
//   y = A u: partial sums over the thread's columns, summed over the 16 lanes
//   of a row by DPP moves, to LDS;                              -- barrier
//   w = tau y - |tau|^2 (u^* y) / 2 u; the next column first, to LDS;
//                                                               -- barrier
//   the rest of A -= u w^* + w u^*.
// The norm and u^* y are sums over the 16 columns' lanes, by every wavefront
// for itself.
// What bounds a step is the issue of its instructions (4 cycles each on the
// SIMD of its wavefront), about half of them the products at n = 64, and the
// latencies between its two barriers: hence few wavefronts (a barrier costs
// 11 cycles with 4, 45 with 8, 132 with 16, and what is not a product is paid
// once per wavefront), and 16-lane rows, whose sums complete within one.
// The matrix is scaled by a power of two to a largest diagonal entry near 1,
// so that squares neither overflow nor matter when they underflow.
// --------------------------------------------------------------------------
template <typename S, int NT> struct ReduceShared {
    S x[2][kMaxM];          // the column being reduced below its diagonal (zero above), by step parity
    S y[2][kMaxM];          // A u, by step parity
    S z[kMaxM], tau[kMaxM];
    double d[kMaxM], e[kMaxM];
    double red[NT / 64];
};

template <int I, int N, typename F> __device__ __forceinline__ void each(F f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        each<I + 1, N>(f);
    }
}
__device__ __forceinline__ double row_sum(double x) {
    x += dpp_f64<0xB1>(x);
    x += dpp_f64<0x4E>(x);
    x += dpp_f64<0x141>(x);
    return x + dpp_f64<0x140>(x);
}
__device__ __forceinline__ cplx row_sum(cplx x) { return {row_sum(x.re), row_sum(x.im)}; }


template <typename S, int NT, int NA, int NB, int NL>
struct Reducer {
    using SC = Scal<S>;
    static constexpr int PR = NT / 16;
    S A[NA][NB - NL];
    S* priv;                 // this thread's LDS slots, NT apart
    ReduceShared<S, NT>& sh;
    S* refl;                 // the next column of reflectors
    int n, ldr, ci, ri;

    __device__ __forceinline__ Reducer(ReduceShared<S, NT>& s, S* p) : priv(p), sh(s) {
        ci = threadIdx.x & 15;
        ri = threadIdx.x >> 4;
    }
    template <int a, int b> __device__ __forceinline__ S get() const {
        if constexpr (b < NL) return priv[(a * NL + b) * NT];
        else return A[a][b - NL];
    }
    template <int a, int b> __device__ __forceinline__ void put(S v) {
        if constexpr (b < NL) priv[(a * NL + b) * NT] = v;
        else A[a][b - NL] = v;
    }
    // keeps the compiler from reading several column blocks' operands ahead,
    // where the matrix leaves no registers for them
    static __device__ __forceinline__ void fence_block() {
        if constexpr (NL > 0) __builtin_amdgcn_sched_barrier(0);
    }
    // column j below its diagonal (block b = j / 16, the thread's entries v),
    // to LDS for the next step and to the workspace as reflector j; entry
    // j + 1 of the reflector (z) follows at the end
    template <int A0, typename F> __device__ __forceinline__ void publish(int j, S* xn, F v) {
        if (ci == (j & 15))
            each<A0, NA>([&](auto a) {
                const int i = PR * a() + ri;
                const S m = sel(i > j, v(a), SC::zero());
                xn[i] = m;
                refl[i] = m;
                fence_block();
            });
        refl += ldr;
    }

    // step j in column block B0; B1 = the block of column j + 1
    template <int B0, int B1> __device__ __forceinline__ void step(int j) {
        constexpr int A0 = 16 * B0 / PR;
        constexpr bool kKeep = NL == 0;  // u and y of the thread's columns in registers, else read again
        const S* x = sh.x[j & 1];
        S* y = sh.y[j & 1];
        const int dj = j + 1;
        // the reflector of column j: beta = -sign(Re alpha) ||x||, z = alpha - beta,
        // tau = 2 / u^T u, from u itself so that the rounding of beta does not
        // cost orthogonality (complex: -1 / (beta conj(z)))
        const S alpha = x[dj];
        S uk[kKeep ? NB : 1], ur[NA];
        double s2 = 0.0;
        each<B0, NB>([&](auto b) {
            const S xi = x[16 * b() + ci];
            if constexpr (kKeep) uk[b()] = xi;
            s2 += norm2(xi);
        });
        each<A0, NA>([&](auto a) { ur[a()] = x[PR * a() + ri]; });
        s2 = row_sum(s2);
        const bool flat = !(s2 > 1e-200);  // (nothing, beside a largest diagonal entry near 1)
        const double inv = rsqrt_acc(s2), ar = SC::re(alpha);
        double nrm = s2 * inv;
        if constexpr (sizeof(S) == sizeof(cplx)) nrm = fma(0.5 * inv, fma(-nrm, nrm, s2), nrm);  // (tau is taken from it)
        nrm = flat ? 0.0 : nrm;
        const double beta = -copysign(nrm, ar);
        const S z = alpha - SC::fromc(mkc(beta));
        S tau;
        if constexpr (sizeof(S) == sizeof(cplx)) tau = copysign(rcp_acc(nrm * norm2(z)), ar) * z;
        else tau = 2.0 * rcp_acc(fma(z, z, fma(-ar, ar, s2)));
        tau = sel(flat, SC::zero(), tau);
        // (every thread writes the same values)
        sh.e[j] = beta;
        sh.z[j] = z;
        sh.tau[j] = tau;
        auto patch = [&](int i, S xi) { return sel(i == dj, z, xi); };
        if constexpr (kKeep) each<B0, NB>([&](auto b) { uk[b()] = patch(16 * b() + ci, uk[b()]); });
        auto ucol = [&](auto b) {
            if constexpr (kKeep) return uk[b()];
            else return patch(16 * b() + ci, x[16 * b() + ci]);
        };
        each<A0, NA>([&](auto a) { ur[a()] = patch(PR * a() + ri, ur[a()]); });
        // y = A u
        S s[NA - A0];
        each<A0, NA>([&](auto a) { s[a() - A0] = SC::zero(); });
        each<B0, NB>([&](auto b) {
            const S ub = ucol(b);
            each<A0, NA>([&](auto a) { s[a() - A0] = fma_s(get<a(), b()>(), ub, s[a() - A0]); });
            fence_block();
        });
        row_sums(s, [&](int a, S v) { y[PR * (A0 + a) + ri] = v; });
        lds_barrier();
        // w = tau y - |tau|^2 (u^* y) / 2 u
        S yk[kKeep ? NB : 1], wr[NA];
        double q = 0.0;
        each<B0, NB>([&](auto b) {
            const S yb = y[16 * b() + ci];
            if constexpr (kKeep) yk[b()] = yb;
            q += re_conj_mul(ucol(b), yb);
            fence_block();
        });
        each<A0, NA>([&](auto a) { wr[a()] = mulr(tau, y[PR * a() + ri]); });
        const double c = -0.5 * re_conj_mul(tau, tau * row_sum(q));  // (|tau|^2 alone may overflow)
        each<A0, NA>([&](auto a) { wr[a()] = wr[a()] + ur[a()] * c; });
        auto update = [&](auto b) {
            const S ub = ucol(b);
            S yb;
            if constexpr (kKeep) yb = yk[b()];
            else yb = y[16 * b() + ci];
            const S wb = mulr(tau, yb) + ub * c;
            each<A0, NA>([&](auto a) {
                put<a(), b()>(upd_s(get<a(), b()>(), ur[a()], wb, wr[a()], ub));
            });
            fence_block();
        };
        // the next column first; the rest needs no other thread's data (x and
        // y alternate between two buffers)
        update(std::integral_constant<int, B1>{});
        publish<A0>(dj, sh.x[(j & 1) ^ 1], [&](auto a) { return get<a(), B1>(); });
        lds_barrier();
        each<B0, NB>([&](auto b) {
            if constexpr (b() != B1) update(b);
        });
    }

    template <int B0> __device__ __forceinline__ void run() {
        if constexpr (B0 < NB) {
            const int end = 16 * B0 + 15 < n - 1 ? 16 * B0 + 15 : n - 1;
            for (int j = 16 * B0; j < end; ++j) step<B0, B0>(j);
            bool more = false;
            if constexpr (B0 + 1 < NB) {
                more = 16 * B0 + 15 < n - 1;
                if (more) step<B0, B0 + 1>(16 * B0 + 15);
            }
            // the block's diagonal of T (no later step changes it, and none
            // keeps the block's registers for it)
            each<16 * B0 / PR, NA>([&](auto a) {
                if (PR * a() + ri == 16 * B0 + ci) sh.d[16 * B0 + ci] = SC::re(get<a(), B0>());
            });
            if (more) run<B0 + 1>();
        }
    }
};

// Columns of X to solve for; 0 when there is nothing to do (the window is not
// full, or no snapshot came since the latest complete solve).
__device__ __forceinline__ int trid_begin(const SolveArgs& a) {
    DevState* st = a.st;
    const int n = window_cols(a.m, a.buildup, st);
    if (n == 0) {
        if (threadIdx.x == 0) {
            st->solve_status = ST_E_NOT_READY;
            st->r_eff = 0;
        }
        return 0;
    }
    if (st->vprev_valid && st->pushes == st->vprev_push) {
        if (threadIdx.x == 0) st->skipped = 1;
        return 0;
    }
    return n;
}

template <typename S, int NT, int NA, int NB, int NL>
__device__ __forceinline__ void reduce_body(const SolveArgs& a, ReduceShared<S, NT>& sh, S* dyn) {
    const int tid = threadIdx.x;
    const TridWork<S> w(a);
    const int n = trid_begin(a);
    if (tid == 0) w.hdr[0] = (double)n;
    if (n == 0) return;
    Reducer<S, NT, NA, NB, NL> R(sh, dyn + tid);
    R.refl = w.refl;
    R.n = n;
    R.ldr = w.ldr;
    constexpr int PR = NT / 16;
    const int oldest = a.st->oldest, slots = a.slots;
    each<0, NA>([&](auto ai) {
        each<0, NB>([&](auto bi) {
            const int i = PR * ai() + R.ri, j = 16 * bi() + R.ci;
            S v = Scal<S>::zero();
            if (i < n && j < n)  // (lanes along j: the conjugate of entry (j, i))
                v = Scal<S>::cj(gram_at<S>(a.G, slot_of(oldest, j, slots), slot_of(oldest, i, slots), slots));
            R.template put<ai(), bi()>(v);
            R.fence_block();
        });
    });
    // the power of two that brings the largest diagonal entry to [1/2, 1)
    double g = 0.0;
    for (int i = tid; i < n; i += NT) {
        const int si = slot_of(oldest, i, slots);
        g = fmax(g, fabs(Scal<S>::re(gram_at<S>(a.G, si, si, slots))));
    }
    auto block_max = [&](double v) {
        v = wave_max(v);
        if ((tid & 63) == 0) sh.red[tid >> 6] = v;
        lds_barrier();
        double r = sh.red[0];
        for (int k = 1; k < NT / 64; ++k) r = fmax(r, sh.red[k]);
        lds_barrier();
        return r;
    };
    g = block_max(g);
    const int ex = __builtin_amdgcn_frexp_exp(g);
    each<0, NA>([&](auto ai) {
        each<0, NB>([&](auto bi) { R.template put<ai(), bi()>(scale_pow2(R.template get<ai(), bi()>(), -ex)); });
    });
    R.template publish<0>(0, sh.x[0], [&](auto a) { return R.template get<a(), 0>(); });
    lds_barrier();
    R.template run<0>();
    if (tid == 0) sh.e[n - 1] = 0.0;
    // the reflectors' stores have landed before their entries j + 1 are replaced
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    // T / scale, scale = the largest Gershgorin radius; a Gram that is not finite
    // (a loaded window; pushes reject such snapshots) leaves a T that is not, and
    // is solved as zero: rank 0
    g = 0.0;
    for (int i = tid; i < n; i += NT) {
        const double rad = fabs(sh.d[i]) + (i > 0 ? fabs(sh.e[i - 1]) : 0.0) + fabs(sh.e[i]);
        g = rad <= DBL_MAX ? fmax(g, rad) : (double)INFINITY;
    }
    double scale = block_max(g);
    if (!(scale <= DBL_MAX)) {
        for (int i = tid; i < n; i += NT) sh.d[i] = sh.e[i] = 0.0;
        scale = 0.0;
        lds_barrier();
    }
    const double inv = scale > 0.0 ? 1.0 / scale : 0.0;
    for (int i = tid; i < n; i += NT) {
        const double e0 = i > 0 ? sh.e[i - 1] * inv : 0.0;
        // (a floor far below the resolution of the counts, 2^-100 in e, keeps
        // the minors of a decoupled T from vanishing)
        w.de[i] = double2{sh.d[i] * inv, fmax(e0 * e0, 0x1p-200)};
        w.e[i] = sh.e[i] * inv;
        if (i + 1 < n) {
            w.tau[i] = sh.tau[i];
            w.refl[(size_t)i * w.ldr + i + 1] = sh.z[i];
        }
    }
    // rows past the matrix, decoupled and above every bracket: no sign changes
    for (int i = n + tid; i < trid_padded(n); i += NT) w.de[i] = double2{2.0, 0.0};
    if (tid == 0) w.hdr[1] = __builtin_ldexp(scale, ex);
}

// --------------------------------------------------------------------------
// k_trid_values: eigenvalue k of T / scale by one wavefront.  64 equally
// spaced points of its bracket per round give 6 bits, so ten rounds of n
// steps replace the 34 (m = 128) of the two lanes per eigenvalue that one
// workgroup has: the Sturm counts are the solve's largest arithmetic, and
// the eigenvalues are independent, so they go to as many CUs as there are
// eigenvalues.  T comes through scalar loads (the same for all lanes).
// --------------------------------------------------------------------------
// Eigenvalues below x: sign changes of the leading principal minors
// p_k = (d_k - x) p_{k-1} - e_{k-1}^2 p_{k-2}, rescaled by powers of two every
// fourth step.  The signs are shifted into a word and the changes counted
// eight steps at a time; an exact zero counts as either sign (its
// neighbours have opposite signs, so one change is counted in any case).
struct SturmRow { double t[16]; };  // eight pairs of T
__device__ __forceinline__ SturmRow sturm_load(scalar_ptr<double> de, int k) {
    SturmRow r;
#pragma unroll
    for (int u = 0; u < 16; ++u) r.t[u] = de[2 * k + u];
    return r;
}
// `row` holds the pairs 1 .. 8 before and after the call
__device__ __forceinline__ int sturm_count64(scalar_ptr<double> de, int npad, double x, SturmRow& row) {
    double p0 = 1.0, p1 = de[0] - x;
    auto hi = [](double v) { return (unsigned)(__builtin_bit_cast(unsigned long long, v) >> 32); };
    unsigned sg = hi(p1) >> 31;
    int cnt = (int)sg;
    for (int k = 1; k < npad; k += 8) {
        // (the next eight pairs are on their way while these are used)
        const SturmRow nx = sturm_load(de, k + 8 < npad ? k + 8 : 1);
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const double p2 = fma(row.t[2 * u] - x, p1, -(row.t[2 * u + 1] * p0));
            p0 = p1;
            p1 = p2;
            sg = __builtin_amdgcn_alignbit(sg, hi(p2), 31);
            if (u % 4 == 3) {
                const int ex = -__builtin_amdgcn_frexp_exp(p1);
                p0 = __builtin_ldexp(p0, ex);
                p1 = __builtin_ldexp(p1, ex);
            }
        }
        cnt += __builtin_popcount((sg ^ (sg >> 1)) & 0xffu);
        row = nx;
    }
    return cnt;
}

// eigenvalue k of T / scale (n x n), the same in every lane
__device__ __forceinline__ double multisect(scalar_ptr<double> de, int n, int k) {
    const int lane = threadIdx.x & 63, npad = trid_padded(n);
    // (off centre, so that an eigenvalue of zero comes out as 1e-19 and not as an
    // exact zero)
    double lo = -1.0 - 8.0 * kEps, hi = 1.0 + 4.0 * kEps;
    SturmRow row = sturm_load(de, 1);
    constexpr double part = 1.0 / 65.0;
    // Ten rounds, 2 / 65^10 = 1.5e-18: the counts of a graded T resolve its small
    // eigenvalues far below eps ||T||, and the vectors of neighbours among them
    // are as orthogonal as their difference is exact (after nine rounds, 9.7e-17,
    // V^T V was off by 3e-14 at m = 32, r = 10 where ten leave 6e-15)
    for (int it = 0; it < 10; ++it) {
        const double wd = hi - lo;
        const double x = fma(wd, (double)(lane + 1) * part, lo);
        const uint64_t mask = __ballot(sturm_count64(de, npad, x, row) > k);
        const int f = mask ? __builtin_ctzll(mask) : 64;  // first point above the eigenvalue
        hi = f == 64 ? hi : fma(wd, (double)(f + 1) * part, lo);
        lo = f == 0 ? lo : fma(wd, (double)f * part, lo);
    }
    return 0.5 * (lo + hi);
}

// Windows of so few columns have a wavefront of k_trid_vectors find each
// eigenvalue: without the launch of k_trid_values a push and its modes take 50
// us for 52 at m = 2, r = 1.
constexpr int kInlineValues = 8;

template <typename S> __device__ __forceinline__ void values_body(const SolveArgs& a) {
    const TridWork<S> w(a);
    const int n = (int)as_scalar(w.hdr)[0];
    const auto de = as_scalar(reinterpret_cast<const double*>(w.de));
    const int k = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (k >= n || a.m <= kInlineValues) return;
    const double l = multisect(de, n, k);
    if ((threadIdx.x & 63) == 0) w.lam[k] = l;
}

// --------------------------------------------------------------------------
// k_trid_vectors
// --------------------------------------------------------------------------
constexpr int kVecThreads = 512;

// Dynamic LDS of the vectors kernel for m columns and nv vectors: the
// multipliers of the twisted factorizations (a row of 64 lanes per step, steps
// in groups of four and a spare row), then over them V_r and T (column stride
// m + 1, real and imaginary parts apart).
template <typename S> __host__ __device__ inline size_t vec_lds(int m, int nv) {
    const size_t cw = sizeof(S) / sizeof(double);
    const size_t lu = 64 * (size_t)(m + 4), vt = 2 * cw * (size_t)(m + 1) * nv;
    return sizeof(double) * (lu > vt ? lu : vt);
}

// argmax over the 16 lanes of a row (lowest index on ties)
__device__ __forceinline__ void row_argmax(double& v, int& i) {
    auto lvl = [&](auto ctrl) {
        constexpr int C = decltype(ctrl)::value;
        const double ov = dpp_f64<C>(v);
        const int oi = __builtin_amdgcn_mov_dpp(i, C, 0xF, 0xF, true);
        const bool take = ov > v || (ov == v && oi < i);
        v = take ? ov : v;
        i = take ? oi : i;
    };
    lvl(std::integral_constant<int, 0xB1>{});
    lvl(std::integral_constant<int, 0x4E>{});
    lvl(std::integral_constant<int, 0x124>{});
    lvl(std::integral_constant<int, 0x128>{});
}
// Z <- H_0 ... H_{n-2} Z for the 16-lane row's vector, entry 16 t + hl in
// z[t]: the vectors are independent, so a reflector costs a row its partial
// dot, four DPP sums and the update, and no barrier.  The entries of the next two
// or four reflectors are on their way meanwhile (a step is shorter than the
// L2's latency).
template <typename S, int NE>
__device__ __forceinline__ void back_transform(S (&z)[NE], const S* refl, const S* s_tau, int n) {
    using SC = Scal<S>;
    const int hl = threadIdx.x & 15;
    auto load = [&](int j, S (&v)[NE], S& tau, auto t0) {
        tau = s_tau[j];
        const S* p = refl + (size_t)(16 * NE) * j + hl;
        each<t0(), NE>([&](auto t) { v[t()] = p[16 * t()]; });
    };
    auto apply = [&](const S (&v)[NE], S tau, auto t0) {
        S p0 = SC::zero(), p1 = SC::zero();
        each<t0(), NE>([&](auto t) {
            if constexpr (t() % 2) p1 = fma_s(SC::cj(v[t()]), z[t()], p1);
            else p0 = fma_s(SC::cj(v[t()]), z[t()], p0);
        });
        const S f = mulr(tau, row_sum(p0 + p1)) * -1.0;
        each<t0(), NE>([&](auto t) { z[t()] = fma_s(v[t()], f, z[t()]); });
    };
    // blocks of 16 reflectors from the last on; reflector j is zero above row
    // j + 1, so block t0 leaves the entries before 16 t0 alone
    constexpr int D = NE * sizeof(S) <= 64 ? 4 : 2;
    auto block = [&](auto t0) {
        const int jlo = 16 * t0(), jhi = 16 * t0() + 15 < n - 2 ? 16 * t0() + 15 : n - 2;
        if (jhi < jlo) return;
        S u[D][NE], tau[D];
#pragma unroll
        for (int q = 0; q < D; ++q) load(jhi - q > jlo ? jhi - q : jlo, u[q], tau[q], t0);
        for (int j = jhi; j >= jlo; j -= D)
            each<0, D>([&](auto q) {
                if (j - q() >= jlo) {
                    apply(u[q()], tau[q()], t0);
                    load(j - q() - D > jlo ? j - q() - D : jlo, u[q()], tau[q()], t0);
                }
            });
    };
    each<0, NE>([&](auto t) { block(std::integral_constant<int, NE - 1 - t()>{}); });
}

__device__ __forceinline__ void coef_store(const SolveArgs& a, int i, int q, double v) {
    const int64_t o = (int64_t)i * a.r + q;
    if (a.coef_f64) reinterpret_cast<double*>(a.Bpod)[o] = v;
    else reinterpret_cast<float*>(a.Bpod)[o] = (float)v;
}
__device__ __forceinline__ void coef_store(const SolveArgs& a, int i, int q, cplx v) {
    const int64_t o = (int64_t)i * 2 * a.r + 2 * q;
    if (a.coef_f64) {
        reinterpret_cast<double*>(a.Bpod)[o] = v.re;
        reinterpret_cast<double*>(a.Bpod)[o + 1] = v.im;
    } else {
        reinterpret_cast<float*>(a.Bpod)[o] = (float)v.re;
        reinterpret_cast<float*>(a.Bpod)[o + 1] = (float)v.im;
    }
}

__device__ __forceinline__ v4d mfma64(double a, double b, v4d c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

template <typename S> struct VecShared {
    double lam[kMaxM];       // eigenvalues of T / scale
    double d[kMaxM], e[kMaxM];          // T / scale
    double2 fb[2][kMaxM + 8];           // (e, next d) of the factorizations' steps, forward and backward
    S tau[kMaxM];
    double sig[kMaxM];       // sigma, descending
    double lsel[kRMax];      // eigenvalue of vector v
    double nrm[2][kRMax];
    double mag[kRMax];
    int tw[kRMax];
    int near;                // two of the selected eigenvalues nearly coincide
};

template <typename S, int NE>
__device__ __forceinline__ void vectors_body(const SolveArgs& a, VecShared<S>& sh, double* dyn) {
    using SC = Scal<S>;
    constexpr bool CPLX = sizeof(S) == sizeof(cplx);
    constexpr int CW = CPLX ? 2 : 1;
    const TridWork<S> w(a);
    const int n = (int)as_scalar(w.hdr)[0];
    if (n == 0) return;
    const int tid = threadIdx.x, lane = tid & 63, hl = tid & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const double scale = as_scalar(w.hdr)[1];
    const int nv = a.r < n ? a.r : n;
    const bool inl = NE == 2 && a.m <= kInlineValues;  // (NE = 2: windows of up to 32 columns)
    if (inl && wave < n) {
        const double l = multisect(as_scalar(reinterpret_cast<const double*>(w.de)), n, wave);
        if (lane == 0) sh.lam[wave] = l;
    }
    for (int i = tid; i < n; i += kVecThreads) {
        if (!inl) sh.lam[i] = w.lam[i];
        sh.d[i] = w.de[i].x;
        sh.e[i] = w.e[i];
        if (i + 1 < n) sh.tau[i] = w.tau[i];
    }
    if (tid == 0) sh.near = 0;
    lds_barrier();
    const int nsteps = n - 1, npad = (n + 2) / 4 * 4;
    for (int i = tid; i < npad + 4; i += kVecThreads) {  // (past the last step: harmless values)
        const bool in = i < nsteps;
        sh.fb[0][i] = in ? double2{sh.e[i], sh.d[i + 1]} : double2{0.0, 2.0};
        sh.fb[1][i] = in ? double2{sh.e[n - 2 - i], sh.d[n - 2 - i]} : double2{0.0, 2.0};
    }
    // order by |lambda| descending (ties: larger index first); sigma =
    // sqrt(|lambda| scale).  Two lanes count the larger ones of an eigenvalue.
    for (int i2 = tid; i2 < 2 * n; i2 += kVecThreads) {
        const int i = i2 >> 1, h = i2 & 1;
        const double li = sh.lam[i], ai = fabs(li);
        int rank = 0;
#pragma unroll 4
        for (int k = h; k < n; k += 2) {
            const double ak = fabs(sh.lam[k]);
            rank += (ak > ai) || (ak == ai && k > i);
        }
        rank += __builtin_amdgcn_mov_dpp(rank, 0xB1, 0xF, 0xF, true);
        if (h == 0) {
            const double s = sqrt(ai * scale);
            sh.sig[rank] = s;
            a.sigma[rank] = s;
            if (rank < nv) sh.lsel[rank] = li;
        }
    }
    for (int i = n + tid; i < a.m; i += kVecThreads) a.sigma[i] = 0.0;
    lds_barrier();
    // rank: the leading sigma above rcond sigma_1 (none if sigma_1 = 0)
    int ke;
    {
        const double s0 = sh.sig[0];
        const bool low = lane < nv && !(s0 > 0.0 && sh.sig[lane < nv ? lane : 0] > a.rcond * s0);
        const uint64_t mask = __ballot(low);
        ke = mask ? __builtin_ctzll(mask) : nv;
    }
    // ---- eigenvectors of T by twisted factorizations of T - lambda_v I, the
    // forward L D L^T in lane v and the backward U D U^T in lane 32 + v of one
    // wavefront, step i of both in row i of M: L_i, and U_{n-1-i}
    double* M = dyn;
    const double tiny = 0x1p-900;
    const int vl = lane & 31, back = lane >> 5;
    if (wave == 0) {
        const double lam = sh.lsel[vl < ke ? vl : 0];
        const double2* T = sh.fb[back];
        double D = sh.d[back ? n - 1 : 0] - lam;
        double2 t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) t[u] = T[u];
        double* out = M + lane;
        for (int i = 0; i < npad; i += 4) {
            double2 nx[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) nx[u] = T[i + 4 + u];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                D = D == 0.0 ? tiny : D;
                const double l = t[u].x * rcp_fast(D);
                out[64 * u] = l;
                D = fma(-l, t[u].x, t[u].y - lam);
                t[u] = nx[u];
            }
            out += 256;
        }
    }
    lds_barrier();
    const int v = tid >> 4;  // a 16-lane row per vector
    const bool live = v < ke;
    if (live) {
        const double lam = sh.lsel[v];
        double best = -1e308;
        int tw = 0;
        for (int k = hl; k < n; k += 16) {
            double g = sh.d[k] - lam;
            if (k > 0) g -= M[64 * (k - 1) + v] * sh.e[k - 1];
            if (k + 1 < n) g -= M[64 * (n - 2 - k) + 32 + v] * sh.e[k];
            if (-fabs(g) > best) {
                best = -fabs(g);
                tw = k;
            }
        }
        row_argmax(best, tw);
        if (hl == 0) sh.tw[v] = tw;
    }
    // near coincidences, for the re-orthogonalization below
    for (int p = tid; p < ke * ke; p += kVecThreads)
        if (p % ke < p / ke && fabs(sh.lsel[p % ke] - sh.lsel[p / ke]) <= 1e-8) sh.near = 1;
    lds_barrier();
    // z_tw = 1, z_i = -L_i z_{i+1} (i < tw), z_{i+1} = -U_{i+1} z_i (i >= tw),
    // over the multipliers; lanes that are done write a spare row
    if (wave == 0) {
        const int tw = vl < ke ? sh.tw[vl] : 0;
        const int start = back ? n - 2 - tw : tw - 1;
        const int spare = npad;
        auto row = [&](int s) { return M + 64 * (s <= start ? start - s : spare) + lane; };
        int most = start;
        for (int off = 32; off >= 1; off >>= 1) {
            const int o = __shfl_xor(most, off, 64);
            most = o > most ? o : most;
        }
        double z = 1.0, nn = 0.0, l[4];
        M[64 * spare + lane] = 0.0;
#pragma unroll
        for (int u = 0; u < 4; ++u) l[u] = *row(u);
        for (int s = 0; s <= most; s += 4) {
            double nl[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) nl[u] = *row(s + 4 + u);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                z = s + u <= start ? -l[u] * z : 0.0;
                nn = fma(z, z, nn);
                *row(s + u) = z;
                l[u] = nl[u];
            }
        }
        sh.nrm[back][vl] = nn;
    }
    lds_barrier();
    // ---- from here on a 16-lane row per vector, entry 16 t + hl in z[t]
    S z[NE];
    {
        const int tw = live ? sh.tw[v] : 0;
        const double sc = live ? rsqrt_acc(1.0 + sh.nrm[0][v] + sh.nrm[1][v]) : 0.0;
#pragma unroll
        for (int t = 0; t < NE; ++t) {
            const int i = 16 * t + hl;
            double x = 0.0;
            if (live && i < n) x = sc * (i < tw ? M[64 * i + v] : i > tw ? M[64 * (n - 1 - i) + 32 + v] : 1.0);
            z[t] = SC::fromc(mkc(x));
        }
    }
    lds_barrier();
    if (sh.near) {
        // nearly coincident eigenvalues: Gram-Schmidt in selection order (one wavefront)
        double* Zs = dyn;  // Zs[i + v n]
#pragma unroll
        for (int t = 0; t < NE; ++t)
            if (live && 16 * t + hl < n) Zs[16 * t + hl + v * n] = SC::re(z[t]);
        lds_barrier();
        if (wave == 0) {
            for (int q = 1; q < ke; ++q) {
                for (int p = 0; p < q; ++p) {
                    if (fabs(sh.lsel[q] - sh.lsel[p]) > 1e-8) continue;
                    double* zq = Zs + q * n;
                    const double* zp = Zs + p * n;
                    double dot = 0.0;
                    for (int i = lane; i < n; i += 64) dot += zp[i] * zq[i];
                    dot = wave_sum(dot);
                    double nn = 0.0;
                    for (int i = lane; i < n; i += 64) {
                        const double zi = zq[i] - dot * zp[i];
                        zq[i] = zi;
                        nn += zi * zi;
                    }
                    nn = wave_sum(nn);
                    const double sc = nn > 0.0 ? rsqrt_acc(nn) : 0.0;
                    for (int i = lane; i < n; i += 64) zq[i] *= sc;
                }
            }
        }
        lds_barrier();
#pragma unroll
        for (int t = 0; t < NE; ++t)
            if (live && 16 * t + hl < n) z[t] = SC::fromc(mkc(Zs[16 * t + hl + v * n]));
        lds_barrier();
    }
    if (4 * wave < ke) back_transform<S, NE>(z, w.refl, sh.tau, n);  // (whole wavefronts without a vector skip)
    // canonical V_r: the entry of largest modulus (lowest index on ties) real positive
    const int ld = n + 1;
    double* Vs = dyn;                             // Vs[c (ld nv) + q ld + i], c = 0 real, 1 imaginary
    double* Ts = dyn + (size_t)CW * ld * nv;
    const int cs = ld * nv;
    {
        double best = -1.0;
        int bi = 0;
#pragma unroll
        for (int t = 0; t < NE; ++t) {
            const int i = 16 * t + hl;
            const double m2 = i < n ? SC::absv(z[t]) : -1.0;
            if (m2 > best) {
                best = m2;
                bi = i;
            }
        }
        row_argmax(best, bi);
        S piv = SC::zero();
#pragma unroll
        for (int t = 0; t < NE; ++t) piv = sel(16 * t + hl == bi, z[t], piv);
        piv = row_sum(piv);  // (one lane holds it)
        const S ph = SC::cj(SC::phase(piv));
        if (live) {
#pragma unroll
            for (int t = 0; t < NE; ++t) {
                const int i = 16 * t + hl;
                if (i < n) {
                    const S x = mulr(z[t], ph);
                    const cplx c = SC::toc(x);
                    Vs[v * ld + i] = c.re;
                    if (CPLX) Vs[cs + v * ld + i] = c.im;
                    store_s<S>(a.V, i + (int64_t)v * a.m, x);
                } else if (i < a.m) {
                    store_s<S>(a.V, i + (int64_t)v * a.m, SC::zero());
                }
            }
        }
    }
    lds_barrier();
    // POD coefficients V_r Sigma^-1 (row-major: lanes along a row)
    {
        const int q = tid & 31;
        if (q < ke) {
            const double is = 1.0 / sh.sig[q];
            for (int i = tid >> 5; i < n; i += kVecThreads / 32) {
                S x = SC::fromc(cplx{Vs[q * ld + i] * is, CPLX ? Vs[cs + q * ld + i] * is : 0.0});
                coef_store(a, i, q, x);
            }
        }
    }
    // ---- T = xty V_r, xty[i][j] = <x_i, x_{j+1}>, on the matrix cores
    // (16 x 16 x 4, A from the Gram: 16 consecutive slots of a column)
    const int li = lane & 15, lk = lane >> 4;
    const int slots = a.slots, oldest = a.st->oldest;
    for (int ti = wave; 16 * ti < n; ti += kVecThreads / 64) {
        v4d acc[2][CW];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int c = 0; c < CW; ++c) acc[q][c] = v4d{0, 0, 0, 0};
        const int i = 16 * ti + li;
        const double* gp = a.G + (size_t)CW * slot_of(oldest, i < n ? i : 0, slots);
        constexpr int U = CPLX ? 4 : 8;
        for (int k0 = 0; k0 < n; k0 += 4 * U) {
            double gr[U], gim[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + 4 * u + lk;
                const bool in = i < n && k < n;
                const double* g = gp + (size_t)CW * slots * slot_of(oldest, k < n ? k + 1 : 1, slots);
                gr[u] = in ? g[0] : 0.0;
                gim[u] = CPLX && in ? g[CW - 1] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + 4 * u + lk;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int c = 16 * q + li;
                    const bool in = k < n && c < ke;
                    const double vr = in ? Vs[c * ld + k] : 0.0;
                    acc[q][0] = mfma64(gr[u], vr, acc[q][0]);
                    if constexpr (CPLX) {
                        const double vi = in ? Vs[cs + c * ld + k] : 0.0;
                        acc[q][0] = mfma64(-gim[u], vi, acc[q][0]);
                        acc[q][1] = mfma64(gr[u], vi, acc[q][1]);
                        acc[q][1] = mfma64(gim[u], vr, acc[q][1]);
                    }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int c = 0; c < CW; ++c)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int row = 16 * ti + lk + 4 * u, col = 16 * q + li;
                    if (row < n && col < ke) Ts[c * cs + col * ld + row] = acc[q][c][u];
                }
    }
    lds_barrier();
    // ---- A~[p][q] = (V_r^* T)[p][q] / (sigma_p sigma_q)
    if (wave < 4 && 16 * (wave & 1) < ke && 16 * (wave >> 1) < ke) {
        const int p0 = 16 * (wave & 1), q0 = 16 * (wave >> 1);
        v4d re = v4d{0, 0, 0, 0}, im = v4d{0, 0, 0, 0};
        const int p = p0 + li, q = q0 + li;
        const double* vp = Vs + (p < ke ? p : 0) * ld;
        const double* tq = Ts + (q < ke ? q : 0) * ld;
#pragma unroll 4
        for (int k0 = 0; k0 < n; k0 += 4) {
            const int k = k0 + lk;
            const bool in = k < n;
            const double vr = in && p < ke ? vp[k] : 0.0, tr = in && q < ke ? tq[k] : 0.0;
            re = mfma64(vr, tr, re);
            if constexpr (CPLX) {
                const double vi = in && p < ke ? vp[cs + k] : 0.0, ti = in && q < ke ? tq[cs + k] : 0.0;
                re = mfma64(vi, ti, re);
                im = mfma64(vr, ti, im);
                im = mfma64(-vi, tr, im);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int pp = p0 + lk + 4 * u;
            if (pp < ke && q < ke) {
                const double f = 1.0 / (sh.sig[pp] * sh.sig[q]);
                store_s<S>(a.At, pp + (int64_t)q * ke, SC::fromc(mkc(re[u] * f, im[u] * f)));
            }
        }
    }
    if (tid == 0) {
        DevState* st = a.st;
        st->skipped = 0;
        st->r_eff = ke;
        st->sweeps = 0;
        st->solve_status = ke < nv || ke == 0 ? ST_W_RANK : ST_OK;
        st->vprev_valid = nv >= n && n == a.m ? 1 : 0;
        st->vprev_push = st->pushes;
        st->warm = 0;
    }
}

// ------------------------------------------------------------------ kernels
// Size classes, by the stream's window length (a build-up start's partial
// windows use their stream's class).
enum { kClassS = 0, kClassL = 1, kClassX = 2 };

template <typename S, int CLS> struct Cls;
template <> struct Cls<double, kClassS> { static constexpr int NT = 256; };
template <> struct Cls<double, kClassL> { static constexpr int NT = 256; };
template <> struct Cls<double, kClassX> { static constexpr int NT = 512; };
template <> struct Cls<cplx, kClassS> { static constexpr int NT = 256; };
template <> struct Cls<cplx, kClassL> { static constexpr int NT = 512; };

template <typename S, int CLS>
__device__ __forceinline__ void reduce_class(const SolveArgs& a, ReduceShared<S, Cls<S, CLS>::NT>& sh, double* dyn) {
    S* d = reinterpret_cast<S*>(dyn);
    if constexpr (sizeof(S) == sizeof(cplx)) {
        if constexpr (CLS == kClassS) {
            reduce_body<S, 256, 2, 2, 0>(a, sh, d);
        } else {
            if (a.m <= 64) reduce_body<S, 512, 2, 4, 0>(a, sh, d);
            else reduce_body<S, 512, 4, 8, 0>(a, sh, d);
        }
    } else if constexpr (CLS == kClassS) {
        if (a.m <= 32) reduce_body<S, 256, 2, 2, 0>(a, sh, d);
        else reduce_body<S, 256, 4, 4, 0>(a, sh, d);
    } else if constexpr (CLS == kClassL) {
        if (a.m <= 96) reduce_body<S, 256, 6, 6, 0>(a, sh, d);
        else reduce_body<S, 256, 8, 8, 0>(a, sh, d);
    } else {
        if (a.m <= 192) reduce_body<S, 512, 6, 12, 0>(a, sh, d);
        else reduce_body<S, 512, 8, 16, 4>(a, sh, d);
    }
}

template <typename S, int CLS>
__global__ __launch_bounds__((Cls<S, CLS>::NT))
void k_trid_reduce(SolveArgs a) {
    extern __shared__ double dyn[];
    __shared__ ReduceShared<S, Cls<S, CLS>::NT> sh;
    reduce_class<S, CLS>(a, sh, dyn);
}
// (The item is read through a scalar pointer: read as plain memory, its fields
// sit in vector registers across the whole reduction, and the m > 128 form
// spilled 1826 of its matrix, now 11 as in the kernel of one window.)
template <typename S, int CLS>
__global__ __launch_bounds__((Cls<S, CLS>::NT))
void k_trid_reduce_grouped(const SolveArgs* __restrict__ items) {
    extern __shared__ double dyn[];
    __shared__ ReduceShared<S, Cls<S, CLS>::NT> sh;
    const SolveArgs a = *(const SolveArgs*)as_scalar(items + blockIdx.x);
    reduce_class<S, CLS>(a, sh, dyn);
}
// A dense push's Gram finalize followed by the reduction of the window it
// completes, in one launch: one kernel boundary fewer on the single-push
// step.  A rejected snapshot leaves the state as it was, and the solve then
// repeats the previous one or finds nothing new (skipped).
template <int CLS>
__global__ __launch_bounds__((Cls<double, CLS>::NT))
void k_finalize_reduce(double* G, const double* partials, int nblk, SolveArgs a) {
    extern __shared__ double dyn[];
    __shared__ ReduceShared<double, Cls<double, CLS>::NT> sh;
    gram_finalize_body<Cls<double, CLS>::NT>(G, partials, nblk, a.m, a.slots, a.st);
    __syncthreads();
    reduce_class<double, CLS>(a, sh, dyn);
}

template <typename S>
__global__ __launch_bounds__(256)
void k_trid_values(SolveArgs a) {
    values_body<S>(a);
}
template <typename S>
__global__ __launch_bounds__(256)
void k_trid_values_grouped(const SolveArgs* __restrict__ items) {
    values_body<S>(items[blockIdx.y]);
}

template <typename S, int CLS>
__device__ __forceinline__ void vectors_class(const SolveArgs& a, VecShared<S>& sh, double* dyn) {
    constexpr bool CPLX = sizeof(S) == sizeof(cplx);
    const int rows = trid_rows(a.m, CPLX);
    if constexpr (CLS == kClassS) {
        if (CPLX || rows == 32) vectors_body<S, 2>(a, sh, dyn);
        else if constexpr (!CPLX) vectors_body<S, 4>(a, sh, dyn);
    } else if constexpr (CLS == kClassL) {
        if (rows == 128) vectors_body<S, 8>(a, sh, dyn);
        else vectors_body<S, CPLX ? 4 : 6>(a, sh, dyn);
    } else {
        if (rows == 192) vectors_body<S, 12>(a, sh, dyn);
        else vectors_body<S, 16>(a, sh, dyn);
    }
}
template <typename S, int CLS>
__global__ __launch_bounds__(kVecThreads)
void k_trid_vectors(SolveArgs a) {
    extern __shared__ double dyn[];
    __shared__ VecShared<S> sh;
    vectors_class<S, CLS>(a, sh, dyn);
}
template <typename S, int CLS>
__global__ __launch_bounds__(kVecThreads)
void k_trid_vectors_grouped(const SolveArgs* __restrict__ items) {
    extern __shared__ double dyn[];
    __shared__ VecShared<S> sh;
    const SolveArgs a = items[blockIdx.x];
    vectors_class<S, CLS>(a, sh, dyn);
}

template <typename K> hipError_t set_lds(K kern, size_t lds) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}
// dynamic LDS of the reduction: the private slots of the first four column
// blocks of windows beyond 192 columns
inline size_t reduce_lds(int m) { return m > 192 ? sizeof(double) * 8 * 4 * 512 : 0; }

// values and vectors of one window
template <typename S, int CLS> hipError_t launch_rest(const SolveArgs& a, hipStream_t s) {
    hipError_t e = hipSuccess;
    if (a.m > kInlineValues) {
        hipLaunchKernelGGL(k_trid_values<S>, dim3((a.m + 3) / 4), dim3(256), 0, s, a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const size_t lds = vec_lds<S>(a.m, a.r < a.m ? a.r : a.m);
    if ((e = set_lds(k_trid_vectors<S, CLS>, lds)) != hipSuccess) return e;
    hipLaunchKernelGGL((k_trid_vectors<S, CLS>), dim3(1), dim3(kVecThreads), lds, s, a);
    return hipGetLastError();
}
template <typename S, int CLS> hipError_t launch_one(const SolveArgs& a, hipStream_t s) {
    const size_t lds = reduce_lds(a.m);
    hipError_t e = set_lds(k_trid_reduce<S, CLS>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_trid_reduce<S, CLS>), dim3(1), dim3(Cls<S, CLS>::NT), lds, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return launch_rest<S, CLS>(a, s);
}
template <int CLS> hipError_t launch_fused(double* G, const double* partials, int nblk, const SolveArgs& a, hipStream_t s) {
    const size_t lds = reduce_lds(a.m);
    hipError_t e = set_lds(k_finalize_reduce<CLS>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_finalize_reduce<CLS>, dim3(1), dim3(Cls<double, CLS>::NT), lds, s, G, partials, nblk, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return launch_rest<double, CLS>(a, s);
}
template <typename S, int CLS> hipError_t launch_group(const SolveArgs* items, int n, int mmax, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const size_t lds = CLS == kClassX ? reduce_lds(mmax) : 0, vlds = vec_lds<S>(mmax, kRMax < mmax ? kRMax : mmax);
    hipError_t e = set_lds(k_trid_reduce_grouped<S, CLS>, lds);
    if (e == hipSuccess) e = set_lds(k_trid_vectors_grouped<S, CLS>, vlds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_trid_reduce_grouped<S, CLS>), dim3(n), dim3(Cls<S, CLS>::NT), lds, s, items);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (mmax > kInlineValues) {
        hipLaunchKernelGGL(k_trid_values_grouped<S>, dim3((mmax + 3) / 4, n), dim3(256), 0, s, items);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_trid_vectors_grouped<S, CLS>), dim3(n), dim3(kVecThreads), vlds, s, items);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_solve_trid(const SolveArgs& a, hipStream_t s) {
    if (a.r > kRMax || a.m > kMaxM) return hipErrorInvalidValue;
    if (a.cplx) {
        if (a.m <= 32) return launch_one<cplx, kClassS>(a, s);
        if (a.m <= 128) return launch_one<cplx, kClassL>(a, s);
        return launch_solve_trid_wide(&a, nullptr, 1, s);
    }
    if (a.m <= 64) return launch_one<double, kClassS>(a, s);
    if (a.m <= 128) return launch_one<double, kClassL>(a, s);
    return launch_one<double, kClassX>(a, s);
}

hipError_t launch_finalize_solve_trid(double* G, const double* partials, int nblk, const SolveArgs& a,
                                      hipStream_t s) {
    if (a.r > kRMax || a.m > kMaxM || a.cplx) return hipErrorInvalidValue;
    if (a.m <= 64) return launch_fused<kClassS>(G, partials, nblk, a, s);
    if (a.m <= 128) return launch_fused<kClassL>(G, partials, nblk, a, s);
    // (the largest windows' reduction needs every register: the finalize runs apart)
    const hipError_t e = launch_gram_finalize(G, partials, nblk, a.m, a.slots, a.st, s);
    return e != hipSuccess ? e : launch_one<double, kClassX>(a, s);
}

int trid_class(int m, int cplx) { return cplx ? (m <= 32 ? 0 : m <= 128 ? 1 : 2) : (m <= 64 ? 0 : m <= 128 ? 1 : 2); }

hipError_t launch_trid_grouped(const SolveArgs* const items[3], const int count[3], hipStream_t s, int m_small) {
    hipError_t e = launch_group<double, kClassX>(items[2], count[2], kMaxM, s);
    if (e == hipSuccess) e = launch_group<double, kClassL>(items[1], count[1], 128, s);
    if (e == hipSuccess) e = launch_group<double, kClassS>(items[0], count[0], m_small, s);
    return e;
}

hipError_t launch_trid_grouped_cplx(const SolveArgs* const items[3], const int count[3], hipStream_t s) {
    hipError_t e = count[2] > 0 ? launch_solve_trid_wide(nullptr, items[2], count[2], s) : hipSuccess;
    if (e == hipSuccess) e = launch_group<cplx, kClassL>(items[1], count[1], 128, s);
    if (e == hipSuccess) e = launch_group<cplx, kClassS>(items[0], count[0], 32, s);
    return e;
}

}  // namespace dmd
