// FP64 small solves of streaming DMD, run on the GPU after each Gram update.
//
// k_solve_sym (one workgroup):
//   * gathers xtx = X^* X (the first m window columns) from the physical Gram;
//   * eigendecomposition xtx V = V diag(d) by cyclic two-sided Jacobi with
//     parallel (round-robin) ordering: every round applies m/2 disjoint
//     rotations at once;  real symmetric or complex Hermitian;
//   * sigma = sqrt(|d|) sorted descending with V's columns permuted alike
//     (Algorithm 1), truncation to r_eff <= r resolvable values;
//   * A~ = Sigma^-1 V^* (X^* X') V Sigma^-1 from the Gram block xty without
//     forming U (Eq. Atilde; Algorithm 2; Sec. 3.4);
//   * POD coefficients V Sigma^-1 (Sec. 2.1, step 2).
// k_solve_eig (one workgroup):
//   * A~ W = W Lambda: Householder reduction to Hessenberg form, QR iteration
//     (real A~: double shifts; complex: Wilkinson shifts) to the Schur form
//     A~ = Z T Z^*, eigenvectors of T by back substitution, W = Z Y;
//   * eigenpairs sorted (|lambda| descending, arg ascending), W's columns
//     scaled to unit norm with the largest-modulus entry real positive;
//   * mode amplitudes b = (W Lambda)^-1 alpha_1 (Sec. 3.3) and the background
//     mode argmin |log lambda| (Algorithm 3);
//   * DMD coefficients C = V Sigma^-1 W for the projection Phi = X' C (Eq. Phi)
//     and the background coefficients C[:, bg] b_bg lambda_bg^m.
#include <type_traits>

#include "solve_common.h"

namespace dmd {
namespace {

// Round-robin tournament: in round `rd` (0 .. M-2) pair i (0 .. M/2-1) is (p, q);
// every index appears in exactly one pair per round and every pair of indices
// meets once per sweep.
__device__ __forceinline__ void rr_pair(int rd, int i, int M, int& p, int& q) {
    const int n1 = M - 1;
    if (i == 0) {
        p = n1;
        q = rd;
    } else {
        p = rd + i;
        if (p >= n1) p -= n1;
        q = rd - i;
        if (q < 0) q += n1;
    }
}

// Rotation (c, s) with c^2 + s^2 = 1 to working precision that annihilates
// the off-diagonal of the real 2x2 [[a, g], [g, b]] (g > 0): t = tan(phi) is
// the root of t^2 + 2 theta t - 1 = 0 of smaller modulus, theta = (b-a)/(2g).
__device__ __forceinline__ void jacobi_cs(double a, double b, double g, double& c, double& s) {
    const double theta = 0.5 * (b - a) * rcp_fast(g);
    double t;
    if (fabs(theta) > 1e100) {
        t = 0.5 * rcp_fast(theta);
    } else {
        const double q = fma(theta, theta, 1.0);
        const double den = fabs(theta) + q * rsqrt_acc(q);
        t = copysign(rcp_fast(den), theta);
        if (theta == 0.0) t = 1.0;
    }
    c = rsqrt_acc(fma(t, t, 1.0));
    s = t * c;
}

// Copies the results block (state, sigma, lambda) to its pinned host mirror so
// that the host reads a consistent snapshot of this solve after one event wait.
__device__ void publish(const SolveArgs& a) {
    __syncthreads();
    const int n4 = a.res_bytes / 4;
    const uint32_t* src = reinterpret_cast<const uint32_t*>(a.res_block);
    volatile uint32_t* dst = reinterpret_cast<volatile uint32_t*>(a.res_host);
    for (int i = threadIdx.x; i < n4; i += blockDim.x) dst[i] = src[i];
    __threadfence_system();
}

// --------------------------------------------------------------------------
// k_solve_sym
// --------------------------------------------------------------------------

// C = op(A) B for M x M matrices with leading dimension ld (op = identity or
// conjugate transpose).  LDS path: each thread owns a 4 x 4 block with rows
// strided by 16 so that a wavefront reads 16 consecutive rows per access.
template <typename S, int NT, bool CONJ_A>
__device__ void gemm_sq(S* __restrict__ C, const S* __restrict__ A, const S* __restrict__ B, int M, int ld) {
    using SC = Scal<S>;
    const int nrg = (M + 63) / 64;  // row/column super-groups of 64
    for (int t = threadIdx.x; t < 256 * nrg * nrg; t += NT) {
        const int g = t / 256, w = t % 256;
        const int i0 = (g % nrg) * 64 + (w % 16), j0 = (g / nrg) * 64 + (w / 16);
        S acc[4][4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[r][c] = SC::zero();
        for (int k = 0; k < M; ++k) {
            S av[4], bv[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = i0 + 16 * r;
                av[r] = i < M ? (CONJ_A ? SC::cj(A[k + (size_t)i * ld]) : A[i + (size_t)k * ld]) : SC::zero();
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int j = j0 + 16 * c;
                bv[c] = j < M ? B[k + (size_t)j * ld] : SC::zero();
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[r][c] = acc[r][c] + mulr(av[r], bv[c]);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int i = i0 + 16 * r, j = j0 + 16 * c;
                if (i < M && j < M) C[i + (size_t)j * ld] = acc[r][c];
            }
    }
}

template <typename S> __device__ __forceinline__ S load_s(const double* p, int64_t i);
template <> __device__ __forceinline__ double load_s<double>(const double* p, int64_t i) { return p[i]; }
template <> __device__ __forceinline__ cplx load_s<cplx>(const double* p, int64_t i) { return cplx{p[2 * i], p[2 * i + 1]}; }

// Common end of the symmetric solves: sigma sorted descending (stable in the
// index) with V permuted alike (Algorithm 1), the rank r_eff, canonical V_r,
// A~ = Sigma^-1 V_r^* xty V_r Sigma^-1 (Eq. Atilde, Algorithm 2), the POD
// coefficients V_r Sigma^-1 and the status.
// s_sig[i]: sigma of eigenvector i (i < m); Vc: eigenvectors by column
// (leading dimension ld), the first nvec of them valid (nvec >= r_eff);
// spare1, spare2: M x ld scratch.
template <typename S, int NT, int AHEAD = 1>
__device__ void sym_tail(const SolveArgs& a, int ld, S* Vc, S* spare1, S* spare2, double* s_sig, int* s_perm,
                         int nvec, int sweeps, bool converged, int warm) {
    using SC = Scal<S>;
    const int tid = threadIdx.x;
    const int slots = a.slots;
    DevState* st = a.st;
    const int m = window_cols(a.m, a.buildup, st);  // columns of X (fewer during a build-up start)
    const int ldv = a.m;                            // storage stride of V and V_full
    const int oldest = st->oldest;
    const int nw = NT / 64, lane = tid & 63, wv = tid >> 6;
    __shared__ int s_reff;
    for (int i = m + tid; i < a.m; i += NT) a.sigma[i] = 0.0;
    // sigma = sqrt(|d|), sorted descending (stable in the index)
    for (int i = tid; i < m; i += NT) {
        const double si = s_sig[i];
        int rank = 0;
        for (int j = 0; j < m; ++j) {
            const double sj = s_sig[j];
            rank += (sj > si) || (sj == si && j < i);
        }
        s_perm[rank] = i;
        a.sigma[rank] = si;
    }
    __syncthreads();
    if (tid == 0) {
        const double s0 = s_sig[s_perm[0]];
        int k = 0;
        if (s0 > 0.0) {
            const double thr = a.rcond * s0;
            const int lim = a.r < m ? a.r : m;
            while (k < lim && s_sig[s_perm[k]] > thr) ++k;
        }
        s_reff = k;
    }
    // the eigenvectors in sigma order, kept for the next solve's warm start
    // (only when all m are known and the window is full)
    const bool keep_full = nvec >= m && m == ldv;
    if (keep_full) {
        for (int idx = tid; idx < m * m; idx += NT) {
            const int i = idx % m, k = idx / m;
            store_s<S>(a.Vfull, i + (int64_t)k * ldv, Vc[i + (size_t)s_perm[k] * ld]);
        }
    }
    __syncthreads();
    const int k_eff = s_reff;

    // canonical V_r: column perm[k] of V, phase so that its largest-modulus
    // entry (lowest index on ties) is real positive
    S* Vr = spare1;  // m x k_eff, leading dimension ld
    for (int k = wv; k < k_eff; k += nw) {
        const int col = s_perm[k];
        double best = -1.0;
        int bi = 0;
        for (int i = lane; i < m; i += 64) {
            const double v = SC::absv(Vc[i + (size_t)col * ld]);
            if (v > best) { best = v; bi = i; }
        }
        for (int off = 32; off >= 1; off >>= 1) {
            const double ob = __shfl_xor(best, off, 64);
            const int oi = __shfl_xor(bi, off, 64);
            if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
        }
        const S ph = SC::cj(SC::phase(Vc[bi + (size_t)col * ld]));
        for (int i = lane; i < m; i += 64) {
            const S v = mulr(Vc[i + (size_t)col * ld], ph);
            Vr[i + (size_t)k * ld] = v;
            store_s<S>(a.V, i + (int64_t)k * ldv, v);
        }
        for (int i = m + lane; i < ldv; i += 64) store_s<S>(a.V, i + (int64_t)k * ldv, SC::zero());
    }
    __syncthreads();

    // T = xty V_r (m x k_eff) with xty[i][j] = <x_i, x_{j+1}>
    S* T = spare2;
    for (int idx = tid; idx < m * k_eff; idx += NT) {
        const int i = idx % m, b = idx / m;
        const int si = slot_of(oldest, i, slots);
        const S acc = ordered_dot<AHEAD>(SC::zero(), 0, 1, m,
                                     [&](int j) { return gram_at<S>(a.G, si, slot_of(oldest, j + 1, slots), slots); },
                                     [&](int j) { return Vr[j + (size_t)b * ld]; });
        T[i + (size_t)b * ld] = acc;
    }
    __syncthreads();

    // A~[p][q] = (V_r^* T)[p][q] / (sigma_p sigma_q)
    for (int idx = tid; idx < k_eff * k_eff; idx += NT) {
        const int p = idx % k_eff, q = idx / k_eff;
        const S acc = ordered_dot<AHEAD>(SC::zero(), 0, 1, m, [&](int i) { return SC::cj(Vr[i + (size_t)p * ld]); },
                                     [&](int i) { return T[i + (size_t)q * ld]; });
        const double sp = s_sig[s_perm[p]], sq = s_sig[s_perm[q]];
        store_s<S>(a.At, p + (int64_t)q * k_eff, acc * (1.0 / (sp * sq)));
    }
    // POD coefficients V_r Sigma^-1 (row-major m x r, real or interleaved complex)
    const int cw = (sizeof(S) == sizeof(cplx)) ? 2 : 1;
    for (int idx = tid; idx < m * k_eff; idx += NT) {
        const int i = idx / k_eff, q = idx % k_eff;
        const S v = Vr[i + (size_t)q * ld] * (1.0 / s_sig[s_perm[q]]);
        const cplx cv = SC::toc(v);
        const int64_t o = (int64_t)i * cw * a.r + (int64_t)cw * q;
        if (a.coef_f64) {
            double* B = reinterpret_cast<double*>(a.Bpod);
            B[o] = cv.re;
            if (cw == 2) B[o + 1] = cv.im;
        } else {
            float* B = reinterpret_cast<float*>(a.Bpod);
            B[o] = (float)cv.re;
            if (cw == 2) B[o + 1] = (float)cv.im;
        }
    }
    if (tid == 0) {
        const int lim = a.r < m ? a.r : m;
        st->skipped = 0;
        st->r_eff = k_eff;
        st->sweeps = sweeps;
        st->solve_status = converged ? (k_eff < lim ? ST_W_RANK : ST_OK) : ST_E_CONVERGENCE;
        if (k_eff == 0) st->solve_status = ST_W_RANK;
        st->vprev_valid = (converged && keep_full) ? 1 : 0;
        st->vprev_push = st->pushes;
        st->warm = warm;
    }
}

// LDS: matrices in dynamic LDS (real, M <= 64); else in the global workspace.
// PMAX: largest number of rotation pairs per round (M / 2).
template <typename S, int NT, bool LDS, int PMAX>
__device__ void solve_sym_body(const SolveArgs& a, int M) {
    using SC = Scal<S>;
    extern __shared__ double dyn[];
    const int tid = threadIdx.x;
    const int slots = a.slots;
    DevState* st = a.st;
    // the columns of X; a partial window (build-up) is the leading block of
    // the zero-padded M x M matrix, whose padding no rotation touches
    const int m = window_cols(a.m, a.buildup, st);
    if (m == 0) {
        if (tid == 0) {
            st->solve_status = ST_E_NOT_READY;
            st->r_eff = 0;
        }
        return;
    }
    if (st->vprev_valid && st->pushes == st->vprev_push) {
        // no snapshot was accepted since the last converged solve: its results stand
        if (tid == 0) st->skipped = 1;
        return;
    }
    const int oldest = st->oldest;
    const int ld = M + 1;  // odd leading dimension: column accesses spread over LDS banks
    const size_t MM = (size_t)M * ld;
    S* bufA;
    if constexpr (LDS) bufA = reinterpret_cast<S*>(dyn);
    else bufA = reinterpret_cast<S*>(a.work);
    S* bufV = bufA + MM;
    S* bufQ = bufV + MM;
    const int P = M / 2;

    __shared__ double s_c[PMAX], s_s[PMAX];
    __shared__ S s_e[PMAX];
    __shared__ int s_p[PMAX], s_q[PMAX];
    __shared__ int s_rot, s_warm;
    __shared__ double s_red[NT / 64];
    __shared__ double s_sig[2 * PMAX];
    __shared__ int s_perm[2 * PMAX];

    if (tid == 0) {
        // warm start from the previous solve's eigenvectors when the window
        // moved by exactly one snapshot (or not at all) since then
        int w = 0;
        if (a.warm_start && st->vprev_valid) {
            if (st->pushes == st->vprev_push + 1) w = 1;
            else if (st->pushes == st->vprev_push) w = 2;
        }
        s_warm = w;
    }
    // xtx = Gram of the first m window columns; padded to even M with a decoupled zero
    for (int idx = tid; idx < M * M; idx += NT) {
        const int i = idx % M, j = idx / M;
        S v = SC::zero();
        if (i < m && j < m) v = gram_at<S>(a.G, slot_of(oldest, i, slots), slot_of(oldest, j, slots), slots);
        bufA[i + (size_t)j * ld] = v;
    }
    __syncthreads();
    const int warm = s_warm;
    if (warm) {
        // Q = previous eigenvectors with rows shifted by one window position:
        // row i of Q is row i+1 of the previous V and the last row is the
        // previous first row (the departed snapshot), so Q stays unitary and
        // Q^* xtx Q is close to diagonal.
        const int shift = warm == 1 ? 1 : 0;
        for (int idx = tid; idx < M * M; idx += NT) {
            const int i = idx % M, j = idx / M;
            S v = (i == j) ? SC::one() : SC::zero();
            if (i < m && j < m) {
                int src = i + shift;
                if (src >= m) src -= m;
                v = load_s<S>(a.Vfull, src + (int64_t)j * a.m);
            }
            bufQ[i + (size_t)j * ld] = v;
        }
        __syncthreads();
        gemm_sq<S, NT, false>(bufV, bufA, bufQ, M, ld);  // T = xtx Q
        __syncthreads();
        gemm_sq<S, NT, true>(bufA, bufQ, bufV, M, ld);   // B = Q^* T
        __syncthreads();
        for (int idx = tid; idx < M * M; idx += NT) {    // exact Hermitian symmetry
            const int i = idx % M, j = idx / M;
            if (i < j) {
                const cplx u = SC::toc(bufA[i + (size_t)j * ld]), w = conj(SC::toc(bufA[j + (size_t)i * ld]));
                const S avg = SC::fromc(0.5 * (u + w));
                bufA[i + (size_t)j * ld] = avg;
                bufA[j + (size_t)i * ld] = SC::cj(avg);
            } else if (i == j) {
                bufA[i + (size_t)i * ld] = SC::fromc(mkc(SC::re(bufA[i + (size_t)i * ld])));
            }
        }
    }
    for (int idx = tid; idx < M * M; idx += NT) {
        const int i = idx % M, j = idx / M;
        bufV[i + (size_t)j * ld] = (i == j) ? SC::one() : SC::zero();
    }
    __syncthreads();

    // rotation floor: entries below 1e-18 * trace cannot move any eigenvalue
    // that a Gram accumulated in FP64 resolves
    double tr = 0.0;
    for (int i = tid; i < m; i += NT) tr += fabs(SC::re(bufA[i + (size_t)i * ld]));
    for (int off = 32; off >= 1; off >>= 1) tr += __shfl_xor(tr, off, 64);
    if ((tid & 63) == 0) s_red[tid >> 6] = tr;
    __syncthreads();
    tr = 0.0;
    for (int w = 0; w < NT / 64; ++w) tr += s_red[w];
    const double floor_abs = 1e-18 * tr;
    const double tol = a.tol;
    S* A = bufA;
    S* V = bufV;
    const int nw = NT / 64, lane = tid & 63, wv = tid >> 6;

    int sweep = 0;
    bool converged = false;
    for (; sweep < a.max_sweeps; ++sweep) {
        if (tid == 0) s_rot = 0;
        __syncthreads();
        for (int rd = 0; rd < M - 1; ++rd) {
            if (tid < P) {
                int p, q;
                rr_pair(rd, tid, M, p, q);
                const S apq = A[p + (size_t)q * ld];
                const double app = SC::re(A[p + (size_t)p * ld]);
                const double aqq = SC::re(A[q + (size_t)q * ld]);
                const double g = SC::absv(apq);
                double c = 1.0, s = 0.0;
                S e = SC::one();
                if (g > floor_abs && g * g > tol * tol * fabs(app * aqq)) {
                    jacobi_cs(app, aqq, g, c, s);
                    e = SC::phase(apq);
                    s_rot = 1;
                }
                s_c[tid] = c;
                s_s[tid] = s;
                s_e[tid] = e;
                s_p[tid] = p;
                s_q[tid] = q;
            }
            __syncthreads();
            // A <- J^* A J on 2x2 blocks (rows of pair k, columns of pair l), k <= l,
            // mirrored so that A stays exactly Hermitian.  Each half-wavefront
            // owns one row pair (its rotation is uniform) and its lanes walk l.
            for (int k = 2 * wv + (lane >> 5); k < P; k += 2 * nw) {
                const double sk = s_s[k], ck = s_c[k];
                const S ek = s_e[k];
                const int p = s_p[k], q = s_q[k];
                for (int l = k + (lane & 31); l < P; l += 32) {
                    const double sl = s_s[l];
                    if (sk == 0.0 && sl == 0.0) continue;
                    if (l == k) {
                        // the pair's own 2x2 block, rotated exactly as the others
                        // (in the basis where a_pq = g e is real): the new
                        // off-diagonal is zero up to rounding of (c, s)
                        const double aa = SC::re(A[p + (size_t)p * ld]), bb = SC::re(A[q + (size_t)q * ld]);
                        const double g = SC::absv(A[p + (size_t)q * ld]);
                        const double cs = ck * sk, c2 = ck * ck, s2 = sk * sk;
                        const double na = c2 * aa - 2.0 * cs * g + s2 * bb;
                        const double nb = s2 * aa + 2.0 * cs * g + c2 * bb;
                        const double nx = cs * (aa - bb) + (c2 - s2) * g;
                        A[p + (size_t)p * ld] = SC::fromc(mkc(na));
                        A[q + (size_t)q * ld] = SC::fromc(mkc(nb));
                        A[p + (size_t)q * ld] = nx * ek;
                        A[q + (size_t)p * ld] = SC::cj(nx * ek);
                        continue;
                    }
                    const int u = s_p[l], v = s_q[l];
                    const double cl = s_c[l];
                    const S el = s_e[l];
                    const S apu = A[p + (size_t)u * ld], apv = A[p + (size_t)v * ld];
                    const S aqu = A[q + (size_t)u * ld], aqv = A[q + (size_t)v * ld];
                    // rows: p' = c p - s e q ;  q' = s conj(e) p + c q
                    const S bpu = ck * apu - sk * mulr(ek, aqu);
                    const S bpv = ck * apv - sk * mulr(ek, aqv);
                    const S bqu = sk * mulr(SC::cj(ek), apu) + ck * aqu;
                    const S bqv = sk * mulr(SC::cj(ek), apv) + ck * aqv;
                    // columns: u' = c u - s conj(e) v ;  v' = s e u + c v
                    const S npu = cl * bpu - sl * mulr(SC::cj(el), bpv);
                    const S npv = sl * mulr(el, bpu) + cl * bpv;
                    const S nqu = cl * bqu - sl * mulr(SC::cj(el), bqv);
                    const S nqv = sl * mulr(el, bqu) + cl * bqv;
                    A[p + (size_t)u * ld] = npu;
                    A[p + (size_t)v * ld] = npv;
                    A[q + (size_t)u * ld] = nqu;
                    A[q + (size_t)v * ld] = nqv;
                    A[u + (size_t)p * ld] = SC::cj(npu);
                    A[v + (size_t)p * ld] = SC::cj(npv);
                    A[u + (size_t)q * ld] = SC::cj(nqu);
                    A[v + (size_t)q * ld] = SC::cj(nqv);
                }
            }
            // V <- V J: one wavefront per pair, lanes over rows
            for (int k = wv; k < P; k += nw) {
                const double sk = s_s[k];
                if (sk == 0.0) continue;
                const double ck = s_c[k];
                const S ek = s_e[k];
                const int p = s_p[k], q = s_q[k];
                for (int i = lane; i < M; i += 64) {
                    const S vp = V[i + (size_t)p * ld], vq = V[i + (size_t)q * ld];
                    V[i + (size_t)p * ld] = ck * vp - sk * mulr(SC::cj(ek), vq);
                    V[i + (size_t)q * ld] = sk * mulr(ek, vp) + ck * vq;
                }
            }
            __syncthreads();
        }
        if (s_rot == 0) {
            converged = true;
            break;
        }
        __syncthreads();
    }

    // eigenvalues d, then eigenvectors of xtx: V (cold) or Q V (warm)
    for (int i = tid; i < m; i += NT) s_sig[i] = sqrt(fabs(SC::re(A[i + (size_t)i * ld])));
    __syncthreads();
    S* Vc;
    S* spare1;
    S* spare2;
    if (warm) {
        gemm_sq<S, NT, false>(bufA, bufQ, bufV, M, ld);
        Vc = bufA;
        spare1 = bufV;
        spare2 = bufQ;
    } else {
        Vc = bufV;
        spare1 = bufA;
        spare2 = bufQ;
    }
    sym_tail<S, NT, kAhead<S, LDS>>(a, ld, Vc, spare1, spare2, s_sig, s_perm, m, sweep + (converged ? 1 : 0), converged, warm);
}

template <typename S, int NT, bool LDS, int PMAX>
__global__ __launch_bounds__(NT)
void k_solve_sym(SolveArgs a, int M) {
    solve_sym_body<S, NT, LDS, PMAX>(a, M);
}

// Grouped form: one workgroup per stream (independent solves run on separate CUs).
template <typename S, int NT, bool LDS, int PMAX>
__global__ __launch_bounds__(NT)
void k_solve_sym_grouped(const SolveArgs* __restrict__ items) {
    const SolveArgs a = items[blockIdx.x];
    solve_sym_body<S, NT, LDS, PMAX>(a, a.m + (a.m & 1));
}

// --------------------------------------------------------------------------
// k_solve_eig: A~ (k x k, k <= 32) in LDS, 4 wavefronts.  The Hessenberg
// reduction, the QR iteration and the triangular solves are one wavefront's
// (chains of dependent steps); products with all eigenvectors are shared.
//
// M holds H in rows 0 .. 31 and the accumulated transformation Z in rows
// 32 .. 63 of the same columns: a transformation from the right is one
// instruction stream for the 64 lanes (lane = row of either), and H's rows
// past the active ones are zero there, so no lane needs a mask.  Odd column
// stride: lanes along a row (lane = column) and along a column hit different
// banks.
//
// Bound by the latency of those chains.  Against one wavefront with H and Z in
// arrays of their own and b always from a pivoted elimination: r = 10 real
// 117 -> 66 us, r = 20 330 -> 169, r = 32 857 -> 362, r = 24 complex 685 -> 471;
// 24 windows of a tick 878 -> 419.
// --------------------------------------------------------------------------
constexpr int LDM = 65;
constexpr int kEigCols = 39;  // 32, and the (zero) columns that a run of eight may reach past them
constexpr int kEigThreads = 256;
constexpr int LDH = kRMax + 1;  // column stride of the eigenvector matrices

template <int I, int N, typename F> __device__ __forceinline__ void each_i(F f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        each_i<I + 1, N>(f);
    }
}
__device__ __forceinline__ double sqr(double a) { return a * a; }
__device__ __forceinline__ double sqr(cplx a) { return fma(a.im, a.im, a.re * a.re); }
__device__ __forceinline__ double fmac(double a, double b, double c) { return fma(a, b, c); }
__device__ __forceinline__ cplx fmac(cplx a, cplx b, cplx c) {
    return {fma(-a.im, b.im, fma(a.re, b.re, c.re)), fma(a.im, b.re, fma(a.re, b.im, c.im))};
}
__device__ __forceinline__ cplx fmac(double a, cplx b, cplx c) { return {fma(a, b.re, c.re), fma(a, b.im, c.im)}; }
__device__ __forceinline__ double other_half_sum(double x) {  // x of this lane plus x of lane ^ 32
    return row_fold<32>(x, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ cplx other_half_sum(cplx x) { return {other_half_sum(x.re), other_half_sum(x.im)}; }
// a / b by the reciprocal of |b|^2 where that is in range
__device__ __forceinline__ cplx div_fast(cplx a, cplx b) {
    const double b2 = sqr(b);
    if (b2 > 1e-280 && b2 < 1e280) return rcp_acc(b2) * mul_conj(a, b);
    return cdiv(a, b);
}

// Householder reduction of H to upper Hessenberg form, Z accumulating: column
// c's reflector u (kept unnormalized, in hv) from the left (lane = column, its
// rows c+1 .. in registers, eight at a time) and from the right (lane = row of
// H or Z).  Entries past the matrix meet zeros of u.
template <typename S>
__device__ __forceinline__ void hessenberg(S* M, S* hv, int k, int lane) {
    using SC = Scal<S>;
    for (int c = 0; c + 2 < k; ++c) {
        const int len = k - c - 1;  // rows c+1 .. k-1
        const S* col = M + c * LDM + c + 1;
        const S xl = lane < len ? col[lane < len ? lane : 0] : SC::zero();
        const S x0 = col[0];
        const double tail2 = wave_sum(lane >= 1 && lane < len ? sqr(xl) : 0.0);
        if (__builtin_amdgcn_readfirstlane(tail2 == 0.0)) continue;
        const double ax0 = SC::absv(x0), alpha = sqrt(ax0 * ax0 + tail2);
        const S ph = SC::phase(x0);
        wave_sync();
        if (lane < 32) hv[lane] = lane == 0 ? x0 + ph * alpha : xl;
        wave_sync();
        const double tau = 1.0 / (alpha * (alpha + ax0));
        S r[32];
        auto reflect = [&](S* p, int stride, bool left) {
            S w0 = SC::zero(), w1 = SC::zero();
            each_i<0, 4>([&](auto ch) {
                if (8 * ch() < len)
                    each_i<0, 8>([&](auto u) {
                        constexpr int i = 8 * ch() + u();
                        r[i] = p[i * stride];
                        const S v = left ? SC::cj(hv[i]) : hv[i];
                        if constexpr (i % 2) w1 = fmac(r[i], v, w1);
                        else w0 = fmac(r[i], v, w0);
                    });
            });
            const S w = (w0 + w1) * -tau;
            each_i<0, 4>([&](auto ch) {
                if (8 * ch() < len)
                    each_i<0, 8>([&](auto u) {
                        constexpr int i = 8 * ch() + u();
                        p[i * stride] = fmac(left ? hv[i] : SC::cj(hv[i]), w, r[i]);
                    });
            });
        };
        reflect(M + (lane & 31) * LDM + c + 1, 1, true);  // (both halves of the wavefront alike)
        wave_sync();
        reflect(M + (c + 1) * LDM + lane, LDM, false);
        wave_sync();
        if (lane < len) M[c * LDM + c + 1 + lane] = lane == 0 ? ph * -alpha : SC::zero();
        wave_sync();
    }
}

// Deflation: the largest l in [1, hi] with a negligible subdiagonal entry
// (set to zero), else 0.
template <typename S>
__device__ __forceinline__ int deflate(S* M, int hi, int lane, double hmax) {
    using SC = Scal<S>;
    bool small = false;
    if (lane >= 1 && lane <= hi) {
        const double sub = SC::absv(M[(lane - 1) * LDM + lane]);
        double scale = SC::absv(M[lane * LDM + lane]) + SC::absv(M[(lane - 1) * LDM + lane - 1]);
        if (scale == 0.0) scale = hmax;
        small = sub <= kEps * scale;
    }
    const unsigned long long mask = __ballot(small);
    const int l = mask ? 63 - __clzll(mask) : 0;
    wave_sync();
    if (l > 0 && lane == 0) M[(l - 1) * LDM + l] = SC::zero();
    wave_sync();
    return l;
}

// Real Schur form of the real upper Hessenberg H: implicit double-shift
// (Francis) QR -- each sweep chases a 3 x 3 Householder bulge started from
// the first column of (H - mu1)(H - mu2), mu1,2 the eigenvalues of the
// trailing 2 x 2 block (an exceptional pair every 10th sweep), so that a
// complex-conjugate pair converges together in real arithmetic.
//
// A step is one chain: the reflector from (x, y, z) (in registers: u =
// (x + sign(x) s, y, z), s = ||(x, y, z)||, tau = 2 / u^T u, by the
// hardware estimates plus Newton steps), the three rows (lane = column), LDS,
// the three columns (lane = row of H or Z), and the next (x, y, z) from the
// lanes that hold them.  22 sweeps of a 20 x 20 matrix take about 73 us,
// deflation checks included (about 750 cycles a step); with the rows of Z apart
// from H's and masked writes a step took 1000 to 1200.
__device__ __forceinline__ void real_schur(double* M, int k, int lane, int max_iter, double hmax, int& total,
                                           bool& failed) {
    auto h = [&](int i, int j) -> double& { return M[j * LDM + i]; };
    const int j = lane & 31;
    int nn = k - 1, its = 0;
    while (nn >= 0) {
        const int l = deflate(M, nn, lane, hmax);
        if (l >= nn - 1) {  // a 1 x 1 or 2 x 2 block splits off
            nn = l - 1;
            its = 0;
            continue;
        }
        if (its >= max_iter) {
            failed = true;
            break;
        }
        ++its;
        ++total;
        // shift pair by its sum s and product t
        double s, t;
        {
            const double a11 = h(nn - 1, nn - 1), a12 = h(nn - 1, nn), a21 = h(nn, nn - 1), a22 = h(nn, nn);
            if (its % 10 == 0) {
                const double e = fabs(a21) + fabs(h(nn - 1, nn - 2));
                const double mu = a22 + 0.75 * e;
                s = 2.0 * mu;
                t = mu * mu + 0.4375 * e * e;
            } else {
                s = a11 + a22;
                t = a11 * a22 - a12 * a21;
            }
        }
        double x, y, z;
        {
            const double h00 = h(l, l), h10 = h(l + 1, l);
            x = h00 * h00 + h(l, l + 1) * h10 - s * h00 + t;
            y = h10 * (h00 + h(l + 1, l + 1) - s);
            z = h10 * h(l + 2, l + 1);
            // (products of entries: scaled, so that their squares stay in range)
            const int e = -__builtin_amdgcn_frexp_exp(fmax(fabs(x), fmax(fabs(y), fabs(z))));
            x = ldexp(x, e);
            y = ldexp(y, e);
            z = ldexp(z, e);
        }
        for (int kk = l; kk < nn; ++kk) {
            double* row = M + j * LDM + kk;     // rows kk .. kk+2 of column j
            double* col = M + kk * LDM + lane;  // columns kk .. kk+2 of row `lane`
            const double r0 = row[0], r1 = row[1], r2 = row[2];
            const double yz2 = fma(y, y, z * z), s2 = fma(x, x, yz2);
            const bool none = !(s2 > 1e-300);   // (nothing to annihilate: z and y are zero, or vanish beside H)
            const double u = x + copysign(s2 * rsqrt_acc(s2), x), u0 = none ? 0.0 : u;
            // (tau = 2 / u^T u from u itself and not from the norms: I - tau u u^T is
            // then orthogonal to the rounding of tau alone)
            const double half_tau = none ? 0.0 : rcp_acc(fma(u, u, yz2)), tau = 2.0 * half_tau;
            const double ru = fma(u0, r0, fma(y, r1, z * r2)), f = half_tau * (ru + ru);
            // the entries below the subdiagonal of column kk-1 become zero
            const bool below = kk > l && j == kk - 1;
            const double n0 = fma(-f, u0, r0), n1 = fma(-f, y, r1), n2 = fma(-f, z, r2);
            row[0] = n0;
            row[1] = below && !none ? 0.0 : n1;
            row[2] = below && !none && kk + 2 <= nn ? 0.0 : n2;
            wave_sync();
            const double c0 = col[0], c1 = col[LDM], c2 = col[2 * LDM];
            const double g = tau * fma(u0, c0, fma(y, c1, z * c2));
            const double d0 = fma(-g, u0, c0);
            col[0] = d0;
            col[LDM] = fma(-g, y, c1);
            col[2 * LDM] = fma(-g, z, c2);
            wave_sync();
            // rows kk+1 .. kk+3 of column kk (z = 0 exactly when the next step has two rows)
            x = lane_f64(d0, kk + 1);
            y = lane_f64(d0, kk + 2);
            z = kk + 3 <= nn ? lane_f64(d0, kk + 3) : 0.0;
        }
    }
}

// Complex Schur form of the complex upper Hessenberg H: single-shift QR with
// Wilkinson shifts, one rotation per step (as the real sweep).
__device__ __forceinline__ void complex_schur(cplx* M, int k, int lane, int max_iter, double hmax, int& total,
                                              bool& failed) {
    auto h = [&](int i, int j) -> cplx& { return M[j * LDM + i]; };
    const int j = lane & 31;
    int hi = k - 1, iter = 0;
    while (hi > 0) {
        const int l = deflate(M, hi, lane, hmax);
        if (l == hi) {
            --hi;
            iter = 0;
            continue;
        }
        if (iter >= max_iter) {
            failed = true;
            break;
        }
        ++iter;
        ++total;
        // Wilkinson shift: eigenvalue of the trailing 2x2 closer to H[hi][hi];
        // every 10th iteration an exceptional shift
        const cplx ta = h(hi - 1, hi - 1), tb = h(hi - 1, hi), tc = h(hi, hi - 1), td = h(hi, hi);
        cplx mu;
        if (iter % 10 == 0) {
            mu = td + mkc(0.75 * cabs(tc));
        } else {
            const cplx half = 0.5 * (ta - td);
            const cplx disc = csqrt(half * half + tb * tc);
            const cplx mu1 = td + half + disc, mu2 = td + half - disc;
            // (a+d)/2 +- disc == d + (a-d)/2 +- disc
            mu = (cabs(mu1 - td) <= cabs(mu2 - td)) ? mu1 : mu2;
        }
        cplx x = h(l, l) - mu, y = h(l + 1, l);
        for (int kk = l; kk < hi; ++kk) {
            cplx* row = M + j * LDM + kk;
            cplx* col = M + kk * LDM + lane;
            const cplx ru = row[0], rv = row[1];
            // G = [[c, s], [-conj(s), c]] with G [x; y] = [rho; 0]:
            // c = |x| / r, s = (x / |x|) conj(y) / r, r^2 = |x|^2 + |y|^2
            double c;
            cplx s;
            const double x2 = abs2(x), y2 = abs2(y);
            if (x2 > 1e-250 && y2 > 1e-250 && x2 < 1e250 && y2 < 1e250) {
                const double rx = rsqrt_acc(x2), rr = rsqrt_acc(x2 + y2);
                c = x2 * rx * rr;
                s = (rx * rr) * mul_conj(x, y);
            } else if (y2 == 0.0) {
                c = 1.0;
                s = mkc(0.0);
            } else if (x2 == 0.0) {
                c = 0.0;
                s = mkc(1.0);
            } else {
                const double ax = cabs(x), rr = hypot(ax, cabs(y));
                c = ax / rr;
                s = (1.0 / rr) * mul_conj(cplx{x.re / ax, x.im / ax}, y);
            }
            const bool below = kk > l && j == kk - 1;
            row[0] = c * ru + s * rv;
            row[1] = below ? mkc(0.0) : c * rv - conj_mul(s, ru);
            wave_sync();
            const cplx u = col[0], v = col[LDM];
            const cplx nc = c * u + mul_conj(v, s);
            col[0] = nc;
            col[LDM] = c * v - u * s;
            wave_sync();
            // rows kk+1, kk+2 of column kk (not used past the last step)
            x = cplx{lane_f64(nc.re, kk + 1), lane_f64(nc.im, kk + 1)};
            y = cplx{lane_f64(nc.re, kk + 2), lane_f64(nc.im, kk + 2)};
        }
    }
}

// Triangularizes each 2 x 2 diagonal block [[a, b], [c, d]], c != 0, of a real
// Schur form held as complex values: with u = (lambda_1 - d, c) / ||.||,
// lambda_1 an eigenvalue of the block, the rotation G = [[u0, -conj(u1)],
// [u1, conj(u0)]] gives G^* B G = [[lambda_1, .], [0, lambda_2]].
__device__ __forceinline__ void split_blocks(cplx* M, int k, int lane) {
    const int j = lane & 31;
    for (int i = 0; i + 1 < k; ++i) {
        const double c = M[i * LDM + i + 1].re;
        if (__builtin_amdgcn_readfirstlane(c == 0.0)) continue;
        const double a = M[i * LDM + i].re, b = M[(i + 1) * LDM + i].re, d = M[(i + 1) * LDM + i + 1].re;
        const double half = 0.5 * (a - d), disc = half * half + b * c;
        cplx l1;
        if (disc >= 0.0) l1 = mkc(0.5 * (a + d) + copysign(sqrt(disc), half));
        else l1 = cplx{0.5 * (a + d), sqrt(-disc)};
        cplx u0 = l1 - mkc(d), u1 = mkc(c);
        const double nu = 1.0 / sqrt(abs2(u0) + abs2(u1));
        u0 = nu * u0;
        u1 = nu * u1;
        wave_sync();
        {
            cplx* row = M + j * LDM + i;  // rows i, i+1 (zero before column i)
            const cplx r0 = row[0], r1 = row[1];
            row[0] = conj_mul(u0, r0) + conj_mul(u1, r1);
            row[1] = u0 * r1 - u1 * r0;
        }
        wave_sync();
        {
            cplx* col = M + i * LDM + lane;  // columns i, i+1 (H zero past row i+1)
            const cplx c0 = col[0], c1 = col[LDM];
            col[0] = c0 * u0 + c1 * u1;
            col[LDM] = mul_conj(c1, u0) - mul_conj(c0, u1);
        }
        wave_sync();
        if (lane == 0) M[i * LDM + i + 1] = mkc(0.0);
        wave_sync();
        ++i;  // the next row belongs to this block
    }
}

// LDS of the eig solve.
struct EigShared {
    cplx M[LDM * kEigCols];                  // H over Z, complex
    union {
        double R[LDM * kEigCols];            // real A~: H over Z until the real Schur form
        cplx Y[LDH * LDH];                   // then the eigenvectors of T, then W in sorted order
    };
    union {
        double hvr[40];
        cplx hv[40];
    };
    cplx lam[kRMax], ls[kRMax];              // eigenvalues: Schur order, sorted
    cplx al[kRMax];                          // POD coefficients alpha_1 of the first snapshot
    cplx x[kRMax];                           // expansion of alpha_1 in the unscaled eigenvectors
    cplx b[kRMax];                           // mode amplitudes
    int piv[kRMax];                          // pivot rows of the elimination for b
    double mod[kRMax], arg[kRMax], isig[kRMax];
    cplx fbg;                                // lambda_bg^m
    int bg, total, failed, redo;
};

// Whether the amplitudes b reproduce the first snapshot with the published W
// and lambda: |alpha_1 - W Lambda b| <= 64 eps |alpha_1|.  b comes from the
// triangle of the Schur vectors, before pairs were made conjugate and columns
// scaled.  A nearly defective A~ (a window with a linear trend) has nearly
// parallel eigenvectors and large b that cancel, and those last changes to W then
// cost up to the size of alpha_1 itself: such a window is solved again.
__device__ __forceinline__ void check_amplitudes(EigShared& sh, int k) {
    const int lane = threadIdx.x & 63, i = lane & 31, hf = lane >> 5;
    if (lane < 32) sh.x[i] = i < k ? sh.ls[i] * sh.b[i] : mkc(0.0);
    wave_sync();
    cplx r = hf ? mkc(0.0) : sh.al[i] * -1.0;
    for (int q0 = 16 * hf; q0 < 16 * hf + 16 && q0 < k; q0 += 4) {
        cplx y[4], xx[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            y[u] = sh.Y[i + (q0 + u) * LDH];
            xx[u] = sh.x[q0 + u];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) r = fmac(y[u], xx[u], r);
    }
    r = other_half_sum(r);
    const double n2 = wave_sum(lane < k ? sqr(r) : 0.0), a2 = wave_sum(lane < k ? sqr(sh.al[i]) : 0.0);
    if (lane == 0) sh.redo = !(n2 <= (64.0 * kEps) * (64.0 * kEps) * a2);
}

// b = (W Lambda)^-1 alpha_1 (Sec. 3.3) by Gaussian elimination with partial
// pivoting on the published W and lambda.
//
// H over Z is free by now: its first rows take W Lambda.  Thread (i, g) keeps
// the entries of row i in columns g, g + 8, .. in registers and copies them to
// LDS, where a step reads column c and the pivot row; what it leaves in columns
// up to c is not used again.  Rows stay in place; every wavefront finds the
// pivot row by itself (32 bits hold the leading bits of an entry's square and
// its row), so that a step has one barrier.  A zero pivot (an eigenvalue of
// zero) gives its mode amplitude 0.  0.45 us a step.
__device__ __forceinline__ void solve_amplitudes(EigShared& sh, int k) {
    const int tid = threadIdx.x, lane = tid & 63, i = tid & 31, g = tid >> 5;
    cplx* A = sh.M;
    cplx own[4], rhs = mkc(0.0);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int q = g + 8 * u;
        own[u] = i < k && q < k ? sh.Y[i + q * LDH] * sh.ls[q] : mkc(0.0);
        A[q * LDM + i] = own[u];
    }
    if (g == 0) {
        rhs = sh.al[i];
        sh.hv[i] = rhs;
    }
    __syncthreads();
    bool free_row = i < k;
    each_i<0, 4>([&](auto ph) {  // steps 8 ph .. 8 ph + 7: columns before 8 ph are done
        const int end = 8 * ph() + 8 < k ? 8 * ph() + 8 : k;
        for (int c = 8 * ph(); c < end; ++c) {
            const cplx aic = A[c * LDM + i];
            const unsigned hi = (unsigned)(__builtin_bit_cast(unsigned long long, abs2(aic)) >> 32);
            unsigned key = free_row ? (hi & ~31u) | (unsigned)(31 - i) : 0u;
            auto lvl = [&](auto ctrl) {
                const unsigned o = (unsigned)__builtin_amdgcn_mov_dpp((int)key, decltype(ctrl)::value, 0xF, 0xF, true);
                key = o > key ? o : key;
            };
            lvl(std::integral_constant<int, 0xB1>{});
            lvl(std::integral_constant<int, 0x4E>{});
            lvl(std::integral_constant<int, 0x141>{});
            lvl(std::integral_constant<int, 0x140>{});
            const auto sw = __builtin_amdgcn_permlane16_swap(key, key, false, false);
            const int p = __builtin_amdgcn_readfirstlane(31 - (int)((sw[0] > sw[1] ? sw[0] : sw[1]) & 31u));
            const cplx pv = A[c * LDM + p];
            cplx top[4];
            each_i<ph(), 4>([&](auto u) { top[u()] = A[(g + 8 * u()) * LDM + p]; });
            const cplx rp = sh.hv[p];
            if (tid == p) sh.piv[c] = p;
            free_row = free_row && i != p;
            const cplx f = div_fast(aic, pv) * -1.0;
            if (free_row && abs2(pv) > 0.0) {
                each_i<ph(), 4>([&](auto u) {
                    own[u()] = fmac(f, top[u()], own[u()]);
                    A[(g + 8 * u()) * LDM + i] = own[u()];
                });
                if (g == 0) {
                    rhs = fmac(f, rp, rhs);
                    sh.hv[i] = rhs;
                }
            }
            __syncthreads();
        }
    });
    if (tid < 64) {
        const int l = i < k ? i : k - 1, p = sh.piv[l];
        cplx r = sh.hv[p];
        const cplx pv = A[l * LDM + p];
        const cplx inv = abs2(pv) > 0.0 ? div_fast(mkc(1.0), pv) : mkc(0.0);
        cplx cn = A[(k - 1) * LDM + p], b = mkc(0.0);
        for (int c = k - 1; c >= 0; --c) {
            const cplx cc = cn;
            cn = A[(c > 0 ? c - 1 : 0) * LDM + p];
            const cplx x = r * inv, xc = {lane_f64(x.re, c), lane_f64(x.im, c)};
            if (l == c) b = xc;
            if (l < c) r = fmac(cc * -1.0, xc, r);
        }
        if (lane < k) sh.b[lane] = b;
    }
}

// C = V_r Sigma^-1 W: a thread keeps a row of V_r Sigma^-1 in registers, W
// (sorted) is in LDS.  Windows of up to 64 (128) columns have four (two)
// threads for a row, each with its share of the columns of C; several rows of W for two
// columns are read at a time.  With a thread per row, complex rows for real V and
// one row of W at a time it took 26 us of the solve's 189 (m = 64, r = 20), now 169 in all.
template <typename S>
__device__ __forceinline__ void coef_rows(const SolveArgs& a, EigShared& sh, int m, int k) {
    using SC = Scal<S>;
    constexpr int U = sizeof(S) == sizeof(cplx) ? 2 : 4;  // rows of W read at a time (registers)
    const int ldv = a.m, bgq = sh.bg;
    const cplx fbg = sh.b[bgq] * sh.fbg;
    const int parts = m <= 64 ? 4 : m <= 128 ? 2 : 1, rows = kEigThreads / parts;
    const int part = __builtin_amdgcn_readfirstlane(threadIdx.x / rows);
    for (int i = threadIdx.x % rows; i < m; i += rows) {
        // (columns past k-1 read column k-1 and are zeroed: every load in flight at once)
        S vrow[kRMax];
#pragma unroll
        for (int p = 0; p < kRMax; ++p) {
            vrow[p] = reinterpret_cast<const S*>(a.V)[(unsigned)((p < k ? p : k - 1) * ldv) + (unsigned)i];
        }
#pragma unroll
        for (int p = 0; p < kRMax; ++p) vrow[p] = p < k ? vrow[p] * sh.isig[p] : SC::zero();
        auto emit = [&](int q, const cplx& acc) {
            if (q == bgq && a.Bbg) {
                // background coefficients beta_i = C[i][bg] b_bg lambda_bg^m
                const cplx bt = acc * fbg;
                if (a.coef_f64) {
                    reinterpret_cast<double*>(a.Bbg)[2 * i] = bt.re;
                    reinterpret_cast<double*>(a.Bbg)[2 * i + 1] = bt.im;
                } else {
                    reinterpret_cast<float*>(a.Bbg)[2 * i] = (float)bt.re;
                    reinterpret_cast<float*>(a.Bbg)[2 * i + 1] = (float)bt.im;
                }
            }
            const int64_t o = (int64_t)i * 2 * a.r + 2 * q;
            if (a.coef_f64) {
                double* B = reinterpret_cast<double*>(a.Bphi);
                B[o] = acc.re;
                B[o + 1] = acc.im;
            } else {
                float* B = reinterpret_cast<float*>(a.Bphi);
                B[o] = (float)acc.re;
                B[o + 1] = (float)acc.im;
            }
        };
        for (int q = 2 * part; q < k; q += 2 * parts) {
            const cplx* w0 = sh.Y + q * LDH;
            const cplx* w1 = sh.Y + (q + 1 < k ? q + 1 : q) * LDH;
            cplx a0 = mkc(0.0), a1 = mkc(0.0), b0 = mkc(0.0), b1 = mkc(0.0);
            each_i<0, kRMax / U>([&](auto ch) {
                constexpr int p = U * ch();
                if (p < k) {  // (rows of W past k-1 are finite and meet zeros)
                    __builtin_amdgcn_sched_barrier(0);
                    cplx y0[U], y1[U];
                    each_i<0, U>([&](auto u) {
                        y0[u()] = w0[p + u()];
                        y1[u()] = w1[p + u()];
                    });
                    each_i<0, U>([&](auto u) {
                        constexpr int e = u();
                        if constexpr (e % 2) {
                            a1 = fmac(vrow[p + e], y0[e], a1);
                            b1 = fmac(vrow[p + e], y1[e], b1);
                        } else {
                            a0 = fmac(vrow[p + e], y0[e], a0);
                            b0 = fmac(vrow[p + e], y1[e], b0);
                        }
                    });
                }
            });
            emit(q, a0 + a1);
            if (q + 1 < k) emit(q + 1, b0 + b1);
        }
    }
}

__device__ __forceinline__ void solve_eig_body(const SolveArgs& a, EigShared& sh) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    DevState* st = a.st;
    const int status0 = st->solve_status;
    const int k = st->r_eff;
    const int m = window_cols(a.m, a.buildup, st);  // columns of X
    if (st->skipped) {
        publish(a);
        return;
    }
    if (status0 == ST_E_NOT_READY || k == 0) {
        if (tid == 0 && status0 != ST_E_NOT_READY) st->solves += 1;
        publish(a);
        return;
    }
    // H = A~, Z = I (columns and rows past k zero)
    if (a.cplx) {
        for (int idx = tid; idx < LDM * kEigCols; idx += kEigThreads) {
            const int i = idx % LDM, jj = idx / LDM;
            const bool in = i < k && jj < k;
            const int64_t o = in ? 2 * (i + jj * k) : 0;
            const double re = a.At[o], im = a.At[o + 1];
            sh.M[idx] = in ? cplx{re, im} : mkc(i == jj + 32 && jj < 32 ? 1.0 : 0.0);
        }
    } else {
        for (int idx = tid; idx < LDM * kEigCols; idx += kEigThreads) {
            const int i = idx % LDM, jj = idx / LDM;
            const bool in = i < k && jj < k;
            const double v = a.At[in ? i + jj * k : 0];
            sh.R[idx] = in ? v : i == jj + 32 && jj < 32 ? 1.0 : 0.0;
        }
    }
    if (tid < kRMax) {
        const double sg = tid < k ? a.sigma[tid] : 1.0;
        sh.isig[tid] = 1.0 / sg;
        cplx al = mkc(0.0);  // Sigma_r V_r^* e_1 (Sec. 3.3)
        if (tid < k) {
            const int64_t o = (int64_t)tid * a.m;
            al = a.cplx ? sg * cplx{a.V[2 * o], -a.V[2 * o + 1]} : mkc(sg * a.V[o]);
        }
        sh.al[tid] = al;
    }
    __syncthreads();
    if (wave == 0) {
        int total = 0;
        bool failed = false;
        double hmax = 0.0;
        if (a.cplx) {
            hessenberg<cplx>(sh.M, sh.hv, k, lane);
            for (int idx = lane; idx < k * k; idx += 64) hmax = fmax(hmax, cabs(sh.M[(idx / k) * LDM + idx % k]));
            hmax = wave_max(hmax);
            complex_schur(sh.M, k, lane, a.max_qr_iter, hmax, total, failed);
            wave_sync();
        } else {
            hessenberg<double>(sh.R, sh.hvr, k, lane);
            for (int idx = lane; idx < k * k; idx += 64) hmax = fmax(hmax, fabs(sh.R[(idx / k) * LDM + idx % k]));
            hmax = wave_max(hmax);
            real_schur(sh.R, k, lane, a.max_qr_iter, hmax, total, failed);
            wave_sync();
            for (int jj = 0; jj < kEigCols; ++jj) sh.M[jj * LDM + lane] = mkc(sh.R[jj * LDM + lane]);
            wave_sync();
            split_blocks(sh.M, k, lane);
        }
        const double smallnum = (hmax > 0.0 ? hmax : 1.0) * kEps;
        // ---- eigenvectors of the triangular T: (T - t_qq) y = 0, y_q = 1 (lane q)
        const int q = lane & 31;
        const cplx lq = sh.M[q * LDM + q];
        cplx* Yq = sh.Y + q * LDH;
        if (lane < 32)
            for (int i = 0; i < LDH; ++i) Yq[i] = mkc(i == q ? 1.0 : 0.0);
        if (lane < k) sh.lam[lane] = lq;
        wave_sync();
        for (int i = k - 2; i >= 0; --i) {
            cplx a0 = mkc(0.0), a1 = mkc(0.0);
            for (int j0 = i + 1; j0 < k; j0 += 4) {  // (y_j = 0 past q; T's columns past k are zero)
                cplx tt[4], yy[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int jj = j0 + u < k ? j0 + u : k - 1;
                    tt[u] = sh.M[(j0 + u) * LDM + i];
                    yy[u] = Yq[jj];
                }
                a0 = fmac(tt[0], yy[0], a0);
                a1 = fmac(tt[1], yy[1], a1);
                a0 = fmac(tt[2], yy[2], a0);
                a1 = fmac(tt[3], yy[3], a1);
            }
            cplx d = sh.M[i * LDM + i] - lq;
            if (abs2(d) < smallnum * smallnum) d = mkc(smallnum);
            if (i < q && lane < 32) Yq[i] = -div_fast(a0 + a1, d);
            wave_sync();
        }
        if (lane == 0) {
            sh.total = total;
            sh.failed = failed;
        }
    }
    __syncthreads();
    // ---- W = Z Y over T (8 columns at a time), and meanwhile the expansion
    // x = Y^-1 Z^* alpha_1 of the first snapshot's coefficients in the columns
    // of Z Y
    if (wave == 3) {
        const int q = lane & 31, hf = lane >> 5;
        cplx g = mkc(0.0);
        for (int i = 16 * hf; i < 16 * hf + 16; i += 4) {
            cplx zz[4], xx[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                zz[u] = conj(sh.M[q * LDM + 32 + i + u]);
                xx[u] = sh.al[i + u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) g = fmac(zz[u], xx[u], g);
        }
        g = other_half_sum(g);
        cplx yn = sh.Y[q + (k - 1) * LDH];
        for (int jj = k - 1; jj >= 1; --jj) {
            const cplx yc = yn;
            yn = sh.Y[q + (jj - 1) * LDH];
            const cplx xj = {lane_f64(g.re, jj), lane_f64(g.im, jj)};
            if (q < jj) g = g - yc * xj;
        }
        wave_sync();
        if (lane < 32) sh.x[q] = g;
    }
    __syncthreads();
    {
        const int i = tid & 31;
        cplx w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int q = (tid >> 5) + 8 * u;
            w[u] = mkc(0.0);
            if (q < k)
                for (int j0 = 0; j0 <= q; j0 += 4) {
                    cplx zz[4], yy[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        zz[e] = sh.M[(j0 + e) * LDM + 32 + i];
                        yy[e] = j0 + e <= q ? sh.Y[j0 + e + q * LDH] : mkc(0.0);
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) w[u] = fmac(zz[e], yy[e], w[u]);
                }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int q = (tid >> 5) + 8 * u;
            if (q < k) sh.M[q * LDM + i] = w[u];  // (rows 0 .. 31: T is no longer needed)
        }
    }
    __syncthreads();
    if (wave == 0 && !a.cplx) {
        // A real A~ has a spectrum closed under conjugation.  The two members
        // of a conjugate pair come with independent rounding; pair them up
        // and make the member with negative imaginary part the exact
        // conjugate of its partner (eigenvector and expansion too), and make
        // numerically real eigenvalues exactly real, so that the order of
        // eigenpairs does not depend on rounding.
        const double dl2 = 1e-20;
        const bool live = lane < k;
        const cplx lq = live ? sh.lam[lane] : mkc(0.0);
        const double cut = dl2 * abs2(lq), im2 = lq.im * lq.im;
        const bool neg = live && lq.im < 0.0 && im2 > cut, pos = live && lq.im > 0.0 && im2 > cut;
        const unsigned long long mpos = __ballot(pos), mneg = __ballot(neg);
        int partner = -1;
        double best = 1e300;
        for (int p = 0; p < k; ++p) {
            const cplx lp = sh.lam[p];
            const double d = sqr(lp.re - lq.re) + sqr(lp.im + lq.im);
            if (neg && ((mpos >> p) & 1) && d < best) {
                best = d;
                partner = p;
            }
        }
        // accept the pairing only if it is a bijection between the two halves
        bool ok = __popcll(mpos) == __popcll(mneg) && __ballot(neg && partner < 0) == 0;
        for (int p = 0; p < k; ++p) ok = ok && __popcll(__ballot(neg && partner == p)) <= 1;
        wave_sync();
        if (ok && live) {
            if (partner >= 0) {
                sh.lam[lane] = conj(sh.lam[partner]);
                sh.x[lane] = conj(sh.x[partner]);
                for (int i = 0; i < k; ++i) sh.M[lane * LDM + i] = conj(sh.M[partner * LDM + i]);
            } else if (!pos) {
                sh.lam[lane].im = 0.0;
            }
        }
        wave_sync();
    }
    __syncthreads();
    if (tid < k) {
        sh.mod[tid] = cabs(sh.lam[tid]);
        sh.arg[tid] = atan2(sh.lam[tid].im, sh.lam[tid].re);
    }
    __syncthreads();
    // ---- normalise column q (8 lanes): unit norm, largest-modulus entry
    // (lowest index on ties) real positive; rank by |lambda| descending, arg
    // ascending; b = x / (scale lambda), the mode amplitudes (W Lambda)^-1 alpha_1
    {
        const int q = tid >> 3, e = tid & 7;
        const bool live = q < k;
        cplx w[4];
        double nrm2 = 0.0, best = -1.0;
        int bi = 0, rank = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = e + 8 * u;
            w[u] = live && i < k ? sh.M[q * LDM + i] : mkc(0.0);
            const double v = abs2(w[u]);
            nrm2 += v;
            if (i < k && v > best) {
                best = v;
                bi = i;
            }
            const double mq = sh.mod[live ? q : 0], aq = sh.arg[live ? q : 0];
            if (i < k) {
                const double mp = sh.mod[i], ap = sh.arg[i];
                rank += (mp > mq) || (mp == mq && ap < aq) || (mp == mq && ap == aq && i < q);
            }
        }
        auto lvl = [&](auto ctrl) {
            constexpr int C = decltype(ctrl)::value;
            nrm2 += dpp_f64<C>(nrm2);
            rank += __builtin_amdgcn_mov_dpp(rank, C, 0xF, 0xF, true);
            const double ov = dpp_f64<C>(best);
            const int oi = __builtin_amdgcn_mov_dpp(bi, C, 0xF, 0xF, true);
            if (ov > best || (ov == best && oi < bi)) {
                best = ov;
                bi = oi;
            }
        };
        lvl(std::integral_constant<int, 0xB1>{});
        lvl(std::integral_constant<int, 0x4E>{});
        lvl(std::integral_constant<int, 0x141>{});
        if (live) {
            const cplx piv = sh.M[q * LDM + bi];
            const double ap = cabs(piv);
            const cplx ph = ap > 0.0 ? cplx{piv.re / ap, -piv.im / ap} : mkc(1.0);
            const cplx scale_q = (nrm2 > 0.0 ? 1.0 / sqrt(nrm2) : 1.0) * ph;
            const cplx lq = sh.lam[q];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = e + 8 * u;
                if (i < k) {
                    const cplx x = w[u] * scale_q;
                    sh.Y[i + rank * LDH] = x;  // sorted, canonical W
                    a.W[2 * (i + (int64_t)rank * k)] = x.re;
                    a.W[2 * (i + (int64_t)rank * k) + 1] = x.im;
                }
            }
            if (e == 0) {
                sh.ls[rank] = lq;
                a.lam[2 * rank] = lq.re;
                a.lam[2 * rank + 1] = lq.im;
                sh.b[rank] = cdiv(sh.x[q], scale_q * lq);
            }
        }
    }
    __syncthreads();
    // ---- the background mode argmin |log lambda| (Algorithm 3; lowest index
    // on ties, over lambda != 0; mode 0 if none) and its factor b_i lambda_i^m
    // for the newest snapshot
    if (wave == 0) {
        bool ok = false;
        double d = 0.0;
        if (lane < k) {
            const cplx lq = sh.ls[lane];
            const double mod = cabs(lq);
            if (mod > 0.0) {
                ok = true;
                d = hypot(log(mod), atan2(lq.im, lq.re));
            }
        }
        int bi = lane;
        for (int off = 32; off >= 1; off >>= 1) {
            const bool ook = __shfl_xor((int)ok, off, 64) != 0;
            const double od = __shfl_xor(d, off, 64);
            const int oi = __shfl_xor(bi, off, 64);
            const bool take = ook && (!ok || od < d || (od == d && oi < bi));
            if (take) {
                ok = true;
                d = od;
                bi = oi;
            }
        }
        bi = ok ? bi : 0;
        if (lane == 0) {
            sh.bg = bi;
            st->bg_index = bi;
            // lambda^m = |lambda|^m e^{i m arg lambda}
            const cplx lb = sh.ls[bi];
            const double pm = pow(cabs(lb), (double)m), th = (double)m * atan2(lb.im, lb.re);
            sh.fbg = cplx{pm * cos(th), pm * sin(th)};
        }
    } else if (wave == 1) {
        check_amplitudes(sh, k);
    }
    __syncthreads();
    if (sh.redo) {
        solve_amplitudes(sh, k);
        __syncthreads();
    }
    if (tid < k) {
        a.amp[2 * tid] = sh.b[tid].re;
        a.amp[2 * tid + 1] = sh.b[tid].im;
    }
    // ---- C = V_r Sigma^-1 W (m x k complex), row-major with row stride 2 r
    if (a.cplx) coef_rows<cplx>(a, sh, m, k);
    else coef_rows<double>(a, sh, m, k);
    if (tid == 0) {
        st->qr_iters = sh.total;
        if (sh.failed) st->solve_status = ST_E_CONVERGENCE;
        st->solves += 1;
    }
    publish(a);
}

__global__ __launch_bounds__(kEigThreads, 2)
void k_solve_eig(SolveArgs a) {
    __shared__ EigShared sh;
    solve_eig_body(a, sh);
    if (a.snap_st) {
        // the snapshot of this solve (state and mode coefficients) for the
        // projections that may run beside the next push
        __syncthreads();
        const uint4* B = static_cast<const uint4*>(a.Bphi);
        uint4* out = static_cast<uint4*>(a.snap_B);
        for (int i = threadIdx.x; i < a.snap_n16; i += blockDim.x) out[i] = B[i];
        if (threadIdx.x == 0) *a.snap_st = *a.st;
    }
}

__global__ __launch_bounds__(kEigThreads, 2)
void k_solve_eig_grouped(const SolveArgs* __restrict__ items) {
    __shared__ EigShared sh;
    const SolveArgs a = items[blockIdx.x];
    solve_eig_body(a, sh);
}

// --------------------------------------------------------------------------
// k_solve_trid_wide: Hermitian windows of more than 128 columns (the others
// are solved in trid_solve.hip), by a method with O(m)
// dependent steps instead of O(m) per Jacobi sweep, for large windows:
//   1. Householder reduction of xtx to a real symmetric tridiagonal T
//      (Hermitian input: complex reflectors, T still real);
//   2. all eigenvalues of T by multisection: 256 / m lanes per eigenvalue
//      (m rounded up to a power of two) evaluate Sturm counts at equally
//      spaced points of its bracket;
//   3. eigenvectors of T for the r largest |eigenvalues| by twisted
//      factorizations (forward L D L^T and backward U D U^T of T - lambda I,
//      twist where |gamma_k| is smallest, then the two one-term recurrences),
//      re-orthogonalized where two eigenvalues nearly coincide;
//   4. back-transformation by the reflectors, one half-wavefront per vector.
// The result feeds the same tail as the Jacobi solve.
// --------------------------------------------------------------------------

// Eigenvalues of the tridiagonal (d, e2 = e^2), scaled so that every Gershgorin
// radius is at most 1, below x: sign changes of the leading principal minors
// p_k = (d_k - x) p_{k-1} - e_{k-1}^2 p_{k-2} (an exact zero counts as a sign
// change), rescaled by powers of two to stay in range.  |p_k| grows at most
// threefold per step, so the range is checked every fourth step.
__device__ __forceinline__ int sturm_count(const double* __restrict__ d, const double* __restrict__ e2, int n,
                                           double x) {
    double a = 1.0, b = d[0] - x;
    if (b == 0.0) b = -0x1p-900;
    int cnt = b < 0.0;
    auto step = [&](int k) {
        double c = fma(d[k] - x, b, -e2[k - 1] * a);
        if (c == 0.0) c = -copysign(0x1p-900, b);
        cnt += (int)(((unsigned long long)__double_as_longlong(c) ^ (unsigned long long)__double_as_longlong(b)) >> 63);
        a = b;
        b = c;
    };
    auto rescale = [&]() {
        const double ab = fabs(b);
        if (ab > 0x1p500 || ab < 0x1p-500) {
            const double sc = ab > 1.0 ? 0x1p-500 : 0x1p500;
            a *= sc;
            b *= sc;
        }
    };
    int k = 1;
    for (; k + 3 < n; k += 4) {
        step(k);
        step(k + 1);
        step(k + 2);
        step(k + 3);
        rescale();
    }
    for (; k < n; ++k) {
        step(k);
        rescale();
    }
    return cnt;
}

__device__ __forceinline__ cplx shfl_xor_c(cplx v, int off, int width) {
    return cplx{__shfl_xor(v.re, off, width), __shfl_xor(v.im, off, width)};
}

// Householder reflector of column j (one wavefront): H = I - tau v v^* maps
// x = A[j+1.., j] to (beta, 0, ..); v = (1, x[1..] / (alpha - beta)) is stored
// over x[1..] and into vbuf, with tau, beta = e_j and d_j = A[j][j].
__device__ void householder_col(cplx* A, int ld, int n, int j, cplx* vbuf, cplx* s_tau, double* s_e, double* s_d) {
    using S = cplx;
    using SC = Scal<S>;
    const int lane = threadIdx.x & 63;
    const int L = n - j - 1;
    S* col = A + (size_t)j * ld + (j + 1);
    double xn2 = 0.0;
    for (int i = 1 + lane; i < L; i += 64) {
        const double ax = SC::absv(col[i]);
        xn2 += ax * ax;
    }
    xn2 = wave_sum(xn2);
    const S alpha = col[0];
    const double ar = SC::re(alpha), aa = SC::absv(alpha);
    S tau = SC::zero(), scal = SC::zero();
    double beta = ar;
    if (!(xn2 == 0.0 && aa == ar)) {
        beta = -copysign(sqrt(aa * aa + xn2), ar);
        tau = (SC::fromc(mkc(beta)) - alpha) * (1.0 / beta);
        scal = cdiv(SC::one(), alpha - SC::fromc(mkc(beta)));
    }
    for (int i = 1 + lane; i < L; i += 64) {
        const S v = mulr(col[i], scal);
        col[i] = v;
        vbuf[i] = v;
    }
    if (lane == 0) {
        vbuf[0] = SC::one();
        s_tau[j] = tau;
        s_e[j] = beta;
        s_d[j] = SC::re(A[j + (size_t)j * ld]);
    }
}

__device__ void solve_trid_body(const SolveArgs& a) {
    using S = cplx;
    constexpr int NT = 1024;
    using SC = Scal<S>;
    extern __shared__ double dyn[];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    const int slots = a.slots;
    DevState* st = a.st;
    const int m = window_cols(a.m, a.buildup, st), n = m;  // fewer columns during a build-up start
    if (m == 0) {
        if (tid == 0) {
            st->solve_status = ST_E_NOT_READY;
            st->r_eff = 0;
        }
        return;
    }
    if (st->vprev_valid && st->pushes == st->vprev_push) {
        if (tid == 0) st->skipped = 1;
        return;
    }
    const int oldest = st->oldest;
    const int ld = n + 1;
    const int nv = a.r < n ? a.r : n;  // eigenvectors computed: the r largest |eigenvalues|

    __shared__ double s_d[kMaxM], s_e[kMaxM], s_e2[kMaxM], s_lam[kMaxM];
    __shared__ S s_tau[kMaxM], s_v0[kMaxM], s_v1[kMaxM], s_p[kMaxM];
    __shared__ double s_sig[kMaxM];
    __shared__ int s_perm[kMaxM], s_sel[kRMax], s_tw[kRMax];
    __shared__ double s_zsc[kRMax];
    __shared__ double s_scale;

    // storage: A (n x ld) in the workspace; the multipliers of the twisted
    // factorizations (2 n nv doubles) in LDS,
    // later the eigenvectors during the back-transformation; Z (n x nv) and
    // the tail's scratch after A in the workspace
    S* A = reinterpret_cast<S*>(a.work);
    double* LU = dyn;
    S* Z = reinterpret_cast<S*>(a.work) + (size_t)n * ld;
    S* spare1 = Z + (size_t)n * ld;
    S* spare2 = spare1 + (size_t)n * ld;

    for (int idx = tid; idx < n * n; idx += NT) {
        const int i = idx % n, j = idx / n;
        A[i + (size_t)j * ld] = gram_at<S>(a.G, slot_of(oldest, i, slots), slot_of(oldest, j, slots), slots);
    }
    __syncthreads();

    // ---- 1. Householder tridiagonalization: T = Q^* xtx Q, Q = H_0 ... H_{n-2},
    // H_j = I - tau_j v_j v_j^*, v_j = (1, A[j+2.., j]) acting on rows j+1..
    // Per column: p = tau A22 v, then A22 -= v w^* + w v^* with w = p + c v,
    // c = -tau (p^* v) / 2.  Wavefront 0 updates the next column first and
    // builds its reflector while the others update the rest (two barriers
    // per column).  Row j+1 of A22 is never used again and is not updated.
    if (wv == 0) householder_col(A, ld, n, 0, s_v0, s_tau, s_e, s_d);
    __syncthreads();
    for (int j = 0; j + 1 < n; ++j) {
        const int L = n - j - 1;
        const S* v = (j & 1) ? s_v1 : s_v0;
        S* vnext = (j & 1) ? s_v0 : s_v1;
        const S tau = s_tau[j];
        S* A22 = A + (size_t)(j + 1) * ld + (j + 1);
        {
            int G = 64;
            while (G > 1 && G * L > NT) G >>= 1;
            const int gi = tid / G, gl = tid % G;
            for (int i = gi; i < L; i += NT / G) {
                const S* ci = A22 + (size_t)i * ld;
                S acc = ordered_dot<kAhead<S, false>>(SC::zero(), gl, G, L, [&](int k) { return SC::cj(ci[k]); },
                                       [&](int k) { return v[k]; });
                acc = group_sum(acc, G);
                if (gl == 0) s_p[i] = mulr(tau, acc);
            }
        }
        __syncthreads();
        S pv = SC::zero();
        for (int k = lane; k < L; k += 64) pv = pv + mulr(SC::cj(s_p[k]), v[k]);
        pv = group_sum(pv, 64);
        const S c = mulr(tau, pv) * (-0.5);
        if (wv == 0) {
            const S v0 = v[0], w0 = s_p[0] + mulr(c, v0);
            for (int k = lane; k < L; k += 64) {
                const S vk = v[k], wk = s_p[k] + mulr(c, vk);
                A22[k] = A22[k] - (mulr(vk, SC::cj(w0)) + mulr(wk, SC::cj(v0)));
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (j + 2 < n) householder_col(A, ld, n, j + 1, vnext, s_tau, s_e, s_d);
        } else {
            // every element is read before the chunk's writes (no two
            // iterations touch the same element), so that the reads of a
            // chunk overlap instead of waiting behind the previous write
            const int L1 = L - 1, NW = NT - 64;
            auto upd = [&](int idx, S a) {
                const int k = 1 + idx % L1, i = 1 + idx / L1;
                const S vk = v[k], vi = v[i];
                const S wk = s_p[k] + mulr(c, vk), wi = s_p[i] + mulr(c, vi);
                return a - (mulr(vk, SC::cj(wi)) + mulr(wk, SC::cj(vi)));
            };
            auto at = [&](int idx) -> S& { return A22[(1 + idx % L1) + (size_t)(1 + idx / L1) * ld]; };
            constexpr int U = 4;
            int idx = tid - 64;
            for (; idx + (U - 1) * NW < L1 * L1; idx += U * NW) {
                S x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) x[u] = at(idx + u * NW);
#pragma unroll
                for (int u = 0; u < U; ++u) at(idx + u * NW) = upd(idx + u * NW, x[u]);
            }
            for (; idx < L1 * L1; idx += NW) at(idx) = upd(idx, at(idx));
        }
        __syncthreads();
    }
    if (tid == 0) {
        s_d[n - 1] = SC::re(A[(n - 1) + (size_t)(n - 1) * ld]);
        s_e[n - 1] = 0.0;
        double g = 0.0;
        for (int i = 0; i < n; ++i) {
            const double r = fabs(s_d[i]) + (i > 0 ? fabs(s_e[i - 1]) : 0.0) + fabs(s_e[i]);
            g = r > g ? r : g;
        }
        s_scale = g;
    }
    __syncthreads();
    const double scale = s_scale;
    const double inv = scale > 0.0 ? 1.0 / scale : 0.0;
    for (int i = tid; i < n; i += NT) {
        s_d[i] *= inv;
        s_e[i] *= inv;
        s_e2[i] = s_e[i] * s_e[i];
    }
    __syncthreads();

    // ---- 2. eigenvalues: G lanes per eigenvalue, bracket [-1, 1] split into
    // G+1 parts per iteration until its width is at most eps (absolute,
    // ||T|| <= 1).  The Sturm counts are FP64 work on one CU, so about 256
    // lanes (G = 256 / m) finish first: more lanes per eigenvalue save
    // iterations but cost more in total than they save.
    {
        int np2 = 1;
        while (np2 < n) np2 <<= 1;
        int G = 256 / np2;
        G = G > 64 ? 64 : (G < 1 ? 1 : G);
        const int gi = tid / G, gl = tid % G;
        const int gshift = (tid & 63) / G * G;  // first lane of the group inside the wavefront
        int iters = 1;
        {
            double w = 2.0;
            while (w > kEps) {
                w /= (double)(G + 1);
                ++iters;
            }
        }
        double lo = -1.0 - 4.0 * kEps, hi = 1.0 + 4.0 * kEps;
        if (64 * wv < G * n)  // wavefronts with no eigenvalue skip the search
        for (int it = 0; it < iters; ++it) {
            const double x = lo + (hi - lo) * (double)(gl + 1) / (double)(G + 1);
            const bool above = gi < n ? sturm_count(s_d, s_e2, n, x) > gi : true;
            const uint64_t mask = __ballot(above);
            const uint64_t grp = (G == 64) ? mask : ((mask >> gshift) & ((1ull << G) - 1));
            if (grp == 0) {
                lo = lo + (hi - lo) * (double)G / (double)(G + 1);
            } else {
                const int f = __builtin_ctzll(grp);  // first point above the eigenvalue
                const double nlo = f == 0 ? lo : lo + (hi - lo) * (double)f / (double)(G + 1);
                hi = lo + (hi - lo) * (double)(f + 1) / (double)(G + 1);
                lo = nlo;
            }
        }
        if (gi < n && gl == 0) s_lam[gi] = 0.5 * (lo + hi);
    }
    __syncthreads();

    // order by |lambda| descending (ties: larger lambda first); sigma = sqrt(|lambda|)
    for (int i = tid; i < n; i += NT) {
        const double li = s_lam[i], ai = fabs(li);
        int rank = 0;
        for (int j2 = 0; j2 < n; ++j2) {
            const double aj = fabs(s_lam[j2]);
            rank += (aj > ai) || (aj == ai && j2 > i);
        }
        s_perm[rank] = i;
        s_sig[rank] = sqrt(ai * scale);
        if (rank < nv) s_sel[rank] = i;
    }
    __syncthreads();

    // ---- 3. eigenvectors of T by twisted factorizations.  The forward
    // L D L^T (wavefront 0, lane v) and backward U D U^T (wavefront 1, lane v)
    // factorizations of T - lambda_v I run side by side; the twist index
    // (argmin |gamma_k|, lowest k on ties) is a wavefront reduction; the two
    // one-term recurrences from the twist run side by side again; the norm is
    // summed in the order of a single serial pass (up, then down), so the
    // vectors do not depend on how the work is split.
    double* Lm = LU;                   // Lm[i * nv + v], i < n-1
    double* Um = LU + (size_t)n * nv;  // Um[i * nv + v], 1 <= i < n
    const double tiny = 0x1p-900;
    if (tid < nv) {
        const int v = tid;
        const double lam = s_lam[s_sel[v]];
        double Dp = s_d[0] - lam;
        for (int i = 0; i + 1 < n; ++i) {
            if (Dp == 0.0) Dp = tiny;
            const double l = s_e[i] * rcp_fast(Dp);
            Lm[(size_t)i * nv + v] = l;
            Dp = s_d[i + 1] - lam - l * s_e[i];
        }
    } else if (tid >= 64 && tid < 64 + nv) {
        const int v = tid - 64;
        const double lam = s_lam[s_sel[v]];
        double Dm = s_d[n - 1] - lam;
        for (int i = n - 1; i >= 1; --i) {
            if (Dm == 0.0) Dm = tiny;
            const double u = s_e[i - 1] * rcp_fast(Dm);
            Um[(size_t)i * nv + v] = u;
            Dm = s_d[i - 1] - lam - u * s_e[i - 1];
        }
    }
    __syncthreads();
    // twist index: argmin |gamma_k|, gamma_k = (d_k - lam) - L_{k-1} e_{k-1} - U_{k+1} e_k
    for (int v = wv; v < nv; v += NT / 64) {
        const double lam = s_lam[s_sel[v]];
        double best = 1e308;
        int tw = 0;
        for (int k = lane; k < n; k += 64) {
            double g = s_d[k] - lam;
            if (k > 0) g -= Lm[(size_t)(k - 1) * nv + v] * s_e[k - 1];
            if (k + 1 < n) g -= Um[(size_t)(k + 1) * nv + v] * s_e[k];
            if (fabs(g) < best) {
                best = fabs(g);
                tw = k;
            }
        }
        for (int off = 32; off >= 1; off >>= 1) {
            const double ob = __shfl_xor(best, off, 64);
            const int ot = __shfl_xor(tw, off, 64);
            if (ob < best || (ob == best && ot < tw)) {
                best = ob;
                tw = ot;
            }
        }
        if (lane == 0) s_tw[v] = tw;
    }
    __syncthreads();
    // z_tw = 1, z_i = -L_i z_{i+1} (i < tw; wavefront 0), z_{i+1} = -U_{i+1} z_i (i >= tw; wavefront 1)
    if (tid < nv) {
        const int v = tid, tw = s_tw[v];
        S* zc = Z + (size_t)v * ld;
        double z = 1.0;
        zc[tw] = SC::one();
        for (int i = tw - 1; i >= 0; --i) {
            z = -Lm[(size_t)i * nv + v] * z;
            zc[i] = SC::fromc(mkc(z));
        }
    } else if (tid >= 64 && tid < 64 + nv) {
        const int v = tid - 64, tw = s_tw[v];
        S* zc = Z + (size_t)v * ld;
        double z = 1.0;
        for (int i = tw; i + 1 < n; ++i) {
            z = -Um[(size_t)(i + 1) * nv + v] * z;
            zc[i + 1] = SC::fromc(mkc(z));
        }
    }
    __syncthreads();
    if (tid < nv) {
        const int v = tid, tw = s_tw[v];
        const S* zc = Z + (size_t)v * ld;
        double nrm2 = 1.0;
        for (int i = tw - 1; i >= 0; --i) {
            const double z = SC::re(zc[i]);
            nrm2 += z * z;
        }
        for (int i = tw; i + 1 < n; ++i) {
            const double z = SC::re(zc[i + 1]);
            nrm2 += z * z;
        }
        s_zsc[v] = rsqrt_acc(nrm2);
    }
    __syncthreads();
    for (int idx = tid; idx < n * nv; idx += NT) {
        const int i = idx % n, v = idx / n;
        S* zc = Z + (size_t)v * ld;
        zc[i] = zc[i] * s_zsc[v];
    }
    __syncthreads();
    // the eigenvectors move into LDS (over the multipliers) for the rest of the work
    S* Zs = reinterpret_cast<S*>(LU);  // Zs[i + v n]
    for (int idx = tid; idx < n * nv; idx += NT) {
        const int i = idx % n, v = idx / n;
        Zs[i + (size_t)v * n] = Z[i + (size_t)v * ld];
    }
    __syncthreads();
    // nearly coincident eigenvalues: Gram-Schmidt in selection order (one wavefront)
    if (wv == 0) {
        for (int q = 1; q < nv; ++q) {
            for (int p = 0; p < q; ++p) {
                if (fabs(s_lam[s_sel[q]] - s_lam[s_sel[p]]) > 1e-8) continue;
                S* zq = Zs + (size_t)q * n;
                const S* zp = Zs + (size_t)p * n;
                double dot = 0.0;
                for (int i = lane; i < n; i += 64) dot += SC::re(zp[i]) * SC::re(zq[i]);
                dot = wave_sum(dot);
                double nn = 0.0;
                for (int i = lane; i < n; i += 64) {
                    const double zi = SC::re(zq[i]) - dot * SC::re(zp[i]);
                    zq[i] = SC::fromc(mkc(zi));
                    nn += zi * zi;
                }
                nn = wave_sum(nn);
                const double sc = nn > 0.0 ? rsqrt_acc(nn) : 0.0;
                for (int i = lane; i < n; i += 64) zq[i] = zq[i] * sc;
            }
        }
    }
    __syncthreads();

    // ---- 4. back-transformation Z <- H_0 ... H_{n-2} Z, one half-wavefront per
    // vector (columns are independent: no barrier between reflectors)
    {
        const int hw = tid >> 5, hl = tid & 31;
        for (int v = hw; v < nv; v += NT / 32) {
            S* zc = Zs + (size_t)v * n;
            for (int j = n - 2; j >= 0; --j) {
                const S tau = s_tau[j];
                const int L = n - j - 1;
                const S* vj = A + (size_t)j * ld + (j + 1);  // v_0 = 1 is implicit
                S w = SC::zero();
                for (int i = hl; i < L; i += 32) {
                    const S vi = i == 0 ? SC::one() : vj[i];
                    w = w + mulr(SC::cj(vi), zc[j + 1 + i]);
                }
                for (int off = 16; off >= 1; off >>= 1) w = w + shfl_xor_c(w, off, 32);
                const S f = mulr(tau, w);
                for (int i = hl; i < L; i += 32) {
                    const S vi = i == 0 ? SC::one() : vj[i];
                    zc[j + 1 + i] = zc[j + 1 + i] - mulr(vi, f);
                }
            }
        }
    }
    __syncthreads();
    for (int idx = tid; idx < n * nv; idx += NT) {
        const int i = idx % n, v = idx / n;
        Z[i + (size_t)v * ld] = Zs[i + (size_t)v * n];
    }
    // eigenvector index k of the tail = selection rank k (columns of Z)
    for (int i = tid; i < n; i += NT) s_perm[i] = i;
    __syncthreads();
    sym_tail<S, NT, kAhead<S, false>>(a, ld, Z, spare1, spare2, s_sig, s_perm, nv, 0, true, 0);
}

__global__ __launch_bounds__(1024)
void k_solve_trid_wide(SolveArgs a) {
    solve_trid_body(a);
}
__global__ __launch_bounds__(1024)
void k_solve_trid_wide_grouped(const SolveArgs* __restrict__ items) {
    const SolveArgs a = items[blockIdx.x];
    solve_trid_body(a);
}

}  // namespace

hipError_t launch_solve_sym(const SolveArgs& a, hipStream_t s) {
    if (a.r > kRMax || a.m > kMaxM) return hipErrorInvalidValue;
    const int M = a.m + (a.m & 1);
    if (!a.cplx && M <= 64) {
        const size_t lds = 3 * sizeof(double) * (size_t)M * (M + 1);
        auto kern = k_solve_sym<double, 1024, true, 32>;
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3(1), dim3(1024), lds, s, a, M);
    } else if (!a.cplx) {
        hipLaunchKernelGGL((k_solve_sym<double, 1024, false, kMaxM / 2>), dim3(1), dim3(1024), 0, s, a, M);
    } else {
        hipLaunchKernelGGL((k_solve_sym<cplx, 1024, false, kMaxM / 2>), dim3(1), dim3(1024), 0, s, a, M);
    }
    return hipGetLastError();
}

// Hermitian windows of more than 128 columns: one window by value, or n items.
hipError_t launch_solve_trid_wide(const SolveArgs* one, const SolveArgs* items, int n, hipStream_t s) {
    const size_t lds = sizeof(double) * 2 * kMaxM * kRMax;
    const void* kern = one ? reinterpret_cast<const void*>(k_solve_trid_wide)
                           : reinterpret_cast<const void*>(k_solve_trid_wide_grouped);
    hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    if (one) hipLaunchKernelGGL(k_solve_trid_wide, dim3(1), dim3(1024), lds, s, *one);
    else hipLaunchKernelGGL(k_solve_trid_wide_grouped, dim3(n), dim3(1024), lds, s, items);
    return hipGetLastError();
}

hipError_t launch_solve_eig(const SolveArgs& a, hipStream_t s) {
    if (a.r > kRMax) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_solve_eig, dim3(1), dim3(kEigThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace dmd

namespace dmd {

hipError_t launch_eig_grouped(const SolveArgs* items, int n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_solve_eig_grouped, dim3(n), dim3(kEigThreads), 0, s, items);
    return hipGetLastError();
}

hipError_t launch_jacobi_grouped(const SolveArgs* items_lds, int n_lds, const SolveArgs* items_glb, int n_glb,
                                 hipStream_t s) {
    if (n_lds > 0) {
        const size_t lds = 3 * sizeof(double) * 64 * 65;  // sized for M <= 64
        auto kern = k_solve_sym_grouped<double, 1024, true, 32>;
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3(n_lds), dim3(1024), lds, s, items_lds);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (n_glb > 0) {
        hipLaunchKernelGGL((k_solve_sym_grouped<double, 1024, false, kMaxM / 2>), dim3(n_glb), dim3(1024), 0, s,
                           items_glb);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}


}  // namespace dmd
