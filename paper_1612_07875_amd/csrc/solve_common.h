// Device helpers shared by the small solves (symmetric eigenproblems and the
// eigenproblem of A~): FP64 reciprocals, lane exchanges and reductions, and
// access to the Gram.
#pragma once
#include <cfloat>

#include "cplx.h"
#include "dmd_internal.h"

namespace dmd {
namespace {

constexpr int kRMax = 32;         // largest truncation rank handled by k_solve_eig
constexpr double kEps = DBL_EPSILON;

// acc + sum of fa(k) * fb(k) over k = k0, k0 + step, ... < L, added in that
// order.  The operands of U consecutive terms are read before their
// products, so that their memory latencies overlap: a loop that reads,
// waits and multiplies one term at a time pays a full round trip per term,
// which the workspace forms of the solves (matrix and coefficients in
// global memory) cannot afford.  The sum is the plain loop's, bit for bit.
// U = 1 is the plain loop (the LDS forms: their register count decides
// whether a solve fits beside a running projection).
template <int U, typename S, typename FA, typename FB>
__device__ __forceinline__ S ordered_dot(S acc, int k0, int step, int L, FA fa, FB fb) {
    int k = k0;
    if constexpr (U > 1) {
        for (; k + (U - 1) * step < L; k += U * step) {
            S x[U], y[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                x[u] = fa(k + u * step);
                y[u] = fb(k + u * step);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) acc = acc + mulr(x[u], y[u]);
        }
    }
    for (; k < L; k += step) acc = acc + mulr(fa(k), fb(k));
    return acc;
}
// terms read ahead by the workspace forms: 8 real or 4 complex values
template <typename S, bool LDS> constexpr int kAhead = LDS ? 1 : (sizeof(S) == sizeof(double) ? 8 : 4);

template <typename S> __device__ __forceinline__ S gram_at(const double* G, int a, int b, int slots);
template <> __device__ __forceinline__ double gram_at<double>(const double* G, int a, int b, int slots) {
    return G[a + (int64_t)b * slots];
}
template <> __device__ __forceinline__ cplx gram_at<cplx>(const double* G, int a, int b, int slots) {
    const double* p = G + 2 * (a + (int64_t)b * slots);
    return cplx{p[0], p[1]};
}

template <typename S> __device__ __forceinline__ void store_s(double* out, int64_t i, S v);
template <> __device__ __forceinline__ void store_s<double>(double* out, int64_t i, double v) { out[i] = v; }
template <> __device__ __forceinline__ void store_s<cplx>(double* out, int64_t i, cplx v) {
    out[2 * i] = v.re;
    out[2 * i + 1] = v.im;
}

// 1/sqrt(x) to full FP64 accuracy: hardware estimate plus two Newton steps
// (the estimate carries ~23 correct bits).  A dependent FP64 operation takes 6
// cycles and any instruction about 4 of its wavefront's issue, so this replaces
// the longer correctly rounded sqrt/division sequences on the latency-bound
// paths.
__device__ __forceinline__ double rsqrt_acc(double x) {
    double y = __builtin_amdgcn_rsq(x);
    const double h = 0.5 * x;
    double e = fma(-h * y, y, 0.5);
    y = fma(y, e, y);
    e = fma(-h * y, y, 0.5);
    return fma(y, e, y);
}
// 1/x to ~46 bits (estimate plus one Newton step).
__device__ __forceinline__ double rcp_fast(double x) {
    const double y = __builtin_amdgcn_rcp(x);
    return fma(y, fma(-x, y, 1.0), y);
}
// 1/x to full FP64 accuracy (estimate plus two Newton steps).
__device__ __forceinline__ double rcp_acc(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = fma(y, fma(-x, y, 1.0), y);
    return fma(y, fma(-x, y, 1.0), y);
}

// A double from another lane of the same 16-lane row, by a DPP lane pattern
// (a register move, no trip through the LDS crossbar as __shfl_xor takes).
template <int CTRL> __device__ __forceinline__ double dpp_f64(double x) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    // (every pattern used reads a lane of its row, so there is no old value to keep)
    const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)(b & 0xffffffffull), CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
// op(x of this lane, x of the lane OFF = 16 or 32 away) for a commutative op,
// by a swap of 16-lane rows (32-lane halves) between two copies of x: after
// it one copy holds the even row's values in both rows of a pair and the
// other the odd row's.  Register moves of about 10 cycles, where __shfl_xor
// takes a trip through the LDS crossbar (83 cycles measured, 123 with 16
// wavefronts on the CU).
template <int OFF, typename OP> __device__ __forceinline__ double row_fold(double x, OP op) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const unsigned lo = (unsigned)(b & 0xffffffffull), hi = (unsigned)(b >> 32);
    auto join = [](unsigned l, unsigned h) {
        return __builtin_bit_cast(double, ((unsigned long long)h << 32) | l);
    };
    if constexpr (OFF == 16) {
        const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        return op(join(l[0], h[0]), join(l[1], h[1]));
    } else {
        const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        return op(join(l[0], h[0]), join(l[1], h[1]));
    }
}
// Sum over each aligned group of G lanes (G = 1, 2, 4, .., 64; every lane of
// the group active), the same value in every lane of the group: neighbour
// pairs, then pairs of pairs (quad permutations 1,0,3,2 and 2,3,0,1); then
// the mirror of each 8-lane half-row and of each 16-lane row, which read a
// lane of the other half whose partial sum equals its own by then; then the
// 16- and 32-lane halves by row swaps.  Each step adds a value to its
// partner's in either order, so all lanes end bitwise equal.
__device__ __forceinline__ double group_sum(double x, int G) {
    if (G >= 2) x += dpp_f64<0xB1>(x);
    if (G >= 4) x += dpp_f64<0x4E>(x);
    if (G >= 8) x += dpp_f64<0x141>(x);
    if (G >= 16) x += dpp_f64<0x140>(x);
    if (G >= 32) x = row_fold<16>(x, [](double a, double b) { return a + b; });
    if (G >= 64) x = row_fold<32>(x, [](double a, double b) { return a + b; });
    return x;
}
__device__ __forceinline__ cplx group_sum(cplx x, int G) { return cplx{group_sum(x.re, G), group_sum(x.im, G)}; }
__device__ __forceinline__ double wave_sum(double x) { return group_sum(x, 64); }
__device__ __forceinline__ double wave_max(double x) {
    x = fmax(x, dpp_f64<0xB1>(x));
    x = fmax(x, dpp_f64<0x4E>(x));
    x = fmax(x, dpp_f64<0x141>(x));
    x = fmax(x, dpp_f64<0x140>(x));
    x = row_fold<16>(x, [](double a, double b) { return fmax(a, b); });
    return row_fold<32>(x, [](double a, double b) { return fmax(a, b); });
}
// Ordering of LDS accesses among the lanes of one wavefront: LDS executes a
// wavefront's instructions in issue order, so a compiler-level fence at
// wavefront scope is all that a one-wavefront workgroup needs between a
// write and another lane's read (no wait for outstanding LDS work).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
// x of lane src (src the same in every lane), read from the register file.
__device__ __forceinline__ double lane_f64(double x, int src) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const int lo = __builtin_amdgcn_readlane((int)(unsigned)(b & 0xffffffffull), src);
    const int hi = __builtin_amdgcn_readlane((int)(unsigned)(b >> 32), src);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

}  // namespace
}  // namespace dmd
