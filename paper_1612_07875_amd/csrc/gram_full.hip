// Whole Gram of a window, G = X^* X for its k <= m+1 columns (Algorithm 1's
// first step; Sec. 2.1 step 1), on the matrix cores.
//
// The result is cut into 16 x 16 tiles; only tiles on or above the diagonal
// are computed (G is symmetric) and mirrored.  The n rows are split into
// `nsplit` ranges and the tiles into groups: a workgroup of 8 wavefronts takes
// one group of at most 32 tiles over one range, tile w + 8 u in wavefront w,
// so that the four SIMDs get equal shares to within a tile.
// It stages the group's columns, 64 (FP32 data) or 32 (FP64 data) rows at a
// time, in one of two LDS buffers (16-byte loads into registers during the
// previous stage's products); each range's tiles are summed in FP64 in a fixed
// order by a second kernel, which also writes the Gram (physical slot
// indexing) and the window state.
//
// What bounds it: the staging.  A group loads its columns from the fabric at
// 2.5 to 3 TB/s over the chip whatever the size (strips of 256 bytes per
// column), so a tile's operands are to be used by many tiles; the products of
// a stage run while the next one is loaded.  The matrix cores take 1.1 ms of
// the 1.6 to 1.8 at n = 2^20, k = 257 in FP64 (64 x 64 tiles with a tile pair's
// columns per workgroup: 2.6 ms and 0.2 for the sum of the row ranges, in 15
// workgroups), 0.11 of 0.24 ms at n = 2,073,600, k = 65 in FP32 (0.53 + 0.56).
// Groups of consecutive tiles, which stage nearly all columns each, took 2.7 ms
// at k = 257; loads under a branch, which the compiler moves behind the
// products, 2.2 ms.
//
// Precision of the products and of the in-tile accumulation:
//   FP64    v_mfma_f64_16x16x4f64, data widened exactly to FP64;
//   FP32    v_mfma_f32_16x16x4f32, FP32 accumulation;
//   BF16X3  v_mfma_f32_16x16x32_bf16 on x = hi + lo (hi = bf16(x),
//           lo = bf16(x - hi)): hi*hi + hi*lo + lo*hi, FP32 accumulation.
// FP32 and BF16X3 sums depend on how the rows are split and ordered: the
// ranges come from gram_full_splits (by the window length alone) and rows are
// taken in order, whatever the groups.  FP64 ranges follow the shape.
//
// Fragment layouts (checked on the device): 16x16x4 A[l%16][l/16],
// B[l/16][l%16]; 16x16x32 A[l%16][8(l/16)+e], B[8(l/16)+e][l%16];
// D f32 [4(l/16)+v][l%16], D f64 [(l/16)+4v][l%16].
#include <type_traits>

#include "dmd_internal.h"

namespace dmd {
namespace {

constexpr int kThreads = 256;      // copies
constexpr int kTileThreads = 512;
constexpr int kTileWaves = kTileThreads / 64;
constexpr int kMaxPerWave = 4;     // tiles of a wavefront
constexpr int kGroupTiles = kTileWaves * kMaxPerWave;

typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

enum Mode { MODE_F64 = 0, MODE_F32 = 1, MODE_BF16X3 = 2 };

template <int MODE> struct MAcc { using type = v4f; };
template <> struct MAcc<MODE_F64> { using type = v4d; };

constexpr int kMaxBlocks = (kMaxM + 1 + 15) / 16;                      // 17
constexpr int kMaxTiles = kMaxBlocks * (kMaxBlocks + 1) / 2;          // 153
constexpr int kMaxParts = 5, kMaxGroups = kMaxParts * (kMaxParts - 1) / 2;

// The tiles by group.  The column blocks are cut into parts, and a group stages
// two of them (one or two parts: everything): it computes the tiles between
// the two and a share of the tiles within each, so that all groups have about
// the same columns to load and the same tiles to compute.
struct GramPlan {
    int ngroup;
    uint8_t first[kMaxGroups + 1];             // tiles first[g] .. first[g+1] - 1 are group g's
    uint8_t ti[kMaxTiles], tj[kMaxTiles];      // column blocks, ti <= tj
    uint8_t a0[kMaxGroups], na[kMaxGroups], b0[kMaxGroups], nb[kMaxGroups];  // staged block ranges
};

struct GramFullArgs {
    const void* ring;
    int64_t ld, n;
    int m, slots, oldest_override;  // oldest_override >= 0: use it instead of the state's
    int kcols;                      // columns of the window (<= m+1)
    int nb, ntri;                   // 16-column blocks, tiles on or above the diagonal
    int nsplit;                     // row ranges
    int64_t rows_per_split;
    double* partial;                // [nsplit][ntri][256], a tile's 4 accumulator values lane by lane
    const DevState* st;
    int mode;
    GramPlan plan;
};

// Stage geometry: rows, and the column stride in LDS (four 4-byte banks more
// than the rows, so that the 16 columns of a fragment's 16-byte reads cover
// all banks).
template <typename TX> struct Stage {
    static constexpr int PER = 16 / sizeof(TX);  // elements per 16-byte load
    static constexpr int R = 16 * PER;           // rows
    static constexpr int LD = R + PER;           // elements per column
};

template <typename TX, int MODE, int NLD>
__global__ __launch_bounds__(kTileThreads)
void k_gram_tiles(GramFullArgs a) {
    constexpr int PER = Stage<TX>::PER, R = Stage<TX>::R, LD = Stage<TX>::LD;
    constexpr int TPC = R / PER;  // 16-byte loads per column and stage
    using AccT = typename MAcc<MODE>::type;
    using V = typename std::conditional<PER == 4, float4, double2>::type;
    // (one array, addressed by offsets: pointers kept in variables would turn
    // its accesses into flat ones)
    extern __shared__ double lds64[];
    TX* const lds = reinterpret_cast<TX*>(lds64);

    // Workgroup b goes to XCD b % 8 (dispatch order): consecutive tasks, the
    // groups of one row range, share an XCD and read their columns through
    // its L2.
    const int per = gridDim.x >> 3, task = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    const int ngroup = a.plan.ngroup;
    if (task >= a.nsplit * ngroup) return;
    const int split = task / ngroup, group = task % ngroup;
    const int t_begin = a.plan.first[group], t_end = a.plan.first[group + 1];
    const int ca = 16 * a.plan.a0[group], wa = 16 * a.plan.na[group];  // staged columns ca .. ca + wa - 1,
    const int cb = 16 * a.plan.b0[group], wb = 16 * a.plan.nb[group];  // then cb .. cb + wb - 1
    const int oldest = a.oldest_override >= 0 ? a.oldest_override : a.st->oldest;
    const int kcols = a.oldest_override >= 0 ? a.kcols : min(a.kcols, a.st->count);
    if (kcols <= 0) return;  // (no entry is written back)
    const TX* ring = reinterpret_cast<const TX*>(a.ring);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const int ncol = wa + wb;
    const int bufsz = ncol * LD;  // two buffers, then a spare column for the loads beyond the group's columns

    const int64_t r_begin = (int64_t)split * a.rows_per_split;
    const int64_t r_end = min(a.n, r_begin + a.rows_per_split);

    // this thread's loads of a stage: column t / TPC, rows q PER .. (columns
    // past the window read its last one: their products are not written back)
    const TX* src[NLD];
    int dst[NLD];
    bool inside[NLD];
#pragma unroll
    for (int u = 0; u < NLD; ++u) {
        const int t = threadIdx.x + u * kTileThreads, c = t / TPC, q = t % TPC;
        const int g = min(c < wa ? ca + c : cb + c - wa, kcols - 1);
        src[u] = ring + (int64_t)slot_of(oldest, g, a.slots) * a.ld + q * PER;
        // FP32 products take the rows in order, four k-steps of a lane side by
        // side: row r of 16 sits at 4 (r % 4) + r / 4
        dst[u] = (c < ncol ? c * LD : 2 * bufsz) + (MODE == MODE_F32 ? q / 4 * 16 + q % 4 : q * PER);
        inside[u] = c < ncol;
    }
    auto put = [&](int b, int u, V v) {
        TX* d = lds + (inside[u] ? b * bufsz : 0) + dst[u];
        if constexpr (MODE == MODE_F32) {
            d[0] = v.x;
            d[4] = v.y;
            d[8] = v.z;
            d[12] = v.w;
        } else {
            *reinterpret_cast<V*>(d) = v;
        }
    };

    // the wavefront's tiles: t_begin + wave + 8 u
    const int ntile = max(0, (t_end - t_begin - wave + kTileWaves - 1) / kTileWaves);
    int ao[kMaxPerWave], bo[kMaxPerWave];
#pragma unroll
    for (int u = 0; u < kMaxPerWave; ++u) {
        const int t = u < ntile ? t_begin + wave + kTileWaves * u : t_begin;
        auto at = [&](int blk) {  // the block's first staged column
            const int c = 16 * blk;
            return c >= ca && c < ca + wa ? c - ca : c - cb + wa;
        };
        ao[u] = (at(a.plan.ti[t]) + li) * LD;
        bo[u] = (at(a.plan.tj[t]) + li) * LD;
    }
    AccT acc[kMaxPerWave];
#pragma unroll
    for (int u = 0; u < kMaxPerWave; ++u) acc[u] = AccT{0, 0, 0, 0};

    auto products = [&](int b, auto nt) __attribute__((always_inline)) {
        const TX* L = lds + b * bufsz;
        constexpr int NT = decltype(nt)::value;
        if constexpr (NT == 0) {
            return;
        } else if constexpr (MODE == MODE_BF16X3) {
#pragma unroll
            for (int k0 = 0; k0 < R; k0 += 32)
#pragma unroll
                for (int u = 0; u < NT; ++u) {
                    v8bf ahi, alo, bhi, blo;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float x = (float)L[ao[u] + k0 + 8 * lk + e], y = (float)L[bo[u] + k0 + 8 * lk + e];
                        ahi[e] = (__bf16)x;
                        alo[e] = (__bf16)(x - (float)ahi[e]);
                        bhi[e] = (__bf16)y;
                        blo[e] = (__bf16)(y - (float)bhi[e]);
                    }
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(alo, bhi, acc[u], 0, 0, 0);
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, blo, acc[u], 0, 0, 0);
                    acc[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ahi, bhi, acc[u], 0, 0, 0);
                }
        } else {
            // a lane's 16 bytes hold its operands of PER k-steps (FP64: any
            // order of the rows will do, as long as both operands agree)
#pragma unroll
            for (int k0 = 0; k0 < R; k0 += 4 * PER) {
                V av[NT], bv[NT];
#pragma unroll
                for (int u = 0; u < NT; ++u) {
                    av[u] = *reinterpret_cast<const V*>(L + ao[u] + k0 + PER * lk);
                    bv[u] = *reinterpret_cast<const V*>(L + bo[u] + k0 + PER * lk);
                }
                auto mma = [&](auto get) {
#pragma unroll
                    for (int u = 0; u < NT; ++u) {
                        if constexpr (MODE == MODE_F64)
                            acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)get(av[u]), (double)get(bv[u]), acc[u], 0, 0, 0);
                        else
                            acc[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(get(av[u]), get(bv[u]), acc[u], 0, 0, 0);
                    }
                };
                mma([](const V& v) { return v.x; });
                mma([](const V& v) { return v.y; });
                if constexpr (PER == 4) {
                    mma([](const V& v) { return v.z; });
                    mma([](const V& v) { return v.w; });
                }
            }
        }
    };
    // full stages pipelined, the ragged last one after
    const int nfull = r_end > r_begin ? (int)((r_end - r_begin) / R) : 0;
    auto run = [&](auto nt) __attribute__((always_inline)) {
        if (nfull > 0) {
#pragma unroll
            for (int u = 0; u < NLD; ++u)
                put(0, u, *reinterpret_cast<const V*>(src[u] + r_begin));
            __syncthreads();
        }
        for (int st = 0; st < nfull; ++st) {
            // (no branch around the loads, which would make the compiler wait
            // for them before the products: the last stage is loaded twice)
            const int64_t rn = r_begin + (int64_t)(st + 1 < nfull ? st + 1 : st) * R;
            V nx[NLD];
#pragma unroll
            for (int u = 0; u < NLD; ++u) nx[u] = *reinterpret_cast<const V*>(src[u] + rn);
            __builtin_amdgcn_sched_barrier(0);  // (the loads are issued before the products)
            products(st & 1, nt);
#pragma unroll
            for (int u = 0; u < NLD; ++u) put((st & 1) ^ 1, u, nx[u]);
            __syncthreads();
        }
        const int64_t r0 = r_begin + (int64_t)nfull * R;
        if (r0 < r_end) {
            const int L = nfull & 1;
#pragma unroll
            for (int u = 0; u < NLD; ++u) {
                const int q = (threadIdx.x + u * kTileThreads) % TPC;
                auto at = [&](int i) { return r0 + q * PER + i < r_end ? src[u][r0 + i] : TX(0); };
                if constexpr (PER == 4) put(L, u, V{at(0), at(1), at(2), at(3)});
                else put(L, u, V{at(0), at(1)});
            }
            __syncthreads();
            products(L, nt);
        }
    };
    switch (ntile) {  // (the same barriers in every case)
        case 4: run(std::integral_constant<int, 4>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 1: run(std::integral_constant<int, 1>{}); break;
        default: run(std::integral_constant<int, 0>{}); break;
    }

#pragma unroll
    for (int u = 0; u < kMaxPerWave; ++u) {
        if (u >= ntile) break;
        double* out = a.partial + ((int64_t)split * a.ntri + t_begin + wave + kTileWaves * u) * 256 + lane;
#pragma unroll
        for (int v = 0; v < 4; ++v) out[64 * v] = (double)acc[u][v];
    }
}

// Sum the row ranges' tiles in a fixed order and write G (both triangles): one
// workgroup per tile, its threads in four quarters of the ranges (a tile's sum
// is a chain of loads, bound by latency: with 3 workgroups of one chain per
// entry it took longer than the products).
// set_window = 1: the Gram came with a new window (slots 0 .. kcols-1), so the
// window state is set; 2: the Gram of the current window was recomputed.  In
// both cases the previous eigenvectors no longer describe the Gram.
__global__ __launch_bounds__(1024)
void k_gram_reduce(GramFullArgs a, double* __restrict__ G, DevState* __restrict__ st, int set_window) {
    __shared__ double part[3][256];
    const int tile = blockIdx.x, e = threadIdx.x & 255, quarter = threadIdx.x >> 8;
    const int ti = a.plan.ti[tile], tj = a.plan.tj[tile];
    const int oldest = a.oldest_override >= 0 ? a.oldest_override : st->oldest;
    const int kcols = a.oldest_override >= 0 ? a.kcols : min(a.kcols, st->count);
    const int lane = e & 63, v = e >> 6;
    const int i = 16 * ti + (a.mode == MODE_F64 ? (lane >> 4) + 4 * v : 4 * (lane >> 4) + v);
    const int j = 16 * tj + (lane & 15);
    const bool in = i < kcols && j < kcols && i <= j;
    const int each = (a.nsplit + 3) / 4, p0 = quarter * each, p1 = min(a.nsplit, p0 + each);
    double s = 0.0;
    if (in) {
        const double* p = a.partial + (int64_t)tile * 256 + e;
        const int64_t step = (int64_t)a.ntri * 256;
#pragma unroll 8
        for (int q = p0; q < p1; ++q) s += p[q * step];
    }
    if (quarter) part[quarter - 1][e] = s;
    __syncthreads();
    if (quarter == 0 && in) {
        s = ((s + part[0][e]) + part[1][e]) + part[2][e];
        const int si = slot_of(oldest, i, a.slots), sj = slot_of(oldest, j, a.slots);
        G[si + (int64_t)sj * a.slots] = s;
        G[sj + (int64_t)si * a.slots] = s;
    }
    if (set_window && tile == 0 && threadIdx.x == 0) {
        if (set_window == 1) {
            st->oldest = a.oldest_override;
            st->count = a.kcols;
        }
        st->pushes += 1;
        st->vprev_valid = 0;
    }
}

// Copy k columns of X (n x k, leading dimension ldx) into ring slots 0 .. k-1.
template <typename TX>
__global__ __launch_bounds__(kThreads)
void k_copy_columns(const TX* __restrict__ X, int64_t ldx, TX* __restrict__ ring, int64_t ld, int64_t n, int k) {
    const int c = blockIdx.y;
    if (c >= k) return;
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads)
        ring[(int64_t)c * ld + i] = X[(int64_t)c * ldx + i];
}

}  // namespace

// Sizing of the partial tiles (and the row ranges of the FP32 and BF16X3
// sums): 64 x 64 tiles of the window, times ranges.
int gram_full_tiles(int m) {
    const int t = (m + 1 + 63) / 64;
    return t * (t + 1) / 2;
}

int gram_full_splits(int m) {
    // about 512 (range, tile) pairs; a multiple of 8 where there are 8 or more
    const int ntri = gram_full_tiles(m);
    int s = (512 + ntri - 1) / ntri;
    s = s > 128 ? 128 : s;
    return s >= 8 ? s / 8 * 8 : (s < 1 ? 1 : s);
}

namespace {
// The plan of nb column blocks in P parts; false if a group would hold more
// tiles than a workgroup's wavefronts have accumulators for.
bool make_plan(int nb, int P, GramPlan* p) {
    *p = GramPlan{};
    int lo[kMaxParts + 1];
    for (int i = 0; i <= P; ++i) lo[i] = nb * i / P;
    struct Group { int I, J, n; uint8_t ti[kGroupTiles], tj[kGroupTiles]; } g[kMaxGroups];
    int ng = 0;
    if (P == 1) g[ng++] = Group{0, 0, 0, {}, {}};
    for (int i = 0; i < P; ++i)
        for (int j = i + 1; j < P; ++j) g[ng++] = Group{i, j, 0, {}, {}};
    auto add = [&](Group& q, int i, int j) {
        if (q.n == kGroupTiles) return false;
        q.ti[q.n] = (uint8_t)i;
        q.tj[q.n++] = (uint8_t)j;
        return true;
    };
    for (int q = 0; q < ng; ++q)
        if (g[q].I != g[q].J)
            for (int i = lo[g[q].I]; i < lo[g[q].I + 1]; ++i)
                for (int j = lo[g[q].J]; j < lo[g[q].J + 1]; ++j)
                    if (!add(g[q], i, j)) return false;
    for (int part = 0; part < P; ++part)
        for (int i = lo[part]; i < lo[part + 1]; ++i)
            for (int j = i; j < lo[part + 1]; ++j) {
                int best = -1;
                for (int q = 0; q < ng; ++q)
                    if ((g[q].I == part || g[q].J == part) && (best < 0 || g[q].n < g[best].n)) best = q;
                if (!add(g[best], i, j)) return false;
            }
    p->ngroup = ng;
    int at = 0;
    for (int q = 0; q < ng; ++q) {
        p->first[q] = (uint8_t)at;
        for (int t = 0; t < g[q].n; ++t) {
            p->ti[at] = g[q].ti[t];
            p->tj[at++] = g[q].tj[t];
        }
        p->a0[q] = (uint8_t)lo[g[q].I];
        p->na[q] = (uint8_t)(lo[g[q].I + 1] - lo[g[q].I]);
        p->b0[q] = (uint8_t)lo[g[q].J];
        p->nb[q] = (uint8_t)(g[q].I == g[q].J ? 0 : lo[g[q].J + 1] - lo[g[q].J]);
    }
    p->first[ng] = (uint8_t)at;
    return true;
}

template <typename TX, int MODE> hipError_t launch_tiles(const GramFullArgs& a, hipStream_t s) {
    const int grid = (a.nsplit * a.plan.ngroup + 7) / 8 * 8;
    int blocks = 0;  // staged by the widest group
    for (int g = 0; g < a.plan.ngroup; ++g)
        if (a.plan.na[g] + a.plan.nb[g] > blocks) blocks = a.plan.na[g] + a.plan.nb[g];
    const size_t lds = sizeof(TX) * Stage<TX>::LD * (2 * 16 * (size_t)blocks + 1);
    const int nld = (16 * blocks * (Stage<TX>::R / Stage<TX>::PER) + kTileThreads - 1) / kTileThreads;
    auto go = [&](auto kern) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3(grid), dim3(kTileThreads), lds, s, a);
        return hipGetLastError();
    };
    switch (nld) {
        case 1: return go(k_gram_tiles<TX, MODE, 1>);
        case 2: return go(k_gram_tiles<TX, MODE, 2>);
        case 3: return go(k_gram_tiles<TX, MODE, 3>);
        case 4: return go(k_gram_tiles<TX, MODE, 4>);
        default: return go(k_gram_tiles<TX, MODE, 5>);
    }
}
}  // namespace

hipError_t launch_gram_full(const void* ring, int64_t ld, int64_t n, int m, int slots, int elem_f64,
                            int precision, int kcols, int oldest_override, double* partial, double* G,
                            DevState* st, int set_window, hipStream_t s) {
    GramFullArgs a{};
    a.ring = ring;
    a.ld = ld;
    a.n = n;
    a.m = m;
    a.slots = slots;
    a.oldest_override = oldest_override;
    a.kcols = kcols;
    a.nb = (kcols + 15) / 16;
    a.ntri = a.nb * (a.nb + 1) / 2;
    a.partial = partial;
    a.st = st;
    // FP64 data always accumulates in FP64; FP32 data in the stream's precision
    a.mode = MODE_F32;
    if (elem_f64 || precision == 3 /*FP64*/) a.mode = MODE_F64;
    else if (precision == 2 /*BF16X3*/) a.mode = MODE_BF16X3;
    // parts: as few as the accumulators allow, and for the fixed row ranges
    // as many as make up 192 workgroups
    const int fixed = a.mode == MODE_F64 ? 0 : gram_full_splits(m);
    bool ok = false;
    for (int P = 1; P <= kMaxParts && P <= a.nb; ++P) {
        if (P == 2) continue;  // (two parts are one group)
        GramPlan p;
        if (!make_plan(a.nb, P, &p)) continue;
        a.plan = p;
        ok = true;
        if (!fixed || fixed * p.ngroup >= 192) break;
    }
    if (!ok) return hipErrorInvalidValue;
    if (a.mode == MODE_F64) {
        // as many ranges as fill the chip with one workgroup per CU, at least
        // two stages each and no more than the partial tiles' buffer holds
        const int64_t cap = (int64_t)gram_full_tiles(m) * gram_full_splits(m) * 4096 / (256 * a.ntri);
        const int64_t stages = (n + 63) / 64;
        int64_t sp = 256 / a.plan.ngroup;
        sp = sp < cap ? sp : cap;
        sp = sp < (stages + 1) / 2 ? sp : (stages + 1) / 2;
        a.nsplit = (int)(sp < 1 ? 1 : sp);
    } else {
        a.nsplit = fixed;
    }
    const int64_t granule = 64;
    a.rows_per_split = ((n + a.nsplit - 1) / a.nsplit + granule - 1) / granule * granule;
    hipError_t e;
    if (elem_f64) e = launch_tiles<double, MODE_F64>(a, s);
    else if (a.mode == MODE_F64) e = launch_tiles<float, MODE_F64>(a, s);
    else if (a.mode == MODE_BF16X3) e = launch_tiles<float, MODE_BF16X3>(a, s);
    else e = launch_tiles<float, MODE_F32>(a, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_gram_reduce, dim3(a.ntri), dim3(1024), 0, s, a, G, st, set_window);
    return hipGetLastError();
}

hipError_t launch_copy_columns(const void* X, int64_t ldx, void* ring, int64_t ld, int64_t n, int k, int elem_f64,
                               hipStream_t s) {
    const int64_t per = (int64_t)kThreads * 8;
    const unsigned gx = (unsigned)((n + per - 1) / per);
    dim3 grid(gx < 4096 ? gx : 4096, k);
    if (elem_f64)
        hipLaunchKernelGGL(k_copy_columns<double>, grid, dim3(kThreads), 0, s, static_cast<const double*>(X), ldx,
                           static_cast<double*>(ring), ld, n, k);
    else
        hipLaunchKernelGGL(k_copy_columns<float>, grid, dim3(kThreads), 0, s, static_cast<const float*>(X), ldx,
                           static_cast<float*>(ring), ld, n, k);
    return hipGetLastError();
}

}  // namespace dmd
