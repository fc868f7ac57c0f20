// Frame preprocessing (GLIM Sec. IV-A; Sec. III-C, Preprocessing): voxel-grid
// downsampling, exact k-nearest-neighbour search and neighbour covariances with
// plane-to-plane regularisation and oriented normals.
//
// Device pipeline:
//   1. one 64-bit word per point (FP64 voxel key | point), sorted; a scan of the
//      key changes numbers the voxels; three lanes per voxel sum its run in input
//      order (FP64, one lane per coordinate).
//   2. k-NN on a hierarchy of six uniform grids (cells of 2r, 4r, ..., 64r).  The
//      grids are nested, so one sort of the points by the Morton code of their 2r
//      cell makes every cell of every grid a contiguous range of it, and one hash
//      table holds the ranges of all six.  Sixteen (or 32) lanes per query look up
//      the 27 cells around its own, take their points together and keep the k best
//      (distance, index) pairs sorted across the lanes; the result is final once
//      the k-th distance is below the distance to the unvisited region (strictly,
//      with a 1e-9 relative margin), otherwise the k-th pair is an upper bound
//      that picks the coarser grid to search.  Queries that would read many
//      candidates, or whose coarsest cells hold too few, go to a pass with a wave
//      per query.
//   3. one thread per point: mean and covariance of its neighbours (FP64),
//      cyclic Jacobi eigen-decomposition, normal = smallest eigenvector,
//      oriented towards the sensor, C = I - (1 - 1e-3) n n^T.
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <climits>
#include <cmath>
#include <string>
#include <vector>

#include "vg_device.h"

namespace vg {
namespace {

constexpr int kPBits = 21;                       // bits per axis of a preprocessing key
constexpr int64_t kPBias = 1ll << (kPBits - 1);  // keys live in [-2^20, 2^20)
constexpr uint64_t kPEmpty = ~0ull;
constexpr double kEpsReg = 1e-3;

// Voxel keys of the frame relative to its lowest, packed x | y | z (lexicographic).
struct DsKeys {
    int64_t q0[3];
    int32_t wy, wz;
    int32_t idx_bits;   // low bits of a word that hold the point (0: a separate array)
};

__global__ void k_ds_words(const double* __restrict__ xyz, int64_t n, double r, DsKeys K, uint64_t* __restrict__ word,
                           int32_t* __restrict__ idx) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint64_t q[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) q[a] = (uint64_t)((int64_t)floor(xyz[3 * i + a] / r) - K.q0[a]);
    const uint64_t key = (((q[0] << K.wy) | q[1]) << K.wz) | q[2];
    word[i] = (key << K.idx_bits) | (K.idx_bits ? (uint64_t)i : 0ull);
    if (idx != nullptr) idx[i] = (int32_t)i;
}

// 1 where a new voxel starts among the sorted words
struct KeyChange {
    const uint64_t* word;
    int32_t idx_bits;
    __host__ __device__ int32_t operator()(int64_t i) const {
        return i == 0 || (word[i - 1] >> idx_bits) != (word[i] >> idx_bits) ? 1 : 0;
    }
};

// first element of every voxel; their number goes to pinned host memory
__global__ void k_ds_starts(const int32_t* __restrict__ scan, int64_t n, int32_t* __restrict__ start,
                            int32_t* __restrict__ h_count) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t v = scan[i];
    if (i == 0 || scan[i - 1] != v) start[v - 1] = (int32_t)i;
    if (i == n - 1) {
        start[v] = (int32_t)n;
        *h_count = v;
    }
}

__device__ __forceinline__ uint64_t spread21(uint64_t v) {
    uint64_t x = v & 0x1fffffull;
    x = (x | (x << 32)) & 0x1f00000000ffffull;
    x = (x | (x << 16)) & 0x1f0000ff0000ffull;
    x = (x | (x << 8)) & 0x100f00f00f00f00full;
    x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

constexpr int kGrids = 6;       // cell sizes 2r, 4r, ..., 64r
// Workgroups of a launch at most: a launch holds fewer than 2^32 threads, and frames
// of 2^27 points and more with 16 or 32 lanes a point would not.  4 M queries of 16
// lanes take milliseconds, so a launch per range costs them nothing.
constexpr int64_t kMaxGroups = 1 << 18;
// Slots of the cell table are 32-bit numbers, and a point has up to kGrids cells: one
// entry has to stay empty, or a search for a missing cell would not end.
constexpr uint32_t kMaxTableBits = 32;
constexpr int64_t kMaxCellPoints = ((1ll << kMaxTableBits) - 1) / kGrids;

// The nested grids: cells are counted from c0, a multiple of the coarsest cell, so
// a cell of grid g is a 2r cell's coordinates shifted by g.
struct Cells {
    double h;            // finest cell size, 2r
    int64_t c0[3];
    int32_t hi[3];       // last 2r cell per axis (the cloud's, with a margin of one cell)
    int32_t w;           // bits per axis
    int32_t idx_bits;    // low bits of a sort word that hold the point (0: a separate array)
    uint32_t lg;         // table entries = 2^lg, lg <= 32
};
__device__ __forceinline__ uint32_t slot_mask(const Cells& C) { return (uint32_t)((1ull << C.lg) - 1ull); }
// Table key of a grid's cell: the Morton code under a leading one, shifted, so the
// grids' keys differ by the place of their highest bit.
__device__ __forceinline__ uint64_t cell_key(const Cells& C, uint64_t code2r, int g) {
    return ((1ull << (3 * C.w)) | code2r) >> (3 * g);
}
__device__ __forceinline__ uint32_t cell_slot(uint64_t key, uint32_t lg) {
    return (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> (64 - lg));
}
__device__ __forceinline__ int32_t cell_coord(const Cells& C, double x, int a) {
    return (int32_t)((int64_t)floor(x / C.h) - C.c0[a]);
}

// Voxel centroids: three lanes per voxel, one per coordinate, eight points in
// flight: the FP64 sum of its run in input order, then the mean; and the sort word
// of its 2r cell.  (One thread per voxel with one point in flight: 45 us for 107k
// raw points, most of it the chain of gathers.)
constexpr int kCentPerWave = 21;
__global__ __launch_bounds__(256) void k_ds_centroids(const double* __restrict__ xyz, const uint64_t* __restrict__ word,
                                                      const int32_t* __restrict__ idx, int32_t ds_bits,
                                                      const int32_t* __restrict__ start, int64_t m, Cells C,
                                                      double* __restrict__ out, int32_t* __restrict__ out_counts,
                                                      uint64_t* __restrict__ cword, int32_t* __restrict__ cidx) {
    const int lane = threadIdx.x & 63, g = lane / 3, k = lane % 3;
    const int64_t v = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * kCentPerWave + g;
    if (g >= kCentPerWave || v >= m) return;
    const int32_t j0 = start[v], j1 = start[v + 1];
    const uint64_t mask = (1ull << ds_bits) - 1ull;
    constexpr int kStep = 8;
    double s = 0.0;
    for (int32_t j = j0; j < j1; j += kStep) {
        double x[kStep];
#pragma unroll
        for (int q = 0; q < kStep; ++q)
            if (j + q < j1) {
                const int64_t p = idx != nullptr ? (int64_t)idx[j + q] : (int64_t)(word[j + q] & mask);
                x[q] = xyz[3 * p + k];
            }
#pragma unroll
        for (int q = 0; q < kStep; ++q)
            if (j + q < j1) s += x[q];
    }
    const double c = s / (double)(j1 - j0);
    out[3 * v + k] = c;
    // the three coordinates' cells meet in the first lane of the voxel
    const uint64_t part = spread21((uint64_t)cell_coord(C, c, k)) << (2 - k);
    const uint64_t p1 = __shfl_down(part, 1), p2 = __shfl_down(part, 2);
    if (k == 0) {
        out_counts[v] = j1 - j0;
        cword[v] = ((part | p1 | p2) << C.idx_bits) | (C.idx_bits ? (uint64_t)v : 0ull);
        if (cidx != nullptr) cidx[v] = (int32_t)v;
    }
}

__global__ void k_fill_cells(u64x2* p, int64_t n) {
    const int64_t step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) p[i] = u64x2{kPEmpty, 0ull};
}

// A point in cell order.
struct alignas(32) CellPoint {
    double x, y, z;
    int64_t i;           // its index in the cloud
};

// Points in cell order, and the range of every cell of every grid: the first
// point of a range writes its start, the last its end (the low and high halves of
// the entry's second word), whichever comes first inserts the key.
__global__ void k_cells(const double* __restrict__ xyz, const uint64_t* __restrict__ cword, const int32_t* __restrict__ cidx,
                        int64_t m, Cells C, CellPoint* __restrict__ pts, u64x2* __restrict__ table) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= m) return;
    const uint64_t w = cword[t], code = w >> C.idx_bits;
    const int64_t i = cidx != nullptr ? (int64_t)cidx[t] : (int64_t)(w & ((1ull << C.idx_bits) - 1ull));
    pts[t] = CellPoint{xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2], i};
    const uint64_t prev = t > 0 ? cword[t - 1] >> C.idx_bits : 0ull, next = t + 1 < m ? cword[t + 1] >> C.idx_bits : 0ull;
    const uint32_t mask = slot_mask(C);
    for (int g = 0; g < kGrids; ++g) {
        const bool first = t == 0 || (prev >> (3 * g)) != (code >> (3 * g));
        const bool last = t + 1 == m || (next >> (3 * g)) != (code >> (3 * g));
        if (!first && !last) break;   // inside a range of this grid: inside one of every coarser grid too
        const uint64_t key = cell_key(C, code, g);
        uint32_t h = cell_slot(key, C.lg);
        for (;;) {
            const unsigned long long was = atomicCAS((unsigned long long*)&table[h], (unsigned long long)kPEmpty,
                                                     (unsigned long long)key);
            if (was == kPEmpty || was == key) break;
            h = (h + 1u) & mask;
        }
        int32_t* range = reinterpret_cast<int32_t*>(reinterpret_cast<uint64_t*>(&table[h]) + 1);
        if (first) range[0] = (int32_t)t;
        if (last) range[1] = (int32_t)(t + 1);
    }
}

// squared distance with every operation rounded on its own: this file is
// compiled with -ffp-contract=off, so no multiply-add is fused
__device__ __forceinline__ double sqdist_rn(double ax, double ay, double az, double bx, double by, double bz) {
    const double dx = bx - ax, dy = by - ay, dz = bz - az;
    const double xx = dx * dx, yy = dy * dy, zz = dz * dz;
    return (xx + yy) + zz;
}

__device__ __forceinline__ bool pair_less(double d, int32_t j, double D, int32_t J) {
    return d < D || (d == D && j < J);
}

// Compare-exchange of (d, j) with the lane at xor o: the lane keeps the smaller
// pair if `low`, else the larger.
__device__ __forceinline__ void exchange(double& d, int32_t& j, int o, bool low) {
    const double od = __shfl_xor(d, o);
    const int32_t oj = __shfl_xor(j, o);
    const bool less = pair_less(od, oj, d, j);
    if (less == low) {
        d = od;
        j = oj;
    }
}

// The G smallest pairs seen by a group of G lanes, ascending over the lanes: one
// new pair per lane is sorted (bitonic) and merged into the kept list.
template <int G>
__device__ __forceinline__ void keep_smallest(double& D, int32_t& I, double d, int32_t j, int gl) {
    // new pairs in descending order
#pragma unroll
    for (int size = 2; size <= G; size <<= 1)
#pragma unroll
        for (int o = size >> 1; o > 0; o >>= 1) {
            const bool up = (gl & size) != 0 && size < G;   // ascending half of a bitonic run
            exchange(d, j, o, ((gl & o) == 0) == up);
        }
    // the smaller of list[l] and new[l] (ascending against descending) are the G
    // smallest, and form a bitonic sequence
    if (pair_less(d, j, D, I)) {
        D = d;
        I = j;
    }
#pragma unroll
    for (int o = G >> 1; o > 0; o >>= 1) exchange(D, I, o, (gl & o) == 0);
}

// Candidates of one query in the (2R + 1)^3 cells of grid g around its own, taken
// by a group of G lanes: each lane looks up a cell, the cells' ranges are laid end
// to end, and every lane takes every G-th candidate.  Cells whose box lies beyond
// the bound are skipped (margin for the rounding of the box and the distances).
// Returns false, with nothing taken, if more than `most` candidates would be read.
template <int G>
struct GroupLds {
    int32_t start[G], before[G];
};
struct Query {
    double x[3];
    int32_t c[3];        // its 2r cell
};
template <int G, bool LIMITED>
__device__ __forceinline__ bool scan_cube(const Cells& C, const u64x2* __restrict__ table,
                                          const CellPoint* __restrict__ pts, const Query& q, int g, int R, double bound,
                                          int kk, int gl, GroupLds<G>& S, int& budget, double& D, int32_t& I) {
    const double h = C.h * (double)(1 << g);
    const int side = 2 * R + 1;
    const int64_t cells = (int64_t)side * side * side;
    const uint32_t mask = slot_mask(C);
    constexpr int PASSES = LIMITED ? (27 + G - 1) / G : 1;   // LIMITED: R = 1, all cells counted before any point is read
    for (int64_t base = 0; base < cells; base += (int64_t)G * PASSES) {
        int32_t from[PASSES], cnt[PASSES];
        int total = 0;
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            const int64_t j = base + p * G + gl;
            from[p] = 0;
            cnt[p] = 0;
            if (j < cells) {
                const int32_t o[3] = {(int32_t)(j / (side * side)) - R, (int32_t)((j / side) % side) - R,
                                      (int32_t)(j % side) - R};
                bool in = true;
                double e2 = 0.0;
                uint64_t code = 0;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const int32_t x = (q.c[a] >> g) + o[a];
                    in = in && x >= 0 && x <= (C.hi[a] >> g);
                    const double lo = (double)((int64_t)x * (1ll << g) + C.c0[a]) * C.h;
                    const double e = fmax(0.0, fmax(lo - q.x[a], q.x[a] - (lo + h)));
                    e2 += e * e;
                    code |= spread21((uint64_t)(uint32_t)x) << (2 - a);
                }
                if (in && !(e2 * (1.0 - 1e-9) > bound)) {
                    const uint64_t key = (1ull << (3 * (C.w - g))) | code;
                    uint32_t s = cell_slot(key, C.lg);
                    for (;;) {
                        const u64x2 t = table[s];
                        if (t.x == key) {
                            from[p] = (int32_t)(uint32_t)t.y;
                            cnt[p] = (int32_t)(uint32_t)(t.y >> 32) - from[p];
                            break;
                        }
                        if (t.x == kPEmpty) break;
                        s = (s + 1u) & mask;
                    }
                }
            }
            total += cnt[p];
        }
        if constexpr (LIMITED) {
            int all = total;
#pragma unroll
            for (int o = G >> 1; o > 0; o >>= 1) all += __shfl_xor(all, o);
            budget -= all;
            if (budget < 0) return false;
        }
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            // exclusive prefix of the lanes' counts, and each cell's start shifted by it
            int incl = cnt[p];
#pragma unroll
            for (int o = 1; o < G; o <<= 1) {
                const int up = __shfl_up(incl, o, G);
                if (gl >= o) incl += up;
            }
            const int sum = __shfl(incl, G - 1, G);
            S.before[gl] = incl - cnt[p];
            S.start[gl] = from[p] - (incl - cnt[p]);
            __builtin_amdgcn_wave_barrier();
            for (int c0 = 0; c0 < sum; c0 += G) {
                const int c = c0 + gl;
                double d = INFINITY;
                int32_t j = INT_MAX;
                if (c < sum) {
                    int cell = 0;   // the last cell whose candidates start at or before c
#pragma unroll
                    for (int o = G >> 1; o > 0; o >>= 1)
                        if (S.before[cell + o] <= c) cell += o;
                    const CellPoint pt = pts[S.start[cell] + c];
                    d = sqdist_rn(q.x[0], q.x[1], q.x[2], pt.x, pt.y, pt.z);
                    j = (int32_t)pt.i;
                }
                // merged only if some lane's candidate beats the group's k-th pair
                const double kD = __shfl(D, kk - 1, G);
                const int32_t kI = __shfl(I, kk - 1, G);
                const bool better = pair_less(d, j, kD, kI);
                int any = better ? 1 : 0;
#pragma unroll
                for (int o = G >> 1; o > 0; o >>= 1) any |= __shfl_xor(any, o);
                if (any) keep_smallest<G>(D, I, d, j, gl);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    return true;
}

// Whether the k-th distance kD is final after the (2R + 1)^3 cells of grid g: the
// cells cover the cloud, or the distance to the first cell outside is larger.
__device__ __forceinline__ bool settled(const Cells& C, const Query& q, int g, int R, double kD) {
    const double h = C.h * (double)(1 << g);
    bool all = true;
    double b = INFINITY;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int32_t c = q.c[a] >> g;
        all = all && c - R <= 0 && c + R >= (C.hi[a] >> g);
        const double lo = (double)((int64_t)(c - R) * (1ll << g) + C.c0[a]) * C.h;
        b = fmin(b, fmin(q.x[a] - lo, lo + (double)(2 * R + 1) * h - q.x[a]));
    }
    return all || (b > 0.0 && kD < b * b * (1.0 - 1e-9));
}

constexpr int kBudget = 1024;   // candidates a query may scan before it is handed to the wave-wide pass

// Exact k-NN, G lanes per query (G >= k), queries from t0 on in cell order.
//
// A pass over grid g lists the k best pairs among the points of the cells it
// visits.  If it cannot prove them final, its k-th pair P is still an upper
// bound of the true k-th pair (its points are a subset of the cloud), so the
// next pass starts on the first coarser grid whose cells are at least sqrt(d(P))
// wide and skips cells whose box lies farther than sqrt(d(P)): every point of the
// true k best lies within that distance, so the pass still finds all of them.
//
// Bound by latency: a query is a chain of table reads, point reads and merges.
// One thread per query kept 640 waves busy with 27 cells each one after another
// (40k points, k = 10: 482 us, and 286 us for the queries handed over).
template <int G>
__global__ __launch_bounds__(256) void k_knn(Cells C, const u64x2* __restrict__ table, const CellPoint* __restrict__ pts,
                                             int64_t t0, int64_t m, int k, int32_t* __restrict__ nbr,
                                             double* __restrict__ nd2, int32_t* __restrict__ hard,
                                             double* __restrict__ hard_bound, int32_t* __restrict__ n_hard) {
    __shared__ GroupLds<G> s_lds[256 / G];
    const int gl = threadIdx.x % G;
    const int64_t t = t0 + (int64_t)blockIdx.x * (256 / G) + threadIdx.x / G;
    if (t >= m) return;
    GroupLds<G>& S = s_lds[threadIdx.x / G];
    const CellPoint me = pts[t];
    Query q{{me.x, me.y, me.z}, {0, 0, 0}};
#pragma unroll
    for (int a = 0; a < 3; ++a) q.c[a] = cell_coord(C, q.x[a], a);
    const int kk = (int)min((int64_t)k, m);
    double bound = INFINITY;
    int budget = kBudget;
    bool done = false;
    double D = INFINITY;
    int32_t I = INT_MAX;
    for (int g = 0; g < kGrids && !done; ++g) {
        const double h = C.h * (double)(1 << g);
        if (g < kGrids - 1 && bound < INFINITY && h * h <= bound) continue;   // cells too small for the bound
        D = INFINITY;
        I = INT_MAX;
        if (!scan_cube<G, true>(C, table, pts, q, g, 1, bound, kk, gl, S, budget, D, I)) break;
        const double kD = __shfl(D, kk - 1, G);
        if (kD < INFINITY) {
            done = settled(C, q, g, 1, kD);
            bound = kD;
        }
    }
    if (done) {
        if (gl < k) {
            const bool ok = gl < kk;
            nbr[me.i * k + gl] = ok ? I : -1;
            nd2[me.i * k + gl] = ok ? D : INFINITY;
        }
    } else if (gl == 0) {
        const int32_t s = atomicAdd(n_hard, 1);
        hard[s] = (int32_t)t;
        hard_bound[s] = bound;
    }
}

// The queries handed over, one wave each: the same search without a budget from the
// first grid that fits the bound, then ever larger cubes of the coarsest cells,
// and every point once a cube would hold more cells than a quarter of the points.
__global__ __launch_bounds__(64) void k_knn_wave(Cells C, const u64x2* __restrict__ table,
                                                 const CellPoint* __restrict__ pts, int64_t m, int k,
                                                 const int32_t* __restrict__ hard, const double* __restrict__ hard_bound,
                                                 const int32_t* __restrict__ n_hard, int32_t* __restrict__ nbr,
                                                 double* __restrict__ nd2) {
    __shared__ GroupLds<64> S;
    const int lane = threadIdx.x;
    const int kk = (int)min((int64_t)k, m);
    const int32_t total = *n_hard;
    for (int32_t s = blockIdx.x; s < total; s += gridDim.x) {
        const CellPoint me = pts[hard[s]];
        Query q{{me.x, me.y, me.z}, {0, 0, 0}};
#pragma unroll
        for (int a = 0; a < 3; ++a) q.c[a] = cell_coord(C, q.x[a], a);
        double bound = hard_bound[s];
        double D = INFINITY;
        int32_t I = INT_MAX;
        bool done = false;
        int unused = 0;
        for (int g = 0, R = 1; !done;) {
            const double h = C.h * (double)(1 << g);
            if (g < kGrids - 1 && bound < INFINITY && h * h <= bound) {
                ++g;
                continue;
            }
            D = INFINITY;
            I = INT_MAX;
            const int64_t side = 2 * R + 1;
            if (R > 1 && side * side * side > m / 4 + 64) {
                for (int64_t p0 = 0; p0 < m; p0 += 64) {
                    const int64_t p = p0 + lane;
                    double d = INFINITY;
                    int32_t j = INT_MAX;
                    if (p < m) {
                        const CellPoint pt = pts[p];
                        d = sqdist_rn(q.x[0], q.x[1], q.x[2], pt.x, pt.y, pt.z);
                        j = (int32_t)pt.i;
                    }
                    const double kD = __shfl(D, kk - 1);
                    const int32_t kI = __shfl(I, kk - 1);
                    if (__any(pair_less(d, j, kD, kI))) keep_smallest<64>(D, I, d, j, lane);
                }
                done = true;
            } else {
                scan_cube<64, false>(C, table, pts, q, g, R, bound, kk, lane, S, unused, D, I);
                const double kD = __shfl(D, kk - 1);
                if (kD < INFINITY) {
                    done = settled(C, q, g, R, kD);
                    bound = kD;
                }
                if (g < kGrids - 1) ++g;
                else R *= 2;
            }
        }
        if (lane < k) {
            const bool ok = lane < kk;
            nbr[me.i * k + lane] = ok ? I : -1;
            nd2[me.i * k + lane] = ok ? D : INFINITY;
        }
    }
}

// One Jacobi rotation in the (p, q) plane: annihilates a[p][q] (Golub & Van Loan,
// symmetric Schur decomposition), accumulates the rotation into v.
template <int P, int Q, int R>
__device__ __forceinline__ void jacobi_rot(double (&a)[3][3], double (&v)[3][3]) {
    const double apq = a[P][Q];
    if (apq == 0.0) return;
    const double tau = (a[Q][Q] - a[P][P]) / (2.0 * apq);
    double t;
    if (fabs(tau) > 1e150) {
        t = 0.5 / tau;
    } else {
        t = (tau >= 0.0 ? 1.0 : -1.0) / (fabs(tau) + sqrt(1.0 + tau * tau));
    }
    const double c = 1.0 / sqrt(1.0 + t * t), s = t * c;
    a[P][P] -= t * apq;
    a[Q][Q] += t * apq;
    a[P][Q] = a[Q][P] = 0.0;
    const double arp = a[R][P], arq = a[R][Q];
    a[R][P] = a[P][R] = c * arp - s * arq;
    a[R][Q] = a[Q][R] = s * arp + c * arq;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const double vp = v[i][P], vq = v[i][Q];
        v[i][P] = c * vp - s * vq;
        v[i][Q] = s * vp + c * vq;
    }
}

__global__ void k_cov_normals(const double* __restrict__ xyz, const int32_t* __restrict__ nbr, int64_t m, int k,
                              double ox, double oy, double oz, double* __restrict__ cov,
                              double* __restrict__ cov_raw, double* __restrict__ nrm) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    const int32_t* row = nbr + i * k;
    int kk = 0;
    double mx = 0.0, my = 0.0, mz = 0.0;
    for (int s = 0; s < k; ++s) {
        const int32_t j = row[s];
        if (j < 0) break;
        mx += xyz[3 * j + 0];
        my += xyz[3 * j + 1];
        mz += xyz[3 * j + 2];
        ++kk;
    }
    const double inv = 1.0 / (double)kk;
    mx *= inv;
    my *= inv;
    mz *= inv;
    double cxx = 0, cxy = 0, cxz = 0, cyy = 0, cyz = 0, czz = 0;
    for (int s = 0; s < kk; ++s) {
        const int32_t j = row[s];
        const double dx = xyz[3 * j + 0] - mx, dy = xyz[3 * j + 1] - my, dz = xyz[3 * j + 2] - mz;
        cxx += dx * dx;
        cxy += dx * dy;
        cxz += dx * dz;
        cyy += dy * dy;
        cyz += dy * dz;
        czz += dz * dz;
    }
    cxx *= inv;
    cxy *= inv;
    cxz *= inv;
    cyy *= inv;
    cyz *= inv;
    czz *= inv;
    double* cr = cov_raw + 6 * i;
    cr[0] = cxx;
    cr[1] = cxy;
    cr[2] = cxz;
    cr[3] = cyy;
    cr[4] = cyz;
    cr[5] = czz;
    double a[3][3] = {{cxx, cxy, cxz}, {cxy, cyy, cyz}, {cxz, cyz, czz}};
    double v[3][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}};
    const double scale = cxx * cxx + cyy * cyy + czz * czz + 2.0 * (cxy * cxy + cxz * cxz + cyz * cyz);
    for (int sweep = 0; sweep < 32; ++sweep) {
        const double off = a[0][1] * a[0][1] + a[0][2] * a[0][2] + a[1][2] * a[1][2];
        if (off == 0.0 || off <= 1e-34 * scale) break;
        jacobi_rot<0, 1, 2>(a, v);
        jacobi_rot<0, 2, 1>(a, v);
        jacobi_rot<1, 2, 0>(a, v);
    }
    // smallest eigenvalue's column (first index on ties)
    int c = 0;
    if (a[1][1] < a[c][c]) c = 1;
    if (a[2][2] < a[c][c]) c = 2;
    double nx = c == 0 ? v[0][0] : (c == 1 ? v[0][1] : v[0][2]);
    double ny = c == 0 ? v[1][0] : (c == 1 ? v[1][1] : v[1][2]);
    double nz = c == 0 ? v[2][0] : (c == 1 ? v[2][1] : v[2][2]);
    const double px = xyz[3 * i + 0], py = xyz[3 * i + 1], pz = xyz[3 * i + 2];
    if (nx * (ox - px) + ny * (oy - py) + nz * (oz - pz) < 0.0) {
        nx = -nx;
        ny = -ny;
        nz = -nz;
    }
    double* no = nrm + 3 * i;
    no[0] = nx;
    no[1] = ny;
    no[2] = nz;
    const double w = 1.0 - kEpsReg;
    double* co = cov + 6 * i;
    co[0] = 1.0 - w * nx * nx;
    co[1] = -w * nx * ny;
    co[2] = -w * nx * nz;
    co[3] = 1.0 - w * ny * ny;
    co[4] = -w * ny * nz;
    co[5] = 1.0 - w * nz * nz;
}

// Leading principal minors of [a b c; b d e; c e f] all positive (each operation
// rounded on its own: this file is compiled without contraction).
__device__ __forceinline__ bool spd6(const double* c) {
    const double a = c[0], b = c[1], cc = c[2], d = c[3], e = c[4], f = c[5];
    const double m2 = a * d - b * b;
    const double det = a * (d * f - e * e) - b * (b * f - cc * e) + cc * (b * e - cc * d);
    return a > 0.0 && m2 > 0.0 && det > 0.0;
}

// Check of a cloud's arrays, and its bounding box: each workgroup takes a share of
// the points and writes its part to pinned host memory, where the host joins them.
// Bound by its reads (24 B per point, 72-96 B with covariances and normals).  On the
// host the same loops took 1.4 ms for a 140k-point submap's source and map, more than
// the two uploads and builds together.
__global__ __launch_bounds__(256) void k_check(const double* __restrict__ xyz, const double* __restrict__ cov,
                                               const double* __restrict__ nrm, int64_t n, CheckPart* __restrict__ out) {
    __shared__ CheckPart s[4];
    double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    int32_t flags = 0;
    int64_t bad = INT64_MAX;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double x = xyz[3 * i + a];
            if (!isfinite(x)) flags |= kBadXyz;
            lo[a] = fmin(lo[a], x);
            hi[a] = fmax(hi[a], x);
            if (nrm != nullptr && !isfinite(nrm[3 * i + a])) flags |= kBadNormal;
        }
        if (cov != nullptr) {
            double c[6];
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                c[k] = cov[6 * i + k];
                if (!isfinite(c[k])) flags |= kBadCov;
            }
            if (!spd6(c)) bad = min(bad, i);
        }
    }
#pragma unroll
    for (int w = 32; w >= 1; w >>= 1) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            lo[a] = fmin(lo[a], __shfl_xor(lo[a], w));
            hi[a] = fmax(hi[a], __shfl_xor(hi[a], w));
        }
        flags |= __shfl_xor(flags, w);
        bad = min(bad, (int64_t)__shfl_xor((long long)bad, w));
    }
    if ((threadIdx.x & 63) == 0) {
        CheckPart& p = s[threadIdx.x >> 6];
        for (int a = 0; a < 3; ++a) {
            p.box[a] = lo[a];
            p.box[3 + a] = hi[a];
        }
        p.bad = bad;
        p.flags = flags;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        CheckPart p = s[0];
        for (int w = 1; w < 4; ++w) {
            for (int a = 0; a < 3; ++a) {
                p.box[a] = fmin(p.box[a], s[w].box[a]);
                p.box[3 + a] = fmax(p.box[3 + a], s[w].box[3 + a]);
            }
            p.bad = min(p.bad, s[w].bad);
            p.flags |= s[w].flags;
        }
        for (int a = 0; a < 3; ++a) p.first[a] = xyz[a];
        out[blockIdx.x] = p;
    }
}

int grid_of(int64_t n, int b = 256) { return (int)((n + b - 1) / b); }

int bits_for(uint64_t max_value) {
    int b = 0;
    while (b < 64 && (max_value >> b) != 0) ++b;
    return b;
}

// Sort of n words by their bits above idx_bits (the points ride in the low bits),
// or of (word, point) pairs where idx_bits is 0.
hipError_t sort_words(void* tmp, size_t& bytes, uint64_t* in, uint64_t* out, int32_t* i_in, int32_t* i_out, int64_t n,
                      int idx_bits, int key_bits, hipStream_t st) {
    const int end = std::max(1, key_bits + idx_bits);
    if (i_in == nullptr) return hipcub::DeviceRadixSort::SortKeys(tmp, bytes, in, out, (int)n, idx_bits, std::max(end, idx_bits + 1), st);
    return hipcub::DeviceRadixSort::SortPairs(tmp, bytes, in, out, i_in, i_out, (int)n, 0, end, st);
}

// every output array of a cloud in one allocation
hipError_t alloc_cloud(vg_cloud* c, int64_t m, int k) {
    const size_t nd = (size_t)m * (3 + 6 + 6 + 3 + k), ni = (size_t)m * (1 + k);
    void* b = nullptr;
    hipError_t e = c->pool->get(&b, sizeof(double) * (nd ? nd : 1) + sizeof(int32_t) * (ni ? ni : 1));
    if (e != hipSuccess) return e;
    c->block = b;
    double* d = (double*)b;
    c->xyz = d;
    c->cov = d + 3 * m;
    c->cov_raw = d + 9 * m;
    c->nrm = d + 15 * m;
    c->d2 = d + 18 * m;
    int32_t* i = (int32_t*)(d + (nd ? nd : 1));
    c->counts = i;
    c->nbr = i + m;
    return hipSuccess;
}

}  // namespace

void free_cloud(vg_cloud* c) {
    if (c->block) c->pool->put(c->block);
    c->block = nullptr;
    c->xyz = c->cov = c->cov_raw = c->nrm = c->d2 = nullptr;
    c->counts = c->nbr = nullptr;
}

vg_status preprocess_frame(vg_context* ctx, Scratch& sc, const double* d_xyz, int64_t n, const double box[6], double r,
                           int k, const double sensor[3], vg_cloud* out) {
    hipStream_t st = ctx->stream;
    out->k = k;
    out->m = 0;
    if (n == 0) {
        VG_HIP(alloc_cloud(out, 0, k));
        return VG_OK;
    }
    // 1. downsampling.  The key range follows from the frame's bounding box (floor
    // and division are monotone).
    DsKeys K{};
    int64_t span[3];
    for (int a = 0; a < 3; ++a) {
        const double lo = std::floor(box[a] / r), hi = std::floor(box[3 + a] / r);
        if (!(lo >= -(double)kPBias && hi < (double)kPBias)) {
            set_error("downsampling voxel key outside the packable range (|floor(x / r)| >= 2^20 on an axis)");
            return VG_ERR_KEY_RANGE;
        }
        K.q0[a] = (int64_t)lo;
        span[a] = (int64_t)hi - (int64_t)lo;
    }
    K.wy = bits_for((uint64_t)span[1]);
    K.wz = bits_for((uint64_t)span[2]);
    const int ds_bits = bits_for((uint64_t)span[0]) + K.wy + K.wz, ib = bits_for((uint64_t)(n - 1));
    const bool packed = ds_bits + ib <= 64 && ib > 0;
    K.idx_bits = packed ? ib : 0;
    uint64_t *w0, *w1;
    int32_t *i0 = nullptr, *i1 = nullptr, *scan, *start;
    VG_HIP(sc.get(&w0, n));
    VG_HIP(sc.get(&w1, n));
    VG_HIP(sc.get(&scan, n));
    VG_HIP(sc.get(&start, n + 1));
    if (!packed) {
        VG_HIP(sc.get(&i0, n));
        VG_HIP(sc.get(&i1, n));
    }
    const hipcub::CountingInputIterator<int64_t> cnt(0);
    const hipcub::TransformInputIterator<int32_t, KeyChange, hipcub::CountingInputIterator<int64_t>> heads(
        cnt, KeyChange{w1, K.idx_bits});
    size_t b1 = 0, b2 = 0;
    (void)sort_words(nullptr, b1, w0, w1, i0, i1, n, K.idx_bits, ds_bits, st);
    (void)hipcub::DeviceScan::InclusiveSum(nullptr, b2, heads, scan, (int)n);
    const size_t tmp_bytes = std::max(b1, b2) + 256;
    char* tmp = nullptr;
    VG_HIP(sc.get(&tmp, tmp_bytes));
    k_ds_words<<<grid_of(n), 256, 0, st>>>(d_xyz, n, r, K, w0, i0);
    VG_HIP(hipGetLastError());
    size_t tb = tmp_bytes;
    VG_HIP(sort_words(tmp, tb, w0, w1, i0, i1, n, K.idx_bits, ds_bits, st));
    tb = tmp_bytes;
    VG_HIP(hipcub::DeviceScan::InclusiveSum(tmp, tb, heads, scan, (int)n, st));
    k_ds_starts<<<grid_of(n), 256, 0, st>>>(scan, n, start, ctx->h_small);
    VG_HIP(hipGetLastError());
    VG_HIP(hipStreamSynchronize(st));
    const int64_t m = ctx->h_small[0];
    if (m > kMaxCellPoints) {
        set_error("too many downsampled points (" + std::to_string(m) + "; at most " + std::to_string(kMaxCellPoints) + ")");
        return VG_ERR_CAPACITY;
    }
    VG_HIP(alloc_cloud(out, m, k));
    out->m = m;
    // 2. cells and the neighbour search (no host round trip)
    Cells C{};
    C.h = 2.0 * r;
    int64_t widest = 0;
    for (int a = 0; a < 3; ++a) {
        // a centroid lies in its points' box up to rounding: one cell of margin
        const int64_t lo = (int64_t)std::floor(box[a] / C.h) - 1, hi = (int64_t)std::floor(box[3 + a] / C.h) + 1;
        C.c0[a] = (lo >> (kGrids - 1)) << (kGrids - 1);
        C.hi[a] = (int32_t)(hi - C.c0[a]);
        widest = std::max<int64_t>(widest, C.hi[a]);
    }
    C.w = std::max(bits_for((uint64_t)widest), kGrids);
    const int cb = bits_for((uint64_t)(m - 1));
    const bool cpacked = 3 * C.w + cb <= 64 && cb > 0;
    C.idx_bits = cpacked ? cb : 0;
    C.lg = 6;   // at most six cells per point: load factor <= 3/4 (up to 2^29 points), and mostly below 1/4
    while (C.lg < kMaxTableBits && (1ull << C.lg) < 8ull * (uint64_t)m) ++C.lg;
    uint64_t *cw0, *cw1;
    int32_t *ci0 = nullptr, *ci1 = nullptr, *hard, *n_hard;
    CellPoint* pts;
    u64x2* table;
    double* hard_bound;
    VG_HIP(sc.get(&cw0, m));
    VG_HIP(sc.get(&cw1, m));
    if (!cpacked) {
        VG_HIP(sc.get(&ci0, m));
        VG_HIP(sc.get(&ci1, m));
    }
    VG_HIP(sc.get(&pts, m));
    VG_HIP(sc.get(&table, ((size_t)1 << C.lg) + 1));   // the entry behind the table: the handed-over queries' count
    VG_HIP(sc.get(&hard, m));
    VG_HIP(sc.get(&hard_bound, m));
    char* ctmp = nullptr;
    size_t ctb = 0;
    (void)sort_words(nullptr, ctb, cw0, cw1, ci0, ci1, m, C.idx_bits, 3 * C.w, st);
    ctb += 256;
    VG_HIP(sc.get(&ctmp, ctb));
    n_hard = reinterpret_cast<int32_t*>(reinterpret_cast<uint64_t*>(table + ((size_t)1 << C.lg)) + 1);
    const int64_t entries = ((int64_t)1 << C.lg) + 1;
    k_fill_cells<<<(int)std::min<int64_t>((entries + 255) / 256, 1 << 22), 256, 0, st>>>(table, entries);
    VG_HIP(hipGetLastError());
    k_ds_centroids<<<grid_of(m, 4 * kCentPerWave), 256, 0, st>>>(d_xyz, w1, i1, K.idx_bits, start, m, C, out->xyz,
                                                                out->counts, cw0, ci0);
    VG_HIP(hipGetLastError());
    VG_HIP(sort_words(ctmp, ctb, cw0, cw1, ci0, ci1, m, C.idx_bits, 3 * C.w, st));
    k_cells<<<grid_of(m), 256, 0, st>>>(out->xyz, cw1, ci1, m, C, pts, table);
    VG_HIP(hipGetLastError());
    // 16 lanes hold the best 16 pairs, 32 the best 32
    const int per = k <= 16 ? 16 : 8;   // queries a workgroup
    for (int64_t t0 = 0; t0 < m; t0 += kMaxGroups * per) {
        const int grid = (int)std::min<int64_t>(kMaxGroups, (m - t0 + per - 1) / per);
        if (k <= 16) k_knn<16><<<grid, 256, 0, st>>>(C, table, pts, t0, m, k, out->nbr, out->d2, hard, hard_bound, n_hard);
        else k_knn<32><<<grid, 256, 0, st>>>(C, table, pts, t0, m, k, out->nbr, out->d2, hard, hard_bound, n_hard);
        VG_HIP(hipGetLastError());
    }
    k_knn_wave<<<4096, 64, 0, st>>>(C, table, pts, m, k, hard, hard_bound, n_hard, out->nbr, out->d2);
    VG_HIP(hipGetLastError());
    // 3. covariances and normals
    k_cov_normals<<<grid_of(m), 256, 0, st>>>(out->xyz, out->nbr, m, k, sensor[0], sensor[1], sensor[2], out->cov,
                                               out->cov_raw, out->nrm);
    VG_HIP(hipGetLastError());
    // the points' bounding box and point 0, for the sources and maps made from the cloud
    const vg_status rc = launch_check(ctx, out->xyz, nullptr, nullptr, m);
    if (rc != VG_OK) return rc;
    VG_HIP(hipStreamSynchronize(st));
    const CheckPart c = joined_check(ctx, m);
    for (int a = 0; a < 6; ++a) out->box[a] = c.box[a];
    for (int a = 0; a < 3; ++a) out->first[a] = c.first[a];
    return VG_OK;
}

static int check_grid(int64_t n) { return (int)std::min<int64_t>(kCheckParts, (n + 255) / 256); }

vg_status launch_check(vg_context* ctx, const double* d_xyz, const double* d_cov, const double* d_nrm, int64_t n) {
    k_check<<<check_grid(n), 256, 0, ctx->stream>>>(d_xyz, d_cov, d_nrm, n, reinterpret_cast<CheckPart*>(ctx->h_small));
    VG_HIP(hipGetLastError());
    return VG_OK;
}

CheckPart joined_check(const vg_context* ctx, int64_t n) {
    const CheckPart* part = reinterpret_cast<const CheckPart*>(ctx->h_small);
    CheckPart p = part[0];
    for (int k = 1; k < check_grid(n); ++k) {
        for (int a = 0; a < 3; ++a) {
            p.box[a] = std::min(p.box[a], part[k].box[a]);
            p.box[3 + a] = std::max(p.box[3 + a], part[k].box[3 + a]);
        }
        p.bad = std::min(p.bad, part[k].bad);
        p.flags |= part[k].flags;
    }
    return p;
}

}  // namespace vg
