// Gaussian voxel map construction (GLIM Sec. III-C, Preprocessing): every point
// x falls in voxel floor(x / r); a voxel stores the average of its points' means
// and the average of their covariances.
//
// Device pipeline, all levels of a map together (a level's pass over a submap is
// a few microseconds of work behind ~25 launches, so the launches are shared):
// one 64-bit word per (level, point) holding level | block | voxel in block |
// point -> one sort -> one scan that numbers the voxels and the blocks -> the
// level sizes go to the host (the build's only synchronization), one allocation
// -> voxel sums in ascending point order in FP64 (deterministic) -> records in
// three layouts -> open-addressing insert of the blocks with 64-bit atomicCAS.
// Bound by launches and their gaps.  A 128-ring sweep (four levels, 40k points)
// from raw points to its first linearization: 3.91 ms with two sorts, 25 launches,
// three synchronizations and 18 allocations per level, 2.96 ms with this.
#include <hipcub/hipcub.hpp>

#include <algorithm>
#include <climits>
#include <vector>

#include "vg_device.h"

namespace vg {

// One level as the build kernels see it.
struct BuildLevel {
    double r;
    int64_t K0[3];        // absolute key of the map origin
    int32_t bmin[3];      // first block per axis (biased block coordinates)
    int32_t wy, wz;       // bits of the block's y and z offsets in a code
    int32_t v0;           // first voxel of the level among all levels'
    uint32_t log2cap;
    uint64_t* slots;
    float* rec32;
    float* recN;
    double* rec64;
    uint64_t* keys;
    int32_t* counts;
};
struct BuildLevels {
    BuildLevel lv[kMaxLevels];
    int32_t L;
    int32_t code_bits;    // a code: level << code_bits | block offsets << 6 | voxel in the block
    int32_t idx_bits;     // low bits of a sort word that hold the point (0: a separate array)
};

// Voxel code of a biased voxel key inside a level: (block offsets from the
// level's first block) << 6 | position in the block.  Ascending codes are
// ascending blocks (x, y, z), voxels x fastest inside a block: record order.
__device__ __forceinline__ uint64_t voxel_code(const BuildLevel& b, uint32_t ux, uint32_t uy, uint32_t uz) {
    const uint64_t x = (ux >> kBlockShift) - (uint32_t)b.bmin[0], y = (uy >> kBlockShift) - (uint32_t)b.bmin[1],
                   z = (uz >> kBlockShift) - (uint32_t)b.bmin[2];
    return (((((x << b.wy) | y) << b.wz) | z) << 6) | block_local(ux, uy, uz);
}

__device__ __forceinline__ void code_key(const BuildLevel& b, uint64_t code, uint32_t u[3]) {
    const uint32_t local = (uint32_t)code & 63u;
    const uint64_t blk = code >> 6;
    const uint32_t z = (uint32_t)(blk & ((1ull << b.wz) - 1)), y = (uint32_t)((blk >> b.wz) & ((1ull << b.wy) - 1)),
                   x = (uint32_t)(blk >> (b.wz + b.wy));
    u[0] = ((x + (uint32_t)b.bmin[0]) << kBlockShift) | (local & 3u);
    u[1] = ((y + (uint32_t)b.bmin[1]) << kBlockShift) | ((local >> 2) & 3u);
    u[2] = ((z + (uint32_t)b.bmin[2]) << kBlockShift) | (local >> 4);
}

// Sort word of every (level, point).  Bound by its reads of xyz (24 B per point);
// the key range was checked on the host from the cloud's bounding box (floor and
// division are monotone), so nothing is flagged here.
__global__ void k_map_codes(const double* __restrict__ xyz, int64_t n, BuildLevels B, uint64_t* __restrict__ word,
                            int32_t* __restrict__ idx) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double x[3] = {xyz[3 * i], xyz[3 * i + 1], xyz[3 * i + 2]};
    for (int l = 0; l < B.L; ++l) {
        const BuildLevel& b = B.lv[l];
        uint32_t u[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) u[a] = (uint32_t)((int64_t)floor(x[a] / b.r) - b.K0[a] + kKeyBias);
        const uint64_t code = ((uint64_t)l << B.code_bits) | voxel_code(b, u[0], u[1], u[2]);
        word[(int64_t)l * n + i] = (code << B.idx_bits) | (B.idx_bits ? (uint64_t)i : 0ull);
        if (idx != nullptr) idx[(int64_t)l * n + i] = (int32_t)i;
    }
}

// Heads of the sorted words: 1 in the low word where a voxel starts, 1 in the
// high word where a block starts.
struct HeadOf {
    const uint64_t* word;
    int32_t idx_bits;
    __host__ __device__ uint64_t operator()(int64_t i) const {
        if (i == 0) return (1ull << 32) | 1ull;
        const uint64_t a = word[i - 1] >> idx_bits, b = word[i] >> idx_bits;
        return (a != b ? 1ull : 0ull) | ((a >> 6) != (b >> 6) ? 1ull << 32 : 0ull);
    }
};

// From the scanned heads: code and first element of every voxel, first voxel of
// every block; the first voxel and block of every level and the totals go to
// `info` (pinned host memory, read after the build's one synchronization).
__global__ void k_map_voxels(const uint64_t* __restrict__ word, const uint64_t* __restrict__ scan, int64_t n, int64_t N,
                             int32_t idx_bits, uint64_t* __restrict__ vcode, int32_t* __restrict__ vstart,
                             int32_t* __restrict__ bfirst, int32_t* __restrict__ info) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    const uint64_t s = scan[i], p = i > 0 ? scan[i - 1] : 0ull;
    const int32_t v = (int32_t)(uint32_t)s - 1, b = (int32_t)(s >> 32) - 1;
    if ((uint32_t)s != (uint32_t)p) {
        vcode[v] = word[i] >> idx_bits;
        vstart[v] = (int32_t)i;
        if ((s >> 32) != (p >> 32)) bfirst[b] = v;
    }
    if (i % n == 0) {
        info[2 * (i / n)] = v;
        info[2 * (i / n) + 1] = b;
    }
    if (i == N - 1) {
        vstart[v + 1] = (int32_t)N;
        bfirst[b + 1] = v + 1;
        info[2 * (N / n)] = v + 1;
        info[2 * (N / n) + 1] = b + 1;
    }
}

// Per-voxel statistics: FP64 sums of its points in ascending point order, then the
// average, written as records in record order.  Nine lanes per voxel, one per
// component (a point's 3 coordinates and 6 covariances are then two contiguous
// reads, and the serial FP64 chains of a voxel's components run side by side),
// with the loads of eight points in flight: a voxel's sum is a chain of dependent
// additions, and one thread per voxel with one load at a time spent it waiting
// (65-200 us a level for the coarse levels of a 32-ring sweep and for 1M points).
constexpr int kVoxPerWave = 7;
__global__ __launch_bounds__(256) void k_map_stats(const double* __restrict__ xyz, const double* __restrict__ cov,
                                                   const uint64_t* __restrict__ word, const int32_t* __restrict__ idx,
                                                   const uint64_t* __restrict__ vcode, const int32_t* __restrict__ vstart,
                                                   int32_t V, BuildLevels B) {
    const int lane = threadIdx.x & 63, g = lane / 9, k = lane % 9;
    const int64_t v = ((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * kVoxPerWave + g;
    if (g >= kVoxPerWave || v >= V) return;
    const uint64_t code = vcode[v];
    const int l = (int)(code >> B.code_bits);
    const BuildLevel& b = B.lv[l];
    const int32_t j0 = vstart[v], j1 = vstart[v + 1];
    const uint64_t mask = (1ull << B.idx_bits) - 1ull;
    const double* src = k < 3 ? xyz + k : cov + (k - 3);
    const int64_t stride = k < 3 ? 3 : 6;
    constexpr int kStep = 8;
    double s = 0.0;
    int32_t j = j0;
    for (; j + kStep <= j1; j += kStep) {
        double x[kStep];
#pragma unroll
        for (int q = 0; q < kStep; ++q) {
            const int64_t i = idx != nullptr ? (int64_t)idx[j + q] : (int64_t)(word[j + q] & mask);
            x[q] = src[stride * i];
        }
#pragma unroll
        for (int q = 0; q < kStep; ++q) s += x[q];
    }
    {
        double x[kStep - 1];
        const int rest = j1 - j;
#pragma unroll
        for (int q = 0; q < kStep - 1; ++q)
            if (q < rest) {
                const int64_t i = idx != nullptr ? (int64_t)idx[j + q] : (int64_t)(word[j + q] & mask);
                x[q] = src[stride * i];
            }
#pragma unroll
        for (int q = 0; q < kStep - 1; ++q)
            if (q < rest) s += x[q];
    }
    const int32_t cnt = j1 - j0;
    const double m = s / (double)cnt;
    uint32_t u[3];
    code_key(b, code & ((1ull << B.code_bits) - 1ull), u);
    const int64_t w = v - b.v0;
    b.rec64[kRec64 * w + k] = m;
    b.recN[kRecN * w + k] = (float)m;
    float* r32 = b.rec32 + kRec32 * w;
    if (k < 3) {
        const int64_t q = (int64_t)(k == 0 ? u[0] : (k == 1 ? u[1] : u[2])) - kKeyBias + b.K0[k];
        const double centre = (double)q * b.r + 0.5 * b.r;
        r32[k] = (float)(m - centre);
        b.recN[kRecN * w + 9 + k] = 0.f;
    } else {
        reinterpret_cast<double*>(r32 + 4)[k - 3] = m;   // covariance, FP64 (8-byte aligned: records are 64 B)
    }
    if (k == 0) {
        r32[3] = (float)cnt;
        b.rec64[kRec64 * w + 9] = 0.0;
        b.keys[w] = pack_key((int64_t)u[0] - kKeyBias, (int64_t)u[1] - kKeyBias, (int64_t)u[2] - kKeyBias);
        b.counts[w] = cnt;
    }
}

// One thread per occupied block: occupancy mask of its records, then insertion
// of (block key | first record, mask) into the block table of its level.
__global__ void k_map_blocks(const uint64_t* __restrict__ vcode, const int32_t* __restrict__ bfirst, int32_t NB,
                             BuildLevels B) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= NB) return;
    const int32_t v0 = bfirst[t], v1 = bfirst[t + 1];
    uint64_t occ = 0;
    for (int32_t v = v0; v < v1; ++v) occ |= 1ull << (vcode[v] & 63);
    const uint64_t code = vcode[v0];
    const BuildLevel& b = B.lv[code >> B.code_bits];
    uint32_t u[3];
    code_key(b, code & ((1ull << B.code_bits) - 1ull), u);
    const uint64_t key = block_key(u[0], u[1], u[2]);
    const uint64_t entry = (key << kBaseBits) | (uint64_t)(v0 - b.v0);
    const uint32_t mask = (1u << b.log2cap) - 1u;
    uint32_t h = slot_of(key, b.log2cap);
    for (uint32_t it = 0; it <= mask; ++it) {
        const unsigned long long prev = atomicCAS((unsigned long long*)(b.slots + 2 * (uint64_t)h),
                                                  (unsigned long long)kEmpty, (unsigned long long)entry);
        if (prev == (unsigned long long)kEmpty) {
            b.slots[2 * (uint64_t)h + 1] = occ;
            return;
        }
        h = (h + 1u) & mask;
    }
}

// 16-byte fill (table entries).
__global__ void k_fill_entries(u64x2* p, int64_t n, uint64_t v) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = u64x2{v, v};
}

__global__ void k_iota(int32_t* p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = (int32_t)i;
}

static int grid_of(int64_t n, int b = 256) { return (int)((n + b - 1) / b); }

static int bits_for(uint64_t max_value) {
    int b = 0;
    while (b < 64 && (max_value >> b) != 0) ++b;
    return b;
}

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Levels [l0, l0 + L) of a map, built together: box is the cloud's bounding box
// (min xyz, max xyz).  The arrays of these levels are one allocation, *block.
static vg_status build_levels(vg_context* ctx, Scratch& sc, const double* d_xyz, const double* d_cov, int64_t n,
                              const double box[6], Level* lv, int L, void** block) {
    hipStream_t st = ctx->stream;
    BuildLevels B{};
    B.L = L;
    int code_bits = 0;
    for (int l = 0; l < L; ++l) {
        Level& q = lv[l];
        BuildLevel& b = B.lv[l];
        b.r = q.r;
        int32_t nb[3];
        for (int a = 0; a < 3; ++a) {
            b.K0[a] = q.K0[a];
            const double lo = std::floor(box[a] / q.r), hi = std::floor(box[3 + a] / q.r);
            // the difference to the origin's key in double first: it may not fit an integer
            if (!(lo - (double)q.K0[a] >= -(double)kKeyBias && hi - (double)q.K0[a] < (double)kKeyBias)) {
                set_error("voxel key outside the packable range (|q - q_origin| >= 8192 voxels on an axis)");
                return VG_ERR_KEY_RANGE;
            }
            q.kmin[a] = (int32_t)((int64_t)lo - q.K0[a]);
            q.kmax[a] = (int32_t)((int64_t)hi - q.K0[a]);
            b.bmin[a] = (q.kmin[a] + kKeyBias) >> kBlockShift;
            nb[a] = ((q.kmax[a] + kKeyBias) >> kBlockShift) - b.bmin[a];
        }
        b.wy = bits_for((uint64_t)nb[1]);
        b.wz = bits_for((uint64_t)nb[2]);
        code_bits = std::max(code_bits, bits_for((uint64_t)nb[0]) + b.wy + b.wz + 6);
    }
    const int64_t N = n * L;
    B.code_bits = code_bits;
    const int word_bits = code_bits + bits_for((uint64_t)(L - 1));
    const int ib = bits_for((uint64_t)(n - 1));
    // the point rides in the word's low bits where they fit (a stable sort by code
    // in one array); otherwise words and points are sorted as pairs
    const bool packed = word_bits + ib <= 64;
    B.idx_bits = packed ? ib : 0;
    uint64_t *w0, *w1, *scan, *vcode;
    int32_t *i0 = nullptr, *i1 = nullptr, *vstart, *bfirst;
    VG_HIP(sc.get(&w0, N));
    VG_HIP(sc.get(&w1, N));
    VG_HIP(sc.get(&scan, N));
    VG_HIP(sc.get(&vcode, N));
    VG_HIP(sc.get(&vstart, N + 1));
    VG_HIP(sc.get(&bfirst, N + 1));
    if (!packed) {
        VG_HIP(sc.get(&i0, N));
        VG_HIP(sc.get(&i1, N));
    }
    const int end_bit = std::max(1, word_bits + B.idx_bits);
    size_t b1 = 0, b2 = 0;
    const hipcub::CountingInputIterator<int64_t> cnt(0);
    const hipcub::TransformInputIterator<uint64_t, HeadOf, hipcub::CountingInputIterator<int64_t>> heads(
        cnt, HeadOf{w1, B.idx_bits});
    if (packed) (void)hipcub::DeviceRadixSort::SortKeys(nullptr, b1, w0, w1, (int)N, B.idx_bits, end_bit);
    else (void)hipcub::DeviceRadixSort::SortPairs(nullptr, b1, w0, w1, i0, i1, (int)N, 0, end_bit);
    (void)hipcub::DeviceScan::InclusiveSum(nullptr, b2, heads, scan, (int)N);
    size_t tmp_bytes = std::max(b1, b2) + 256;
    char* tmp = nullptr;
    VG_HIP(sc.get(&tmp, tmp_bytes));
    k_map_codes<<<grid_of(n), 256, 0, st>>>(d_xyz, n, B, w0, i0);
    VG_HIP(hipGetLastError());
    size_t tb = tmp_bytes;
    if (packed) VG_HIP(hipcub::DeviceRadixSort::SortKeys(tmp, tb, w0, w1, (int)N, B.idx_bits, end_bit, st));
    else VG_HIP(hipcub::DeviceRadixSort::SortPairs(tmp, tb, w0, w1, i0, i1, (int)N, 0, end_bit, st));
    tb = tmp_bytes;
    VG_HIP(hipcub::DeviceScan::InclusiveSum(tmp, tb, heads, scan, (int)N, st));
    int32_t* info = ctx->h_small;
    k_map_voxels<<<grid_of(N), 256, 0, st>>>(w1, scan, n, N, B.idx_bits, vcode, vstart, bfirst, info);
    VG_HIP(hipGetLastError());
    VG_HIP(hipStreamSynchronize(st));
    size_t bytes = 0;
    const int32_t V_all = info[2 * L], NB_all = info[2 * L + 1];
    for (int l = 0; l < L; ++l) {
        Level& q = lv[l];
        q.V = info[2 * (l + 1)] - info[2 * l];
        q.n_blocks = info[2 * (l + 1) + 1] - info[2 * l + 1];
        if (q.V > kMaxVoxels) {
            set_error("too many voxels in one level");
            return VG_ERR_CAPACITY;
        }
        B.lv[l].v0 = info[2 * l];
        // block table: power of two >= 4 x blocks (load factor <= 1/4)
        uint32_t lg = 6;
        while ((1ull << lg) < 4ull * (uint64_t)q.n_blocks) ++lg;
        q.log2cap = lg;
        bytes += 16ull << lg;
    }
    const size_t table_bytes = bytes;   // every level's table first, so that one fill covers them
    for (int l = 0; l < L; ++l)
        bytes += align256(4 * kRec32 * (size_t)lv[l].V) + align256(4 * kRecN * (size_t)lv[l].V) +
                 align256(8 * kRec64 * (size_t)lv[l].V) + align256(8 * (size_t)lv[l].V) + align256(4 * (size_t)lv[l].V);
    VG_HIP(ctx->pool->get(block, bytes));
    char* p = (char*)*block;
    for (int l = 0; l < L; ++l) {
        lv[l].slots = (uint64_t*)p;
        p += 16ull << lv[l].log2cap;
    }
    for (int l = 0; l < L; ++l) {
        Level& q = lv[l];
        const size_t V = (size_t)q.V;
        auto take = [&](size_t b) { char* r = p; p += align256(b); return r; };
        q.rec32 = (float*)take(4 * kRec32 * V);
        q.recN = (float*)take(4 * kRecN * V);
        q.rec64 = (double*)take(8 * kRec64 * V);
        q.keys = (uint64_t*)take(8 * V);
        q.counts = (int32_t*)take(4 * V);
        BuildLevel& b = B.lv[l];
        b.log2cap = q.log2cap;
        b.slots = q.slots;
        b.rec32 = q.rec32;
        b.recN = q.recN;
        b.rec64 = q.rec64;
        b.keys = q.keys;
        b.counts = q.counts;
    }
    k_fill_entries<<<grid_of((int64_t)(table_bytes / 16)), 256, 0, st>>>((u64x2*)*block, (int64_t)(table_bytes / 16), kEmpty);
    VG_HIP(hipGetLastError());
    k_map_stats<<<grid_of(V_all, 4 * kVoxPerWave), 256, 0, st>>>(d_xyz, d_cov, w1, i1, vcode, vstart, V_all, B);
    VG_HIP(hipGetLastError());
    k_map_blocks<<<grid_of(NB_all), 256, 0, st>>>(vcode, bfirst, NB_all, B);
    VG_HIP(hipGetLastError());
    return VG_OK;
}

vg_status build_map(vg_context* ctx, Scratch& sc, const double* d_xyz, const double* d_cov, int64_t n,
                    const double box[6], const double* resolutions, int L, vg_voxelmap* m) {
    for (int l = 0; l < L; ++l) {
        m->lv[l].r = resolutions[l];
        for (int a = 0; a < 3; ++a) m->lv[l].K0[a] = (int64_t)llround(m->origin[a] / resolutions[l]);
    }
    if (n == 0) {
        constexpr size_t kTable = 16 * 64;
        VG_HIP(ctx->pool->get(&m->blocks[0], kTable * L));
        k_fill_entries<<<1, 64 * L, 0, ctx->stream>>>((u64x2*)m->blocks[0], 64 * L, kEmpty);
        VG_HIP(hipGetLastError());
        for (int l = 0; l < L; ++l) {
            m->lv[l].log2cap = 6;
            m->lv[l].slots = (uint64_t*)((char*)m->blocks[0] + kTable * l);
        }
        return VG_OK;
    }
    // all levels in one go; clouds too large for the library's 32-bit item counts, or
    // whose temporaries for all levels (50 B a point and level) do not fit, level by level
    if (n * L < (int64_t)1 << 30) {
        vg_status rc;
        {
            Scratch all(&sc);
            rc = build_levels(ctx, all, d_xyz, d_cov, n, box, m->lv, L, &m->blocks[0]);
        }
        if (rc != VG_ERR_OOM || L == 1) return rc;
        set_error("");
    }
    for (int l = 0; l < L; ++l) {
        Scratch one(&sc);
        const vg_status rc = build_levels(ctx, one, d_xyz, d_cov, n, box, m->lv + l, 1, &m->blocks[l]);
        if (rc != VG_OK) return rc;
    }
    return VG_OK;
}

// Order of a small level's records by key, on the host: the key's offset in the level's
// key box, sorted by digits from the lowest.
static void order_on_host(const Level& lv, const std::vector<uint64_t>& keys, std::vector<int32_t>& order) {
    const size_t V = keys.size();
    const int by = bits_for((uint64_t)(lv.kmax[1] - lv.kmin[1])), bz = bits_for((uint64_t)(lv.kmax[2] - lv.kmin[2]));
    const int bits = bits_for((uint64_t)(lv.kmax[0] - lv.kmin[0])) + by + bz;
    std::vector<uint64_t> code(V), code2(V);
    std::vector<int32_t> order2(V);
    for (size_t v = 0; v < V; ++v) {
        int64_t q[3];
        unpack_key(keys[v], q);
        code[v] = ((((uint64_t)(q[0] - lv.kmin[0]) << by) | (uint64_t)(q[1] - lv.kmin[1])) << bz) |
                  (uint64_t)(q[2] - lv.kmin[2]);
        order[v] = (int32_t)v;
    }
    constexpr int kDigit = 10;
    for (int s = 0; s < bits; s += kDigit) {
        uint32_t at[1 << kDigit] = {};
        for (size_t v = 0; v < V; ++v) ++at[(code[v] >> s) & ((1u << kDigit) - 1)];
        uint32_t sum = 0;
        for (uint32_t& n : at) {
            const uint32_t k = n;
            n = sum;
            sum += k;
        }
        for (size_t v = 0; v < V; ++v) {
            const uint32_t to = at[(code[v] >> s) & ((1u << kDigit) - 1)]++;
            code2[to] = code[v];
            order2[to] = order[v];
        }
        code.swap(code2);
        order.swap(order2);
    }
}

// A level in canonical order (ascending lexicographic key): its records are in
// block order, and no kernel needs the canonical one, so the rows are ordered here:
// levels of up to kHostOrder voxels on the host, where a sort's launches on the
// device take longer (2,000 voxels: 66 us a call, 130 us on the device; 15,500: 362
// and 414; 31,000: 696 and 691).
constexpr int64_t kHostOrder = 1 << 14;
vg_status export_level(vg_context* ctx, const Level& lv, int64_t* keys, double* means, double* covs,
                       int64_t* counts) {
    hipStream_t st = ctx->stream;
    const int64_t V = lv.V;
    if (V == 0) return VG_OK;
    std::vector<uint64_t> k((size_t)V);
    std::vector<int32_t> c((size_t)V), l2r((size_t)V);
    std::vector<double> r((size_t)V * kRec64);
    Scratch sc(ctx);
    if (V > kHostOrder) {
        uint64_t* ks = nullptr;
        int32_t *id = nullptr, *order = nullptr;
        char* tmp = nullptr;
        size_t tb = 0;
        (void)hipcub::DeviceRadixSort::SortPairs(nullptr, tb, lv.keys, ks, id, order, (int)V, 0, 3 * kKeyBits);
        VG_HIP(sc.get(&ks, V));
        VG_HIP(sc.get(&id, V));
        VG_HIP(sc.get(&order, V));
        VG_HIP(sc.get(&tmp, tb + 256));
        k_iota<<<grid_of(V), 256, 0, st>>>(id, V);
        VG_HIP(hipGetLastError());
        tb += 256;
        VG_HIP(hipcub::DeviceRadixSort::SortPairs(tmp, tb, lv.keys, ks, id, order, (int)V, 0, 3 * kKeyBits, st));
        VG_HIP(hipMemcpyAsync(l2r.data(), order, sizeof(int32_t) * V, hipMemcpyDeviceToHost, st));
    }
    VG_HIP(hipMemcpyAsync(k.data(), lv.keys, sizeof(uint64_t) * V, hipMemcpyDeviceToHost, st));
    VG_HIP(hipMemcpyAsync(c.data(), lv.counts, sizeof(int32_t) * V, hipMemcpyDeviceToHost, st));
    VG_HIP(hipMemcpyAsync(r.data(), lv.rec64, sizeof(double) * kRec64 * V, hipMemcpyDeviceToHost, st));
    VG_HIP(hipStreamSynchronize(st));
    if (V <= kHostOrder) order_on_host(lv, k, l2r);
    for (int64_t v = 0; v < V; ++v) {
        int64_t q[3];
        const int64_t w = l2r[v];
        unpack_key(k[w], q);
        if (keys)
            for (int a = 0; a < 3; ++a) keys[3 * v + a] = q[a] + lv.K0[a];
        if (means)
            for (int a = 0; a < 3; ++a) means[3 * v + a] = r[kRec64 * w + a];
        if (covs)
            for (int a = 0; a < 6; ++a) covs[6 * v + a] = r[kRec64 * w + 3 + a];
        if (counts) counts[v] = c[w];
    }
    return VG_OK;
}

void free_map(vg_voxelmap* m) {
    for (int l = 0; l < kMaxLevels; ++l) {
        if (m->blocks[l]) m->pool->put(m->blocks[l]);
        m->blocks[l] = nullptr;
        m->lv[l] = Level{};
    }
}

// ---------------------------------------------------------------- source clouds

__device__ __forceinline__ uint64_t spread21(uint64_t v) {
    uint64_t x = v & 0x1fffffull;
    x = (x | (x << 32)) & 0x1f00000000ffffull;
    x = (x | (x << 16)) & 0x1f0000ff0000ffull;
    x = (x | (x << 8)) & 0x100f00f00f00f00full;
    x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

// Sort word of a point: the Morton code of its 0.25 m cell around the source
// origin (21 bits per axis, offset by 2^20), with the point in the low idx_bits.
// Only `keep` bits per axis and the offset's top bit are interleaved: the bits
// between are the complement of the top bit for every cell of the cloud, so they
// never decide between two codes that agree above them, and the order is the full
// code's.  idx: the points as a separate array where they don't fit the word.
__global__ void k_morton(const double* __restrict__ xyz, int64_t n, double ox, double oy, double oz, int32_t keep,
                         int32_t idx_bits, uint64_t* __restrict__ word, int32_t* __restrict__ idx) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double o[3] = {ox, oy, oz};
    uint64_t q[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double c = floor((xyz[3 * i + a] - o[a]) * 4.0) + 1048576.0;
        c = fmin(fmax(c, 0.0), 2097151.0);
        const uint64_t u = (uint64_t)c;
        q[a] = keep >= 20 ? u : ((u >> 20) << keep) | (u & ((1ull << keep) - 1ull));
    }
    const uint64_t code = (spread21(q[0]) << 2) | (spread21(q[1]) << 1) | spread21(q[2]);
    word[i] = (code << idx_bits) | (idx_bits ? (uint64_t)i : 0ull);
    if (idx != nullptr) idx[i] = (int32_t)i;
}

// FP32 value >= x (round up).
__device__ __forceinline__ float f32_up(double x) {
    float f = (float)x;
    if ((double)f < x) f = nextafterf(f, INFINITY);
    return f;
}

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o));
    return v;
}

// Bounds of one chunk from the FP32 offsets the kernels read, one point per lane
// of a wave: a ball around the anchor (radius bounds every point's distance) and
// an axis-aligned box in the source frame (centre offset from the anchor, half
// extents bounding every point).  Returns the radius.
__device__ __forceinline__ float chunk_bounds(const float d[3], bool live, int lane, float* __restrict__ o) {
    const double x[3] = {d[0], d[1], d[2]};
    const double m = fmax(0.0, wave_max(live ? x[0] * x[0] + x[1] * x[1] + x[2] * x[2] : 0.0));
    float ctr[3], half[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double lo = wave_min(live ? x[a] : INFINITY), hi = wave_max(live ? x[a] : -INFINITY);
        ctr[a] = (float)(0.5 * (lo + hi));
        half[a] = f32_up(fmax(hi - (double)ctr[a], (double)ctr[a] - lo));
    }
    const float rad = f32_up(sqrt(m));
    if (lane < 8) {
        const float v = lane == 0 ? ctr[0] : lane == 1 ? ctr[1] : lane == 2 ? ctr[2] : lane == 3 ? rad
                      : lane == 4 ? half[0] : lane == 5 ? half[1] : lane == 6 ? half[2] : 0.f;
        o[lane] = v;
    }
    return rad;
}

// Value of lane i (uniform).
__device__ __forceinline__ double lane_value(double v, int i) {
    const uint64_t u = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, i),
                   hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), i);
    return __longlong_as_double((int64_t)(((uint64_t)hi << 32) | lo));
}

// Layout of a source, one wave per 64-point chunk: its points in Morton order
// (gathered by row), the anchor (the centroid, FP64 sum in that order: keeps the
// FP32 offsets, and so their rounding, as small as the chunk allows), every array,
// the chunk's bounds, and an upper bound of its points' distance from the source
// origin.  Bound by its ~300 B per point of reads and writes.  The anchors and
// bounds were passes of their own with one thread per chunk, whose serial walk
// over 64 strided points took 44 and 24 us at any size.
__global__ __launch_bounds__(256) void k_layout(const double* __restrict__ xyz, const double* __restrict__ cov,
                                                const double* __restrict__ nrm, const uint64_t* __restrict__ word,
                                                const int32_t* __restrict__ idx, int32_t idx_bits, int64_t n,
                                                int64_t n_pad, double ox, double oy, double oz,
                                                float* __restrict__ dxyz, float* __restrict__ cov32,
                                                float* __restrict__ nrm32, double* __restrict__ anchor,
                                                float* __restrict__ cbound, float* __restrict__ axyz,
                                                double* __restrict__ xyz64, double* __restrict__ cov64,
                                                double* __restrict__ nrm64, int32_t* __restrict__ perm,
                                                double* __restrict__ extent, PointSrc* __restrict__ self, PointSrc me) {
    const int lane = threadIdx.x & 63;
    const int64_t c = (int64_t)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t i = c * kChunk + lane;
    if (c * kChunk >= n_pad) return;
    const int npts = (int)min<int64_t>(kChunk, n - c * kChunk);
    const bool live = lane < npts;
    int64_t s = 0;
    double x[3] = {0.0, 0.0, 0.0};
    if (live) {
        s = idx != nullptr ? (int64_t)idx[i] : (int64_t)(word[i] & ((1ull << idx_bits) - 1ull));
#pragma unroll
        for (int a = 0; a < 3; ++a) x[a] = xyz[3 * s + a];
    }
    double an[3] = {0.0, 0.0, 0.0};
    for (int k = 0; k < npts; ++k) {
#pragma unroll
        for (int a = 0; a < 3; ++a) an[a] += lane_value(x[a], k);
    }
    const double inv = 1.0 / (double)npts;
    float d[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        an[a] *= inv;
        asm("" : "+v"(an[a]));   // the offsets are taken from the rounded anchor, not from a fused product
        d[a] = live ? (float)(x[a] - an[a]) : 0.f;
        dxyz[a * n_pad + i] = d[a];
        axyz[a * n_pad + i] = live ? (float)x[a] : 0.f;
        xyz64[a * n_pad + i] = x[a];
    }
    perm[i] = live ? (int32_t)s : -1;
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const double v = live ? cov[6 * s + k] : 0.0;
        cov32[k * n_pad + i] = (float)v;
        cov64[k * n_pad + i] = v;
    }
    if (nrm != nullptr) {
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double v = live ? nrm[3 * s + a] : 0.0;
            nrm32[a * n_pad + i] = (float)v;
            nrm64[a * n_pad + i] = v;
        }
    }
    const float rad = chunk_bounds(d, live, lane, cbound + 8 * c);
    if (lane < 3) anchor[3 * c + lane] = lane == 0 ? an[0] : lane == 1 ? an[1] : an[2];
    if (lane == 0) {
        const double e0 = an[0] - ox, e1 = an[1] - oy, e2 = an[2] - oz;
        extent[c] = sqrt(e0 * e0 + e1 * e1 + e2 * e2) + (double)rad;
        if (c == 0) *self = me;
    }
}

// Largest of n values (n >= 1), to pinned host memory; one workgroup.
__global__ __launch_bounds__(1024) void k_max(const double* __restrict__ v, int64_t n, double* __restrict__ out) {
    __shared__ double s[16];
    double m = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) m = fmax(m, v[i]);
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 16; ++w) m = fmax(m, s[w]);
        *out = m;
    }
}

vg_status layout_source(vg_context* ctx, Scratch& sc, vg_source* s, const double* d_xyz, const double* d_cov,
                        const double* d_nrm, const double box[6]) {
    hipStream_t st = ctx->stream;
    const int64_t n = s->n, n_pad = s->n_pad;
    if (n == 0) return VG_OK;
    // low bits per axis that hold every cell's distance from the origin's cell
    int keep = 0;
    for (int a = 0; a < 3; ++a) {
        const double lo = std::floor((box[a] - s->origin[a]) * 4.0), hi = std::floor((box[3 + a] - s->origin[a]) * 4.0);
        while (keep < 20 && !(lo >= -(double)(1ll << keep) && hi < (double)(1ll << keep))) ++keep;
    }
    const int code_bits = 3 * (keep + 1), ib = bits_for((uint64_t)(n - 1));
    const bool packed = code_bits + ib <= 64;
    const int idx_bits = packed ? ib : 0;
    uint64_t *w0, *w1;
    int32_t *i0 = nullptr, *i1 = nullptr;
    double* ext;
    VG_HIP(sc.get(&w0, n));
    VG_HIP(sc.get(&w1, n));
    VG_HIP(sc.get(&ext, s->n_chunks));
    if (!packed) {
        VG_HIP(sc.get(&i0, n));
        VG_HIP(sc.get(&i1, n));
    }
    const int end_bit = code_bits + idx_bits;
    size_t tb = 0;
    if (packed) (void)hipcub::DeviceRadixSort::SortKeys(nullptr, tb, w0, w1, (int)n, idx_bits, end_bit);
    else (void)hipcub::DeviceRadixSort::SortPairs(nullptr, tb, w0, w1, i0, i1, (int)n, 0, end_bit);
    char* tmp = nullptr;
    tb += 256;
    VG_HIP(sc.get(&tmp, tb));
    k_morton<<<grid_of(n), 256, 0, st>>>(d_xyz, n, s->origin[0], s->origin[1], s->origin[2], keep, idx_bits, w0, i0);
    VG_HIP(hipGetLastError());
    if (packed) VG_HIP(hipcub::DeviceRadixSort::SortKeys(tmp, tb, w0, w1, (int)n, idx_bits, end_bit, st));
    else VG_HIP(hipcub::DeviceRadixSort::SortPairs(tmp, tb, w0, w1, i0, i1, (int)n, 0, end_bit, st));
    k_layout<<<grid_of(s->n_chunks, 4), 256, 0, st>>>(d_xyz, d_cov, d_nrm, w1, i1, idx_bits, n, n_pad, s->origin[0],
                                                      s->origin[1], s->origin[2], s->dxyz, s->cov, s->nrm, s->anchor,
                                                      s->cbound, s->axyz, s->xyz64, s->cov64, s->nrm64, s->perm, ext, s->self,
                                                      PointSrc{s->dxyz, s->axyz, s->xyz64, s->perm, s->anchor, s->cbound, n, n_pad, 0});
    VG_HIP(hipGetLastError());
    double* h = reinterpret_cast<double*>(ctx->h_small);
    k_max<<<1, 1024, 0, st>>>(ext, s->n_chunks, h);
    VG_HIP(hipGetLastError());
    VG_HIP(hipStreamSynchronize(st));
    s->extent = h[0];
    return VG_OK;
}

// New positions of sources and their chunk bounds, one wave per chunk: the offsets
// are taken from the kept anchors, and the bounds from the offsets while they are
// in registers.  A source's rows start at row0 of `in`.  Bound by its ~70 B per
// point, 12 or 24 of them gathered in the sources' order of chunks: a line of `in`
// holds rows of many chunks, so the workgroups are numbered in eight contiguous
// ranges, one per XCD, and the lines of a source are fetched by one L2 only; the
// absolute positions, which the compensated kernels do not read, are stored past the
// caches and leave them to `in` and the offsets.  One launch for all sources of a
// batch (nb workgroups each); 64 sources of 100k points, a call: 126 us (0.41 GB),
// 149 us with ordinary stores and 155 us without the ranges too.
template <typename S>
__global__ __launch_bounds__(256) void k_set_points(const S* __restrict__ in, const PointSrc* __restrict__ src,
                                                    uint32_t nb, uint32_t n_items) {
    const uint32_t per = (n_items + kParts - 1) / kParts;
    const uint32_t item = (blockIdx.x % kParts) * per + blockIdx.x / kParts;
    if (blockIdx.x / kParts >= per || item >= n_items) return;
    const PointSrc q = src[item / nb];
    const int lane = threadIdx.x & 63;
    const int64_t c = (int64_t)(item % nb) * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t i = c * kChunk + lane;
    if (c * kChunk >= q.n) return;
    const bool live = i < q.n;
    float d[3] = {0.f, 0.f, 0.f};
    if (live) {
        const int64_t s = q.row0 + q.perm[i];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double x = (double)in[3 * s + a];
            d[a] = (float)(x - q.anchor[3 * c + a]);
            q.dxyz[a * q.n_pad + i] = d[a];
            __builtin_nontemporal_store((float)x, q.axyz + a * q.n_pad + i);
            __builtin_nontemporal_store(x, q.xyz64 + a * q.n_pad + i);
        }
    }
    chunk_bounds(d, live, lane, q.cbound + 8 * c);
}

vg_status set_points(vg_context* ctx, const PointSrc* d_src, int64_t n_src, int64_t max_chunks, const void* d_xyz,
                     int dtype) {
    if (max_chunks <= 0) return VG_OK;
    const int64_t nb = (max_chunks + 3) / 4;   // workgroups per source
    const int64_t step = std::max<int64_t>(1, (1ll << 22) / nb);
    for (int64_t s0 = 0; s0 < n_src; s0 += step) {
        const uint32_t items = (uint32_t)(nb * std::min(step, n_src - s0));
        const unsigned grid = (unsigned)(kParts * ((items + kParts - 1) / kParts));
        if (dtype == 0)
            k_set_points<float><<<grid, 256, 0, ctx->stream>>>((const float*)d_xyz, d_src + s0, (uint32_t)nb, items);
        else
            k_set_points<double><<<grid, 256, 0, ctx->stream>>>((const double*)d_xyz, d_src + s0, (uint32_t)nb, items);
        VG_HIP(hipGetLastError());
    }
    return VG_OK;
}

}  // namespace vg
