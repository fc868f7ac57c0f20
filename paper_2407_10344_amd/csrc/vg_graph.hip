// Two-node expansion of linearized factors and device assembly of the
// block-sparse normal equations of a pose graph (GLIM Sec. III-C: a matching
// cost factor between poses T_i and T_j yields H_ii, H_ij, H_jj, b_i, b_j).
//
// A factor's relative pose is T = T_j^-1 T_i (source node i, target node j).
// With right perturbations T_i Exp(xi_i), T_j Exp(xi_j), the relative tangent is
// xi = xi_i - Ad(T^-1) xi_j to first order, so with A = Ad(T^-1):
//   H_ii = H, H_ij = -H A, H_ji = H_ij^T, H_jj = A^T H A, b_i = b, b_j = -A^T b.
//
// Assembly is deterministic: every block of the BSR matrix has a fixed list of
// contributions (built on the host, in factor order), summed in that order in
// FP64.  A node's diagonal block has one contribution per factor of the node, so
// the node's entries of the right-hand side are summed along with it.
#include <algorithm>
#include <map>

#include "vg_device.h"
#include "vg_timeline.h"

struct vg_graph {
    vg_context* ctx = nullptr;
    int64_t N = 0, F = 0, nnzb = 0;
    int64_t longest = 0;                     // contributions of a block at most
    std::vector<int64_t> row_ptr, col_idx;   // BSR structure (host copy)
    // contributions: per block slot, a list of (factor, kind); kind 0 ii, 1 ij, 2 ji, 3 jj
    int32_t* d_blk_ptr = nullptr;   // nnzb + 1
    int32_t* d_blk_item = nullptr;  // packed (factor << 2 | kind)
    int32_t* d_blk_node = nullptr;  // nnzb: the node of a diagonal block, else -1
    uint32_t magic = 0;
};

namespace vg {

// Entry (i, j) of A = Ad(T^-1) for T = (R, t): T^-1 = (R', t') = (R^T, -R^T t) and
// Ad = [[R', 0], [(t')x R', R']].  P (uniform): R row-major, t.
__device__ __forceinline__ double adjoint_entry(const double* __restrict__ P, int i, int j) {
    const int i3 = i % 3, j3 = j % 3;
    // column j3 of R' is row j3 of R
    const double c0 = j3 == 0 ? P[0] : (j3 == 1 ? P[3] : P[6]);
    const double c1 = j3 == 0 ? P[1] : (j3 == 1 ? P[4] : P[7]);
    const double c2 = j3 == 0 ? P[2] : (j3 == 1 ? P[5] : P[8]);
    double tp[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) tp[a] = -(P[a] * P[9] + P[3 + a] * P[10] + P[6 + a] * P[11]);
    const double x0 = i3 == 0 ? 0.0 : (i3 == 1 ? tp[2] : -tp[1]);
    const double x1 = i3 == 0 ? -tp[2] : (i3 == 1 ? 0.0 : tp[0]);
    const double x2 = i3 == 0 ? tp[1] : (i3 == 1 ? -tp[0] : 0.0);
    const double low = (x0 * c0 + x1 * c1) + x2 * c2;
    const double rot = i3 == 0 ? c0 : (i3 == 1 ? c1 : c2);
    return (i < 3) == (j < 3) ? rot : (i < 3 ? 0.0 : low);
}

// One workgroup per BSR block: its contributions are dealt to the waves in rounds of
// WAVES, lane k < 36 of a wave making entry (k / 6, k % 6) of one contribution
// and, for a diagonal block, lanes 36..41 the node's right-hand side; the workgroup
// adds a round's contributions in list order.  Bound by the chain of dependent
// loads (list, factor row, pose) of the longest list, so the list is read once by
// the lanes and, with four waves, the rounds are few: a node of 20 factors takes
// five.  Making A in place (a few selects and nine multiply-adds per lane) leaves no
// launch and no buffer for it.  500 nodes, 5,000 factors: 55 us a call with separate
// kernels for A, blocks and right-hand side, 45 us so, most of it the host ordering
// the two streams.
// A graph of many blocks fills the device however long a chain takes, and most of its
// blocks have one contribution, which leaves three of four waves idle: a block costs
// 0.75 ns with one wave and 1.6 ns with four, a contribution of the longest list 0.73
// and 0.22 us.  So one wave from 600 blocks per contribution on: 20,000 nodes and
// 200,000 factors (248,000 blocks, lists of 42) 184 us (four waves 406), 25,000 blocks
// with lists of 34 41 us (49); four waves for 12,000 blocks with lists of 34, 23 us
// (one 25), and for 600 nodes all to all (360,000 blocks, lists of 599), 641 us (755).
constexpr int64_t kBlocksPerContribution = 600;
template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void k_graph_assemble(
    const int32_t* __restrict__ blk_ptr, const int32_t* __restrict__ blk_item, const int32_t* __restrict__ blk_node,
    const double* __restrict__ poses, const double* __restrict__ lin, double* __restrict__ values,
    double* __restrict__ rhs, int64_t n_blocks) {
    __shared__ double sH[WAVES][36], sA[WAVES][36], sHA[WAVES][36], sB[WAVES][6], sV[2][WAVES][42];
    for (int64_t s = blockIdx.x; s < n_blocks; s += gridDim.x) {
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int r = lane / 6, c = lane % 6;   // of lanes 0..35; r == 6: the right-hand side
        const int32_t i0 = blk_ptr[s], i1 = blk_ptr[s + 1];
        const int32_t node = blk_node[s];
        double acc = 0.0;
        int buf = 0;
        for (int32_t base = i0; base < i1; base += 64) {
            const int32_t mine = base + lane < i1 ? blk_item[base + lane] : 0;
            const int cnt = min(64, i1 - base);
            for (int k0 = 0; k0 < cnt; k0 += WAVES, buf ^= 1) {
                const int k = k0 + wave;
                if (k < cnt) {   // uniform per wave
                    const int32_t item = __builtin_amdgcn_readlane(mine, k);
                    const int64_t f = item >> 2;
                    const int kind = item & 3;
                    const double* row = lin + (int64_t)kOutRow * f + 1;   // H (36), b (6)
                    const double h = lane < 42 ? row[lane] : 0.0;
                    double v = h;   // kind 0: H and b
                    if (kind != 0) {
                        if (lane < 36) {
                            sA[wave][lane] = adjoint_entry(poses + 12 * f, r, c);
                            sH[wave][lane] = h;
                        } else if (lane < 42) {
                            sB[wave][c] = h;
                        }
                        __builtin_amdgcn_wave_barrier();
                        if (lane < 36) {   // H A
                            double x = 0.0;
#pragma unroll
                            for (int q = 0; q < 6; ++q) x += sH[wave][6 * r + q] * sA[wave][6 * q + c];
                            sHA[wave][lane] = x;
                        }
                        __builtin_amdgcn_wave_barrier();
                        if (lane < 36) {
                            if (kind == 3) {          // A^T (H A)
                                v = 0.0;
#pragma unroll
                                for (int p = 0; p < 6; ++p) v += sA[wave][6 * p + r] * sHA[wave][6 * p + c];
                            } else {                  // -H A or its transpose
                                v = -sHA[wave][kind == 1 ? lane : 6 * c + r];
                            }
                        } else if (lane < 42) {       // -A^T b (used for kind 3)
                            double x = 0.0;
#pragma unroll
                            for (int q = 0; q < 6; ++q) x += sA[wave][6 * q + c] * sB[wave][q];
                            v = -x;
                        }
                    }
                    if (lane < 42) sV[buf][wave][lane] = v;
                }
                __syncthreads();   // (the sums of the round before last are done with this half of sV)
                if (threadIdx.x < 42) {
                    for (int w = 0; w < min(WAVES, cnt - k0); ++w) acc += sV[buf][w][threadIdx.x];
                }
            }
        }
        if (threadIdx.x < 36) values[36 * s + threadIdx.x] = acc;
        else if (threadIdx.x < 42 && node >= 0) rhs[6 * (int64_t)node + threadIdx.x - 36] = acc;
        __syncthreads();   // the next block's rounds start on the same half of sV
    }
}

}  // namespace vg

using namespace vg;

namespace {
constexpr uint32_t kGraphMagic = 0x62A90001u;
bool graph_ok(const vg_graph* g) { return g != nullptr && g->magic == kGraphMagic; }
vg_status g_invalid(const char* m) {
    set_error(m);
    return VG_ERR_INVALID_ARG;
}
void graph_free(vg_graph* g) {
    if (g->d_blk_ptr) (void)hipFree(g->d_blk_ptr);
    if (g->d_blk_item) (void)hipFree(g->d_blk_item);
    if (g->d_blk_node) (void)hipFree(g->d_blk_node);
}
template <typename T>
hipError_t up(T** d, const std::vector<T>& h) {
    hipError_t e = device_alloc((void**)d, sizeof(T) * std::max<size_t>(h.size(), 1));
    if (e == hipSuccess && !h.empty()) e = hipMemcpy(*d, h.data(), sizeof(T) * h.size(), hipMemcpyHostToDevice);
    return e;
}
}  // namespace

extern "C" vg_status vg_create_graph(vg_context* ctx, int64_t N, int64_t F, const int64_t* node_i,
                                     const int64_t* node_j, vg_graph** out) try {
    set_error("");
    if (!context_ok(ctx)) {
        set_error("invalid context");
        return VG_ERR_STATE;
    }
    if (out == nullptr) return g_invalid("out is NULL");
    *out = nullptr;
    if (N < 1 || F < 0 || N >= (1ll << 30) || F >= (1ll << 29)) return g_invalid("N or F out of range");
    if (F > 0 && (node_i == nullptr || node_j == nullptr)) return g_invalid("node arrays are NULL");
    for (int64_t f = 0; f < F; ++f)
        if (node_i[f] < 0 || node_i[f] >= N || node_j[f] < 0 || node_j[f] >= N || node_i[f] == node_j[f])
            return g_invalid("factor nodes must be distinct and in [0, N)");
    // blocks: (r, c) -> ordered contribution list
    std::map<std::pair<int64_t, int64_t>, std::vector<int32_t>> blocks;
    for (int64_t f = 0; f < F; ++f) {
        const int64_t i = node_i[f], j = node_j[f];
        blocks[{i, i}].push_back((int32_t)(f << 2 | 0));
        blocks[{i, j}].push_back((int32_t)(f << 2 | 1));
        blocks[{j, i}].push_back((int32_t)(f << 2 | 2));
        blocks[{j, j}].push_back((int32_t)(f << 2 | 3));
    }
    for (int64_t n = 0; n < N; ++n) blocks[{n, n}];   // every node has a diagonal block
    auto* g = new vg_graph();
    AtExit drop([&] {
        graph_free(g);
        delete g;
    });
    g->ctx = ctx;
    g->N = N;
    g->F = F;
    g->row_ptr.assign(N + 1, 0);
    std::vector<int32_t> bptr, bitem, bnode;
    bptr.push_back(0);
    for (auto& kv : blocks) {
        g->row_ptr[kv.first.first + 1] += 1;
        g->col_idx.push_back(kv.first.second);
        for (int32_t it : kv.second) bitem.push_back(it);
        g->longest = std::max<int64_t>(g->longest, (int64_t)bitem.size() - bptr.back());
        bptr.push_back((int32_t)bitem.size());
        bnode.push_back(kv.first.first == kv.first.second ? (int32_t)kv.first.first : -1);
    }
    for (int64_t n = 0; n < N; ++n) g->row_ptr[n + 1] += g->row_ptr[n];
    g->nnzb = (int64_t)g->col_idx.size();
    hipError_t e = hipSetDevice(ctx->device);
    if (e == hipSuccess) e = up(&g->d_blk_ptr, bptr);
    if (e == hipSuccess) e = up(&g->d_blk_item, bitem);
    if (e == hipSuccess) e = up(&g->d_blk_node, bnode);
    if (e != hipSuccess) return hip_fail(e, "graph upload");
    drop.armed = false;
    g->magic = kGraphMagic;
    *out = g;
    return VG_OK;
} VG_NO_THROW

extern "C" vg_status vg_graph_structure(const vg_graph* g, int64_t* nnz_blocks, int64_t* row_ptr, int64_t* col_idx) try {
    set_error("");
    if (!graph_ok(g)) {
        set_error("invalid graph");
        return VG_ERR_STATE;
    }
    if (nnz_blocks) *nnz_blocks = g->nnzb;
    if (row_ptr) std::copy(g->row_ptr.begin(), g->row_ptr.end(), row_ptr);
    if (col_idx) std::copy(g->col_idx.begin(), g->col_idx.end(), col_idx);
    return VG_OK;
} VG_NO_THROW

extern "C" vg_status vg_graph_assemble_async(vg_graph* g, const double* d_poses, const double* d_lin,
                                             double* d_values, double* d_rhs) try {
    const vg::TimelineRange range_("vg_graph_assemble_async");
    set_error("");
    if (!graph_ok(g)) {
        set_error("invalid graph");
        return VG_ERR_STATE;
    }
    if ((g->F > 0 && (d_poses == nullptr || d_lin == nullptr)) || d_values == nullptr || d_rhs == nullptr)
        return g_invalid("NULL device pointer");
    VG_HIP(hipSetDevice(g->ctx->device));
    hipStream_t st = g->ctx->stream;
    const int grid = (int)std::min<int64_t>(g->nnzb, 1 << 22);
    if (g->nnzb > kBlocksPerContribution * g->longest)
        k_graph_assemble<1><<<grid, 64, 0, st>>>(g->d_blk_ptr, g->d_blk_item, g->d_blk_node, d_poses, d_lin, d_values,
                                                 d_rhs, g->nnzb);
    else
        k_graph_assemble<4><<<grid, 256, 0, st>>>(g->d_blk_ptr, g->d_blk_item, g->d_blk_node, d_poses, d_lin, d_values,
                                                  d_rhs, g->nnzb);
    VG_HIP(hipGetLastError());
    return VG_OK;
} VG_NO_THROW

extern "C" vg_status vg_graph_destroy(vg_graph* g) try {
    set_error("");
    if (!graph_ok(g)) {
        set_error("invalid graph");
        return VG_ERR_STATE;
    }
    (void)hipSetDevice(g->ctx->device);
    (void)hipStreamSynchronize(g->ctx->stream);
    graph_free(g);
    g->magic = 0;
    delete g;
    return VG_OK;
} VG_NO_THROW
