// Internal declarations of the VGICP device library (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <memory>
#include <mutex>
#include <string>
#include <unordered_map>
#include <utility>
#include <vector>

#include "vgicp.h"

namespace vg {

// ---------------------------------------------------------------- constants

constexpr int kMaxLevels = 4;
constexpr int kChunk = 64;              // points per anchor chunk == one wavefront
constexpr int kKeyBits = 14;            // bits per axis of a packed relative voxel key
constexpr int kKeyBias = 1 << (kKeyBits - 1);   // relative keys live in [-8192, 8191]
constexpr int kBlockShift = 2;          // voxel blocks of 4 x 4 x 4
constexpr int kBlockBits = kKeyBits - kBlockShift;   // 12 bits per axis of a block key
constexpr int kBaseBits = 28;           // first-record index bits of a block entry
constexpr uint64_t kBaseMask = (1ull << kBaseBits) - 1;
// voxels per level: records are addressed by 32-bit byte offsets (64 B each), so
// fewer than 2^26; this also keeps a valid entry word from ever being all ones
constexpr int64_t kMaxVoxels = ((int64_t)1 << 26) - 1;
constexpr uint64_t kEmpty = ~0ull;      // empty block-table entry
constexpr int kTerms = 28;              // e, 21 upper-triangular H, 6 b
// partial row of a tile (FP64): 28 terms, inliers per level, then the work the
// tile did: source points walked (chunks not culled), table lookups per level
// (point-levels inside the level's key box), chunks walked
constexpr int kRowInl = kTerms;                  // 4: points with a voxel, per level
constexpr int kRowWalk = kRowInl + 4;            // 1: source points walked
constexpr int kRowProbe = kRowWalk + 1;          // 4: table lookups, per level
constexpr int kRowChunks = kRowProbe + 4;        // 1: chunks walked
constexpr int kRow = 40;
constexpr int kWork = 8;                // per-factor work counts: walked points, walked chunks, lookups (4), 0, 0
constexpr int kMaxTileChunks = 128;     // chunks whose data a tile holds in LDS at once
constexpr int kMaxTilePoints = 32768;   // points per tile (taken in batches of kMaxTileChunks chunks)
constexpr int kGroup = 4;               // tiles per unit (workgroup) at most
constexpr int kRec32 = 16;              // floats per compensated voxel record (64 B: 4 FP32 + 6 FP64)
constexpr int kRecN = 12;               // floats per absolute-FP32 voxel record
constexpr int kRec64 = 10;              // doubles per FP64 voxel record
constexpr int kOutRow = 43;             // e, H (36), b (6)
constexpr int kParts = 8;               // XCDs of an MI355X: workgroups go to them round-robin

enum Mode { kLin = 0, kEval = 1, kBwd = 2, kCount = 3 };
enum Prec { kN32 = VG_FP32, kC32 = VG_FP32_COMPENSATED, kF64 = VG_FP64 };

// ---------------------------------------------------------------- device descriptors

// One level of a target voxel map as the kernels see it.
struct LevelDesc {
    const uint64_t* slots;   // 2^log2cap block entries of two words:
                             //   [(36-bit block key << 28) | first record, 64-bit occupancy]
    const float* rec32;      // V x 16 floats (64 B): mean - voxel centre (3 FP32), count (FP32), cov (6 FP64)
    const float* recN;       // V x 12: FP32 absolute mean (3), cov (6), pad
    const double* rec64;     // V x 10: absolute mean (3), cov (6), pad
    uint32_t log2cap;
    int32_t scale;           // r_coarsest / r_l (power of two)
    int32_t log2scale;       // log2 of scale
    float r, inv_r;
    double r64, inv_r64;
    int64_t K0[3];           // absolute key of the map origin at this level
    int32_t kmin[3], kmax[3];// bounding box of the level's relative keys (empty: min > max)
    int32_t kbox0[3];        // the same box as kbox0 + [0, kboxw] (empty level: the single key 0)
    uint32_t kboxw[3];
    double blo[3], bhi[3];   // the same box in metres, target frame (empty level: blo > bhi)
};

// One factor: a source cloud (internal Morton order) matched into a target map.
struct FactorDesc {
    const float* dxyz;       // 3 x n_pad SoA offsets from the chunk anchor
    const float* cov;        // 6 x n_pad SoA covariances
    const float* nrm;        // 3 x n_pad SoA normals or nullptr
    const double* anchor;    // n_chunks x 3 absolute anchors (source frame)
    const float* cbound;     // n_chunks x 8: chunk bounds around the anchor (m): box centre offset (3),
                             //   ball radius, box half extents (3), 0
    const float* axyz;       // 3 x n_pad absolute FP32 positions
    const double* xyz64;     // 3 x n_pad absolute FP64 positions
    const double* cov64;     // 6 x n_pad FP64 covariances
    const double* nrm64;     // 3 x n_pad FP64 normals or nullptr
    const int32_t* perm;     // internal index -> caller index
    int64_t n, n_pad;
    int64_t grad_offset;     // first row of this source in the concatenated point gradient
    int64_t grad_slab;       // -1 if no other factor of the batch uses this source; otherwise the
                             //   first row of this factor's own rows in the per-factor gradient
                             //   buffer, summed per source in factor order afterwards
    int32_t L;
    int32_t pad_;
    double src_origin[3];    // o_s: the re-centring origin of the source
    double viewpoint[3];     // target viewpoint (target frame) for surface validation
    LevelDesc lv[kMaxLevels];
};

// One source whose positions are replaced from rows of a device buffer.
struct PointSrc {
    float* dxyz;
    float* axyz;
    double* xyz64;
    const int32_t* perm;
    const double* anchor;
    float* cbound;
    int64_t n, n_pad;
    int64_t row0;            // its first row in the buffer
};

// A source used by several factors of a batch: its rows of the point gradient
// are the sum, in factor order, of those factors' rows in the per-factor buffer.
struct SharedSrc {
    int64_t row0;            // first of its rows among all shared sources' rows
    int64_t n;               // points
    int64_t grad_offset;     // first row in the concatenated point gradient
    int32_t f0, f1;          // its factors' entries [f0, f1) in the slab-offset list
};

// Device buffers one launch of the tile kernel and reduction works in.
struct Workspace {
    double* partials;        // n_tiles x kRow
    float* posef;            // F x 16 staged FP32 poses
    int64_t* work;           // F x kWork work counts, or nullptr
};

// One Levenberg-Marquardt iteration (every pointer on the device; lambda nullptr:
// none).  The proposal and the acceptance leave the FP32 poses of the tile launch
// that follows, and the reduction of the evaluation of the candidates ends with
// accepting or rejecting them.
struct LmArgs {
    double* lambda;          // F damping factors
    double* poses;           // F x 12 poses T
    double* cand;            // F x 12 candidates T Exp(delta)
    int32_t* valid;          // F: the damped matrix was SPD
    const double* lin;       // F x kOutRow linearization rows at T
    float* posef;            // F x 16 FP32 poses for the next tile launch, or nullptr
    double* e_out;           // error at T and decision, at column `col` of rows of `stride`, or nullptr
    int32_t* accepted;
    int32_t stride, col;
};

struct Tile {
    int32_t factor;
    int32_t chunk0;          // first chunk of the factor's source
    int32_t nchunks;
    int32_t row0;            // its partial row (a unit of tiles: that of its first tile)
};

// ---------------------------------------------------------------- host objects

struct Level {
    double r = 0;
    int64_t K0[3] = {0, 0, 0};
    int64_t V = 0;
    uint32_t log2cap = 0;      // block-table entries = 2^log2cap
    int64_t n_blocks = 0;
    uint64_t* slots = nullptr; // 2 words per entry
    float* rec32 = nullptr;
    float* recN = nullptr;
    double* rec64 = nullptr;
    uint64_t* keys = nullptr;   // V packed relative keys (record order)
    int32_t* counts = nullptr;  // V points per voxel (record order)
    int32_t kmin[3] = {1, 1, 1}, kmax[3] = {0, 0, 0};   // relative key bounding box
};

}  // namespace vg

namespace vg {

// hipMalloc on the current device.  Out of memory, it gives back what every context
// there keeps idle and tries again.  Leaves no error in the runtime when it fails.
hipError_t device_alloc(void** p, size_t bytes);

// Device memory that a context keeps: blocks of its clouds, maps, sources and batches
// for the next ones, and a workspace for the calls that build them.  The runtime
// hands out memory of 2 MiB and more by mapping it, unless a block of that very size
// was freed just before: 290 us against 12 us.  128-ring frames of differing sizes:
// 1,515 us each, 735 us with kept blocks.
// Blocks from kPooled on are rounded up by at most an eighth and kept when their
// object is destroyed, up to kKeepBlocks in all (the oldest are freed first); an idle
// block of up to one and a half times the rounded size is taken again.  They are
// given back with the context, or when any allocation of the library on the device
// fails (so is the workspace, unless a call is using it).  A block is taken back once
// the device is idle, as hipFree would wait, so no stream of any user still reads
// it.  Objects share the pool, which any thread may call.
struct BlockPool {
    static constexpr size_t kPooled = (size_t)2 << 20, kKeepBlocks = (size_t)256 << 20;
    explicit BlockPool(int device);
    ~BlockPool();
    BlockPool(const BlockPool&) = delete;
    BlockPool& operator=(const BlockPool&) = delete;
    hipError_t get(void** p, size_t bytes);
    void put(void* p);
    void close();     // frees what is kept; blocks put later are freed at once
    void give_back(); // frees what is idle
    // the workspace for one call, grown to `need` (0: as it is) when the call ends
    void* workspace(size_t* bytes);
    void end_workspace(size_t need);
    void drop_workspace();   // by the call that holds it
    const int device;
private:
    void release_locked(size_t limit);
    std::mutex mu;
    bool closed = false;
    size_t kept = 0;
    std::vector<std::pair<void*, size_t>> idle;   // oldest first
    std::unordered_map<void*, size_t> live;
    void* ws = nullptr;
    size_t ws_bytes = 0;
    int ws_users = 0;
};

}  // namespace vg

struct vg_context {
    int device = 0;
    std::shared_ptr<vg::BlockPool> pool;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    int32_t* h_small = nullptr;  // pinned host words that those calls' kernels write their sizes to
    int num_cu = 0;
    void* scratch = nullptr;     // this device's fixed scratch array (device address), or nullptr
    std::string arch;
    std::string name;
    uint32_t magic = 0;
};

struct vg_voxelmap {
    vg_context* ctx = nullptr;
    int L = 0;
    double origin[3] = {0, 0, 0};
    vg::Level lv[vg::kMaxLevels];
    void* blocks[vg::kMaxLevels] = {};   // the allocations that hold every level's arrays
    std::shared_ptr<vg::BlockPool> pool;
    int users = 0;
    uint32_t magic = 0;
};

struct vg_source {
    vg_context* ctx = nullptr;
    std::shared_ptr<vg::BlockPool> pool;
    int64_t n = 0, n_pad = 0, n_chunks = 0;
    double origin[3] = {0, 0, 0};
    bool has_normals = false;
    float* dxyz = nullptr;
    float* cov = nullptr;
    float* nrm = nullptr;
    double* anchor = nullptr;
    float* cbound = nullptr;   // per chunk: box centre offset (3), ball radius, box half extents (3), 0 (m)
    float* axyz = nullptr;
    double* xyz64 = nullptr;
    double* cov64 = nullptr;
    double* nrm64 = nullptr;
    int32_t* perm = nullptr;   // internal -> caller
    void* block = nullptr;     // the allocation that holds every array above and self
    vg::PointSrc* self = nullptr;   // device table of one entry: this source, rows from 0
    double extent = 0.0;       // upper bound of |mu - origin| over its points (m), from the chunk bounds
    int users = 0;
    uint32_t magic = 0;
};

// A preprocessed frame (downsampled points, neighbours, covariances, normals).
struct vg_cloud {
    vg_context* ctx = nullptr;
    std::shared_ptr<vg::BlockPool> pool;
    int64_t m = 0;              // downsampled points
    int32_t k = 0;              // neighbours per point
    double* xyz = nullptr;      // m x 3
    double* cov = nullptr;      // m x 6 regularised
    double* cov_raw = nullptr;  // m x 6 neighbour covariance
    double* nrm = nullptr;      // m x 3
    int32_t* counts = nullptr;  // m input points per voxel
    int32_t* nbr = nullptr;     // m x k
    double* d2 = nullptr;       // m x k
    void* block = nullptr;      // one allocation holding every array above
    double first[3] = {0, 0, 0};// host copy of point 0 (origins of sources / maps made from the cloud)
    double box[6] = {0, 0, 0, 0, 0, 0};   // host copy of the points' bounding box
    uint32_t magic = 0;
};

struct vg_batch {
    vg_context* ctx = nullptr;
    std::shared_ptr<vg::BlockPool> pool;
    int64_t F = 0;
    int L = 0;
    vg_batch_options opt{};
    std::vector<vg_source*> src;
    std::vector<vg_voxelmap*> tgt;
    std::vector<vg::FactorDesc> h_fac;
    std::vector<vg::Tile> h_tiles;
    std::vector<int32_t> h_tile_first;   // F + 1
    std::vector<vg::Tile> h_units;       // units: runs of whole tiles of one factor
    std::vector<int32_t> h_unit_first;   // F + 1
    int64_t total_points = 0;
    int64_t grad_rows = 0;               // rows of the concatenated point gradient
    int block = 256, tile_points = 2048, blocks_per_cu = 0;
    int tile_order = 1;                  // 1 contiguous per XCD, 2 round-robin over XCDs
    // device buffers, carved from one block
    char* dblock = nullptr;
    char* sched = nullptr;          // large rows, or tables and rows of a launch shape set after creation
    vg::FactorDesc* d_fac = nullptr;
    vg::Tile* d_units = nullptr;
    int32_t* d_tile_first = nullptr;
    double* d_partials = nullptr;
    double* d_poses = nullptr;
    float* d_posef = nullptr;       // F x 16 staged FP32 poses
    double* d_out = nullptr;        // F x 43
    int64_t* d_inliers = nullptr;   // F x L
    int64_t* d_work = nullptr;      // F x kWork work counts of the last linearize / evaluate / overlap
    double* d_e = nullptr;          // F (evaluate)
    double* d_lm = nullptr;         // LM scratch
    // sources shared by several factors (deterministic point gradients)
    std::vector<vg::SharedSrc> h_shared;
    std::vector<int64_t> h_slab_off;     // per shared source, its factors' slab rows, factor order
    int64_t slab_rows = 0;
    int64_t shared_rows = 0;
    vg::SharedSrc* d_shared = nullptr;
    vg::PointSrc* d_points = nullptr;    // its distinct sources in order of first use
    int64_t n_sources = 0, max_chunks = 0;
    int64_t* d_slab_off = nullptr;
    void* d_gslab = nullptr;             // per-factor point gradients (grown on first use)
    size_t gslab_bytes = 0;
    double max_source_extent = 0.0;      // largest |mu - o_s| over the batch's sources (m)
    // pinned host staging (one upload, one download), carved from one block
    char* hblock = nullptr;
    double* h_poses = nullptr;
    double* h_out = nullptr;
    int64_t* h_inliers = nullptr;
    unsigned char* h_lm = nullptr;  // error and decision histories of short LM runs
    size_t h_lm_bytes = 0;
    uint32_t magic = 0;
};

namespace vg {

// ---------------------------------------------------------------- error state

void set_error(const std::string& msg);
bool context_ok(const vg_context* c);
vg_status hip_fail(hipError_t e, const char* what);

#define VG_HIP(call)                                        \
    do {                                                    \
        hipError_t _e = (call);                             \
        if (_e != hipSuccess) return vg::hip_fail(_e, #call);\
    } while (0)

// Ends every entry point of the ABI (a function-try-block): an exception, which is the
// host's memory running out, becomes a status.  The message is short enough for the
// string to hold it without allocating.
vg_status out_of_host_memory();
#define VG_NO_THROW                         \
    catch (...) {                           \
        return vg::out_of_host_memory();    \
    }

// Runs f at the end of its scope, also on exceptions, unless disarmed.
template <typename F>
struct AtExit {
    F f;
    bool armed = true;
    explicit AtExit(F g) : f(g) {}
    AtExit(const AtExit&) = delete;
    AtExit& operator=(const AtExit&) = delete;
    ~AtExit() {
        if (armed) f();
    }
};

// ---------------------------------------------------------------- scratch

constexpr size_t kKeepWorkspace = (size_t)1 << 30;   // a larger call's temporaries are freed with it
constexpr int kCheckParts = 256;                     // workgroups of a cloud's check at most
constexpr int kSmallWords = 8192;                    // pinned words of a context

// Temporaries of one call, carved from the context's workspace (the calls of a
// context are ordered on its stream, so a later call may write them while the
// host is ahead of the device); what does not fit is allocated and freed, and the
// workspace grows to the call's total afterwards, up to kKeepWorkspace, so calls of
// similar size allocate nothing.
struct Scratch {
    vg_context* ctx;
    size_t ws_bytes = 0;   // (initialised before ws, whose initialiser sets it)
    char* ws;
    size_t off = 0, need = 0, parts = 0;   // parts: the most that one part of the call needed
    Scratch* whole = nullptr;
    std::vector<void*> ptrs;
    explicit Scratch(vg_context* c) : ctx(c), ws((char*)c->pool->workspace(&ws_bytes)) {}
    // temporaries of a part of a call, behind those of the call
    explicit Scratch(Scratch* of) : ctx(of->ctx), ws_bytes(of->ws_bytes), ws(of->ws), off(of->off), whole(of) {}
    Scratch(const Scratch&) = delete;
    Scratch& operator=(const Scratch&) = delete;
    ~Scratch() {
        if (!ptrs.empty()) (void)hipStreamSynchronize(ctx->stream);   // also on early error returns
        for (void* p : ptrs) (void)hipFree(p);
        need += parts;
        if (whole) whole->parts = need > whole->parts ? need : whole->parts;
        else ctx->pool->end_workspace(need <= kKeepWorkspace ? need : 0);
    }
    template <typename T>
    hipError_t get(T** p, size_t count) {
        const size_t bytes = (sizeof(T) * (count ? count : 1) + 255) & ~(size_t)255;
        need += bytes;
        *p = nullptr;
        if (ws && off + bytes <= ws_bytes) {
            *p = (T*)(ws + off);
            off += bytes;
            return hipSuccess;
        }
        void* q = nullptr;
        hipError_t e = device_alloc(&q, bytes);
        if (e != hipSuccess && ws && off == 0 && !whole) {   // too small for this call, and in its way
            ctx->pool->drop_workspace();
            ws = nullptr;
            e = device_alloc(&q, bytes);
        }
        if (e == hipSuccess) ptrs.push_back(q);
        *p = (T*)q;
        return e;
    }
};

// ---------------------------------------------------------------- launchers (device code)

// One workgroup's share of the check of a cloud's arrays, in pinned host memory.
constexpr int32_t kBadXyz = 1, kBadCov = 2, kBadNormal = 4;   // some value is not finite
struct CheckPart {
    double box[6];       // min xyz, max xyz
    double first[3];     // point 0
    int64_t bad;         // lowest point whose covariance is not SPD (INT64_MAX: none)
    int32_t flags;
    int32_t pad;
};
static_assert(sizeof(CheckPart) * kCheckParts <= sizeof(int32_t) * kSmallWords, "the parts fit the pinned words");
// check n >= 1 points (covariances and normals may be nullptr); the result may be
// read with joined_check once the stream has been waited for
vg_status launch_check(vg_context* ctx, const double* d_xyz, const double* d_cov, const double* d_nrm, int64_t n);
CheckPart joined_check(const vg_context* ctx, int64_t n);

// every level of m (its origin is set) from n points; box: their bounding box
vg_status build_map(vg_context* ctx, Scratch& sc, const double* d_xyz, const double* d_cov, int64_t n,
                    const double box[6], const double* resolutions, int L, vg_voxelmap* m);
vg_status export_level(vg_context* ctx, const Level& lv, int64_t* keys, double* means, double* covs,
                       int64_t* counts);
void free_map(vg_voxelmap* m);

// frame preprocessing: d_xyz n x 3 FP64 device input with bounding box `box`; fills every array of *out
vg_status preprocess_frame(vg_context* ctx, Scratch& sc, const double* d_xyz, int64_t n, const double box[6], double r,
                           int k, const double sensor[3], vg_cloud* out);
void free_cloud(vg_cloud* c);

// every array of s from device FP64 arrays in caller order, and its extent; box: the points' bounding box
vg_status layout_source(vg_context* ctx, Scratch& sc, vg_source* s, const double* d_xyz, const double* d_cov,
                        const double* d_nrm, const double box[6]);
// new positions of n_src sources (device table) from d_xyz, with their chunk bounds
vg_status set_points(vg_context* ctx, const PointSrc* d_src, int64_t n_src, int64_t max_chunks, const void* d_xyz,
                     int dtype);

// launch the tile kernel of a mode over the tiles of factors [f0, f1) (their poses are staged to FP32
// first where the kernel reads them so, unless `staged` says that they are)
// ws: the buffers of the launch (the batch's own, or a caller-provided scratch)
vg_status launch_tiles(vg_batch* b, const Workspace& ws, int mode, const double* d_poses, const double* d_grad_e,
                       void* d_grad_points, int points_dtype, int64_t f0, int64_t f1, bool staged = false);
// whether the batch's kernels of a mode read FP32 poses staged in ws.posef
bool reads_staged_poses(const vg_batch* b, int mode);
vg_status launch_reduce(vg_batch* b, const Workspace& ws, int mode, const double* d_poses, int32_t f0, int32_t f1,
                        double* d_out, int64_t* d_inliers, const double* d_grad_e, const double* d_jr,
                        double* d_grad_xi, const LmArgs& lm = LmArgs{});
// the batch's poses from pinned host memory to b->d_poses, and to ws.posef where a mode's kernels read
// them so (the tile launch that follows is then `staged`)
vg_status launch_pose_upload(vg_batch* b, const Workspace& ws, int mode, const double* h_poses);
// copy of a multiple of 8 bytes between device and pinned host memory by a kernel
vg_status launch_copy(vg_context* ctx, const void* src, void* dst, size_t bytes);
// rows of shared sources: sum of their factors' per-factor rows in factor order
vg_status launch_grad_combine(vg_batch* b, void* d_grad_points, int points_dtype);
vg_status launch_correspondences(vg_batch* b, const double* d_pose, int64_t factor, int64_t* d_keys,
                                 int32_t* d_found);
vg_status launch_zero(vg_context* ctx, void* d_ptr, size_t bytes);
vg_status launch_se3_retract(vg_context* ctx, int64_t F, const double* d_T0, const double* d_xi, double* d_T,
                             double* d_jr);
// candidates of every factor from its linearization row
vg_status launch_lm_propose(vg_batch* b, const double* d_out, const LmArgs& lm);
vg_status launch_fill(vg_context* ctx, double* d_ptr, int64_t n, double v);

}  // namespace vg
