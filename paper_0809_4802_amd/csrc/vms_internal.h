// Internal declarations of libvms (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <string>
#include <type_traits>
#include <vector>

#include "vms.h"

namespace vms {

constexpr int kBlock = 256;          // threads per workgroup for streaming kernels
constexpr int kRedBlocks = 1024;     // workgroups of the grid-wide reductions
constexpr int kMaxRestart = 128;
constexpr int kDrMax = 33;           // vectors kept by deflated restarting (k <= 32, +1 for a complex pair)
// Deflated restarting: what the host hands the device between two cycles, packed (doubles,
// each block column-major): the basis coefficients P ((m+1) x kk, ld m+1), the kept block of H
// ((kk+1) x kk), its triangle R (kk x kk), Q^T ((kk+1) x (kk+1)) and the free-pressure sums of
// the kept vectors (kk).
constexpr int kDrOffH = (kMaxRestart + 1) * kDrMax;
constexpr int kDrOffR = kDrOffH + (kDrMax + 1) * kDrMax;
constexpr int kDrOffQt = kDrOffR + kDrMax * kDrMax;
constexpr int kDrOffSvs = kDrOffQt + (kDrMax + 1) * (kDrMax + 1);
constexpr int kDrUpload = kDrOffSvs + kDrMax;
#ifndef VMS_DOT_CHUNKS
#define VMS_DOT_CHUNKS 64          // upper bound on the workgroups (partials) per GMRES dot slot
#endif
constexpr int kTileNodes = 64;           // max nodes owned by one assembly tile
// Tiles of the residual alone.  Measured at 41,400 nodes with a body force, 195,000 nodes transient:
// 256 threads and 32 nodes 22.8 and 43.2 us, 24 nodes 26.1 and 53, 64 nodes 24 and 45, 128 threads 27
// and 49 (the registers allow three waves a SIMD; a bound of four spills: 25 and 47).
constexpr int kResidualThreads = 256;     // threads per tile
constexpr int kResidualNodes = 32;        // max nodes owned by one
constexpr int kResidualSlots = 2048;      // max element rows staged by one (64 KB)
constexpr int kNoSlot = 0xffff;           // slot of a vertex that the tile does not own (or does not number)
constexpr int kTileMaxNodes = 255;       // max nodes staged by one tile (8-bit local numbers)
#ifndef VMS_TILE_BLOCKS_FP64
#define VMS_TILE_BLOCKS_FP64 280
#endif
#ifndef VMS_TILE_BLOCKS_DET
#define VMS_TILE_BLOCKS_DET 64
#endif
#ifndef VMS_TILE_BLOCKS_FP32
#define VMS_TILE_BLOCKS_FP32 870
#endif
#ifndef VMS_LDS_BLOCK_STRIDE
#define VMS_LDS_BLOCK_STRIDE 17
#endif
#ifndef VMS_MIXED_LDS_FP64
#define VMS_MIXED_LDS_FP64 1
#endif
// accumulator type of the staged blocks in the mixed-precision assembly
using MixedAcc = std::conditional_t<VMS_MIXED_LDS_FP64 != 0, double, float>;
constexpr size_t kMixedAccSize = sizeof(MixedAcc);
constexpr int kTileBlocksFP64 = VMS_TILE_BLOCKS_FP64;   // max 4x4 blocks staged in LDS per tile (FP64 values)
constexpr int kTileBlocksFP32 = VMS_TILE_BLOCKS_FP32;   // same for FP32 values
constexpr int kTileBlocksDet = VMS_TILE_BLOCKS_DET;     // blocks per one-wavefront tile (deterministic contexts)

// Dynamic LDS of a tile: block values (each 4x4 block padded to 17 entries so that the
// lanes of a wave, which update the same entry of different blocks, spread over the LDS
// banks), rhs rows and residual rows.
constexpr int kLdsBlockStride = VMS_LDS_BLOCK_STRIDE;
__host__ __device__ constexpr size_t align16(size_t x) { return (x + 15) & ~size_t(15); }
__host__ __device__ constexpr size_t tile_lds_bytes(int64_t nblocks, int64_t nnodes, size_t elt) {
    return align16(nblocks * kLdsBlockStride * elt) + 2 * nnodes * 4 * 8;
}
// The most dynamic LDS that any context's tiles take, of the assembly (a row has at most kTileMaxNodes
// blocks; a staged node three double4) and of the residual alone.
constexpr size_t kTileLdsMax =
    std::max(tile_lds_bytes(std::max(kTileBlocksFP64, kTileMaxNodes), kTileNodes, sizeof(double)),
             kMixedAccSize == sizeof(double) ? size_t(0) : tile_lds_bytes(kTileBlocksFP32, kTileNodes, kMixedAccSize)) +
    96 * size_t(kTileMaxNodes);
constexpr size_t kResidualLdsMax = 32 * (size_t(kResidualSlots) + 3 * kTileMaxNodes);
static_assert(kTileLdsMax <= 163840 - 1024 && kResidualLdsMax <= 163840 - 1024, "LDS of a CU");

// Four-wide vector of a precision (one node's dofs, one block row).
template <typename T>
struct Vec4;
template <>
struct Vec4<double> {
    using type = double4;
};
template <>
struct Vec4<float> {
    using type = float4;
};

// The same in a caller's array, which is only promised to be aligned to its entries: accessed in one wide
// load or store that asks for no more.
template <typename T>
struct CallerVec4;
template <>
struct CallerVec4<double> {
    typedef double type __attribute__((ext_vector_type(4), aligned(8)));
};
template <>
struct CallerVec4<float> {
    typedef float type __attribute__((ext_vector_type(4), aligned(4)));
};

// Lane exchanges of a double by DPP (two 32-bit moves; no LDS round trip).  CTRL: a
// quad_perm pattern, or 0x140 (row_mirror: lane i <-> 15 - i in a row of 16), 0x141
// (row_half_mirror: lane i <-> 7 - i in a group of 8) and 0x138 (a shift by one lane).  Every lane of the wave must be active.
template <int CTRL>
__device__ __forceinline__ double dpp_mov(double v) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double read_lane(double v, int l) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l),
                            __builtin_amdgcn_readlane(__double2loint(v), l));
}

// v of lane l to lane l + 1; lane 0 gets first.  Every lane of the wave must be active.
__device__ __forceinline__ double wave_shift(double v, double first) {
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(first), __double2loint(v), 0x138, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(first), __double2hiint(v), 0x138, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}

// Sum over the eight lanes of an aligned group (every lane gets it).
__device__ __forceinline__ double group8_sum(double v) {
    v += dpp_mov<0xB1>(v);           // quad_perm [1,0,3,2]: lane ^ 1
    v += dpp_mov<0x4E>(v);           // quad_perm [2,3,0,1]: lane ^ 2
    return v + dpp_mov<0x141>(v);    // the other quad of the eight
}

// Sum over the 64 lanes of the wave (every lane gets it): rows of 16 by DPP, then the four
// row sums read back as scalars.  Every lane of the wave must be active.
__device__ __forceinline__ double wave_sum(double v) {
    v = group8_sum(v);
    v += dpp_mov<0x140>(v);          // the other eight of the row
    return (read_lane(v, 0) + read_lane(v, 16)) + (read_lane(v, 32) + read_lane(v, 48));
}

// Gauss-Jordan inverse of a 4x4 block (partial pivoting); false if singular.  Rows are exchanged by
// selects: an index that depends on the pivot puts the block in scratch memory, which made the
// block-Jacobi setup of 274,625 nodes take 39.7 us (mixed), now 14.1.
__device__ __forceinline__ bool invert4(const double (&in)[4][4], double (&out)[4][4]) {
    double m[4][8];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            m[r][c] = in[r][c];
            m[r][4 + c] = (r == c) ? 1.0 : 0.0;
        }
    bool ok = true;
#pragma unroll
    for (int col = 0; col < 4; ++col) {
        int piv = col;
        double best = fabs(m[col][col]);
#pragma unroll
        for (int r = col + 1; r < 4; ++r)
            if (fabs(m[r][col]) > best) {
                best = fabs(m[r][col]);
                piv = r;
            }
        ok = ok && best > 0.0;
#pragma unroll
        for (int r = col + 1; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const double t = m[col][c], v = m[r][c];
                m[col][c] = piv == r ? v : t;
                m[r][c] = piv == r ? t : v;
            }
        const double ip = 1.0 / m[col][col];
#pragma unroll
        for (int c = 0; c < 8; ++c) m[col][c] *= ip;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if (r == col) continue;
            const double f = m[r][col];
#pragma unroll
            for (int c = 0; c < 8; ++c) m[r][c] -= f * m[col][c];
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) out[r][c] = m[r][4 + c];
    return ok;
}

// Device-resident state of one GMRES cycle (Hessenberg matrix, Givens
// rotations, residual estimate).  Updated by single-lane finalisers so that
// the Arnoldi loop never waits for the host.
struct GmresState {
    double H[(kMaxRestart + 1) * kMaxRestart];   // Hessenberg, column-major, ld = kMaxRestart + 1
    double R[(kMaxRestart + 1) * kMaxRestart];   // its Givens-rotated triangle, same layout
    double cs[kMaxRestart];
    double sn[kMaxRestart];
    double g[kMaxRestart + 1];     // rotated right-hand side (final entries)
    double gin[kMaxRestart + 1];   // entry i before rotation i (gin[k] = residual estimate)
    double y[kMaxRestart];
    double scoef[kMaxRestart];     // s = Q^T u_m: second-pass coefficients of a cycle's last vector
    double svs[kMaxRestart + 1];   // free-pressure sum of every final basis vector
    double tol_abs;                // stop when |g[k]| <= tol_abs
    double beta;                   // norm of the cycle's initial residual
    double kappa;                  // coarse pressure correction: 1 / (sum of free p-p entries), 0 = off
    double su;                     // sum of the free pressure entries of u_j
    double rho;                    // norm of u_j after its second pass
    double rho_m;                  // the same of a cycle's last vector
    double cj;                     // q_j . w
    double hh;                     // provisional subdiagonal of column j (norm estimate of u_{j+1})
    int reorth;                    // 0: one Gram-Schmidt pass; otherwise a delayed second pass
    int k;                         // Arnoldi steps completed in this cycle
    int done;                      // 0 while the cycle runs; 1 once it stopped (converged or
                                   // breakdown), later kernels idle
    unsigned gen;                  // cycle number (host-assigned) reported with the progress word
    uint64_t* progress;            // host-mapped progress word: gen << 32 | k << 1 | done
    const void* A;                 // the cycle's matrix, where P and A are applied one after the other
    // deflated restarting: the cycle starts with dk kept vectors V[0 .. dk-1], whose
    // columns of H (rows 0 .. dk) and R the host set; dr_qt is Q^T of the QR factors of that
    // (dk + 1) x dk block (column-major), dr_c the cycle's least-squares right-hand side
    double dr_qt[(kDrMax + 1) * (kDrMax + 1)];
    double dr_c[kDrMax + 1];
};
// the host staging of deflated restarting: a GmresState (padded), then the packed upload
constexpr size_t kDrStateBytes = (sizeof(GmresState) + 255) & ~size_t(255);
constexpr int kDrTagWord = 4;        // word of the progress page: number of the cycle whose state was handed over
constexpr size_t kDrStagingBytes = kDrStateBytes + sizeof(double) * kDrUpload;

// Grid-wide reduction scratch.
struct RedScratch {
    double partial[kRedBlocks * (kMaxRestart + 1)];
    unsigned counter;
};

}  // namespace vms

struct vms_ctx {
    int device = 0;
    int32_t n_nodes = 0;
    int32_t n_elems = 0;
    int64_t nb = 0;
    vms_precision prec = VMS_FP64;
    int32_t max_restart = 50;
    int32_t n_dir = 0;
    int32_t n_pressure_pins = 0;     // Dirichlet pressure dofs (the coarse pressure mode needs one)

    // mesh (device, library-owned copies)
    double4* xyz4 = nullptr;         // [n_nodes] (x, y, z, 0)
    int4* tets = nullptr;            // [n_elems]
    uint8_t* dmask = nullptr;        // [n_nodes] bit c set: dof 4i+c is Dirichlet
    int32_t* dlist = nullptr;        // [n_dir] Dirichlet dofs

    // block pattern (device)
    int32_t* rowptr = nullptr;       // [n_nodes + 1]
    int32_t* colidx = nullptr;       // [nb]
    int32_t* diagpos = nullptr;      // [n_nodes]
    int32_t* tpos = nullptr;         // [nb] position of the transposed block
    // assembly tiles: tile t owns the block rows of a contiguous node range and stages the nodes
    // its elements touch (owned ones first) in LDS; it works through its items, one per
    // (element e, owned vertex a), in the vertex order a, a^1, a^2, a^3: items = (e, four 8-bit
    // local node numbers, four 16-bit tile-local block slots of the owned row; bit 15 of the
    // first slot marks a = 0)
    int32_t n_tiles = 0;
    int4* tile_meta = nullptr;       // [n_tiles][2]: (first node, end node, first block, blocks),
                                     // (first item, end item, first staged node, staged nodes)
    int32_t* tile_nodes = nullptr;   // [staged nodes of all tiles]
    uint4* items = nullptr;          // [4 n_elems]
    uint16_t* bmask = nullptr;       // [nb] Dirichlet bits of the column node (0..3) and the row
                                     // node (4..7), bit 8 on diagonal blocks
    double* tile_part = nullptr;     // [max(n_tiles, n_rtiles)][2] partial sums of the residual norm
    // tiles of the residual alone (element.hip, residual_kernel): its own node ranges, one item per
    // element and tile, and a slot per element and vertex, those of a node side by side
    int32_t n_rtiles = 0;
    int4* rtile_meta = nullptr;      // [n_rtiles][2]: (first node, end node, first staged node, staged nodes),
                                     // (first item, end item, first slot, slots)
    int32_t* rtile_nodes = nullptr;  // [staged nodes of all residual tiles]
    uint4* ritems = nullptr;
    int32_t* n2e_ptr = nullptr;      // [n_nodes + 1] elements at the nodes before
    size_t rtile_lds[2] = {};        // dynamic LDS bytes of the largest residual tile; [1]: with a previous
                                     // velocity or a body force
    int32_t tile_threads = 256;      // threads per assembly tile (64: deterministic context)
    size_t tile_lds = 0;             // dynamic LDS bytes of the largest tile (steady)
    size_t tile_lds_tr = 0;          // same with the previous velocity staged (transient)

    // Newton workspaces (device)
    void* A = nullptr;               // [nb][16] of the ctx precision
    double* rhs = nullptr;           // [4 n_nodes]
    double* du = nullptr;            // [4 n_nodes]
    double* rnorm = nullptr;         // [4] device scalars
    int32_t* flags = nullptr;        // [8] device flags: [2] singular preconditioner blocks, [3] non-finite
                                     // learned blocks; [4..7] the two 64-bit element flags (element.hip)
    uint32_t elem_gen = 0;           // call number of the element flags (advanced by each element launch)

    // Krylov workspaces (device); T = double (FP64 ctx) or float (mixed)
    void* V = nullptr;               // [(max_restart + 1)][4 n_nodes]
    void* w = nullptr;               // [4 n_nodes]
    void* z = nullptr;               // [4 n_nodes]
    void* d = nullptr;               // [4 n_nodes] correction accumulated by a solve
    void* r = nullptr;               // [4 n_nodes] inner residual
    void* Minv = nullptr;            // [n_nodes][16] preconditioner blocks
    void* AP = nullptr;              // [nb][16] A P: each block times the preconditioner block of its column
    void* Az = nullptr;              // [4 n_nodes] A z, z = 1 on every free pressure dof
    void* pp = nullptr;              // [nb] the entries of A that couple two free pressures (condensed systems)
    double* x64 = nullptr;           // [4 n_nodes] the iterate before a deflated GMRES cycle
    // mixed context created with basis_fp64: the FP64 basis, w and z
    double* V64 = nullptr;           // [(max_restart + 1)][4 n_nodes]
    double* w64 = nullptr;
    double* z64 = nullptr;
    double* r64 = nullptr;           // [4 n_nodes]
    vms::GmresState* gs = nullptr;
    vms::RedScratch* red = nullptr;
    // progress of the running GMRES cycle, written by the device into pinned host memory so
    // that the host can follow it without synchronising the stream
    uint64_t* progress_host = nullptr;
    uint64_t* progress_dev = nullptr;
    // GMRES norms that the host reads (the true residual, the right-hand side, the inner residual),
    // written by the device into the same pinned allocation, 64 bytes after the progress word, and
    // then their tags, which the host polls for: no copy kernel and no stream synchronisation per read
    double* scal_host = nullptr;
    double* scal_dev = nullptr;
    uint64_t scal_seq = 0;               // tag of the last norm launched (words 1 .. 3 of the progress page)
    uint32_t cycle_gen = 0;
    std::vector<int64_t> cycle_timed;    // timed launches of the cycle: (step, slot, generation)
    // a full restart cycle's Arnoldi steps recorded once as a graph (replayed with one launch)
    hipStream_t cap_stream = nullptr;    // stream the graph is captured on
    hipGraphExec_t cycle_exec = nullptr;
    int cycle_exec_m = 0;                // restart length of cycle_exec, times 2, + 1 for an FP64 basis
    // graphs of deflated cycles (steps j0 .. m-1), keyed by (m, j0)
    hipGraphExec_t dr_exec[4] = {nullptr, nullptr, nullptr, nullptr};
    int dr_exec_key[4] = {0, 0, 0, 0};
    double* dr_p = nullptr;              // [(kMaxRestart + 1) kDrMax] device copy of the basis coefficients
    void* dr_pinned = nullptr;           // mapped host memory [kDrStagingBytes]: a GmresState written by the
                                         // device (kDrStateBytes), then the packed upload it reads
    void* dr_mapped = nullptr;           // its device address
    int64_t prof_cycles = 0;             // cycles seen while the phase timers are on
    bool prof_force = false;             // a sampled cycle: every launch of a timed phase is timed

    // uncondensed system (vms_create_opts.full_system): a solver-only child context over the
    // n_nodes + n_elems block rows (its n_nodes field counts block rows), and the positions of
    // the element contributions in its pattern
    vms_ctx* full = nullptr;
    int32_t* full_cc = nullptr;      // [nb] position of condensed-pattern block k in the full pattern
    int32_t* full_epos = nullptr;    // [n_elems][9]: (node a, elem) a = 0..3, (elem, node b) b = 0..3, (elem, elem)
    int32_t linearization = VMS_LIN_NEWTON;   // tangent of the element kernels (vms_set_linearization)
    int32_t full_nodes = 0;          // in the child: number of node block rows (0 in other contexts)
    double* zfull = nullptr;         // in the child: [4 n_nodes] coarse vector (free pressures + fine response)

    // learned preconditioner (device, float)
    float* feats = nullptr;          // [n_nodes][25]
    float* hid = nullptr;            // [n_nodes][64]
    float* pblk = nullptr;           // [n_nodes][16]
    float* gblk = nullptr;           // [n_nodes][16] D^-1 blocks (features, training)
    float* gdel = nullptr;           // [n_nodes][16] dL/dDelta (training)
    float* tvec = nullptr;           // [3][4 n_nodes] training vectors
    float* wgrad = nullptr;          // [kRedBlocks][VMS_PC_NWEIGHTS] partial weight gradients
    float* fscal = nullptr;          // [8] float scalars

    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    std::string err;

    // phase timers
    uint32_t prof_mask = 0;                // phases being timed
    int32_t prof_every = 1;                // time every n-th launch of a phase
    int64_t prof_seen[VMS_NPHASES] = {};   // launches seen per phase
    int64_t prof_gen = 0;                  // pending-slot generation (bumped by each flush)
    std::vector<hipEvent_t> prof_ev;       // pairs
    std::vector<int> prof_phase;           // pending slot -> phase
    std::vector<double> prof_bytes;        // pending slot -> algorithmic bytes
    int prof_used = 0;
    double prof_ms[VMS_NPHASES] = {};
    double prof_acc_bytes[VMS_NPHASES] = {};
    int64_t prof_count[VMS_NPHASES] = {};
};

namespace vms {

int set_error(vms_ctx* ctx, int code, const std::string& msg);
int check_hip(vms_ctx* ctx, hipError_t e, const char* what);
inline size_t elt_size(const vms_ctx* c) { return c->prec == VMS_FP64 ? 8 : 4; }
inline unsigned long long* element_flags(vms_ctx* c) { return reinterpret_cast<unsigned long long*>(c->flags + 4); }

// phase timers (ctx.cpp): a scope records an event pair around the launches it encloses
int prof_begin(vms_ctx* c, int phase, double bytes, hipStream_t s);
void prof_end(vms_ctx* c, int slot, hipStream_t s);
// Drops a pending timed launch (one that returned without work) from the accumulators.
void prof_void(vms_ctx* c, int slot, int64_t gen);
struct PhaseScope {
    vms_ctx* c;
    int slot;
    int64_t gen;
    hipStream_t s;
    PhaseScope(vms_ctx* c_, int phase, double bytes, hipStream_t s_) : c(c_), slot(-1), gen(0), s(s_) {
        if ((c->prof_mask >> phase) & 1u) {
            slot = prof_begin(c, phase, bytes, s);
            gen = c->prof_gen;
        }
    }
    ~PhaseScope() {
        if (slot >= 0) prof_end(c, slot, s);
    }
};

// element kernels (element.hip)
hipError_t tile_kernels_configure();
// rglob (may be null) receives the assembled residual rows; every launch leaves the norm's
// partial sums per tile in ctx->tile_part, which launch_norm_finalize adds into out.
int launch_condense(vms_ctx* ctx, const double* u, const double* u_prev, const double* beta,
                    double nu, double inv_dt, const double* body, void* A, double* rhs,
                    double* rglob, hipStream_t s);
int launch_residual(vms_ctx* ctx, const double* u, const double* u_prev, const double* beta,
                    double nu, double inv_dt, const double* body, double* rglob, hipStream_t s);
int launch_norm_finalize(vms_ctx* ctx, double* out, hipStream_t s);    // after launch_condense
int launch_residual_norm(vms_ctx* ctx, double* out, hipStream_t s);    // after launch_residual
int check_element_flags(vms_ctx* ctx, hipStream_t s);
// Resolves this device's address of the no-allocation entry point's static scratch (once per
// device; called by vms_create with the context's device current).
int noalloc_scratch_init(vms_ctx* ctx);
// Uncondensed system (ctx->full must exist): assembly into vals / rhs of the full pattern, and
// the Newton update from its solution dx.
int launch_full_assemble(vms_ctx* ctx, const double* u, const double* u_prev, const double* beta, double nu,
                         double inv_dt, const double* body, void* vals, double* rhs, hipStream_t s);
int launch_full_update(vms_ctx* ctx, const double* dx, double* u, double* beta, hipStream_t s);

// linear algebra (krylov.hip)
hipError_t small_cycle_configure();
int launch_fill(void* p, size_t bytes, hipStream_t s);
int launch_spmv(vms_ctx* ctx, const void* A, const void* x, void* y, hipStream_t s);
int launch_bj_setup(vms_ctx* ctx, const void* A, void* Minv, hipStream_t s);
int gmres_solve(vms_ctx* ctx, const void* A, const double* b, double* x,
                const vms_solve_opts* opts, vms_solve_info* info, hipStream_t s);

// learned preconditioner (learned_pc.hip)
int learned_blocks(vms_ctx* ctx, const void* A, const float* weights, void* Minv_out,
                   int out_is_double, hipStream_t s);

}  // namespace vms
