// Condensed-system linear algebra on gfx950: 4x4 block-CSR SpMV, block
// preconditioners and restarted GMRES(m).
//
// The paper solves each Newton system with a Krylov method at tolerance 1e-12
// and a 50-iteration cap and aborts on failure (Section 6); the method and the
// preconditioner are left to PETSc defaults.  This library uses right-
// preconditioned restarted GMRES with 4x4 block-Jacobi (or its learned
// correction), judges success by the true residual ||b - A x|| recomputed at
// every restart, and reports failure instead of aborting.
//
// GPU layout: all vectors are node-interleaved (4 n_nodes entries, dofs
// (vx, vy, vz, p) of a node adjacent) so that a 4x4 block multiplies one
// 32-byte (FP64) or 16-byte (FP32) segment.  The Hessenberg matrix, the Givens
// rotations and the residual estimate live in device memory, updated by single
// workgroups beside the streaming ones, so an Arnoldi step is a fixed
// sequence of launches with no host round trip.  The rotations publish the
// progress in a host-mapped word: after every column where the host issues the
// steps, at the stop and at the end in recorded cycles and those of small systems.
#include <cstdio>
#include <cstdlib>
#include <cstddef>
#include <vector>

#include "deflate.h"
#include "vms_internal.h"

namespace vms {
namespace {

inline int grid_for(int64_t n, int block = kBlock) { return (int)((n + block - 1) / block); }

// Workgroups are dispatched to the 8 XCDs round-robin by linear id, and each XCD has its own
// L2, which keeps its lines across kernel boundaries.  The Arnoldi kernels (SpMV, dots, update)
// give XCD k the k-th eighth of the rows, so that the slices of a vector one of them writes
// and the next one reads (and most SpMV gathers, the mesh being numbered brick by brick) stay
// in the same XCD's L2: slot of workgroup b in a grid of g (a multiple of 8).
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_slot(int b, int g) { return (b % kXcds) * (g / kXcds) + b / kXcds; }
inline int xcd_round(int g) { return (g + kXcds - 1) / kXcds * kXcds; }

__device__ __forceinline__ double ld_agent(const double* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}


__global__ void fill_kernel(uint4* p, size_t n16) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n16; i += (size_t)gridDim.x * blockDim.x)
        p[i] = make_uint4(0u, 0u, 0u, 0u);
}

// Publishes the cycle's progress (completed columns k, done flag) to the host-mapped word.
__device__ __forceinline__ void report_progress(uint64_t* progress, unsigned gen, int k, int done) {
    const uint64_t word = ((uint64_t)gen << 32) | ((uint64_t)k << 1) | (uint64_t)(done ? 1 : 0);
    __hip_atomic_store(progress, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ void report_progress(GmresState* gs, int k, int done) {
    report_progress(gs->progress, gs->gen, k, done);
}

// The done flag, where a workgroup of the same launch may set it (columns_rotate beside the rows of an
// SpMV or the last dots' sums): whoever misses it does work that no later launch reads.
__device__ __forceinline__ int ld_done(const GmresState* gs) {
    return __hip_atomic_load(&gs->done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void set_done(GmresState* gs) {
    __hip_atomic_store(&gs->done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// What the end of a column needs from the cycle state, loaded ahead.
struct GivensCtx {
    double tol_abs;
    uint64_t* progress;
    unsigned gen;
    int report;             // 1: publish the progress after every column; 0: only when the cycle stops
};

// a . b over four entries, with its roundings written out: left to the compiler, which of the first
// two products is rounded by itself depends on the code around it, and the sums of two kernels that
// have to give the same bits would differ.
template <typename T>
__device__ __forceinline__ T dot4(T a0, T a1, T a2, T a3, T b0, T b1, T b2, T b3) {
    return fma(a3, b3, fma(a2, b2, fma(a0, b0, a1 * b1)));
}
template <typename V4>
__device__ __forceinline__ auto dot4(const V4& a, const V4& b) {
    return dot4(a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w);
}

// Givens rotation of column jc (held in LDS, rows 0 .. jc+1), with the rotations of columns
// 0 .. jc-1 in LDS (cl, sl) and gj the rotated right-hand side entry jc.  The rotated column
// (rows 0 .. jc) goes to Rl in LDS, for the workgroup to store; the rotation, g, the residual
// estimate, k and the done flag go to the cycle state, and the progress is published.
// Returns 1 when the cycle stops.  Called by one whole wave, which issues no memory access in the
// chain (inside a launch that streams vectors, every such access would queue behind the
// stream).  In the chain x_{i+1} = c_i y_i - s_i x_i lane i holds rotation i and hands x_{i+1} to
// lane i + 1 by a DPP shift: a multiply, an FMA and the shift per rotation (lane i's x is right,
// and stays so, from round i on).  One lane fetching the operands from LDS took 65 ns a rotation.
// i0 > 0: rows 0 .. i0-1 of the column were already rotated (Rl) and x0 is row i0.  next: receives the
// right-hand side's entry jc + 1.
__device__ int givens_column(int jc, const double* col, double* cl, double* sl, double gj, double* Rl,
                             const GivensCtx& gc, GmresState* gs, int i0, double x0, double* next = nullptr) {
    const int lane = threadIdx.x & 63;
    double x = i0 > 0 ? x0 : col[0];
    const double hn = col[jc + 1];
    for (int base = i0; base < jc; base += 64) {
        const int i = base + lane, n = min(64, jc - base);
        const bool on = lane < n;
        const double c = on ? cl[i] : 0.0, s = on ? sl[i] : 0.0, y = on ? col[i + 1] : 0.0;
        double xi = x;                                 // what enters rotation i
        for (int k = 1; k < n; ++k) xi = wave_shift(fma(c, y, -(s * xi)), x);
        if (on) Rl[i] = fma(c, xi, s * y);
        x = read_lane(fma(c, y, -(s * xi)), n - 1);
    }
    const double d = hypot(x, hn);
    const double cs = d > 0.0 ? x / d : 1.0;
    const double sn = d > 0.0 ? hn / d : 0.0;
    const double gnext = -sn * gj;
    const bool conv = fabs(gnext) <= gc.tol_abs;
    const bool breakdown = !(hn > 1e-300 * (fabs(d) + 1e-300)) || !isfinite(hn) || !isfinite(gnext);
    const int stop = (conv || breakdown) ? 1 : 0;
    if (lane == 0) {
        Rl[jc] = d;
        gs->cs[jc] = cs;
        gs->sn[jc] = sn;
        cl[jc] = cs;
        sl[jc] = sn;
        gs->g[jc] = cs * gj;
        gs->gin[jc + 1] = gnext;
        gs->k = jc + 1;
        if (stop) set_done(gs);
        if (stop || gc.report) report_progress(gc.progress, gc.gen, jc + 1, stop);
    }
    if (next) *next = gnext;
    return stop;
}

// The rotations that step j makes due, by one workgroup: column j-1 of H became final with the
// update of step j (columns_close), and this rotates it, which gives the residual estimate, k = j
// and, on convergence or breakdown, the done flag; a zero hh (an invariant Krylov space) makes
// column j final too and closes the cycle there.  Nothing of the Arnoldi recurrence waits for it:
// it runs as workgroup 0 of the next step's SpMV launch, the longest of the step's three (inside
// the update it was the last to end, 1.2 us after the streaming workgroups at cavity 32^3).  A
// stop it finds takes effect from that step's dots on; the columns and vectors formed meanwhile
// lie beyond the final basis.  tail: the last vector's second pass (its norm in rho_m), with no
// column j.  dk: the vectors kept by deflated restarting; columns 0 .. dk-1 of
// H are the kept block (rows 0 .. dk), set by the host together with their rotated form (R) and
// Q^T, and step dk starts the Arnoldi recurrence with the cycle's right-hand side c in dr_c.
constexpr int kQtMax = (kDrMax + 1) * (kDrMax + 1);
constexpr int kQtLoads = (kQtMax + kBlock - 1) / kBlock;
__device__ void columns_rotate(int j, int dk, GmresState* gs, int report, bool tail = false) {
    constexpr int ld = kMaxRestart + 1;
    __shared__ double Hc[kMaxRestart + 2];              // the column
    __shared__ double cl[kMaxRestart], sl[kMaxRestart];
    __shared__ double Rl[kMaxRestart + 1];              // the column rotated
    __shared__ double qt[kQtMax];                       // Q^T of the kept block, column-major, ld dk + 1
    __shared__ double src[kDrMax + 1];                  // what it is applied to
    __shared__ double dr_x0;                            // row dk of a column after Q^T
    __shared__ int stop_l;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool dr_first = dk > 0 && j == dk;
    const int jm = max(j - 1, 0);
    // one round of loads, none under a condition of its own lane (indices clamped instead)
    const int row = min(tid, ld - 1), rot = min(tid, kMaxRestart - 1);
    const double h_t = gs->H[(size_t)jm * ld + row], cs_t = gs->cs[rot], sn_t = gs->sn[rot];
    const double rho = tail ? gs->rho_m : gs->rho, hh = gs->hh, gprev = gs->gin[jm];
    const int done = gs->done;
    const GivensCtx gc{gs->tol_abs, gs->progress, gs->gen, report};
    double c_t = 0.0, qt_t[kQtLoads];
    if (dk > 0) {
        c_t = gs->dr_c[min(tid, kDrMax)];
#pragma unroll
        for (int q = 0; q < kQtLoads; ++q) qt_t[q] = gs->dr_qt[min(tid + kBlock * q, kQtMax - 1)];
    }
    if (done) return;                                   // uniform: written by an earlier launch
    if (tid <= j) Hc[tid] = h_t;
    if (tid < j) {
        cl[tid] = cs_t;
        sl[tid] = sn_t;
    }
    if (dk > 0) {
        if (tid <= dk) src[tid] = dr_first ? c_t : h_t;
#pragma unroll
        for (int q = 0; q < kQtLoads; ++q)
            if (tid < kBlock && tid + kBlock * q < kQtMax) qt[tid + kBlock * q] = qt_t[q];
    }
    __syncthreads();
    // Q^T of the kept block on rows 0 .. dk -- of the cycle's right-hand side at step dk, of
    // column j-1 at later steps
    auto apply_qt = [&](double* out) {
        double t = 0.0;
        if (tid <= dk) {
#pragma unroll 4
            for (int l = 0; l <= dk; ++l) t += qt[l * (dk + 1) + tid] * src[l];
            if (tid < dk) out[tid] = t;
            else dr_x0 = t;
        }
    };
    if (dk > 0 && j >= dk) {
        apply_qt(dr_first ? gs->g : Rl);
        __syncthreads();
    }
    if (wave == 0) {
        int st = 0;
        if (dr_first) {
            // the kept block's residual estimate; the columns 0 .. dk-1 are done
            st = (fabs(dr_x0) <= gc.tol_abs || !(rho > 0.0) || !isfinite(dr_x0)) ? 1 : 0;
            if (lane == 0) {
                gs->gin[dk] = dr_x0;
                gs->k = dk;
                if (st) set_done(gs);
                if (st || gc.report) report_progress(gc.progress, gc.gen, dk, st);
            }
        } else if (j > 0) {
            st = givens_column(j - 1, Hc, cl, sl, gprev, Rl, gc, gs, dk, dr_x0);
            if (!(rho > 0.0)) {
                st = 1;                      // u_j vanished: column j-1 closes the cycle
                if (lane == 0) {
                    set_done(gs);
                    report_progress(gc.progress, gc.gen, j, 1);
                }
            }
        }
        if (lane == 0) stop_l = st;
    }
    __syncthreads();
    if (j > 0 && tid < j && !dr_first) gs->R[(size_t)(j - 1) * ld + tid] = Rl[tid];
    if (tail || stop_l || !(rho > 0.0) || hh > 0.0) return;   // uniform
    // the Krylov space is invariant: column j is final with a zero subdiagonal
    __syncthreads();
    if (tid <= j) Hc[tid] = gs->H[(size_t)j * ld + tid];
    if (tid == j) Hc[j + 1] = 0.0;
    if (dk > 0 && tid <= dk) src[tid] = gs->H[(size_t)j * ld + tid];
    __syncthreads();
    if (dk > 0) {
        apply_qt(Rl);
        __syncthreads();
    }
    if (wave == 0) {
        givens_column(j, Hc, cl, sl, gs->gin[j], Rl, gc, gs, dk, dr_x0);
        if (lane == 0) {
            set_done(gs);
            report_progress(gc.progress, gc.gen, j + 1, 1);
        }
    }
    __syncthreads();
    if (tid <= j) gs->R[(size_t)j * ld + tid] = Rl[tid];
}

// ---------------------------------------------------------------------------------- SpMV
// Eight lanes per block row.  Lane (q, r), q = 0, 1 and r = 0..3, owns output dof r and the
// row's blocks q, q + 2, q + 4, ...: it reads row r of each (4 contiguous values) and the
// 4-vector of the column node.  The first kSpmvUnroll blocks of a lane are all loaded before
// any is used, so that its loads are in flight together (a row of this mesh has at most 15
// blocks, i.e. 8 per lane); the two halves of a row are summed with one lane exchange.
// MODE 0: y = A x.  MODE 1: y = b - A x.  MODE 2: y = A x + (kappa S) b with kappa and S (the
// coarse pressure scale and the free-pressure sum of x) taken from the GMRES state.  Grids of at
// most kSpmvXcdMaxGrid workgroups (about one round of residency) take their rows through
// xcd_slot; larger ones keep the linear order, in which the whole chip streams one window of
// the matrix (measured at 64^3: 53.9 us linear, 56.5 us mapped; at 32^3 8.5 and 8.3 us).
constexpr int kSpmvLanes = 8;
constexpr int kSpmvXcdMaxGrid = 2048;
constexpr int kSpmvUnroll = 8;

// Component I of a quad's four values (lane r of the quad holds component r): a DPP quad_perm
// broadcast.  Every lane of the quad must be active.
template <int I>
__device__ __forceinline__ float quad_bcast(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), I * 0x55, 0xF, 0xF, false));
}
template <int I>
__device__ __forceinline__ double quad_bcast(double v) {
    return dpp_mov<I * 0x55>(v);
}

// The four lanes of a block row need the same 4-vector x of the block's column: each loads one
// component and the quad exchanges them by DPP, so that x is requested once per quad instead
// of four times (as many bytes as the matrix block otherwise).  The four lanes share the row
// and the block sequence, so a quad is active or inactive as a whole.
// ROT: the launch of Arnoldi step rot_j + 1, whose workgroup 0 makes the rotations that step rot_j
// left due (columns_rotate); the others take the rows, XCD for XCD as without it.  With MODE 0 that step
// multiplies by the caller's matrix, whose address is the cycle state's: a recorded step serves every
// matrix that the context solves with.
template <typename TA, typename TX, typename TY, typename TACC, int MODE, typename TB = double, bool ROT = false>
__global__ __launch_bounds__(kBlock) void spmv_kernel(int n_rows, const int32_t* __restrict__ rowptr,
                                                      const int32_t* __restrict__ colidx,
                                                      const TA* __restrict__ A, const TX* __restrict__ x,
                                                      const TB* __restrict__ b, TY* __restrict__ y, GmresState* gs,
                                                      int rot_j = 0, int dk = 0, int report = 0) {
    int slot;
    if (ROT && MODE == 0) A = static_cast<const TA*>(gs->A);
    if (ROT) {
        if (blockIdx.x == 0) {
            __builtin_amdgcn_s_setprio(3);
            if (rot_j >= dk) columns_rotate(rot_j, dk, gs, report);
            return;
        }
        const int g = gridDim.x - 1, q = blockIdx.x % kXcds;      // workgroup b runs on XCD b mod 8
        slot = g <= kSpmvXcdMaxGrid ? q * (g / kXcds) + blockIdx.x / kXcds - (q == 0 ? 1 : 0) : blockIdx.x - 1;
    } else {
        slot = gridDim.x <= kSpmvXcdMaxGrid ? xcd_slot(blockIdx.x, gridDim.x) : blockIdx.x;
    }
    // a finished GMRES cycle reads no blocks and stores nothing; the flag is read alongside the
    // row bounds, which the block loads wait for anyway
    const int skip = ROT ? ld_done(gs) : 0;
    constexpr int Q = kSpmvLanes / 4;
    // the blocks of A P are the context's, the others may be a caller's
    using VA = typename std::conditional_t<ROT && MODE == 2, Vec4<TA>, CallerVec4<TA>>::type;
    const int tid = slot * blockDim.x + threadIdx.x;
    const int row = tid / kSpmvLanes, sub = tid % kSpmvLanes;
    const int q = sub >> 2, r = sub & 3;
    TACC acc = TACC(0);
    if (row < n_rows) {
        const int k0 = rowptr[row], k1 = skip ? k0 : rowptr[row + 1];
        int cols[kSpmvUnroll];
#pragma unroll
        for (int u = 0; u < kSpmvUnroll; ++u) {
            const int k = k0 + q + u * Q;
            cols[u] = k < k1 ? colidx[k] : -1;
        }
        VA av[kSpmvUnroll];
        TX xr[kSpmvUnroll];
#pragma unroll
        for (int u = 0; u < kSpmvUnroll; ++u) {
            if (cols[u] >= 0) {
                av[u] = *reinterpret_cast<const VA*>(A + (size_t)(k0 + q + u * Q) * 16 + r * 4);
                xr[u] = x[(size_t)cols[u] * 4 + r];
            } else {
                av[u] = VA{TA(0), TA(0), TA(0), TA(0)};
                xr[u] = TX(0);
            }
        }
#pragma unroll
        for (int u = 0; u < kSpmvUnroll; ++u) {
            const TX x0 = quad_bcast<0>(xr[u]), x1 = quad_bcast<1>(xr[u]), x2 = quad_bcast<2>(xr[u]),
                     x3 = quad_bcast<3>(xr[u]);
            acc += dot4<TACC>(av[u].x, av[u].y, av[u].z, av[u].w, x0, x1, x2, x3);
        }
        // rows longer than kSpmvUnroll blocks per lane (other meshes)
        for (int k = k0 + q + kSpmvUnroll * Q; k < k1; k += Q) {
            const VA a = *reinterpret_cast<const VA*>(A + (size_t)k * 16 + r * 4);
            const TX xc = x[(size_t)colidx[k] * 4 + r];
            const TX x0 = quad_bcast<0>(xc), x1 = quad_bcast<1>(xc), x2 = quad_bcast<2>(xc), x3 = quad_bcast<3>(xc);
            acc += dot4<TACC>(a.x, a.y, a.z, a.w, x0, x1, x2, x3);
        }
    }
    acc += __shfl_xor(acc, 4, 64);       // lanes 4q + r of a row: q = 0 and q = 1
    if (row < n_rows && q == 0 && !skip) {
        if (MODE == 1)
            y[4 * (size_t)row + r] = TY(TACC(b[4 * (size_t)row + r]) - acc);
        else if (MODE == 2)
            y[4 * (size_t)row + r] = TY(acc + TACC(gs->kappa * gs->su) * TACC(b[4 * (size_t)row + r]));
        else
            y[4 * (size_t)row + r] = TY(acc);
    }
}

inline int spmv_grid(int n_rows) { return xcd_round((int)(((int64_t)kSpmvLanes * n_rows + kBlock - 1) / kBlock)); }

// --------------------------------------------------------------------------- block-Jacobi
// Inverse of each 4x4 diagonal block in FP64 (Gauss-Jordan, partial pivoting),
// stored in the preconditioner precision.  A singular block is replaced by the
// identity and counted in flags[2].
// Inverts the FP64 4x4 block D into out (precision TM); a singular block becomes the
// identity and is counted in flags[2].
template <typename TM>
__device__ void invert_block_store(const double (&D)[4][4], TM* __restrict__ out, int32_t* flags) {
    double m[4][4];
    const bool ok = invert4(D, m);
    if (!ok) atomicAdd(&flags[2], 1);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) out[r * 4 + c] = ok ? TM(m[r][c]) : TM(r == c ? 1 : 0);
}

template <typename TA, typename TM>
__global__ void bj_setup_kernel(int n, const int32_t* __restrict__ diagpos, const TA* __restrict__ A,
                                TM* __restrict__ Minv, int32_t* flags) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const TA* Dp = A + (size_t)diagpos[i] * 16;
    double D[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int c = 0; c < 4; ++c) D[r][c] = double(Dp[r * 4 + c]);
    invert_block_store<TM>(D, Minv + (size_t)i * 16, flags);
}

// Uncondensed system (node rows 0..nn, element rows after them; each element row holds the
// element's K_fc blocks, its K_ff block padded to 4x4 and nothing else).  The node diagonal
// blocks of that system have a zero pressure-pressure entry, so their plain inverse is no
// preconditioner.  Node row i instead gets the inverse of the diagonal block of the Schur
// complement, K_cc(i,i) - sum_e K_cf(i,e) K_ff(e)^-1 K_fc(e,i) (Section 5), formed from the
// assembled blocks and the element rows' inverses already in Minv.
template <typename TA, typename TM>
__global__ void schur_diag_pc_kernel(int nn, const int32_t* __restrict__ rowptr, const int32_t* __restrict__ colidx,
                                     const int32_t* __restrict__ diagpos, const TA* __restrict__ A,
                                     TM* __restrict__ Minv, int32_t* flags) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nn) return;
    double D[4][4];
    {
        const TA* Dp = A + (size_t)diagpos[i] * 16;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) D[r][c] = double(Dp[r * 4 + c]);
    }
    for (int k = rowptr[i]; k < rowptr[i + 1]; ++k) {
        const int e = colidx[k];
        if (e < nn) continue;
        int kf = -1;                                   // block (e, i) in element row e
        for (int q = rowptr[e]; q < rowptr[e + 1]; ++q)
            if (colidx[q] == i) kf = q;
        if (kf < 0) continue;
        const TA* Cf = A + (size_t)k * 16;
        const TA* Fc = A + (size_t)kf * 16;
        const TM* P = Minv + (size_t)e * 16;
        double W[4][4];                                // K_ff^-1 K_fc (padded)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                double t = 0.0;
#pragma unroll
                for (int q = 0; q < 3; ++q) t += double(P[r * 4 + q]) * double(Fc[q * 4 + c]);
                W[r][c] = t;
            }
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                double t = 0.0;
#pragma unroll
                for (int q = 0; q < 3; ++q) t += double(Cf[r * 4 + q]) * W[q][c];
                D[r][c] -= t;
            }
    }
    invert_block_store<TM>(D, Minv + (size_t)i * 16, flags);
}

// ------------------------------------------------------------------------ reductions
// Block-level sum of NV values per thread into s[0..NV) (result valid in thread 0).
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* lds) {
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = wave_sum(v[q]);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int q = 0; q < NV; ++q) lds[w * NV + q] = v[q];
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            double t = 0.0;
            for (int ww = 0; ww < kBlock / 64; ++ww) t += lds[ww * NV + q];
            v[q] = t;
        }
    }
}

// Last-arriving workgroup detection (partials written before the fence).
__device__ __forceinline__ bool arrive_last(unsigned* counter) {
    __shared__ bool last;
    if (threadIdx.x == 0) {
        __threadfence();
        const unsigned prev = atomicAdd(counter, 1u);
        last = prev == gridDim.x - 1;
    }
    __syncthreads();
    return last;
}

// Inside the last-arriving workgroup: out[i] = sum_k part[i * ld + k], k < nk, for i < nvec.
// Threads form groups of P lanes (P a power of two, P <= 64) per vector; each lane sums a
// fixed stride of partials and the group combines them with shuffles (fixed order).
__device__ void reduce_partials(const double* part, int ld, int nvec, int nk, double* out) {
    int P = 64;
    while (P > 1 && P * nvec > (int)blockDim.x) P >>= 1;
    const int i = threadIdx.x / P, lane = threadIdx.x % P;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    if (i < nvec) {
        const double* pi = part + (size_t)i * ld;
        int k = lane;
        for (; k + 3 * P < nk; k += 4 * P) {
            s0 += ld_agent(pi + k);
            s1 += ld_agent(pi + k + P);
            s2 += ld_agent(pi + k + 2 * P);
            s3 += ld_agent(pi + k + 3 * P);
        }
        for (; k < nk; k += P) s0 += ld_agent(pi + k);
    }
    double sum = (s0 + s1) + (s2 + s3);
    for (int off = P / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, 64);
    if (i < nvec && lane == 0) out[i] = sum;
}

// dof idx is a pressure dof without a Dirichlet condition
__device__ __forceinline__ bool free_pressure(const uint8_t* __restrict__ dmask, int idx) {
    return (idx & 3) == 3 && !(dmask[idx >> 2] & 8u);
}

// Coarse correction on the constant pressure mode: kappa = 1 / sum of the entries of A
// that couple two free pressure dofs (= 1 / (z^T A z) for z = 1 on the free pressure dofs).
// That sum is the Galerkin coarse operator of the mode.  It is only meaningful when the mode
// is nearly singular because one pressure dof is pinned: there the sum is the coupling to the
// pinned dof, about 1 / (2 n_nodes) of the summed magnitudes.  Without a pin (open or
// traction-free boundaries) the pressure-pressure block annihilates constants and the sum is
// rounding noise: the caller then passes enabled = 0 (the noise of FP32-stored entries can
// exceed any fixed fraction of the magnitudes, and kappa = 1 / noise would swamp the Krylov
// space).  As a guard, the correction is also off when |sum| <= 1e-8 x the summed magnitudes.
// The entries come packed from ap_rows_kernel (pp: one per block, zero where they do not count), kPpAhead
// of a row in flight.  Read from the matrix, one by one behind their columns' masks and 64 bytes
// apart, they took 172 us at 64^3 (mixed) and 31 us at 32^3; now 21 and 9.  With n_nodes = 0, kappa is 0.
constexpr int kPpAhead = 8;
template <typename TA>
__global__ __launch_bounds__(kBlock) void coarse_setup_kernel(int n_nodes, const int32_t* __restrict__ rowptr,
                                                              const TA* __restrict__ pp, RedScratch* red,
                                                              GmresState* gs) {
    __shared__ double lds[(kBlock / 64) * 2];
    double v[2] = {0.0, 0.0};
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_nodes; i += gridDim.x * blockDim.x) {
        const int k1 = rowptr[i + 1];
        for (int k = rowptr[i]; k < k1; k += kPpAhead) {
            TA a[kPpAhead];
#pragma unroll
            for (int q = 0; q < kPpAhead; ++q) a[q] = pp[min(k + q, k1 - 1)];
#pragma unroll
            for (int q = 0; q < kPpAhead; ++q)
                if (k + q < k1) {
                    v[0] += double(a[q]);
                    v[1] += fabs(double(a[q]));
                }
        }
    }
    block_sum<2>(v, lds);
    if (threadIdx.x == 0) {
        red->partial[blockIdx.x] = v[0];
        red->partial[kRedBlocks + blockIdx.x] = v[1];
    }
    if (!arrive_last(&red->counter)) return;
    __threadfence();
    __shared__ double tot[2];
    reduce_partials(red->partial, kRedBlocks, 2, gridDim.x, tot);
    __syncthreads();
    if (threadIdx.x == 0) {
        const bool usable = isfinite(tot[0]) && fabs(tot[0]) > 1e-8 * tot[1];
        gs->kappa = usable ? 1.0 / tot[0] : 0.0;
        red->counter = 0u;
    }
}

// Coarse vector of the uncondensed system: 1 on the free node pressures and, on each element
// row, the fine response -K_ff^-1 K_fc 1_p (K_fc columns of prescribed dofs are zero).  The
// response vanishes up to rounding unless the element touches a pinned pressure (the
// gradients of an element sum to zero); with it, 1_p^T A z equals the Schur complement's
// 1_p^T S 1_p, which the plain indicator (zero pressure-pressure block) would miss.
template <typename TA, typename TM>
__global__ void full_coarse_vector_kernel(int nn, int n_rows, const int32_t* __restrict__ rowptr,
                                          const int32_t* __restrict__ colidx, const TA* __restrict__ A,
                                          const TM* __restrict__ Minv, const uint8_t* __restrict__ dmask,
                                          double* __restrict__ zvec) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_rows) return;
    double* zi = zvec + 4 * (size_t)i;
    if (i < nn) {
        zi[0] = zi[1] = zi[2] = 0.0;
        zi[3] = (dmask[i] & 8u) ? 0.0 : 1.0;
        return;
    }
    double t[3] = {0.0, 0.0, 0.0};
    for (int k = rowptr[i]; k < rowptr[i + 1]; ++k) {
        const int b = colidx[k];
        if (b >= nn || (dmask[b] & 8u)) continue;
#pragma unroll
        for (int q = 0; q < 3; ++q) t[q] += double(A[(size_t)k * 16 + 4 * q + 3]);
    }
    const TM* P = Minv + (size_t)i * 16;
#pragma unroll
    for (int r = 0; r < 3; ++r)
        zi[r] = -(double(P[4 * r]) * t[0] + double(P[4 * r + 1]) * t[1] + double(P[4 * r + 2]) * t[2]);
    zi[3] = 0.0;
}

// kappa = 1 / (1_p^T A z) for the explicit coarse vector z, switched off (as for the condensed
// system) when the sum is below 1e-8 x the summed magnitudes of the free pressure rows' terms.
template <typename TA>
__global__ __launch_bounds__(kBlock) void full_coarse_setup_kernel(int nn, const int32_t* __restrict__ rowptr,
                                                                   const int32_t* __restrict__ colidx,
                                                                   const TA* __restrict__ A,
                                                                   const uint8_t* __restrict__ dmask,
                                                                   const double* __restrict__ zvec, int enabled,
                                                                   RedScratch* red, GmresState* gs) {
    __shared__ double lds[(kBlock / 64) * 2];
    double v[2] = {0.0, 0.0};
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nn; i += gridDim.x * blockDim.x) {
        if (dmask[i] & 8u) continue;
        for (int k = rowptr[i]; k < rowptr[i + 1]; ++k) {
            const double* zc = zvec + 4 * (size_t)colidx[k];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const double a = double(A[(size_t)k * 16 + 12 + q]);
                v[0] += a * zc[q];
                v[1] += fabs(a * zc[q]);
            }
        }
    }
    block_sum<2>(v, lds);
    if (threadIdx.x == 0) {
        red->partial[blockIdx.x] = v[0];
        red->partial[kRedBlocks + blockIdx.x] = v[1];
    }
    if (!arrive_last(&red->counter)) return;
    __threadfence();
    __shared__ double tot[2];
    reduce_partials(red->partial, kRedBlocks, 2, gridDim.x, tot);
    __syncthreads();
    if (threadIdx.x == 0) {
        const bool usable = isfinite(tot[0]) && fabs(tot[0]) > 1e-8 * tot[1];
        gs->kappa = (enabled && usable) ? 1.0 / tot[0] : 0.0;
        red->counter = 0u;
    }
}

// A cycle's initial residual r: per workgroup the partial sums of its squares and of its free
// pressure entries (added by cycle_v0_kernel, so that no workgroup has to wait for the last one).
// With r64, r is first formed as r64 scaled (FP32 cycles start from the FP64 residual scaled to
// one); with x_save, the iterate is kept there before a deflated cycle.
template <typename T>
__global__ __launch_bounds__(kBlock) void cycle_norm_kernel(int n, const double* __restrict__ r64, double scale,
                                                            T* __restrict__ r, const double* __restrict__ x,
                                                            double* __restrict__ x_save,
                                                            const uint8_t* __restrict__ dmask, RedScratch* red) {
    __shared__ double lds[(kBlock / 64) * 2];
    double v[2] = {0.0, 0.0};
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        if (r64) r[i] = T(r64[i] * scale);
        if (x_save) x_save[i] = x[i];
        const double e = double(r[i]);
        v[0] += e * e;
        if (free_pressure(dmask, i)) v[1] += e;
    }
    block_sum<2>(v, lds);
    if (threadIdx.x == 0) {
        red->partial[blockIdx.x] = v[0];
        red->partial[kRedBlocks + blockIdx.x] = v[1];
    }
}

// Starts the cycle from the nparts partials: its norm to gs->beta, g = beta e_1, k = 0, the done
// flag and the matrix of a cycle that applies P and A one after the other (workgroup 0), and
// V[0] = r / beta (V0 = V + j0 n for a deflated cycle).  Every workgroup adds the partials itself, in
// the same order.
template <typename T>
__global__ __launch_bounds__(kBlock) void cycle_v0_kernel(int n, const T* __restrict__ r, T* __restrict__ V0,
                                                          int nparts, const RedScratch* red, GmresState* gs,
                                                          double tol_abs, int reorth, unsigned gen,
                                                          const void* A) {
    __shared__ double tot[2];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    const double e = i < n ? double(r[i]) : 0.0;
    reduce_partials(red->partial, kRedBlocks, 2, nparts, tot);
    __syncthreads();
    const double nrm = sqrt(tot[0]);
    if (i < n) V0[i] = nrm > 0.0 ? T(e / nrm) : T(0);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        gs->su = nrm > 0.0 ? tot[1] / nrm : 0.0;
        gs->beta = nrm;
        gs->g[0] = nrm;
        gs->gin[0] = nrm;
        gs->k = 0;
        gs->tol_abs = tol_abs;
        gs->done = (nrm <= tol_abs || !(nrm > 0.0)) ? 1 : 0;
        gs->reorth = reorth;
        gs->gen = gen;
        gs->A = A;
        report_progress(gs, 0, gs->done);
    }
}

// Deflated restarting: V[c] = sum_l P(l, c) V[l] for the kept columns c < kk (l < mv), in
// place -- each thread owns one entry of every vector and reads all of them before it writes.
// P is staged in LDS (every thread reads the same entry: a broadcast); KMAX >= kk bounds the
// accumulators.
template <typename T, int KMAX>
__global__ __launch_bounds__(kBlock) void dr_basis_kernel(int n, int mv, int kk, const double* __restrict__ P,
                                                          int ldp, T* __restrict__ V) {
    __shared__ double Pl[(kMaxRestart + 1) * KMAX];     // Pl[l KMAX + c]
    for (int e = threadIdx.x; e < mv * KMAX; e += blockDim.x) {
        const int l = e / KMAX, c = e % KMAX;
        Pl[e] = c < kk ? P[(size_t)c * ldp + l] : 0.0;
    }
    __syncthreads();
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const size_t N = (size_t)n;
    double acc[KMAX];
#pragma unroll
    for (int c = 0; c < KMAX; ++c) acc[c] = 0.0;
#pragma unroll 4
    for (int l = 0; l < mv; ++l) {
        const double v = double(V[(size_t)l * N + i]);
#pragma unroll
        for (int c = 0; c < KMAX; ++c) acc[c] += Pl[l * KMAX + c] * v;
    }
#pragma unroll
    for (int c = 0; c < KMAX; ++c)
        if (c < kk) V[(size_t)c * N + i] = T(acc[c]);
}

template <typename T>
void launch_dr_basis(int n, int mv, int kk, const double* P, int ldp, T* V, hipStream_t s) {
    if (kk <= 12)
        dr_basis_kernel<T, 12><<<grid_for(n), kBlock, 0, s>>>(n, mv, kk, P, ldp, V);
    else if (kk <= 20)
        dr_basis_kernel<T, 20><<<grid_for(n), kBlock, 0, s>>>(n, mv, kk, P, ldp, V);
    else
        dr_basis_kernel<T, kDrMax><<<grid_for(n), kBlock, 0, s>>>(n, mv, kk, P, ldp, V);
}

// Deflated restarting: the kept block of H and its factors from the host's packed staging (mapped
// memory, read here once) into the cycle state (columns 0 .. kk-1 of H and R, zero below their last
// row), and the np basis coefficients P into Pd for dr_basis_kernel.  One workgroup.
constexpr int kDrLoadThreads = 1024;
__global__ __launch_bounds__(kDrLoadThreads) void dr_load_kernel(int kk, int np, const double* __restrict__ up,
                                                                 double* __restrict__ Pd, GmresState* gs) {
    constexpr int ld = kMaxRestart + 1;
    const int tid = threadIdx.x;
    for (int e = tid; e < np; e += kDrLoadThreads) Pd[e] = up[e];
    for (int e = tid; e < kk * ld; e += kDrLoadThreads) {
        const int col = e / ld, row = e % ld;
        gs->H[e] = row <= kk ? up[kDrOffH + col * (kk + 1) + row] : 0.0;
        gs->R[e] = row < kk ? up[kDrOffR + col * kk + row] : 0.0;
    }
    for (int e = tid; e < (kk + 1) * (kk + 1); e += kDrLoadThreads) gs->dr_qt[e] = up[kDrOffQt + e];
    for (int e = tid; e < kk; e += kDrLoadThreads) gs->svs[e] = up[kDrOffSvs + e];
}

// A P for the Arnoldi steps: block (i, b) times the preconditioner block of node b, so that
// the step's SpMV applies the preconditioner on the fly.  Four lanes per block, lane r forms
// row r; the product is summed in FP64 and stored in T.
template <typename T, typename V4>
__device__ __forceinline__ T ap_entry(const V4& a, T m0, T m1, T m2, T m3) {
    return T(dot4<double>(a.x, a.y, a.z, a.w, m0, m1, m2, m3));
}
// The same with lane q of the quad holding row q's entry of the column.
template <typename T, typename V4>
__device__ __forceinline__ T ap_quad(const V4& a, T m) {
    return ap_entry<T>(a, quad_bcast<0>(m), quad_bcast<1>(m), quad_bcast<2>(m), quad_bcast<3>(m));
}
template <typename T>
__global__ void ap_blocks_kernel(int64_t nb, const int32_t* __restrict__ colidx, const T* __restrict__ A,
                                 const T* __restrict__ Minv, T* __restrict__ AP) {
    const int64_t tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t k = tid >> 2;
    const int r = (int)(tid & 3);
    if (k >= nb) return;
    using V4 = typename Vec4<T>::type;
    const auto a = *reinterpret_cast<const typename CallerVec4<T>::type*>(A + k * 16 + r * 4);
    const T* M = Minv + (size_t)colidx[k] * 16;
    T o[4];
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) o[cc] = ap_entry<T>(a, M[cc], M[4 + cc], M[8 + cc], M[12 + cc]);
    *reinterpret_cast<V4*>(AP + k * 16 + r * 4) = V4{o[0], o[1], o[2], o[3]};
}

// The same by rows, with what the coarse pressure mode needs of A: A z for z = 1 on every free pressure
// dof (per row, the sum of the pressure columns of the blocks whose column node has a free pressure,
// in order), and, if pp is given, the entries that couple two free pressures.  Four lanes per block
// row, lane r holding row r of the block and of its column's preconditioner block; kApAhead blocks in
// flight.  As three launches that each read the matrix, this and the sum of pp took 363 us at 64^3
// (mixed) and 60 us at 32^3; now 115 + 21 and 17 + 9.  With 8 FP32 blocks in flight 144 and 18.6; with
// every lane loading the whole preconditioner block (4 in flight) 168 and 20.
template <typename T>
__global__ __launch_bounds__(kBlock) void ap_rows_kernel(int n_rows, const int32_t* __restrict__ rowptr,
                                                         const int32_t* __restrict__ colidx, const T* __restrict__ A,
                                                         const T* __restrict__ Minv, const uint8_t* __restrict__ dmask,
                                                         T* __restrict__ AP, T* __restrict__ Az, T* __restrict__ pp) {
    constexpr int kApAhead = 64 / sizeof(T);             // most rows of a tetrahedral mesh at once in FP32
    using V4 = typename Vec4<T>::type;
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    const int row = tid >> 2, r = tid & 3;
    if (row >= n_rows) return;
    const int k1 = rowptr[row + 1];
    const bool row_free = !(dmask[row] & 8u);
    double acc = 0.0;
    for (int kb = rowptr[row]; kb < k1; kb += kApAhead) {
        typename CallerVec4<T>::type a[kApAhead];
        V4 m[kApAhead];
        bool col_free[kApAhead];
#pragma unroll
        for (int u = 0; u < kApAhead; ++u) {
            const int k = min(kb + u, k1 - 1), col = colidx[k];
            a[u] = *reinterpret_cast<const typename CallerVec4<T>::type*>(A + (size_t)k * 16 + r * 4);
            col_free[u] = !(dmask[col] & 8u);
            m[u] = *reinterpret_cast<const V4*>(Minv + (size_t)col * 16 + r * 4);
        }
#pragma unroll
        for (int u = 0; u < kApAhead; ++u) {
            if (kb + u >= k1) continue;                  // the four lanes of a row agree
            const size_t k = (size_t)kb + u;
            *reinterpret_cast<V4*>(AP + k * 16 + r * 4) =
                V4{ap_quad<T>(a[u], m[u].x), ap_quad<T>(a[u], m[u].y), ap_quad<T>(a[u], m[u].z),
                   ap_quad<T>(a[u], m[u].w)};
            if (col_free[u]) acc += double(a[u].w);
            if (pp && r == 3) pp[k] = row_free && col_free[u] ? a[u].w : T(0);
        }
    }
    Az[4 * (size_t)row + r] = T(acc);
}

// t = P v = Minv v + z kappa S(v), S(v) = gs->su (the free-pressure sum of the step's vector):
// the preconditioner of an Arnoldi step applied on its own, for steps whose matrix is stored
// in a lower precision than the basis (the step then multiplies by A itself, so that its
// operator is exactly A P, the one the FP64 residual and the correction P V y see).  Idle once
// the cycle has stopped.
template <typename TM, typename T>
__global__ void precond_apply_kernel(int n_nodes, const TM* __restrict__ Minv, const T* __restrict__ v,
                                     const uint8_t* __restrict__ dmask, const double* __restrict__ zvec,
                                     const GmresState* gs, T* __restrict__ t) {
    if (gs->done) return;
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    const int node = tid >> 2, r = tid & 3;
    if (node >= n_nodes) return;
    using M4 = typename Vec4<TM>::type;
    using V4 = typename Vec4<T>::type;
    const M4 m = *reinterpret_cast<const M4*>(Minv + (size_t)node * 16 + r * 4);
    const V4 x = *reinterpret_cast<const V4*>(v + 4 * (size_t)node);
    double acc = double(m.x) * double(x.x) + double(m.y) * double(x.y) + double(m.z) * double(x.z) +
                 double(m.w) * double(x.w);
    if (zvec)
        acc += gs->kappa * gs->su * zvec[4 * (size_t)node + r];
    else if (r == 3 && !(dmask[node] & 8u))
        acc += gs->kappa * gs->su;
    t[4 * (size_t)node + r] = T(acc);
}

// ------------------------------------------------------------------- Arnoldi step kernels
// Gram-Schmidt with delayed reorthogonalisation and a single reduction per step (the DCGS2
// scheme of Swirydowicz et al. / Bielich et al., written here for right-preconditioned
// Arnoldi).  Entering step j, q_0 .. q_{j-1} are final and V[j] holds u_j, the next vector
// after one classical Gram-Schmidt pass, normalised by an estimate; column j-1 of H is
// provisional.  B = A P is the preconditioned operator, S(v) the sum of the free pressure
// entries of v.
//   spmv         w = (A P) u_j + kappa S(u_j) A z = B u_j, from the stored blocks of A P (S(u_j)
//                carried in gs); a step whose matrix is stored in a lower precision than its
//                basis instead applies P (precond_apply) and then A
//   dots         slots per (chunk, y): y < j -> (q_y . u_j, q_y . w);  y = j -> (u_j . u_j,
//                u_j . w);  y = j + 1 -> (w . w, S(w))    -> part[slot][chunk], stride = chunks
//   update       every workgroup sums the slots itself (step_scalars, same order everywhere):
//                s = Q^T u_j, rho = sqrt(u_j . u_j - |s|^2), so that q_j = (u_j - Q s)/rho is
//                u_j's second pass; with t = Q^T w and c = (t, c_j), c_j = (u_j . w - s . t) / rho
//                = q_j . w, and the provisional subdiagonal of column j is
//                hh = sqrt(w . w - |c|^2) / rho (Pythagoras).  Then q_j = (u_j - Q s) / rho over
//                V[j] and u_{j+1} = (w - Q t - c_j q_j) / (rho hh) to V[j+1].  Workgroup 0
//                instead does the Hessenberg columns (columns_close): column j-1 becomes final,
//                H(0:j-1, j-1) += hh' s and H(j, j-1) = hh' rho (hh': its provisional
//                subdiagonal), and H(0:j, j) = (c - H s) / rho, H(j+1, j) = hh.  The Givens
//                rotation of column j-1, the residual estimate and the done flag follow in
//                workgroup 0 of the next step's spmv (columns_rotate).
// Three launches per step (a separate one-workgroup reduction cost more than every update
// workgroup summing the partials of kFusedChunks chunks again).  The tail of a cycle, the
// second pass of the last vector, is dots + reduce_kernel + columns_kernel.
// An estimate that loses digits to cancellation only scales u_{j+1}; the next step measures
// its norm directly (u . u), so the final subdiagonal hh rho is exact to rounding.  With
// reorthogonalisation off, s is taken as 0 (one Gram-Schmidt pass, the norm still measured).
// The chunks of a slot go to the XCDs through xcd_slot (when their count is a multiple of 8),
// matching the rows the update and the SpMV give each XCD.
constexpr int kDotChunks = VMS_DOT_CHUNKS;       // bound on the chunks (partials) per dot slot
constexpr int kDotThreads = 256;
constexpr int kDotUnrollF32 = 3;     // strides per pass for FP32 vectors (FP64: 1, register-bound)
static_assert(2 * (kMaxRestart + 2) * kDotChunks <= kRedBlocks * (kMaxRestart + 1), "dot slots exceed scratch");


// One thread's share of a chunk [i0, i1) of one dot slot: KIND 0 (q . u, q . w), 1 (u . u, u . w),
// 2 (w . w, S(w)).  kDotUnroll strides per pass, all loaded before any is used; indices past
// the chunk are clamped to its last node and weighted 0 (no branch around a load).  Three
// strides for FP32 vectors (the slot's loads then take one memory round at 32^3); FP64 keeps
// one, where nine 32-byte loads in flight cost more occupancy than they save.
template <int KIND, typename V4>
__device__ __forceinline__ void dot_chunk(const V4* __restrict__ q4, const V4* __restrict__ u4,
                                          const V4* __restrict__ w4, const uint8_t* __restrict__ dmask, int i0,
                                          int i1, double& a0, double& a1) {
    constexpr int kDotUnroll = sizeof(V4) <= 16 ? kDotUnrollF32 : 1;
    for (int ib = i0 + (int)threadIdx.x; ib < i1; ib += kDotUnroll * (int)blockDim.x) {
        V4 bv[kDotUnroll], xv[kDotUnroll], uv[kDotUnroll];
        uint8_t mk[kDotUnroll];
#pragma unroll
        for (int r = 0; r < kDotUnroll; ++r) {
            const int i = min(ib + r * (int)blockDim.x, i1 - 1);
            bv[r] = w4[i];
            if (KIND == 0) xv[r] = q4[i];
            if (KIND <= 1) uv[r] = u4[i];
            if (KIND == 2) mk[r] = dmask[i];
        }
#pragma unroll
        for (int r = 0; r < kDotUnroll; ++r) {
            const double wt = ib + r * (int)blockDim.x < i1 ? 1.0 : 0.0;
            const V4 b = bv[r];
            if (KIND == 0) {
                const V4 q = xv[r], u = uv[r];
                a0 += wt * double(dot4(q, u));
                a1 += wt * double(dot4(q, b));
            } else if (KIND == 1) {
                const V4 u = uv[r];
                a0 += wt * double(dot4(u, u));
                a1 += wt * double(dot4(u, b));
            } else {
                a0 += wt * double(dot4(b, b));
                a1 += (mk[r] & 8u) ? 0.0 : wt * double(b.w);
            }
        }
    }
}

// The same for G finished vectors x, which share the loads of u and w: a vector by itself costs three
// loads per entry, two a pair four, and the large meshes' dots are bound by what the L2s deliver.
template <int G, typename V4>
__device__ __forceinline__ void dot_chunk_group(const V4* const (&x)[G], const V4* __restrict__ u4,
                                                const V4* __restrict__ w4, int i0, int i1, double (&a)[2 * G]) {
    constexpr int kDotUnroll = sizeof(V4) <= 16 ? kDotUnrollF32 : 1;
    for (int ib = i0 + (int)threadIdx.x; ib < i1; ib += kDotUnroll * (int)blockDim.x) {
        V4 bv[kDotUnroll], uv[kDotUnroll], xv[kDotUnroll][G];
#pragma unroll
        for (int r = 0; r < kDotUnroll; ++r) {
            const int i = min(ib + r * (int)blockDim.x, i1 - 1);
            bv[r] = w4[i];
            uv[r] = u4[i];
#pragma unroll
            for (int g = 0; g < G; ++g) xv[r][g] = x[g][i];
        }
#pragma unroll
        for (int r = 0; r < kDotUnroll; ++r) {
            const double wt = ib + r * (int)blockDim.x < i1 ? 1.0 : 0.0;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                a[2 * g] += wt * double(dot4(xv[r][g], uv[r]));
                a[2 * g + 1] += wt * double(dot4(xv[r][g], bv[r]));
            }
        }
    }
}

// Workgroup rows 0 .. ceil(j / G) - 1 take G finished vectors each, the next one u_j, the last one w.
template <typename T, int G>
__global__ __launch_bounds__(kDotThreads) void dots_kernel(int n_nodes, int j, const T* __restrict__ V,
                                                           const T* __restrict__ w,
                                                           const uint8_t* __restrict__ dmask,
                                                           double* __restrict__ part, const GmresState* gs) {
    // a finished cycle reads nothing (the replayed steps after convergence cost only their
    // launches); its partials are left as they are, and the update and the tail test the flag too
    if (gs->done) return;
    using V4 = typename Vec4<T>::type;
    const int groups = (j + G - 1) / G;
    const int row = blockIdx.y;
    const int y = row < groups ? G * row : j + (row - groups);       // the first vector
    const size_t N4 = (size_t)n_nodes;          // float4 / double4 entries per vector
    const V4* v4 = reinterpret_cast<const V4*>(V);
    const V4* u4 = v4 + (size_t)j * N4;
    const V4* w4 = reinterpret_cast<const V4*>(w);
    const int per = (n_nodes + gridDim.x - 1) / gridDim.x;
    const int chunk = gridDim.x % kXcds == 0 ? xcd_slot(blockIdx.x, gridDim.x) : blockIdx.x;
    const int i0 = chunk * per, i1 = min(n_nodes, i0 + per);
    double a[2 * G] = {};
    int slots = 2;
    if (row < groups) {
        if constexpr (G == 1) {
            dot_chunk<0>(v4 + (size_t)y * N4, u4, w4, dmask, i0, i1, a[0], a[1]);
        } else {
            // the last group's missing vectors repeat its last one and are not stored
            slots = 2 * min(G, j - y);
            const V4* x[G];
#pragma unroll
            for (int g = 0; g < G; ++g) x[g] = v4 + (size_t)min(y + g, j - 1) * N4;
            dot_chunk_group<G>(x, u4, w4, i0, i1, a);
        }
    } else if (y == j) {
        dot_chunk<1>(v4, u4, w4, dmask, i0, i1, a[0], a[1]);
    } else {
        dot_chunk<2>(v4, u4, w4, dmask, i0, i1, a[0], a[1]);
    }
    __shared__ double lds[2 * G][kDotThreads / 64];
#pragma unroll
    for (int q = 0; q < 2 * G; ++q) {
        a[q] = wave_sum(a[q]);
        if ((threadIdx.x & 63) == 0) lds[q][threadIdx.x >> 6] = a[q];
    }
    __syncthreads();
    if ((int)threadIdx.x < slots) {
        double t = 0.0;
        for (int k = 0; k < kDotThreads / 64; ++k) t += lds[threadIdx.x][k];
        part[(size_t)(2 * y + threadIdx.x) * gridDim.x + chunk] = t;
    }
}

// The Hessenberg bookkeeping of step j, for one workgroup of kBlock threads.  It needs the
// step's sums, and nothing of the Arnoldi recurrence waits for it, so it runs as workgroup 0 of
// the update launch, with the sums that workgroup formed in LDS (in), and, for the cycle's
// tail, as a launch of its own after reduce_kernel (in = nullptr: column j-1 only, inputs from
// the cycle state).
//  * u_j's second pass makes column j-1 final: H(0:j-1, j-1) += hh' s and H(j, j-1) = hh' rho,
//    hh' being the provisional subdiagonal stored at step j-1; columns_rotate takes it from there.
//  * column j: H(0:j, j) = (c - H s) / rho with c = (t, c_j), H(j+1, j) = hh.  A zero hh means
//    an invariant Krylov space: column j is final and closes the cycle.
//  * at the first step of a deflated cycle, c = beta (s, rho) is the least-squares right-hand side.
// Every value of the cycle state is loaded in one round (columns_load: the update issues it right
// behind the loads of the step's partials, which it needs first), the columns 0 .. j-2 that H s
// needs included (lane = row, wave w = the columns l = w mod 4, kColFirst of them per lane; more in
// batches).  No load stands under a condition of its own lane, which would become a branch with a
// full wait: the indices are clamped, the values selected.
struct StepIn {
    const double* sums;     // s_i = sums[2i] (before the reorthogonalisation switch), t_i = sums[2i+1]
    double rho, cj, hh;
    int reorth;
};

constexpr int kColFirst = 12;                           // H loads per lane in the first round
struct ColLoads {
    double beta, hprev;
    double hp;              // H(tid, j-1)
    double hv[kColFirst];   // H(lane, wave + 4 q)
};

__device__ __forceinline__ ColLoads columns_load(int j, const GmresState* gs, bool last) {
    constexpr int ld = kMaxRestart + 1, kWaves = kBlock / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int jm = max(j - 1, 0);
    ColLoads c;
    c.beta = gs->beta;
    c.hprev = gs->H[(size_t)jm * ld + j];
    c.hp = gs->H[(size_t)jm * ld + min(tid, ld - 1)];
    if (!last && j > 1)
#pragma unroll
        for (int q = 0; q < kColFirst; ++q) c.hv[q] = gs->H[(size_t)min(wave + kWaves * q, j - 2) * ld + lane];
    return c;
}

__device__ void columns_close(int j, int dk, GmresState* gs, const StepIn* in, const ColLoads& c) {
    constexpr int ld = kMaxRestart + 1;
    constexpr int kWaves = kBlock / 64;
    constexpr int kBatch = 64;                           // further H loads per batch
    static_assert(kMaxRestart <= 128 && kBlock >= 64 + kMaxRestart, "two row passes; rows on waves 1..");
    __shared__ double Hc[kMaxRestart + 2];              // column j-1, final
    __shared__ double sv[kMaxRestart];                  // s
    __shared__ double hpart[kWaves][kMaxRestart];       // H s, per column class
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool dr_first = dk > 0 && j == dk;
    auto rowmax = [&](int l) { return l < dk ? dk : l + 1; };   // last nonzero row of column l
    const int r = tid - 64;                             // row of column j (waves 1 ..)
    const bool last = in == nullptr;                    // the tail: column j-1 only
    const bool hs_on = !last && j > 1;                  // columns 0 .. j-2 take part in H s
    const int reorth = in ? in->reorth : gs->reorth;
    const double rho = in ? in->rho : gs->rho_m, hh = in ? in->hh : 0.0, cj = in ? in->cj : 0.0;
    double s_t = 0.0, t_r = 0.0;
    if (tid < j) s_t = in ? in->sums[2 * tid] : gs->scoef[tid];
    if (!last && r >= 0 && r < j) t_r = in->sums[2 * r + 1];
    if (tid < j) sv[tid] = reorth ? s_t : 0.0;
    __syncthreads();
    if (j > 0 && tid <= j) {
        if (dr_first) {
            // column dk-1 is the kept block's last column: final as the host set it
            Hc[tid] = tid < j ? c.hp : c.hprev;
            gs->dr_c[tid] = c.beta * (tid < dk ? sv[tid] : rho);
        } else {
            const double h = tid < j ? c.hp + c.hprev * sv[tid] : c.hprev * rho;
            Hc[tid] = h;
            gs->H[(size_t)(j - 1) * ld + tid] = h;
        }
    }
    if (last) return;
    if (hs_on) {
        double acc[2] = {0.0, 0.0};
#pragma unroll
        for (int q = 0; q < kColFirst; ++q) {
            const int l = wave + kWaves * q;
            if (l <= j - 2) acc[0] += (lane <= rowmax(l) ? c.hv[q] : 0.0) * sv[l];
        }
        for (int p = 0; p < 2; ++p) {
            const int i = lane + 64 * p;
            if (i > j) break;
            const int lbeg = wave + (p == 0 ? kWaves * kColFirst : kWaves * (63 / kWaves));
            for (int l0 = lbeg; l0 <= j - 2; l0 += kWaves * kBatch) {
                double hb[kBatch];
#pragma unroll
                for (int q = 0; q < kBatch; ++q) {
                    const int l = l0 + kWaves * q;
                    hb[q] = (l <= j - 2 && i <= rowmax(l)) ? gs->H[(size_t)l * ld + i] : 0.0;
                }
#pragma unroll
                for (int q = 0; q < kBatch; ++q) {
                    const int l = l0 + kWaves * q;
                    if (l <= j - 2) acc[p] += hb[q] * sv[l];
                }
            }
        }
        if (lane <= j) hpart[wave][lane] = acc[0];
        if (lane + 64 <= j) hpart[wave][lane + 64] = acc[1];
    }
    __syncthreads();
    if (rho > 0.0 && r >= 0 && r <= j) {
        double hs = 0.0;
        if (j > 0 && reorth) {
            if (hs_on)
                for (int w = 0; w < kWaves; ++w) hs += hpart[w][r];
            hs += Hc[r] * sv[j - 1];
        }
        const double h = ((r < j ? t_r : cj) - hs) / rho;
        gs->H[(size_t)j * ld + r] = h;
        if (r == j) gs->H[(size_t)j * ld + j + 1] = hh;
    }
}

// The tail of a cycle (one workgroup of kRedThreads): the dot slots of the last vector u_m are
// summed (eight lanes per slot, eight chunks each, loaded in one predicated round), and one wave
// forms rho (the norm of u_m after its second pass), S(q_m) and s, which columns_close needs
// to make column m-1 final.  eps_dot: relative accuracy of the dot products (precision of the
// stored vectors); a squared norm that cancels below eps_dot times its input is a numerical
// breakdown.  A vanished or non-finite rho is stored as 0, which makes columns_rotate close
// the cycle at column m-1.  (Inside a cycle the update launch forms the same sums itself,
// step_scalars below.)  Workgroup 1 makes the rotations that the last step left due; it reads
// nothing that workgroup 0 writes.
constexpr int kRedThreads = 1024;
constexpr int kSlotLanes = 8;                               // lanes per dot slot
constexpr int kSlotChunks = 64 / kSlotLanes;                // chunks per lane
constexpr int kSlotGroups = kRedThreads / kSlotLanes;       // slots per round
constexpr int kSlotRounds = (2 * (kMaxRestart + 2) + kSlotGroups - 1) / kSlotGroups;
static_assert(kDotChunks <= 64, "a slot has at most 64 chunks");

__global__ __launch_bounds__(kRedThreads) void reduce_kernel(int j, int nchunks, const double* __restrict__ part,
                                                             GmresState* gs, double eps_dot, int dk, int report) {
    if (blockIdx.x == 1) {
        columns_rotate(j - 1, dk, gs, report);
        return;
    }
    __shared__ double sums[2 * (kMaxRestart + 2)];
    __shared__ double svl[kMaxRestart + 1];
    __shared__ double su_l;
    __shared__ int flags[2];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ns = 2 * (j + 2);
    const int grp = tid / kSlotLanes, sub = tid % kSlotLanes;
    double pv[kSlotRounds][kSlotChunks];
#pragma unroll
    for (int r = 0; r < kSlotRounds; ++r) {
        const int slot = grp + kSlotGroups * r;
#pragma unroll
        for (int c = 0; c < kSlotChunks; ++c) {
            const int ch = sub * kSlotChunks + c;
            pv[r][c] = (slot < ns && ch < nchunks) ? part[(size_t)slot * nchunks + ch] : 0.0;
        }
    }
    if (tid < j) svl[tid] = gs->svs[tid];
    if (tid == 0) {
        flags[0] = ld_done(gs);
        flags[1] = gs->reorth;
        su_l = gs->su;
    }
#pragma unroll
    for (int r = 0; r < kSlotRounds; ++r) {
        double a = 0.0;
#pragma unroll
        for (int c = 0; c < kSlotChunks; ++c) a += pv[r][c];
        a = group8_sum(a);
        const int slot = grp + kSlotGroups * r;
        if (sub == 0 && slot < ns) sums[slot] = a;
    }
    __syncthreads();
    if (flags[0]) return;
    const int reorth = flags[1];
    // sums: s_i = sums[2i] (i < j), then u.u at 2j (the t slots are not used here)
    for (int i = tid; i < j; i += kRedThreads) gs->scoef[i] = reorth ? sums[2 * i] : 0.0;
    if (wave != 0) return;
    // |s|^2 and s.S(q) over i < j
    double a[2] = {0.0, 0.0};
    for (int i = lane; i < j; i += 64) {
        const double si = reorth ? sums[2 * i] : 0.0;
        a[0] += si * si;
        a[1] += si * svl[i];
    }
    a[0] = wave_sum(a[0]);
    a[1] = wave_sum(a[1]);
    if (lane != 0) return;
    const double r2 = sums[2 * j] - a[0];
    double rho = j > 0 ? (r2 > eps_dot * sums[2 * j] ? sqrt(r2) : 0.0) : 1.0;
    if (!(rho > 0.0) || !isfinite(rho)) rho = 0.0;
    gs->svs[j] = j == 0 ? su_l : (rho > 0.0 ? (su_l - a[1]) / rho : 0.0);     // S(q_j)
    gs->rho_m = rho;
}

// Sum over the four lanes of an aligned group (every lane gets it; all lanes active).
__device__ __forceinline__ double group4_sum(double v) {
    v += dpp_mov<0xB1>(v);
    return v + dpp_mov<0x4E>(v);
}

// The tail of a cycle: column j-1 from the last vector's second pass, and its rotation.
__global__ __launch_bounds__(kBlock) void columns_kernel(int j, int dk, GmresState* gs) {
    const ColLoads c = columns_load(j, gs, true);
    if (gs->done) return;
    columns_close(j, dk, gs, nullptr, c);
    __syncthreads();
    columns_rotate(j, dk, gs, 1, true);
}

// ------------------------------------------------------------- fused step (3 launches per step)
// The update launch forms the step's sums itself: every workgroup reads the dot partials
// (kFusedChunks per slot, four lanes per slot) and forms rho, c_j, hh exactly as the reduction
// kernel does, in the same order everywhere, so all workgroups agree bitwise.  The basis loads
// of the first batch are issued before, and wait out, that work.  Workgroup 0 also stores the
// free-pressure sums S(q_j), S(u_{j+1}) for later steps and runs columns_close from LDS.
constexpr int kFusedChunks = 16;                                     // dot partials per slot
constexpr int kFusedLanes = 4;                                       // lanes per slot
constexpr int kFusedPer = kFusedChunks / kFusedLanes;                // partials per lane
constexpr int kFusedSlots = kBlock / kFusedLanes;                    // slots per round
constexpr int kFusedRounds = 2;                                      // rounds loaded ahead (62 steps)
static_assert(kFusedChunks % kXcds == 0 && kFusedChunks <= kDotChunks, "fused dot chunks");
// Large meshes: the dots write kWideChunks partials per slot (more workgroups streaming the
// basis when j is small), slot_sum_kernel adds them, and the update reads one sum per slot.
constexpr int kWideChunks = 64;
// Two finished vectors a workgroup there: an Arnoldi step at 64^3 (mixed) 110.0 -> 105.9 us, at 56^3
// (FP64) 142.9 -> 136.8; three 106.1 and 140.0, four 108.8 and 142.3 (fewer workgroups).  At 16 chunks
// (12^3 .. 50^3 nodes) pairs gain nothing, there being too few workgroups as it is.
constexpr int kWideGroup = 2;                                         // finished vectors per dot workgroup
constexpr int kWideMinNodes = 131072;
constexpr int kWideSumOffset = 2 * (kMaxRestart + 2) * kWideChunks;   // sums after the partials
static_assert(kWideChunks <= kDotChunks && kWideChunks % kXcds == 0 && kWideChunks <= 64, "wide dot chunks: one a lane");
static_assert(kWideSumOffset + 2 * (kMaxRestart + 2) <= kRedBlocks * (kMaxRestart + 1), "wide sums exceed scratch");

// sums[y] = the nchunks partials of slot y added in chunk order, a wave per slot, its lanes holding the
// partials (idle once the cycle has stopped).  One round of loads, whole lines; a thread per slot read
// them 512 bytes apart from its neighbours' and took 1.2 us more per step (64^3 mixed 111.3 -> 110.1).
// Letting the last dots workgroup of a slot add them saves the launch and costs more (114.4): every
// workgroup then waits for its partials and an atomic.
__global__ __launch_bounds__(kBlock) void slot_sum_kernel(int j, int nchunks, const double* __restrict__ part,
                                                          double* __restrict__ sums, const GmresState* gs) {
    if (gs->done) return;
    const int lane = threadIdx.x & 63;
    const int y = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
    if (y >= 2 * (j + 2)) return;
    const double v = lane < nchunks ? part[(size_t)y * nchunks + lane] : 0.0;
    double t = 0.0;
#pragma unroll
    for (int c = 0; c < kWideChunks; ++c) t += read_lane(v, c);
    if (lane == 0) sums[y] = t;
}

struct StepLds {
    double sums[2 * (kMaxRestart + 2)];
    double svl[kMaxRestart + 1];
    double su;              // S(u_j)
    int flags[2];           // done, reorth
};

struct StepOut {
    double rho, cj, hh;
    double su_next;         // S(u_{j+1})
    double svj;             // S(q_j)
};

// The loads of step_scalars, which a caller may follow with its own before it waits for them.
struct StepLoads {
    double pv[kFusedRounds][kFusedPer];
    double svl, su;
    int done, reorth;
};
__device__ __forceinline__ StepLoads step_load(int j, int nchunks, const double* __restrict__ part,
                                               const GmresState* gs) {
    const int tid = threadIdx.x;
    const int ns = 2 * (j + 2);
    const int grp = tid / kFusedLanes, sub = tid % kFusedLanes;
    // part[slot][0 .. nchunks) is contiguous (stride nchunks): lane sub of a slot reads its
    // kFusedPer consecutive partials.  Only the rounds that hold slots are issued; inside one,
    // every load is unconditional (slot and chunk clamped to valid ones) and weighted 0 when
    // absent, since a load under a per-lane condition becomes a branch with a full wait.
    const int rounds = (ns + kFusedSlots - 1) / kFusedSlots;
    StepLoads s;
#pragma unroll
    for (int r = 0; r < kFusedRounds; ++r) {
        const int slot = grp + kFusedSlots * r;
        const size_t base = (size_t)min(slot, ns - 1) * nchunks;
#pragma unroll
        for (int c = 0; c < kFusedPer; ++c) s.pv[r][c] = 0.0;
        if (r < rounds) {
#pragma unroll
            for (int c = 0; c < kFusedPer; ++c) s.pv[r][c] = part[base + min(sub * kFusedPer + c, nchunks - 1)];
        }
    }
    s.svl = gs->svs[min(tid, kMaxRestart)];
    s.done = gs->done;
    s.reorth = gs->reorth;
    s.su = gs->su;
    return s;
}

// The step's scalars from its sums (s_i, t_i, ...), the free-pressure sums svl of the final vectors
// and su of u_j.  Every wave forms them itself (the wave sums leave them in every lane), so that no
// second barrier is needed; all lanes and workgroups do the same operations in the same order.
__device__ __forceinline__ StepOut step_scalars_of(int j, double eps_dot, const double* sums, const double* svl,
                                                   double su, int reorth) {
    const int lane = threadIdx.x & 63;
    double a[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    for (int i = lane; i < j; i += 64) {
        const double si = reorth ? sums[2 * i] : 0.0, ti = sums[2 * i + 1], pi = svl[i];
        a[0] += si * si;
        a[1] += si * ti;
        a[2] += si * pi;
        a[3] += ti * ti;
        a[4] += ti * pi;
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) a[q] = wave_sum(a[q]);
    const double r2 = sums[2 * j] - a[0];
    double rho = j > 0 ? (r2 > eps_dot * sums[2 * j] ? sqrt(r2) : 0.0) : 1.0;
    if (!(rho > 0.0) || !isfinite(rho)) rho = 0.0;
    const double svj = j == 0 ? su : (rho > 0.0 ? (su - a[2]) / rho : 0.0);
    double cj = 0.0, hh = 0.0, sun = 0.0;
    if (rho > 0.0) {
        cj = (sums[2 * j + 1] - a[1]) / rho;
        const double cc = a[3] + cj * cj;
        const double pw = sums[2 * j + 3] - a[4] - cj * svj;
        const double h2 = sums[2 * j + 2] - cc;
        hh = h2 > eps_dot * sums[2 * j + 2] ? sqrt(h2) / rho : 0.0;
        if (!isfinite(hh)) hh = 0.0;
        sun = hh > 0.0 ? pw / (rho * hh) : 0.0;
    }
    return StepOut{rho, cj, hh, sun, svj};
}

// Returns false (uniformly) when the cycle is done.  Every thread of the workgroup calls it.
__device__ __forceinline__ bool step_scalars(int j, int nchunks, const double* __restrict__ part, const StepLoads& s,
                                             double eps_dot, StepLds& L, StepOut& o) {
    const int tid = threadIdx.x;
    const int ns = 2 * (j + 2);
    const int grp = tid / kFusedLanes, sub = tid % kFusedLanes;
    if (tid < j) L.svl[tid] = s.svl;
    if (tid == 0) {
        L.flags[0] = s.done;
        L.flags[1] = s.reorth;
        L.su = s.su;
    }
#pragma unroll
    for (int r = 0; r < kFusedRounds; ++r) {
        double a = 0.0;
#pragma unroll
        for (int c = 0; c < kFusedPer; ++c) {
            const int slot = grp + kFusedSlots * r;
            a += (slot < ns && sub * kFusedPer + c < nchunks) ? s.pv[r][c] : 0.0;
        }
        a = group4_sum(a);
        const int slot = grp + kFusedSlots * r;
        if (sub == 0 && slot < ns) L.sums[slot] = a;
    }
    for (int s0 = kFusedSlots * kFusedRounds; s0 < ns; s0 += kFusedSlots) {   // longer restarts
        const int slot = s0 + grp;
        double a = 0.0;
#pragma unroll
        for (int c = 0; c < kFusedPer; ++c) {
            const int ch = sub * kFusedPer + c;
            a += (slot < ns && ch < nchunks) ? part[(size_t)slot * nchunks + ch] : 0.0;
        }
        a = group4_sum(a);
        if (sub == 0 && slot < ns) L.sums[slot] = a;
    }
    __syncthreads();
    if (L.flags[0]) return false;              // the cycle stopped in an earlier launch
    o = step_scalars_of(j, eps_dot, L.sums, L.svl, L.su, L.flags[1]);
    return true;
}

// The vector rows are split in eighths of xrows rows, one per XCD: the rows whose dot products
// the dots launch formed on that XCD, so that their reads here hit its L2.
template <typename T, int R>
__global__ __launch_bounds__(kBlock, sizeof(T) * R > 8 ? 4 : 5) void update_fused_kernel(int n, int xrows, int j, T* __restrict__ V,
                                                              const T* __restrict__ w, int nchunks,
                                                              const double* __restrict__ part, GmresState* gs,
                                                              double eps_dot, int dk) {
    __shared__ StepLds L;
    StepOut o;
    if (blockIdx.x == 0) {
        // the launch lasts as long as this workgroup: its waves go first on their CU
        __builtin_amdgcn_s_setprio(3);
        const StepLoads sl = step_load(j, nchunks, part, gs);
        const ColLoads c = columns_load(j, gs, false);
        if (!step_scalars(j, nchunks, part, sl, eps_dot, L, o)) return;
        if (threadIdx.x == 0) {
            gs->rho = o.rho;
            gs->cj = o.cj;
            gs->hh = o.hh;
            gs->su = o.su_next;     // S(u_{j+1}); the other workgroups read only S(u_j), unused there
            gs->svs[j] = o.svj;
        }
        const StepIn in{L.sums, o.rho, o.cj, o.hh, L.flags[1]};
        columns_close(j, dk, gs, &in, c);
        return;
    }
    // R rows per thread, each row's loads coalesced across the workgroup; workgroup b runs on
    // XCD b mod 8 and takes the (b-1)/8-th block of R * blockDim rows of that XCD's eighth
    const int bb = blockIdx.x - 1;
    const int base = ((bb + 1) % kXcds) * xrows, end = min(n, base + xrows);
    int idx[R], ix[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        idx[r] = base + ((bb / kXcds) * R + r) * (int)blockDim.x + (int)threadIdx.x;
        ix[r] = idx[r] < n ? idx[r] : n - 1;     // every thread takes part in the step's sums
    }
    const size_t N = (size_t)n;
    T* uj = V + (size_t)j * N;
    double aq[R], aw[R];
    T v0[8][R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        aq[r] = double(uj[ix[r]]);
        aw[r] = double(w[ix[r]]);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int r = 0; r < R; ++r) v0[q][r] = V[(size_t)min(q, max(j - 1, 0)) * N + ix[r]];
    if (!step_scalars(j, nchunks, part, step_load(j, nchunks, part, gs), eps_dot, L, o)) return;
    const bool reorth = L.flags[1] != 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        if (q < j) {
            const double sq = reorth ? L.sums[2 * q] : 0.0, tq = L.sums[2 * q + 1];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                aq[r] -= sq * double(v0[q][r]);
                aw[r] -= tq * double(v0[q][r]);
            }
        }
    }
    int i = 8;
    for (; i + 8 <= j; i += 8) {
        double vv[8][R];
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int r = 0; r < R; ++r) vv[q][r] = double(V[(size_t)(i + q) * N + ix[r]]);
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const double sq = reorth ? L.sums[2 * (i + q)] : 0.0, tq = L.sums[2 * (i + q) + 1];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                aq[r] -= sq * vv[q][r];
                aw[r] -= tq * vv[q][r];
            }
        }
    }
    for (; i < j; ++i) {
        const double sq = reorth ? L.sums[2 * i] : 0.0, tq = L.sums[2 * i + 1];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const double v = double(V[(size_t)i * N + ix[r]]);
            aq[r] -= sq * v;
            aw[r] -= tq * v;
        }
    }
    const double rho = o.rho, cj = o.cj, hh = o.hh;
    if (!(rho > 0.0)) return;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (idx[r] >= end) continue;             // beyond the vector or this XCD's eighth
        const double q = aq[r] / rho;
        uj[idx[r]] = T(q);
        if (hh > 0.0) V[(size_t)(j + 1) * N + idx[r]] = T((aw[r] - cj * q) / (rho * hh));
    }
}

// ---------------------------------------------------------------- cycles of small systems
// All Arnoldi steps of a cycle and its tail in one launch of one workgroup, for systems of at most
// kSmallNodes nodes and cycles of at most kSmallSteps columns.  Such a step's three launches are
// start-up, hand-over between XCDs and serial latency, of which the vectors' work is a fraction;
// here the vectors in progress, H and the rotations stay in LDS, the basis in the CU's caches, and a
// step is four barriers.  The last wave keeps H beside the others' work: it forms the step's
// scalars, makes column j-1 final beside the update, rotates it beside the next SpMV and forms
// column j beside the next dots.  The others load the basis vectors they need next before they wait
// at a barrier.  Twelve waves: with sixteen (128 registers) these loads spill and a step takes 0.6 us
// more, without them it takes 0.6 us more too; with all waves taking part in everything, 1.8.
// A step of a 125-node FP64 system takes 9.0 us against 11.9 by launches, and an inexact-Newton solve
// on it 1386 us against 1862.  With the cycle's ends, us per step at restart 50, FP64 and mixed, against
// launches: 27 nodes 6.2 and 6.2, 64 nodes 7.2 and 6.7 (12.5 and 12.6), 125 nodes 9.7 and 8.7 (12.8 and
// 12.7), 150 nodes 11.4 and 10.4 (12.8 and 12.7), 175 nodes 11.8 and 10.5 (13.0 and 12.8).  The line lies
// at two 64-node parts of a dot product; the launches are not yet ahead at 176 nodes, the most whose rows
// these waves hold, and sixteen waves at 210 nodes (14.8 and 13.4 against 12.5 and 12.4) are behind.
// Keeping the first vectors in LDS too gains nothing.  Up to 58 columns H stays in LDS, a row per lane.
// Every sum is formed in the order of the three kernels (a wave takes a slot's 64-node parts in
// turn) and with the same roundings, so that a cycle gives the same bits on either path.
constexpr int kSmallNodes = 128;
constexpr int kSmallBlocks = 4096;          // blocks of the matrix (their columns are kept in LDS)
constexpr int kSmallSteps = 58;             // columns; rows of H one per lane
constexpr int kSmallThreads = 768;          // three waves a SIMD: 168 registers
constexpr int kSmallWaves = kSmallThreads / 64 - 1;      // beside the wave that keeps H
constexpr int kSmallWorkers = 64 * kSmallWaves;
constexpr int kSmallLd = 61;                // odd: a row of H across its columns spreads over the banks
constexpr int kSmallSlots = 4;              // dot slots of a wave at a time
static_assert(kSmallNodes <= kDotThreads, "one dot chunk, one node per lane and part");
static_assert(4 * kSmallNodes <= kSmallWorkers, "one row of the vectors per worker");
static_assert(kSmallSteps + 3 <= kSmallLd && kSmallSteps + 2 <= 64, "rows");

__device__ __forceinline__ void wave_sync() {           // LDS of one wave: order its accesses
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <typename T>
struct SmallLds {
    T u[4 * kSmallNodes], w[4 * kSmallNodes];   // u_j, B u_j
    double H[kSmallSteps + 1][kSmallLd];        // columns of H
    double sums[2 * 64];                        // the step's slots
    double svl[kSmallSteps + 2];                // free-pressure sums of the final vectors
    double cl[64], sl[64], Rl[66];
    double qt[kQtMax], c[kDrMax + 1];           // deflated restarting: Q^T, the right-hand side
    StepOut o;
    int done;
    uint16_t ptr[kSmallNodes + 1];              // row bounds and columns of the blocks
    uint8_t col[kSmallBlocks];
};

// Sums over the wave of eight values at once, as a reduce-scatter: lane l returns that of value
// 4 (l & 1) + (l & 2) + (l >> 2 & 1).  Lanes are added in the order of wave_sum.
__device__ __forceinline__ double wave_sum8(double (&v)[8]) {
    const int lane = threadIdx.x & 63;
    const bool b0 = lane & 1, b1 = lane & 2, b2 = lane & 4;
    double a[4], c[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] = (b0 ? v[4 + i] : v[i]) + dpp_mov<0xB1>(b0 ? v[i] : v[4 + i]);   // lane ^ 1
#pragma unroll
    for (int i = 0; i < 2; ++i) c[i] = (b1 ? a[2 + i] : a[i]) + dpp_mov<0x4E>(b1 ? a[i] : a[2 + i]);   // lane ^ 2
    double t = (b2 ? c[1] : c[0]) + dpp_mov<0x1B>(dpp_mov<0x141>(b2 ? c[0] : c[1]));                    // lane ^ 4
    t += dpp_mov<0x128>(t);                                                                             // lane ^ 8
    t += __shfl_xor(t, 16, 64);
    return t + __shfl_xor(t, 32, 64);
}

// The finished vectors of dot slots y0, y0 + kSmallWaves, ... at part's nodes.
template <typename T>
__device__ __forceinline__ void small_load(int n_nodes, int j, int y0, int part, const T* V,
                                           typename Vec4<T>::type (&x)[kSmallSlots]) {
    using V4 = typename Vec4<T>::type;
    const int node = min(64 * part + ((int)threadIdx.x & 63), n_nodes - 1);
#pragma unroll
    for (int q = 0; q < kSmallSlots; ++q)
        x[q] = reinterpret_cast<const V4*>(V)[(size_t)min(y0 + kSmallWaves * q, max(j - 1, 0)) * n_nodes + node];
}

// The wave's dot slots of the step into L.sums; x: the first part's vectors (small_load).
template <typename T>
__device__ __forceinline__ void small_dots(int n_nodes, int j, const T* V, SmallLds<T>& L,
                                           const uint8_t* __restrict__ dmask,
                                           typename Vec4<T>::type (&x)[kSmallSlots]) {
    using V4 = typename Vec4<T>::type;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const V4* u4 = reinterpret_cast<const V4*>(L.u);
    const V4* w4 = reinterpret_cast<const V4*>(L.w);
    for (int y0 = wave; y0 <= j + 1; y0 += kSmallWaves * kSmallSlots) {
        double t = 0.0;
        for (int part = 0; 64 * part < n_nodes; ++part) {
            const int node = min(64 * part + lane, n_nodes - 1);
            const bool in = 64 * part + lane < n_nodes;
            if (part > 0 || y0 > wave) small_load(n_nodes, j, y0, part, V, x);
            const bool masked = (dmask[node] & 8u) != 0;
            const V4 u = u4[node], b = w4[node];
            double d[2 * kSmallSlots];
#pragma unroll
            for (int q = 0; q < kSmallSlots; ++q) {
                const int y = y0 + kSmallWaves * q;              // uniform over the wave
                double d0 = 0.0, d1 = 0.0;
                if (y <= j) {
                    const V4 v = y < j ? x[q] : u;
                    d0 = double(dot4(v, u));
                    d1 = double(dot4(v, b));
                } else if (y == j + 1) {
                    d0 = double(dot4(b, b));
                    d1 = masked ? 0.0 : double(b.w);
                }
                d[2 * q] = in ? d0 : 0.0;
                d[2 * q + 1] = in ? d1 : 0.0;
            }
            t += wave_sum8(d);
        }
        const int i = 4 * (lane & 1) + (lane & 2) + ((lane >> 2) & 1), y = y0 + kSmallWaves * (i >> 1);
        if (lane < 8 && y <= j + 1) L.sums[2 * y + (i & 1)] = t;
    }
}

// What the books' wave keeps of a step until its column is formed: lane i holds s_i and t_i.
struct SmallStep {
    double s, t, rho, cj, hh;
};

// Column j-1 of H becomes final (first part of columns_close), lane = row; dr_first: the right-hand
// side of a deflated cycle instead.
template <typename T>
__device__ __forceinline__ void small_final(int j, int dk, SmallLds<T>& L, const SmallStep& p, double beta,
                                            GmresState* gs) {
    const int r = threadIdx.x & 63;
    if (j > 0 && r <= j) {
        if (dk > 0 && j == dk) {
            const double cr = beta * (r < dk ? p.s : p.rho);
            L.c[r] = cr;
            gs->dr_c[r] = cr;
        } else {
            const double hp = L.H[j - 1][r], hprev = L.H[j - 1][j];
            const double h = r < j ? hp + hprev * p.s : hprev * p.rho;
            wave_sync();
            L.H[j - 1][r] = h;
        }
    }
    wave_sync();
}

// Column j of H from the step's sums (second part of columns_close), lane = row.
template <typename T>
__device__ __forceinline__ void small_column(int j, int dk, SmallLds<T>& L, const SmallStep& p, int reorth) {
    if (!(p.rho > 0.0)) return;
    const int r = threadIdx.x & 63;
    auto rowmax = [&](int l) { return l < dk ? dk : l + 1; };   // last nonzero row of column l
    const int rr = min(r, kSmallLd - 1);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int l0 = 0; l0 <= j - 2; l0 += 8) {
        double h[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) h[q] = L.H[min(l0 + q, j - 2)][rr];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (l0 + q <= j - 2) acc[q & 3] += (r <= rowmax(l0 + q) ? h[q] : 0.0) * read_lane(p.s, l0 + q);
    }
    const double s_last = j > 0 ? read_lane(p.s, j - 1) : 0.0;
    if (r <= j) {
        double hs = 0.0;
        if (j > 0 && reorth) {
            if (j > 1)
#pragma unroll
                for (int q = 0; q < 4; ++q) hs += acc[q];
            hs += L.H[j - 1][r] * s_last;
        }
        L.H[j][r] = ((r < j ? p.t : p.cj) - hs) / p.rho;
        if (r == j) L.H[j][j + 1] = p.hh;
    }
    wave_sync();
}

// The rotations that step j left due, by one wave (columns_rotate); gcur: the right-hand side's entry
// at the next rotation.  Sets L.done when the cycle stops.
template <typename T>
__device__ void small_rotate(int j, int dk, SmallLds<T>& L, double rho, double hh, double& gcur, GivensCtx gc,
                             bool tail, GmresState* gs) {
    constexpr int ld = kMaxRestart + 1;
    const int lane = threadIdx.x & 63;
    const bool dr_first = dk > 0 && j == dk;
    // Q^T of the kept block on rows 0 .. dk of src: rows 0 .. dk-1 into out, the last one returned
    auto apply_qt = [&](const double* src, double* out) {
        double t = 0.0;
        if (lane <= dk) {
#pragma unroll 4
            for (int l = 0; l <= dk; ++l) t += L.qt[l * (dk + 1) + lane] * src[l];
            if (lane < dk) out[lane] = t;
        }
        wave_sync();
        return read_lane(t, dk);
    };
    auto rotate = [&](int jc) {
        double* col = L.H[jc];
        const double x0 = dk > 0 ? apply_qt(col, L.Rl) : 0.0;
        double gnext;
        const int st = givens_column(jc, col, L.cl, L.sl, gcur, L.Rl, gc, gs, dk, x0, &gnext);
        wave_sync();
        gcur = gnext;
        if (lane <= jc) gs->R[(size_t)jc * ld + lane] = L.Rl[lane];
        wave_sync();
        return st;
    };
    int st = 0;
    if (dr_first) {
        const double x0 = apply_qt(L.c, gs->g);
        st = (fabs(x0) <= gc.tol_abs || !(rho > 0.0) || !isfinite(x0)) ? 1 : 0;
        gcur = x0;
        if (lane == 0) {
            gs->gin[dk] = x0;
            gs->k = dk;
            if (st) set_done(gs);
            if (st || gc.report) report_progress(gc.progress, gc.gen, dk, st);
        }
    } else if (j > 0) {
        st = rotate(j - 1);
        if (!(rho > 0.0)) {
            st = 1;                          // u_j vanished: column j-1 closes the cycle
            if (lane == 0) {
                set_done(gs);
                report_progress(gc.progress, gc.gen, j, 1);
            }
        }
    }
    if (!(tail || st || !(rho > 0.0) || hh > 0.0)) {
        // the Krylov space is invariant: column j (formed by now) is final with a zero subdiagonal
        if (lane == 0) L.H[j][j + 1] = 0.0;
        wave_sync();
        rotate(j);
        st = 1;
        if (lane == 0) {
            set_done(gs);
            report_progress(gc.progress, gc.gen, j + 1, 1);
        }
    }
    if (st && lane == 0) L.done = 1;
}

template <typename T>
__global__ __launch_bounds__(kSmallThreads) void small_cycle_kernel(int n_nodes, int dk, int end,
                                                                    const int32_t* __restrict__ rowptr,
                                                                    const int32_t* __restrict__ colidx,
                                                                    const T* __restrict__ AP, const T* __restrict__ Az,
                                                                    const uint8_t* __restrict__ dmask, T* V,
                                                                    GmresState* gs, double eps_dot) {
    constexpr int ld = kMaxRestart + 1;
    constexpr int kRows = kSmallWorkers / kSpmvLanes;          // rows per pass of the SpMV
    constexpr int Q = kSpmvLanes / 4;
    constexpr int kBatch = 64 / sizeof(T);                    // basis vectors and blocks of a lane in flight
    constexpr int kUnroll = 32 / sizeof(T);
    using V4 = typename Vec4<T>::type;
    extern __shared__ __align__(16) unsigned char small_smem[];
    SmallLds<T>& L = *reinterpret_cast<SmallLds<T>*>(small_smem);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool books = __builtin_amdgcn_readfirstlane(wave) == kSmallWaves;     // the wave that keeps H
    const int n = 4 * n_nodes;
    if (gs->done) return;
    const int reorth = gs->reorth;
    const double beta = gs->beta, kappa = gs->kappa;
    for (int i = tid; i < n; i += kSmallThreads) L.u[i] = V[(size_t)dk * n + i];
    for (int e = tid; e < dk * (dk + 1); e += kSmallThreads)
        L.H[e / (dk + 1)][e % (dk + 1)] = gs->H[(size_t)(e / (dk + 1)) * ld + e % (dk + 1)];
    if (dk > 0)
        for (int e = tid; e < (dk + 1) * (dk + 1); e += kSmallThreads) L.qt[e] = gs->dr_qt[e];
    if (tid < dk) L.svl[tid] = gs->svs[tid];
    for (int i = tid; i <= n_nodes; i += kSmallThreads) L.ptr[i] = (uint16_t)rowptr[i];
    for (int k = tid; k < rowptr[n_nodes]; k += kSmallThreads) L.col[k] = (uint8_t)colidx[k];
    if (tid == 0) L.done = 0;
    __syncthreads();
    // the two kinds of waves run loops of their own (their registers are then not held side by
    // side), which meet at the same barriers: four per step, and the tail's
    if (books) {
        double su = gs->su, gcur = gs->gin[0];
        SmallStep p{0.0, 0.0, 0.0, 0.0, 0.0};
        GivensCtx gc{gs->tol_abs, gs->progress, gs->gen, 0};
        __builtin_amdgcn_s_setprio(3);
        int j = dk;
        for (; j < end; ++j) {
            if (j > dk) small_rotate(j - 1, dk, L, p.rho, p.hh, gcur, gc, false, gs);
            __syncthreads();
            if (L.done) break;
            if (j > dk) small_column(j - 1, dk, L, p, reorth);
            __syncthreads();
            const StepOut o = step_scalars_of(j, eps_dot, L.sums, L.svl, su, reorth);
            p = SmallStep{reorth && lane < j ? L.sums[2 * lane] : 0.0, lane < j ? L.sums[2 * lane + 1] : 0.0, o.rho,
                          o.cj, o.hh};
            if (lane == 0) L.o = o;
            __syncthreads();
            small_final(j, dk, L, p, beta, gs);
            if (lane == 0) {
                L.svl[j] = o.svj;
                gs->svs[j] = o.svj;
            }
            if (!(o.hh > 0.0)) small_column(j, dk, L, p, reorth);     // the rotation closes column j
            su = o.su_next;
            __syncthreads();
        }
        if (j == end) {
            // the second pass of the last vector completes the last column
            small_rotate(end - 1, dk, L, p.rho, p.hh, gcur, gc, false, gs);
            __syncthreads();
            if (!L.done) {
                small_column(end - 1, dk, L, p, reorth);
                __syncthreads();
                const double si = reorth && lane < end ? L.sums[2 * lane] : 0.0;
                double a[2] = {0.0, 0.0};
                if (lane < end) {
                    a[0] += si * si;
                    a[1] += si * L.svl[lane];
                    gs->scoef[lane] = si;
                }
                a[0] = wave_sum(a[0]);
                a[1] = wave_sum(a[1]);
                const double r2 = L.sums[2 * end] - a[0];
                double rho = r2 > eps_dot * L.sums[2 * end] ? sqrt(r2) : 0.0;
                if (!(rho > 0.0) || !isfinite(rho)) rho = 0.0;
                if (lane == 0) {
                    gs->svs[end] = rho > 0.0 ? (su - a[1]) / rho : 0.0;
                    gs->rho_m = rho;
                }
                small_final(end, dk, L, SmallStep{si, 0.0, rho, 0.0, 0.0}, beta, gs);
                gc.report = 1;
                small_rotate(end, dk, L, rho, 1.0, gcur, gc, true, gs);
            }
        }
    } else {
        const int sub = tid % kSpmvLanes, quad = sub >> 2, r = sub & 3;
        const int iv = min(tid, n - 1);                        // the worker's vector row
        double su = gs->su;
        int j = dk;
        for (; j < end; ++j) {
            // w = (A P) u_j + kappa S(u_j) A z
            for (int row0 = 0; row0 < n_nodes; row0 += kRows) {
                const int row = row0 + tid / kSpmvLanes;
                T acc = T(0);
                if (row < n_nodes) {
                    const int k1 = L.ptr[row + 1];
                    const T az = Az[4 * (size_t)row + r];
                    for (int kb = L.ptr[row] + quad; kb < k1; kb += kUnroll * Q) {
                        V4 av[kUnroll];
#pragma unroll
                        for (int u = 0; u < kUnroll; ++u)
                            if (kb + u * Q < k1) av[u] = *reinterpret_cast<const V4*>(AP + (size_t)(kb + u * Q) * 16 + r * 4);
#pragma unroll
                        for (int u = 0; u < kUnroll; ++u) {
                            if (kb + u * Q >= k1) continue;          // the four lanes of a quad agree
                            const T xr = L.u[L.col[kb + u * Q] * 4 + r];
                            const T x0 = quad_bcast<0>(xr), x1 = quad_bcast<1>(xr), x2 = quad_bcast<2>(xr),
                                    x3 = quad_bcast<3>(xr);
                            acc += dot4<T>(av[u].x, av[u].y, av[u].z, av[u].w, x0, x1, x2, x3);
                        }
                    }
                    acc += __shfl_xor(acc, 4, 64);               // the eight lanes of a row agree
                    if (quad == 0) L.w[4 * row + r] = acc + T(kappa * su) * az;
                }
            }
            V4 x[kSmallSlots];                                 // loads that need not wait for the barrier
            small_load(n_nodes, j, wave, 0, V, x);
            __syncthreads();
            if (L.done) break;
            small_dots(n_nodes, j, V, L, dmask, x);
            T v[kBatch];                                       // nor these for the scalars
            if (64 * wave < n) {
#pragma unroll
                for (int q = 0; q < kBatch; ++q) v[q] = V[(size_t)min(q, max(j - 1, 0)) * n + iv];
            }
            __syncthreads();
            __syncthreads();
            // q_j and u_{j+1}
            const StepOut o = L.o;
            if (o.rho > 0.0 && 64 * wave < n) {
                const double s_l = reorth && lane < j ? L.sums[2 * lane] : 0.0;
                const double t_l = lane < j ? L.sums[2 * lane + 1] : 0.0;
                double aq = double(L.u[iv]), aw = double(L.w[iv]);
                for (int l0 = 0; l0 < j; l0 += kBatch) {
#pragma unroll
                    for (int q = 0; q < kBatch; ++q)
                        if (l0 + q < j) {
                            aq -= read_lane(s_l, l0 + q) * double(v[q]);
                            aw -= read_lane(t_l, l0 + q) * double(v[q]);
                        }
                    if (l0 + kBatch < j)
#pragma unroll
                        for (int q = 0; q < kBatch; ++q) v[q] = V[(size_t)min(l0 + kBatch + q, j - 1) * n + iv];
                }
                const double q = aq / o.rho;
                if (tid < n) {
                    V[(size_t)j * n + tid] = T(q);
                    if (o.hh > 0.0) {
                        const T un = T((aw - o.cj * q) / (o.rho * o.hh));
                        V[(size_t)(j + 1) * n + tid] = un;
                        L.u[tid] = un;
                    }
                }
            }
            su = o.su_next;
            __syncthreads();
        }
        if (j == end) {
            __syncthreads();
            if (!L.done) {
                V4 x[kSmallSlots];
                small_load(n_nodes, end, wave, 0, V, x);
                small_dots(n_nodes, end, V, L, dmask, x);
                __syncthreads();
            }
        }
    }
    __syncthreads();
    // H for the host (deflated restarting)
    for (int e = tid; e < end * (end + 1); e += kSmallThreads)
        gs->H[(size_t)(e / (end + 1)) * ld + e % (end + 1)] = L.H[e / (end + 1)][e % (end + 1)];
}

// What the host needs of a full cycle to deflate the next one (dr_prepare), written into its mapped
// staging by the back-substitution's workgroup (every thread of it; y finished): rows 0 .. m of H and
// the cycle state from y on, then the cycle number with release order, which the host polls for.
// The host works on it while the device finishes the cycle and forms the true residual.
__device__ void dr_export(int m, const GmresState* gs, GmresState* out, uint64_t* tag) {
    constexpr int ld = kMaxRestart + 1;
    for (int e = threadIdx.x; e < m * (m + 1); e += blockDim.x) {
        const size_t at = (size_t)(e / (m + 1)) * ld + e % (m + 1);
        out->H[at] = gs->H[at];
    }
    constexpr size_t first = offsetof(GmresState, y), words = (sizeof(GmresState) - first) / sizeof(uint64_t);
    static_assert(first % sizeof(uint64_t) == 0 && sizeof(GmresState) % sizeof(uint64_t) == 0, "whole words");
    const uint64_t* src = reinterpret_cast<const uint64_t*>(reinterpret_cast<const char*>(gs) + first);
    uint64_t* dst = reinterpret_cast<uint64_t*>(reinterpret_cast<char*>(out) + first);
    for (size_t e = threadIdx.x; e < words; e += blockDim.x) dst[e] = src[e];
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(tag, (uint64_t)gs->gen, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// y = R^{-1} g for the k x k triangle of the rotated Hessenberg matrix (one workgroup): the
// triangle and the reciprocals of its diagonal are staged in LDS (column batches, loads in
// flight together), then one wave eliminates
// column by column, lane l holding entries l and l + 64 of the right-hand side; the pivot
// entry is broadcast with readlane, so the sequential chain is a multiply and an FMA per column.
__global__ __launch_bounds__(kBlock) void backsub_kernel(GmresState* gs, int m, GmresState* out,
                                                         uint64_t* tag) {
    const int k = gs->k;
    if (k == 0 && !out) return;
    constexpr int ld = kMaxRestart + 1;
    __shared__ double Rl[kMaxRestart * kMaxRestart];
    __shared__ double rinv[kMaxRestart];
    // staging: lane = row (two halves), wave w = the columns col = w mod 4, eight columns of a
    // lane loaded before any is stored (clamped column, so no branch around a load)
    constexpr int kWaves = kBlock / 64, kCols = 8;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int c0 = wave; c0 < k; c0 += kWaves * kCols) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int row = lane + 64 * half;
            if (row >= k) break;
            double rv[kCols];
#pragma unroll
            for (int q = 0; q < kCols; ++q) rv[q] = gs->R[(size_t)min(c0 + kWaves * q, k - 1) * ld + row];
#pragma unroll
            for (int q = 0; q < kCols; ++q) {
                const int col = c0 + kWaves * q;
                if (col < k && row <= col) {
                    Rl[col * k + row] = rv[q];
                    if (row == col) rinv[col] = 1.0 / rv[q];
                }
            }
        }
    }
    double g0 = 0.0, g1 = 0.0;
    if (threadIdx.x < 64) {
        g0 = threadIdx.x < k ? gs->g[threadIdx.x] : 0.0;
        g1 = threadIdx.x + 64 < k ? gs->g[threadIdx.x + 64] : 0.0;
    }
    __syncthreads();
    const int l = threadIdx.x;
    if (l < 64)
        for (int col = k - 1; col >= 0; --col) {
            const double yc = read_lane(col < 64 ? g0 : g1, col & 63) * rinv[col];
            if (l == 0) gs->y[col] = yc;
            if (l < col) g0 -= Rl[col * k + l] * yc;
            if (l + 64 < col) g1 -= Rl[col * k + l + 64] * yc;
        }
    if (!out) return;
    __syncthreads();
    dr_export(m, gs, out, tag);
}

// The same for restart lengths up to 64, by one wave: lane l holds row l of the triangle, so that
// an elimination step is two lane reads, a multiply and an FMA with no memory access in the chain
// (the staged form reads its operands from LDS in every step: 10 us for 50 columns, 4 us so).
constexpr int kBacksubLanes = 64;
__global__ __launch_bounds__(kBlock) void backsub_wave_kernel(GmresState* gs, int m, GmresState* out, uint64_t* tag) {
    constexpr int ld = kMaxRestart + 1;
    const int l = threadIdx.x;
    if (l < kBacksubLanes) {
        double row[kBacksubLanes];
#pragma unroll
        for (int col = 0; col < kBacksubLanes; ++col) row[col] = gs->R[(size_t)col * ld + l];
        const double diag = gs->R[(size_t)l * ld + l], gl = gs->g[l];
        const int k = gs->k;
        double g = l < k ? gl : 0.0, y = 0.0;
        const double rinv = 1.0 / diag;
#pragma unroll
        for (int col = kBacksubLanes - 1; col >= 0; --col) {
            if (col < k) {
                const double yc = read_lane(g, col) * read_lane(rinv, col);
                if (l == col) y = yc;
                if (l < col) g -= row[col] * yc;
            }
        }
        if (l < k) gs->y[l] = y;
    }
    if (!out) return;
    __syncthreads();
    dr_export(m, gs, out, tag);
}

// t = sum_{i<k} y_i V_i
template <typename T>
__global__ __launch_bounds__(kBlock) void combine_kernel(int n, const T* __restrict__ V, const GmresState* gs,
                                                         T* __restrict__ t) {
    const int k = gs->k;
    if (k == 0) return;
    __shared__ double ys[kMaxRestart];
    for (int i = threadIdx.x; i < k; i += blockDim.x) ys[i] = gs->y[i];
    __syncthreads();
    const int idx = xcd_slot(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;   // basis slices in this XCD's L2
    if (idx >= n) return;
    const size_t N = (size_t)n;
    double sacc = 0.0;
    int i = 0;
    for (; i + 8 <= k; i += 8) {
        double vv[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) vv[q] = double(V[(size_t)(i + q) * N + idx]);
#pragma unroll
        for (int q = 0; q < 8; ++q) sacc += ys[i + q] * vv[q];
    }
    for (; i < k; ++i) sacc += ys[i] * double(V[(size_t)i * N + idx]);
    t[idx] = T(sacc);
}

// Partial sums of the free pressure entries of t (for the coarse term of P t; added by
// precond_accumulate_kernel)
template <typename T>
__global__ __launch_bounds__(kBlock) void free_pressure_sum_kernel(int n_nodes, const T* __restrict__ t,
                                                                   const uint8_t* __restrict__ dmask,
                                                                   RedScratch* red, const GmresState* gs) {
    if (gs->k == 0) return;
    __shared__ double lds[kBlock / 64];
    double v[1] = {0.0};
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n_nodes; i += gridDim.x * blockDim.x)
        if (!(dmask[i] & 8u)) v[0] += double(t[4 * (size_t)i + 3]);
    block_sum<1>(v, lds);
    if (threadIdx.x == 0) red->partial[blockIdx.x] = v[0];
}

// x += xscale P t = xscale (Minv t + z kappa (1_p^T t))  (x in TX: double for the FP64 solution,
// float for an inner correction; xscale is the norm of the residual an FP32 cycle was given
// scaled to one).  z is the indicator of the free pressure dofs 1_p, or the explicit vector zvec.
// Every workgroup adds the nparts partials of 1_p^T t itself, in the same order.
template <typename TM, typename T, typename TX>
__global__ __launch_bounds__(kBlock) void precond_accumulate_kernel(int n_nodes, const TM* __restrict__ Minv,
                                                                    const T* __restrict__ t,
                                                                    const uint8_t* __restrict__ dmask,
                                                                    const double* __restrict__ zvec,
                                                                    const GmresState* gs, int nparts,
                                                                    const RedScratch* red, double xscale,
                                                                    TX* __restrict__ x) {
    if (gs->k == 0) return;
    __shared__ double st;
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    const int node = min(tid >> 2, n_nodes - 1), r = tid & 3;
    using M4 = typename Vec4<TM>::type;
    using V4 = typename Vec4<T>::type;
    const M4 m = *reinterpret_cast<const M4*>(Minv + (size_t)node * 16 + r * 4);
    const V4 v = *reinterpret_cast<const V4*>(t + 4 * (size_t)node);
    const TX x0 = x[4 * (size_t)node + r];
    const uint32_t dm = dmask[node];
    reduce_partials(red->partial, kRedBlocks, 1, nparts, &st);
    __syncthreads();
    if ((tid >> 2) >= n_nodes) return;
    double s = double(m.x) * double(v.x) + double(m.y) * double(v.y) + double(m.z) * double(v.z) +
               double(m.w) * double(v.w);
    if (zvec)
        s += gs->kappa * st * zvec[4 * (size_t)node + r];
    else if (r == 3 && !(dm & 8u))
        s += gs->kappa * st;
    x[4 * (size_t)node + r] = TX(double(x0) + xscale * s);
}

// FP64 norm of a vector of any precision into out (device) via partials.
template <typename T>
__global__ __launch_bounds__(kBlock) void norm_kernel(int n, const T* __restrict__ r, RedScratch* red,
                                                      double* out, uint64_t* tag_out, uint64_t tag) {
    __shared__ double lds[kBlock / 64];
    double v[1] = {0.0};
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const double x = double(r[i]);
        v[0] += x * x;
    }
    block_sum<1>(v, lds);
    if (threadIdx.x == 0) red->partial[blockIdx.x] = v[0];
    if (!arrive_last(&red->counter)) return;
    __threadfence();
    __shared__ double tot;
    reduce_partials(red->partial, kRedBlocks, 1, gridDim.x, &tot);
    __syncthreads();
    if (threadIdx.x == 0) {
        // out and tag_out are pinned host memory (the context's mapped page): the value, then its
        // tag with release order, which the host polls for
        __hip_atomic_store(out, sqrt(tot), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        red->counter = 0u;
        __hip_atomic_store(tag_out, tag, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

__global__ void zero_count_kernel(int32_t* p) {
    if (threadIdx.x == 0) *p = 0;
}

template <typename TS, typename TD>
__global__ void convert_kernel(int n, const TS* __restrict__ s, TD* __restrict__ d, double scale) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) d[i] = TD(double(s[i]) * scale);
}

template <typename T>
__global__ void axpy64_kernel(int n, double alpha, const T* __restrict__ d, double* __restrict__ x) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] += alpha * double(d[i]);
}

// Workgroups of a grid-wide reduction: each one pays a device-scope fence and an atomic on the
// arrival counter, which costs more than streaming a few more elements per thread.
#ifndef VMS_RED_GRID_MAX
#define VMS_RED_GRID_MAX 128
#endif
static_assert(VMS_RED_GRID_MAX <= kRedBlocks, "reduction grid exceeds the partials");
inline int red_grid(int64_t n) { return std::max(1, std::min(VMS_RED_GRID_MAX, grid_for(n))); }

// Launches the norm of r (n entries) into mapped scalar k with a fresh tag.
template <typename T>
void launch_norm(vms_ctx* c, int n, const T* r, int k, hipStream_t s) {
    norm_kernel<T><<<red_grid(n), kBlock, 0, s>>>(n, r, c->red, c->scal_dev + k, c->progress_dev + 1 + k,
                                                  ++c->scal_seq);
}

// Waits for a word of the mapped page: spins on it (the launches after the one that writes it are
// already ordered), with a stream query every 256 spins so that a failed or drained stream ends the
// wait.  read_scalar: mapped scalar k of the last launch_norm.
int wait_word(vms_ctx* c, int word, uint64_t want, const char* what, hipStream_t s) {
    const uint64_t* tag = c->progress_host + word;
    for (unsigned spin = 0;; ++spin) {
        if (__atomic_load_n(tag, __ATOMIC_ACQUIRE) == want) return VMS_OK;
        if ((spin & 255u) == 255u) {
            const hipError_t q = hipStreamQuery(s);
            if (q == hipSuccess) {
                if (__atomic_load_n(tag, __ATOMIC_ACQUIRE) == want) return VMS_OK;
                return set_error(c, VMS_EHIP, std::string(what) + ": the stream finished without the value");
            }
            if (q != hipErrorNotReady) return check_hip(c, q, what);
        }
    }
}

int read_scalar(vms_ctx* c, int k, double* h, hipStream_t s) {
    if (int rc = wait_word(c, 1 + k, c->scal_seq, "read scalar", s)) return rc;
    *h = *reinterpret_cast<volatile const double*>(c->scal_host + k);
    return VMS_OK;
}

#ifndef VMS_LEAD_STEPS
#define VMS_LEAD_STEPS 3
#endif
constexpr int kLeadSteps = VMS_LEAD_STEPS;   // Arnoldi steps the host may issue ahead of the device

// The device's progress word for cycle gen: completed columns (-1 before the cycle has
// reported), *done = 1 once the cycle stopped (converged or broke down).
int read_progress(const vms_ctx* c, uint32_t gen, int* done) {
    const uint64_t word = __atomic_load_n(c->progress_host, __ATOMIC_ACQUIRE);
    if ((uint32_t)(word >> 32) != gen) {
        *done = 0;
        return -1;
    }
    *done = (int)(word & 1u);
    return (int)((word >> 1) & 0x7fffffffu);
}

// Waits, without synchronising the stream, until cycle gen has completed `need` columns or
// stopped.  Returns 1 if it stopped, 0 if the columns are there (or the stream ran dry), a
// negative status on a HIP error.
int wait_progress(vms_ctx* c, uint32_t gen, int need, hipStream_t s) {
    for (unsigned spin = 0;; ++spin) {
        int done = 0;
        const int k = read_progress(c, gen, &done);
        if (done) return 1;
        if (k >= need) return 0;
        if ((spin & 255u) == 255u) {
            const hipError_t q = hipStreamQuery(s);
            if (q == hipSuccess) {           // every launch has finished: the word is final
                read_progress(c, gen, &done);
                return done;
            }
            if (q != hipErrorNotReady) {
                (void)check_hip(c, q, "gmres: stream query");
                return -1;
            }
        }
    }
}

// Launches one GMRES(m) cycle on A d = r0 with right preconditioner Minv, adding the Krylov
// correction xscale Minv (V y) (+ coarse term) to x (double or float).  r0 is the cycle's initial
// residual (precision T), formed here as r64 scaled when r64 is given; x_save receives x as it is
// before the cycle; with to_deflate, a full cycle hands the host what dr_prepare needs.  The host follows the device's progress through the mapped word,
// keeps at most kLeadSteps steps queued ahead of it and stops issuing steps once the cycle has
// converged; nothing here synchronises the stream.  finish_cycle gives the number of steps
// once the caller has synchronised.
// Cycle graphs are on unless VMS_CYCLE_GRAPHS=0 in the environment (read at every cycle).
inline bool cycle_graphs_enabled() {
    const char* e = std::getenv("VMS_CYCLE_GRAPHS");
    return !(e && e[0] == '0');
}

// The Krylov basis and work vectors of precision T: the context's own (its precision), or the
// FP64 set a mixed context allocates for solves with an FP64 basis.
template <typename T>
T* basis_vectors(vms_ctx* c, int which) {
    const bool own = sizeof(T) == elt_size(c);
    void* p[3] = {own ? c->V : c->V64, own ? c->w : c->w64, own ? c->z : c->z64};
    return static_cast<T*>(p[which]);
}

// One restart cycle: T the precision of the basis and of its arithmetic, TM that of the stored
// matrix, its A P blocks, A z and the preconditioner blocks, TX that of the iterate x.
// With TM != T the steps apply P and A (Amat) in two passes instead of the stored A P blocks.
template <typename T, typename TX, typename TM = T>
int run_cycle(vms_ctx* c, T* r0, const TM* Minv, TX* x, double tol_abs, int m, int budget, int cgs2,
              hipStream_t s, double xscale = 1.0, int j0 = 0, const TM* Amat = nullptr, const double* r64 = nullptr,
              double r64_scale = 1.0, double* x_save = nullptr, bool to_deflate = false) {
    constexpr bool split = !std::is_same<TM, T>::value;
    if (split && !Amat) return set_error(c, VMS_EINVAL, "gmres: no matrix for the split operator");
    const int n = 4 * c->n_nodes;
    const TM* AP = (const TM*)c->AP;
    const TM* Az = (const TM*)c->Az;
    T* V = basis_vectors<T>(c, 0);
    T* w = basis_vectors<T>(c, 1);
    T* z = basis_vectors<T>(c, 2);
    // recorded graphs are told apart by restart length, kept vectors and basis precision; every address in
    // them is the context's (the caller's matrix is found through the cycle state)
    const int pbit = sizeof(T) == 8 ? 1 : 0;
    const uint32_t gen = ++c->cycle_gen;
    c->cycle_timed.clear();
    const double* x_old = nullptr;
    if constexpr (std::is_same<TX, double>::value) x_old = x;
    cycle_norm_kernel<T><<<red_grid(n), kBlock, 0, s>>>(n, r64, r64_scale, r0, x_old, x_save, c->dmask, c->red);
    // a deflated cycle puts the residual after the kept vectors and runs steps j0 .. m-1
    cycle_v0_kernel<T><<<grid_for(n), kBlock, 0, s>>>(n, r0, V + (size_t)j0 * n, red_grid(n), c->red, c->gs, tol_abs,
                                                      cgs2, gen, Amat);
    const int steps = std::min(m - j0, budget);
    const double vb = (double)n * sizeof(T);      // bytes of one Krylov vector
    // algorithmic bytes of the Arnoldi SpMV: blocks and column indices, row pointers, the input
    // and output vectors once (the coarse-pressure vector A z it also reads is not credited)
    const double spmv_bytes = (double)c->nb * (16.0 * sizeof(TM) + 4.0) + 4.0 * (c->n_nodes + 1) + 2.0 * vb;
    const bool wide = c->n_nodes >= kWideMinNodes;
    const int nch = wide ? kWideChunks : std::max(1, std::min(kFusedChunks, (c->n_nodes + kDotThreads - 1) / kDotThreads));
    // rows of the vectors whose dots the workgroups on one XCD form (the dots take their chunks
    // in xcd_slot order when there are a multiple of 8 of them), which the update reads there too
    const int xrows = nch % kXcds == 0 ? 4 * ((c->n_nodes + nch - 1) / nch) * (nch / kXcds)
                                       : (n + kXcds - 1) / kXcds;
    double* part = c->red->partial;
    const double eps_dot = sizeof(T) == 8 ? 1e-14 : 1e-6;
    // timed launches per step, so that steps issued after convergence (their kernels return
    // at once) can be dropped from the phase timers
    auto keep = [&](int jj, const PhaseScope& ph) {
        if (ph.slot >= 0) {
            c->cycle_timed.push_back(jj);
            c->cycle_timed.push_back(ph.slot);
            c->cycle_timed.push_back(ph.gen);
        }
    };
    auto timed = [&](int phase, double bytes, int j, hipStream_t st, auto&& launch) {
        PhaseScope ph(c, phase, bytes, st);
        launch();
        keep(j, ph);
    };
    auto launch_dots = [&](int j, hipStream_t st) {
        if (wide)
            dots_kernel<T, kWideGroup><<<dim3(nch, (j + kWideGroup - 1) / kWideGroup + 2), kDotThreads, 0, st>>>(
                c->n_nodes, j, V, w, c->dmask, part, c->gs);
        else
            dots_kernel<T, 1><<<dim3(nch, j + 2), kDotThreads, 0, st>>>(c->n_nodes, j, V, w, c->dmask, part, c->gs);
    };
    // the Arnoldi steps and the tail on stream st; with lead, the host keeps at most kLeadSteps
    // steps queued ahead of the device and stops issuing once the cycle has converged
    auto issue = [&](int steps_, bool lead, hipStream_t st) -> int {
        steps_ += j0;                                     // the last column index
        for (int j = j0; j < steps_; ++j) {
            if (lead && j - j0 >= kLeadSteps) {
                const int sw = wait_progress(c, gen, j - kLeadSteps, st);
                if (sw < 0) return VMS_EHIP;
                if (sw == 1) break;
            }
            // w = A P u_j = (A P) u_j + kappa S(u_j) A z, or A (P u_j) with z = P u_j
            if constexpr (split) {
                timed(VMS_PH_PCAPPLY, (double)c->n_nodes * (16.0 * sizeof(TM) + 8.0 * sizeof(T)), j, st, [&] {
                    precond_apply_kernel<TM, T><<<grid_for(n), kBlock, 0, st>>>(c->n_nodes, Minv, V + (size_t)j * n,
                                                                              c->dmask, c->zfull, c->gs, z);
                });
                timed(VMS_PH_SPMV, spmv_bytes, j, st, [&] {
                    spmv_kernel<TM, T, T, T, 0, double, true><<<1 + spmv_grid(c->n_nodes), kBlock, 0, st>>>(
                        c->n_nodes, c->rowptr, c->colidx, (const TM*)nullptr, z, (const double*)nullptr, w, c->gs, j - 1, j0,
                        lead ? 1 : 0);
                });
            } else {
                timed(VMS_PH_SPMV, spmv_bytes, j, st, [&] {
                    spmv_kernel<TM, T, T, T, 2, TM, true><<<1 + spmv_grid(c->n_nodes), kBlock, 0, st>>>(
                        c->n_nodes, c->rowptr, c->colidx, AP, V + (size_t)j * n, Az, w, c->gs, j - 1, j0,
                        lead ? 1 : 0);
                });
            }
            timed(VMS_PH_DOTS, (j + 2) * vb, j, st, [&] {
                launch_dots(j, st);
            });
            timed(VMS_PH_UPDATE, (j + 4) * vb, j, st, [&] {
                if (wide) slot_sum_kernel<<<(2 * (j + 2) + kBlock / 64 - 1) / (kBlock / 64), kBlock, 0, st>>>(j, nch, part, part + kWideSumOffset, c->gs);
                // two vector rows per thread halve the workgroups that each form the step's
                // scalars, except for FP64 vectors on small meshes, where one row per thread
                // keeps more waves streaming the basis
                const double* sums = wide ? part + kWideSumOffset : part;
                const int nsum = wide ? 1 : nch;
                if (sizeof(T) == 4 || wide)
                    update_fused_kernel<T, 2><<<1 + kXcds * grid_for(xrows, 2 * kBlock), kBlock, 0, st>>>(
                        n, xrows, j, V, w, nsum, sums, c->gs, eps_dot, j0);
                else
                    update_fused_kernel<T, 1><<<1 + kXcds * grid_for(xrows, kBlock), kBlock, 0, st>>>(
                        n, xrows, j, V, w, nsum, sums, c->gs, eps_dot, j0);
            });
        }
        // the second pass of the last vector completes the last column
        launch_dots(steps_, st);
        reduce_kernel<<<2, kRedThreads, 0, st>>>(steps_, nch, part, c->gs, eps_dot, j0, lead ? 1 : 0);
        columns_kernel<<<1, kBlock, 0, st>>>(steps_, j0, c->gs);
        return VMS_OK;
    };
    // With the phase timers on, every prof_every-th cycle is launched directly and every launch
    // of a timed phase in it is timed (events cannot time launches inside a graph).
    const bool graphs = steps == m - j0 && cycle_graphs_enabled();
    const bool sampled = c->prof_mask != 0 && c->prof_cycles++ % c->prof_every == 0;
    bool small = false;
    if constexpr (!split) {
        // with the timers on, only in place of a graph: partial cycles are timed launch by launch
        small = c->n_nodes <= kSmallNodes && c->nb <= kSmallBlocks && j0 + steps <= kSmallSteps && !sampled &&
                (c->prof_mask == 0 || graphs);
        if (small)
            small_cycle_kernel<T><<<1, kSmallThreads, sizeof(SmallLds<T>), s>>>(
                c->n_nodes, j0, j0 + steps, c->rowptr, c->colidx, AP, Az, c->dmask, V, c->gs, eps_dot);
    }
    if (small) {
        // done: one launch
    } else if (graphs && !sampled && j0 > 0) {
        // a full deflated cycle: one recorded graph per (m, j0), kept in a small cache
        const int key = (m * 256 + j0) * 2 + pbit;
        int slot = -1;
        for (int q = 0; q < 4; ++q)
            if (c->dr_exec[q] && c->dr_exec_key[q] == key) slot = q;
        if (slot < 0) {
            slot = 0;
            for (int q = 0; q < 4; ++q)
                if (!c->dr_exec[q]) {
                    slot = q;
                    break;
                }
            int rc = VMS_OK;
            if (!c->cap_stream &&
                (rc = check_hip(c, hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking), "capture stream")))
                return rc;
            if (c->dr_exec[slot]) {
                (void)hipGraphExecDestroy(c->dr_exec[slot]);
                c->dr_exec[slot] = nullptr;
            }
            if ((rc = check_hip(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeThreadLocal),
                                "begin capture")))
                return rc;
            const uint32_t mask = c->prof_mask;
            c->prof_mask = 0;
            rc = issue(m - j0, false, c->cap_stream);
            c->prof_mask = mask;
            hipGraph_t g = nullptr;
            const hipError_t e = hipStreamEndCapture(c->cap_stream, &g);
            if (rc) return rc;
            if ((rc = check_hip(c, e, "end capture"))) return rc;
            rc = check_hip(c, hipGraphInstantiate(&c->dr_exec[slot], g, nullptr, nullptr, 0), "graph instantiate");
            (void)hipGraphDestroy(g);
            if (rc) return rc;
            c->dr_exec_key[slot] = key;
        }
        if (int rc = check_hip(c, hipGraphLaunch(c->dr_exec[slot], s), "graph launch")) return rc;
    } else if (graphs && !sampled) {
        // a full cycle: replay the recorded steps (the kernels after convergence return at once)
        if (!c->cycle_exec || c->cycle_exec_m != m * 2 + pbit) {
            int rc = VMS_OK;
            if (!c->cap_stream &&
                (rc = check_hip(c, hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking), "capture stream")))
                return rc;
            if (c->cycle_exec) {
                (void)hipGraphExecDestroy(c->cycle_exec);
                c->cycle_exec = nullptr;
            }
            if ((rc = check_hip(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeThreadLocal),
                                "begin capture")))
                return rc;
            const uint32_t mask = c->prof_mask;      // nothing is timed inside the graph
            c->prof_mask = 0;
            rc = issue(m, false, c->cap_stream);
            c->prof_mask = mask;
            hipGraph_t g = nullptr;
            const hipError_t e = hipStreamEndCapture(c->cap_stream, &g);
            if (rc) return rc;
            if ((rc = check_hip(c, e, "end capture"))) return rc;
            rc = check_hip(c, hipGraphInstantiate(&c->cycle_exec, g, nullptr, nullptr, 0), "graph instantiate");
            (void)hipGraphDestroy(g);
            if (rc) return rc;
            c->cycle_exec_m = m * 2 + pbit;
        }
        if (int rc = check_hip(c, hipGraphLaunch(c->cycle_exec, s), "graph launch")) return rc;
    } else {
        c->prof_force = graphs && sampled;
        const int rc = issue(steps, true, s);
        c->prof_force = false;
        if (rc) return rc;
    }
    // y = R^{-1} g on the device
    GmresState* out = to_deflate && steps == m - j0 ? static_cast<GmresState*>(c->dr_mapped) : nullptr;
    uint64_t* tag = c->progress_dev + kDrTagWord;
    if (m <= kBacksubLanes)
        backsub_wave_kernel<<<1, out ? kBlock : kBacksubLanes, 0, s>>>(c->gs, m, out, tag);
    else
        backsub_kernel<<<1, kBlock, 0, s>>>(c->gs, m, out, tag);
    combine_kernel<T><<<xcd_round(grid_for(n)), kBlock, 0, s>>>(n, V, c->gs, z);
    free_pressure_sum_kernel<T><<<red_grid(c->n_nodes), kBlock, 0, s>>>(c->n_nodes, z, c->dmask, c->red, c->gs);
    precond_accumulate_kernel<TM, T, TX><<<grid_for(n), kBlock, 0, s>>>(
        c->n_nodes, Minv, z, c->dmask, c->zfull, c->gs, red_grid(c->n_nodes), c->red, xscale, x);
    return check_hip(c, hipGetLastError(), "gmres cycle launch");
}

// After the caller has synchronised the stream: Arnoldi steps of the last cycle (*stopped = 1
// when the cycle ended on its own residual estimate or a breakdown, not on the step budget).
// Timed launches of steps issued after convergence are dropped.
int finish_cycle(vms_ctx* c, int* stopped = nullptr) {
    int done = 0;
    const int k = std::max(0, read_progress(c, c->cycle_gen, &done));
    if (stopped) *stopped = done;
    for (size_t i = 0; i + 2 < c->cycle_timed.size(); i += 3)
        if (c->cycle_timed[i] >= k) prof_void(c, (int)c->cycle_timed[i + 1], c->cycle_timed[i + 2]);
    c->cycle_timed.clear();
    return k;
}

// Deflated restarting after a full cycle of m steps that kept j0 vectors of its predecessor: the
// cycle's Hessenberg matrix, solution y and right-hand side (dr_export) give the harmonic Ritz
// vectors to keep (dr_setup), packed into the staging.  Host work only: it runs while the device
// ends the cycle and forms the true residual (0.1 ms at m = 50, k = 10, of which the device hides
// about 40 us).  *kk: the vectors the next cycle can start with (0: a plain restart).
int dr_prepare(vms_ctx* c, int m, int j0, int deflate, hipStream_t s, int* kk) {
    constexpr int ld = kMaxRestart + 1;
    *kk = 0;
    if (int rc = wait_word(c, kDrTagWord, c->cycle_gen, "read cycle state", s)) return rc;
    const GmresState* h = reinterpret_cast<const GmresState*>(c->dr_pinned);
    double* up = reinterpret_cast<double*>(reinterpret_cast<char*>(c->dr_pinned) + kDrStateBytes);
    const double rho = h->rho_m;
    if (!(rho > 0.0) || !std::isfinite(rho)) return VMS_OK;
    // Hbar (m+1) x m, entries below each column's last row cleared: the kept block's columns end
    // at row j0, an Arnoldi column j at row j + 1
    std::vector<double> Hb((size_t)(m + 1) * m, 0.0);
    for (int j = 0; j < m; ++j) {
        const int last = j < j0 ? j0 : j + 1;
        for (int i = 0; i <= last; ++i) Hb[(size_t)j * (m + 1) + i] = h->H[(size_t)j * ld + i];
    }
    // rc = c - Hbar y, c = beta e_1 (plain cycle) or beta (s, rho) in the kept basis
    std::vector<double> rcv(m + 1, 0.0);
    if (j0 > 0)
        for (int i = 0; i <= j0; ++i) rcv[i] = h->dr_c[i];
    else
        rcv[0] = h->beta;
    for (int j = 0; j < m; ++j)
        for (int i = 0; i <= m; ++i) rcv[i] -= Hb[(size_t)j * (m + 1) + i] * h->y[j];
    DrSetup S;
    const int k = dr_setup(m, deflate, Hb.data(), m + 1, rcv.data(), &S);
    if (k <= 0 || k >= m || k > kDrMax) return VMS_OK;
    // P for the stored basis: V[m] holds u_m, whose final vector is q_m = (u_m - V s) / rho
    const int mp = m + 1;
    for (int col = 0; col < k; ++col) {
        const double pm = S.P[(size_t)col * mp + m];
        for (int l = 0; l < m; ++l) up[col * mp + l] = S.P[(size_t)col * mp + l] - pm * h->scoef[l] / rho;
        up[col * mp + m] = pm / rho;
        double sv = 0.0;
        for (int l = 0; l <= m; ++l) sv += S.P[(size_t)col * mp + l] * h->svs[l];
        up[kDrOffSvs + col] = sv;
    }
    std::copy(S.Hk.begin(), S.Hk.end(), up + kDrOffH);
    std::copy(S.R.begin(), S.R.end(), up + kDrOffR);
    std::copy(S.Qt.begin(), S.Qt.end(), up + kDrOffQt);
    *kk = k;
    return VMS_OK;
}

// The kept block of H, its QR factors and the free-pressure sums go to the cycle state, and the
// basis is recombined in place: the next cycle starts with kk vectors.
template <typename T>
int dr_apply(vms_ctx* c, int m, int kk, hipStream_t s) {
    const int n = 4 * c->n_nodes, mp = m + 1;
    const double* up = reinterpret_cast<const double*>(static_cast<const char*>(c->dr_mapped) + kDrStateBytes);
    dr_load_kernel<<<1, kDrLoadThreads, 0, s>>>(kk, kk * mp, up, c->dr_p, c->gs);
    launch_dr_basis<T>(n, mp, kk, c->dr_p, mp, basis_vectors<T>(c, 0), s);
    return check_hip(c, hipGetLastError(), "deflation launch");
}

}  // namespace

hipError_t small_cycle_configure() {
    hipError_t e = hipFuncSetAttribute((const void*)small_cycle_kernel<float>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(SmallLds<float>));
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)small_cycle_kernel<double>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)sizeof(SmallLds<double>));
    return e;
}

int launch_fill(void* p, size_t bytes, hipStream_t s) {
    if (bytes == 0) return VMS_OK;
    if (bytes % 16 != 0 || ((uintptr_t)p % 16) != 0) {
        // every buffer of the library is a multiple of 16 bytes and 16-byte aligned
        return set_error(nullptr, VMS_EINVAL, "fill: unaligned buffer");
    }
    const size_t n16 = bytes / 16;
    const int g = (int)std::min<size_t>((n16 + kBlock - 1) / kBlock, 8192);
    fill_kernel<<<g, kBlock, 0, s>>>((uint4*)p, n16);
    return VMS_OK;
}

int launch_spmv(vms_ctx* c, const void* A, const void* x, void* y, hipStream_t s) {
    if (c->prec == VMS_FP64)
        spmv_kernel<double, double, double, double, 0><<<spmv_grid(c->n_nodes), kBlock, 0, s>>>(
            c->n_nodes, c->rowptr, c->colidx, (const double*)A, (const double*)x, (const double*)nullptr, (double*)y, nullptr);
    else
        spmv_kernel<float, float, float, float, 0><<<spmv_grid(c->n_nodes), kBlock, 0, s>>>(
            c->n_nodes, c->rowptr, c->colidx, (const float*)A, (const float*)x, (const double*)nullptr, (float*)y, nullptr);
    return check_hip(c, hipGetLastError(), "spmv launch");
}

int launch_bj_setup(vms_ctx* c, const void* A, void* Minv, hipStream_t s) {
    zero_count_kernel<<<1, 64, 0, s>>>(c->flags + 2);      // singular blocks of this setup
    PhaseScope ph(c, VMS_PH_PCSETUP, (double)c->n_nodes * (32.0 * elt_size(c) + 4.0), s);
    if (c->prec == VMS_FP64)
        bj_setup_kernel<double, double><<<grid_for(c->n_nodes), kBlock, 0, s>>>(c->n_nodes, c->diagpos,
                                                                              (const double*)A, (double*)Minv,
                                                                              c->flags);
    else
        bj_setup_kernel<float, float><<<grid_for(c->n_nodes), kBlock, 0, s>>>(c->n_nodes, c->diagpos,
                                                                            (const float*)A, (float*)Minv,
                                                                            c->flags);
    return check_hip(c, hipGetLastError(), "bj setup launch");
}

// Block-Jacobi for the uncondensed system: K_ff^-1 on element rows, the Schur diagonal
// inverse on node rows.
static int launch_full_pc_setup(vms_ctx* c, const void* A, void* Minv, hipStream_t s) {
    int rc = launch_bj_setup(c, A, Minv, s);
    if (rc) return rc;
    const int nn = c->full_nodes;
    if (c->prec == VMS_FP64)
        schur_diag_pc_kernel<double, double><<<grid_for(nn), kBlock, 0, s>>>(
            nn, c->rowptr, c->colidx, c->diagpos, (const double*)A, (double*)Minv, c->flags);
    else
        schur_diag_pc_kernel<float, float><<<grid_for(nn), kBlock, 0, s>>>(
            nn, c->rowptr, c->colidx, c->diagpos, (const float*)A, (float*)Minv, c->flags);
    return check_hip(c, hipGetLastError(), "schur diagonal setup launch");
}

// A P and A z for the Arnoldi steps (after the preconditioner blocks are set), and for condensed systems
// the coarse pressure mode's kappa (set before, for uncondensed ones).
template <typename T>
static void launch_ap_setup_t(vms_ctx* c, const T* A, int coarse_pressure, hipStream_t s) {
    if (c->zfull) {
        const int g = (int)((4 * c->nb + kBlock - 1) / kBlock);
        ap_blocks_kernel<T><<<g, kBlock, 0, s>>>(c->nb, c->colidx, A, (const T*)c->Minv, (T*)c->AP);
        spmv_kernel<T, double, T, double, 0><<<spmv_grid(c->n_nodes), kBlock, 0, s>>>(
            c->n_nodes, c->rowptr, c->colidx, A, c->zfull, (const double*)nullptr, (T*)c->Az, nullptr);
        return;
    }
    T* pp = coarse_pressure ? (T*)c->pp : nullptr;
    ap_rows_kernel<T><<<grid_for(4 * (int64_t)c->n_nodes), kBlock, 0, s>>>(
        c->n_nodes, c->rowptr, c->colidx, A, (const T*)c->Minv, c->dmask, (T*)c->AP, (T*)c->Az, pp);
    const int nk = pp ? c->n_nodes : 0;
    coarse_setup_kernel<T><<<red_grid(nk), kBlock, 0, s>>>(nk, c->rowptr, pp, c->red, c->gs);
}

int launch_ap_setup(vms_ctx* c, const void* A, int coarse_pressure, hipStream_t s) {
    const double es = elt_size(c);
    PhaseScope ph(c, VMS_PH_PCAPPLY, (double)c->nb * (32.0 * es + 4.0) + (double)c->n_nodes * 16.0 * es, s);
    if (c->prec == VMS_FP64)
        launch_ap_setup_t(c, (const double*)A, coarse_pressure, s);
    else
        launch_ap_setup_t(c, (const float*)A, coarse_pressure, s);
    return check_hip(c, hipGetLastError(), "A P setup launch");
}

// FP64 residual r64 = b - A x and its norm, which read_scalar(c, 0, ..) waits for.
static void launch_true_residual(vms_ctx* c, const void* A, const double* b, const double* x, hipStream_t s) {
    const int n = 4 * c->n_nodes;
    if (c->prec == VMS_FP64)
        spmv_kernel<double, double, double, double, 1><<<spmv_grid(c->n_nodes), kBlock, 0, s>>>(
            c->n_nodes, c->rowptr, c->colidx, (const double*)A, x, b, c->r64, nullptr);
    else
        spmv_kernel<float, double, double, double, 1><<<spmv_grid(c->n_nodes), kBlock, 0, s>>>(
            c->n_nodes, c->rowptr, c->colidx, (const float*)A, x, b, c->r64, nullptr);
    launch_norm<double>(c, n, c->r64, 0, s);
}

int gmres_solve(vms_ctx* c, const void* A, const double* b, double* x, const vms_solve_opts* o,
                vms_solve_info* info, hipStream_t s) {
    const int n = 4 * c->n_nodes;
    vms_solve_info inf{};
    const int m = o->restart > 0 ? std::min(o->restart, c->max_restart) : c->max_restart;
    const int max_iters = o->max_iters > 0 ? o->max_iters : 100000;
    const double rtol = o->rtol > 0 ? o->rtol : 1e-8;
    const int refine_max = o->refine_max > 0 ? o->refine_max : 30;
    // mixed ctx: inner_rtol <= 0 restarts every FP32 cycle from the FP64 residual; a positive
    // value runs FP32 restart cycles on the FP32 residual until it falls below inner_rtol
    const bool sweeps = o->inner_rtol > 0;
    const double inner_rtol = o->inner_rtol;
    // deflated restarting keeps part of every full cycle's basis; it needs the second
    // Gram-Schmidt pass (the cycle's residual is orthogonalised against the kept vectors)
    // mixed ctx with an FP64 basis: FP64 cycles on the FP32-stored matrix and preconditioner
    const bool basis64 = c->prec != VMS_FP64 && o->basis_fp64;
    const int deflate = o->deflate;
    if (deflate != 0) {
        if (deflate < 0 || deflate > kDrMax - 1 || deflate > m - 2)
            return set_error(c, VMS_EINVAL, "gmres: deflate must lie in 1 .. min(32, restart - 2)");
        if (c->prec != VMS_FP64 && !basis64 && sweeps)
            return set_error(c, VMS_EINVAL, "gmres: deflate needs inner_rtol <= 0");
        if (c->full_nodes > 0)
            return set_error(c, VMS_EINVAL, "gmres: deflate is for condensed systems only");
    }
    const int cgs2 = deflate > 0 ? 1 : o->cgs2;
    int rc;
    if (basis64 && !c->V64)
        return set_error(c, VMS_EINVAL, "gmres: basis_fp64 needs a context created with basis_fp64");
    // the constant-pressure coarse mode exists only when a pressure dof is prescribed
    const int coarse_pressure = o->coarse_pressure && c->n_pressure_pins > 0;

    // preconditioner blocks
    if (o->pc == VMS_PC_LEARNED && o->pc_weights) {
        rc = learned_blocks(c, A, o->pc_weights, c->Minv, c->prec == VMS_FP64, s);
        if (rc == VMS_ENONFINITE) {
            inf.fell_back_to_bj = 1;
            if ((rc = launch_bj_setup(c, A, c->Minv, s))) return rc;
        } else if (rc) {
            return rc;
        }
    } else if (c->full_nodes > 0) {
        if ((rc = launch_full_pc_setup(c, A, c->Minv, s))) return rc;
    } else {
        if ((rc = launch_bj_setup(c, A, c->Minv, s))) return rc;
    }
    if (c->zfull) {
        const int nn = c->full_nodes;
        if (c->prec == VMS_FP64) {
            full_coarse_vector_kernel<double, double><<<grid_for(c->n_nodes), kBlock, 0, s>>>(
                nn, c->n_nodes, c->rowptr, c->colidx, (const double*)A, (const double*)c->Minv, c->dmask, c->zfull);
            full_coarse_setup_kernel<double><<<red_grid(nn), kBlock, 0, s>>>(
                nn, c->rowptr, c->colidx, (const double*)A, c->dmask, c->zfull, coarse_pressure, c->red, c->gs);
        } else {
            full_coarse_vector_kernel<float, float><<<grid_for(c->n_nodes), kBlock, 0, s>>>(
                nn, c->n_nodes, c->rowptr, c->colidx, (const float*)A, (const float*)c->Minv, c->dmask, c->zfull);
            full_coarse_setup_kernel<float><<<red_grid(nn), kBlock, 0, s>>>(
                nn, c->rowptr, c->colidx, (const float*)A, c->dmask, c->zfull, coarse_pressure, c->red, c->gs);
        }
    }
    if ((rc = launch_ap_setup(c, A, coarse_pressure, s))) return rc;
    launch_norm<double>(c, n, b, 1, s);
    double bn = 0.0;
    if ((rc = read_scalar(c, 1, &bn, s))) return rc;
    if (!std::isfinite(bn)) return set_error(c, VMS_ENONFINITE, "gmres: non-finite right-hand side");
    // singular diagonal blocks of the preconditioner setup (applied as the identity), read
    // once the stream is drained at the end of the call
    int32_t singular = 0;
    auto read_singular = [&]() {
        return check_hip(c, hipMemcpyAsync(&singular, c->flags + 2, sizeof singular, hipMemcpyDeviceToHost, s),
                         "read singular-block count");
    };
    if (bn == 0.0) {
        if ((rc = launch_fill(x, n * sizeof(double), s))) return rc;
        if ((rc = read_singular())) return rc;
        if ((rc = check_hip(c, hipStreamSynchronize(s), "sync"))) return rc;
        inf.true_rel_res = 0.0;
        inf.singular_blocks = singular;
        if (info) *info = inf;
        return VMS_OK;
    }
    const double tol = rtol * bn;
    double rn = 0.0;
    int iters = 0;
    int status = VMS_OK;
    const bool learned = o->pc == VMS_PC_LEARNED && o->pc_weights && !inf.fell_back_to_bj;
    const int learned_budget = learned ? max_iters / 2 : max_iters;
    bool using_learned = learned;
    bool pending = false;          // an FP64 cycle was launched and not yet counted
    int j0 = 0;                    // vectors the cycle in flight kept from its predecessor
    bool dr_out = false;           // the cycle in flight hands the host its state for deflation
    bool dr_live = deflate > 0;    // deflation still in use in this solve
    double rn_start = 0.0;         // true residual before the cycle in flight
    for (;;) {
        launch_true_residual(c, A, b, x, s);
        // the host's part of the next deflated restart, while the device gets to the residual: after a
        // full cycle that did not stop, when the budgets leave room for another
        int kk = 0;
        if (pending && dr_out) {
            if ((rc = wait_word(c, kDrTagWord, c->cycle_gen, "read cycle state", s))) return rc;
            int stopped = 0;
            const int k = read_progress(c, c->cycle_gen, &stopped);
            const int after = iters + k - j0;
            if (k == m && !stopped && after < max_iters && !(using_learned && after >= learned_budget) &&
                (rc = dr_prepare(c, m, j0, deflate, s, &kk)))
                return rc;
        }
        if ((rc = read_scalar(c, 0, &rn, s))) return rc;
        int last_k = -1;
        if (pending) {
            int stopped = 0;
            last_k = finish_cycle(c, &stopped);
            iters += last_k - j0;
            inf.restarts++;
            pending = false;
            if (j0 > 0 && !(rn <= rn_start)) {
                // A deflated cycle cannot raise the residual in exact arithmetic (y = 0 is
                // feasible); when it does, the kept block's Arnoldi relation has drifted from the
                // stored vectors (in FP32 storage the rounding of the recombined basis adds up
                // over cycles).  Its correction is undone and the solve restarts plainly.
                if ((rc = check_hip(c, hipMemcpyAsync(x, c->x64, sizeof(double) * n, hipMemcpyDeviceToDevice, s),
                                    "restore iterate")))
                    return rc;
                launch_true_residual(c, A, b, x, s);
                if ((rc = read_scalar(c, 0, &rn, s))) return rc;
                dr_live = false;
                kk = 0;
                inf.deflation_stopped = 1;
            }
        }
        if (o->log_residuals && inf.logged < o->log_max) {
            convert_kernel<double, float><<<grid_for(n), kBlock, 0, s>>>(
                n, c->r64, o->log_residuals + (size_t)inf.logged * n, 1.0);
            inf.logged++;
        }
        if (!std::isfinite(rn)) {
            status = set_error(c, VMS_ENONFINITE, "gmres: non-finite residual");
            break;
        }
        if (rn <= tol) break;
        if (last_k == 0) {
            status = set_error(c, VMS_ENOCONV_GMRES, "gmres: stagnation (no Arnoldi progress)");
            break;
        }
        if (iters >= max_iters) {
            status = set_error(c, VMS_ENOCONV_GMRES, "gmres: iteration cap reached before rtol");
            break;
        }
        if (using_learned && iters >= learned_budget) {
            // the learned blocks did not deliver within half the budget: continue from the
            // current iterate with plain block-Jacobi
            if ((rc = launch_bj_setup(c, A, c->Minv, s))) return rc;
            if ((rc = launch_ap_setup(c, A, coarse_pressure, s))) return rc;
            using_learned = false;
            inf.fell_back_to_bj = 1;
            kk = 0;                // the kept basis belongs to the old operator
        }
        // the next cycle's kept vectors (0: a plain restart)
        if (kk > 0) {
            rc = (c->prec == VMS_FP64 || basis64) ? dr_apply<double>(c, m, kk, s) : dr_apply<float>(c, m, kk, s);
            if (rc) return rc;
        }
        j0 = kk;
        rn_start = rn;
        double* x_save = j0 > 0 ? c->x64 : nullptr;
        // while the learned blocks are on trial, no cycle runs past half of the budget, so that
        // the switch to block-Jacobi above happens there
        const int cap = using_learned ? learned_budget : max_iters;
        dr_out = dr_live && cap - iters >= m - j0;
        if (c->prec == VMS_FP64) {
            // one restart cycle on the FP64 residual; the true residual is recomputed above
            if ((rc = run_cycle<double, double, double>(c, c->r64, (const double*)c->Minv, x, tol, m, cap - iters,
                                                cgs2, s, 1.0, j0, nullptr, nullptr, 1.0, x_save, dr_out)))
                return rc;
            pending = true;
        } else if (basis64) {
            // the same on the FP32-stored matrix and preconditioner, applied one after the other
            // (the stored A P blocks are rounded products, not the operator the residual sees)
            if ((rc = run_cycle<double, double, float>(c, c->r64, (const float*)c->Minv, x, tol, m, cap - iters,
                                                       cgs2, s, 1.0, j0, (const float*)A, nullptr, 1.0, x_save, dr_out)))
                return rc;
            pending = true;
        } else if (!sweeps) {
            // FP64 refinement at every restart: one FP32 cycle on A d = r / ||r|| (r = b - A x in FP64,
            // A the FP32-stored matrix), its correction added to the FP64 x as ||r|| P V y.  Every
            // cycle thus starts from a residual that is exact to FP32 rounding of a unit vector; a
            // residual recomputed in FP32 from an FP32 correction carries an error near
            // eps32 |A| |d|, which on hard systems the following cycles spend their steps on.
            inf.refinements++;
            if ((rc = run_cycle<float, double, float>(c, (float*)c->r, (const float*)c->Minv, x, tol / rn, m, cap - iters, cgs2,
                                               s, rn, j0, nullptr, c->r64, 1.0 / rn, x_save, dr_out)))
                return rc;
            pending = true;
        } else {
            // FP64 iterative refinement: FP32 restarted GMRES on A d = r / ||r||, then x += ||r|| d
            if (inf.refinements >= refine_max) {
                status = set_error(c, VMS_ENOCONV_GMRES, "gmres: refinement cap reached before rtol");
                break;
            }
            inf.refinements++;
            float* rr = (float*)c->r;      // unit-norm residual of this sweep
            float* d = (float*)c->d;       // FP32 correction
            float* q = c->tvec;            // inner residual rr - A d
            convert_kernel<double, float><<<grid_for(n), kBlock, 0, s>>>(n, c->r64, rr, 1.0 / rn);
            if ((rc = launch_fill(d, n * sizeof(float), s))) return rc;
            // one sweep is asked for 0.9 of the remaining reduction (never below inner_rtol)
            const double inner_tol = std::max(inner_rtol, 0.9 * tol / rn);
            float* cycle_r = rr;
            int progress = 0;
            while (iters < cap) {
                if ((rc = run_cycle<float, float>(c, cycle_r, (const float*)c->Minv, d, inner_tol, m,
                                                  cap - iters, cgs2, s)))
                    return rc;
                spmv_kernel<float, float, float, float, 1, float><<<spmv_grid(c->n_nodes), kBlock, 0, s>>>(
                    c->n_nodes, c->rowptr, c->colidx, (const float*)A, d, rr, q, nullptr);
                launch_norm<float>(c, n, q, 2, s);
                double qn = 0.0;
                if ((rc = read_scalar(c, 2, &qn, s))) return rc;     // synchronises
                int stopped = 0;
                const int k = finish_cycle(c, &stopped);
                iters += k;
                progress += k;
                inf.restarts++;
                if (k == 0) break;
                if (o->log_residuals && inf.logged < o->log_max) {
                    convert_kernel<float, float><<<grid_for(n), kBlock, 0, s>>>(
                        n, q, o->log_residuals + (size_t)inf.logged * n, 1.0);
                    inf.logged++;
                }
                if (!(qn > inner_tol) || !std::isfinite(qn)) break;
                // The FP32 inner residual has a rounding floor near eps32 |A| |d|: when the cycle's own
                // estimate reached inner_tol but the recomputed residual did not, the sweep ends and the
                // FP64 refinement continues from the new iterate.
                if (stopped) break;
                cycle_r = q;
            }
            axpy64_kernel<float><<<grid_for(n), kBlock, 0, s>>>(n, rn, d, x);
            if (progress == 0) {
                status = set_error(c, VMS_ENOCONV_GMRES, "gmres: stagnation (no Arnoldi progress)");
                break;
            }
        }
    }
    // the per-cycle reads above wait only for their norms; the call returns with the stream drained
    if (int rs = read_singular()) return rs;
    if (int rs = check_hip(c, hipStreamSynchronize(s), "sync")) return rs;
    inf.singular_blocks = singular;
    inf.iters = iters;
    inf.true_rel_res = rn / bn;
    if (info) *info = inf;
    return status;
}

}  // namespace vms

using namespace vms;

extern "C" int vms_bsr_spmv(vms_ctx* c, const void* bsr_vals, const void* x, void* y, hipStream_t s) {
    if (!c || !bsr_vals || !x || !y) return set_error(c, VMS_EINVAL, "vms_bsr_spmv: NULL argument");
    return launch_spmv(c, bsr_vals, x, y, s);
}

extern "C" int vms_gmres_solve(vms_ctx* c, const void* bsr_vals, const double* b, double* x,
                               const vms_solve_opts* opts, vms_solve_info* info, hipStream_t s) {
    if (!c || !bsr_vals || !b || !x || !opts) return set_error(c, VMS_EINVAL, "vms_gmres_solve: NULL argument");
    if (opts->restart > c->max_restart)
        return set_error(c, VMS_EINVAL, "vms_gmres_solve: restart exceeds the allocated basis");
    return gmres_solve(c, bsr_vals, b, x, opts, info, s);
}
