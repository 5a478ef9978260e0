// Learned correction of the 4x4 block-Jacobi preconditioner (FP32 kernels).
//
// The paper leaves the Krylov preconditioner open (Section 6).  Per node i a
// two-layer perceptron maps 25 features of the condensed tangent's block row
// to a 4x4 correction Delta_i, and the preconditioner block becomes
// P_i = D_i^-1 (I + Delta_i) with Delta_i zeroed on Dirichlet rows/columns.
// With a zero output layer this is exactly block-Jacobi.  Training minimises
// mean_s ||r_s - A P r_s||^2 / ||r_s||^2 over residual samples produced by the
// method's own GMRES solves:
//   e = r - A P r,  ds = dL/d(P r) = -2 A^T e / ||r||^2,
//   dL/dDelta_i = D_i^-T ds_i r_i^T (masked),  then the MLP backward and Adam.
// A^T e uses the transposed-block map of the symmetric block pattern.  Weight
// gradients are reduced per workgroup and then across workgroups in a fixed
// order (deterministic).
#include "vms_internal.h"

namespace vms {
namespace {

constexpr int NIN = VMS_PC_NIN, NHID = VMS_PC_NHID, NOUT = VMS_PC_NOUT, NW = VMS_PC_NWEIGHTS;
constexpr int OFF_W1 = 0, OFF_B1 = NHID * NIN, OFF_W2 = OFF_B1 + NHID, OFF_B2 = OFF_W2 + NOUT * NHID;

inline int grid_for(int64_t n, int block = kBlock) { return (int)((n + block - 1) / block); }

// Features of node i (see vms.h) and D_i^-1 (float, row-major).  Four lanes per node, lane r = row r of
// the blocks, kFeatAhead blocks in flight: the launch reads every block of the matrix once, a whole
// block per quad and load.  With a lane per node (64 bytes apart, a block at a time) and the inverse
// in scratch memory it took 17.6 us at 32^3 (mixed); now 13.3, most of it FP64 arithmetic (4 or 16
// blocks in flight take the same).
constexpr int kFeatAhead = 8;

// Entry r of four, by selects: the empty asm keeps the compiler from indexing them in scratch memory.
__device__ __forceinline__ double by_lane(int r, double a, double b, double c, double d) {
    asm("" : "+v"(a));
    asm("" : "+v"(b));
    asm("" : "+v"(c));
    asm("" : "+v"(d));
    return r < 2 ? (r == 0 ? a : b) : (r == 2 ? c : d);
}

template <typename TA>
__global__ __launch_bounds__(kBlock) void features_kernel(int n, const int32_t* __restrict__ rowptr,
                                                          const int32_t* __restrict__ diagpos,
                                                          const TA* __restrict__ A, const uint8_t* __restrict__ dmask,
                                                          float* __restrict__ feats, float* __restrict__ dinv,
                                                          int32_t* flags) {
    using V4 = typename CallerVec4<TA>::type;
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    const int i = tid >> 2, r = tid & 3;
    if (i >= n) return;                         // the four lanes of a quad agree
    const int dp = diagpos[i], k1 = rowptr[i + 1];
    const V4* rows = reinterpret_cast<const V4*>(A) + r;
    const V4 d = rows[4 * (size_t)dp];
    const double dr[4] = {double(d.x), double(d.y), double(d.z), double(d.w)};
    double off = 0.0;
    for (int k = rowptr[i]; k < k1; k += kFeatAhead) {
        V4 b[kFeatAhead];
#pragma unroll
        for (int q = 0; q < kFeatAhead; ++q) b[q] = rows[4 * (size_t)min(k + q, k1 - 1)];
#pragma unroll
        for (int q = 0; q < kFeatAhead; ++q)
            if (k + q < k1 && k + q != dp)
                off += fabs(double(b[q].x)) + fabs(double(b[q].y)) + fabs(double(b[q].z)) + fabs(double(b[q].w));
    }
    double D[4][4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        D[0][c] = dpp_mov<0x00>(dr[c]);          // quad broadcasts of rows 0 .. 3
        D[1][c] = dpp_mov<0x55>(dr[c]);
        D[2][c] = dpp_mov<0xAA>(dr[c]);
        D[3][c] = dpp_mov<0xFF>(dr[c]);
    }
    double fro = 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) fro += D[q >> 2][q & 3] * D[q >> 2][q & 3];
    fro = sqrt(fro);
    float* x = feats + (size_t)i * NIN;
    const double ifro = fro > 0.0 ? 1.0 / fro : 0.0;
#pragma unroll
    for (int c = 0; c < 4; ++c) x[4 * r + c] = float(dr[c] * ifro);
    const double drr = by_lane(r, dr[0], dr[1], dr[2], dr[3]);
    x[17 + r] = float(log1p(off / fmax(fabs(drr), 1e-300)));
    x[21 + r] = (dmask[i] & (1u << r)) ? 1.f : 0.f;
    double Di[4][4];
    const bool ok = invert4(D, Di);
    if (r == 0) {
        x[16] = float(log(fmax(fro, 1e-300)));
        if (!ok) atomicAdd(&flags[2], 1);
    }
    if (!dinv) return;
    float op[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const double v = by_lane(r, Di[0][c], Di[1][c], Di[2][c], Di[3][c]);
        op[c] = ok ? float(v) : (r == c ? 1.f : 0.f);
    }
    *reinterpret_cast<float4*>(dinv + (size_t)i * 16 + 4 * r) = make_float4(op[0], op[1], op[2], op[3]);
}

// Four consecutive values of a caller's array, as floats.
typedef float f32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 load4(const float* p) {
    return *reinterpret_cast<const CallerVec4<float>::type*>(p);
}
__device__ __forceinline__ f32x4 load4(const double* p) {
    const auto v = *reinterpret_cast<const CallerVec4<double>::type*>(p);
    return f32x4{float(v.x), float(v.y), float(v.z), float(v.w)};
}

// The network runs on the matrix cores (v_mfma_f32_16x16x4: FP32 inputs, products and sums), a
// wave taking 16 nodes at a time.  With g = lane / 16 and c = lane % 16 the instruction takes
// A[row c][k g], B[k g][column c] and keeps D[row 4g + i][column c] in register i.  The order
// of the summed index is free, so a D of one product is the B (or A) of the next without moving
// a value between lanes: register i of lane group g is simply index 4g + i.
constexpr int kMlpNodes = 16;                 // nodes per wave and pass
constexpr int kHidTiles = NHID / 16;          // 16-row tiles of the hidden layer
constexpr int kInSteps = (NIN + 3) / 4;       // four inputs per instruction
constexpr int kInTiles = (NIN + 1 + 15) / 16; // 16-column tiles of the inputs and the bias
static_assert(NHID % 16 == 0 && NOUT == 16, "tiles of the network");

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// MLP forward per node and P_i = D_i^-1 (I + Delta_i); hidden activations kept for backward.
// One lane per node walked the 2,624 products serially with every weight read from LDS: 31 us
// for 35,937 nodes, about half a wave per SIMD.  As 44 matrix instructions per 16 nodes (under
// 2 us of arithmetic) it takes 12.5 us: the latency of the weights, the inputs and tanh.
constexpr int kFwdBlocks = 512;               // workgroups at most: each wave loads the weights once
template <typename TM>
__global__ __launch_bounds__(kBlock) void forward_kernel(int n, const float* __restrict__ feats,
                                                         const float* __restrict__ wts,
                                                         const float* __restrict__ dinv,
                                                         const uint8_t* __restrict__ dmask,
                                                         float* __restrict__ hid, TM* __restrict__ P,
                                                         int32_t* flags) {
    __shared__ __align__(16) float sm[kBlock / 64][kMlpNodes][NOUT + 4];   // I + Delta of a wave's nodes
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, c = lane & 15;
    float w1[kHidTiles][kInSteps], w2[kHidTiles][4];
    f32x4 b1[kHidTiles], b2;
#pragma unroll
    for (int t = 0; t < kHidTiles; ++t) {
#pragma unroll
        for (int k = 0; k < kInSteps; ++k) {
            const int f = 4 * k + g;
            w1[t][k] = f < NIN ? wts[OFF_W1 + (16 * t + c) * NIN + min(f, NIN - 1)] : 0.f;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            w2[t][i] = wts[OFF_W2 + c * NHID + 16 * t + 4 * g + i];
            b1[t][i] = wts[OFF_B1 + 16 * t + 4 * g + i];
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) b2[i] = wts[OFF_B2 + 4 * g + i];
    const int waves = gridDim.x * (kBlock / 64);
    // every wave of the workgroup makes the same number of passes (the barriers below)
    for (int64_t n0 = (int64_t)blockIdx.x * (kBlock / 64) * kMlpNodes; n0 < n; n0 += (int64_t)waves * kMlpNodes) {
        const int64_t node = n0 + wave * kMlpNodes + c;
        const bool live = node < n;
        const size_t i0 = (size_t)(live ? node : n - 1);
        float x[kInSteps];
#pragma unroll
        for (int k = 0; k < kInSteps; ++k) {
            const int f = 4 * k + g;
            x[k] = f < NIN ? feats[i0 * NIN + min(f, NIN - 1)] : 0.f;
        }
        const f32x4 dr = *reinterpret_cast<const f32x4*>(dinv + i0 * 16 + 4 * g);   // row g of D^-1
        const uint32_t dm = dmask[i0];
        f32x4 y = b2;
#pragma unroll
        for (int t = 0; t < kHidTiles; ++t) {
            f32x4 z = b1[t];
#pragma unroll
            for (int k = 0; k < kInSteps; ++k) z = mfma4(w1[t][k], x[k], z);
#pragma unroll
            for (int i = 0; i < 4; ++i) z[i] = tanhf(z[i]);
            if (hid && live) *reinterpret_cast<f32x4*>(hid + i0 * NHID + 16 * t + 4 * g) = z;
#pragma unroll
            for (int i = 0; i < 4; ++i) y = mfma4(w2[t][i], z[i], y);
        }
        // y: row g of the node's Delta
        f32x4 m;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const bool masked = (dm & (1u << g)) || (dm & (1u << q));
            m[q] = (g == q ? 1.f : 0.f) + (masked ? 0.f : y[q]);
        }
        *reinterpret_cast<f32x4*>(&sm[wave][c][4 * g]) = m;
        __syncthreads();
        float o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const f32x4 mk = *reinterpret_cast<const f32x4*>(&sm[wave][c][4 * k]);
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] += dr[k] * mk[q];
        }
        if (live) {
            using V4 = typename CallerVec4<TM>::type;
            *reinterpret_cast<V4*>(P + i0 * 16 + 4 * g) = V4{TM(o[0]), TM(o[1]), TM(o[2]), TM(o[3])};
            if (!(isfinite(o[0]) && isfinite(o[1]) && isfinite(o[2]) && isfinite(o[3]))) atomicAdd(&flags[3], 1);
        }
        __syncthreads();
    }
}
inline int forward_grid(int n) { return std::min(kFwdBlocks, grid_for(n, kMlpNodes * (kBlock / 64))); }

// ------------------------------------------------------------------------ residual samples
// The samples of a batch go through the matrix together, up to eight at a time, so that each of
// A P r and A^T e reads it once for all of them: 20 + 17 us for eight samples at 35,937 nodes
// (FP32), where a pass per sample took 8 x (12.5 + 12.6) us and four more launches a sample.  Vectors of a group are interleaved per node
// as [node][dof][S], S = 1, 2, 4 or 8 the group's size rounded up: a block's column of S
// samples is S adjacent 4-byte values per dof.  Eight lanes share a block row as in the
// solver's SpMV: lane (q, r) takes row r of blocks q, q + 2, ...
constexpr int kGroupMax = 8;
constexpr int kRowLanes = 8;
constexpr int kBatchUnroll = 4;               // blocks of a lane in flight
constexpr int kBatchBlocks = 2048;            // workgroups at most: two sums a sample each
static_assert((2 * kGroupMax) * (kBatchBlocks + 1) <= kRedBlocks * (kMaxRestart + 1), "batch sums exceed scratch");

template <int I>
__device__ __forceinline__ float quad_get(float v) {       // component I of a quad's four values
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), I * 0x55, 0xF, 0xF, false));
}

template <int S>
__device__ __forceinline__ void load_group(const float* __restrict__ p, float (&v)[S]) {
    if constexpr (S >= 4) {
#pragma unroll
        for (int k = 0; k < S / 4; ++k) {
            const f32x4 x = reinterpret_cast<const f32x4*>(p)[k];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[4 * k + q] = x[q];
        }
    } else {
#pragma unroll
        for (int k = 0; k < S; ++k) v[k] = p[k];
    }
}
template <int S>
__device__ __forceinline__ void store_group(float* __restrict__ p, const float (&v)[S]) {
    if constexpr (S >= 4) {
#pragma unroll
        for (int k = 0; k < S / 4; ++k)
            reinterpret_cast<f32x4*>(p)[k] = f32x4{v[4 * k], v[4 * k + 1], v[4 * k + 2], v[4 * k + 3]};
    } else {
#pragma unroll
        for (int k = 0; k < S; ++k) p[k] = v[k];
    }
}

// t = P r for the group's samples (node-local 4x4 products); samples past nb are zero.
template <int S>
__global__ void group_apply_kernel(int n, int nb, const float* __restrict__ P, const float* __restrict__ r,
                                   float* __restrict__ t) {
    const int64_t tid = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (tid >= 4 * (int64_t)n) return;
    const f32x4 p = *reinterpret_cast<const f32x4*>(P + tid * 4);
    const size_t N = 4 * (size_t)n;
    float x[S], o[S];
#pragma unroll
    for (int b = 0; b < S; ++b) x[b] = b < nb ? r[b * N + tid] : 0.f;
#pragma unroll
    for (int b = 0; b < S; ++b)
        o[b] = p[0] * quad_get<0>(x[b]) + p[1] * quad_get<1>(x[b]) + p[2] * quad_get<2>(x[b]) +
               p[3] * quad_get<3>(x[b]);
    store_group<S>(t + tid * S, o);
}

// Sums of S values over the wave, as a reduce-scatter: lane l < S returns that of sample
// bit-reversed l.  The order is fixed.
template <int S>
__device__ __forceinline__ double group_wave_sum(double (&v)[S]) {
    const int lane = threadIdx.x & 63;
    int off = 1;
#pragma unroll
    for (int w = S / 2; w >= 1; w >>= 1) {
        const bool up = (lane & off) != 0;
#pragma unroll
        for (int i = 0; i < w; ++i) {
            const double send = up ? v[i] : v[w + i], keep = up ? v[w + i] : v[i];
            v[i] = keep + __shfl_xor(send, off, 64);
        }
        off <<= 1;
    }
    for (; off < 64; off <<= 1) v[0] += __shfl_xor(v[0], off, 64);
    return v[0];
}
template <int S>
__device__ __forceinline__ int group_sum_index(int lane) {
    int s = 0;
#pragma unroll
    for (int w = S / 2, b = 0; w >= 1; w >>= 1, ++b) s += ((lane >> b) & 1) * w;
    return s;
}

// e = r - A t for the group, and per workgroup the partial sums of e^2 (part[s][workgroup]) and
// r^2 (part[S + s][workgroup]) of every sample s: no atomics, so that training is reproducible.
template <typename TA, int S>
__global__ __launch_bounds__(kBlock) void group_residual_kernel(int n, int nb, const int32_t* __restrict__ rowptr,
                                                                const int32_t* __restrict__ colidx,
                                                                const TA* __restrict__ A, const float* __restrict__ t,
                                                                const float* __restrict__ rb, float* __restrict__ e,
                                                                double* __restrict__ part) {
    const int sub = threadIdx.x % kRowLanes, q = sub >> 2, r = sub & 3;
    constexpr int Q = kRowLanes / 4;
    const size_t N = 4 * (size_t)n;
    double se[S], sr[S];
#pragma unroll
    for (int b = 0; b < S; ++b) se[b] = sr[b] = 0.0;
    for (int row = (blockIdx.x * kBlock + threadIdx.x) / kRowLanes; row < n; row += gridDim.x * (kBlock / kRowLanes)) {
        const int k1 = rowptr[row + 1];
        float acc[S], rv[S];
#pragma unroll
        for (int b = 0; b < S; ++b) {
            acc[b] = 0.f;
            rv[b] = b < nb ? rb[b * N + 4 * (size_t)row + r] : 0.f;
        }
        for (int k0 = rowptr[row] + q; k0 < k1; k0 += kBatchUnroll * Q) {
            int col[kBatchUnroll];
            f32x4 a[kBatchUnroll];
            float x[kBatchUnroll][S];
#pragma unroll
            for (int u = 0; u < kBatchUnroll; ++u) {
                const int k = k0 + u * Q;
                col[u] = k < k1 ? colidx[k] : -1;
            }
#pragma unroll
            for (int u = 0; u < kBatchUnroll; ++u)
                if (col[u] >= 0) {
                    a[u] = load4(A + (size_t)(k0 + u * Q) * 16 + r * 4);
                    load_group<S>(t + ((size_t)col[u] * 4 + r) * S, x[u]);
                }
#pragma unroll
            for (int u = 0; u < kBatchUnroll; ++u)
                if (col[u] >= 0) {                 // the four lanes of a quad agree
#pragma unroll
                    for (int b = 0; b < S; ++b)
                        acc[b] += a[u][0] * quad_get<0>(x[u][b]) + a[u][1] * quad_get<1>(x[u][b]) +
                                  a[u][2] * quad_get<2>(x[u][b]) + a[u][3] * quad_get<3>(x[u][b]);
                }
        }
        float ev[S];
#pragma unroll
        for (int b = 0; b < S; ++b) {
            const float other = __shfl_xor(acc[b], 4, 64);
            ev[b] = b < nb ? rv[b] - (acc[b] + other) : 0.f;
            if (q == 0) {
                se[b] += double(ev[b]) * double(ev[b]);
                sr[b] += double(rv[b]) * double(rv[b]);
            }
        }
        if (q == 0) store_group<S>(e + (4 * (size_t)row + r) * S, ev);
    }
    __shared__ double ls[kBlock / 64][2 * S];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const double te = group_wave_sum<S>(se), tr = group_wave_sum<S>(sr);
    if (lane < S) {
        ls[wave][group_sum_index<S>(lane)] = te;
        ls[wave][S + group_sum_index<S>(lane)] = tr;
    }
    __syncthreads();
    if (threadIdx.x < 2 * S) {
        double v = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) v += ls[w][threadIdx.x];
        part[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = v;
    }
}

// sums[i] = the nb partials of sum i in a fixed order (one workgroup a sum: strided serial
// sums, then a pairwise tree in LDS)
__global__ __launch_bounds__(kBlock) void group_sums_kernel(int nb, const double* __restrict__ part,
                                                            double* __restrict__ sums) {
    __shared__ double ls[kBlock];
    const double* p = part + (size_t)blockIdx.x * nb;
    double s = 0.0;
    for (int i = threadIdx.x; i < nb; i += kBlock) s += p[i];
    ls[threadIdx.x] = s;
    __syncthreads();
    for (int h = kBlock / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h) ls[threadIdx.x] += ls[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = ls[0];
}

// g = A^T e through the transposed-block map, and straight from it the gradient of the blocks:
//   gdelta_i (+)= sum_s scale_s D_i^-T g_s r_s^T,  scale_s = -2 / (nbatch ||r_s||^2),
// added to the earlier groups' unless first; workgroup 0 also adds the group's loss
// sum_s ||e_s||^2 / (nbatch ||r_s||^2).  Lane r takes row r of a block, so that its own value of
// e serves the block's four columns; the quad's partial columns meet once per block row.
template <typename TA, int S>
__global__ __launch_bounds__(kBlock) void group_grad_kernel(int n, int nb, const int32_t* __restrict__ rowptr,
                                                            const int32_t* __restrict__ colidx,
                                                            const int32_t* __restrict__ tpos,
                                                            const TA* __restrict__ A, const float* __restrict__ e,
                                                            const float* __restrict__ rb,
                                                            const float* __restrict__ dinv,
                                                            const double* __restrict__ sums, int nbatch, int first,
                                                            float* __restrict__ gdelta, float* __restrict__ loss) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        float l = first ? 0.f : loss[0];
        for (int b = 0; b < nb; ++b)
            if (sums[S + b] > 0.0) l += float(sums[b] / (nbatch * sums[S + b]));
        loss[0] = l;
    }
    const int sub = threadIdx.x % kRowLanes, q = sub >> 2, r = sub & 3;
    constexpr int Q = kRowLanes / 4;
    const size_t N = 4 * (size_t)n;
    float scale[S];
#pragma unroll
    for (int b = 0; b < S; ++b) {
        const double rr = b < nb ? sums[S + b] : 0.0;
        scale[b] = rr > 0.0 ? float(-2.0 / (nbatch * rr)) : 0.f;
    }
    for (int row = (blockIdx.x * kBlock + threadIdx.x) / kRowLanes; row < n; row += gridDim.x * (kBlock / kRowLanes)) {
        const int k1 = rowptr[row + 1];
        float rv[S], di[4];
#pragma unroll
        for (int b = 0; b < S; ++b) rv[b] = b < nb ? rb[b * N + 4 * (size_t)row + r] : 0.f;
#pragma unroll
        for (int k = 0; k < 4; ++k) di[k] = dinv[(size_t)row * 16 + 4 * k + r];
        float acc[4][S];                           // this lane's part of column c
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int b = 0; b < S; ++b) acc[c][b] = 0.f;
        for (int k0 = rowptr[row] + q; k0 < k1; k0 += kBatchUnroll * Q) {
            int col[kBatchUnroll], tp[kBatchUnroll];
            f32x4 a[kBatchUnroll];
            float x[kBatchUnroll][S];
#pragma unroll
            for (int u = 0; u < kBatchUnroll; ++u) {
                const int k = k0 + u * Q;
                col[u] = k < k1 ? colidx[k] : -1;
                tp[u] = k < k1 ? tpos[k] : 0;
            }
#pragma unroll
            for (int u = 0; u < kBatchUnroll; ++u)
                if (col[u] >= 0) {
                    a[u] = load4(A + (size_t)tp[u] * 16 + r * 4);
                    load_group<S>(e + ((size_t)col[u] * 4 + r) * S, x[u]);
                }
#pragma unroll
            for (int u = 0; u < kBatchUnroll; ++u)
                if (col[u] >= 0) {
#pragma unroll
                    for (int c = 0; c < 4; ++c)
#pragma unroll
                        for (int b = 0; b < S; ++b) acc[c][b] += a[u][c] * x[u][b];
                }
        }
        // column c of the quad's four rows: a reduce-scatter, lane r keeps column r; then the
        // two halves of the row
        const bool x1 = (r & 1) != 0, x2 = (r & 2) != 0;
        float gv[S];
#pragma unroll
        for (int b = 0; b < S; ++b) {
            const float lo = (x2 ? acc[2][b] : acc[0][b]) + __shfl_xor(x2 ? acc[0][b] : acc[2][b], 2, 64);
            const float hi = (x2 ? acc[3][b] : acc[1][b]) + __shfl_xor(x2 ? acc[1][b] : acc[3][b], 2, 64);
            float v = (x1 ? hi : lo) + __shfl_xor(x1 ? lo : hi, 1, 64);
            gv[b] = v + __shfl_xor(v, 4, 64);
        }
        // row r of the gradient block: (D^-T g)_r r^T (the halves hold the same values)
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
        f32x4* dst = reinterpret_cast<f32x4*>(gdelta + (size_t)row * 16 + 4 * r);
        if (!first) o = *dst;
#pragma unroll
        for (int b = 0; b < S; ++b) {
            const float dg = di[0] * quad_get<0>(gv[b]) + di[1] * quad_get<1>(gv[b]) + di[2] * quad_get<2>(gv[b]) +
                             di[3] * quad_get<3>(gv[b]);
            const float r0 = quad_get<0>(rv[b]), r1 = quad_get<1>(rv[b]), r2 = quad_get<2>(rv[b]),
                        r3 = quad_get<3>(rv[b]);
            if (b < nb) {
                const float s = scale[b] * dg;
                o[0] += s * r0;
                o[1] += s * r1;
                o[2] += s * r2;
                o[3] += s * r3;
            }
        }
        if (q == 0) *dst = o;
    }
}

// MLP backward, partial weight gradients per workgroup.  Both contractions are matrix products
// over the nodes: gz = (gy W2) (1 - h^2) per node, then gW1 += gz^T [x 1] and gW2 += gy^T h, 64
// instructions per 16 nodes and wave, the weight gradients staying in 48 accumulators.  (13 us for
// 35,937 nodes; one thread per weight over nodes staged in LDS read two LDS words per product
// and took 99 us.)  gz comes out as D[node 4g + i][hidden c], which is the A operand of the second
// product as it stands.
constexpr int kBwdNodes = kMlpNodes * (kBlock / 64);
__global__ __launch_bounds__(kBlock) void backward_kernel(int n, const float* __restrict__ feats,
                                                          const float* __restrict__ hid,
                                                          const float* __restrict__ gdelta,
                                                          const uint8_t* __restrict__ dmask,
                                                          const float* __restrict__ wts, float* __restrict__ wpart) {
    __shared__ float lw[kBlock / 64][NW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int g = lane >> 4, c = lane & 15;
    float w2[kHidTiles][4];                        // W2[4g + s][16t + c]
#pragma unroll
    for (int t = 0; t < kHidTiles; ++t)
#pragma unroll
        for (int s = 0; s < 4; ++s) w2[t][s] = wts[OFF_W2 + (4 * g + s) * NHID + 16 * t + c];
    f32x4 a1[kHidTiles][kInTiles], a2[kHidTiles];
    float ab2 = 0.f;                               // sum of gy[., c] over this lane group's nodes
#pragma unroll
    for (int t = 0; t < kHidTiles; ++t) {
        a2[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int f = 0; f < kInTiles; ++f) a1[t][f] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int64_t step = (int64_t)gridDim.x * kBwdNodes;
    for (int64_t n0 = (int64_t)blockIdx.x * kBwdNodes + wave * kMlpNodes; n0 < n; n0 += step) {
        // gy of node n0 + c, outputs 4g .. 4g + 3 (zero past the last node)
        f32x4 gyr = {0.f, 0.f, 0.f, 0.f};
        if (n0 + c < n) {
            gyr = *reinterpret_cast<const f32x4*>(gdelta + (size_t)(n0 + c) * 16 + 4 * g);
            const uint32_t dm = dmask[n0 + c];
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if ((dm & (1u << g)) || (dm & (1u << s))) gyr[s] = 0.f;
        }
        // node n0 + 4g + i: output gradient c, hidden unit 16t + c, input 16f + c (the bias is
        // an input of one)
        float gyc[4], h[4][kHidTiles], x[4][kInTiles];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t node = n0 + 4 * g + i;
            const bool live = node < n;
            const size_t nd = (size_t)(live ? node : n - 1);
            const uint32_t dm = dmask[nd];
            const bool off = !live || (dm & (1u << (c >> 2))) || (dm & (1u << (c & 3)));
            const float gv = gdelta[nd * 16 + c];
            gyc[i] = off ? 0.f : gv;
#pragma unroll
            for (int t = 0; t < kHidTiles; ++t) h[i][t] = hid[nd * NHID + 16 * t + c];
#pragma unroll
            for (int f = 0; f < kInTiles; ++f) {
                const int k = 16 * f + c;
                const float xv = feats[nd * NIN + min(k, NIN - 1)];
                x[i][f] = k < NIN ? xv : (k == NIN ? 1.f : 0.f);
            }
            ab2 += gyc[i];
        }
#pragma unroll
        for (int t = 0; t < kHidTiles; ++t) {
            f32x4 gz = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 4; ++s) gz = mfma4(gyr[s], w2[t][s], gz);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float z = gz[i] * (1.f - h[i][t] * h[i][t]);
#pragma unroll
                for (int f = 0; f < kInTiles; ++f) a1[t][f] = mfma4(z, x[i][f], a1[t][f]);
                a2[t] = mfma4(gyc[i], h[i][t], a2[t]);
            }
        }
    }
    ab2 += __shfl_xor(ab2, 16, 64);
    ab2 += __shfl_xor(ab2, 32, 64);
    float* l = lw[wave];
#pragma unroll
    for (int t = 0; t < kHidTiles; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int hd = 16 * t + 4 * g + i;     // row of a1
#pragma unroll
            for (int f = 0; f < kInTiles; ++f) {
                const int k = 16 * f + c;
                if (k < NIN) l[OFF_W1 + hd * NIN + k] = a1[t][f][i];
                if (k == NIN) l[OFF_B1 + hd] = a1[t][f][i];
            }
            l[OFF_W2 + (4 * g + i) * NHID + 16 * t + c] = a2[t][i];
        }
    if (g == 0) l[OFF_B2 + c] = ab2;
    __syncthreads();
    for (int wi = threadIdx.x; wi < NW; wi += kBlock) {
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) s += lw[w][wi];
        wpart[(size_t)blockIdx.x * NW + wi] = s;
    }
}

// grad = sum of the partials (fixed order); Adam update when lr > 0.  A workgroup takes 32
// adjacent weights, eight threads a weight sharing its partials (one thread a weight was a
// serial chain of 256 loads on eleven workgroups: 63 us, now 5 us).
constexpr int kAdamWeights = 32, kAdamLanes = kBlock / kAdamWeights;
__global__ __launch_bounds__(kBlock) void adam_kernel(int nparts, const float* __restrict__ wpart,
                                                      float* __restrict__ wts, float* __restrict__ mstate,
                                                      float* __restrict__ vstate, int step, float lr,
                                                      float* __restrict__ grad_out) {
    __shared__ float ls[kAdamLanes][kAdamWeights];
    const int k = threadIdx.x % kAdamWeights, q = threadIdx.x / kAdamWeights;
    const int wi = blockIdx.x * kAdamWeights + k;
    float s = 0.f;
    if (wi < NW) {
#pragma unroll 8
        for (int p = q; p < nparts; p += kAdamLanes) s += wpart[(size_t)p * NW + wi];
    }
    ls[q][k] = s;
    __syncthreads();
    if (q != 0 || wi >= NW) return;
    float g = 0.f;
#pragma unroll
    for (int p = 0; p < kAdamLanes; ++p) g += ls[p][k];
    if (grad_out) grad_out[wi] = g;
    if (!(lr > 0.f)) return;
    const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
    const float m = b1 * mstate[wi] + (1.f - b1) * g;
    const float v = b2 * vstate[wi] + (1.f - b2) * g * g;
    mstate[wi] = m;
    vstate[wi] = v;
    const float mh = m / (1.f - powf(b1, (float)step));
    const float vh = v / (1.f - powf(b2, (float)step));
    wts[wi] -= lr * mh / (sqrtf(vh) + eps);
}

__global__ void reset_pc_flags_kernel(int32_t* flags) {
    if (threadIdx.x == 0) {
        flags[2] = 0;
        flags[3] = 0;
    }
}

constexpr int kBwdBlocks = 256;

int features(vms_ctx* c, const void* A, float* feats, float* dinv, hipStream_t s) {
    if (c->prec == VMS_FP64)
        features_kernel<double><<<grid_for(4 * (int64_t)c->n_nodes), kBlock, 0, s>>>(c->n_nodes, c->rowptr, c->diagpos,
                                                                       (const double*)A, c->dmask, feats, dinv,
                                                                       c->flags);
    else
        features_kernel<float><<<grid_for(4 * (int64_t)c->n_nodes), kBlock, 0, s>>>(c->n_nodes, c->rowptr, c->diagpos,
                                                                      (const float*)A, c->dmask, feats, dinv,
                                                                      c->flags);
    return check_hip(c, hipGetLastError(), "features launch");
}

// One group of samples (nb of the batch of nbatch, interleaved S to a node) through P, A and
// A^T: t and e are scratch of 4 n S floats each.
template <typename TA, int S>
void launch_group(vms_ctx* c, const TA* A, int nb, int nbatch, int first, const float* r, const float* P,
                  const float* dinv, float* t, float* e, float* gdelta, float* loss, hipStream_t s) {
    const int n = c->n_nodes;
    const int g = std::min(kBatchBlocks, grid_for((int64_t)kRowLanes * n));
    double* part = c->red->partial;                        // reduction scratch: idle here
    double* sums = part + (size_t)2 * S * g;
    group_apply_kernel<S><<<grid_for(4 * (int64_t)n), kBlock, 0, s>>>(n, nb, P, r, t);
    group_residual_kernel<TA, S><<<g, kBlock, 0, s>>>(n, nb, c->rowptr, c->colidx, A, t, r, e, part);
    group_sums_kernel<<<2 * S, kBlock, 0, s>>>(g, part, sums);
    group_grad_kernel<TA, S><<<g, kBlock, 0, s>>>(n, nb, c->rowptr, c->colidx, c->tpos, A, e, r, dinv, sums, nbatch,
                                                  first, gdelta, loss);
}

// The batch in groups of at most eight samples.  The group's vectors live in the Krylov basis,
// which holds nothing between solves; a context whose basis is too short for the group (a
// restart length below 2 S - 1 in FP32) takes smaller groups, down to one sample at a time in
// the context's own training vectors.
template <typename TA>
void launch_batch(vms_ctx* c, const TA* A, const float* r_batch, int nbatch, const float* P, const float* dinv,
                  float* gdelta, float* loss, hipStream_t s) {
    const size_t N = 4 * (size_t)c->n_nodes;
    const size_t room = (size_t)(c->max_restart + 1) * sizeof(TA) / sizeof(float);   // FP32 vectors in the basis
    int cap = kGroupMax;
    while (cap > 1 && 2 * (size_t)cap > room) cap >>= 1;
    for (int b0 = 0; b0 < nbatch; b0 += cap) {
        const int nb = std::min(cap, nbatch - b0);
        const float* r = r_batch + b0 * N;
        int S = 1;
        while (S < nb) S <<= 1;
        float* t = S == 1 ? c->tvec : (float*)c->V;
        float* e = t + N * S;
        auto go = [&](auto sz) {
            launch_group<TA, decltype(sz)::value>(c, A, nb, nbatch, b0 == 0, r, P, dinv, t, e, gdelta, loss, s);
        };
        if (S == 1) go(std::integral_constant<int, 1>{});
        else if (S == 2) go(std::integral_constant<int, 2>{});
        else if (S == 4) go(std::integral_constant<int, 4>{});
        else go(std::integral_constant<int, 8>{});
    }
}

}  // namespace

int learned_blocks(vms_ctx* c, const void* A, const float* weights, void* Minv_out, int out_is_double,
                   hipStream_t s) {
    PhaseScope ph(c, VMS_PH_PCSETUP, (double)c->n_nodes * (32.0 * elt_size(c) + 4.0), s);
    reset_pc_flags_kernel<<<1, 64, 0, s>>>(c->flags);
    int rc = features(c, A, c->feats, c->gblk, s);   // gblk holds D^-1 here
    if (rc) return rc;
    if (out_is_double)
        forward_kernel<double><<<forward_grid(c->n_nodes), kBlock, 0, s>>>(c->n_nodes, c->feats, weights, c->gblk,
                                                                      c->dmask, nullptr, (double*)Minv_out, c->flags);
    else
        forward_kernel<float><<<forward_grid(c->n_nodes), kBlock, 0, s>>>(c->n_nodes, c->feats, weights, c->gblk,
                                                                     c->dmask, nullptr, (float*)Minv_out, c->flags);
    if ((rc = check_hip(c, hipGetLastError(), "learned blocks launch"))) return rc;
    int32_t h[4];
    if ((rc = check_hip(c, hipMemcpyAsync(h, c->flags, sizeof h, hipMemcpyDeviceToHost, s), "read flags"))) return rc;
    if ((rc = check_hip(c, hipStreamSynchronize(s), "sync"))) return rc;
    if (h[2] || h[3]) return set_error(c, VMS_ENONFINITE, "learned preconditioner produced a non-finite block");
    return VMS_OK;
}

}  // namespace vms

using namespace vms;

extern "C" int vms_pc_features(vms_ctx* c, const void* bsr_vals, float* feats, hipStream_t s) {
    if (!c || !bsr_vals || !feats) return set_error(c, VMS_EINVAL, "vms_pc_features: NULL argument");
    return features(c, bsr_vals, feats, nullptr, s);
}

extern "C" int vms_pc_blocks(vms_ctx* c, const void* bsr_vals, const float* weights, float* P, hipStream_t s) {
    if (!c || !bsr_vals || !P) return set_error(c, VMS_EINVAL, "vms_pc_blocks: NULL argument");
    int rc = features(c, bsr_vals, c->feats, c->gblk, s);
    if (rc) return rc;
    if (!weights) {   // plain block-Jacobi: P = D^-1
        return check_hip(c, hipMemcpyAsync(P, c->gblk, (size_t)c->n_nodes * 16 * sizeof(float),
                                           hipMemcpyDeviceToDevice, s), "copy blocks");
    }
    forward_kernel<float><<<forward_grid(c->n_nodes), kBlock, 0, s>>>(c->n_nodes, c->feats, weights, c->gblk, c->dmask,
                                                                 nullptr, P, c->flags);
    return check_hip(c, hipGetLastError(), "pc blocks launch");
}

extern "C" int vms_pc_train_step(vms_ctx* c, const void* bsr_vals, const float* r_batch, int32_t nbatch,
                                 float* weights, float* adam_state, int32_t step, float lr, float* grad_out,
                                 float* loss_out, hipStream_t s) {
    if (!c || !bsr_vals || !r_batch || !weights || nbatch <= 0)
        return set_error(c, VMS_EINVAL, "vms_pc_train_step: NULL argument or empty batch");
    if (lr > 0.f && (!adam_state || step < 1))
        return set_error(c, VMS_EINVAL, "vms_pc_train_step: Adam needs adam_state and step >= 1");
    const int n = c->n_nodes;
    float* dinv = c->gblk;             // D^-1 blocks
    float* P = c->pblk;                // preconditioner blocks
    float* gdelta = c->gdel;           // [n][16]
    float* loss = c->fscal;
    int rc = features(c, bsr_vals, c->feats, dinv, s);
    if (rc) return rc;
    forward_kernel<float><<<forward_grid(n), kBlock, 0, s>>>(n, c->feats, weights, dinv, c->dmask, c->hid, P,
                                                             c->flags);
    if (c->prec == VMS_FP64)
        launch_batch<double>(c, (const double*)bsr_vals, r_batch, nbatch, P, dinv, gdelta, loss, s);
    else
        launch_batch<float>(c, (const float*)bsr_vals, r_batch, nbatch, P, dinv, gdelta, loss, s);
    const int nparts = std::min(kBwdBlocks, std::max(1, (n + kBwdNodes - 1) / kBwdNodes));
    backward_kernel<<<nparts, kBlock, 0, s>>>(n, c->feats, c->hid, gdelta, c->dmask, weights, c->wgrad);
    adam_kernel<<<grid_for(NW, kAdamWeights), kBlock, 0, s>>>(nparts, c->wgrad, weights, adam_state,
                                                adam_state ? adam_state + NW : nullptr, step, lr, grad_out);
    if (loss_out)
        if ((rc = check_hip(c, hipMemcpyAsync(loss_out, loss, sizeof(float), hipMemcpyDeviceToDevice, s), "loss")))
            return rc;
    return check_hip(c, hipGetLastError(), "train step launch");
}
