// The featureless convolution (Section 3.1, "Featureless Convolutions",
// Eq. 9-10): when every input carries the constant feature 1, the feature
// matrix drops out and Z = G~ Phi_0, where G~[i, m] adds up the values of
// basis function m along row i and Phi_0 is an M x P matrix.
//
// Forward: a group of kFLanes lanes per row takes the row's edges in turn,
// evaluates their basis values (or reads them), and adds them up in float64,
// lane partial sums first and then across the lanes, so the sums do not depend
// on scheduling; the group then writes Z[i, :] = G~[i, :] Phi_0, a lane per
// output channel.  Backward: dPhi_0 = G~^T dZ; a block makes G~ of kDRows rows
// at a time in LDS and keeps its part of the product in registers, and the
// blocks' parts are added in order (G~ reaches memory only where dZ is wide).
#include <type_traits>

#include "basis.hpp"
#include "common.hpp"
#include "spmm.hpp"

namespace sbc {
namespace {

constexpr int kFLanes = 16;
constexpr int kFThreads = 256;

// Sum over the 16 lanes of a DPP row, in every lane: xor 1, xor 2, then the
// mirrored quads and halves.  (Moves within the vector ALU; as shuffles through
// LDS the 4 steps of M float64 sums took longer than the edges.)
__device__ __forceinline__ double row16_sum(double x) {
#define SBC_STEP(ctrl)                                                              \
    do {                                                                            \
        const int64_t u = __builtin_bit_cast(int64_t, x);                           \
        const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)u, ctrl, 0xf, 0xf, true); \
        const uint32_t hi =                                                         \
            (uint32_t)__builtin_amdgcn_mov_dpp((int)(u >> 32), ctrl, 0xf, 0xf, true); \
        x += __builtin_bit_cast(double, (int64_t)(((uint64_t)hi << 32) | lo));      \
    } while (0)
    SBC_STEP(0xB1);   // quad_perm [1, 0, 3, 2]
    SBC_STEP(0x4E);   // quad_perm [2, 3, 0, 1]
    SBC_STEP(0x141);  // row_half_mirror
    SBC_STEP(0x140);  // row_mirror
#undef SBC_STEP
    return x;
}

constexpr int kSumsGiven = -1;  // (a mode of the product alone, below)

// G~[r, :] in every lane of the row's group (sl: the lane in it).
// kMode: 0 basis values read from v; 1 windowed point monomials; 2 event
// offsets with decay; 3 the weighted monomials (Eq. 11), whose common factor
// 1 / W_i is taken out of the row's sums.
template <int M, int kMode>
__device__ __forceinline__ void row_sums(int64_t r, int sl, const int32_t *__restrict__ row_ptr,
                                         const int32_t *__restrict__ col_idx, int64_t nnz_bound,
                                         const float *__restrict__ v, const sbc_geometry &g,
                                         double (&acc)[M]) {
    // entries past nnz_bound (a malformed pattern) are not read
    const int64_t e1 = row_ptr[r + 1] < nnz_bound ? (int64_t)row_ptr[r + 1] : nnz_bound;
    const int64_t e0 = row_ptr[r] < e1 ? (int64_t)row_ptr[r] : e1;
    const double inv_r = kMode == 1 || kMode == 3 ? 1.0 / (double)g.radius : 0.0;
    const float inv_tau = kMode == 2 ? 1.0f / g.tau : 0.f;
    float qx = 0.f, qy = 0.f, qz = 0.f;
    if constexpr (kMode == 1 || kMode == 3) {
        qx = g.x_out[3 * r];
        qy = g.x_out[3 * r + 1];
        qz = g.x_out[3 * r + 2];
    }
#pragma unroll
    for (int m = 0; m < M; ++m) acc[m] = 0.0;
    for (int64_t e = e0 + sl; e < e1; e += kFLanes) {
        if constexpr (kMode == 3) {
            const int64_t j = col_idx[e];
            const float px = g.x_in[3 * j], py = g.x_in[3 * j + 1], pz = g.x_in[3 * j + 2];
            const double w = point_weight(qx, qy, qz, px, py, pz, inv_r);
            const double x = ((double)qx - (double)px) * inv_r;
            const double y = ((double)qy - (double)py) * inv_r;
            const double z = ((double)qz - (double)pz) * inv_r;
            const double wx = w * x, wy = w * y, wz = w * z;
            acc[0] += w;
            acc[1] += wx;
            acc[2] += wy;
            acc[3] += wz;
            acc[4] += wx * x;
            acc[5] += wy * y;
            acc[6] += wz * z;
            acc[7] += wx * y;
            acc[8] += wx * z;
            acc[9] += wy * z;
        } else {
            float b[M];
            if constexpr (kMode == 0) {
#pragma unroll
                for (int m = 0; m < M; ++m) b[m] = v[e * M + m];
            } else if constexpr (kMode == 1) {
                const int64_t j = col_idx[e];
                point_basis<M>(qx, qy, qz, g.x_in[3 * j], g.x_in[3 * j + 1], g.x_in[3 * j + 2],
                               inv_r, b);
            } else {
                const int64_t j = col_idx[e];
                const int k = event_index(g.px[r] - g.px[j], g.py[r] - g.py[j]);
                const float d = event_decay(g.t[r], g.t[j], inv_tau);
#pragma unroll
                for (int m = 0; m < M; ++m) b[m] = m == k ? d : 0.f;
            }
#pragma unroll
            for (int m = 0; m < M; ++m) acc[m] += (double)b[m];
        }
    }
#pragma unroll
    for (int m = 0; m < M; ++m) acc[m] = row16_sum(acc[m]);
    if constexpr (kMode == 3) {
        const double s = acc[0] != 0.0 ? 1.0 / acc[0] : 0.0;
#pragma unroll
        for (int m = 0; m < M; ++m) acc[m] *= s;
    }
}

// Z = G~ Phi_0, or (not kWritesZ) G~ itself, [n_rows, M].
template <int M, int kMode, bool kWritesZ>
__global__ void __launch_bounds__(kFThreads)
    featureless_kernel(int32_t n_rows, const int32_t *__restrict__ row_ptr,
                       const int32_t *__restrict__ col_idx, int64_t nnz_bound,
                       const float *__restrict__ v, sbc_geometry g,
                       const float *__restrict__ Phi, int32_t P, float *__restrict__ out) {
    const int sl = threadIdx.x % kFLanes;
    const int64_t r = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kFLanes;
    if (r >= n_rows) return;  // a group leaves as a whole
    double acc[M];
    row_sums<M, kMode>(r, sl, row_ptr, col_idx, nnz_bound, v, g, acc);
    if constexpr (!kWritesZ) {
        if (sl < M) {
            float x = 0.f;
#pragma unroll
            for (int m = 0; m < M; ++m)
                if (m == sl) x = (float)acc[m];
            out[r * M + sl] = x;
        }
        return;
    }
    for (int32_t p = sl; p < P; p += kFLanes) {
        double z = 0.0;
#pragma unroll
        for (int m = 0; m < M; ++m) z += acc[m] * (double)Phi[(int64_t)m * P + p];
        out[r * P + p] = (float)z;
    }
}

// Rows of G~ a block makes at a time, and the columns of dZ a row of its threads
// takes (blockIdx.y: which NC kDCols).
constexpr int kDRows = 64;
constexpr int kDCols = 64;
constexpr int kDBlocks = 512;  // partial products: two blocks per CU

// part[x][m, p] = sum over the block's rows r of G~[r, m] dZ[r, p].  Thread
// (column p of kDCols, row group q of 4) sums the rows r = q mod 4 in float64;
// the groups are added in order.  Where there are at most 32 columns a row of
// threads is 32 wide and there are 8 groups.  NC: columns a thread takes, kDCols
// apart.  kMode kSumsGiven: the row sums are read from v [n_rows, M].
template <int M, int kMode, int NC>
__global__ void __launch_bounds__(kFThreads)
    featureless_dphi_kernel(int32_t n_rows, const int32_t *__restrict__ row_ptr,
                            const int32_t *__restrict__ col_idx, int64_t nnz_bound,
                            const float *__restrict__ v, sbc_geometry g,
                            const float *__restrict__ dZ, int32_t P, float *__restrict__ part) {
    __shared__ double G[kDRows][M];  // (float32 values)
    __shared__ double sums[kFThreads];
    const int tid = threadIdx.x, sl = tid % kFLanes;
    const int32_t p0 = blockIdx.y * (NC * kDCols);
    const int width = P - p0 <= 32 ? 32 : 64;
    const int32_t p = p0 + tid % width;
    const int q = tid / width, groups = kFThreads / width;
    double acc[NC][M];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int m = 0; m < M; ++m) acc[c][m] = 0.0;
    for (int64_t r0 = (int64_t)blockIdx.x * kDRows; r0 < n_rows; r0 += (int64_t)gridDim.x * kDRows) {
        if constexpr (kMode == kSumsGiven) {
            for (int x = tid; x < kDRows * M; x += kFThreads)
                (&G[0][0])[x] = r0 + x / M < n_rows ? (double)v[r0 * M + x] : 0.0;
        } else
#pragma unroll 1
        for (int i = tid / kFLanes; i < kDRows; i += kFThreads / kFLanes) {
            double s[M];
            const bool on = r0 + i < n_rows;  // the same for a whole group
            if (on) row_sums<M, kMode>(r0 + i, sl, row_ptr, col_idx, nnz_bound, v, g, s);
            if (sl < M) {
                float x = 0.f;
#pragma unroll
                for (int m = 0; m < M; ++m)
                    if (m == sl) x = on ? (float)s[m] : 0.f;
                G[i][sl] = (double)x;
            }
        }
        __syncthreads();
        if (p < P) {
            const int64_t left = n_rows - r0;
            const int rows = left < kDRows ? (int)left : kDRows;
            // 4 rows' loads in flight (rows past the last: G is 0 there)
            static_assert(kDRows % (4 * 8) == 0, "whole steps");
            for (int i = q; i < rows; i += 4 * groups) {
                float z[4][NC];
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int c = 0; c < NC; ++c)
                        z[u][c] = i + u * groups < rows && p + c * kDCols < P
                                      ? dZ[(r0 + i + u * groups) * P + p + c * kDCols]
                                      : 0.f;
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int c = 0; c < NC; ++c)
#pragma unroll
                        for (int m = 0; m < M; ++m)
                            acc[c][m] += G[i + u * groups][m] * (double)z[u][c];
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int m = 0; m < M; ++m) {
            sums[tid] = acc[c][m];
            __syncthreads();
            if (q == 0 && p + c * kDCols < P) {
                double t = 0.0;
                for (int k = 0; k < groups; ++k) t += sums[k * width + tid];
                part[((int64_t)blockIdx.x * M + m) * P + p + c * kDCols] = (float)t;
            }
            __syncthreads();
        }
}

// dPhi[x] = sum over blocks of part[block][x], in block order within 16 groups
// of consecutive blocks (a thread per position and group), then over the groups.
__global__ void __launch_bounds__(256)
    featureless_reduce_kernel(const float *__restrict__ part, int32_t n_parts, int32_t total,
                              float *__restrict__ dPhi) {
    __shared__ double s[16][16];
    const int g = threadIdx.x / 16, t = threadIdx.x % 16;
    const int32_t x = blockIdx.x * 16 + t;
    const int32_t per = (n_parts + 15) / 16;
    const int32_t b0 = g * per, b1 = b0 + per < n_parts ? b0 + per : n_parts;
    double a = 0.0;
    if (x < total)
        for (int32_t b = b0; b < b1; b += 8) {
            float y[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) y[j] = b + j < b1 ? part[(int64_t)(b + j) * total + x] : 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) a += (double)y[j];
        }
    s[g][t] = a;
    __syncthreads();
    if (g == 0 && x < total) {
        double r = 0.0;
#pragma unroll
        for (int k = 0; k < 16; ++k) r += s[k][t];
        dPhi[x] = (float)r;
    }
}

int32_t dphi_blocks(int32_t n) {
    const int32_t b = (n + kDRows - 1) / kDRows;
    return b < kDBlocks ? b : kDBlocks;
}

// Up to this many columns the blocks make the row sums as they go, for every 64
// columns again; beyond it a pass of its own makes them once, and a thread takes
// two columns.  32768 rows, M 8, 20 entries: 128 columns 26 us by the first way,
// 256 columns 45 and 34 us, 1024 columns 121 and 81.  What is left against a float32
// matrix product of the stored sums (37 and 74 us) are the float64 sums, which
// are kept; four columns a thread took 108 (registers).
constexpr int kSumsColumns = 128;

// f(M, mode) for the basis of a call
template <typename F>
void featureless_dispatch(const float *v, const sbc_geometry *g, int32_t M, F f) {
    using std::integral_constant;
    auto at = [&](auto m, auto mode) { f(m, mode); };
#define SBC_FL(MM, MODE) at(integral_constant<int, MM>{}, integral_constant<int, MODE>{})
    if (v) {
        if (M == 4) SBC_FL(4, 0);
        else if (M == 8) SBC_FL(8, 0);
        else SBC_FL(10, 0);
    } else if (g->basis == SBC_BASIS_EVENT8) {
        SBC_FL(8, 2);
    } else if (g->basis == SBC_BASIS_WMONO10) {
        SBC_FL(10, 3);
    } else if (M == 4) {
        SBC_FL(4, 1);
    } else {
        SBC_FL(8, 1);
    }
#undef SBC_FL
}

sbc_status check_featureless(const sbc_csr *csr, const float *v, const sbc_geometry *g,
                             int32_t M, int32_t P) {
    SBC_TRY(check_csr(csr));
    if (M != 4 && M != 8 && M != 10) return fail(SBC_ERR_UNSUPPORTED, "M must be 4, 8 or 10");
    if (P <= 0) return fail(SBC_ERR_INVALID_ARG, "P must be > 0");
    if (!v) {
        SBC_TRY(check_geometry(g, csr->n_rows, csr->n_cols));
        if (g->basis == SBC_BASIS_EVENT_DECAYS)
            return fail(SBC_ERR_UNSUPPORTED, "the learned-decay basis needs v here");
        if (sbc_basis_size(g->basis) != M)
            return fail(SBC_ERR_INVALID_ARG, "M does not match the geometry's basis");
    }
    return SBC_OK;
}

}  // namespace
}  // namespace sbc

using namespace sbc;

extern "C" size_t sbc_featureless_workspace_size(int32_t n_out, int32_t M, int32_t P) {
    if (n_out < 0 || M <= 0 || P <= 0) return 0;
    return align_up((size_t)dphi_blocks(n_out) * M * P * 4) +
           (P > kSumsColumns ? align_up((size_t)n_out * M * 4) : 0);
}

extern "C" sbc_status sbc_featureless_forward(const sbc_csr *csr, const float *v,
                                              const sbc_geometry *geometry, int32_t M,
                                              const float *Phi, int32_t P, float *Z,
                                              hipStream_t stream) {
    clear_error();
    SBC_TRY(check_featureless(csr, v, geometry, M, P));
    if (csr->n_rows == 0) return SBC_OK;
    if (!Phi || !Z) return fail(SBC_ERR_INVALID_ARG, "Phi or Z is null");
    trace_before("featureless_fwd", stream);
    const sbc_geometry g = geometry ? *geometry : sbc_geometry{};
    featureless_dispatch(v, geometry, M, [&](auto m, auto mode) {
        hipLaunchKernelGGL((featureless_kernel<decltype(m)::value, decltype(mode)::value, true>),
                           dim3(grid_for((int64_t)csr->n_rows * kFLanes, kFThreads)),
                           dim3(kFThreads), 0, stream, csr->n_rows, csr->row_ptr, csr->col_idx,
                           csr->nnz_bound, v, g, Phi, P, Z);
    });
    SBC_LAUNCH_CHECK();
    trace_after("featureless_fwd", stream);
    return SBC_OK;
}

extern "C" sbc_status sbc_featureless_backward(const sbc_csr *csr, const float *v,
                                               const sbc_geometry *geometry, int32_t M,
                                               const float *dZ, int32_t P, float *dPhi,
                                               void *workspace, size_t workspace_bytes,
                                               hipStream_t stream) {
    clear_error();
    SBC_TRY(check_featureless(csr, v, geometry, M, P));
    if (!dPhi) return fail(SBC_ERR_INVALID_ARG, "dPhi is null");
    const int32_t n = csr->n_rows;
    if (n > 0 && !dZ) return fail(SBC_ERR_INVALID_ARG, "dZ is null");
    const size_t need = sbc_featureless_workspace_size(n, M, P);
    if (!workspace || workspace_bytes < need)
        return fail(SBC_ERR_WORKSPACE, "workspace smaller than sbc_featureless_workspace_size()");
    if (n == 0) return fill_i32(reinterpret_cast<int32_t *>(dPhi), 0, (int64_t)M * P, stream);
    float *part = static_cast<float *>(workspace);
    const sbc_geometry g = geometry ? *geometry : sbc_geometry{};
    const int32_t blocks = dphi_blocks(n);
    float *sums = reinterpret_cast<float *>(static_cast<char *>(workspace) +
                                            align_up((size_t)blocks * M * P * 4));
    trace_before("featureless_rowsum", stream);
    featureless_dispatch(v, geometry, M, [&](auto m, auto mode) {
        constexpr int kM = decltype(m)::value, kMode = decltype(mode)::value;
        auto product = [&](auto kernel, int columns, const float *vals) {
            hipLaunchKernelGGL(kernel,
                               dim3((unsigned)blocks, (unsigned)((P + columns - 1) / columns)),
                               dim3(kFThreads), 0, stream, n, csr->row_ptr, csr->col_idx,
                               csr->nnz_bound, vals, g, dZ, P, part);
        };
        if (P <= kSumsColumns) {
            product(featureless_dphi_kernel<kM, kMode, 1>, kDCols, v);
        } else {
            hipLaunchKernelGGL((featureless_kernel<kM, kMode, false>),
                               dim3(grid_for((int64_t)n * kFLanes, kFThreads)), dim3(kFThreads), 0,
                               stream, n, csr->row_ptr, csr->col_idx, csr->nnz_bound, v, g,
                               nullptr, P, sums);
            product(featureless_dphi_kernel<kM, kSumsGiven, 2>, 2 * kDCols, sums);
        }
    });
    SBC_LAUNCH_CHECK();
    trace_after("featureless_rowsum", stream);
    trace_before("featureless_dphi", stream);
    hipLaunchKernelGGL(featureless_reduce_kernel, dim3(grid_for((int64_t)M * P, 16)), dim3(256), 0,
                       stream, part, blocks, M * P, dPhi);
    SBC_LAUNCH_CHECK();
    trace_after("featureless_dphi", stream);
    return SBC_OK;
}
