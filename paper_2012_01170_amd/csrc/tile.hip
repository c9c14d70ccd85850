// Host side of the tile passes (tile.hpp), the fragments of the weights and
// the reduction of the weight gradient's partial sums.
#include "tile.hpp"

#include "common.hpp"
#include "split.hpp"
#include "tile_args.hpp"

namespace sbc {
namespace {

// W [M, Ci, Co] as the contraction's B operand, B[m, c, n] = W[m, c, n] or
// (transposed) W[m, n, c], in the order the waves load it: per slice of 32
// channels c, basis function and part, per block of 16 columns, lane by lane,
// 8 consecutive channels each; zero past C and N.  A thread makes one lane's 8.
template <typename WT, int NB>
__global__ void __launch_bounds__(256)
    tile_frag_kernel(const WT *__restrict__ W, int32_t M, int32_t Ci, int32_t Co, bool transposed,
                     int32_t slices, uint16_t *__restrict__ frag) {
    const int32_t C = transposed ? Co : Ci, N = transposed ? Ci : Co;
    const int32_t ncb = (N + 15) / 16;
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= (int64_t)slices * M * ncb * 64) return;
    const int lane = (int)(x % 64);
    const int32_t cb = (int32_t)(x / 64 % ncb);
    const int64_t sk = x / 64 / ncb;  // slice * M + m
    const int32_t s = (int32_t)(sk / M), m = (int32_t)(sk % M);
    const int32_t n = 16 * cb + (lane & 15);
    float f[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int32_t c = s * kTileCS + 8 * (lane >> 4) + j;
        f[j] = 0.f;
        if (c < C && n < N) {
            const int64_t at = transposed ? ((int64_t)m * Ci + n) * Co + c
                                          : ((int64_t)m * Ci + c) * Co + n;
            if constexpr (sizeof(WT) == 2) f[j] = __uint_as_float((uint32_t)W[at] << 16);
            else f[j] = quiet(W[at]);
        }
    }
    uint32_t w[3][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) split2(f[2 * j], f[2 * j + 1], w[0][j], w[1][j], w[2][j]);
#pragma unroll
    for (int q = 0; q < NB; ++q)
        *reinterpret_cast<uint4 *>(frag + (((sk * NB + q) * ncb + cb) * 64 + lane) * 8) =
            make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]);
}

// dW[m, c, p] = sum over splits of part[split][c_P][m][c_Q].  A block of 256
// threads owns 64 consecutive positions; 16 groups of 16 threads (four
// positions each) sum a contiguous range of splits in order, then the groups
// are added in order.
__global__ void __launch_bounds__(256)
    tile_dw_reduce_kernel(const float *__restrict__ part, int32_t n_parts, int32_t M, int32_t CP,
                          int32_t CQ, bool p_is_in, float *__restrict__ dW) {
    __shared__ float sums[16][64];
    const int64_t total = (int64_t)CP * M * CQ;
    const int g = threadIdx.x / 16, tq = threadIdx.x % 16;
    const int64_t off = (int64_t)blockIdx.x * 64 + 4 * tq;
    const int32_t per = (n_parts + 15) / 16;
    const int32_t b0 = g * per, b1 = b0 + per < n_parts ? b0 + per : n_parts;
    float s[4] = {0.f, 0.f, 0.f, 0.f};
    if (total % 4 == 0) {
        if (off < total)
            for (int32_t b = b0; b < b1; b += 8) {
                float4 v[8];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    v[j] = b + j < b1 ? *reinterpret_cast<const float4 *>(
                                            part + (int64_t)(b + j) * total + off)
                                      : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    s[0] += v[j].x;
                    s[1] += v[j].y;
                    s[2] += v[j].z;
                    s[3] += v[j].w;
                }
            }
    } else {
        for (int32_t b = b0; b < b1; ++b)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (off + k < total) s[k] += part[(int64_t)b * total + off + k];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) sums[g][4 * tq + k] = s[k];
    __syncthreads();
    if (threadIdx.x >= 64) return;
    const int64_t x = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (x >= total) return;
    float t = 0.f;
#pragma unroll
    for (int q = 0; q < 16; ++q) t += sums[q][threadIdx.x];
    const int32_t q = (int32_t)(x % CQ);
    const int32_t m = (int32_t)(x / CQ % M), c = (int32_t)(x / CQ / M);
    if (p_is_in) dW[((int64_t)m * CP + c) * CQ + q] = t;
    else dW[((int64_t)m * CQ + q) * CP + c] = t;
}

// Whether tiles of 64 rows are taken where the rows are short (half the weight
// bytes per row): the tiles then still give two blocks per CU, and a wave's sums
// of 64 rows leave registers for the products (not for M > 10, nor for M = 10
// with more than 64 columns).
bool contract_tall(int32_t M, int32_t n_rows, int32_t N) {
    if (M > 10 || (M == 10 && N > 64)) return false;
    const int32_t chunks = (N + 127) / 128;
    return ((int64_t)n_rows + 63) / 64 * chunks >= 512;
}

}  // namespace

bool tile_available(int32_t M, int32_t C_in, int32_t C_out) {
    return (M == 4 || M == 8 || M == 10 || M == 16 || M == 24 || M == 32) && C_in >= 8 &&
           C_out >= 8 && C_in <= 512 && C_out <= 512;
}

size_t tile_frag_bytes(int32_t M, int32_t C, int32_t N, bool bf16) {
    // (slices of 32 channels, blocks of 16 columns)
    return (size_t)((C + kTileCS - 1) / kTileCS * kTileCS) * M * ((N + 15) / 16 * 16) * 2 * (bf16 ? 1 : 3);
}

sbc_status tile_contract(const TilePattern &p, const float *v, const KGeo &g, int mode, int32_t M,
                         const void *X, const void *W, bool w_transposed, bool bf16, int32_t C,
                         int32_t N, float *out, void *frag, hipStream_t stream,
                         const char *trace) {
    if (p.n_rows <= 0) return SBC_OK;
    const int32_t slices = (C + kTileCS - 1) / kTileCS;
    const int32_t Ci = w_transposed ? N : C, Co = w_transposed ? C : N;
    const int64_t lanes = (int64_t)slices * M * ((N + 15) / 16) * 64;
    uint16_t *fr = static_cast<uint16_t *>(frag);
    trace_before(trace, stream);
    if (bf16)
        hipLaunchKernelGGL((tile_frag_kernel<uint16_t, 1>), dim3(grid_for(lanes, 256)), dim3(256),
                           0, stream, static_cast<const uint16_t *>(W), M, Ci, Co, w_transposed,
                           slices, fr);
    else
        hipLaunchKernelGGL((tile_frag_kernel<float, 3>), dim3(grid_for(lanes, 256)), dim3(256), 0,
                           stream, static_cast<const float *>(W), M, Ci, Co, w_transposed, slices,
                           fr);
    SBC_LAUNCH_CHECK();
    const TileContractArgs a{p, v, g, mode, X, C, fr, N, out,
                             contract_tall(M, p.n_rows, N)};
    SBC_TRY(M <= 10 ? launch_contract_4_8_10(M, bf16, a, stream)
                    : launch_contract_16_24_32(M, bf16, a, stream));
    trace_after(trace, stream);
    return SBC_OK;
}

size_t tile_dw_bytes(int32_t n_rows, int32_t M, int32_t C_P, int32_t C_Q) {
    return (size_t)dw_splits(n_rows, M, C_P, C_Q) * C_P * M * C_Q * sizeof(float);
}

sbc_status tile_weight_gradient(const TilePattern &p, const float *v, const KGeo &g, int mode,
                                int32_t M, const void *P, const void *Q, bool bf16, int32_t C_in,
                                int32_t C_out, float *dW, void *part, hipStream_t stream,
                                const char *trace) {
    const int32_t CP = p.transposed ? C_in : C_out, CQ = p.transposed ? C_out : C_in;
    const int32_t S = p.n_rows > 0 ? dw_splits(p.n_rows, M, CP, CQ) : 0;
    float *pt = static_cast<float *>(part);
    trace_before(trace, stream);
    if (S > 0) SBC_TRY(launch_dw(M, bf16, TileDwArgs{p, v, g, mode, P, CP, Q, CQ, pt, S}, stream));
    const int64_t total = (int64_t)CP * M * CQ;
    hipLaunchKernelGGL(tile_dw_reduce_kernel, dim3(grid_for(total, 64)), dim3(256), 0, stream, pt,
                       S, M, CP, CQ, p.transposed, dW);
    SBC_LAUNCH_CHECK();
    trace_after(trace, stream);
    return SBC_OK;
}

}  // namespace sbc
