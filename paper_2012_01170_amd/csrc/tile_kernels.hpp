// Device code of the tile passes (tile.hpp), for any channel counts.
//
// Both passes gather a tile of rows of G = [N^(m) X]_m, one slice of CS
// channels for all M basis functions at a time, split the float32 sums into
// their bf16 parts (split.hpp) in LDS, and contract the slice on the bf16
// matrix cores, so G never reaches memory and any channel count is a number
// of slices:
//   tile_contract_kernel   out tile += G slice x B slice over the slices (the
//                          forward, and the input gradient on the transposed
//                          pattern);
//   tile_dw_kernel         a block keeps P^T G of one slice in registers over
//                          its tiles (the weight gradient).
// Measured against the separate kernels they replace (gather to memory,
// float32 contraction): 64 ragged clouds of up to 256 points, 16 entries a
// row, M 8, 128 -> 128 channels, forward 115 -> 57 us, both gradients 186 ->
// 145 us; 128 clouds of 1024, weighted M 10, 64 -> 64, forward 237 -> 134 us,
// both gradients 490 -> 322 us.  They do not serve all sizes better: which do is
// estimated (route_cost.hpp).  Errors against float64 fall from 5e-7 to 2e-7
// (the split products, split.hpp).
#pragma once

#include <type_traits>

#include "common.hpp"
#include "edge_basis.hpp"
#include "split.hpp"
#include "tile.hpp"

namespace sbc {

__device__ __forceinline__ void tile_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
}

// What the stage holds of an entry, beside its other end:
//   kValues   its M basis values;
//   kCompact  point bases of M = 8 and 10: u = (x'_i - x_j) / r and the weight;
//   kEvents   event bases: the offset index and the M / 8 decays (or their
//             derivatives) of that offset, the only values that are not zero.
// The shorter forms leave room for all entries of a wave's rows, which are then
// staged once for all slices.
enum StageKind { kValues = 0, kCompact = 1, kEvents = 2 };

// Stage kind of a basis mode.
__host__ __device__ constexpr StageKind stage_kind(int32_t M, int mode) {
    return mode == SBC_BASIS_MONO8 + 1 || mode == SBC_BASIS_WMONO10 + 1 ? kCompact
           : mode == 0 || M == 4                                        ? kValues
                                                                        : kEvents;
}

// words of a staged entry
template <int M, StageKind kKind>
constexpr int stage_words() {
    return kKind == kCompact ? 4 : kKind == kEvents ? 1 + M / 8 : M;
}

// Offset index (8: none, a same-pixel edge) and decays of an event edge, in the
// expressions of the basis values kernel.
template <int M>
__device__ __forceinline__ void event_entry(int mode, const KGeo &g, int32_t i, int32_t j,
                                            float *out) {
    constexpr int Mv = M / 8;
    const int4 a = g.ev[i], b = g.ev[j];
    const int k = event_index(a.x - b.x, a.y - b.y);
    out[0] = __int_as_float(k >= 0 ? k : 8);
    if constexpr (Mv == 1) {
        out[1] = event_decay(a.z, b.z, g.inv_tau);
    } else {
        const float dt = (float)((int64_t)a.z - (int64_t)b.z);
#pragma unroll
        for (int q = 0; q < Mv; ++q) {
            const float x = expf(-g.decays[(k >= 0 ? k : 0) * Mv + q] * dt);
            out[1 + q] = mode == kDecayDerivMode ? -dt * x : x;
        }
    }
}

// u and the weight of an edge of a point basis, each float64 rounded once.  The
// monomials are formed from them in float32 where they are used (values()), so a
// value w x y has up to five roundings, of its three factors and two products,
// where sbc_basis_eval and the separate kernels form it in float64 and round
// once (basis.hpp): 5 * 2^-24 against 2^-24 of it, and not the same bits.  The
// differences and 1 - |u|^2, where float32 would cancel, are float64 on both.
// The results are nearer to float64 than the separate kernels' all the same,
// whose float32 sums of M C products lose more (5e-7 against 2e-7 in the header).
// Weight: (1 - |u|^2)^2 (M = 8), (1 - |u|) / W_i (M = 10; 0 where W_i = 0).
template <int M>
__device__ __forceinline__ float4 compact_entry(const KGeo &g, int32_t i, int32_t j) {
    const float *q = g.x_out + 3 * (int64_t)i, *s = g.x_in + 3 * (int64_t)j;
    const float qx = q[0], qy = q[1], qz = q[2], px = s[0], py = s[1], pz = s[2];
    const double ux = ((double)qx - (double)px) * g.inv_r;
    const double uy = ((double)qy - (double)py) * g.inv_r;
    const double uz = ((double)qz - (double)pz) * g.inv_r;
    double w;
    if constexpr (M == 10) {
        const double W = g.wsum[i];
        w = W != 0.0 ? point_weight(qx, qy, qz, px, py, pz, g.inv_r) / W : 0.0;
    } else {
        const double a = 1.0 - (ux * ux + uy * uy + uz * uz);
        w = a * a;
    }
    return make_float4((float)ux, (float)uy, (float)uz, (float)w);
}

// row0 + up, at most n_rows (the sum may pass 2^31)
__host__ __device__ constexpr int32_t row_at(int32_t row0, int32_t up, int32_t n_rows) {
    return row0 < n_rows - up ? row0 + up : n_rows;
}

// Entries a wave stages at once (entry SW weighs nothing: the slots past a
// row's end read it).  Compact entries move as 16 bytes, so a stage (one per
// wave, in an array) starts and ends on 16 bytes.
template <int M, int SW, StageKind kKind>
struct alignas(16) TileStage {
    static constexpr int NV = stage_words<M, kKind>();
    float v[SW + 1][NV];
    int32_t nb[SW + 1];
};

// The gather of one wave's RPW consecutive rows, 32 channels (a slice) at a
// time: LPR lanes a row, NL loads of VEC channels a lane and entry.  What
// bounds it is the cache lines a CU can wait for at once (about 10 TB/s over
// the chip with lines of 128 bytes used whole, half of that with 64-byte
// pieces of them), so an entry's float32 slice is one whole line.  The
// products run on the matrix cores as 16 independent 4 x 4 outer products (an
// entry's 4 basis functions x 4 lanes' channels; float32): as plain FMAs, M
// per channel and entry, they kept the vector ALU busy longer than the loads.
template <int M, bool kXbf, StageKind kKind, int RPW, int SW, int U_>
struct TileGather {
    static constexpr int LPR = 64 / RPW;
    static_assert(LPR == 4 || LPR == 8, "a row is 4 or 8 lanes");
    static constexpr int VEC = kXbf && LPR == 4 ? 8 : 4;
    static constexpr int CS = 32;
    static constexpr int NL = CS / (LPR * VEC);
    static constexpr int VT = NL * VEC;      // channels per lane
    static constexpr int U = U_;             // entries of a row loaded together
    static constexpr int MG = (M + 3) / 4;   // groups of 4 basis functions
    using Stage = TileStage<M, SW, kKind>;
    // sums of basis function 4 g + r and the lane's channel k: [g][k][r]
    using Acc = floatx4[MG][VT];
    using Raw = typename std::conditional<
        kXbf, typename std::conditional<VEC == 8, uint4, uint2>::type, float4>::type;

    const TilePattern &p;
    const float *v;
    const KGeo &g;
    int mode;
    const void *X;
    int32_t C;
    bool vec;  // rows of X start on a load's bytes
    Stage &st;
    int lane, rl, piece;
    int32_t row_begin, wb, we, lo, hi;
    int32_t bound;  // lane l <= RPW: first entry of row row_begin + l
    bool staged;    // the whole wave's entries are in the stage

    __device__ __forceinline__ TileGather(const TilePattern &p_, const float *v_, const KGeo &g_,
                                          int mode_, const void *X_, int32_t C_, Stage &st_)
        : p(p_), v(v_), g(g_), mode(mode_), X(X_), C(C_),
          vec(C_ % VEC == 0 && (reinterpret_cast<uintptr_t>(X_) & (sizeof(Raw) - 1)) == 0), st(st_) {
        lane = threadIdx.x & 63;
        rl = lane / LPR;
        piece = lane % LPR;
        if (lane < Stage::NV) st.v[SW][lane] = kKind == kEvents && lane == 0 ? __int_as_float(8) : 0.f;
    }

    // row bounds of the wave's rows (clamped into [0, nnz])
    __device__ __forceinline__ void begin(int32_t row0) {
        row_begin = row0;
        const int32_t b = p.ptr[row_at(row0, lane < RPW ? lane : RPW, p.n_rows)];
        bound = b < 0 ? 0 : (b < g.nnz ? b : g.nnz);
        wb = __builtin_amdgcn_readlane(bound, 0);
        we = __builtin_amdgcn_readlane(bound, RPW);
        lo = __shfl(bound, rl, 64);
        hi = __shfl(bound, rl + 1, 64);
        // (a malformed pattern's bounds need not ascend: stay inside the wave's)
        lo = lo > wb ? lo : wb;
        hi = hi < we ? hi : we;
        staged = false;
    }

    // entries [c0, min(we, c0 + SW)) into the stage
    __device__ __forceinline__ void stage(int32_t c0) {
        const int32_t end = we < c0 + SW ? we : c0 + SW;
        tile_wave_sync();  // the previous entries are read
#pragma unroll 1
        for (int32_t e0 = c0; e0 < end; e0 += 64) {
            const int32_t e = e0 + lane;
            if (e < end) {
                const int32_t other = p.idx[e];
                int s = 0;
#pragma unroll
                for (int q = 1; q < RPW; ++q) s += __builtin_amdgcn_readlane(bound, q) <= e ? 1 : 0;
                // (a malformed pattern's row stays inside the rows)
                const int32_t row = row_begin + s < p.n_rows ? row_begin + s : p.n_rows - 1;
                const int32_t i = p.transposed ? other : row, j = p.transposed ? row : other;
                st.nb[e - c0] = other;
                // (slots without an entry read a row the wave reads anyway: one
                // row for all waves made its cache line the bottleneck)
                if (e == c0) st.nb[SW] = other;
                if constexpr (kKind == kCompact) {
                    *reinterpret_cast<float4 *>(st.v[e - c0]) = compact_entry<M>(g, i, j);
                } else {
                    float b[Stage::NV];
                    if constexpr (kKind == kEvents) {
                        event_entry<M>(mode, g, i, j, b);
                    } else if (mode == 0) {
                        edge_basis<M, 0>(g, v, i, j, p.perm ? (int64_t)p.perm[e] : (int64_t)e,
                                         g.inv_r, g.inv_tau, b);
                    } else if constexpr (M == 4) {
                        edge_basis<M, SBC_BASIS_MONO4 + 1>(g, v, i, j, 0, g.inv_r, g.inv_tau, b);
                    }
#pragma unroll
                    for (int m = 0; m < Stage::NV; ++m) st.v[e - c0][m] = b[m];
                }
            }
        }
        tile_wave_sync();
    }

    // this lane's basis functions (4 g + lane % 4) of a staged entry
    __device__ __forceinline__ void values(int32_t at, float (&w)[MG]) const {
        const int t = lane & 3;
        if constexpr (kKind == kValues) {
#pragma unroll
            for (int q = 0; q < MG; ++q) {
                if constexpr (M % 4 == 0) w[q] = st.v[at][4 * q + t];
                else w[q] = 4 * q + t < M ? st.v[at][4 * q + t < M ? 4 * q + t : 0] : 0.f;
            }
        } else if constexpr (kKind == kEvents) {
            constexpr int Mv = M / 8;
            const int k = __float_as_int(st.v[at][0]);
            if constexpr (4 % Mv == 0) {  // the lane's decay is the same in every group
                const float d = st.v[at][1 + t % Mv];
#pragma unroll
                for (int q = 0; q < MG; ++q) w[q] = (4 * q + t) / Mv == k ? d : 0.f;
            } else {
                float d[Mv];
#pragma unroll
                for (int q = 0; q < Mv; ++q) d[q] = st.v[at][1 + q];
#pragma unroll
                for (int q = 0; q < MG; ++q) {
                    const int m = 4 * q + t, r = m % Mv;
                    float x = d[0];
#pragma unroll
                    for (int z = 1; z < Mv; ++z) x = r == z ? d[z] : x;
                    w[q] = m / Mv == k ? x : 0.f;
                }
            }
        } else {
            const float4 e = *reinterpret_cast<const float4 *>(st.v[at]);
            // [1, x, y, z], [xx, yy, zz, xy] and for M = 10 [xz, yz, 0, 0],
            // times the weight
            const float f = t == 0 ? 1.f : t == 1 ? e.x : t == 2 ? e.y : e.z;
            const float a = t == 1 ? e.y : t == 2 ? e.z : e.x;
            const float b = t == 0 ? e.x : t == 2 ? e.z : e.y;
            const float as = a * e.w;
            w[0] = f * e.w;
            w[1] = as * b;
            if constexpr (MG == 3) w[2] = t < 2 ? as * e.z : 0.f;
        }
    }

    // the lane's channel k of slice `slice`: NL pieces of VEC, LPR VEC apart
    __device__ __forceinline__ int32_t channel(int32_t slice, int k) const {
        return slice * CS + k / VEC * (LPR * VEC) + piece * VEC + k % VEC;
    }

    // channels c .. c + VEC - 1 of row j (channels past C read channel C - 1,
    // or the row's first)
    template <bool kVec>
    __device__ __forceinline__ Raw load(int32_t j, int32_t c) const {
        if constexpr (kVec) {
            const int32_t cc = c < C ? c : 0;
            if constexpr (kXbf)
                return *reinterpret_cast<const Raw *>(static_cast<const uint16_t *>(X) +
                                                      (int64_t)j * C + cc);
            else
                return *reinterpret_cast<const Raw *>(static_cast<const float *>(X) +
                                                      (int64_t)j * C + cc);
        } else if constexpr (kXbf) {
            const uint16_t *r = static_cast<const uint16_t *>(X) + (int64_t)j * C;
            uint32_t w[VEC / 2];
#pragma unroll
            for (int k = 0; k < VEC / 2; ++k) {
                const int32_t a = c + 2 * k < C ? c + 2 * k : C - 1;
                const int32_t b = c + 2 * k + 1 < C ? c + 2 * k + 1 : C - 1;
                w[k] = (uint32_t)r[a] | ((uint32_t)r[b] << 16);
            }
            if constexpr (VEC == 8) return make_uint4(w[0], w[1], w[2], w[3]);
            else return make_uint2(w[0], w[1]);
        } else {
            const float *r = static_cast<const float *>(X) + (int64_t)j * C;
            float f[VEC];
#pragma unroll
            for (int k = 0; k < VEC; ++k) f[k] = r[c + k < C ? c + k : C - 1];
            return make_float4(f[0], f[1], f[2], f[3]);
        }
    }

    // a loaded piece as float32 (0 where the slot holds no entry)
    static __device__ __forceinline__ void unpack(const Raw &r, bool on, float *f) {
        if constexpr (kXbf) {
            uint32_t w[VEC / 2];
            w[0] = r.x;
            w[1] = r.y;
            if constexpr (VEC == 8) {
                w[2] = r.z;
                w[3] = r.w;
            }
#pragma unroll
            for (int k = 0; k < VEC / 2; ++k) {
                const uint32_t x = on ? w[k] : 0u;
                f[2 * k] = __uint_as_float(x << 16);
                f[2 * k + 1] = __uint_as_float(x & 0xFFFF0000u);
            }
        } else {
            f[0] = on ? r.x : 0.f;
            f[1] = on ? r.y : 0.f;
            f[2] = on ? r.z : 0.f;
            f[3] = on ? r.w : 0.f;
        }
    }

    // acc = the lane's sums of slice `slice` (entries in pattern order)
    __device__ __forceinline__ void slice_sums(int32_t slice, Acc &acc) {
#pragma unroll
        for (int q = 0; q < MG; ++q)
#pragma unroll
            for (int k = 0; k < VT; ++k) acc[q][k] = floatx4{0.f, 0.f, 0.f, 0.f};
        // (two loops: with the choice inside, its two kinds of load were merged
        // into single words)
        if (vec) add_entries<true>(slice, acc);
        else add_entries<false>(slice, acc);
        // channels past C weigh nothing whatever was read for them
#pragma unroll
        for (int k = 0; k < VT; ++k)
            if (channel(slice, k) >= C) {
#pragma unroll
                for (int q = 0; q < MG; ++q) acc[q][k] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
    }

    // Groups of U entries per row: the rows of X of the next group are loaded
    // while this group is summed.
    template <bool kVec>
    __device__ __forceinline__ void add_entries(int32_t slice, Acc &acc) {
#pragma unroll 1
        for (int32_t c0 = wb; c0 < we; c0 += SW) {
            if (!staged) {
                stage(c0);
                staged = we - wb <= SW;
            }
            int32_t e = (lo > c0 ? lo : c0) - c0;
            const int32_t end = (hi < c0 + SW ? hi : c0 + SW) - c0;
            // the most entries any row still has (wave-uniform)
            int32_t left = end - e;
#pragma unroll
            for (int d = LPR; d < 64; d <<= 1) {
                const int32_t o = __shfl_xor(left, d, 64);
                left = o > left ? o : left;
            }
            left = __builtin_amdgcn_readfirstlane(left);
            if (left <= 0) continue;
            struct Group {
                Raw f[U][NL];
            };
            auto fetch = [&](int32_t e1, Group &q) {
                int32_t j[U];
#pragma unroll
                for (int u = 0; u < U; ++u) j[u] = st.nb[e1 + u < end ? e1 + u : SW];
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int l = 0; l < NL; ++l)
                        q.f[u][l] = load<kVec>(j[u], channel(slice, l * VEC));
            };
            Group q;
            fetch(e, q);
#pragma unroll 1
            for (;;) {
                Group n;
                if (left > U) fetch(e + U, n);
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (u < left) {
                        const bool on = e + u < end;
                        float x[VT], w[MG];
                        values(on ? e + u : SW, w);
#pragma unroll
                        for (int l = 0; l < NL; ++l) unpack(q.f[u][l], on, x + l * VEC);
#pragma unroll
                        for (int m = 0; m < MG; ++m)
#pragma unroll
                            for (int k = 0; k < VT; ++k)
                                acc[m][k] = __builtin_amdgcn_mfma_f32_4x4x1f32(w[m], x[k],
                                                                               acc[m][k], 0, 0, 0);
                    }
                left -= U;
                if (left <= 0) break;
                q = n;
                e += U;
            }
        }
    }

    // the split parts of the lane's sums of basis functions 4 g .. 4 g + 3 into
    // the planes [3][rows][S], column 32 (m - 4 g) + channel of the slice
    template <int S, int ROWS>
    __device__ __forceinline__ void store(uint16_t (*planes)[ROWS][S], int local_row,
                                          const Acc &acc, int g_) const {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (4 * g_ + r < M) {
#pragma unroll
                for (int l = 0; l < NL; ++l) {
                    uint32_t w[3][VEC / 2];
#pragma unroll
                    for (int k = 0; k < VEC / 2; ++k)
                        split2(acc[g_][l * VEC + 2 * k][r], acc[g_][l * VEC + 2 * k + 1][r],
                               w[0][k], w[1][k], w[2][k]);
#pragma unroll
                    for (int t = 0; t < 3; ++t) {
                        uint16_t *o = &planes[t][local_row][32 * r + l * (LPR * VEC) + piece * VEC];
                        if constexpr (VEC == 8)
                            *reinterpret_cast<uint4 *>(o) =
                                make_uint4(w[t][0], w[t][1], w[t][2], w[t][3]);
                        else
                            *reinterpret_cast<uint2 *>(o) = make_uint2(w[t][0], w[t][1]);
                    }
                }
            }
    }
};

// Logical tile of block b of n: consecutive blocks go to the 8 XCDs in turn,
// so each XCD gets one contiguous range of tiles (rows near each other gather
// from the same neighbourhood, which then sits in one L2).
__device__ __forceinline__ int32_t tile_of_block(int32_t b, int32_t n) {
    const int32_t per = n / 8, rem = n % 8;
    const int32_t x = b % 8, l = b / 8;
    return x < rem ? x * (per + 1) + l : rem * (per + 1) + (x - rem) * per + l;
}

constexpr int kTileThreads = 256;
constexpr int kTileWaves = 4;

// Stage entries per wave that `bytes` of LDS hold (at most 384).
template <int M, StageKind kKind>
constexpr int stage_entries(int bytes) {
    const int n = (bytes / (kTileWaves * 4 * (stage_words<M, kKind>() + 1)) - 1) / 32 * 32;
    return n > 384 ? 384 : n;
}

// Entries of a row loaded together: what a wave's registers leave (256 with two
// blocks a CU) beside its sums and `kept` accumulators.
template <int M, bool kXbf, int RPW, int kept>
constexpr int tile_u() {
    const int vt = RPW == 16 ? 8 : 4;
    const int per = (kXbf ? vt / 2 : vt) * 2;  // registers per entry, two groups
    const int left = 168 - (M + 3) / 4 * 4 * vt - kept;
    const int u = left / per;
    return u < 2 ? 2 : u > 8 ? 8 : u;
}
template <int M, bool kXbf, int RPW, int kept>
constexpr int kTileU = tile_u<M, kXbf, RPW, kept>();

// Tiles of TR rows of the contraction.  Four basis functions' 32 channels are
// in LDS at a time (128 columns, TR x 816 bytes for the three parts); the
// stage fills what two blocks a CU leave.
template <int M, int TR, StageKind kKind>
struct TileShape {
    static constexpr int RPW = TR / kTileWaves;
    static constexpr int S = 128 + 8;  // 4 mod 64 dwords: 16 rows' b128 reads on distinct banks
    static constexpr int SW = stage_entries<M, kKind>(81920 - 3 * TR * S * 2);
    static_assert(SW >= 64, "a stage of at least 64 entries");
};

// LDS of a tile: the planes of four basis functions' columns, then the stages.
template <int M, bool kXbf, StageKind kKind, int TR, int NCBW, int WCB>
struct ContractTile {
    using T = TileShape<M, TR, kKind>;
    static constexpr int WRB = TR / 16 / (kTileWaves / NCBW);
    // entries loaded together: as many as the accumulators leave registers for
    static constexpr int U = kTileU<M, kXbf, TR / kTileWaves, WRB * WCB * 4>;
    using Gather = TileGather<M, kXbf, kKind, T::RPW, T::SW, U>;
    static constexpr int plane_bytes = 3 * TR * T::S * 2;
    static constexpr int bytes = plane_bytes + kTileWaves * (int)sizeof(typename Gather::Stage);
    static_assert(plane_bytes % 16 == 0 && bytes <= 81920, "aligned stages, two blocks a CU");
};

// out tile [TR, 16 NCBW WCB] of columns from blockIdx.y's chunk.  Waves:
// NCBW column groups x 4 / NCBW row groups, each WCB column blocks (16 NCBW
// columns apart) and WRB row blocks.  B comes as fragments (tile_frag_kernel)
// straight from L2, 6 M C N bytes for every TR rows.  The second block of the
// CU covers this one's gather.
template <int M, bool kXbf, StageKind kKind, int TR, int NCBW, int WCB>
__device__ __forceinline__ void contract_tile(char *lds, int32_t row0, const TilePattern &p,
                                              const float *__restrict__ v, const KGeo &g, int mode,
                                              const void *__restrict__ X, int32_t C,
                                              const uint16_t *__restrict__ frag, int32_t N,
                                              float *__restrict__ out) {
    using CT = ContractTile<M, kXbf, kKind, TR, NCBW, WCB>;
    using T = typename CT::T;
    using Gather = typename CT::Gather;
    constexpr int NRG = kTileWaves / NCBW;
    constexpr int WRB = CT::WRB;
    constexpr int NB = kXbf ? 1 : 3;
    auto planes = reinterpret_cast<uint16_t(*)[TR][T::S]>(lds);
    auto stage = reinterpret_cast<typename Gather::Stage *>(lds + CT::plane_bytes);

    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int lr = lane >> 4, lc = lane & 15;
    const int wc = w % NCBW, wr = w / NCBW;
    const int32_t ncb = (N + 15) / 16;
    const int32_t cb0 = blockIdx.y * NCBW * WCB;
    const int32_t slices = (C + Gather::CS - 1) / Gather::CS;

    Gather G(p, v, g, mode, X, C, stage[w]);
    G.begin(row0 + w * T::RPW);

    floatx4 sum[WRB][WCB];
#pragma unroll
    for (int u = 0; u < WRB; ++u)
#pragma unroll
        for (int t = 0; t < WCB; ++t) sum[u][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    int32_t cb[WCB];
#pragma unroll
    for (int t = 0; t < WCB; ++t) {
        const int32_t c = cb0 + wc + NCBW * t;
        cb[t] = c < ncb ? c : ncb - 1;  // a column block past N: computed, not stored
    }

#pragma unroll 1
    for (int32_t s = 0; s < slices; ++s) {
        typename Gather::Acc acc;
        G.slice_sums(s, acc);
        // k-step m: basis function m's 32 channels
        auto load_b = [&](int m, bf16x8 (&bb)[WCB][NB]) {
            const uint16_t *f = frag + ((int64_t)(s * M + m) * NB) * ncb * 512 + lane * 8;
#pragma unroll
            for (int t = 0; t < WCB; ++t)
#pragma unroll
                for (int q = 0; q < NB; ++q)
                    bb[t][q] = *reinterpret_cast<const bf16x8 *>(f + ((int64_t)q * ncb + cb[t]) * 512);
        };
        bf16x8 b[2][WCB][NB];
        load_b(0, b[0]);
        // the slice's small products (added once, so they live only here)
        floatx4 lo[WRB][WCB];
#pragma unroll
        for (int u = 0; u < WRB; ++u)
#pragma unroll
            for (int t = 0; t < WCB; ++t) lo[u][t] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int mg = 0; mg < Gather::MG; ++mg) {
            __syncthreads();  // the previous columns are multiplied
            G.template store<T::S, TR>(planes, w * T::RPW + G.rl, acc, mg);
            __syncthreads();
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = 4 * mg + r;
                if (m < M) {
                    if (m + 1 < M) load_b(m + 1, b[(m + 1) & 1]);
#pragma unroll
                    for (int u = 0; u < WRB; ++u) {
                        bf16x8 a[3];
#pragma unroll
                        for (int q = 0; q < 3; ++q)
                            a[q] = *reinterpret_cast<const bf16x8 *>(
                                &planes[q][16 * (wr + NRG * u) + lc][32 * r + 8 * lr]);
#pragma unroll
                        for (int t = 0; t < WCB; ++t)
                            mma_split<3, NB>(a, b[m & 1][t], sum[u][t], lo[u][t]);
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < WRB; ++u)
#pragma unroll
            for (int t = 0; t < WCB; ++t) sum[u][t] = finish(sum[u][t], lo[u][t]);
    }
#pragma unroll
    for (int u = 0; u < WRB; ++u)
#pragma unroll
        for (int t = 0; t < WCB; ++t) {
            const int32_t col = 16 * (cb0 + wc + NCBW * t) + lc;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int32_t row = row0 + 16 * (wr + NRG * u) + 4 * lr + r;
                if (row < p.n_rows && col < N) out[(int64_t)row * N + col] = sum[u][t][r];
            }
        }
}

// Most entries a row, in the mean, for which tiles of 64 rows are taken: they
// halve the weights' bytes per row, but a wave then gathers 16 rows by pieces of
// 64 bytes, where 8 rows take whole lines of 128.  128 clouds of 1024, 64 -> 64,
// 64 rows against 32: M 8, 5 entries a row 99 and 127 us, 16: 187 and 182, 45:
// 526 and 429; values given, 16: 226 and 174.  Three parts of the weights for
// more than 64 columns weigh more (16 entries: 218 and 218).  Event entries are
// shorter to gather, and their rows' lengths differ more: 64 rows throughout
// (300k events, 14 entries: 305 and 309; 64 -> 128, 373 and 450).
template <bool kXbf, int COLS>
constexpr int kTallEntries = !kXbf && COLS > 64 ? 16 : 10;
template <StageKind kKind>
constexpr bool kAlwaysTall = kKind == kEvents;

// kTall: tiles of 64 rows, or where there is a choice the pattern's own entry
// count (the host knows a bound alone) decides between 64 and 32 rows; the grid
// is that of 32 then, and the blocks past the last tile of 64 end at once.
template <int M, bool kXbf, StageKind kKind, bool kTall, int NCBW, int WCB>
__global__ void __launch_bounds__(kTileThreads, 2)
    tile_contract_kernel(TilePattern p, const float *__restrict__ v, KGeo g, int mode,
                         const void *__restrict__ X, int32_t C,
                         const uint16_t *__restrict__ frag, int32_t N, float *__restrict__ out) {
    using Low = ContractTile<M, kXbf, kKind, 32, NCBW, WCB>;
    if constexpr (kTall && kAlwaysTall<kKind>) {
        __shared__ __attribute__((aligned(16))) char
            lds[ContractTile<M, kXbf, kKind, 64, NCBW, WCB>::bytes];
        contract_tile<M, kXbf, kKind, 64, NCBW, WCB>(lds, tile_of_block(blockIdx.x, gridDim.x) * 64,
                                                     p, v, g, mode, X, C, frag, N, out);
    } else if constexpr (kTall) {
        using Tall = ContractTile<M, kXbf, kKind, 64, NCBW, WCB>;
        __shared__ __attribute__((aligned(16))) char
            lds[Tall::bytes > Low::bytes ? Tall::bytes : Low::bytes];
        const int64_t entries = p.ptr[p.n_rows];
        if (entries <= (int64_t)kTallEntries<kXbf, 16 * NCBW * WCB> * p.n_rows) {
            const int32_t tiles = p.n_rows / 64 + (p.n_rows % 64 != 0);
            if ((int32_t)blockIdx.x < tiles)
                contract_tile<M, kXbf, kKind, 64, NCBW, WCB>(
                    lds, tile_of_block(blockIdx.x, tiles) * 64, p, v, g, mode, X, C, frag, N, out);
            return;
        }
        contract_tile<M, kXbf, kKind, 32, NCBW, WCB>(lds, tile_of_block(blockIdx.x, gridDim.x) * 32,
                                                     p, v, g, mode, X, C, frag, N, out);
    } else {
        __shared__ __attribute__((aligned(16))) char lds[Low::bytes];
        contract_tile<M, kXbf, kKind, 32, NCBW, WCB>(lds, tile_of_block(blockIdx.x, gridDim.x) * 32,
                                                     p, v, g, mode, X, C, frag, N, out);
    }
}

// ---------------------------------------------------------------- weight gradient
typedef short s16x4v __attribute__((ext_vector_type(4)));

// Eight consecutive k (rows) of one column per lane from a row-major tile:
// lane l of a 16-lane group gets column l of the 16 at p and rows 0..7 (two
// transposing LDS reads of 4 rows x 16 columns each; the lane's own address
// is row l / 4, columns 4 (l % 4)..+3 of the tile).
template <int S>
__device__ __forceinline__ bf16x8 lds_rows8(const uint16_t *p) {
    typedef __attribute__((address_space(3))) s16x4v *lds_t;
    const s16x4v a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)(p));
    const s16x4v b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)(p + 4 * S));
    typedef short s16x8v __attribute__((ext_vector_type(8)));
    const s16x8v r = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, r);
}

// One k-step of 32 rows per tile; four basis functions' 32 channels (8 column
// blocks, two per wave) are in LDS at a time.
template <int M, int NPB, StageKind kKind>
struct DwShape {
    static constexpr int TR = 32;
    static constexpr int RPW = TR / kTileWaves;
    static constexpr int MG = (M + 3) / 4;
    static constexpr int S = 128 + 16;        // 8 mod 64 dwords: the four rows of a
    static constexpr int SP = NPB * 16 + 16;  // transposing read on distinct banks
    static constexpr int SW = stage_entries<M, kKind>(81920 - 3 * TR * (S + SP) * 2);
    static_assert(SW >= 32, "a stage of at least 32 entries");
};

// Block (x, y): split x of the row tiles, slice y % slices of Q's channels and
// chunk y / slices (16 NPB channels) of P's.  part[x][c_P][m][c_Q].
template <int M, bool kXbf, StageKind kKind, int NPB>
__global__ void __launch_bounds__(kTileThreads, (M <= 16 ? 2 : 1))
    tile_dw_kernel(TilePattern p, const float *__restrict__ v, KGeo g, int mode,
                   const void *__restrict__ P, int32_t CP, const void *__restrict__ Q, int32_t CQ,
                   int32_t n_tiles, float *__restrict__ part) {
    using T = DwShape<M, NPB, kKind>;
    constexpr int NA = kXbf ? 1 : 3;  // parts of P
    constexpr int U = kTileU<M, kXbf, T::RPW, (M <= 16 ? T::MG * 2 * NPB * 4 : 64)>;
    using Gather = TileGather<M, kXbf, kKind, T::RPW, T::SW, U>;
    static_assert((3 * T::S + NA * T::SP) * T::TR * 2 +
                      kTileWaves * sizeof(typename Gather::Stage) <= 81920, "two blocks a CU");
    __shared__ __attribute__((aligned(16))) uint16_t dpl[3][T::TR][T::S];
    __shared__ __attribute__((aligned(16))) uint16_t ppl[NA][T::TR][T::SP];
    __shared__ __attribute__((aligned(16))) typename Gather::Stage stage[kTileWaves];

    const int lane = threadIdx.x & 63;
    const int w = threadIdx.x >> 6;
    const int lr = lane >> 4, lc = lane & 15;
    const int32_t slices = (CQ + Gather::CS - 1) / Gather::CS;
    const int32_t slice = blockIdx.y % slices, pc0 = (blockIdx.y / slices) * NPB * 16;

    // column block 2 w + n of each group of basis functions
    floatx4 sum[T::MG][NPB][2];
#pragma unroll
    for (int q = 0; q < T::MG; ++q)
#pragma unroll
        for (int a = 0; a < NPB; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) sum[q][a][b] = floatx4{0.f, 0.f, 0.f, 0.f};

    Gather G(p, v, g, mode, Q, CQ, stage[w]);
    // P rows of a tile: 8 threads a row, 2 NPB channels each
    constexpr int PV = 2 * NPB;
    const int prow = threadIdx.x >> 3, pcol = (threadIdx.x & 7) * PV;
    constexpr int PB = kXbf ? 2 * PV : 16;  // bytes of a load
    const bool pvec = CP % PV == 0 && (reinterpret_cast<uintptr_t>(P) & (PB - 1)) == 0;
    // this XCD's contiguous range of tiles, interleaved over its blocks
    const int32_t nb = gridDim.x, xs = nb < 8 ? nb : 8;
    const int32_t x = blockIdx.x % xs, l = blockIdx.x / xs;
    const int32_t bx = nb / xs + (x < nb % xs ? 1 : 0);
    // (ranges in proportion to the blocks that share them)
    const int32_t before = x * (nb / xs) + (x < nb % xs ? x : nb % xs);
    const int32_t t0 = (int32_t)((int64_t)n_tiles * before / nb);
    const int32_t t1 = (int32_t)((int64_t)n_tiles * (before + bx) / nb);
#pragma unroll 1
    for (int32_t t = t0 + l; t < t1; t += bx) {
        const int32_t row0 = t * T::TR;
        G.begin(row0 + w * T::RPW);
        typename Gather::Acc acc;
        G.slice_sums(slice, acc);
        // the tile's P rows (zero past the last row and channel)
        float pv[PV];
        {
            const int32_t r = row0 + prow, c = pc0 + pcol;
            const bool on = r < p.n_rows;
            const int64_t base = (int64_t)(on ? r : 0) * CP;
            if (pvec) {
                const int32_t cc = c < CP ? c : 0;
                if constexpr (kXbf) {
                    const uint16_t *s = static_cast<const uint16_t *>(P) + base + cc;
                    uint32_t u[PV / 2];
                    if constexpr (PV == 8) {
                        const uint4 q = *reinterpret_cast<const uint4 *>(s);
                        u[0] = q.x; u[1] = q.y; u[2] = q.z; u[3] = q.w;
                    } else {
                        const uint2 q = *reinterpret_cast<const uint2 *>(s);
                        u[0] = q.x; u[1] = q.y;
                    }
#pragma unroll
                    for (int k = 0; k < PV / 2; ++k) {
                        pv[2 * k] = __uint_as_float(u[k] << 16);
                        pv[2 * k + 1] = __uint_as_float(u[k] & 0xFFFF0000u);
                    }
                } else {
                    const float *s = static_cast<const float *>(P) + base + cc;
#pragma unroll
                    for (int k = 0; k < PV; k += 4) {
                        const float4 q = *reinterpret_cast<const float4 *>(s + k);
                        pv[k] = q.x; pv[k + 1] = q.y; pv[k + 2] = q.z; pv[k + 3] = q.w;
                    }
                }
            } else {
#pragma unroll
                for (int k = 0; k < PV; ++k) {
                    const int64_t a = base + (c + k < CP ? c + k : CP - 1);
                    if constexpr (kXbf)
                        pv[k] = __uint_as_float((uint32_t) static_cast<const uint16_t *>(P)[a] << 16);
                    else
                        pv[k] = static_cast<const float *>(P)[a];
                }
            }
#pragma unroll
            for (int k = 0; k < PV; ++k)
                pv[k] = !on || c + k >= CP ? 0.f : quiet(pv[k]);
        }
        __syncthreads();  // the previous tile is multiplied
        {
            uint32_t u[3][PV / 2];
#pragma unroll
            for (int k = 0; k < PV / 2; ++k)
                split2(pv[2 * k], pv[2 * k + 1], u[0][k], u[1][k], u[2][k]);
#pragma unroll
            for (int q = 0; q < NA; ++q) {
                uint16_t *o = &ppl[q][prow][pcol];
                if constexpr (PV == 8)
                    *reinterpret_cast<uint4 *>(o) = make_uint4(u[q][0], u[q][1], u[q][2], u[q][3]);
                else
                    *reinterpret_cast<uint2 *>(o) = make_uint2(u[q][0], u[q][1]);
            }
        }
        const int trow = 8 * lr + (lc >> 2), tcol = 4 * (lc & 3);
#pragma unroll
        for (int mg = 0; mg < T::MG; ++mg) {
            if (mg > 0) __syncthreads();  // the previous columns are multiplied
            G.template store<T::S, T::TR>(dpl, w * T::RPW + G.rl, acc, mg);
            __syncthreads();
            // (two row blocks at a time: the fragments of four, with D's, spilled)
#pragma unroll
            for (int i0 = 0; i0 < NPB; i0 += 2) {
                bf16x8 a[2][NA];
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int q = 0; q < NA; ++q)
                        a[i][q] = lds_rows8<T::SP>(&ppl[q][trow][16 * (i0 + i) + tcol]);
#pragma unroll
                for (int n = 0; n < 2; ++n)
                    if (4 * mg + (2 * w + n) / 2 < M) {
                        bf16x8 b[3];
#pragma unroll
                        for (int q = 0; q < 3; ++q)
                            b[q] = lds_rows8<T::S>(&dpl[q][trow][16 * (2 * w + n) + tcol]);
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            floatx4 lo{0.f, 0.f, 0.f, 0.f};
                            mma_split<NA, 3>(a[i], b, sum[mg][i0 + i][n], lo);
                            sum[mg][i0 + i][n] = finish(sum[mg][i0 + i][n], lo);
                        }
                    }
            }
        }
    }
    // column block 2 w + n of group mg: basis function 4 mg + w, channels 16 n ..
    float *o = part + (int64_t)blockIdx.x * CP * M * CQ;
#pragma unroll
    for (int mg = 0; mg < T::MG; ++mg)
#pragma unroll
        for (int i = 0; i < NPB; ++i)
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                const int m = 4 * mg + w;
                const int32_t q = slice * Gather::CS + 16 * n + lc;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int32_t c = pc0 + 16 * i + 4 * lr + r;
                    if (m < M && c < CP && q < CQ)
                        o[((int64_t)c * M + m) * CQ + q] = sum[mg][i][n][r];
                }
            }
}

}  // namespace sbc
