// Subsampling of point clouds (Section 3.1, "Subsampling", and the
// supplementary algorithms): iterative farthest points, its approximation with
// distance updates limited to the ball neighbourhood of each taken point, and
// rejection sampling (taking, in input order, every point no earlier taken
// point has in its ball), alone or followed by the approximation.
//
// One workgroup per cloud, with the cloud's squared distances and sampling
// states in LDS:
//   - rejection sampling is the lexicographically first maximal independent
//     set of the ball graph; it is found in rounds: an undecided point whose
//     earlier neighbours are all decided is taken if none of them was taken,
//     else rejected.  The lowest undecided point always decides, so the rounds
//     end, and a decision depends only on final states, so the result is the
//     sequential one whatever the timing;
//   - farthest points: each step is an argmax over the points not yet taken
//     (ties to the lowest index), then the distances are lowered to the new
//     point (all of them, or its ball neighbours).
// Squared distances are float32 in the canonical form of the neighbour search,
// so every choice is exact.
#include <type_traits>

#include "common.hpp"

namespace sbc {
namespace {

constexpr int kSampMax = 8192;  // points per cloud held in LDS
// Clouds of up to kSampNear points keep their coordinates and row bounds in
// LDS too, and their neighbours where they fit: a farthest-point step is a chain
// (argmax, the chosen point's row, its neighbours, their coordinates, the
// distances), and each link from memory costs several times what it costs from
// LDS.
constexpr int kSampNear = 2048;
constexpr int kCus = 256;  // of an MI355X
// That stage's bytes by the blocks that are to share a CU (160 KB beside 41 KB a
// block of words and states): one takes 2048 points and 24576 neighbours, which
// leaves no room for a second block.  A chain of dependent steps leaves a CU
// idle most of the time, so blocks side by side cost each other little, and with
// more clouds than CUs a stage that keeps them apart costs a whole turn.  Quarter
// of the points by the farthest of all, us with no stage / the full stage for any
// number of clouds / this rule: 256 clouds of 256 points 104 / 51 / 51, 300 of
// them 107 / 90 / 53, 1024 of them 201 / 172 / 98, 512 of 1024 points 471 / 354 /
// 196, 768 of 2048 1243 / 1382 / 933.
__host__ __device__ constexpr int samp_stage_bytes(int per_cu) {
    return per_cu == 1 ? 16 * kSampNear + 16 + 2 * 24576 : per_cu == 2 ? 40448 : 13056;
}

// the canonical form, with no contraction of the products into the sums
__device__ __forceinline__ float sq_dist(const float3 &a, const float3 &b) {
#pragma clang fp contract(off)
    const float dx = a.x - b.x, dy = a.y - b.y, dz = a.z - b.z;
    return (dx * dx + dy * dy) + dz * dz;
}

// Maximum (minimum) over the wave by DPP operands (the value ends in lane 63,
// returned to all): through LDS, as shuffles, each of the six steps is a round
// trip.  Lanes a move leaves out take the identity, so each step is one
// instruction.
template <bool kMax>
__device__ __forceinline__ int32_t wave_extreme(int32_t x) {
    constexpr int32_t id = kMax ? INT32_MIN : INT32_MAX;
#define SBC_DPP(ctrl, rows)                                                             \
    do {                                                                                \
        const int32_t y = __builtin_amdgcn_update_dpp(id, x, ctrl, rows, 0xf, false);   \
        x = kMax ? (y > x ? y : x) : (y < x ? y : x);                                   \
    } while (0)
    SBC_DPP(0x111, 0xf);  // row_shr 1, 2, 4, 8: within 16 lanes
    SBC_DPP(0x112, 0xf);
    SBC_DPP(0x114, 0xf);
    SBC_DPP(0x118, 0xf);
    SBC_DPP(0x142, 0xa);  // row_bcast 15 and 31: across the rows of 16
    SBC_DPP(0x143, 0xc);
#undef SBC_DPP
    return __builtin_amdgcn_readlane(x, 63);
}

struct SampleArgs {
    const float *x;
    const int32_t *splits;
    const int32_t *row_ptr, *col_idx;  // in-place ball CSR (may be null for exact IFP)
    int32_t method, per_cloud;
    int32_t near_cap;                  // clouds of at most this many points take the stage
    const int32_t *out_splits;         // (null in the counting pass of rejection sampling)
    int32_t *out_idx, *counts;
    float *dmin2;
};

// kWrite false: the counting pass (each cloud's number of outputs; rejection
// sampling alone decides its points here to count them); kWrite true: the
// sampling, writing the indices at out_splits[b] and the squared distances.
// T threads: a step scans n / T distances a thread and meets T / 64 waves.
// kPerCu: the blocks a CU is to hold.
template <bool kWrite, int T, int kPerCu>
__global__ void __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(kPerCu * T / 256 < 4 ? kPerCu * T / 256 : 4)))
    sample_kernel(SampleArgs A) {
    constexpr int kStage = samp_stage_bytes(kPerCu);
    // a point's squared distance (its bits), later with the sign for "taken"
    __shared__ __attribute__((aligned(16))) int32_t s_word[kSampMax];
    __shared__ uint8_t s_st[kSampMax];  // 0 undecided, 1 taken, 2 rejected
    // [near_cap] coordinates, [near_cap + 1] row bounds, neighbours in the rest
    __shared__ __attribute__((aligned(16))) char s_stage[kStage];
    __shared__ __attribute__((aligned(16))) int64_t s_best[2][T / 64];
    __shared__ int32_t s_count[T / 64];
    __shared__ int32_t s_cnt;
    constexpr int kWaves = T / 64;
    static_assert(sizeof(s_word) + sizeof(s_st) + kStage + sizeof(s_best) + sizeof(s_count) + 16 <=
                      163840 / kPerCu,
                  "LDS of a CU");
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    float3 *const s_x = reinterpret_cast<float3 *>(s_stage);
    int32_t *const s_ptr = reinterpret_cast<int32_t *>(s_stage + 12 * A.near_cap);
    uint16_t *const s_col = reinterpret_cast<uint16_t *>(s_stage + 16 * A.near_cap + 4);
    const int32_t edge_cap = (kStage - 16 * A.near_cap - 4) / 2;
    const int32_t b = blockIdx.x;
    const int32_t s = A.splits[b], n = A.splits[b + 1] - s;
    const bool rej = A.method == SBC_SAMPLE_REJECTION || A.method == SBC_SAMPLE_APPROX_IFP_REJECTION;
    const bool approx = A.method != SBC_SAMPLE_IFP;
    if (n > kSampMax || n < 0) {  // beyond the LDS state (the caller's bound): no outputs
        if (!kWrite && tid == 0) A.counts[b] = 0;
        return;
    }
    if (!kWrite && A.method != SBC_SAMPLE_REJECTION) {
        if (tid == 0) A.counts[b] = A.per_cloud < n ? A.per_cloud : n;
        return;
    }
    const bool near = n <= A.near_cap;
    int32_t e_first = 0;
    bool cols = false;  // the cloud's neighbours are in s_col
    int32_t e_last = 0;
    if (near) {
        if (approx && n > 0) {
            e_first = A.row_ptr[s];
            const int32_t e_end = A.row_ptr[s + n];
            cols = e_end >= e_first && e_end - e_first <= edge_cap;
            e_last = e_end - e_first;
            if (cols)
                for (int32_t e = tid; e < e_end - e_first; e += T) {
                    // (a neighbour outside the cloud is marked: it never counts)
                    const int32_t k = A.col_idx[e_first + e] - s;
                    s_col[e] = k >= 0 && k < n ? (uint16_t)k : (uint16_t)0xFFFF;
                }
        }
        for (int32_t j = tid; j < n; j += T) {
            const float *p = A.x + 3 * ((int64_t)s + j);
            s_x[j] = make_float3(p[0], p[1], p[2]);
            if (cols) s_ptr[j] = A.row_ptr[s + j] - e_first;
        }
        if (cols && tid == 0) s_ptr[n] = A.row_ptr[s + n] - e_first;
    }
    auto point = [&](int32_t j) {
        if (near) return s_x[j];
        const float *p = A.x + 3 * ((int64_t)s + j);
        return make_float3(p[0], p[1], p[2]);
    };
    // Row j's entries, the neighbour of one (negative: outside the cloud) and a
    // point, from LDS and from memory.  (Bounds that do not ascend belong to no
    // ball pattern: in LDS they are kept inside the staged entries.)
    auto lds_point = [&](int32_t j) { return s_x[j]; };
    auto mem_point = [&](int32_t j) {
        const float *p = A.x + 3 * ((int64_t)s + j);
        return make_float3(p[0], p[1], p[2]);
    };
    auto lds_row = [&](int32_t j, int32_t &e0, int32_t &e1) {
        e0 = s_ptr[j] > 0 ? s_ptr[j] : 0;
        e1 = s_ptr[j + 1] < e_last ? s_ptr[j + 1] : e_last;
    };
    auto mem_row = [&](int32_t j, int32_t &e0, int32_t &e1) {
        e0 = A.row_ptr[s + j];
        e1 = A.row_ptr[s + j + 1];
    };
    auto lds_entry = [&](int32_t e) {
        const uint16_t k = s_col[e];
        return k == 0xFFFF ? -1 : (int32_t)k;
    };
    auto mem_entry = [&](int32_t e) {
        const int32_t k = A.col_idx[e] - s;
        return k < n ? k : -1;
    };
    for (int32_t j = tid; j < n; j += T) {
        s_word[j] = __float_as_int(INFINITY);
        s_st[j] = 0;
    }
    if (tid == 0) s_cnt = 0;
    __syncthreads();
    if (rej) {
        // (where rows and neighbours come from is chosen outside the loops)
        auto decide = [&](auto coords, auto bounds, auto entry) {
            // rounds of the first maximal independent set of the ball graph
            bool more = true;
            while (more) {
                bool undecided = false;
                for (int32_t j = tid; j < n; j += T) {
                    if (s_st[j] != 0) continue;
                    bool pending = false, hit = false;
                    int32_t e, e1;
                    bounds(j, e, e1);
                    for (; e < e1; ++e) {
                        const int32_t k = entry(e);
                        if (k < 0 || k >= j) continue;  // later points (and any outside the cloud)
                        const uint8_t st = s_st[k];
                        if (st == 1) { hit = true; break; }
                        if (st == 0) pending = true;
                    }
                    if (hit) s_st[j] = 2;
                    else if (!pending) s_st[j] = 1;
                    else undecided = true;
                }
                more = __syncthreads_or(undecided);
            }
            // distances to the nearest taken neighbour; count the taken points
            int32_t mine = 0;
            for (int32_t j = tid; j < n; j += T) {
                float d = INFINITY;
                const float3 pj = coords(j);
                int32_t e, e1;
                bounds(j, e, e1);
                for (; e < e1; ++e) {
                    const int32_t k = entry(e);
                    if (k >= 0 && s_st[k] == 1) {
                        const float q = sq_dist(coords(k), pj);
                        d = q < d ? q : d;
                    }
                }
                s_word[j] = __float_as_int(d);
                mine += s_st[j] == 1 ? 1 : 0;
            }
            return mine;
        };
        const int32_t mine = cols ? decide(lds_point, lds_row, lds_entry)
                                  : decide(mem_point, mem_row, mem_entry);
        atomicAdd(&s_cnt, mine);  // an integer count: order-free
        __syncthreads();
    }
    const int32_t taken = s_cnt;
    const int32_t total = A.method == SBC_SAMPLE_REJECTION ? taken
                          : (A.per_cloud < n ? A.per_cloud : n);
    if (!kWrite) {
        if (tid == 0) A.counts[b] = total;
        return;
    }
    const int32_t base = A.out_splits[b];
    int32_t pos = 0;
    if (rej) {
        // the taken points first, in input order: each chunk of T points by wave
        // ballots and the waves' counts
        const int32_t cap = taken < total ? taken : total;
        for (int32_t c0 = 0; c0 < n; c0 += T) {
            const int32_t j = c0 + tid;
            const bool f = j < n && s_st[j] == 1;
            const uint64_t m = __ballot(f);
            if (lane == 0) s_count[w] = (int32_t)__popcll(m);
            __syncthreads();
            int32_t rank = pos + (int32_t)__popcll(m & ((1ull << lane) - 1ull));
#pragma unroll
            for (int q = 0; q < kWaves; ++q) {
                const int32_t c = s_count[q];
                if (q < w) rank += c;
                pos += c;
            }
            if (f && rank < cap) A.out_idx[base + rank] = s + j;
            __syncthreads();
        }
        pos = cap;
    }
    // Farthest points.  A point's word is its squared distance's bits, with the
    // sign set once it is taken: as integers, candidates' words compare as their
    // distances do and taken points' words lie below them all, so a taken point
    // is never taken again (which matters once every remaining distance is 0:
    // coincident points).  Ties go to the lowest index.
    int32_t bk = -1, bi = 0;
    const int32_t n4 = (n + 3) / 4;
    for (int32_t j = tid; j < 4 * n4; j += T)
        s_word[j] = j >= n ? INT32_MIN : s_st[j] == 1 ? s_word[j] | INT32_MIN : s_word[j];
    __syncthreads();
    auto offer = [&](int32_t j, int32_t v) {
        if (v > bk) {
            bk = v;
            bi = j;
        }
    };
    // the word of a point at distance q from the newly taken one
    auto lowered = [](int32_t v, float q) {
        return q < __uint_as_float((uint32_t)v & 0x7FFFFFFFu)
                   ? (int32_t)(__float_as_uint(q) | ((uint32_t)v & 0x80000000u))
                   : v;
    };
    // the workgroup's best candidate from the threads' (bk, bi)
    auto argmax = [&](int32_t it) {
        const int32_t wk = wave_extreme<true>(bk);
        const uint64_t who = __ballot(bk == wk);
        int32_t wi;
        if (__popcll(who) == 1)  // the usual case
            wi = __builtin_amdgcn_readlane(bi, (int)__builtin_ctzll(who));
        else
            wi = wave_extreme<false>(bk == wk ? bi : INT32_MAX);
        // (the word, then the lowest index, in one comparison)
        if (lane == 0)
            s_best[it & 1][w] = (int64_t)(((uint64_t)(uint32_t)wk << 32) | (uint32_t)~wi);
        __syncthreads();
        int64_t c[kWaves];
#pragma unroll
        for (int q = 0; q < kWaves; ++q) c[q] = s_best[it & 1][q];
#pragma unroll
        for (int q = 1; q < kWaves; ++q) c[0] = c[q] > c[0] ? c[q] : c[0];
        return __builtin_amdgcn_readfirstlane((int32_t)~(uint32_t)c[0]);
    };
    // Thread (it - pos) % T keeps the point taken in step it; they are stored T
    // steps at a time (a store in every step would be waited for).
    int32_t mine = 0;
    auto record = [&](int32_t it, int32_t sel) {
        const int32_t slot = (it - pos) % T;
        if (tid == slot) mine = s + sel;
        if ((slot == T - 1 || it + 1 == total) && tid <= slot)
            A.out_idx[base + it - slot + tid] = mine;
    };
    // Steps that lower the chosen point's ball.  Where points, rows and
    // neighbours come from is chosen outside the loop: with the choice inside,
    // every step waited for the memory path's loads and stores.
    auto ball_steps = [&](auto coords, auto bounds, auto entry) {
        for (int32_t it = pos; it < total; ++it) {
            bk = -1;
            bi = 0;
#pragma unroll 2
            for (int32_t j = tid; j < n4; j += T) {
                const int4 k = *reinterpret_cast<const int4 *>(&s_word[4 * j]);
                offer(4 * j, k.x);
                offer(4 * j + 1, k.y);
                offer(4 * j + 2, k.z);
                offer(4 * j + 3, k.w);
            }
            const int32_t sel = argmax(it);
            const float3 ps = coords(sel);
            int32_t e, e1;
            bounds(sel, e, e1);
            for (e += tid; e < e1; e += T) {
                const int32_t k = entry(e);
                if (k < 0) continue;
                const int32_t v = lowered(s_word[k], sq_dist(coords(k), ps));
                s_word[k] = k == sel ? v | INT32_MIN : v;
            }
            // (its ball holds the chosen point itself unless the pattern leaves it
            // out; the two writes of its word agree in any order)
            if (tid == 0) atomicOr(&s_word[sel], INT32_MIN);
            record(it, sel);
            __syncthreads();
        }
    };
    // Steps that lower every point, kept in registers (n <= NP T points, thread
    // tid the points tid, tid + T, ...): no word is shared, so a step has one
    // barrier.
    auto all_steps = [&](auto np) {
        constexpr int NP = decltype(np)::value;
        float3 x[NP];
        int32_t v[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int32_t j = tid + q * T;
            v[q] = j < n ? s_word[j] : INT32_MIN;
            x[q] = j < n ? point(j) : make_float3(0.f, 0.f, 0.f);
        }
        auto offer_all = [&]() {
            bk = -1;
            bi = 0;
#pragma unroll
            for (int q = 0; q < NP; ++q) offer(tid + q * T, v[q]);
        };
        offer_all();
        for (int32_t it = pos; it < total; ++it) {
            const int32_t sel = argmax(it);
            const float3 ps = point(sel);
#pragma unroll
            for (int q = 0; q < NP; ++q) {
                const int32_t j = tid + q * T;
                if (j == sel) v[q] |= INT32_MIN;
                if (j < n) v[q] = lowered(v[q], sq_dist(x[q], ps));
            }
            offer_all();
            record(it, sel);
        }
#pragma unroll
        for (int q = 0; q < NP; ++q)
            if (tid + q * T < n) s_word[tid + q * T] = v[q];
    };
    if (!approx) {
        if (n <= 4 * T) all_steps(std::integral_constant<int, 4>{});
        else if (n <= 8 * T) all_steps(std::integral_constant<int, 8>{});
        else if (n <= 16 * T) all_steps(std::integral_constant<int, 16>{});
        else all_steps(std::integral_constant<int, kSampMax / T>{});
    } else if (cols) {
        ball_steps(lds_point, lds_row, lds_entry);
    } else if (near) {
        ball_steps(lds_point, mem_row, mem_entry);
    } else {
        ball_steps(mem_point, mem_row, mem_entry);
    }
    if (A.dmin2) {
        __syncthreads();
        for (int32_t j = tid; j < n; j += T)
            A.dmin2[s + j] = __uint_as_float((uint32_t)s_word[j] & 0x7FFFFFFFu);
    }
}

}  // namespace
}  // namespace sbc

using namespace sbc;

extern "C" size_t sbc_sampling_workspace_size(int32_t n_batch) {
    if (n_batch < 0) return 0;
    return align_up((size_t)n_batch * 4) + align_up(16) + scan_workspace_bytes(n_batch);
}

extern "C" sbc_status sbc_sample_points(const float *x, const int32_t *splits, int32_t n_batch,
                                        int32_t n_points, int32_t max_cloud,
                                        const sbc_csr *ball, sbc_sampling method,
                                        int32_t per_cloud, int32_t *out_idx,
                                        int32_t *out_splits, float *dmin2, void *workspace,
                                        size_t workspace_bytes, hipStream_t stream) {
    clear_error();
    if (n_batch < 1 || !splits || !out_splits || n_points < 0)
        return fail(SBC_ERR_INVALID_ARG, "n_batch must be >= 1 with splits and out_splits");
    if (method != SBC_SAMPLE_IFP && method != SBC_SAMPLE_APPROX_IFP &&
        method != SBC_SAMPLE_APPROX_IFP_REJECTION && method != SBC_SAMPLE_REJECTION)
        return fail(SBC_ERR_INVALID_ARG, "unknown sampling method");
    if (method != SBC_SAMPLE_REJECTION && per_cloud < 0)
        return fail(SBC_ERR_INVALID_ARG, "per_cloud must be >= 0");
    if (max_cloud < 0 || max_cloud > kSampMax)
        return fail(SBC_ERR_UNSUPPORTED, "clouds of at most 8192 points");
    if (n_points > 0 && (!x || !out_idx)) return fail(SBC_ERR_INVALID_ARG, "x or out_idx is null");
    if (method != SBC_SAMPLE_IFP &&
        (!ball || !ball->row_ptr || ball->n_rows != n_points || ball->n_cols != n_points ||
         (ball->nnz_bound > 0 && !ball->col_idx)))
        return fail(SBC_ERR_INVALID_ARG, "the in-place ball pattern of the points is needed");
    const size_t need = sbc_sampling_workspace_size(n_batch);
    if (!workspace || workspace_bytes < need)
        return fail(SBC_ERR_WORKSPACE, "workspace smaller than sbc_sampling_workspace_size()");
    Carver cv(workspace);
    int32_t *counts = cv.take<int32_t>(n_batch);
    int64_t *total = cv.take<int64_t>(2);
    void *scan_ws = cv.take<char>(scan_workspace_bytes(n_batch));
    SampleArgs A{};
    A.x = x;
    A.splits = splits;
    A.row_ptr = ball ? ball->row_ptr : nullptr;
    A.col_idx = ball ? ball->col_idx : nullptr;
    A.method = method;
    A.per_cloud = per_cloud;
    A.out_idx = out_idx;
    A.counts = counts;
    A.dmin2 = nullptr;
    // counts per cloud (rejection sampling runs once here to count), bounds,
    // then the sampling with its writes
    // A CU is to hold as many blocks as the clouds give each, and three at most, as
    // many as held the words and states of 8192 points alone before there was a
    // stage.  A farthest-point step is a chain: 256 threads where no cloud has more
    // than kSampNear points (a step's scan is then at most 8 distances a thread),
    // else 512.  Rejection's rounds are parallel: 512 threads, and nothing staged
    // where no steps follow or the largest cloud does not fit the stage (rejection
    // alone, 32 clouds of 1024: 86 us with no stage, 115 staged, 78 now; 768 of 6000
    // with it and steps, 228 and 304: the registers hold two blocks a CU).
    const int per_cu = n_batch <= kCus ? 1 : n_batch <= 2 * kCus ? 2 : 3;
    const int32_t fits = (samp_stage_bytes(per_cu) - 4) / 16;
    const int32_t lim = fits < kSampNear ? fits : kSampNear;
    const bool rounds = method == SBC_SAMPLE_REJECTION ||
                        (method == SBC_SAMPLE_APPROX_IFP_REJECTION && max_cloud > lim);
    const bool small = max_cloud <= kSampNear && !rounds;
    // (max_cloud bounds no access: larger clouds are read from memory)
    A.near_cap = method == SBC_SAMPLE_REJECTION ? 0 : max_cloud < lim ? max_cloud : lim;
    auto launch = [&](auto write) {
        constexpr bool kW = decltype(write)::value;
        auto with = [&](auto per) {
            constexpr int P = decltype(per)::value;
            if (small)
                hipLaunchKernelGGL((sample_kernel<kW, 256, P>), dim3(n_batch), dim3(256), 0,
                                   stream, A);
            else
                hipLaunchKernelGGL((sample_kernel<kW, 512, P>), dim3(n_batch), dim3(512), 0,
                                   stream, A);
        };
        if (per_cu == 1) with(std::integral_constant<int, 1>{});
        else if (per_cu == 2) with(std::integral_constant<int, 2>{});
        else with(std::integral_constant<int, 3>{});
    };
    trace_before("sample_count", stream);
    launch(std::false_type{});
    SBC_LAUNCH_CHECK();
    trace_after("sample_count", stream);
    SBC_TRY(exclusive_scan_i32(counts, out_splits, n_batch, total, scan_ws, stream));
    A.out_splits = out_splits;
    A.dmin2 = dmin2;
    trace_before("sample", stream);
    launch(std::true_type{});
    SBC_LAUNCH_CHECK();
    trace_after("sample", stream);
    return SBC_OK;
}
