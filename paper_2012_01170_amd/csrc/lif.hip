// The leaky integrate-and-fire event sampler (the supplementary's event network
// details, and Section 4's stream hierarchy): it turns an event stream into the
// next, coarser one.  Each output cell holds a potential that decays with the
// time since its last update; every input event in its receptive field adds
// 1/n (n = how many cells that event reaches), and when the potential exceeds
// the threshold it is reset and the cell emits an event at the input's time.
//
// A cell's potential depends only on the events of its own receptive field, in
// stream order, so the cells run in parallel:
//   1. each pixel's events are listed, sorted by event index, with their times
//      alongside (counted, placed, then sorted within each pixel; the count
//      also clears the spike flags);
//   2. blocks of 8 cells, a wave per cell: the
//      wave stages the lists of its cell's k x k input pixels in LDS and merges
//      them in parallel, each entry finding its place by binary searches in
//      the other lists; the decay factors exp(-(t_s - t_{s-1}) / decay) of the
//      merged sequence do not depend on the potential and are computed in
//      parallel too.  Then one wave runs the block's recursions
//      v = V e_s + 1/n_s (threshold, reset; float64) side by side, a lane per
//      cell; a spike marks its merged entry, and every wave then sets byte
//      `slot` of event i for the spikes of its cell (slot: the cell's
//      row-major place among the cells event i reaches).  The cells share the staging; those
//      that do not fit together take turns, and one with more events than all
//      of it merges its lists from global memory on another wave, event by
//      event;
//   3. the spikes of each group of 1024 events are counted; a block per group
//      adds up the counts of the groups before it, scans its own events' and
//      writes the output, which are
//      thereby ordered by input event, then cell row, then cell column (the
//      sequential emission order).
#include "common.hpp"
#include "pixel_lists.hpp"

namespace sbc {
namespace {

constexpr int kLifThreads = 64;  // a wave
constexpr int kLifMaxKernel = 5;
constexpr int kGroup = 1024;  // events per block of the emission

struct LifArgs {
    const int32_t *px, *py;
    int32_t n, W, H, Wo, Ho, k, S, pad, nsd;  // nsd: cells per dimension one input can reach
    double decay, thresh, reset;
    const int32_t *pix_start, *list, *list_t;
    int32_t *spikes;                          // [n][words]: byte s is 1 for a spike at slot s
    int32_t words;                            // 4-byte words that hold an event's slots
    uint32_t *status;                         // kFlagInternal on a bad event or slot
};

// Marks the spike of event `ev` at its cell slot `slot` (each once: the slot is
// the cell's).  Both come out of the kernel's own merge, so they are always in
// range; the check keeps a defect there from turning into a store outside the
// words (it raises the status word, which the synchronising call reports,
// instead).  (A byte each and plain stores: with a bit each, set and counted by
// atomics, which leave the XCD's L2, the cells took 117 us instead of 79.)
__device__ __forceinline__ void mark_spike(const LifArgs &A, int64_t ev, int64_t slot) {
    const int64_t nslots = (int64_t)A.nsd * A.nsd;
    if (ev >= 0 && ev < A.n && slot >= 0 && slot < nslots)
        reinterpret_cast<uint8_t *>(A.spikes + ev * A.words)[slot] = 1;
    else
        atomicOr(A.status, kFlagInternal);
}

// Cells o (one dimension) whose receptive field [o*S - pad, o*S - pad + k)
// holds input coordinate x: lo..hi (empty when hi < lo).
__device__ __forceinline__ void cell_range(int32_t x, const LifArgs &A, int32_t n_out,
                                           int32_t &lo, int32_t &hi) {
    const int32_t a = x + A.pad - A.k + 1;  // o * S >= a
    lo = a <= 0 ? 0 : (a + A.S - 1) / A.S;
    hi = (x + A.pad) / A.S;
    hi = hi < n_out - 1 ? hi : n_out - 1;
}

// The receptive field of cell (ox, oy): list q (row-major over the k x k
// pixels) starts at *start and holds *len events; inc is 1/n of its pixel and
// slot the cell's place among the cells that pixel reaches.  Off the sensor:
// an empty list.
__device__ __forceinline__ void field_list(const LifArgs &A, int32_t ox, int32_t oy, int q,
                                           int32_t &start, int32_t &len, double &inc,
                                           int32_t &slot) {
    const int32_t x = ox * A.S - A.pad + q % A.k, y = oy * A.S - A.pad + q / A.k;
    start = len = slot = 0;
    inc = 0.0;
    if (x < 0 || x >= A.W || y < 0 || y >= A.H) return;
    const int32_t p = y * A.W + x;
    start = A.pix_start[p];
    len = A.pix_start[p + 1] - start;
    int32_t lx, hx, ly, hy;
    cell_range(x, A, A.Wo, lx, hx);
    cell_range(y, A, A.Ho, ly, hy);
    inc = 1.0 / (double)((hx - lx + 1) * (hy - ly + 1));  // this cell is one of them
    slot = (oy - ly) * A.nsd + (ox - lx);
}

// One cell on one wave, a list on each of its first k * k lanes: a step takes
// the earliest head (event indices are distinct) and every lane advances the
// potential by it; the taking lane has the entry after its head loaded already.
__device__ __forceinline__ void cell_sequential(const LifArgs &A, int32_t ox, int32_t oy,
                                                int lane) {
#pragma clang fp contract(off)
    constexpr int32_t kNone = INT32_MAX;
    int32_t pos = 0, end = 0, slot = 0;
    double inc = 0.0;
    if (lane < A.k * A.k) {
        int32_t len;
        field_list(A, ox, oy, lane, pos, len, inc, slot);
        end = pos + len;
    }
    int32_t h0 = kNone, t0 = 0, h1 = kNone, t1 = 0;  // the list's next two events
    if (pos < end) {
        h0 = A.list[pos];
        t0 = A.list_t[pos];
    }
    if (pos + 1 < end) {
        h1 = A.list[pos + 1];
        t1 = A.list_t[pos + 1];
    }
    double V = 0.0, T = 0.0;
    for (;;) {
        int32_t best = h0;
#pragma unroll
        for (int d = 1; d < 32; d <<= 1) {
            const int32_t o = __shfl_xor(best, d, 64);
            best = o < best ? o : best;
        }
        best = __builtin_amdgcn_readfirstlane(best);  // (lists sit on lanes below 32)
        if (best == kNone) break;
        const int q = __builtin_ctzll(__ballot(h0 == best));
        const double ti = (double)__shfl(t0, q, 64);
        double v = V * exp(-(ti - T) / A.decay) + __shfl(inc, q, 64);
        if (v > A.thresh) {
            v = A.reset;
            if (lane == q) mark_spike(A, best, slot);
        }
        V = v;
        T = ti;
        if (lane == q) {
            h0 = h1;
            t0 = t1;
            ++pos;
            h1 = kNone;
            if (pos + 1 < end) {
                h1 = A.list[pos + 1];
                t1 = A.list_t[pos + 1];
            }
        }
    }
}

// Cells per block (a wave each while staging and merging; their recursions
// then run side by side on one wave, a lane per cell), and the entries they
// stage together.  The time goes into chains: the merge's searches, then the
// recursions on one wave while the others wait.  33 bytes an entry leave room
// for two blocks a CU, one merging while the other's recursions run: 300k
// events on 128 x 128 pixels, 3 x 3 fields at stride 2 (165 events a cell) take
// 43 us, against 47 with 16 cells in the whole LDS, and 79 where the 8 cells
// need two turns (1024 entries).  Two blocks a CU leave 128 registers; fields of
// 4 x 4 and 5 x 5 spill 25 and 58 of theirs.
template <int K>
struct LifTile {
    static constexpr int kCells = 8;
    static constexpr int kPool = 2048;
};

template <int K>
__global__ void __launch_bounds__(LifTile<K>::kCells * 64)
    __attribute__((amdgpu_waves_per_eu(4))) lif_cell_kernel(LifArgs A) {
#pragma clang fp contract(off)
    constexpr int Q = K * K;
    constexpr int C = LifTile<K>::kCells, MG = LifTile<K>::kPool;
    // cell w's entries from s_moff[w]: its staged lists (list q from off[q]),
    // then the merged sequence
    __shared__ int32_t s_idx[MG];
    __shared__ int32_t s_t[MG];
    __shared__ int32_t m_idx[MG];
    __shared__ int32_t m_t[MG];
    __shared__ uint8_t m_q[MG];
    __shared__ double2 m_ei[MG];  // decay factor and 1/n of each merged event
    __shared__ int32_t s_start[C][Q], s_len[C][Q], s_slot[C][Q], s_L[C], s_moff[C], s_pass[C + 1];
    __shared__ int32_t s_off[C][Q + 1];
    __shared__ double s_inc[C][Q];
    const int w = threadIdx.x / kLifThreads, lane = threadIdx.x % kLifThreads;
    const int64_t cells = (int64_t)A.Wo * A.Ho;
    const int64_t cell = (int64_t)blockIdx.x * C + w;
    const bool valid = cell < cells;
    const int32_t ox = valid ? (int32_t)(cell % A.Wo) : 0, oy = valid ? (int32_t)(cell / A.Wo) : 0;
    if (valid && lane < Q) {
        int32_t start, len, slot;
        double inc;
        field_list(A, ox, oy, lane, start, len, inc, slot);
        s_start[w][lane] = start;
        s_len[w][lane] = len;
        s_slot[w][lane] = slot;
        s_inc[w][lane] = inc;
    }
    __syncthreads();
    // list offsets (in LDS: as registers they spilled) and the longest list
    int32_t L = 0, longest = 0;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int32_t len = valid ? s_len[w][q] : 0;
        if (lane == 0) s_off[w][q] = L;
        L += len;
        longest = len > longest ? len : longest;
    }
    if (lane == 0) {
        s_off[w][Q] = L;
        s_L[w] = L;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        // the cells in order, as many a pass as fit together; pass -1: alone
        int32_t o = 0, pass = 0;
        for (int c = 0; c < C; ++c) {
            if (s_L[c] > MG) {
                s_pass[c] = -1;
                continue;
            }
            if (o + s_L[c] > MG) {
                ++pass;
                o = 0;
            }
            s_pass[c] = pass;
            s_moff[c] = o;
            o += s_L[c];
        }
        s_pass[C] = pass + 1;
    }
    __syncthreads();
    const int32_t passes = s_pass[C];
#pragma unroll 1
    for (int32_t pass = 0; pass < passes; ++pass) {
        const bool staged = valid && s_pass[w] == pass;
        const int32_t mo = staged ? s_moff[w] : 0;
        if (staged) {
            const int32_t *off = s_off[w];
            // stage the lists: the first 64 events of every list in one round of
            // independent loads, longer lists after
            int32_t vi[Q], vt[Q];
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (lane < off[q + 1] - off[q]) {
                    vi[q] = A.list[s_start[w][q] + lane];
                    vt[q] = A.list_t[s_start[w][q] + lane];
                }
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (lane < off[q + 1] - off[q]) {
                    s_idx[mo + off[q] + lane] = vi[q];
                    s_t[mo + off[q] + lane] = vt[q];
                }
            if (longest > kLifThreads)
                for (int q = 0; q < Q; ++q)
                    for (int32_t j = kLifThreads + lane; j < off[q + 1] - off[q]; j += kLifThreads) {
                        s_idx[mo + off[q] + j] = A.list[s_start[w][q] + j];
                        s_t[mo + off[q] + j] = A.list_t[s_start[w][q] + j];
                    }
        }
        __syncthreads();
        if (staged) {
            const int32_t *off = s_off[w];
            // merge: an entry's place is its place in its own list plus, for every
            // other list, the entries there with a smaller event index (binary
            // searches run in lockstep over the lists, so their reads overlap)
            const int steps = 32 - __clz(longest);  // halvings that empty the longest range
            const int32_t *si = s_idx + mo;
            for (int32_t e = lane; e < L; e += kLifThreads) {
                int q = 0;
#pragma unroll
                for (int q2 = 1; q2 < Q; ++q2) q += e >= off[q2] ? 1 : 0;
                const int32_t idx = si[e];
                int32_t base[Q], cnt[Q];
#pragma unroll
                for (int q2 = 0; q2 < Q; ++q2) {
                    base[q2] = off[q2];
                    cnt[q2] = q2 == q ? 0 : off[q2 + 1] - off[q2];
                }
                for (int it = 0; it < steps; ++it)
#pragma unroll
                    for (int q2 = 0; q2 < Q; ++q2)
                        if (cnt[q2] > 0) {
                            const int32_t half = cnt[q2] >> 1;
                            if (si[base[q2] + half] < idx) {
                                base[q2] += half + 1;
                                cnt[q2] -= half + 1;
                            } else {
                                cnt[q2] = half;
                            }
                        }
                int32_t r = e - off[q];
#pragma unroll
                for (int q2 = 0; q2 < Q; ++q2) r += base[q2] - off[q2];
                m_idx[mo + r] = idx;
                m_t[mo + r] = s_t[mo + e];
                m_q[mo + r] = (uint8_t)q;
            }
        }
        __syncthreads();
        if (staged)  // decay factors: T is the previous event's time, 0 before the first
            for (int32_t r = lane; r < L; r += kLifThreads) {
                const double ti = (double)m_t[mo + r];
                const double T = r > 0 ? (double)m_t[mo + r - 1] : 0.0;
                m_ei[mo + r] = make_double2(exp(-(ti - T) / A.decay), s_inc[w][m_q[mo + r]]);
            }
        __syncthreads();
        if (w == 0) {
            // the recursions of the block's staged cells, a lane each; a spike
            // marks its merged entry (bit 7 of m_q) and is passed on after.  The
            // operands of a chunk are read while the chunk before it runs; reads
            // past a cell's end are clamped into the array and unused.
            const int g = lane;
            const bool mine = g < C && (int64_t)blockIdx.x * C + g < cells && s_pass[g] == pass;
            const int32_t go = mine ? s_moff[g] : 0, gL = mine ? s_L[g] : 0;
            constexpr int kC = 4;
            auto at = [&](int32_t r) { return go + r < MG ? go + r : MG - 1; };
            double2 c[kC];
#pragma unroll
            for (int u = 0; u < kC; ++u) c[u] = m_ei[at(u)];
            double V = 0.0;
            for (int32_t r0 = 0; r0 < gL; r0 += kC) {
                double2 n[kC];
#pragma unroll
                for (int u = 0; u < kC; ++u) n[u] = m_ei[at(r0 + kC + u)];
#pragma unroll
                for (int u = 0; u < kC; ++u) {
                    if (r0 + u < gL) {
                        const double v = V * c[u].x + c[u].y;
                        const bool fire = v > A.thresh;
                        V = fire ? A.reset : v;
                        if (fire) m_q[go + r0 + u] |= 0x80;
                    }
                }
#pragma unroll
                for (int u = 0; u < kC; ++u) c[u] = n[u];
            }
        } else if (pass == 0) {
            // cells beyond the staging run alone, a wave each, on the other waves
            for (int g = w - 1; g < C; g += C - 1) {
                const int64_t c = (int64_t)blockIdx.x * C + g;
                if (c < cells && s_pass[g] < 0)
                    cell_sequential(A, (int32_t)(c % A.Wo), (int32_t)(c / A.Wo), lane);
            }
        }
        __syncthreads();
        if (staged)  // the spikes of this wave's cell
            for (int32_t r = lane; r < L; r += kLifThreads) {
                const int q = m_q[mo + r];
                if (q & 0x80)
                    mark_spike(A, m_idx[mo + r], s_slot[w][q & 0x7f]);
            }
        // (the next pass stages where only the merge behind it read, and merges
        // behind a barrier)
    }
}

// Spikes of an event's words and of every group of kGroup events.
__device__ __forceinline__ int32_t event_spikes(const LifArgs &A, int64_t i) {
    int32_t c = 0;
    for (int32_t q = 0; q < A.words; ++q) c += __popc((uint32_t)A.spikes[i * A.words + q]);
    return c;
}

__global__ void __launch_bounds__(256)
    lif_count_kernel(LifArgs A, int32_t *__restrict__ counts) {
    __shared__ int32_t s_sum[4];
    // (the group's words, 256 threads apart)
    const int64_t w0 = (int64_t)blockIdx.x * kGroup * A.words;
    const int64_t all = (int64_t)A.n * A.words;
    const int64_t w1 = w0 + (int64_t)kGroup * A.words < all ? w0 + (int64_t)kGroup * A.words : all;
    int32_t c = 0;
#pragma unroll 4
    for (int64_t q = w0 + threadIdx.x; q < w1; q += 256) c += __popc((uint32_t)A.spikes[q]);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
    if ((threadIdx.x & 63) == 0) s_sum[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
}

// The spikes of kGroup events, four a thread.  offsets: the spikes before each
// group, or null: the block adds up the groups before its own (up to
// kSelfGroups of them).  The last block writes the total, and beside it the
// status, for one copy to the host.
constexpr int kEmitThreads = 256;
constexpr int64_t kSelfGroups = 4096;

__global__ void __launch_bounds__(kEmitThreads)
    lif_emit_kernel(LifArgs A, const int32_t *__restrict__ counts,
                    const int32_t *__restrict__ offsets, const int32_t *__restrict__ t,
                    int64_t capacity, int32_t *__restrict__ out_x, int32_t *__restrict__ out_y,
                    int32_t *__restrict__ out_t, int32_t *__restrict__ out_src,
                    int64_t *__restrict__ total, int64_t *__restrict__ result) {
    constexpr int NW = kEmitThreads / 64, V = kGroup / kEmitThreads;
    __shared__ int64_t s_before[NW];
    __shared__ int32_t s_sum[NW];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    int64_t before = 0;
    if (!offsets)
        for (int64_t q = threadIdx.x; q < (int64_t)blockIdx.x; q += kEmitThreads)
            before += counts[q];
    else if (threadIdx.x == 0)
        before = offsets[blockIdx.x];
    const int32_t i0 = (int32_t)blockIdx.x * kGroup + (int32_t)threadIdx.x * V;
    int32_t m[V], mine = 0;
#pragma unroll
    for (int u = 0; u < V; ++u) {
        m[u] = i0 + u < A.n ? event_spikes(A, i0 + u) : 0;
        mine += m[u];
    }
    int32_t incl = mine;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t y = __shfl_up(incl, d, 64);
        if (lane >= d) incl += y;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) before += __shfl_xor(before, d, 64);
    if (lane == 63) s_sum[w] = incl;
    if (lane == 0) s_before[w] = before;
    __syncthreads();
    int64_t o = incl - mine, all = 0;
#pragma unroll
    for (int q = 0; q < NW; ++q) {
        o += s_before[q] + (q < w ? s_sum[q] : 0);
        all += s_before[q] + s_sum[q];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        *total = all;
        result[0] = all;
        result[1] = *A.status;
    }
#pragma unroll
    for (int u = 0; u < V; ++u) {
        if (m[u] == 0) continue;
        const int32_t i = i0 + u;
        int32_t lx, hx, ly, hy;
        cell_range(A.px[i], A, A.Wo, lx, hx);
        cell_range(A.py[i], A, A.Ho, ly, hy);
        const int32_t ti = t[i];
        for (int32_t q = 0; q < A.words; ++q)
            for (uint32_t b = (uint32_t)A.spikes[(int64_t)i * A.words + q]; b != 0u; b &= b - 1u) {
                const int32_t s = 4 * q + (__ffs((int)b) - 1) / 8;
                if (o < capacity) {
                    out_x[o] = lx + s % A.nsd;
                    out_y[o] = ly + s / A.nsd;
                    out_t[o] = ti;
                    if (out_src) out_src[o] = i;
                }
                ++o;
            }
    }
}

struct LifWs {
    PixelLists pl;
    int32_t *spikes, *counts, *offsets;
    int64_t *result;
    uint32_t *status;
    void *scan_ws;
};

int64_t lif_groups(int32_t n) { return n > 0 ? ((int64_t)n + kGroup - 1) / kGroup : 1; }

int32_t lif_slots(int32_t kernel, int32_t stride) {
    const int32_t nsd = (kernel - 1) / stride + 1;
    return nsd * nsd;
}

LifWs carve_lif(void *base, int32_t n, int64_t npix, int32_t words, size_t *bytes) {
    Carver cv(base);
    const int64_t groups = lif_groups(n);
    LifWs w;
    w.pl = carve_pixel_lists(cv, n, npix);
    w.spikes = cv.take<int32_t>((size_t)n * words);
    w.counts = cv.take<int32_t>(groups);
    w.offsets = cv.take<int32_t>(groups + 1);
    w.result = cv.take<int64_t>(2);
    w.status = cv.take<uint32_t>(4);
    w.scan_ws = cv.take<char>(scan_workspace_bytes(groups));
    if (bytes) *bytes = cv.used;
    return w;
}

sbc_status check_lif_shape(int32_t n, int32_t width, int32_t height, int32_t kernel,
                           int32_t stride) {
    if (n < 0 || width <= 0 || height <= 0)
        return fail(SBC_ERR_INVALID_ARG, "n must be >= 0, width and height > 0");
    if ((int64_t)width * height >= (int64_t)INT32_MAX)
        return fail(SBC_ERR_INVALID_ARG, "width * height must be < 2^31 - 1");
    if (kernel < 1 || kernel > kLifMaxKernel)
        return fail(SBC_ERR_UNSUPPORTED, "kernel must be 1..5");
    if (stride < 1) return fail(SBC_ERR_INVALID_ARG, "stride must be >= 1");
    if ((int64_t)n * lif_slots(kernel, stride) >= (int64_t)INT32_MAX)
        return fail(SBC_ERR_OVERFLOW, "n * cells reached per event must be < 2^31 - 1");
    return SBC_OK;
}

}  // namespace
}  // namespace sbc

using namespace sbc;

extern "C" size_t sbc_lif_workspace_size(int32_t n, int32_t width, int32_t height,
                                         int32_t kernel, int32_t stride) {
    if (check_lif_shape(n, width, height, kernel, stride) != SBC_OK) {
        clear_error();
        return 0;
    }
    size_t bytes = 0;
    carve_lif(nullptr, n, (int64_t)width * height, (lif_slots(kernel, stride) + 3) / 4, &bytes);
    return bytes;
}

extern "C" sbc_status sbc_lif_sample_events(const int32_t *px, const int32_t *py,
                                            const int32_t *t, int32_t n, int32_t width,
                                            int32_t height, int32_t kernel, int32_t stride,
                                            double decay, double v_thresh, double v_reset,
                                            int32_t *out_x, int32_t *out_y, int32_t *out_t,
                                            int32_t *out_src, int64_t capacity,
                                            int64_t *n_out_dev, int64_t *n_out_host,
                                            void *workspace, size_t workspace_bytes,
                                            hipStream_t stream) {
    clear_error();
    SBC_TRY(check_lif_shape(n, width, height, kernel, stride));
    if (!(decay > 0.0)) return fail(SBC_ERR_INVALID_ARG, "decay must be > 0 (inf: no decay)");
    if (n > 0 && (!px || !py || !t)) return fail(SBC_ERR_INVALID_ARG, "null event arrays");
    if (capacity < 0 || (capacity > 0 && (!out_x || !out_y || !out_t)))
        return fail(SBC_ERR_INVALID_ARG, "output arrays are null, or capacity < 0");
    const int64_t npix = (int64_t)width * height;
    const int64_t groups = lif_groups(n);
    size_t need = 0;
    const int32_t words = (lif_slots(kernel, stride) + 3) / 4;
    LifWs ws = carve_lif(workspace, n, npix, words, &need);
    if (!workspace || workspace_bytes < need)
        return fail(SBC_ERR_WORKSPACE, "workspace smaller than sbc_lif_workspace_size()");
    LifArgs A{};
    A.px = px;
    A.py = py;
    A.n = n;
    A.W = width;
    A.H = height;
    A.S = stride;
    A.k = kernel;
    A.pad = (kernel - 1) / 2;
    A.Wo = (width + stride - 1) / stride;
    A.Ho = (height + stride - 1) / stride;
    A.nsd = (kernel - 1) / stride + 1;
    A.decay = decay;
    A.thresh = v_thresh;
    A.reset = v_reset;
    A.pix_start = ws.pl.pix_start;
    A.list = ws.pl.list;
    A.list_t = ws.pl.list_t;
    A.spikes = ws.spikes;
    A.words = words;
    A.status = ws.status;

    SBC_TRY(fill_i32(reinterpret_cast<int32_t *>(ws.status), 0, 1, stream));
    if (n > 0) {
        trace_before("lif_sort", stream);
        SBC_TRY(build_pixel_lists(px, py, t, n, width, height, ws.pl, ws.status, ws.spikes, words,
                                  stream));
        trace_after("lif_sort", stream);
        const int64_t cells = (int64_t)A.Wo * A.Ho;
        trace_before("lif_cells", stream);
#define SBC_LIF_CELLS(KK)                                                                      \
    hipLaunchKernelGGL(lif_cell_kernel<KK>, dim3(grid_for(cells, LifTile<KK>::kCells)),      \
                       dim3(LifTile<KK>::kCells * kLifThreads), 0, stream, A)
        switch (kernel) {
            case 1: SBC_LIF_CELLS(1); break;
            case 2: SBC_LIF_CELLS(2); break;
            case 3: SBC_LIF_CELLS(3); break;
            case 4: SBC_LIF_CELLS(4); break;
            default: SBC_LIF_CELLS(5); break;
        }
#undef SBC_LIF_CELLS
        SBC_LAUNCH_CHECK();
        trace_after("lif_cells", stream);
    }
    trace_before("lif_emit", stream);
    hipLaunchKernelGGL(lif_count_kernel, dim3((unsigned)groups), dim3(256), 0, stream, A,
                       ws.counts);
    SBC_LAUNCH_CHECK();
    const bool self = groups <= kSelfGroups;
    if (!self)
        SBC_TRY(exclusive_scan_i32(ws.counts, ws.offsets, groups, nullptr, ws.scan_ws, stream));
    hipLaunchKernelGGL(lif_emit_kernel, dim3((unsigned)groups), dim3(kEmitThreads), 0, stream, A,
                       ws.counts, self ? nullptr : ws.offsets, t, capacity, out_x, out_y, out_t, out_src,
                       n_out_dev ? n_out_dev : ws.result, ws.result);
    SBC_LAUNCH_CHECK();
    trace_after("lif_emit", stream);
    if (n_out_host) {
        int64_t host[2];
        SBC_HIP_TRY(hipMemcpyAsync(host, ws.result, sizeof(host), hipMemcpyDeviceToHost, stream));
        SBC_HIP_TRY(hipStreamSynchronize(stream));
        const int64_t count = host[0];
        const uint32_t st = (uint32_t)host[1];
        *n_out_host = count;
        if (st & kFlagInternal)
            return fail(SBC_ERR_INTERNAL, "a spike flag index fell outside the flags");
        if (st & kFlagOutOfRange) return fail(SBC_ERR_OUT_OF_RANGE, "pixel outside the sensor");
        if (st & kFlagUnsorted) return fail(SBC_ERR_UNSORTED, "timestamps must be non-decreasing");
        if (count > capacity)
            return fail(SBC_ERR_CAPACITY, "capacity " + std::to_string(capacity) +
                                              " < output events " + std::to_string(count));
    }
    return SBC_OK;
}
