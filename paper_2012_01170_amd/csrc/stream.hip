// The event convolution's deployment form (Section 3.2, Eq. 13-15), for a
// stream fed in batches.  Every pixel x keeps z_x, the decayed sum of the
// features of its events, and tau_x, the time of its last update; an event
// reads its output from the 3 x 3 block around it before updating its own
// pixel.  With learned decays (M_v rates lambda_uv per offset u) a pixel keeps
// one sum per basis function (u, v), each decayed at its own rate; with the
// one rate 1/tau they would all be equal, and one is kept.  A batch does not
// wait for its own events one by one: event i's output is
//   sum over offsets u of W_m(u)^T [ exp(-(t_i - tau_q)/tau) z_q
//                                   + sum over batch events j < i at q of exp(-(t_i - t_j)/tau) f_j ]
// with q = x_i - u and z, tau_q the state before the batch, which is the
// recursion's value (the decays compose).  So a batch is
//   1. the batch's per-pixel lists (stream order),
//   2. G[i, m, :], the bracket above, a thread per (event, offset, 4 channels),
//   3. Y = G W on the matrix cores (the split contraction of the routes),
//   4. the state update, a thread per (pixel, 4 channels) walking the pixel's
//      batch events in order: z <- f_j + exp(-(t_j - tau_x)/tau) z, tau_x <- t_j.
// Decay factors and sums are float64; the state and G are float32.  Batches of
// up to 8192 events do the same in three launches (below, "short batches").
#include "basis.hpp"
#include "common.hpp"
#include "gemm.hpp"
#include "pixel_lists.hpp"

namespace sbc {
namespace {

constexpr int kStreamThreads = 256;
constexpr int kStreamM = 8;  // the 3 x 3 offsets without the centre

// Rates of the basis functions: rates[m] (learned decays, function m = u Mv + v)
// or 1/tau for all (rates null); the state of function m is z[(q Mz + m) C]
// with Mz = M (one sum per function) or z[q C] with Mz = 1 (one for all).
struct StreamRates {
    const float *rates;
    double inv_tau;
    int32_t M, Mv, Mz;
    __device__ double rate(int32_t m) const { return rates ? (double)rates[m] : inv_tau; }
};

__global__ void __launch_bounds__(kStreamThreads)
    stream_gather_kernel(const int32_t *__restrict__ px, const int32_t *__restrict__ py,
                         const int32_t *__restrict__ t, const float *__restrict__ F, int32_t n,
                         int32_t W, int32_t H, StreamRates R, const float *__restrict__ z,
                         const int32_t *__restrict__ z_time,
                         const int32_t *__restrict__ pix_start,
                         const int32_t *__restrict__ list, const int32_t *__restrict__ list_t,
                         int32_t C, float *__restrict__ G) {
    const int32_t chunks = (C + 3) / 4;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (int64_t)n * R.M * chunks) return;
    const int32_t c0 = (int32_t)(g % chunks) * 4;
    const int32_t m = (int32_t)((g / chunks) % R.M);
    const int32_t i = (int32_t)(g / ((int64_t)chunks * R.M));
    // offset u = m / Mv of function m: row-major over the 3 x 3 block, centre skipped
    const int32_t u = m / R.Mv;
    const int k = u < 4 ? u : u + 1;
    const int32_t qx = px[i] - (k % 3 - 1), qy = py[i] - (k / 3 - 1);
    const double lam = R.rate(m);
    const int32_t zm = R.Mz == 1 ? 0 : m;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    if (qx >= 0 && qx < W && qy >= 0 && qy < H) {
        const int32_t q = qy * W + qx;
        const double ti = (double)t[i];
        const double a = exp(-lam * (ti - (double)z_time[q]));
        const float *zq = z + ((int64_t)q * R.Mz + zm) * C;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (c0 + c < C) acc[c] = a * (double)zq[c0 + c];
        const int32_t e1 = pix_start[q + 1];
        for (int32_t e = pix_start[q]; e < e1; ++e) {
            const int32_t j = list[e];
            if (j >= i) break;  // the list is in stream order
            const double b = exp(-lam * (ti - (double)list_t[e]));
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c0 + c < C) acc[c] += b * (double)F[(int64_t)j * C + c0 + c];
        }
    }
    float *row = G + ((int64_t)i * R.M + m) * C;
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (c0 + c < C) row[c0 + c] = (float)acc[c];
}

// A thread per (pixel, state, 4 channels).  The threads of one pixel may sit
// in different waves, so none of them writes the pixel's time, which the
// others read: stream_time_kernel does that afterwards.
__global__ void __launch_bounds__(kStreamThreads)
    stream_update_kernel(const float *__restrict__ F, int64_t npix, StreamRates R,
                         const int32_t *__restrict__ pix_start,
                         const int32_t *__restrict__ list, const int32_t *__restrict__ list_t,
                         int32_t C, float *__restrict__ z, const int32_t *__restrict__ z_time) {
    const int32_t chunks = (C + 3) / 4;
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= npix * R.Mz * chunks) return;
    const int32_t c0 = (int32_t)(g % chunks) * 4;
    const int32_t zm = (int32_t)((g / chunks) % R.Mz);
    const int64_t q = g / ((int64_t)chunks * R.Mz);
    const int32_t e0 = pix_start[q], e1 = pix_start[q + 1];
    if (e0 == e1) return;
    const double lam = R.rate(zm);
    float *zq = z + (q * R.Mz + zm) * C;
    double s[4];
    double last = (double)z_time[q];
#pragma unroll
    for (int c = 0; c < 4; ++c) s[c] = c0 + c < C ? (double)zq[c0 + c] : 0.0;
    for (int32_t e = e0; e < e1; ++e) {
        const int32_t j = list[e];
        const double tj = (double)list_t[e];
        const double a = exp(-lam * (tj - last));
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (c0 + c < C) s[c] = (double)F[(int64_t)j * C + c0 + c] + a * s[c];
        last = tj;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (c0 + c < C) zq[c0 + c] = (float)s[c];
}

// tau_x <- the time of the pixel's last batch event (pixels with none keep theirs).
__global__ void __launch_bounds__(kStreamThreads)
    stream_time_kernel(int64_t npix, const int32_t *__restrict__ pix_start,
                       const int32_t *__restrict__ list_t, int32_t *__restrict__ z_time) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= npix) return;
    const int32_t e0 = pix_start[q], e1 = pix_start[q + 1];
    if (e0 < e1) z_time[q] = list_t[e1 - 1];
}

// ---------------------------------------------------------------- short batches
// A batch of up to kShortBatch events takes three launches instead of twelve: a
// batch of 4096 is launch-bound.  65536 events in 16 batches, 32 channels to 32:
// 796 us by the lists, 343 us here; four rates a pixel, batches of 7639 (12 to
// 12): 641 and 386.  The comparisons grow with n^2, so longer batches (12766:
// equal times by then) stay on the lists.
// On few hot pixels the walks are long chains of dependent loads that also skip
// the later events, where the lists read consecutive entries; with one rate or two
// they are still the faster ones (four batches of 4096 events on 4 pixels, 16
// channels: 4871 -> 3180 us and 5000 -> 4416), with four rates on 4 to 16 pixels
// they are not (5742 -> 7098, 1711 -> 1908).  The host does not see the pixels,
// and the same shape is faster on ordinary streams, so no rule says otherwise.
//   1. links: an event's predecessor in its pixel is the latest earlier event
//      with its key, found by comparing keys with every event of the batch
//      (16.8 M compares for 4096); an event with no later
//      one is its pixel's tail;
//   2. output: a block makes G of 16 events in LDS, a thread per (event,
//      function, 4 channels) that walks the neighbour pixel's events from its
//      tail, and contracts it with W on the matrix cores;
//   3. state: the tails' pixels, each walked from its tail.
// The walks go from late events to early ones; the recursion's sum is the same
// (the decays compose), in float64 as in the longer path.
constexpr int kShortBatch = 8192;
constexpr int kLinkThreads = 1024;  // 16 waves, an event each

// key: the event's pixel (-1 off the sensor); link[i]: the latest earlier event
// of the pixel (-1: none) and the event's time; tail_key[i]: key for a tail, else -1;
// tail[p]: the tail of pixel p.  Pixels without events keep whatever tail[p]
// held: a reader takes tail[p] = j only if 0 <= j < n and tail_key[j] = p, and
// then it is the tail.
//
// A wave compares its event with the whole batch, 64 lanes by 4 keys at a time
// from LDS.  All of it is latency: with 16 lanes an event in blocks of 256 (one
// wave a SIMD, a serial chain of 64 LDS reads) 4096 events took 15.6 us; 64
// lanes an event, blocks of 16 waves and four reads in flight take 7.1.
__global__ void __launch_bounds__(kLinkThreads)
    stream_link_kernel(const int32_t *__restrict__ px, const int32_t *__restrict__ py,
                       const int32_t *__restrict__ t, int32_t n, int32_t W, int32_t H,
                       int2 *__restrict__ link, int32_t *__restrict__ tail_key,
                       int32_t *__restrict__ tail) {
    __shared__ __attribute__((aligned(16))) int32_t key[kShortBatch];
    constexpr int U = 4;          // loads in flight per lane
    constexpr int Q = 64 * 4 * U;  // keys per wave and trip
    const int32_t nq = (n + Q - 1) / Q * Q;  // at most kShortBatch, a multiple of Q
    for (int32_t j0 = threadIdx.x; j0 < nq; j0 += U * kLinkThreads) {
        int32_t x[U], y[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t j = j0 + u * kLinkThreads, jj = j < n ? j : n - 1;
            x[u] = px[jj];
            y[u] = py[jj];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t j = j0 + u * kLinkThreads;
            const bool in = j < n && x[u] >= 0 && x[u] < W && y[u] >= 0 && y[u] < H;
            if (j < nq) key[j] = in ? y[u] * W + x[u] : -1;
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int32_t i = blockIdx.x * (kLinkThreads / 64) + (threadIdx.x >> 6);
    if (i >= n) return;
    const int32_t k = key[i];
    // this lane's keys: the latest match before i, and the latest match of all
    int32_t before = -1, last = -1;
    for (int32_t j0 = 4 * lane; j0 < nq; j0 += Q) {
        int4 q[U];
#pragma unroll
        for (int u = 0; u < U; ++u) q[u] = *reinterpret_cast<const int4 *>(&key[j0 + 256 * u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t v[4] = {q[u].x, q[u].y, q[u].z, q[u].w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int32_t j = j0 + 256 * u + c;
                last = v[c] == k ? j : last;
                before = v[c] == k && j < i ? j : before;
            }
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const int32_t b = __shfl_xor(before, d), a = __shfl_xor(last, d);
        before = b > before ? b : before;
        last = a > last ? a : last;
    }
    if (lane == 0) {
        const bool is_tail = k >= 0 && last == i;
        link[i] = make_int2(k >= 0 ? before : -1, t[i]);
        tail_key[i] = is_tail ? k : -1;
        if (is_tail) tail[k] = i;
    }
}

constexpr int kShortRows = 16;      // events per block: one MFMA row block
constexpr int kShortThreads = 512;  // 8 waves

typedef float floatx4s __attribute__((ext_vector_type(4)));

// LDS row stride of G: 4 mod 64 floats, so the 16 rows x 4 columns an operand
// reads sit on 64 banks.
__host__ __device__ constexpr int32_t short_stride(int32_t K) { return (K + 63) / 64 * 64 + 4; }

__global__ void __launch_bounds__(kShortThreads)
    stream_output_kernel(const int32_t *__restrict__ px, const int32_t *__restrict__ py,
                         const int32_t *__restrict__ t, const float *__restrict__ F, int32_t n,
                         int32_t W, int32_t H, StreamRates R, const float *__restrict__ z,
                         const int32_t *__restrict__ z_time, const int2 *__restrict__ link,
                         const int32_t *__restrict__ tail_key, const int32_t *__restrict__ tail,
                         int32_t C, const float *__restrict__ Wt, int32_t Co,
                         float *__restrict__ Y) {
    extern __shared__ float lds[];
    constexpr int NW = kShortThreads / 64;
    const int32_t K = R.M * C, S = short_stride(K);
    float *G = lds;                                    // [kShortRows][S]
    float *part = lds + (size_t)kShortRows * S;        // [NW][64][4]
    const int32_t chunks = (C + 3) / 4;
    const int32_t i0 = blockIdx.x * kShortRows;
    // whole 16-byte pieces: the state and the features by float4
    const bool vec = C % 4 == 0 && ((reinterpret_cast<uintptr_t>(z) |
                                     reinterpret_cast<uintptr_t>(F)) & 15) == 0;
    for (int32_t x = threadIdx.x; x < kShortRows * R.M * chunks; x += kShortThreads) {
        const int32_t c0 = x % chunks * 4;
        const int32_t m = x / chunks % R.M;
        const int32_t row = x / chunks / R.M, i = i0 + row;
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        // offset u = m / Mv of function m: row-major over the 3 x 3 block, centre skipped
        const int32_t u = m / R.Mv;
        const int k = u < 4 ? u : u + 1;
        const int32_t ii = i < n ? i : n - 1;
        const int32_t qx = px[ii] - (k % 3 - 1), qy = py[ii] - (k / 3 - 1);
        if (i < n && qx >= 0 && qx < W && qy >= 0 && qy < H) {
            const int32_t q = qy * W + qx;
            const double lam = R.rate(m);
            const double ti = (double)t[i];
            int32_t j = tail[q];
            const float *zq = z + ((int64_t)q * R.Mz + (R.Mz == 1 ? 0 : m)) * C + c0;
            const double a = exp(-lam * (ti - (double)z_time[q]));
            float f[4] = {0.f, 0.f, 0.f, 0.f};
            if (vec) {
                const float4 y = *reinterpret_cast<const float4 *>(zq);
                f[0] = y.x; f[1] = y.y; f[2] = y.z; f[3] = y.w;
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (c0 + c < C) f[c] = zq[c];
            }
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c0 + c < C) acc[c] = a * (double)f[c];
            if (j < 0 || j >= n || tail_key[j] != q) j = -1;
            while (j >= 0) {
                const int2 next = link[j];
                if (j < i) {
                    const float *fj = F + (int64_t)j * C + c0;
                    if (vec) {
                        const float4 y = *reinterpret_cast<const float4 *>(fj);
                        f[0] = y.x; f[1] = y.y; f[2] = y.z; f[3] = y.w;
                    } else {
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            if (c0 + c < C) f[c] = fj[c];
                    }
                    const double b = exp(-lam * (ti - (double)next.y));
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[c] += b * (double)f[c];
                }
                j = next.x;
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (c0 + c < C) G[row * S + m * C + c0 + c] = (float)acc[c];
    }
    // K past M C up to a multiple of 4: zeros
    const int32_t K4 = (K + 3) / 4 * 4;
    for (int32_t x = threadIdx.x; x < kShortRows * (K4 - K); x += kShortThreads)
        G[x / (K4 - K) * S + K + x % (K4 - K)] = 0.f;
    __syncthreads();
    // Y rows = G W: 16-column blocks by split K over the waves, the parts added
    // in order
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, lr = lane >> 4, lc = lane & 15;
    const int32_t ncb = (Co + 15) / 16;
    int per = 1;  // column blocks at a time: the largest power of two up to NW
    while (per < NW && per < ncb) per *= 2;
    const int parts = NW / per;
    const int32_t kc = (K4 / 4 + parts - 1) / parts * 4;  // K per part
    const int kp = w / per;
    const int32_t k0 = kp * kc, k1 = k0 + kc < K4 ? k0 + kc : K4;
    for (int32_t cb0 = 0; cb0 < ncb; cb0 += per) {
        const int32_t cb = cb0 + w % per, col = 16 * cb + lc;
        floatx4s acc{0.f, 0.f, 0.f, 0.f};
        if (cb < ncb) {
            const float *a = G + lc * S + lr;
            const bool on = col < Co;
            const float *b = Wt + (on ? col : 0);
            // eight k-steps' loads in flight (steps past the part weigh nothing)
            for (int32_t k = k0; k < k1; k += 32) {
                float av[8], bv[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int32_t kk = k + 4 * q + lr;
                    av[q] = a[k + 4 * q < K4 ? k + 4 * q : 0];
                    bv[q] = b[(int64_t)(kk < K ? kk : K - 1) * Co];
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const bool live = k + 4 * q < k1;
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(
                        live ? av[q] : 0.f, on && live && k + 4 * q + lr < K ? bv[q] : 0.f, acc, 0,
                        0, 0);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) part[(w * 64 + lane) * 4 + r] = acc[r];
        __syncthreads();
        if (kp == 0 && cb < ncb) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                float y = 0.f;
                for (int p = 0; p < parts; ++p) y += part[((p * per + w) * 64 + lane) * 4 + r];
                const int32_t i = i0 + 4 * lr + r;
                if (i < n && col < Co) Y[(int64_t)i * Co + col] = y;
            }
        }
        __syncthreads();
    }
}

// The state of every tail's pixel.  A pixel's threads (its states and 4-channel
// chunks) sit in one block, which reads the pixel's time before it sets it.
__global__ void __launch_bounds__(kStreamThreads)
    stream_state_kernel(const float *__restrict__ F, int32_t n, StreamRates R,
                        const int2 *__restrict__ link, const int32_t *__restrict__ tail_key,
                        int32_t C, int32_t per_block, float *__restrict__ z,
                        int32_t *__restrict__ z_time) {
    const int32_t chunks = (C + 3) / 4, items = R.Mz * chunks;
    const int32_t group = kStreamThreads / per_block;  // threads per event
    const int32_t i = blockIdx.x * per_block + threadIdx.x / group;
    const int32_t q = i < n ? tail_key[i] : -1;
    const int32_t last = q >= 0 ? z_time[q] : 0;
    __syncthreads();  // every thread of the block has its pixel's time
    if (q < 0) return;
    const int32_t ti = link[i].y;
    if (threadIdx.x % group == 0) z_time[q] = ti;
    for (int32_t x = threadIdx.x % group; x < items; x += group) {
        const int32_t c0 = x % chunks * 4, zm = x / chunks;
        const double lam = R.rate(zm);
        float *zq = z + ((int64_t)q * R.Mz + zm) * C + c0;
        const double a = exp(-lam * ((double)ti - (double)last));
        double s[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) s[c] = c0 + c < C ? a * (double)zq[c] : 0.0;
        for (int32_t j = i; j >= 0;) {
            const int2 next = link[j];
            const double b = exp(-lam * ((double)ti - (double)next.y));
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c0 + c < C) s[c] += b * (double)F[(int64_t)j * C + c0 + c];
            j = next.x;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (c0 + c < C) zq[c] = (float)s[c];
    }
}

// LDS of the short batches' output kernel, and whether a batch takes that path:
// its links fit in LDS, and so do 16 rows of G (64 KB: two blocks a CU; wider
// rows, four rates of 28 channels or one of 112, stay on the lists).
size_t short_lds(int32_t K) {
    return ((size_t)kShortRows * short_stride(K) + (size_t)kShortThreads * 4) * 4;
}
bool short_batch(int32_t n, int32_t K) { return n <= kShortBatch && short_lds(K) <= 65536; }

struct StreamWs {
    PixelLists pl;
    uint32_t *status;
    float *G;
    float *part;
    int2 *link;                       // short batches
    int32_t *tail_key, *tail;
};

StreamWs carve_stream(void *base, int32_t n, int64_t npix, int32_t M, int32_t C_in,
                      int32_t C_out, size_t *bytes) {
    Carver cv(base);
    StreamWs w{};
    w.pl = carve_pixel_lists(cv, n, npix);
    w.status = cv.take<uint32_t>(4);
    w.G = cv.take<float>((size_t)n * M * C_in);
    w.part = cv.take<float>(gemm_workspace_floats(n, C_out, (int64_t)M * C_in));
    // a short batch lays its links over the same space, which is larger (the
    // lists hold npix counts and npix + 1 starts, and 28 bytes an event)
    Carver sv(base);
    w.link = sv.take<int2>(n);
    w.tail_key = sv.take<int32_t>(n);
    w.tail = sv.take<int32_t>(npix);
    if (bytes) *bytes = sv.used > cv.used ? sv.used : cv.used;
    return w;
}

sbc_status check_stream(int32_t n, int32_t width, int32_t height, int32_t M, int32_t C_in,
                        int32_t C_out) {
    if (n < 0 || width <= 0 || height <= 0)
        return fail(SBC_ERR_INVALID_ARG, "n must be >= 0, width and height > 0");
    if ((int64_t)width * height >= (int64_t)INT32_MAX)
        return fail(SBC_ERR_INVALID_ARG, "width * height must be < 2^31 - 1");
    if (C_in <= 0 || C_out <= 0) return fail(SBC_ERR_INVALID_ARG, "C_in and C_out must be > 0");
    if ((int64_t)n * M * C_in >= (int64_t)INT32_MAX)
        return fail(SBC_ERR_OVERFLOW, "n * M * C_in must be < 2^31 - 1");
    if ((int64_t)width * height * (M == kStreamM ? 1 : M) * C_in >= (int64_t)INT32_MAX * 2)
        return fail(SBC_ERR_OVERFLOW, "the state has too many entries");
    return SBC_OK;
}

size_t stream_workspace(int32_t n, int32_t width, int32_t height, int32_t M, int32_t C_in,
                        int32_t C_out) {
    if (check_stream(n, width, height, M, C_in, C_out) != SBC_OK) {
        clear_error();
        return 0;
    }
    size_t bytes = 0;
    carve_stream(nullptr, n, (int64_t)width * height, M, C_in, C_out, &bytes);
    return bytes;
}

// One batch: lists, G, Y = G W, state update, times.
sbc_status stream_step(const int32_t *px, const int32_t *py, const int32_t *t, const float *F,
                       int32_t n, int32_t width, int32_t height, StreamRates R, const float *W,
                       int32_t C_in, int32_t C_out, float *z, int32_t *z_time, float *Y,
                       void *workspace, size_t workspace_bytes, hipStream_t stream) {
    if (!z || !z_time) return fail(SBC_ERR_INVALID_ARG, "the state z, z_time is null");
    if (n == 0) return SBC_OK;
    if (!px || !py || !t || !F || !W || !Y)
        return fail(SBC_ERR_INVALID_ARG, "null event, feature, weight or output array");
    const int64_t npix = (int64_t)width * height;
    size_t need = 0;
    StreamWs ws = carve_stream(workspace, n, npix, R.M, C_in, C_out, &need);
    if (!workspace || workspace_bytes < need)
        return fail(SBC_ERR_WORKSPACE, "workspace smaller than the stream's workspace size");
    const int32_t chunks = (C_in + 3) / 4;
    if (short_batch(n, R.M * C_in)) {
        trace_before("stream_lists", stream);
        hipLaunchKernelGGL(stream_link_kernel,
                           dim3(grid_for(n, kLinkThreads / 64)), dim3(kLinkThreads), 0,
                           stream, px, py, t, n, width, height, ws.link, ws.tail_key, ws.tail);
        SBC_LAUNCH_CHECK();
        trace_after("stream_lists", stream);
        trace_before("stream_gather", stream);
        hipLaunchKernelGGL(stream_output_kernel, dim3(grid_for(n, kShortRows)),
                           dim3(kShortThreads), short_lds(R.M * C_in), stream, px, py, t, F, n,
                           width, height, R, z, z_time, ws.link, ws.tail_key, ws.tail, C_in, W,
                           C_out, Y);
        SBC_LAUNCH_CHECK();
        trace_after("stream_gather", stream);
        // events per block: as many as 256 threads hold whole, at least one
        int32_t per_block = 1;
        while (2 * per_block * R.Mz * chunks <= kStreamThreads) per_block *= 2;
        trace_before("stream_update", stream);
        hipLaunchKernelGGL(stream_state_kernel, dim3(grid_for(n, per_block)), dim3(kStreamThreads),
                           0, stream, F, n, R, ws.link, ws.tail_key, C_in, per_block, z, z_time);
        SBC_LAUNCH_CHECK();
        trace_after("stream_update", stream);
        return SBC_OK;
    }
    trace_before("stream_lists", stream);
    SBC_TRY(fill_i32(reinterpret_cast<int32_t *>(ws.status), 0, 1, stream));
    SBC_TRY(build_pixel_lists(px, py, t, n, width, height, ws.pl, ws.status, nullptr, 0, stream));
    trace_after("stream_lists", stream);
    trace_before("stream_gather", stream);
    hipLaunchKernelGGL(stream_gather_kernel,
                       dim3(grid_for((int64_t)n * R.M * chunks, kStreamThreads)),
                       dim3(kStreamThreads), 0, stream, px, py, t, F, n, width, height, R, z,
                       z_time, ws.pl.pix_start, ws.pl.list, ws.pl.list_t, C_in, ws.G);
    SBC_LAUNCH_CHECK();
    trace_after("stream_gather", stream);
    // Y [n, C_out] = G [n, M C_in] x W [M C_in, C_out]
    SBC_TRY(gemm(ws.G, false, (int64_t)R.M * C_in, 1, W, false, C_out, 1, Y, C_out, 1, n, C_out,
                 (int64_t)R.M * C_in, ws.part, stream, "stream_gemm"));
    trace_before("stream_update", stream);
    hipLaunchKernelGGL(stream_update_kernel,
                       dim3(grid_for(npix * R.Mz * chunks, kStreamThreads)),
                       dim3(kStreamThreads), 0, stream, F, npix, R, ws.pl.pix_start, ws.pl.list,
                       ws.pl.list_t, C_in, z, z_time);
    SBC_LAUNCH_CHECK();
    hipLaunchKernelGGL(stream_time_kernel, dim3(grid_for(npix, kStreamThreads)),
                       dim3(kStreamThreads), 0, stream, npix, ws.pl.pix_start, ws.pl.list_t,
                       z_time);
    SBC_LAUNCH_CHECK();
    trace_after("stream_update", stream);
    return SBC_OK;
}

}  // namespace
}  // namespace sbc

using namespace sbc;

extern "C" size_t sbc_event_stream_workspace_size(int32_t n, int32_t width, int32_t height,
                                                  int32_t C_in, int32_t C_out) {
    return stream_workspace(n, width, height, kStreamM, C_in, C_out);
}

extern "C" sbc_status sbc_event_stream_step(const int32_t *px, const int32_t *py,
                                            const int32_t *t, const float *F, int32_t n,
                                            int32_t width, int32_t height, float tau,
                                            const float *W, int32_t C_in, int32_t C_out,
                                            float *z, int32_t *z_time, float *Y,
                                            void *workspace, size_t workspace_bytes,
                                            hipStream_t stream) {
    clear_error();
    SBC_TRY(check_stream(n, width, height, kStreamM, C_in, C_out));
    if (!(tau > 0.f)) return fail(SBC_ERR_INVALID_ARG, "tau must be > 0");
    const StreamRates R{nullptr, 1.0 / (double)tau, kStreamM, 1, 1};
    return stream_step(px, py, t, F, n, width, height, R, W, C_in, C_out, z, z_time, Y, workspace,
                       workspace_bytes, stream);
}

extern "C" size_t sbc_event_stream_decays_workspace_size(int32_t n, int32_t width,
                                                         int32_t height, int32_t n_decays,
                                                         int32_t C_in, int32_t C_out) {
    if (n_decays < 1 || n_decays > 4) return 0;
    return stream_workspace(n, width, height, kStreamM * n_decays, C_in, C_out);
}

extern "C" sbc_status sbc_event_stream_step_decays(const int32_t *px, const int32_t *py,
                                                   const int32_t *t, const float *F, int32_t n,
                                                   int32_t width, int32_t height,
                                                   const float *decays, int32_t n_decays,
                                                   const float *W, int32_t C_in, int32_t C_out,
                                                   float *z, int32_t *z_time, float *Y,
                                                   void *workspace, size_t workspace_bytes,
                                                   hipStream_t stream) {
    clear_error();
    if (n_decays < 1 || n_decays > 4)
        return fail(SBC_ERR_INVALID_ARG, "n_decays must be in 1..4");
    if (!decays) return fail(SBC_ERR_INVALID_ARG, "decays is null");
    const int32_t M = kStreamM * n_decays;
    SBC_TRY(check_stream(n, width, height, M, C_in, C_out));
    const StreamRates R{decays, 0.0, M, n_decays, M};
    return stream_step(px, py, t, F, n, width, height, R, W, C_in, C_out, z, z_time, Y, workspace,
                       workspace_bytes, stream);
}
