// Event preprocessing of the divergence estimator (gfx950): the steps the
// paper applies before estimation (Sec. 6, "Preprocessing"): hot-pixel
// removal, and the "resized and resampled" variant that scales the image
// coordinates to a smaller sensor and keeps a random fraction of the events.
//
// Both produce compacted copies of the windows (order kept) with new CSR
// offsets.  The random keep decision is a counter-based draw: event k of
// window w (k counted from the window start) is kept iff the top 24 bits of
// SplitMix64 at counter seed + (w * 2^32 + k + 1) * 0x9E3779B97F4A7C15 fall
// below keep_frac * 2^24.
#include <utility>

#include "ecmd_internal.hpp"

namespace ecmd {

constexpr int kPreThreads = 1024;
// Events of a workgroup: a chunk of kPreChunk consecutive events of the batch,
// whichever windows they lie in, so that the launches grow with the events and
// not with the windows.  (A chunk per window: 65535 windows of 10 events
// resampled in 1305 us, windows of 100 in 1312, against 228 and 340 with a
// thread per event, and more windows than a grid holds workgroups refused.)
// Whether event e of a chunk is kept is bit e % 64 of the chunk's word e / 64.
constexpr int kPreIter = 8;
constexpr int kPreWords = kPreThreads * kPreIter / 64;
static_assert(kPreChunk == kPreThreads * kPreIter, "a chunk is a workgroup's events");

__device__ __forceinline__ unsigned long long splitmix64(unsigned long long s) {
    unsigned long long z = s;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// The window of event i: the last w in [lo, hi) that starts at or before it.
__device__ __forceinline__ int window_at(const long long* __restrict__ offsets, int lo, int hi, long long i) {
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (offsets[mid] <= i) lo = mid; else hi = mid;
    }
    return lo;
}

// This workgroup's chunk: its first event in the arrays, how many it holds and
// the windows of its first and last event (mostly the same one).
struct Chunk {
    int lo, hi, n;
    long long base;
};

__device__ __forceinline__ Chunk chunk_of(const long long* __restrict__ offsets, int B) {
    Chunk c;
    c.base = offsets[0] + (long long)blockIdx.x * kPreChunk;
    c.n = (int)min((long long)kPreChunk, offsets[B] - c.base);  // >= 1
    c.lo = window_at(offsets, 0, B, c.base);
    const long long last = c.base + c.n - 1;
    c.hi = offsets[c.lo + 1] > last ? c.lo : window_at(offsets, c.lo + 1, B, last);
    return c;
}

__device__ __forceinline__ int window_of(const Chunk& c, const long long* __restrict__ offsets, int e) {
    return c.lo == c.hi ? c.lo : window_at(offsets, c.lo, c.hi + 1, c.base + e);
}

// Pixel floor(y) W + floor(x), or -1 outside the sensor.
__device__ __forceinline__ int pixel_of(float x, float y, int W, int H) {
    return x >= 0.0f && x < (float)W && y >= 0.0f && y < (float)H ? (int)floorf(y) * W + (int)floorf(x) : -1;
}

// Stores the chunk's keep words and its count of kept events; keep(e) for
// event e of the chunk, e < c.n.
template <class F>
__device__ __forceinline__ void store_keep(const Chunk& c, unsigned long long* __restrict__ words,
                                           int* __restrict__ blk_cnt, F&& keep) {
    __shared__ int s_cnt[kPreThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int cnt = 0;
#pragma unroll
    for (int j = 0; j < kPreIter; ++j) {
        const int e = j * kPreThreads + (int)threadIdx.x;
        const unsigned long long m = __ballot(e < c.n && keep(e, j));
        if (lane == 0) words[(long long)blockIdx.x * kPreWords + j * (kPreThreads / 64) + wave] = m;
        cnt += __popcll(m);
    }
    if (lane == 0) s_cnt[wave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int k = 0; k < kPreThreads / 64; ++k) t += s_cnt[k];
        blk_cnt[blockIdx.x] = t;
    }
}

// keep words of the resample: a counter-based draw per event
__global__ __launch_bounds__(kPreThreads) void k_resample_keep(const long long* __restrict__ offsets, int B,
                                                               unsigned long long seed, unsigned thresh24,
                                                               unsigned long long* __restrict__ words,
                                                               int* __restrict__ blk_cnt) {
    const Chunk c = chunk_of(offsets, B);
    const auto keep = [&](int w, long long k) {  // event k of window w
        const unsigned long long ctr = ((unsigned long long)w << 32) + (unsigned long long)k + 1ull;
        return (unsigned)(splitmix64(seed + ctr * 0x9E3779B97F4A7C15ull) >> 40) < thresh24;
    };
    if (c.lo == c.hi) {
        const long long first = c.base - offsets[c.lo];
        store_keep(c, words, blk_cnt, [&](int e, int) { return keep(c.lo, first + e); });
    } else {
        store_keep(c, words, blk_cnt, [&](int e, int) {
            const int w = window_of(c, offsets, e);
            return keep(w, c.base + e - offsets[w]);
        });
    }
}

// ---------------------------------------------------------------- hot pixels
//
// The counts of a window's pixels do not fit LDS, and an atomic per event on
// counters in memory runs at 24 G/s (853 us for 20M events of 16 windows of
// 1280x720).  So the events' pixels are first sorted into bands of kBandPx
// pixels (16 bits per event), each band is counted in LDS and leaves a bitmap
// of its hot pixels (115 KB a window of 1280x720, read from L2 by the keep
// pass).  20M events of 16 windows of 1280x720, filtered and resampled:
// 1800 -> 662 us; counting and marking 1030 -> 295 us (the band passes read
// 8 bytes an event at 2 TB/s, the compaction moves 440 MB at 5 TB/s).
constexpr int kBandPx = 16384;

// Bands of every event of the chunk: -1 outside the sensor.
__device__ __forceinline__ void chunk_pixels(const Chunk& c, const float* __restrict__ x, const float* __restrict__ y,
                                             int W, int H, int (&pix)[kPreIter]) {
#pragma unroll
    for (int j = 0; j < kPreIter; ++j) {
        const int e = j * kPreThreads + (int)threadIdx.x;
        pix[j] = e < c.n ? pixel_of(x[c.base + e], y[c.base + e], W, H) : -1;
    }
}

// A chunk's counters, one per band of each of its windows, lie together from
// its first window's.  They are counted in LDS where at most kBandLds are;
// with more (many small windows) each gets a few events only, and these go to
// the counters in memory.
constexpr int kBandLds = 2048;
static_assert(kMaxBands <= kBandLds, "a window's bands");
__device__ __forceinline__ long long chunk_bands(const Chunk& c, int nb) { return (long long)(c.hi - c.lo + 1) * nb; }

// Counter of the band of this thread's event j, from the chunk's first one.
__device__ __forceinline__ int band_at(const Chunk& c, const long long* __restrict__ offsets, int j, int nb, int pix) {
    return (window_of(c, offsets, j * kPreThreads + (int)threadIdx.x) - c.lo) * nb + pix / kBandPx;
}

__global__ __launch_bounds__(kPreThreads) void k_band_count(const float* __restrict__ x, const float* __restrict__ y,
                                                            const long long* __restrict__ offsets, int B,
                                                            int W, int H, int nb, int* __restrict__ cnt) {
    __shared__ int s_cnt[kBandLds];
    const Chunk c = chunk_of(offsets, B);
    const long long nc = chunk_bands(c, nb);
    int* const out = cnt + (long long)c.lo * nb;
    int pix[kPreIter];
    chunk_pixels(c, x, y, W, H, pix);
    if (nc > kBandLds) {
#pragma unroll
        for (int j = 0; j < kPreIter; ++j)
            if (pix[j] >= 0) atomicAdd(&out[band_at(c, offsets, j, nb, pix[j])], 1);
        return;
    }
    for (int k = threadIdx.x; k < nc; k += kPreThreads) s_cnt[k] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPreIter; ++j)
        if (pix[j] >= 0) atomicAdd(&s_cnt[band_at(c, offsets, j, nb, pix[j])], 1);
    __syncthreads();
    for (int k = threadIdx.x; k < nc; k += kPreThreads)
        if (s_cnt[k]) atomicAdd(&out[k], s_cnt[k]);
}

__global__ __launch_bounds__(kPreThreads) void k_band_scatter(const float* __restrict__ x, const float* __restrict__ y,
                                                              const long long* __restrict__ offsets, int B,
                                                              int W, int H, int nb, long long* __restrict__ cursor,
                                                              uint16_t* __restrict__ list) {
    __shared__ int s_cnt[kBandLds];
    __shared__ long long s_base[kBandLds];
    const Chunk c = chunk_of(offsets, B);
    const long long nc = chunk_bands(c, nb);
    unsigned long long* const cur = (unsigned long long*)cursor + (long long)c.lo * nb;
    int pix[kPreIter], at[kPreIter], rank[kPreIter];
    chunk_pixels(c, x, y, W, H, pix);
    if (nc > kBandLds) {
#pragma unroll
        for (int j = 0; j < kPreIter; ++j)
            if (pix[j] >= 0)
                list[atomicAdd(&cur[band_at(c, offsets, j, nb, pix[j])], 1ull)] = (uint16_t)(pix[j] % kBandPx);
        return;
    }
    for (int k = threadIdx.x; k < nc; k += kPreThreads) s_cnt[k] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPreIter; ++j)
        if (pix[j] >= 0) {
            at[j] = band_at(c, offsets, j, nb, pix[j]);
            rank[j] = atomicAdd(&s_cnt[at[j]], 1);
        }
    __syncthreads();
    for (int k = threadIdx.x; k < nc; k += kPreThreads)
        if (s_cnt[k]) s_base[k] = (long long)atomicAdd(&cur[k], (unsigned long long)s_cnt[k]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPreIter; ++j)
        if (pix[j] >= 0) list[s_base[at[j]] + rank[j]] = (uint16_t)(pix[j] % kBandPx);
}

// The pixel counts of a band of a window in LDS, then one bit per pixel that
// holds more than max_count events.  (After the scatter a band's cursor is its
// end, the one before it its start.)  A workgroup takes `per` bands: one, or
// with many small windows kPreThreads / 64 or more, of which each wave looks at its
// own and clears them where no pixel can hold more than max_count (65535 windows of
// 6 bands: a workgroup for each would be launched to write 2 KB).
__global__ __launch_bounds__(kPreThreads) void k_band_hot(const long long* __restrict__ cursor,
                                                          const uint16_t* __restrict__ list, long long nbands, int per,
                                                          int nb, int words_w, unsigned max_count,
                                                          unsigned long long* __restrict__ hot) {
    __shared__ __align__(16) unsigned s_cnt[kBandPx];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long k0 = (long long)blockIdx.x * per;
    const auto words = [&](long long k) {  // a band's words, and how many
        const int at = (int)(k % nb) * (kBandPx / 64);
        return std::pair<unsigned long long*, int>(hot + k / nb * words_w + at, min(kBandPx / 64, words_w - at));
    };
    const auto first = [&](long long k) { return k ? cursor[k - 1] : 0ll; };
    for (int i = per == 1 ? 0 : wave; i < per && k0 + i < nbands; i += kPreThreads / 64) {
        const long long k = k0 + i;
        if (cursor[k] - first(k) > (long long)max_count) continue;
        const auto [out, nw] = words(k);  // no pixel can hold more
        for (int q = per == 1 ? threadIdx.x : lane; q < nw; q += per == 1 ? kPreThreads : 64) out[q] = 0ull;
    }
    for (int i = 0; i < per && k0 + i < nbands; ++i) {
        const long long k = k0 + i, beg = first(k), end = cursor[k];
        if (end - beg <= (long long)max_count) continue;
        __syncthreads();  // the band before has been read
        for (int q = threadIdx.x; q < kBandPx / 4; q += kPreThreads)
            reinterpret_cast<uint4*>(s_cnt)[q] = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        for (long long q = beg + threadIdx.x; q < end; q += kPreThreads) atomicAdd(&s_cnt[list[q]], 1u);
        __syncthreads();
        const auto [out, nw] = words(k);
        for (int q = wave; q < nw; q += kPreThreads / 64) {
            const unsigned long long m = __ballot(s_cnt[q * 64 + lane] > max_count);
            if (lane == 0) out[q] = m;
        }
    }
}

// The same bitmap from counters in memory, for sensors of more bands than
// the sort takes.
__global__ __launch_bounds__(kPreThreads) void k_pixel_counts(const float* __restrict__ x, const float* __restrict__ y,
                                                              const long long* __restrict__ offsets, int B,
                                                              int W, int H, unsigned* __restrict__ counts) {
    const Chunk c = chunk_of(offsets, B);
    int pix[kPreIter];
    chunk_pixels(c, x, y, W, H, pix);
#pragma unroll
    for (int j = 0; j < kPreIter; ++j)
        if (pix[j] >= 0)
            atomicAdd(&counts[(long long)window_of(c, offsets, j * kPreThreads + (int)threadIdx.x) * W * H + pix[j]], 1u);
}

// Keep words of the hot-pixel filter, from the bitmap or from the counters.
__global__ __launch_bounds__(kPreThreads) void k_hot_keep(const float* __restrict__ x, const float* __restrict__ y,
                                                          const long long* __restrict__ offsets, int B,
                                                          int W, int H, int words_w,
                                                          const unsigned long long* __restrict__ hot,
                                                          const unsigned* __restrict__ counts, unsigned max_count,
                                                          unsigned long long* __restrict__ words,
                                                          int* __restrict__ blk_cnt) {
    const Chunk c = chunk_of(offsets, B);
    int pix[kPreIter];
    chunk_pixels(c, x, y, W, H, pix);
    bool hot_px[kPreIter];
#pragma unroll
    for (int j = 0; j < kPreIter; ++j) {
        hot_px[j] = false;
        if (pix[j] >= 0) {
            const long long w = window_of(c, offsets, j * kPreThreads + (int)threadIdx.x);
            hot_px[j] = hot ? (hot[w * words_w + (pix[j] >> 6)] >> (pix[j] & 63)) & 1ull
                            : counts[w * W * H + pix[j]] > max_count;
        }
    }
    store_keep(c, words, blk_cnt, [&](int, int j) { return !hot_px[j]; });
}

// ---------------------------------------------------------------- compaction

// Exclusive prefix sums of n counts and their total (out[n]): one workgroup,
// four counts a thread and round, the next round's loaded before the scan.
__global__ __launch_bounds__(1024) void k_scan(const int* __restrict__ in, long long n, long long* __restrict__ out) {
    __shared__ long long s_wave[2][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const auto load = [&](long long k) {
        if (k + 4 <= n) return *reinterpret_cast<const int4*>(in + k);
        return make_int4(k < n ? in[k] : 0, k + 1 < n ? in[k + 1] : 0, k + 2 < n ? in[k + 2] : 0, 0);
    };
    long long total = 0;
    int turn = 0;
    int4 next = load(4 * threadIdx.x);
    for (long long base = 0; base < n; base += 4096, turn ^= 1) {
        const long long k = base + 4 * threadIdx.x;
        const int4 c = next;
        next = load(k + 4096);
        const long long v = (long long)c.x + c.y + c.z + c.w;
        long long incl = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const long long u = __shfl_up(incl, o, 64);
            if (lane >= o) incl += u;
        }
        // two rows: the one written here was last read before the barrier of
        // the round between
        if (lane == 63) s_wave[turn][wave] = incl;
        __syncthreads();
        long long run = total + incl - v;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const long long a = s_wave[turn][j];
            if (j < wave) run += a;
            total += a;
        }
        const int part[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (k + j < n) out[k + j] = run;
            run += part[j];
        }
    }
    if (threadIdx.x == 0) out[n] = total;
}

// The kept events in order.
__global__ __launch_bounds__(kPreThreads) void k_keep_scatter(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ t,
    const long long* __restrict__ offsets, int B, const unsigned long long* __restrict__ words,
    const long long* __restrict__ blk, float sx, float sy,
    float* __restrict__ xo, float* __restrict__ yo, float* __restrict__ to) {
    __shared__ int s_pre[kPreWords];
    const long long first = offsets[0] + (long long)blockIdx.x * kPreChunk;
    const int n = (int)min((long long)kPreChunk, offsets[B] - first);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long* const mine = words + (long long)blockIdx.x * kPreWords;
    if (threadIdx.x < 64) {  // one wave: kept events before each word, two words a lane
        const int a = __popcll(mine[2 * lane]), v = a + __popcll(mine[2 * lane + 1]);
        int incl = v;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int u = __shfl_up(incl, o, 64);
            if (lane >= o) incl += u;
        }
        s_pre[2 * lane] = incl - v;
        s_pre[2 * lane + 1] = incl - v + a;
    }
    __syncthreads();
    const long long base = blk[blockIdx.x];
#pragma unroll
    for (int j = 0; j < kPreIter; ++j) {
        const int e = j * kPreThreads + (int)threadIdx.x, wd = j * (kPreThreads / 64) + wave;
        const unsigned long long m = mine[wd];
        if (e < n && (m >> lane & 1ull)) {
            const long long d = base + s_pre[wd] + __popcll(m & ((1ull << lane) - 1ull));
            const long long i = first + e;
            xo[d] = x[i] * sx;
            yo[d] = y[i] * sy;
            to[d] = t[i];
        }
    }
}
static_assert(kPreWords == 128, "two words of a chunk per lane of the scanning wave");

// The windows' new offsets: the kept events before each window's first, by
// kOffLanes lanes a window (a chain of a lane's loads takes 12 us, this 4).
constexpr int kOffLanes = 16;
__global__ __launch_bounds__(256) void k_keep_offsets(const long long* __restrict__ offsets, int B,
                                                      const unsigned long long* __restrict__ words,
                                                      const long long* __restrict__ blk,
                                                      long long* __restrict__ off_out) {
    const long long w = ((long long)blockIdx.x * 256 + threadIdx.x) / kOffLanes;
    const int part = threadIdx.x % kOffLanes;
    if (w > B) return;
    const long long i = offsets[w] - offsets[0], b = i / kPreChunk;
    const int e = (int)(i % kPreChunk);  // 0 where there is no chunk b
    const unsigned long long* const mine = words + b * kPreWords;
    int v = 0;
#pragma unroll
    for (int j = 0; j < kPreWords / kOffLanes; ++j) {
        const int k = j * kOffLanes + part, n = e - k * 64;  // bits of word k that lie before
        if (n > 0) v += __popcll(mine[k] & (n < 64 ? (1ull << n) - 1ull : ~0ull));
    }
#pragma unroll
    for (int o = kOffLanes / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kOffLanes);
    if (part == 0) off_out[w] = blk[b] + v;
}

hipError_t launch_compact(hipStream_t s, const float* x, const float* y, const float* t, const long long* offsets,
                          int B, long long nblk, const unsigned long long* words, const int* blk_cnt,
                          long long* blk, float sx, float sy, float* xo, float* yo, float* to, long long* off_out) {
    k_scan<<<1, 1024, 0, s>>>(blk_cnt, nblk, blk);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (nblk > 0) {
        k_keep_scatter<<<(unsigned)nblk, kPreThreads, 0, s>>>(x, y, t, offsets, B, words, blk, sx, sy, xo, yo, to);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    k_keep_offsets<<<(unsigned)((((long long)B + 1) * kOffLanes + 255) / 256), 256, 0, s>>>(offsets, B, words, blk, off_out);
    return hipGetLastError();
}

hipError_t launch_resample_keep(hipStream_t s, const long long* offsets, int B, long long nblk,
                                unsigned long long seed, unsigned thresh24, unsigned long long* words, int* blk_cnt) {
    if (nblk <= 0) return hipSuccess;
    k_resample_keep<<<(unsigned)nblk, kPreThreads, 0, s>>>(offsets, B, seed, thresh24, words, blk_cnt);
    return hipGetLastError();
}

int hot_bands(int W, int H) {
    const long long nb = ((long long)W * H + kBandPx - 1) / kBandPx;
    return nb <= kMaxBands ? (int)nb : 0;
}

constexpr long long kManyBands = 16384;  // 64 workgroups of k_band_hot per CU

hipError_t launch_hot_keep(hipStream_t s, const float* x, const float* y, const long long* offsets, int B,
                           long long nblk, int W, int H, int nb, int* cnt, long long* cursor,
                           uint16_t* list, unsigned long long* hot, unsigned* counts, unsigned max_count,
                           unsigned long long* words, int* blk_cnt) {
    if (nblk <= 0) return hipSuccess;
    const int words_w = (int)(((long long)W * H + 63) / 64);
    hipError_t e;
    if (nb > 0) {
        k_band_count<<<(unsigned)nblk, kPreThreads, 0, s>>>(x, y, offsets, B, W, H, nb, cnt);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        k_scan<<<1, 1024, 0, s>>>(cnt, (long long)B * nb, cursor);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        k_band_scatter<<<(unsigned)nblk, kPreThreads, 0, s>>>(x, y, offsets, B, W, H, nb, cursor, list);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        const long long nbands = (long long)B * nb;
        const int per = nbands > kManyBands ? kPreThreads / 64 * (int)(1 + (nbands >> 25)) : 1;  // at most 2^21 workgroups
        k_band_hot<<<(unsigned)((nbands + per - 1) / per), kPreThreads, 0, s>>>(cursor, list, nbands, per, nb, words_w,
                                                                               max_count, hot);
    } else {
        k_pixel_counts<<<(unsigned)nblk, kPreThreads, 0, s>>>(x, y, offsets, B, W, H, counts);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_hot_keep<<<(unsigned)nblk, kPreThreads, 0, s>>>(x, y, offsets, B, W, H, words_w, nb > 0 ? hot : nullptr, counts,
                                            max_count, words, blk_cnt);
    return hipGetLastError();
}

// ------------------------------------------------------------ stream windows

// offsets[k] = first event with t >= t_start + k * tau (t non-decreasing)
__global__ void k_stream_bounds(const double* __restrict__ t, long long n, double t_start, double tau, int K,
                                long long* __restrict__ offsets) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k > K) return;
    const double b = t_start + (double)k * tau;
    long long lo = 0, hi = n;
    while (lo < hi) {
        const long long mid = (lo + hi) >> 1;
        if (t[mid] < b) lo = mid + 1; else hi = mid;
    }
    offsets[k] = lo;
}

// t_rel of every event of the K windows, relative to its window start
__global__ __launch_bounds__(kPreThreads) void k_stream_trel(const double* __restrict__ t,
                                                            const long long* __restrict__ offsets, int K,
                                                            double t_start, double tau, float* __restrict__ t_rel) {
    const long long i = offsets[0] + (long long)blockIdx.x * kPreThreads + threadIdx.x;
    if (i >= offsets[K]) return;
    int lo = 0, hi = K;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (offsets[mid] <= i) lo = mid; else hi = mid;
    }
    t_rel[i - offsets[0]] = (float)(t[i] - (t_start + (double)lo * tau));
}

hipError_t launch_stream_bounds(hipStream_t s, const double* t, long long n, double t_start, double tau, int K,
                                long long* offsets) {
    k_stream_bounds<<<(K + 1 + 255) / 256, 256, 0, s>>>(t, n, t_start, tau, K, offsets);
    return hipGetLastError();
}

hipError_t launch_stream_trel(hipStream_t s, const double* t, const long long* offsets, long long n_sel, int K,
                              double t_start, double tau, float* t_rel) {
    if (n_sel <= 0) return hipSuccess;
    k_stream_trel<<<(unsigned)((n_sel + kPreThreads - 1) / kPreThreads), kPreThreads, 0, s>>>(t, offsets, K, t_start,
                                                                                             tau, t_rel);
    return hipGetLastError();
}

}  // namespace ecmd
