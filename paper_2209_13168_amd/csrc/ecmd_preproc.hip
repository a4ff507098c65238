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
#include "ecmd_internal.hpp"

namespace ecmd {

constexpr int kPreThreads = 1024;
// Events of a workgroup: a chunk of one window (the host cuts every window
// into chunks of kPreChunk; blk_start is their prefix).  Whether event e of a
// chunk is kept is bit e % 64 of the chunk's word e / 64.
constexpr int kPreIter = 8;
constexpr int kPreWords = kPreThreads * kPreIter / 64;
static_assert(kPreChunk == kPreThreads * kPreIter, "a chunk is a workgroup's events");

__device__ __forceinline__ unsigned long long splitmix64(unsigned long long s) {
    unsigned long long z = s;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// This workgroup's chunk: its window, the chunk's first event counted from
// the window's start, and how many events it holds.
struct Chunk {
    int w, n;
    long long first, base;  // base: the chunk's first event in the arrays
};

__device__ __forceinline__ Chunk chunk_of(const int* __restrict__ blk_start, int B,
                                          const long long* __restrict__ offsets) {
    int lo = 0, hi = B;  // the last window that starts at or before this chunk
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (blk_start[mid] <= (int)blockIdx.x) lo = mid; else hi = mid;
    }
    Chunk c;
    c.w = lo;
    c.first = (long long)((int)blockIdx.x - blk_start[lo]) * kPreChunk;
    c.base = offsets[lo] + c.first;
    c.n = (int)min((long long)kPreChunk, offsets[lo + 1] - c.base);
    return c;
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
                                                               const int* __restrict__ blk_start,
                                                               unsigned long long seed, unsigned thresh24,
                                                               unsigned long long* __restrict__ words,
                                                               int* __restrict__ blk_cnt) {
    const Chunk c = chunk_of(blk_start, B, offsets);
    store_keep(c, words, blk_cnt, [&](int e, int) {
        const unsigned long long ctr = ((unsigned long long)c.w << 32) + (unsigned long long)(c.first + e) + 1ull;
        return (unsigned)(splitmix64(seed + ctr * 0x9E3779B97F4A7C15ull) >> 40) < thresh24;
    });
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

__global__ __launch_bounds__(kPreThreads) void k_band_count(const float* __restrict__ x, const float* __restrict__ y,
                                                            const long long* __restrict__ offsets, int B,
                                                            const int* __restrict__ blk_start, int W, int H, int nb,
                                                            int* __restrict__ cnt) {
    __shared__ int s_cnt[kMaxBands];
    const Chunk c = chunk_of(blk_start, B, offsets);
    for (int k = threadIdx.x; k < nb; k += kPreThreads) s_cnt[k] = 0;
    int pix[kPreIter];
    chunk_pixels(c, x, y, W, H, pix);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPreIter; ++j)
        if (pix[j] >= 0) atomicAdd(&s_cnt[pix[j] / kBandPx], 1);
    __syncthreads();
    for (int k = threadIdx.x; k < nb; k += kPreThreads)
        if (s_cnt[k]) atomicAdd(&cnt[(long long)c.w * nb + k], s_cnt[k]);
}

__global__ __launch_bounds__(kPreThreads) void k_band_scatter(const float* __restrict__ x, const float* __restrict__ y,
                                                              const long long* __restrict__ offsets, int B,
                                                              const int* __restrict__ blk_start, int W, int H, int nb,
                                                              long long* __restrict__ cursor,
                                                              uint16_t* __restrict__ list) {
    __shared__ int s_cnt[kMaxBands];
    __shared__ long long s_base[kMaxBands];
    const Chunk c = chunk_of(blk_start, B, offsets);
    for (int k = threadIdx.x; k < nb; k += kPreThreads) s_cnt[k] = 0;
    int pix[kPreIter], rank[kPreIter];
    chunk_pixels(c, x, y, W, H, pix);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPreIter; ++j)
        if (pix[j] >= 0) rank[j] = atomicAdd(&s_cnt[pix[j] / kBandPx], 1);
    __syncthreads();
    for (int k = threadIdx.x; k < nb; k += kPreThreads)
        if (s_cnt[k])
            s_base[k] = (long long)atomicAdd((unsigned long long*)&cursor[(long long)c.w * nb + k],
                                             (unsigned long long)s_cnt[k]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPreIter; ++j)
        if (pix[j] >= 0) list[s_base[pix[j] / kBandPx] + rank[j]] = (uint16_t)(pix[j] % kBandPx);
}

// One workgroup per band of a window: its pixel counts in LDS, then one bit
// per pixel that holds more than max_count events.  (After the scatter a
// band's cursor is its end, the one before it its start.)
__global__ __launch_bounds__(kPreThreads) void k_band_hot(const long long* __restrict__ cursor,
                                                          const uint16_t* __restrict__ list, int nb, int words_w,
                                                          unsigned max_count, unsigned long long* __restrict__ hot) {
    __shared__ __align__(16) unsigned s_cnt[kBandPx];
    const long long k = blockIdx.x;
    const int band = (int)(k % nb);
    unsigned long long* const out = hot + k / nb * words_w + band * (kBandPx / 64);
    const int nw = min(kBandPx / 64, words_w - band * (kBandPx / 64));
    const long long beg = k ? cursor[k - 1] : 0, end = cursor[k];
    if (end - beg <= (long long)max_count) {  // no pixel can hold more
        for (int i = threadIdx.x; i < nw; i += kPreThreads) out[i] = 0ull;
        return;
    }
    for (int i = threadIdx.x; i < kBandPx / 4; i += kPreThreads)
        reinterpret_cast<uint4*>(s_cnt)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    for (long long i = beg + threadIdx.x; i < end; i += kPreThreads) atomicAdd(&s_cnt[list[i]], 1u);
    __syncthreads();
    for (int i = threadIdx.x >> 6; i < nw; i += kPreThreads / 64) {
        const unsigned long long m = __ballot(s_cnt[i * 64 + (threadIdx.x & 63)] > max_count);
        if ((threadIdx.x & 63) == 0) out[i] = m;
    }
}

// The same bitmap from counters in memory, for sensors of more bands than
// the sort takes.
__global__ __launch_bounds__(kPreThreads) void k_pixel_counts(const float* __restrict__ x, const float* __restrict__ y,
                                                              const long long* __restrict__ offsets, int B,
                                                              const int* __restrict__ blk_start, int W, int H,
                                                              unsigned* __restrict__ counts) {
    const Chunk c = chunk_of(blk_start, B, offsets);
    int pix[kPreIter];
    chunk_pixels(c, x, y, W, H, pix);
#pragma unroll
    for (int j = 0; j < kPreIter; ++j)
        if (pix[j] >= 0) atomicAdd(&counts[(long long)c.w * W * H + pix[j]], 1u);
}

// Keep words of the hot-pixel filter, from the bitmap or from the counters.
__global__ __launch_bounds__(kPreThreads) void k_hot_keep(const float* __restrict__ x, const float* __restrict__ y,
                                                          const long long* __restrict__ offsets, int B,
                                                          const int* __restrict__ blk_start, int W, int H, int words_w,
                                                          const unsigned long long* __restrict__ hot,
                                                          const unsigned* __restrict__ counts, unsigned max_count,
                                                          unsigned long long* __restrict__ words,
                                                          int* __restrict__ blk_cnt) {
    const Chunk c = chunk_of(blk_start, B, offsets);
    int pix[kPreIter];
    chunk_pixels(c, x, y, W, H, pix);
    bool hot_px[kPreIter];
#pragma unroll
    for (int j = 0; j < kPreIter; ++j) {
        hot_px[j] = false;
        if (pix[j] >= 0)
            hot_px[j] = hot ? (hot[(long long)c.w * words_w + (pix[j] >> 6)] >> (pix[j] & 63)) & 1ull
                            : counts[(long long)c.w * W * H + pix[j]] > max_count;
    }
    store_keep(c, words, blk_cnt, [&](int, int j) { return !hot_px[j]; });
}

// ---------------------------------------------------------------- compaction

// Exclusive prefix sums of n counts and their total (out[n]): one workgroup,
// a run of consecutive counts per thread.
__global__ __launch_bounds__(1024) void k_scan(const int* __restrict__ in, long long n, long long* __restrict__ out) {
    __shared__ long long s_wave[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long per = (n + 1023) / 1024;
    const long long a = min(n, per * threadIdx.x), b = min(n, a + per);
    long long v = 0;
    for (long long k = a; k < b; ++k) v += in[k];
    long long incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long u = __shfl_up(incl, o, 64);
        if (lane >= o) incl += u;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    long long run = incl - v;
    for (int k = 0; k < wave; ++k) run += s_wave[k];
    for (long long k = a; k < b; ++k) {
        out[k] = run;
        run += in[k];
    }
    if (threadIdx.x == 1023) out[n] = run;  // its run ends at n
}

// The kept events in order, and the windows' new offsets (a window starts
// with its first chunk).
__global__ __launch_bounds__(kPreThreads) void k_keep_scatter(
    const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ t,
    const long long* __restrict__ offsets, int B, const int* __restrict__ blk_start,
    const unsigned long long* __restrict__ words, const long long* __restrict__ blk, float sx, float sy,
    float* __restrict__ xo, float* __restrict__ yo, float* __restrict__ to) {
    __shared__ int s_pre[kPreWords];
    const Chunk c = chunk_of(blk_start, B, offsets);
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
        if (e < c.n && (m >> lane & 1ull)) {
            const long long d = base + s_pre[wd] + __popcll(m & ((1ull << lane) - 1ull));
            const long long i = c.base + e;
            xo[d] = x[i] * sx;
            yo[d] = y[i] * sy;
            to[d] = t[i];
        }
    }
}
static_assert(kPreWords == 128, "two words of a chunk per lane of the scanning wave");

__global__ void k_keep_offsets(const int* __restrict__ blk_start, int B, const long long* __restrict__ blk,
                               long long* __restrict__ off_out) {
    const int w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w <= B) off_out[w] = blk[blk_start[w]];
}

hipError_t launch_compact(hipStream_t s, const float* x, const float* y, const float* t, const long long* offsets,
                          int B, const int* blk_start, int nblk, const unsigned long long* words, const int* blk_cnt,
                          long long* blk, float sx, float sy, float* xo, float* yo, float* to, long long* off_out) {
    k_scan<<<1, 1024, 0, s>>>(blk_cnt, nblk, blk);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (nblk > 0) {
        k_keep_scatter<<<nblk, kPreThreads, 0, s>>>(x, y, t, offsets, B, blk_start, words, blk, sx, sy, xo, yo, to);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    k_keep_offsets<<<(B + 1 + 255) / 256, 256, 0, s>>>(blk_start, B, blk, off_out);
    return hipGetLastError();
}

hipError_t launch_resample_keep(hipStream_t s, const long long* offsets, int B, const int* blk_start, int nblk,
                                unsigned long long seed, unsigned thresh24, unsigned long long* words, int* blk_cnt) {
    if (nblk <= 0) return hipSuccess;
    k_resample_keep<<<nblk, kPreThreads, 0, s>>>(offsets, B, blk_start, seed, thresh24, words, blk_cnt);
    return hipGetLastError();
}

int hot_bands(int W, int H) {
    const long long nb = ((long long)W * H + kBandPx - 1) / kBandPx;
    return nb <= kMaxBands ? (int)nb : 0;
}

hipError_t launch_hot_keep(hipStream_t s, const float* x, const float* y, const long long* offsets, int B,
                           const int* blk_start, int nblk, int W, int H, int nb, int* cnt, long long* cursor,
                           uint16_t* list, unsigned long long* hot, unsigned* counts, unsigned max_count,
                           unsigned long long* words, int* blk_cnt) {
    if (nblk <= 0) return hipSuccess;
    const int words_w = (int)(((long long)W * H + 63) / 64);
    hipError_t e;
    if (nb > 0) {
        k_band_count<<<nblk, kPreThreads, 0, s>>>(x, y, offsets, B, blk_start, W, H, nb, cnt);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        k_scan<<<1, 1024, 0, s>>>(cnt, (long long)B * nb, cursor);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        k_band_scatter<<<nblk, kPreThreads, 0, s>>>(x, y, offsets, B, blk_start, W, H, nb, cursor, list);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        k_band_hot<<<(unsigned)(B * nb), kPreThreads, 0, s>>>(cursor, list, nb, words_w, max_count, hot);
    } else {
        k_pixel_counts<<<nblk, kPreThreads, 0, s>>>(x, y, offsets, B, blk_start, W, H, counts);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_hot_keep<<<nblk, kPreThreads, 0, s>>>(x, y, offsets, B, blk_start, W, H, words_w, nb > 0 ? hot : nullptr, counts,
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
