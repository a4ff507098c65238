// HIP kernels of the MI355X divergence estimator (gfx950).
//
// Method: arXiv 2209.13168 -- radial warp eq. (12), event image eq. (13),
// contrast eq. (14), upper bound eqs. (15)-(20), branch and bound Alg. 1.
// Built with -ffp-contract=off: every fp32/fp64 operation below rounds
// exactly as written (the readings are listed in include/ecmd.h).
#include <hip/hip_ext.h>

#include "ecmd_internal.hpp"

namespace ecmd {

// ------------------------------------------------------------ arithmetic

__device__ __forceinline__ float rate_of(float d, float tau) {
    float a = d * tau;
    float den = 1.0f - a;
    return d / den;  // correctly rounded fp32 division
}

__device__ __forceinline__ float grid_d(float d_lo, float d_hi, int L, unsigned j) {
    double span = (double)d_hi - (double)d_lo;
    double v = (double)d_lo + span * ldexp((double)j, -L);
    return (float)v;
}

__device__ __forceinline__ bool inside(float xw, float yw, float Wf, float Hf) {
    return xw >= 0.0f && xw < Wf && yw >= 0.0f && yw < Hf;
}

// floor(v) as an integer in one instruction (saturating for huge |v|,
// which only ever means "outside the image").
__device__ __forceinline__ int cvt_flr(float v) {
    int r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(v));
    return r;
}

// floor of v clamped to [-1, hi]: -1 and hi both mean "outside the image"
// (floor commutes with clamping to integer limits).
__device__ __forceinline__ int flr_clamp(float v, int hi) {
    return cvt_flr(__builtin_amdgcn_fmed3f(v, -1.0f, (float)hi));
}

__device__ __forceinline__ unsigned umax(unsigned a, unsigned b) { return a > b ? a : b; }

__device__ __forceinline__ i128 mk128(long long hi, unsigned long long lo) {
    unsigned __int128 u = ((unsigned __int128)(unsigned long long)hi << 64) | (unsigned __int128)lo;
    return (i128)u;
}

__device__ __forceinline__ void sp128(i128 v, long long& hi, unsigned long long& lo) {
    unsigned __int128 u = (unsigned __int128)v;
    lo = (unsigned long long)u;
    hi = (long long)(unsigned long long)(u >> 64);
}

// Correctly rounded conversion of a 128-bit integer to double: the top 64
// significant bits, with a sticky bit for any below them, are converted
// (one rounding) and scaled by a power of two (exact).
__device__ __forceinline__ double i128_to_double(i128 v) {
    const bool neg = v < 0;
    const unsigned __int128 u = neg ? (unsigned __int128)0 - (unsigned __int128)v : (unsigned __int128)v;
    const unsigned long long hi = (unsigned long long)(u >> 64);
    double r;
    if (hi == 0) {
        r = (double)(unsigned long long)u;
    } else {
        const int sh = 64 - __clzll(hi);
        unsigned long long top = (unsigned long long)(u >> sh);
        top |= (u & ((((unsigned __int128)1) << sh) - 1)) != 0 ? 1ull : 0ull;
        r = ldexp((double)top, sh);
    }
    return neg ? -r : r;
}

// A float no smaller than v >= 0 (the double is within 2^-53 of v, the
// float within 2^-24 of the double, the factor covers both).
__device__ __forceinline__ float ub_float(i128 v) { return (float)(i128_to_double(v) * (1.0 + 0x1p-20)); }

// The smallest integer no smaller than the finite f >= 0.
__device__ __forceinline__ i128 ceil_i128(float f) {
    int e;
    const float m = frexpf(f, &e);  // f = m 2^e, m in [0.5, 1)
    const long long mi = (long long)ldexpf(m, 24);  // f = mi 2^(e - 24) exactly
    const int sh = e - 24;
    if (sh >= 0) return (i128)mi << sh;
    if (sh < -24) return mi > 0 ? (i128)1 : (i128)0;
    return ((i128)mi + (((i128)1 << -sh) - 1)) >> -sh;
}

__device__ __forceinline__ bool improvable(i128 key, unsigned ja, i128 Kinc, unsigned jinc) {
    return key > Kinc || (key == Kinc && (unsigned long long)ja + 1ull < (unsigned long long)jinc);
}

__device__ __forceinline__ int bitlen128(i128 v) {
    unsigned __int128 u = (unsigned __int128)v;
    unsigned long long hi = (unsigned long long)(u >> 64), lo = (unsigned long long)u;
    if (hi) return 128 - __clzll(hi);
    if (lo) return 64 - __clzll(lo);
    return 0;
}

// One step of a DPP wave reduction of a 64-bit value: add the value that
// DPP control CTRL routes to this lane (rows outside ROWMASK add zero).
template <int CTRL, int ROWMASK>
__device__ __forceinline__ unsigned long long dpp_add(unsigned long long v) {
    const unsigned lo = __builtin_amdgcn_update_dpp(0u, (unsigned)v, CTRL, ROWMASK, 0xf, false);
    const unsigned hi = __builtin_amdgcn_update_dpp(0u, (unsigned)(v >> 32), CTRL, ROWMASK, 0xf, false);
    return v + (((unsigned long long)hi << 32) | lo);
}

// The same for a 32-bit value whose wave total fits 32 bits.
__device__ __forceinline__ unsigned wave_total32(unsigned v) {
    v += __builtin_amdgcn_update_dpp(0u, v, 0xB1, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0u, v, 0x4E, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0u, v, 0x141, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0u, v, 0x140, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0u, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0u, v, 0x143, 0xc, 0xf, false);
    return v;
}

// Sum over the 64 lanes of a wave in registers (no LDS): quad swaps, half-row
// and row mirrors give every lane its row's sum; the two row broadcasts then
// carry rows 0-2 into row 3.  The total is valid in lane 63 (all lanes active).
__device__ __forceinline__ unsigned long long wave_total(unsigned long long v) {
    v = dpp_add<0xB1, 0xf>(v);   // quad_perm [1,0,3,2]
    v = dpp_add<0x4E, 0xf>(v);   // quad_perm [2,3,0,1]
    v = dpp_add<0x141, 0xf>(v);  // row_half_mirror
    v = dpp_add<0x140, 0xf>(v);  // row_mirror
    v = dpp_add<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    return v;
}

// ------------------------------------------------------------ window params

// Walk-length classes: inside a tile segment, events are ordered by
// |ax| + |ay| (longest first).  For any interval an event's staircase walk
// is about (|ax| + |ay|)(r_b - r_a) pixels long, so neighbouring lanes of a
// wave then walk similar distances.
constexpr int kNB = 16;
// Guests keep half as many walk classes (kNB / 2 per guest bin).
constexpr int kNG = kNB / 2;
// Prep counters of one tile segment: owned by walk class, then guests by
// bin and walk class, so a segment holds its owned events first and its
// guest bins in increasing order.
constexpr int kTC = kNB + kGuestBins * kNG;

// Guest bin cuts of a window, uniform over its binning range [r_lo, r_hi]
// and non-decreasing whatever the rounding.
__device__ __forceinline__ void set_guest_cuts(WinParam& p) {
    const float span = p.r_hi - p.r_lo;
    float prev = p.r_lo;
    for (int m = 1; m < kGuestBins; ++m) {
        prev = fmaxf(prev, fmaf((float)m * (1.0f / kGuestBins), span, p.r_lo));
        p.gcut[m - 1] = prev;
    }
}

__global__ void k_winparam(const float* __restrict__ tau, const long long* __restrict__ offsets, int B,
                           float d_lo, float d_hi, int W, int H, float cx, float cy, WinParam* __restrict__ wp) {
    int w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= B) return;
    WinParam p;
    p.tau = tau[w];
    p.r_lo = rate_of(d_lo, p.tau);
    p.r_hi = rate_of(d_hi, p.tau);
    const float key_max = (fmaxf(fabsf(cx), fabsf((float)W - cx)) + fmaxf(fabsf(cy), fabsf((float)H - cy))) * p.tau;
    p.kscale = key_max > 0.0f ? (float)kNB / key_max : 0.0f;
    p.n_events = offsets[w + 1] - offsets[w];
    set_guest_cuts(p);
    wp[w] = p;
}

hipError_t launch_winparam(hipStream_t s, const Geometry& g, const float* tau, const long long* offsets, int B,
                           float d_lo, float d_hi, WinParam* wp) {
    if (B <= 0) return hipSuccess;
    k_winparam<<<(B + 255) / 256, 256, 0, s>>>(tau, offsets, B, d_lo, d_hi, g.W, g.H, g.cx, g.cy, wp);
    return hipGetLastError();
}

// ------------------------------------------------------------ prep (a1)

// Window of block b: the largest w with blk_start[w] <= b.
__device__ __forceinline__ int window_of_block(const int* blk_start, int B, int b) {
    int lo = 0, hi = B;
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (blk_start[mid] <= b) lo = mid; else hi = mid;
    }
    return lo;
}

__device__ __forceinline__ int walk_class(float ax, float ay, float kscale) {
    int b = (int)((fabsf(ax) + fabsf(ay)) * kscale);
    return kNB - 1 - min(max(b, 0), kNB - 1);
}

// counters of an owned event and of a guest copy in bin m, inside a window
__device__ __forceinline__ int ctr_own(int t, int b) { return t * kTC + b; }
__device__ __forceinline__ int ctr_guest(int t, int m, int b) { return t * kTC + kNB + m * kNG + (b >> 1); }

// Cuts at which one coordinate of an event, warped by the evaluation's own
// fmaf (v + a r), is still short of the edge e of a band, e being the edge
// the coordinate moves towards as the rate grows (the lower one for a >= 0).
// The test is monotone in the rate, so the cuts at which it holds come
// first.  A guest copy's bin is the larger of its two coordinates' counts:
// the event has not reached the tile while either coordinate is short, and
// the union of two leading runs of cuts is the longer one.  A bin-m copy
// evaluated at rates that are all at most gcut[m - 1] lies outside the tile
// at both ends, on the same side, and adds only to the tile's border.
__device__ __forceinline__ int cuts_short(const WinParam& p, float v, float a, float e) {
    const bool neg = a < 0.0f;
    int m = 0;
#pragma unroll
    for (int k = 0; k < kGuestBins - 1; ++k) m += ((fmaf(a, p.gcut[k], v) < e) != neg) ? 1 : 0;
    return m;
}

// Band edges of the tile grid as floats, in LDS for the prep blocks.
struct PrepCuts {
    float col[kMaxTiles + 1], row[kMaxTiles + 1];
};

__device__ __forceinline__ void load_cuts(const Geometry& g, PrepCuts& c) {
    for (int k = threadIdx.x; k <= g.ntx; k += blockDim.x) c.col[k] = (float)g.colcut[k];
    for (int k = threadIdx.x; k <= g.nty; k += blockDim.x) c.row[k] = (float)g.rowcut[k];
}

// First segment of an event's image: the polarity-aware contrast keeps one
// event image per polarity (p > 0: the second), each tiled alike.
__device__ __forceinline__ int seg_base(const Geometry& g, int pol) { return pol > 0 ? g.nsp : 0; }

// Per-event prep: validity, (ax, ay), reachable tiles and walk class.
struct PrepEv {
    bool ok, valid;
    float x, y, ax, ay;
    int tx0, tx1, ty0, ty1, cls;
};

// Counter of a prepared event's own copy (the one N_low and the certificates
// read; segment base sb): it goes to the tile the event starts in, at the low
// end of the binning range, the corner of its tile rectangle it moves away
// from.  Every other tile is a guest, reached at higher rates only.
__device__ __forceinline__ int own_copy(const Geometry& g, int sb, const PrepEv& e) {
    return ctr_own(sb + (e.ay < 0.0f ? e.ty1 : e.ty0) * g.ntx + (e.ax < 0.0f ? e.tx1 : e.tx0), e.cls);
}

// Counters of its guest copies, in the same order for the counting and the
// scattering passes.
template <class F>
__device__ __forceinline__ void for_each_guest(const Geometry& g, const WinParam& p, const PrepCuts& c, int sb,
                                               const PrepEv& e, F&& f) {
    if (e.tx0 == e.tx1 && e.ty0 == e.ty1) return;
    const int ox = e.ax < 0.0f ? e.tx1 : e.tx0, oy = e.ay < 0.0f ? e.ty1 : e.ty0;
    for (int ty = e.ty0; ty <= e.ty1; ++ty) {
        const int by = cuts_short(p, e.y, e.ay, c.row[e.ay < 0.0f ? ty + 1 : ty]);
        for (int tx = e.tx0; tx <= e.tx1; ++tx) {
            if (ty == oy && tx == ox) continue;
            const int bx = cuts_short(p, e.x, e.ax, c.col[e.ax < 0.0f ? tx + 1 : tx]);
            f(ctr_guest(sb + ty * g.ntx + tx, max(bx, by), e.cls));
        }
    }
}

// All but the tiles: tx0 .. ty1 are the pixels of the box that the event
// spans over the whole search range (clamped to the image), and ok is false
// when that box misses the image.
__device__ __forceinline__ PrepEv prep_box(const Geometry& g, const WinParam& p, float xv, float yv, float tv) {
    PrepEv e;
    e.valid = isfinite(xv) && isfinite(yv) && tv >= 0.0f && tv <= p.tau;
    e.ok = false;
    e.tx0 = e.tx1 = e.ty0 = e.ty1 = 0;
    if (!e.valid) return e;
    const float ux = xv - g.cx, uy = yv - g.cy, delta = p.tau - tv;
    e.x = xv;
    e.y = yv;
    e.ax = ux * delta;
    e.ay = uy * delta;
    const float xa = fmaf(e.ax, p.r_lo, xv), xb = fmaf(e.ax, p.r_hi, xv);
    const float ya = fmaf(e.ay, p.r_lo, yv), yb = fmaf(e.ay, p.r_hi, yv);
    const int kx0 = flr_clamp(fminf(xa, xb), g.W), kx1 = flr_clamp(fmaxf(xa, xb), g.W);
    const int ky0 = flr_clamp(fminf(ya, yb), g.H), ky1 = flr_clamp(fmaxf(ya, yb), g.H);
    e.ok = !(kx1 < 0 || kx0 > g.W - 1 || ky1 < 0 || ky0 > g.H - 1);
    e.tx0 = max(kx0, 0);
    e.ty0 = max(ky0, 0);
    e.tx1 = min(kx1, g.W - 1);
    e.ty1 = min(ky1, g.H - 1);
    e.cls = walk_class(e.ax, e.ay, p.kscale);
    return e;
}

// The tiles of N prepared boxes.  The cuts increase: a band is the count of
// inner cuts at or below the pixel, and each cut is read (as a scalar) once
// for all the thread's events.
template <int N>
__device__ __forceinline__ void prep_tiles(const Geometry& g, PrepEv (&e)[N]) {
    int x0[N] = {}, x1[N] = {}, y0[N] = {}, y1[N] = {};
    for (int k = 1; k < g.ntx; ++k) {
        const int c = g.colcut[k];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            x0[j] += c <= e[j].tx0 ? 1 : 0;
            x1[j] += c <= e[j].tx1 ? 1 : 0;
        }
    }
    for (int k = 1; k < g.nty; ++k) {
        const int c = g.rowcut[k];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            y0[j] += c <= e[j].ty0 ? 1 : 0;
            y1[j] += c <= e[j].ty1 ? 1 : 0;
        }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        e[j].tx0 = x0[j];
        e[j].tx1 = x1[j];
        e[j].ty0 = y0[j];
        e[j].ty1 = y1[j];
    }
}

// Prep workgroups: kPrepPer events per thread, held in registers between the
// counting and the writing.  1024 threads share the chunk's zeroing of the
// counters and its cursor atomics (up to kMaxTiles * kTC of each); with fewer
// events there are too few such chunks to fill the CUs, and 256 threads are
// faster (count / scatter, before prep_tiles: 20M events in 24 tiles 141 / 214 us with 1024
// threads, 165 / 289 with 256; 2M in 8 tiles 24 / 34.8 and 21.6 / 31.0; one
// window of 10k 6.2 / 6.8 with 256, 20 / 34 with chunks of 4096).  Eight
// events per thread: 137 / 306 us for the 20M.
constexpr int kPrepPer = 4, kPrepMany = 1024, kPrepSome = 256;
constexpr long long kPrepFew = 1 << 22;

// A thread's PER events of a chunk, all loads in flight; past the chunk's n
// events the last one again.
template <int PER>
struct PrepIn {
    float x[PER], y[PER], t[PER];
    int p[PER];
    template <int NT>
    __device__ __forceinline__ void load(const float* xs, const float* ys, const float* ts, const signed char* ps,
                                         long long beg, int n) {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const long long i = beg + min(j * NT + (int)threadIdx.x, n - 1);
            x[j] = xs[i];
            y[j] = ys[i];
            t[j] = ts[i];
            p[j] = ps ? ps[i] : 0;
        }
    }
};

// Bound by instructions: the boxes, the tile bands and, for the wave's events
// with guests, their bins (20M events in 24 tiles: 141 us with the cuts read
// and the bands counted event by event, 108 with each cut read once for the
// thread's four; 80M: 641 and 484).
template <int NT, int PER>
__global__ __launch_bounds__(NT) void k_prep_count(
    Geometry g, const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ t_rel,
    const signed char* __restrict__ pol, const long long* __restrict__ offsets, const WinParam* __restrict__ wp, int B,
    const int* __restrict__ blk_start, int* __restrict__ cnt, int* __restrict__ err_flag) {
    extern __shared__ int s_cnt[];  // g.T * kTC counters
    __shared__ PrepCuts s_cuts;
    const int blk = blockIdx.x;
    if (blk >= blk_start[B]) return;  // a grid sized for the largest batch
    const int nc = g.T * kTC;
    for (int k = threadIdx.x; k < nc; k += NT) s_cnt[k] = 0;
    load_cuts(g, s_cuts);
    __syncthreads();
    const int w = window_of_block(blk_start, B, blk);
    const long long beg = offsets[w] + (long long)(blk - blk_start[w]) * (NT * PER);
    const int n = (int)min((long long)(NT * PER), offsets[w + 1] - beg);  // >= 1
    const WinParam p = wp[w];
    PrepIn<PER> in;
    in.template load<NT>(x, y, t_rel, pol, beg, n);
    PrepEv e[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) e[j] = prep_box(g, p, in.x[j], in.y[j], in.t[j]);
    prep_tiles(g, e);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (j * NT + (int)threadIdx.x >= n) break;
        if (!e[j].valid) atomicOr(&err_flag[w], 1);
        if (!e[j].ok) continue;
        const int sb = seg_base(g, in.p[j]);
        atomicAdd(&s_cnt[own_copy(g, sb, e[j])], 1);
        for_each_guest(g, p, s_cuts, sb, e[j], [&](int k) { atomicAdd(&s_cnt[k], 1); });
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nc; k += NT)
        if (s_cnt[k]) atomicAdd(&cnt[(long long)w * nc + k], s_cnt[k]);
}

// Exclusive scan of the counters of every (window, tile, owned/guest bin,
// class) in that order (one workgroup); then the segment of (w, t) starts at
// its first counter, its owned events end where its first guest bin begins,
// and guest bin m ends where bin m + 1 (or the next segment) begins.  The
// rounds are a chain of load, scan and barrier, so each takes kScanPer int4
// per thread, in rows of 64 neighbouring ones, and loads the next round's
// before it scans: 64 windows of 24 tiles (73728 counters) take 41 us
// (a CU's bandwidth), one counter per thread and round took 127.
constexpr int kScanPer = 4;
static_assert(kTC % 4 == 0, "the counters are read four at a time");
__global__ __launch_bounds__(1024) void k_prep_scan(int B, int T, const int* __restrict__ cnt,
                                                    long long* __restrict__ seg_off, int* __restrict__ seg_own,
                                                    unsigned long long* __restrict__ cursor) {
    __shared__ long long s_wave[2][16];
    const long long n4 = (long long)B * T * kTC / 4, n = 4 * n4;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int4* const c4 = reinterpret_cast<const int4*>(cnt);
    const long long first = wv * 64 * kScanPer + lane;
    int4 c[kScanPer], cn[kScanPer];
#pragma unroll
    for (int j = 0; j < kScanPer; ++j) cn[j] = first + 64 * j < n4 ? c4[first + 64 * j] : make_int4(0, 0, 0, 0);
    long long total = 0;
    int turn = 0;
    for (long long base = 0; base < n4; base += 1024 * kScanPer, turn ^= 1) {
        const long long k = base + first;
        long long v[kScanPer];  // inclusive sums of the row's lanes
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) {
            c[j] = cn[j];
            const long long kn = k + 1024 * kScanPer + 64 * j;
            cn[j] = kn < n4 ? c4[kn] : make_int4(0, 0, 0, 0);
            v[j] = (long long)c[j].x + c[j].y + c[j].z + c[j].w;
        }
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
#pragma unroll
            for (int j = 0; j < kScanPer; ++j) {
                const long long a = __shfl_up(v[j], o, 64);
                if (lane >= o) v[j] += a;
            }
        }
        long long row[kScanPer], wave = 0;  // before each row of the wave
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) {
            row[j] = wave;
            wave += __shfl(v[j], 63, 64);
        }
        // two rows: the one written here was last read before the barrier
        // of the round between
        if (lane == 0) s_wave[turn][wv] = wave;
        __syncthreads();
        long long pre = total;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const long long a = s_wave[turn][j];
            if (j < wv) pre += a;
            total += a;
        }
#pragma unroll
        for (int j = 0; j < kScanPer; ++j) {
            if (k + 64 * j >= n4) break;
            ulonglong2* const q = reinterpret_cast<ulonglong2*>(cursor + 4 * (k + 64 * j));
            const long long r3 = pre + row[j] + v[j] - c[j].w, r2 = r3 - c[j].z, r1 = r2 - c[j].y;
            q[0] = make_ulonglong2(r1 - c[j].x, r1);
            q[1] = make_ulonglong2(r2, r3);
        }
    }
    __syncthreads();  // every cursor is visible
    const auto start = [&](long long k) { return k < n ? (long long)cursor[k] : total; };
    for (int st = threadIdx.x; st < B * T; st += 1024) {
        const long long c0 = (long long)st * kTC;
        const long long o0 = start(c0);
        seg_off[st] = o0;
        int* const so = seg_own + (long long)st * (kGuestBins + 1);
        so[0] = (int)(start(c0 + kNB) - o0);
        for (int m = 0; m < kGuestBins; ++m) so[1 + m] = (int)(start(c0 + kNB + (m + 1) * kNG) - o0);
    }
    if (threadIdx.x == 0) seg_off[(long long)B * T] = total;
}

// The same events again; an owned record's rank in its run is what the
// counting atomic returned, and the events stay in registers, so nothing is
// read or worked out a third time (20M events in 24 tiles: 434 -> 195 us, 80M:
// 2160 -> 977).  Only the few guests are counted and then ranked.
template <int NT, int PER>
__global__ __launch_bounds__(NT) void k_prep_scatter(
    Geometry g, const float* __restrict__ x, const float* __restrict__ y, const float* __restrict__ t_rel,
    const signed char* __restrict__ pol, const long long* __restrict__ offsets, const WinParam* __restrict__ wp, int B,
    const int* __restrict__ blk_start, unsigned long long* __restrict__ cursor, const long long* __restrict__ total,
    long long cap, float4* __restrict__ ev) {
    extern __shared__ unsigned long long s_prep[];  // g.T * kTC bases, then as many counts
    const int nc = g.T * kTC;
    unsigned long long* const s_base = s_prep;
    int* const s_cnt = reinterpret_cast<int*>(s_prep + nc);
    __shared__ PrepCuts s_cuts;
    const int blk = blockIdx.x;
    if (blk >= blk_start[B]) return;  // a grid sized for the largest batch
    if (total && *total > cap) return;  // the records would not fit the store: nothing is written
    load_cuts(g, s_cuts);
    for (int k = threadIdx.x; k < nc; k += NT) s_cnt[k] = 0;
    __syncthreads();
    const int w = window_of_block(blk_start, B, blk);
    const long long beg = offsets[w] + (long long)(blk - blk_start[w]) * (NT * PER);
    const int n = (int)min((long long)(NT * PER), offsets[w + 1] - beg);  // >= 1
    const WinParam p = wp[w];
    PrepIn<PER> in;
    in.template load<NT>(x, y, t_rel, pol, beg, n);
    PrepEv e[PER];
    int sb[PER], rank[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) e[j] = prep_box(g, p, in.x[j], in.y[j], in.t[j]);
    prep_tiles(g, e);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        e[j].ok = e[j].ok && j * NT + (int)threadIdx.x < n;
        if (!e[j].ok) continue;
        sb[j] = seg_base(g, in.p[j]);
        rank[j] = atomicAdd(&s_cnt[own_copy(g, sb[j], e[j])], 1);
        for_each_guest(g, p, s_cuts, sb[j], e[j], [&](int k) { atomicAdd(&s_cnt[k], 1); });
    }
    __syncthreads();
    // the owned events have their ranks; the guests are counted again
    for (int k = threadIdx.x; k < nc; k += NT) {
        const int m = s_cnt[k];
        s_base[k] = m ? atomicAdd(&cursor[(long long)w * nc + k], (unsigned long long)m) : 0ull;
        s_cnt[k] = 0;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (!e[j].ok) continue;
        const float4 v = make_float4(e[j].x, e[j].y, e[j].ax, e[j].ay);
        ev[s_base[own_copy(g, sb[j], e[j])] + (unsigned long long)rank[j]] = v;
        for_each_guest(g, p, s_cuts, sb[j], e[j], [&](int k) {
            const int r = atomicAdd(&s_cnt[k], 1);
            ev[s_base[k] + (unsigned long long)r] = v;
        });
    }
}

// Events per prep workgroup.
int prep_chunk(long long max_events) { return (max_events < kPrepFew ? kPrepSome : kPrepMany) * kPrepPer; }

__global__ void k_begin(const unsigned* __restrict__ staged, unsigned* __restrict__ head, int n_head,
                        int* __restrict__ cnt, long long nctr, int* __restrict__ err_flag, int B,
                        Queue* __restrict__ q, int* __restrict__ n_active) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_head) head[i] = staged[i];
    if (i < nctr) cnt[i] = 0;
    if (i < B) err_flag[i] = 0;
    if (q && i < kQueues) {
        q[i].n_items = 0;
        q[i].next = 0;
    }
    if (n_active && i == 0) *n_active = 0;
}

hipError_t launch_begin(hipStream_t s, const unsigned* staged, unsigned* head, int n_head, int* cnt, long long nctr,
                        int* err_flag, int B, Queue* q, int* n_active) {
    const long long n = std::max(std::max((long long)n_head, nctr), (long long)std::max(B, kQueues));
    k_begin<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(staged, head, n_head, cnt, nctr, err_flag, B, q, n_active);
    return hipGetLastError();
}

__global__ void k_fetch(const unsigned* __restrict__ a, unsigned* __restrict__ ha, int na,
                        const unsigned* __restrict__ b, unsigned* __restrict__ hb, int nb) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < na) ha[i] = a[i];
    if (i < nb) hb[i] = b[i];
}

hipError_t launch_fetch(hipStream_t s, const unsigned* a, unsigned* ha, int na, const unsigned* b, unsigned* hb,
                        int nb) {
    k_fetch<<<(std::max(na, nb) + 255) / 256, 256, 0, s>>>(a, ha, na, b, hb, nb);
    return hipGetLastError();
}

// 64 windows' states per workgroup
__global__ __launch_bounds__(256) void k_report(int B, const long long* __restrict__ records,
                                                const int* __restrict__ n_active, const int* __restrict__ err_flag,
                                                const WinState* __restrict__ st, int all, Report* __restrict__ rep,
                                                WinState* __restrict__ hs) {
    __shared__ int s_bad;
    const int finished = n_active ? *n_active : 0;
    if (blockIdx.x == 0) {
        if (threadIdx.x == 0) s_bad = B;
        __syncthreads();
        if (err_flag)
            for (int w = threadIdx.x; w < B; w += 256)
                if (err_flag[w]) atomicMin(&s_bad, w);
        __syncthreads();
        if (threadIdx.x == 0) {
            rep->records = *records;
            rep->finished = finished;
            rep->bad = s_bad;
        }
    }
    if (st && (all || finished + B == 0)) {
        static_assert(sizeof(WinState) % 8 == 0, "copied in 8-byte words");
        constexpr long long words = sizeof(WinState) / 8;
        const unsigned long long* const src = reinterpret_cast<const unsigned long long*>(st);
        unsigned long long* const dst = reinterpret_cast<unsigned long long*>(hs);
        const long long end = min((long long)B, 64ll * (blockIdx.x + 1)) * words;
        for (long long k = 64ll * blockIdx.x * words + threadIdx.x; k < end; k += 256) dst[k] = src[k];
    }
}

hipError_t launch_report(hipStream_t s, int B, const long long* records, const int* n_active, const int* err_flag,
                         const WinState* st, int all, Report* rep, WinState* hs) {
    k_report<<<st ? (B + 63) / 64 : 1, 256, 0, s>>>(B, records, n_active, err_flag, st, all, rep, hs);
    return hipGetLastError();
}

size_t prep_counters(int B, int T) { return (size_t)B * T * kTC; }
size_t seg_own_words(int B, int T) { return (size_t)B * T * (kGuestBins + 1); }

template <int NT, int PER>
static void prep_pass(hipStream_t s, int phase, const Geometry& g, const float* x, const float* y, const float* t_rel,
                      const signed char* pol, const long long* offsets, const WinParam* wp, int B,
                      const int* blk_start, int nblk, int* cnt, long long* seg_off, unsigned long long* cursor,
                      float4* ev, int* err_flag, long long cap) {
    if (phase == 0)
        k_prep_count<NT, PER><<<nblk, NT, sizeof(int) * g.T * kTC, s>>>(g, x, y, t_rel, pol, offsets, wp, B, blk_start,
                                                                        cnt, err_flag);
    else
        k_prep_scatter<NT, PER><<<nblk, NT, (sizeof(unsigned long long) + sizeof(int)) * g.T * kTC, s>>>(
            g, x, y, t_rel, pol, offsets, wp, B, blk_start, cursor,
            cap >= 0 ? seg_off + (long long)B * g.T : nullptr, cap, ev);
}

hipError_t launch_prep(hipStream_t s, int phase, const Geometry& g, const float* x, const float* y,
                       const float* t_rel, const signed char* pol, const long long* offsets, const WinParam* wp, int B,
                       const int* blk_start, int nblk, int chunk, int* cnt, long long* seg_off, int* seg_own,
                       unsigned long long* cursor, float4* ev, int* err_flag, long long cap) {
    if (nblk > 0) {
        if (chunk == kPrepSome * kPrepPer)
            prep_pass<kPrepSome, kPrepPer>(s, phase, g, x, y, t_rel, pol, offsets, wp, B, blk_start, nblk, cnt, seg_off, cursor, ev,
                              err_flag, cap);
        else
            prep_pass<kPrepMany, kPrepPer>(s, phase, g, x, y, t_rel, pol, offsets, wp, B, blk_start, nblk, cnt, seg_off,
                                      cursor, ev, err_flag, cap);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (phase == 0) {
        k_prep_scan<<<1, 1024, 0, s>>>(B, g.T, cnt, seg_off, seg_own, cursor);
        return hipGetLastError();
    }
    return hipSuccess;
}

// ------------------------------------------------------------ evaluation (a2, a3)

// Add one to every pixel of this tile that the staircase walk from pixel
// (kx, ky) to pixel (kxb, kyb) visits (eq. (17)); the start pixel is
// counted by the caller.  While both coordinates still move each step takes
// the corner test below; once one has reached its end the rest is a straight
// run with no test (the two loops visit exactly the pixels of one loop that
// tests every step, and skip its fp64 work on the run).  Corner decisions follow the event's ray through
// (x, y) with direction (ax, ay), in fp64: e = |X - x||ay| - |Y - y||ax|
// compares where the ray meets the next vertical and horizontal pixel
// edges; within 2^-8 px of the corner both side pixels are counted.
// Increments do not return the old count, so no step waits on the LDS;
// the item's sum of squares and its count of increments come from one pass
// over the tile afterwards (no walk counts its own steps).
// The corner test computes X - x as kx - (x - 1) or kx - x (the edge ahead
// is kx + 1 or kx), the same fp64 value as X - x, so decisions do not change.
// Pixels outside the tile are clamped onto its one-cell border (`Ring`),
// whose counts are removed at the end.

// The tile's counters in LDS with a one-cell border: pixel (kx, ky), clamped
// to [xlo, xhi] x [ylo, yhi] = [x0 - 1, x0 + tw] x [y0 - 1, y0 + th], is
// counter ky * rw + kx + base, rw = tw + 2.  Border counters collect every
// increment outside the tile (other tiles, outside the image).  `org` is
// the counter array shifted by base (org[ky * rw + kx] is pixel (kx, ky)),
// so an address is one 24-bit mad and one shift-add.
struct Ring {
    int xlo, xhi, ylo, yhi;
    int rw, base;
    int vxhi, vyhi;  // xhi, yhi held in vector registers (the clamp takes one scalar operand)
};

// v copied into a vector register that the compiler keeps (rather than
// copying it again before every use)
__device__ __forceinline__ int to_vgpr(int v) {
    int r;
    asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "s"(v));
    return r;
}

// a * b + c for 24-bit signed a, b in one instruction, b uniform (left to
// itself the compiler scales both terms of the index separately)
__device__ __forceinline__ int mad24(int a, int b, int c) {
    int r;
    asm("v_mad_i32_i24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(b), "v"(c));
    return r;
}

// v clamped to [lo, hi] (lo <= hi, lo uniform) in one instruction
__device__ __forceinline__ int clampi(int v, int lo, int hi) {
    int r;
    asm("v_med3_i32 %0, %1, %2, %3" : "=v"(r) : "v"(v), "s"(lo), "v"(hi));
    return r;
}

__device__ __forceinline__ unsigned* ring_at(unsigned* org, const Ring& R, int kx, int ky) {
    return org + mad24(ky, R.rw, kx);
}

__device__ __forceinline__ void lds_inc(unsigned* p) {
    atomicAdd(p, 1u);  // the old count is not used: no wait for it
}

__device__ __forceinline__ void tile_add(unsigned* org, const Ring& R, int px, int py) {
    const int cx = clampi(px, R.xlo, R.vxhi), cy = clampi(py, R.ylo, R.vyhi);
    lds_inc(ring_at(org, R, cx, cy));
}

__device__ __forceinline__ void walk_tile(unsigned* org, const Ring& R, int kx, int ky, int kxb,
                                          int kyb, float xf, float yf, float axf, float ayf) {
    // a single step along a row or a column (|dx| + |dy| = 1, i.e.
    // dx^2 + dy^2 = 1) has no corner to test: it visits the end pixel only
    // (the coordinates are clamped to [-1, W] x [-1, H], so the squares are
    // 24-bit products)
    {
        const int dx = kxb - kx, dy = kyb - ky;
        if (__mul24(dx, dx) + __mul24(dy, dy) == 1) {
            tile_add(org, R, kxb, kyb);
            return;
        }
    }
    // step direction of each coordinate (not used once it is at its end)
    const bool px = kxb > kx, py = kyb > ky;
    const int sx = px ? 1 : -1, sy = py ? 1 : -1;
    if (kx != kxb && ky != kyb) {
        // the edges ahead are X = kx + px and Y = ky + py; with the origin
        // moved to (x - px, y - py) (exact in fp64), X - x = kx - xo exactly
        const double xo = (double)xf - (px ? 1.0 : 0.0), yo = (double)yf - (py ? 1.0 : 0.0);
        const double aax = fabs((double)axf), aay = fabs((double)ayf);
        const double thr = (aax + aay) * 0.00390625;
        // both coordinates still move: which edge does the ray meet first
        do {
            const double ex = fabs((double)kx - xo) * aay;
            const double ey = fabs((double)ky - yo) * aax;
            const double e = ex - ey;
            const bool lo = e < -thr, hi = e > thr;
            if (!lo && !hi) {  // the ray passes near the corner: both side pixels
                tile_add(org, R, kx + sx, ky);
                tile_add(org, R, kx, ky + sy);
            }
            kx += !hi ? sx : 0;
            ky += !lo ? sy : 0;
            tile_add(org, R, kx, ky);
        } while (kx != kxb && ky != kyb);
    }
    // one coordinate left: a straight run along a row or a column
    if (kx != kxb) {
        const int cy = clampi(ky, R.ylo, R.vyhi);
        do {
            kx += sx;
            lds_inc(org + mad24(cy, R.rw, clampi(kx, R.xlo, R.vxhi)));
        } while (kx != kxb);
    } else {
        const int cx = clampi(kx, R.xlo, R.vxhi);
        while (ky != kyb) {
            ky += sy;
            lds_inc(org + mad24(clampi(ky, R.ylo, R.vyhi), R.rw, cx));
        }
    }
}

// LDS layout of k_eval: [tile with its border: (tw + 2)(th + 2) counters]
// (region rounded up to 16 bytes)[reduction scratch][queue sizes, 4 bytes spare].  The
// reduction scratch is sized for the largest workgroup (1024 threads).
constexpr int kEvalWaves = kEvalThreads / 64;

// Counter words of the LDS tile region for tiles of up to ring_px counters
// (border included), rounded up to whole 16-byte units so the clear can use
// 16-byte stores.
__host__ __device__ __forceinline__ int eval_counter_words(int ring_px) { return (ring_px + 3) & ~3; }

size_t eval_lds_bytes(int ring_px) {
    return (size_t)eval_counter_words(ring_px) * 4 + 3 * kEvalWaves * 8 + 4 * (1 + kXcd);
}

// Persistent evaluation kernel: each workgroup takes work items (a window's
// tile segment and one or more hypotheses) from the queue until it is
// empty.  For each hypothesis it bins the tile's events in LDS (point: one
// increment per event, interval: one per pixel of the walk) with atomic adds
// that return nothing, then removes the border counters' share and sums the
// squares of the tile's counters in one 16-byte-wide pass that also zeroes
// them for the next hypothesis (the tile region is cleared once, at start).
// An interval takes the segment's owned events, then its guest copies,
// skipping a guest whose walk box misses the tile (all its increments would
// land on the border).  Points and intervals read the guest bins whose lower
// cut lies below the hypothesis's larger rate only (the others are short of
// the tile at every rate it takes).  An endpoint certificate reads the owned
// events only and touches no counter.
template <int NT>
__global__ __launch_bounds__(NT) void k_eval(
    Geometry g, const float4* __restrict__ ev, const long long* __restrict__ seg_off,
    const int* __restrict__ seg_own, const WinParam* __restrict__ wp, const Hyp* __restrict__ hyps,
    const int* __restrict__ act, const Item* __restrict__ items, int qcap, Queue* __restrict__ q, Queue* __restrict__ q_reset,
    Part* __restrict__ part, int HS, unsigned* __restrict__ img_out) {
    constexpr int NW = NT / 64;
    extern __shared__ __align__(16) unsigned smem[];
    const int tid = threadIdx.x;
    unsigned* const tile = smem;
    unsigned long long* const s_red =
        reinterpret_cast<unsigned long long*>(smem + eval_counter_words(g.ring_px));
    // the work item, in the scratch between the hypotheses' sums (thread 0
    // alone has read them last)
    long long* const s_item = reinterpret_cast<long long*>(s_red);
    if (blockIdx.x == 0 && tid < kXcd && q_reset) {
        q_reset[tid].n_items = 0;
        q_reset[tid].next = 0;
    }
    {  // nothing queued (the rounds after the last step): leave before the clear
        int any = 0;
        for (int r = 0; r < kXcd; ++r) any |= q[r].n_items;
        if (any == 0) return;
    }
    {  // every counter of the tile region starts at zero and is zeroed again
       // by the pass that sums each hypothesis's squares
        uint4* const t4 = reinterpret_cast<uint4*>(tile);
        const int n4 = eval_counter_words(g.ring_px) >> 2;
        for (int i = tid; i < n4; i += NT) t4[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    const int home = blockIdx.x % kXcd;
    int qi = 0;  // queues tried so far, starting at this XCD's own (thread 0 only)
    int* const qn = reinterpret_cast<int*>(s_red + 3 * NW);  // queue sizes, read once (thread 0 only; in LDS, not registers)
    if (tid == 0)
        for (int r = 0; r < kXcd; ++r) qn[r] = q[(home + r) % kXcd].n_items;
    for (;;) {
        if (tid == 0) {
            long long got = -1;
            while (qi < kXcd) {
                const int r = (home + qi) % kXcd;
                if (qn[qi] > 0) {
                    const int k = atomicAdd(&q[r].next, 1);
                    if (k < qn[qi]) {
                        got = hyp_slot(r, k, qcap);
                        break;
                    }
                }
                ++qi;
            }
            *s_item = got;
        }
        __syncthreads();
        const long long it = *s_item;
        __syncthreads();
        if (it < 0) break;
        const Item item = items[it];
        const int w = item.w, t = item.t;
        const int ts = t % g.nsp;  // spatial tile of the segment
        const int tx = ts % g.ntx, ty = ts / g.ntx;
        const int x0 = g.colcut[tx], y0 = g.rowcut[ty];
        const int tw = g.colcut[tx + 1] - x0, th = g.rowcut[ty + 1] - y0;
        Ring R;
        R.xlo = x0 - 1;
        R.xhi = x0 + tw;
        R.ylo = y0 - 1;
        R.yhi = y0 + th;
        R.rw = tw + 2;
        R.base = -(R.ylo * R.rw + R.xlo);
        R.vxhi = to_vgpr(R.xhi);
        R.vyhi = to_vgpr(R.yhi);
        unsigned* const org = tile + R.base;   // org[ky * rw + kx]: pixel (kx, ky)
        const int ncnt = R.rw * (th + 2);       // counters, border included
        const int nring = 2 * R.rw + 2 * th;    // border counters
        const float fxlo = (float)R.xlo, fxhi = (float)R.xhi, fylo = (float)R.ylo, fyhi = (float)R.yhi;
        const long long seg = (long long)w * g.T + t;
        const long long beg = seg_off[seg];
        const int* const sown = seg_own + seg * (kGuestBins + 1);
        const float* const gcut = wp[w].gcut;
      for (int gk = 0; gk < item.cnt; ++gk) {
        const int wh = w * HS + act[w * HS + item.r0 + gk];
        const Hyp hp = hyps[wh];
        // guest bins read: those whose lower cut lies below the larger rate
        int nbin = 0;
        {
            const float rmax = fmaxf(hp.ra, hp.rb);
#pragma unroll
            for (int k = 0; k < kGuestBins - 1; ++k) nbin += gcut[k] < rmax ? 1 : 0;
        }

        unsigned long long nlow = 0;
        // the segment's events, indexed from its start with 32-bit offsets
        // (byte offsets fit 32 bits: a segment holds fewer than 2^28 events)
        const char* __restrict__ sev = reinterpret_cast<const char*>(ev + beg);
        const auto at = [sev](unsigned k) { return *reinterpret_cast<const float4*>(sev + (k << 4)); };
        const unsigned nown = (unsigned)sown[0], nseg = (unsigned)sown[1 + nbin];
        unsigned long long ucert = 0;  // certificate: walk pixels of the events inside at both ends
        if (hp.kind == HYP_CERT) {
            // Endpoint certificate of an interval (eqs. (17)-(20) without
            // the walk): the owned events only, no counter is touched.  An
            // event with both endpoint pixels in the image walks through
            // |dkx| + |dky| + 1 distinct image pixels at least.
            const float ra = hp.ra, rb = hp.rb;
            unsigned nl = 0;
            const auto one = [&](const float4& e) {
                const int kxa = flr_clamp(fmaf(e.z, ra, e.x), g.W), kya = flr_clamp(fmaf(e.w, ra, e.y), g.H);
                const int kxb = flr_clamp(fmaf(e.z, rb, e.x), g.W), kyb = flr_clamp(fmaf(e.w, rb, e.y), g.H);
                // both endpoints in the image, i.e. the far one (see the interval path)
                const bool full = ((unsigned)kxb < (unsigned)g.W) & ((unsigned)kyb < (unsigned)g.H);
                nl += full ? 1u : 0u;
                ucert += full ? (unsigned)(abs(kxb - kxa) + abs(kyb - kya) + 1) : 0u;
            };
            constexpr int U = 4;
            constexpr unsigned S = NT;
            unsigned i = tid;
            for (; i + (U - 1) * S < nown; i += U * S) {
                float4 e[U];
#pragma unroll
                for (int k = 0; k < U; ++k) e[k] = at(i + k * S);
#pragma unroll
                for (int k = 0; k < U; ++k) one(e[k]);
            }
            for (; i < nown; i += S) one(at(i));
            nlow = nl;
        } else if (hp.kind == HYP_POINT) {
            // Point hypothesis (eqs. (12)-(13)): U events per thread in
            // flight, loads first, then U increments without branches.
            const float r = hp.ra;
            constexpr int U = 4;
            constexpr unsigned S = NT;
            unsigned i = tid;
            for (; i + (U - 1) * S < nseg; i += U * S) {
                float4 e[U];
#pragma unroll
                for (int k = 0; k < U; ++k) e[k] = at(i + k * S);
                int a[U];
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    const int kx = cvt_flr(__builtin_amdgcn_fmed3f(fmaf(e[k].z, r, e[k].x), fxlo, fxhi));
                    const int ky = cvt_flr(__builtin_amdgcn_fmed3f(fmaf(e[k].w, r, e[k].y), fylo, fyhi));
                    a[k] = mad24(ky, R.rw, kx);
                }
#pragma unroll
                for (int k = 0; k < U; ++k) atomicAdd(org + a[k], 1u);
            }
            for (; i < nseg; i += S) {
                const float4 e = at(i);
                const int kx = cvt_flr(__builtin_amdgcn_fmed3f(fmaf(e.z, r, e.x), fxlo, fxhi));
                const int ky = cvt_flr(__builtin_amdgcn_fmed3f(fmaf(e.w, r, e.y), fylo, fyhi));
                atomicAdd(ring_at(org, R, kx, ky), 1u);
            }
        } else {
            // Interval hypothesis (eqs. (17)-(20)): endpoints, N_low, walk.
            const float ra = hp.ra, rb = hp.rb;
            unsigned nlow32 = 0;
            const auto one = [&](const float4& e, unsigned i) {
                const float xa = fmaf(e.z, ra, e.x), ya = fmaf(e.w, ra, e.y);
                const float xb = fmaf(e.z, rb, e.x), yb = fmaf(e.w, rb, e.y);
                const int kxa = flr_clamp(xa, g.W), kya = flr_clamp(ya, g.H);
                const int kxb = flr_clamp(xb, g.W), kyb = flr_clamp(yb, g.H);
                // both endpoints in the image, i.e. the far one (not clamped to
                // -1, huge as unsigned, nor to W, H): the warp only moves an
                // event away from the FOE as the rate grows, so an event inside
                // at rb is inside at ra <= rb
                nlow32 += (unsigned)(i < nown) & (unsigned)((unsigned)kxb < (unsigned)g.W) &
                          (unsigned)((unsigned)kyb < (unsigned)g.H);
                tile_add(org, R, kxa, kya);
                if (kxa != kxb || kya != kyb) walk_tile(org, R, kxa, kya, kxb, kyb, e.x, e.y, e.z, e.w);
            };
            // Owned events first (N_low counts them), then the guest copies:
            // a guest whose walk box for this interval misses the tile would
            // only increment the discarded border, so it is skipped, tested
            // on the warped coordinates before their floor (for an integer
            // edge e, floor(v) < e exactly when v < e, and the clamp to the
            // image cannot move a coordinate across an edge of the tile).
            // Two events in flight ahead of the one being binned (the loads
            // may read up to two strides past a range: the store is padded by
            // kEvalPad records).
            const float fx0 = (float)x0, fx1 = (float)(x0 + tw), fy0 = (float)y0, fy1 = (float)(y0 + th);
            const auto guest = [&](const float4& e, unsigned i) {
                const float xa = fmaf(e.z, ra, e.x), ya = fmaf(e.w, ra, e.y);
                const float xb = fmaf(e.z, rb, e.x), yb = fmaf(e.w, rb, e.y);
                const bool miss = fmaxf(xa, xb) < fx0 || fminf(xa, xb) >= fx1 || fmaxf(ya, yb) < fy0 || fminf(ya, yb) >= fy1;
                if (!miss) {
                    const int kxa = flr_clamp(xa, g.W), kya = flr_clamp(ya, g.H);
                    const int kxb = flr_clamp(xb, g.W), kyb = flr_clamp(yb, g.H);
                    tile_add(org, R, kxa, kya);
                    if (kxa != kxb || kya != kyb) walk_tile(org, R, kxa, kya, kxb, kyb, e.x, e.y, e.z, e.w);
                }
            };
            const auto run = [&](unsigned i, unsigned lim, auto&& f) {
                if (i < lim) {
                    float4 e0 = at(i), e1 = at(i + NT), e2;
                    for (;;) {
                        e2 = at(i + 2 * NT);
                        f(e0, i);
                        i += NT;
                        if (i >= lim) break;
                        e0 = at(i + 2 * NT);
                        f(e1, i);
                        i += NT;
                        if (i >= lim) break;
                        e1 = at(i + 2 * NT);
                        f(e2, i);
                        i += NT;
                        if (i >= lim) break;
                    }
                }
            };
            run((unsigned)tid, nown, one);
            run(nown + (unsigned)tid, nseg, guest);
            nlow = nlow32;
        }
        // The border counters' squares and counts are removed, then the sums
        // of the counters and of their squares are taken over the whole
        // counter region, 16 bytes per read, and the region is zeroed for the
        // next hypothesis (every counter is zero between hypotheses).  The
        // sum of the counters less the border's is the hypothesis's count of
        // in-tile increments (every increment lands in one counter).  Each
        // thread takes some counters (its own sums may wrap; the workgroup's
        // totals are exact).
        // (A certificate touched no counter: it skips both passes, not the
        // barrier, which also orders thread 0's reads of the reduction
        // scratch before the next writes.)
        __syncthreads();
        unsigned long long sq = ucert, hits = 0;
        if (hp.kind != HYP_CERT) {
            for (int k = tid; k < nring; k += NT) {
                int idx;
                if (k < R.rw) idx = k;                                      // top row
                else if (k < 2 * R.rw) idx = (th + 1) * R.rw + (k - R.rw);  // bottom row
                else idx = (1 + ((k - 2 * R.rw) >> 1)) * R.rw + (((k - 2 * R.rw) & 1) ? R.rw - 1 : 0);
                const unsigned m = tile[idx];
                sq -= (unsigned long long)m * m;
                hits -= m;
            }
            if (img_out) {  // hypothesis wh's image(s): W*H cells per polarity image
                const long long M = (long long)g.W * g.H;
                unsigned* const im = img_out + (long long)wh * M * (g.T / g.nsp) + (long long)(t / g.nsp) * M;
                for (int k = tid; k < tw * th; k += NT) {
                    const int lx = k % tw, ly = k / tw;
                    im[(long long)(y0 + ly) * g.W + (x0 + lx)] = tile[(ly + 1) * R.rw + lx + 1];
                }
            }
            __syncthreads();  // every read of single counters is done before the region is zeroed
            uint4* const t4 = reinterpret_cast<uint4*>(tile);
            const int n4 = (ncnt + 3) >> 2;  // the counters lie in the rounded-up region
            for (int i = tid; i < n4; i += NT) {
                const uint4 v = t4[i];
                t4[i] = make_uint4(0u, 0u, 0u, 0u);
                sq += (unsigned long long)v.x * v.x + (unsigned long long)v.y * v.y +
                      (unsigned long long)v.z * v.z + (unsigned long long)v.w * v.w;
                hits += (unsigned long long)v.x + v.y + v.z + v.w;
            }
        }
        // block reduction of (S, hits, nlow)
        sq = wave_total(sq);
        hits = wave_total(hits);
        // N_low counts owned events (fewer than 2^28 per segment); points have none
        if (hp.kind != HYP_POINT) nlow = wave_total32((unsigned)nlow);
        const int wave = tid >> 6, lane = tid & 63;
        if (lane == 63) {
            s_red[wave] = sq;
            s_red[NW + wave] = hits;
            s_red[2 * NW + wave] = nlow;
        }
        __syncthreads();
        if (tid == 0) {
            unsigned long long a = 0, b = 0, c = 0;
            for (int k = 0; k < NW; ++k) {
                a += s_red[k];
                b += s_red[NW + k];
                c += s_red[2 * NW + k];
            }
            Part pt;
            pt.S = a;
            pt.N = (long long)(hp.kind == HYP_POINT ? b : c);
            pt.U = b;
            pt.pad = 0;
            part[(long long)wh * g.T + t] = pt;
        }
        // no barrier here: every thread zeroed its counters before the one
        // above, and thread 0 reads s_red before the next hypothesis's first
        // barrier, after which s_red is written again
      }
    }
}

// ------------------------------------------------------------ node groups (a2, a3)
//
// Late in a search the nodes are narrow and many lie side by side.  A node
// asks for its centre's point image and, unless it is a leaf, for the
// upper-bound images of its two children, which meet in the centre: three
// passes over the events, in which nearly every event adds the same single
// increment to every image.  k_nodes evaluates a group of up to kMaxNodes
// nodes of a window, in grid order, in one pass: an event whose pixel is the
// same at both ends of the group's hull [ra, rb] has that pixel at every rate
// between (the warp is monotone in the rate).  All events are binned at ra,
// the others are listed, and the counters then go from image to image by the
// listed events' changes alone: to node k's point image (phase 3k), to its
// first child's (3k + 1: the walks' pixels before the centre's) and back, to
// its second child's (3k + 2: the walks' pixels after the centre's) and back.
// A change of a counter from c to c + 1 changes the sum of squares by 2c + 1
// (the atomic returns c), whatever the order of the changes within a phase,
// so each phase's sum of these changes and the sums over the last image give
// every image's S and count of increments exactly.  N of a point image is its
// count of increments; N_low of an interval is the point count at its far
// end (an event inside the image there is inside at every smaller rate).
//
// Each wave makes the changes of its own strip of the tile's rows, so no wave
// waits for another between phases: a wave's LDS operations complete in
// order.  Bound by VALU issue (55% of its limit: 25 instructions an event in
// the pass for up to 3 kMaxNodes images, where k_eval takes about 27 per event
// and image) and by the latency of the returned counts in the phases.  Per
// batch, without and with node groups: 32 windows of 346x260 7.29 and 5.11 ms,
// 64 of 640x480 40.3 and 23.7 ms, 64 of 1280x720 (0.1M-5M events) 207 and
// 170 ms; a late step of the 640x480 batch 4.3 and 0.8 ms (with the binning,
// tiling and host work of today 4.39, 21.7 and 165 ms).
constexpr int kNodePhases = 3 * kMaxNodes;
static_assert(kNodePhases <= 64, "one lane per phase");

// LDS of k_nodes after the counters: [S and count of the last image][phase
// sums of S][of the count][changes of N, per node][steps, per wave][s_full][work item and its queue, queue sizes].
constexpr int kNodeLds = 16 + 12 * kNodePhases + 4 * kMaxNodes + 4 * kEvalWaves + 4 + 4 * (2 + kXcd);
size_t nodes_lds_bytes(int ring_px) { return (size_t)eval_counter_words(ring_px) * 4 + kNodeLds; }

// A step (see k_nodes): the counter before in the low 16 bits, then these.
constexpr int kStepRate = 16, kStepX = 21, kStepY = 23;  // rate index, 2-bit signed direction
constexpr unsigned kStepIn0 = 1u << 25, kStepIn1 = 1u << 26;  // the pixels before, after lie in the strip
constexpr unsigned kStepNone = 31u << kStepRate;
static_assert(3 * kMaxNodes <= 31, "rate index of a step");

__device__ __forceinline__ float lane_f(float v, int k) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k));
}

template <int NT>
__global__ __launch_bounds__(NT, NT == 1024 ? 4 : 6) void k_nodes(
    Geometry g, const float4* __restrict__ ev, const long long* __restrict__ seg_off,
    const int* __restrict__ seg_own, const WinParam* __restrict__ wp, const Hyp* __restrict__ hyps,
    const int* __restrict__ act, const Item* __restrict__ items, int qcap, Queue* __restrict__ q,
    Queue* __restrict__ q_reset, Part* __restrict__ part, int HS, float4* __restrict__ lists, int mcap) {
    constexpr int NW = NT / 64;
    extern __shared__ __align__(16) unsigned smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    unsigned* const tile = smem;
    unsigned long long* const s_fin = reinterpret_cast<unsigned long long*>(smem + eval_counter_words(g.ring_px));
    unsigned long long* const s_dS = s_fin + 2;
    int* const s_dH = reinterpret_cast<int*>(s_dS + kNodePhases);
    int* const s_dN = s_dH + kNodePhases;
    int* const s_cnt = s_dN + kMaxNodes;
    int* const s_full = s_cnt + kEvalWaves;
    int* const s_item = s_full + 1;
    if (blockIdx.x == 0 && tid < kXcd) {
        q_reset[tid].n_items = 0;
        q_reset[tid].next = 0;
    }
    {  // nothing queued: leave before the clear
        int any = 0;
        for (int r = 0; r < kXcd; ++r) any |= q[r].n_items;
        if (any == 0) return;
    }
    {  // counters and sums start at zero and are cleared again by each item
        uint4* const t4 = reinterpret_cast<uint4*>(tile);
        const int n4 = eval_counter_words(g.ring_px) >> 2;
        for (int i = tid; i < n4; i += NT) t4[i] = make_uint4(0u, 0u, 0u, 0u);
        unsigned* const rest = reinterpret_cast<unsigned*>(s_fin);
        for (int i = tid; i < kNodeLds / 4 - 2 - kXcd; i += NT) rest[i] = 0u;
    }
    const int home = blockIdx.x % kXcd;
    int qi = 0;
    int* const qn = s_item + 2;
    if (tid == 0)
        for (int r = 0; r < kXcd; ++r) qn[r] = q[(home + r) % kXcd].n_items;
    const int F = HS / 3;
    for (;;) {
        if (tid == 0) {
            int got = -1;
            while (qi < kXcd) {
                const int r = (home + qi) % kXcd;
                if (qn[qi] > 0) {
                    const int k = atomicAdd(&q[r].next, 1);
                    if (k < qn[qi]) {
                        got = k;
                        s_item[1] = r;
                        break;
                    }
                }
                ++qi;
            }
            *s_item = got;
        }
        __syncthreads();
        const int it = *s_item;
        if (it < 0) break;
        const Item item = items[node_slot(s_item[1], it, qcap)];
        const int w = item.w, t = item.t, m = item.cnt;
        const int ts = t % g.nsp;
        const int tx = ts % g.ntx, ty = ts / g.ntx;
        const int x0 = g.colcut[tx], y0 = g.rowcut[ty];
        const int tw = g.colcut[tx + 1] - x0, th = g.rowcut[ty + 1] - y0;
        Ring R;
        R.xlo = x0 - 1;
        R.xhi = x0 + tw;
        R.ylo = y0 - 1;
        R.yhi = y0 + th;
        R.rw = tw + 2;
        R.base = -(R.ylo * R.rw + R.xlo);
        unsigned* const org = tile + R.base;
        const float fxlo = (float)R.xlo, fxhi = (float)R.xhi, fylo = (float)R.ylo, fyhi = (float)R.yhi;
        const long long seg = (long long)w * g.T + t;
        // lane k holds node k: its slot, the rates of its start, centre and
        // end (a leaf's are its centre's) and whether it has children
        int slot = 0, kids = 0;
        float na = INFINITY, nc = 0.0f, nb = -INFINITY;
        if (lane < m) {
            slot = act[w * HS + item.r0 + lane];
            const Hyp* const hy = hyps + w * HS;
            na = nc = nb = hy[slot].ra;
            kids = hy[F + 2 * slot].kind != HYP_NONE;
            if (kids) {
                na = hy[F + 2 * slot].ra;
                nb = hy[F + 2 * slot + 1].rb;
            }
        }
        float ra = INFINITY, rb = -INFINITY;  // the hull
        for (int k = 0; k < m; ++k) {
            ra = fminf(ra, lane_f(na, k));
            rb = fmaxf(rb, lane_f(nb, k));
        }
        // guest bins read: those whose lower cut lies below the hull's end
        int nbin = 0;
        {
            const float* const gcut = wp[w].gcut;
#pragma unroll
            for (int k = 0; k < kGuestBins - 1; ++k) nbin += gcut[k] < rb ? 1 : 0;
        }
        const char* __restrict__ sev = reinterpret_cast<const char*>(ev + seg_off[seg]);
        const auto at = [sev](unsigned k) { return *reinterpret_cast<const float4*>(sev + (k << 4)); };
        const unsigned nseg = (unsigned)seg_own[seg * (kGuestBins + 1) + 1 + nbin];
        // strips of sr rows, one per wave; (k + 0.5) / sr stays clear of the
        // integers by 0.5 / sr, far more than the rounding for k < 2^15
        const int sr = (th + NW - 1) / NW;
        const float inv = 1.0f / (float)sr;
        const auto strip = [&](int ky) {
            return (int)(((float)clampi(ky - y0, 0, th - 1) + 0.5f) * inv);
        };
        // pixels at both ends of the hull, clamped onto the tile's border
        const auto ends = [&](const float4& e, int& kx, int& ky, int& kxb, int& kyb) {
            kx = cvt_flr(__builtin_amdgcn_fmed3f(fmaf(e.z, ra, e.x), fxlo, fxhi));
            ky = cvt_flr(__builtin_amdgcn_fmed3f(fmaf(e.w, ra, e.y), fylo, fyhi));
            kxb = cvt_flr(__builtin_amdgcn_fmed3f(fmaf(e.z, rb, e.x), fxlo, fxhi));
            kyb = cvt_flr(__builtin_amdgcn_fmed3f(fmaf(e.w, rb, e.y), fylo, fyhi));
        };
        const auto pix = [&](const float4& e, float r, int& kx, int& ky) {  // the pixel in the image
            kx = flr_clamp(fmaf(e.z, r, e.x), g.W);
            ky = flr_clamp(fmaf(e.w, r, e.y), g.H);
        };
        const auto before = [](unsigned long long mask) {  // lanes of the mask before this one
            return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                  __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
        };
        // This wave's part of the lists: the events of its share of the
        // segment that change pixel inside the hull (mcap records), and what
        // becomes of them for its strip (kStepCap mcap words: a strip may
        // hold several times its share of a tile).
        char* const wg_list = reinterpret_cast<char*>(lists) + (size_t)blockIdx.x * NW * node_list_bytes(mcap);
        const auto moved_of = [&](int wv) { return reinterpret_cast<float4*>(wg_list + wv * node_list_bytes(mcap)); };
        const auto steps_of = [&](int wv) { return reinterpret_cast<unsigned*>(moved_of(wv) + mcap); };
        float4* const moved = moved_of(wave);
        int nl = 0;
        const auto bin = [&](const float4& e, bool valid) {
            int kx, ky, kxb, kyb;
            ends(e, kx, ky, kxb, kyb);
            if (valid) lds_inc(ring_at(org, R, kx, ky));
            const bool mv = valid && (kx != kxb || ky != kyb);
            const unsigned long long mask = __ballot(mv);
            const int at_ = nl + before(mask);
            if (mv && at_ < mcap) moved[at_] = e;
            nl += __popcll(mask);
        };
        constexpr int U = 4;
        // (the whole wave runs every iteration, so nl stays uniform)
        unsigned b = (unsigned)wave * 64;
        for (; b + (U - 1) * NT + 63 < nseg; b += U * NT) {
            float4 e[U];
#pragma unroll
            for (int k = 0; k < U; ++k) e[k] = at(b + lane + k * NT);
#pragma unroll
            for (int k = 0; k < U; ++k) bin(e[k], true);
        }
        for (; b < nseg; b += NT) bin(at(min(b + lane, nseg - 1)), b + lane < nseg);
        nl = __builtin_amdgcn_readfirstlane(nl);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        // Most listed events change each coordinate by one pixel at most over
        // the hull.  Such a change is kept as a step: the counter before it,
        // its direction, whether the pixels before and after lie in the strip,
        // and the first of the rates a_0, c_0, b_0, a_1, .. at which it is
        // done (3k: node k's start, 3k + 1: its centre, 3k + 2: its end).  Two changes between the same two
        // rates are one diagonal step, and what its walk visits on the way
        // (walk_tile's corner test) a step from a pixel to itself, which adds
        // to the one child's image only.  A list without room, or an event
        // that moves further, leaves the images to be made one by one from the
        // segment's events (s_full: the groups are cut so narrow that ordinary
        // windows meet neither; windows whose events crowd on few points do).
        if (nl > mcap && lane == 0) *s_full = 1;
        for (int j0 = 0; j0 < min(nl, mcap); j0 += 64) {
            const bool ok = j0 + lane < nl;
            const float4 e = ok ? moved[j0 + lane] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            int kx, ky, kxb, kyb;
            ends(e, kx, ky, kxb, kyb);
            const bool px = kxb > kx, py = kyb > ky;
            const float ex = (float)max(kx, kxb), ey = (float)max(ky, kyb);  // the edges stepped over
            int cx = 1, cy = 1;  // rates at which the step is not done
            for (int k = 0; k < m; ++k) {
                const float a = lane_f(na, k), c = lane_f(nc, k), d = lane_f(nb, k);
                if (k) {
                    cx += (fmaf(e.z, a, e.x) < ex) == px;
                    cy += (fmaf(e.w, a, e.y) < ey) == py;
                }
                cx += (fmaf(e.z, c, e.x) < ex) == px;
                cy += (fmaf(e.w, c, e.y) < ey) == py;
                cx += (fmaf(e.z, d, e.x) < ex) == px;
                cy += (fmaf(e.w, d, e.y) < ey) == py;
            }
            const bool sx = kx != kxb, sy = ky != kyb;
            if (!ok) continue;
            const auto in_tile = [&](int x, int y) {
                return (unsigned)(x - x0) < (unsigned)tw && (unsigned)(y - y0) < (unsigned)th;
            };
            // the step (fx, fy) -> (gx, gy) to the strips of its two pixels
            const auto put = [&](int fx, int fy, int gx, int gy, int rate) {
                const int s0 = strip(fy), s1 = strip(gy);
                const bool fin = in_tile(fx, fy), gin = in_tile(gx, gy);
                const unsigned word = (unsigned)((fy - R.ylo) * R.rw + (fx - R.xlo)) | (unsigned)rate << kStepRate |
                                      ((unsigned)(gx - fx) & 3u) << kStepX | ((unsigned)(gy - fy) & 3u) << kStepY;
                for (int u = 0; u < 2; ++u) {
                    const int s = u ? s1 : s0;
                    const unsigned in = (fin && s == s0 ? kStepIn0 : 0u) | (gin && s == s1 ? kStepIn1 : 0u);
                    if (in) {
                        const int k = atomicAdd(&s_cnt[s], 1);
                        if (k < kStepCap * mcap) steps_of(s)[k] = word | in;
                        else *s_full = 1;
                    }
                    if (s0 == s1) break;
                }
            };
            if (abs(kx - kxb) > 1 || abs(ky - kyb) > 1) {
                *s_full = 1;
                continue;
            }
            const bool diag = sx && sy && cx == cy;
            if (diag && cx % 3 != 0) {
                // the walk itself runs in the image, not on the tile's border
                int ax, ay, bx, by;
                pix(e, ra, ax, ay);
                pix(e, rb, bx, by);
                if (abs(ax - bx) > 1 || abs(ay - by) > 1) *s_full = 1;
                const double xo = (double)e.x - (double)px, yo = (double)e.y - (double)py;
                const double aax = fabs((double)e.z), aay = fabs((double)e.w);
                const double thr = (aax + aay) * 0.00390625;
                const double d = fabs((double)ax - xo) * aay - fabs((double)ay - yo) * aax;
                // x first, y first, or both sides of the corner (pixels off
                // the tile go nowhere)
                if (!(d > thr) && in_tile(bx, ay)) put(bx, ay, bx, ay, cx);
                if (!(d < -thr) && in_tile(ax, by)) put(ax, by, ax, by, cx);
            }
            // the step, or the first of two, to (gx, gy)
            const bool xfirst = sx && (!sy || cx < cy), two = sx && sy && !diag;
            const int gx = xfirst || diag ? kxb : kx, gy = xfirst ? ky : kyb;
            put(kx, ky, gx, gy, xfirst ? cx : cy);
            if (two) put(gx, gy, kxb, kyb, xfirst ? cy : cx);
        }
        __syncthreads();  // the image at ra and the lists are complete
        const bool full = *s_full != 0;
        uint4* const t4 = reinterpret_cast<uint4*>(tile);
        const int n4 = (R.rw * (th + 2) + 3) >> 2;
        if (full) {
            for (int i = tid; i < n4; i += NT) t4[i] = make_uint4(0u, 0u, 0u, 0u);
            R.vxhi = to_vgpr(R.xhi);
            R.vyhi = to_vgpr(R.yhi);
            __syncthreads();
        }
      // once over the last image of the group, or (full) over every image,
      // 3k: node k's point image, 3k + 1 and 3k + 2: its children's.  (Every
      // wave looking through all events for its strip's changes, phase by
      // phase, kept the counters but took 35 ms for 16 windows of 1M events
      // on 128 x 128 pixels; image by image 9.3, 200k events 4.5 and 1.9.)
      for (int im = 0; im < (full ? 3 * m : 1); ++im) {
        const int fk = im / 3, fside = im - 3 * fk;
        if (full && fside && !__builtin_amdgcn_readlane(kids, fk)) continue;  // a leaf
        if (full) {
            const float lo = fside == 1 ? lane_f(na, fk) : lane_f(nc, fk);
            const float hi = fside == 2 ? lane_f(nb, fk) : lane_f(nc, fk);
            int nin = 0;  // events in the tile at the far end
            for (unsigned j = tid; j < nseg; j += NT) {
                const float4 e = at(j);
                int kx, ky, hx, hy;
                pix(e, lo, kx, ky);
                pix(e, hi, hx, hy);
                tile_add(org, R, kx, ky);
                if (kx != hx || ky != hy) walk_tile(org, R, kx, ky, hx, hy, e.x, e.y, e.z, e.w);
                nin += (unsigned)(hx - x0) < (unsigned)tw && (unsigned)(hy - y0) < (unsigned)th;
            }
            if (fside && nin) atomicAdd(s_dN, nin);
        } else {
            const int ns = s_cnt[wave];
            const unsigned* const steps = steps_of(wave);
            // four chunks of steps at a time, kept in registers when they are all
            constexpr int C = 4;
            unsigned sp[C];
            const auto load = [&](int j0) {
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    const int j = j0 + i * 64 + lane;
                    sp[i] = j < ns ? steps[j] : kStepNone;
                }
            };
            load(0);
            // f(step) of every step whose rate index lies in [lo, lo + cnt)
            const auto each_step = [&](int lo, unsigned cnt, auto&& f) {
                for (int j0 = 0; j0 < ns; j0 += C * 64) {
                    if (ns > C * 64) load(j0);
#pragma unroll
                    for (int i = 0; i < C; ++i) {
                        if (j0 + i * 64 >= ns) break;
                        if ((unsigned)((int)(sp[i] >> kStepRate & 31u) - lo) < cnt) f(sp[i]);
                    }
                }
            };
            const auto first = [&](unsigned v) { return tile + (v & 0xFFFFu); };
            const auto second = [&](unsigned v) {
                const int dx = (int)(v << (30 - kStepX)) >> 30, dy = (int)(v << (30 - kStepY)) >> 30;
                return tile + (int)(v & 0xFFFFu) + dx + __mul24(dy, R.rw);
            };
            const auto account = [&](int ph, long long dS, int dH) {
                if (dS != 0) atomicAdd(s_dS + to_vgpr(ph), (unsigned long long)dS);
                if (dH != 0) atomicAdd(s_dH + to_vgpr(ph), dH);
            };
            for (int k = 0; ns > 0 && k < m; ++k) {
                const bool leaf = lane_f(na, k) == lane_f(nb, k);
#pragma unroll 1
                for (int st = 0; st < 4; ++st) {
                    // 0: the last second child's extra pixels go, the points
                    // move to the next centre; 1: first child's extra pixels;
                    // 2: they go; 3: second child's
                    if (st == 0) {
                        each_step(3 * k - 1, 1u, [&](unsigned v) {
                            if (v & kStepIn1) atomicSub(second(v), 1u);
                        });
                    } else if (st == 2) {
                        each_step(3 * k + 1, 1u, [&](unsigned v) {
                            if (v & kStepIn0) atomicSub(first(v), 1u);
                        });
                    } else {
                        each_step(st == 1 ? 3 * k + 1 : 3 * k + 2, 1u, [&](unsigned v) {
                            if (v & (st == 1 ? kStepIn0 : kStepIn1))
                                account(st == 1 ? 3 * k + 1 : 3 * k + 2,
                                        2 * (long long)(int)atomicAdd(st == 1 ? first(v) : second(v), 1u) + 1, 1);
                            const int d = (int)((v & kStepIn1) != 0) - (int)((v & kStepIn0) != 0);
                            if (st == 3 && d) atomicAdd(s_dN + to_vgpr(k), d);
                        });
                    }
                    if (st == 0) {
                        each_step(3 * k - 1, 3u, [&](unsigned v) {
                            const bool in0 = v & kStepIn0, in1 = v & kStepIn1;
                            unsigned o0 = 0, o1 = 0;
                            if (in0) o0 = atomicSub(first(v), 1u);
                            if (in1) o1 = atomicAdd(second(v), 1u);
                            account(3 * k, (in1 ? 2 * (long long)(int)o1 + 1 : 0) - (in0 ? 2 * (long long)(int)o0 - 1 : 0),
                                    (int)in1 - (int)in0);
                        });
                    }
                    // the next part's changes stay behind this one's
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    if (leaf) break;
                }
            }
        }
        // The sums over the last image: the border's counters come off, then
        // one pass over the counters, which zeroes them for the next item.
        __syncthreads();
        unsigned long long sq = 0, hits = 0;
        const int nring = 2 * R.rw + 2 * th;
        for (int k = tid; k < nring; k += NT) {
            int idx;
            if (k < R.rw) idx = k;
            else if (k < 2 * R.rw) idx = (th + 1) * R.rw + (k - R.rw);
            else idx = (1 + ((k - 2 * R.rw) >> 1)) * R.rw + (((k - 2 * R.rw) & 1) ? R.rw - 1 : 0);
            const unsigned v = tile[idx];
            sq -= (unsigned long long)v * v;
            hits -= v;
        }
        __syncthreads();
        for (int i = tid; i < n4; i += NT) {
            const uint4 v = t4[i];
            t4[i] = make_uint4(0u, 0u, 0u, 0u);
            sq += (unsigned long long)v.x * v.x + (unsigned long long)v.y * v.y + (unsigned long long)v.z * v.z +
                  (unsigned long long)v.w * v.w;
            hits += (unsigned long long)v.x + v.y + v.z + v.w;
        }
        sq = wave_total(sq);
        hits = wave_total(hits);
        if (lane == 63) {
            atomicAdd(&s_fin[0], sq);
            atomicAdd(&s_fin[1], hits);
        }
        __syncthreads();
        if (full) {
            if (tid == 0) {
                const int i = __builtin_amdgcn_readlane(slot, fk);
                Part pt;
                pt.S = s_fin[0];
                pt.U = s_fin[1];
                pt.N = fside ? (long long)*s_dN : (long long)s_fin[1];
                pt.pad = 0;
                part[((long long)w * HS + (fside == 0 ? i : F + 2 * i + fside - 1)) * g.T + t] = pt;
                s_fin[0] = s_fin[1] = 0ull;
                *s_dN = 0;
            }
            __syncthreads();
            continue;
        }
        if (tid < 64) {
            // lane p: the image of phase p.  The last image's sums less its
            // extra pixels give the last centre's, less the moves after
            // centre k that centre's.
            const int k = lane / 3, side = lane - 3 * k;
            unsigned long long dS = 0, dH = 0;
            if (lane < kNodePhases) {
                dS = s_dS[lane];
                dH = (unsigned long long)(long long)s_dH[lane];
            }
            unsigned long long ss = side ? 0ull : dS, hh = side ? 0ull : dH;
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned long long s2 = __shfl_down(ss, o, 64), h2 = __shfl_down(hh, o, 64);
                if (lane + o < 64) {
                    ss += s2;
                    hh += h2;
                }
            }
            const unsigned long long Sc = s_fin[0] - s_dS[3 * m - 1] - (side ? ss : ss - dS);
            const unsigned long long Nc = s_fin[1] - (unsigned long long)(long long)s_dH[3 * m - 1] - (side ? hh : hh - dH);
            const int i = __shfl(slot, min(k, 63), 64), hk = __shfl(kids, min(k, 63), 64);
            if (k < m && (side == 0 || hk)) {
                Part pt;
                pt.S = side ? Sc + dS : Sc;
                pt.N = (long long)Nc + (side == 2 ? s_dN[k] : 0);
                pt.U = side ? Nc + dH : Nc;
                pt.pad = 0;
                part[((long long)w * HS + (side == 0 ? i : F + 2 * i + side - 1)) * g.T + t] = pt;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (lane < kNodePhases) {
                s_dS[lane] = 0ull;
                s_dH[lane] = 0;
            }
            if (lane < kMaxNodes) s_dN[lane] = 0;
            if (lane < kEvalWaves + 1) s_cnt[lane] = 0;  // and s_full
            if (lane < 2) s_fin[lane] = 0ull;
        }
      }
        if (full && tid < kEvalWaves + 1) s_cnt[tid] = 0;  // and s_full
    }
}

static const void* nodes_kernel(int nt) {
    switch (nt) {
        case 256: return (const void*)k_nodes<256>;
        case 512: return (const void*)k_nodes<512>;
        default: return (const void*)k_nodes<1024>;
    }
}

hipError_t nodes_occupancy(int* blocks_per_cu, size_t lds_bytes, int nt) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, nodes_kernel(nt), nt, lds_bytes);
}

hipError_t launch_nodes(hipStream_t s, const Geometry& g, int nblocks, int nt, size_t lds_bytes, const float4* ev,
                        const long long* seg_off, const int* seg_own, const WinParam* wp, const Hyp* hyps,
                        const int* act, const Item* items, int qcap, Queue* q, Queue* q_reset, Part* part, int HS,
                        float4* lists, int mcap, hipEvent_t t0, hipEvent_t t1) {
    switch (nt) {
        case 256:
            hipExtLaunchKernelGGL(k_nodes<256>, dim3(nblocks), dim3(256), (uint32_t)lds_bytes, s, t0, t1, 0u, g, ev,
                                  seg_off, seg_own, wp, hyps, act, items, qcap, q, q_reset, part, HS, lists, mcap);
            break;
        case 512:
            hipExtLaunchKernelGGL(k_nodes<512>, dim3(nblocks), dim3(512), (uint32_t)lds_bytes, s, t0, t1, 0u, g, ev,
                                  seg_off, seg_own, wp, hyps, act, items, qcap, q, q_reset, part, HS, lists, mcap);
            break;
        default:
            hipExtLaunchKernelGGL(k_nodes<1024>, dim3(nblocks), dim3(1024), (uint32_t)lds_bytes, s, t0, t1, 0u, g,
                                  ev, seg_off, seg_own, wp, hyps, act, items, qcap, q, q_reset, part, HS, lists, mcap);
    }
    return hipGetLastError();
}

// The evaluation kernel for nt threads per workgroup (256, 512 or 1024).
static const void* eval_kernel(int nt) {
    switch (nt) {
        case 256: return (const void*)k_eval<256>;
        case 512: return (const void*)k_eval<512>;
        default: return (const void*)k_eval<1024>;
    }
}

hipError_t eval_occupancy(int* blocks_per_cu, size_t lds_bytes, int nt) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, eval_kernel(nt), nt, lds_bytes);
}

hipError_t eval_set_lds(size_t bytes) {
    for (int nt : {256, 512, 1024}) {
        hipError_t e = hipFuncSetAttribute(eval_kernel(nt), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(nodes_kernel(nt), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_eval(hipStream_t s, const Geometry& g, int nblocks, int nt, size_t lds_bytes, const float4* ev,
                       const long long* seg_off, const int* seg_own, const WinParam* wp, const Hyp* hyps,
                       const int* act,
                       const Item* items, int qcap, Queue* q, Queue* q_reset, Part* part, int HS,
                       unsigned* img_out, hipEvent_t t0, hipEvent_t t1) {
    // the events (nullable) take the kernel's start and end times from its dispatch
    switch (nt) {
        case 256:
            hipExtLaunchKernelGGL(k_eval<256>, dim3(nblocks), dim3(256), (uint32_t)lds_bytes, s, t0, t1, 0u, g, ev,
                                  seg_off, seg_own, wp, hyps, act, items, qcap, q, q_reset, part, HS, img_out);
            break;
        case 512:
            hipExtLaunchKernelGGL(k_eval<512>, dim3(nblocks), dim3(512), (uint32_t)lds_bytes, s, t0, t1, 0u, g, ev,
                                  seg_off, seg_own, wp, hyps, act, items, qcap, q, q_reset, part, HS, img_out);
            break;
        default:
            hipExtLaunchKernelGGL(k_eval<1024>, dim3(nblocks), dim3(1024), (uint32_t)lds_bytes, s, t0, t1, 0u, g,
                                  ev, seg_off, seg_own, wp, hyps, act, items, qcap, q, q_reset, part, HS, img_out);
    }
    return hipGetLastError();
}

// ------------------------------------------------------------ frontier (a4)

constexpr int NTF = kFrontThreads;
constexpr int NWF = NTF / 64;

// A node group lists at most this share of the events, by the estimate lam
// of emit_hyps.  An event moves at most four times the mean (a corner of the
// sensor, the start of the window), so by less than a pixel.  Measured on 32
// windows of 346x260 and 64 of 640x480, per batch: 0.1 5.03 and 23.7 ms, 0.2
// 5.01 and 23.6, 0.3 5.08 and 23.8 (7.29 and 40.3 without node groups).
constexpr float kNodeShare = 0.2f;
// A window of an image of at most kNodeSmall cells with more than kNodeDense
// events per cell forms none: its walks are short, so plain evaluation is
// cheap, and whole points of events cross pixel edges together and outgrow the
// lists.  us a search, without and with groups: 128x128, 8 windows of 500k
// events (30 per cell) 2816 and 3733, 16 of 1M (61) 6540 and 9270, 16 of 200k
// (12) 2295 and 1863; 346x260 (89960 cells), 6 of 3M (33) 35960 and 21940.
constexpr long long kNodeSmall = 40000, kNodeDense = 24;

// Scratch of the workgroup's scans: each call alternates between two rows, so
// a call needs one barrier (the row it writes was last read before the barrier
// of the call between).  `turn` starts at 0 in every thread and moves alike.
// The frontier is a serial chain of such calls on one workgroup per window;
// with two barriers and a shuffle scan for flags as well a round took 9.9 us
// on one 128 x 128 window, with this and slot_sums' grouped loads 8.8.
struct ScanLds {
    int row[2][NWF];
};

// Exclusive prefix sum of v over the workgroup (in thread order); `total`
// receives the sum.  All threads must call it.
__device__ __forceinline__ int block_scan(int v, ScanLds* sc, int& turn, int& total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int x = v;
    for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    int* const row = sc->row[turn & 1];
    ++turn;
    if (lane == 63) row[wave] = x;
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < NWF; ++k) {
        const int t = row[k];
        if (k < wave) base += t;
        tot += t;
    }
    total = tot;
    return base + x - v;
}

// The same for a flag per thread: a wave's flags are one ballot.
__device__ __forceinline__ int block_rank(bool f, ScanLds* sc, int& turn, int& total) {
    const int wave = threadIdx.x >> 6;
    const unsigned long long m = __ballot(f);
    int* const row = sc->row[turn & 1];
    ++turn;
    if ((threadIdx.x & 63) == 0) row[wave] = __popcll(m);
    __syncthreads();
    int base = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < NWF; ++k) {
        const int t = row[k];
        if (k < wave) base += t;
        tot += t;
    }
    total = tot;
    return base + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Lexicographic maximum of (K, -j) over the workgroup: within each wave by
// lane exchanges, then across the NWF wave winners through LDS.
__device__ __forceinline__ bool lex_better(long long bh, unsigned long long bl, unsigned bj, long long ah,
                                           unsigned long long al, unsigned aj) {
    return bh > ah || (bh == ah && (bl > al || (bl == al && bj < aj)));
}

__device__ __forceinline__ void block_argmax(i128& K, unsigned& j, long long* s_hi, unsigned long long* s_lo,
                                             unsigned* s_j) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    long long h;
    unsigned long long l;
    sp128(K, h, l);
    unsigned jj = j;
    for (int o = 32; o > 0; o >>= 1) {
        const long long oh = __shfl_xor(h, o, 64);
        const unsigned long long ol = __shfl_xor(l, o, 64);
        const unsigned oj = __shfl_xor(jj, o, 64);
        if (lex_better(oh, ol, oj, h, l, jj)) {
            h = oh;
            l = ol;
            jj = oj;
        }
    }
    if (lane == 0) {
        s_hi[wave] = h;
        s_lo[wave] = l;
        s_j[wave] = jj;
    }
    __syncthreads();
    h = s_hi[0];
    l = s_lo[0];
    jj = s_j[0];
    for (int k = 1; k < NWF; ++k)
        if (lex_better(s_hi[k], s_lo[k], s_j[k], h, l, jj)) {
            h = s_hi[k];
            l = s_lo[k];
            jj = s_j[k];
        }
    K = mk128(h, l);
    j = jj;
    __syncthreads();
}

// Sum of the tiles' partial sums of one hypothesis slot.
__device__ __forceinline__ void slot_sums(const Part* pw, int slot, int T, const int* tiles, int nt,
                                          unsigned long long& S, long long& N, unsigned long long& U) {
    S = 0;
    N = 0;
    U = 0;
    // eight tiles' loads in flight (one after another they are a chain of
    // nt memory latencies)
    constexpr int G = 8;
    for (int k = 0; k < nt; k += G) {
        Part q[G];
#pragma unroll
        for (int j = 0; j < G; ++j) q[j] = pw[(long long)slot * T + tiles[min(k + j, nt - 1)]];
#pragma unroll
        for (int j = 0; j < G; ++j)
            if (k + j < nt) {
                S += q[j].S;
                N += q[j].N;
                U += q[j].U;
            }
    }
}

// Work items of the na active slots act[0..na) of window w: groups of up
// to G slots on each non-empty tile, tile-major, appended to the window's
// queue in qf.
__device__ void emit_items(const Search& sp, int w, const int* tiles, int nt, int na, Item* items, int qcap,
                           Queue* qf) {
    int G = sp.G;
    const int qr = w % kXcd;  // this window's queue
    Item* qitems = items + hyp_slot(qr, 0, qcap);
    __shared__ int s_base;
    if (sp.gslots > 0) {  // this step's items with one hypothesis each, all windows alike
        const long long work = (long long)sp.B * na * nt;
        G = (int)max(1ll, min((long long)G, work / sp.gslots));
    }
    const int ng = (na + G - 1) / G;
    if (threadIdx.x == 0) s_base = (ng * nt) ? atomicAdd(&qf[qr].n_items, ng * nt) : 0;
    __syncthreads();
    for (int k = threadIdx.x; k < ng * nt; k += NTF) {
        const int ti = k / ng, gi = k % ng;  // tile-major: items sharing events are adjacent
        Item it;
        it.w = w;
        it.t = tiles[ti];
        it.r0 = gi * G;
        it.cnt = min(G, na - gi * G);
        // within a tile the groups with intervals (the longer items) first
        qitems[s_base + ti * ng + (ng - 1 - gi)] = it;
    }
    __syncthreads();
}

// Node items of window w, tile-major, from the end of its queue's slots:
// group k holds the sorted nodes act[base + gs[k]] up to the next group's start.
__device__ void emit_node_items(int w, const int* tiles, int nt, int base, const int* gs, int ng, int nodes,
                                Item* items, int qcap, Queue* nf) {
    const int qr = w % kXcd;
    Item* const qlast = items + node_slot(qr, 0, qcap);
    __shared__ int s_nbase;
    if (threadIdx.x == 0) s_nbase = (ng * nt) ? atomicAdd(&nf[qr].n_items, ng * nt) : 0;
    __syncthreads();
    for (int k = threadIdx.x; k < ng * nt; k += NTF) {
        const int ti = k / ng, gi = k % ng;
        Item it;
        it.w = w;
        it.t = tiles[ti];
        it.r0 = base + gs[gi];
        it.cnt = (gi + 1 < ng ? gs[gi + 1] : nodes) - gs[gi];
        *(qlast - (s_nbase + k)) = it;
    }
    __syncthreads();
}

// Hypotheses of the selected nodes, the list of active slots, and the work
// items.  q_rem: nodes left in the queue; n_kids: selected nodes with
// children.  When every node the queue can hold after the next step is
// expanded at that step (q_rem + 2 n_kids <= F) and there is no node
// budget, a child's bound value decides nothing but whether it is kept, so
// the children get the endpoint certificate (exact bounds when it fails, in
// the same step).  For the gamma stop a certified child's points are
// bounded by its nearest exactly bounded ancestor's bound instead.
__device__ void emit_hyps(const Search& sp, const WinParam& p, int w, int T, const int* tiles, int nt, int most,
                          const Sel* sl, int n_sel, int q_rem, int n_kids, float kinc, Hyp* hy, int* act,
                          Item* items, int qcap, Queue* qf, ScanLds* sc, int& turn, bool groups) {
    const int F = sp.F, HS = sp.HS;
    const bool cert = sp.cert && sp.max_nodes == 0 && q_rem + 2 * n_kids <= F && q_rem + 2 * n_kids <= sp.CAP;
    // a node's children take the certificate when it is expected to clear
    // the incumbent K_inc (kinc): a failed certificate costs its pass and the
    // exact bound (measured on the three batches: margins of 0.5 to 1.5 x
    // K_inc within 3%, 1.0 best; no prediction: +10% on 1280x720, +25% on
    // 346x260)
    // Nodes that go into node groups.  lam estimates how many pixels an event
    // moves per unit of rate (the mean of |ax| + |ay| over the sensor and the
    // window), so lam times a node's width is about the share of the events
    // that change pixel inside it.
    constexpr unsigned kAlone = 0xFFFFFFFFu;  // (grid indices stay below 2^31)
    __shared__ unsigned s_ja[kMaxF];  // a grouped node's start on the grid, or kAlone
    __shared__ float s_na[kMaxF], s_nb[kMaxF];  // its rates there and at its end
    __shared__ int s_ord[kMaxF], s_gs[kMaxF];
    __shared__ int s_ng;
    const float per = (float)most / (float)max(sp.nwave, 1);  // a wave's events of the fullest tile
    // the share of the events that a group may list
    const float share = fminf(kNodeShare, (float)sp.nlist / fmaxf(per, 1.0f));
    const float lam = p.kscale > 0.0f ? 0.25f * (float)kNB / p.kscale : 0.0f;
    groups = groups && sp.nmax > 0 && (sp.M > kNodeSmall || p.n_events <= kNodeDense * sp.M);
    int nodes = 0;
    for (int i0 = 0; groups && i0 < n_sel; i0 += NTF) {
        const int i = i0 + threadIdx.x;
        bool in = false;
        if (i < n_sel) {
            const float a = rate_of(grid_d(sp.d_lo, sp.d_hi, sp.L, sl[i].ja), p.tau);
            const float b = rate_of(grid_d(sp.d_lo, sp.d_hi, sp.L, sl[i].jb), p.tau);
            in = lam * (b - a) <= share && !(cert && sl[i].kids && sl[i].lc > kinc);
            s_ja[i] = in ? sl[i].ja : kAlone;
            s_na[i] = a;
            s_nb[i] = b;
        }
        int tot;
        block_rank(in, sc, turn, tot);
        nodes += tot;
    }
    int na = 0;  // active slots so far
    for (int h0 = 0; h0 < HS; h0 += NTF) {
        const int h = h0 + threadIdx.x;
        Hyp hp;
        hp.kind = HYP_NONE;
        hp.pad = 0;
        hp.ra = hp.rb = 0.0f;
        if (h < F) {
            if (h < n_sel) {
                hp.kind = HYP_POINT;
                hp.ra = hp.rb = rate_of(grid_d(sp.d_lo, sp.d_hi, sp.L, sl[h].jc), p.tau);
            }
        } else if (h < HS) {
            const int c = h - F, i = c >> 1;
            if (i < n_sel && sl[i].kids) {
                const unsigned a = (c & 1) ? sl[i].jc : sl[i].ja;
                const unsigned b = (c & 1) ? sl[i].jb : sl[i].jc;
                hp.kind = (cert && sl[i].lc > kinc) ? HYP_CERT : HYP_INTERVAL;
                hp.ra = rate_of(grid_d(sp.d_lo, sp.d_hi, sp.L, a), p.tau);
                hp.rb = rate_of(grid_d(sp.d_lo, sp.d_hi, sp.L, b), p.tau);
            }
        }
        if (h < HS) hy[h] = hp;
        const int node = h < F ? h : (h - F) >> 1;
        const bool alone = hp.kind != HYP_NONE && !(nodes && s_ja[node] != kAlone);
        int tot;
        const int r = block_rank(alone, sc, turn, tot);
        if (alone) act[na + r] = h;
        na += tot;
    }
    emit_items(sp, w, tiles, nt, na, items, qcap, qf);
    if (!nodes) return;
    // The grouped nodes in grid order, as k_nodes takes them.  Nodes are
    // disjoint, so their starts on the grid differ, where neighbouring grid
    // points may share a rate (from a depth of about 26 on): by rates a node
    // of no width could come after its wider neighbour.
    for (int i = threadIdx.x; i < n_sel; i += NTF) {
        const unsigned ja = s_ja[i];
        if (ja == kAlone) continue;
        int r = 0;
        for (int k = 0; k < n_sel; ++k) r += s_ja[k] < ja ? 1 : 0;
        s_ord[r] = i;
        act[na + r] = i;
    }
    __syncthreads();
    // A group takes the nodes that follow while its hull lists at most hull
    // of the events: s_gs[r] = the node after the group that starts at r.
    const float hull = share / fmaxf(lam, 1e-7f);
    const long long alone_items = (long long)sp.B * nodes * nt;  // items with one node each, all windows alike
    const int gm = (int)max(1ll, min((long long)sp.nmax, alone_items / max(sp.nslots, 1ll)));
    for (int r = threadIdx.x; r < nodes; r += NTF) {
        const float lim = s_na[s_ord[r]] + hull;
        int e = r + 1;
        while (e < nodes && e < r + gm && s_nb[s_ord[e]] <= lim) ++e;
        s_gs[r] = e;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int n = 0;
        for (int r = 0; r < nodes; ++n) {  // n <= r: entries still needed are not overwritten
            const int e = s_gs[r];
            s_gs[n] = r;
            r = e;
        }
        s_ng = n;
    }
    __syncthreads();
    const int ng = s_ng;
    emit_node_items(w, tiles, nt, na, s_gs, ng, nodes, items, qcap, qf + 2 * kXcd);
}

// Tiles of window w that hold events; s_nt[0]: how many, s_nt[1]: the events
// of the fullest.
__device__ __forceinline__ void nonempty_tiles(int w, int T, const long long* seg_off, int* tiles, int* s_nt,
                                               ScanLds* sc, int& turn) {
    const int t = threadIdx.x;
    int ne = 0, size = 0;
    if (t < T) {
        const long long seg = (long long)w * T + t;
        size = (int)(seg_off[seg + 1] - seg_off[seg]);  // fewer than 2^28
        ne = size > 0 ? 1 : 0;
    }
    if (threadIdx.x == 0) s_nt[1] = 0;
    int tot;
    const int r = block_rank(ne != 0, sc, turn, tot);
    if (ne) {
        tiles[r] = t;
        atomicMax(&s_nt[1], size);
    }
    if (threadIdx.x == 0) *s_nt = tot;
    __syncthreads();
}

__global__ __launch_bounds__(NTF) void k_init(Search sp, const WinParam* __restrict__ wp,
                                              const float* __restrict__ seeds, int B, WinState* __restrict__ st,
                                              Sel* __restrict__ sel, Hyp* __restrict__ hyps, int* __restrict__ act,
                                              Item* __restrict__ items, int qcap, Queue* __restrict__ q, int T,
                                              const long long* __restrict__ seg_off, InitCheck chk) {
    const int w = blockIdx.x;
    const unsigned top = 1u << sp.L;
    Sel* sl = sel + (long long)w * sp.F;
    __shared__ int s_nsel, s_nt[2];
    __shared__ ScanLds s_scan;
    int turn = 0;
    __shared__ int s_tiles[kMaxTiles];
    if (chk.wstat) {
        const int bad = chk.wstat[w] ? chk.wstat[w]
                        : chk.werr[w] ? -1                                  // ECMD_EINVAL
                        : seg_off[(long long)B * T] > chk.cap ? -2 : 0;     // ECMD_ENOMEM
        if (bad) {
            if (threadIdx.x == 0) {
                WinState s = WinState{};
                s.status = bad;
                st[w] = s;
            }
            return;
        }
    }
    if (threadIdx.x == 0) {
        WinState s = WinState{};
        s.Kinc_hi = -1;
        s.Kinc_lo = ~0ull;  // K_inc = -1: the first evaluated point replaces it
        s.j_inc = 0;
        s.active = 1;
        Sel root;
        root.ja = 0;
        root.jb = top;
        root.jc = top >> 1;
        root.kids = (top >= 4) ? 1u : 0u;
        root.lc = INFINITY;  // no evaluation yet: the root's children try the certificate
        root.ub = INFINITY;  // and no bound above them
        sl[0] = root;
        int n_sel = 1;
        if (seeds) {
            const float d = seeds[w];
            if (isfinite(d)) {
                const double span = (double)sp.d_hi - (double)sp.d_lo;
                const double v = ((double)d - (double)sp.d_lo) / span * (double)top;
                long long j = llround(v);
                j = j < 1 ? 1 : (j > (long long)top - 1 ? (long long)top - 1 : j);
                if ((unsigned)j != root.jc && sp.F > 1) {
                    Sel sd;
                    sd.ja = sd.jb = sd.jc = (unsigned)j;
                    sd.kids = 0;
                    sd.lc = 0.0f;
                    sd.ub = INFINITY;
                    sl[1] = sd;
                    n_sel = 2;
                }
                s.seeded = 1;
            }
        }
        s.n_sel = n_sel;
        s.nodes_expanded = 1;
        st[w] = s;
        s_nsel = n_sel;
    }
    __syncthreads();
    nonempty_tiles(w, T, seg_off, s_tiles, s_nt, &s_scan, turn);
    emit_hyps(sp, wp[w], w, T, s_tiles, s_nt[0], s_nt[1], sl, s_nsel, 0, 1, -1.0f, hyps + (long long)w * sp.HS,
              act + (long long)w * sp.HS, items, qcap, q, &s_scan, turn, false);
}

hipError_t launch_init(hipStream_t s, const Search& sp, const WinParam* wp, const float* seeds, int B,
                       WinState* st, Sel* sel, Hyp* hyps, int* act, Item* items, int qcap, Queue* q, int T,
                       const long long* seg_off, InitCheck chk) {
    if (B <= 0) return hipSuccess;
    k_init<<<B, NTF, 0, s>>>(sp, wp, seeds, B, st, sel, hyps, act, items, qcap, q, T, seg_off, chk);
    return hipGetLastError();
}

// The certificate a node's children can expect, from the node's own sums:
// U walk pixels over N_low events inside at both ends, i.e. mean walk
// length l = U / N_low - 1; a child's walks are about half as long, so its
// certificate is about N_low^2 (l/2)(l/2 + 2).  Only the choice between the
// certificate and the exact bound depends on it, never a result.
__device__ __forceinline__ float child_cert(unsigned long long U, long long N) {
    if (N <= 0) return 0.0f;
    const float l = fmaxf((float)U / (float)N - 1.0f, 0.0f) * 0.5f;
    return (float)N * (float)N * l * (l + 2.0f);
}

// Append the children whose keep flag is set to the queue (array order),
// noting an overflow of the capacity.
__device__ __forceinline__ void queue_append(Node* fr, int& n, int CAP, bool keep, const Node& nd, ScanLds* sc,
                                             int& turn, int& overflow) {
    int tot;
    const int r = block_rank(keep, sc, turn, tot);
    if (keep && n + r < CAP) fr[n + r] = nd;
    if (n + tot > CAP) overflow = 1;
    n = min(n + tot, CAP);
}

// One frontier launch of Algorithm 1 for window blockIdx.x: absorb the
// evaluated hypotheses, update the incumbent and queue the improvable
// children (phase 0), then drop queued nodes that can no longer improve,
// decide whether to stop, select the next nodes and emit their hypotheses
// (phase 1).  A child evaluated by its endpoint certificate L <= K_bar is
// queued with key L (marked kNodeCert) when L already shows it improvable;
// otherwise it is queued in its place as a placeholder (kNodeRepair) and its
// exact bound goes to the next evaluation launch, so the queue keeps the
// exact search's order; only then does the window's phase 1 wait for the
// next frontier launch (WinState::n_repair > 0).  Windows are independent, so
// each takes its own steps: a step without a failed certificate costs one
// evaluation and one frontier launch.  A small search is a chain of launches
// (with a launch per phase and an evaluation between them, usually empty, one
// 10k-event window of 128x128 took 901 us, with this 763 us; 32 windows of
// 346x260 7.60 and 7.29 ms).  Every order below is the array order (scans, no
// atomic slot races), so the search is reproducible.
__global__ __launch_bounds__(NTF) void k_frontier(
    Search sp, const WinParam* __restrict__ wp, int B, int T, const long long* __restrict__ seg_off,
    WinState* __restrict__ st, Node* __restrict__ front, Sel* __restrict__ sel, Hyp* __restrict__ hyps,
    int* __restrict__ act, const Part* __restrict__ part, Item* __restrict__ items, int qcap,
    Queue* __restrict__ qf, int* __restrict__ n_active) {
    const int w = blockIdx.x, tid = threadIdx.x;
    __shared__ WinState s;
    __shared__ long long s_hi[NTF];
    __shared__ unsigned long long s_lo[NTF];
    __shared__ unsigned s_j[NTF];
    __shared__ int s_tiles[kMaxTiles], s_nt[2];
    __shared__ ScanLds s_scan;
    int turn = 0;
    __shared__ int s_hist[130];
    __shared__ int s_bstar, s_quota, s_stop, s_take, s_anycert, s_ubmax;
    __shared__ unsigned long long s_pix;
    __shared__ long long s_nbound, s_pruned, s_ncert;
    if (tid == 0) s = st[w];
    __syncthreads();
    if (!s.active || s.steps >= sp.max_steps) return;
    const int F = sp.F, HS = sp.HS, CAP = sp.CAP;
    const long long M = sp.M;
    const WinParam p = wp[w];
    Node* fr = front + (long long)w * CAP;
    Sel* sl = sel + (long long)w * F;
    Hyp* hy = hyps + (long long)w * HS;
    int* ac = act + (long long)w * HS;
    const Part* pw = part + (long long)w * HS * T;
    nonempty_tiles(w, T, seg_off, s_tiles, s_nt, &s_scan, turn);
    const int nt = s_nt[0];
    i128 Kinc = mk128(s.Kinc_hi, s.Kinc_lo);
    unsigned jinc = s.j_inc;
    const bool repaired = s.n_repair > 0;  // phase 0 of this step is done
    if (!repaired) {
        const int n_sel = s.n_sel;

        // (1) centre points: lexicographic max of (K, -j) with the incumbent
        i128 bK = Kinc;
        unsigned bJ = jinc;
        for (int i = tid; i < n_sel; i += NTF) {
            unsigned long long S, U;
            long long N;
            slot_sums(pw, i, T, s_tiles, nt, S, N, U);
            const i128 K = (i128)M * (i128)S - (i128)N * (i128)N;
            const unsigned jc = sl[i].jc;
            if (K > bK || (K == bK && jc < bJ)) { bK = K; bJ = jc; }
        }
        block_argmax(bK, bJ, s_hi, s_lo, s_j);
        Kinc = bK;
        jinc = bJ;
        if (tid == 0) {
            sp128(Kinc, s.Kinc_hi, s.Kinc_lo);
            s.j_inc = jinc;
            s.point_evals += n_sel;
            s.event_hyp += (long long)n_sel * p.n_events;
            s_pix = 0;
            s_nbound = 0;
            s_pruned = 0;
            s_ncert = 0;
        }
        __syncthreads();

        // (2) children of the expanded nodes, appended in slot order
        int n = s.n_front;
        const int n0 = n;
        int overflow = 0, nrep = 0;
        for (int c0 = 0; c0 < 2 * n_sel; c0 += NTF) {
            const int c = c0 + tid;
            bool keep = false, rep = false;
            Node nd;
            if (c < 2 * n_sel && sl[c >> 1].kids) {
                unsigned long long S, U;
                long long N;
                slot_sums(pw, F + c, T, s_tiles, nt, S, N, U);
                const Sel x = sl[c >> 1];
                nd.ja = (c & 1) ? x.jc : x.ja;
                nd.jb = (c & 1) ? x.jb : x.jc;
                nd.ub = x.ub;  // every grid point of the child is one of the parent's
                if (hy[F + c].kind == HYP_CERT) {
                    // S holds U (walk pixels of the events inside at both ends),
                    // a lower bound of sum H_bar.  Two lower bounds of K_bar:
                    // M S_bar >= U^2 (Cauchy-Schwarz over the M cells), and, as
                    // the centre d_c of the expanded node (evaluated this step:
                    // S_c, N_c) is an end of the child, H_bar >= H(d_c) pixel by
                    // pixel, so with X = H_bar - H(d_c) >= 0,
                    // S_bar >= S_c + (sum X)^2 / M and sum X >= U - N_c.
                    unsigned long long Sc, Uc;
                    long long Nc;
                    slot_sums(pw, c >> 1, T, s_tiles, nt, Sc, Nc, Uc);
                    const i128 N2 = (i128)N * (i128)N;
                    const i128 L1 = (i128)S * (i128)S - N2;
                    const i128 X = (long long)S > Nc ? (i128)((long long)S - Nc) : (i128)0;
                    const i128 L2 = (i128)M * (i128)Sc + X * X - N2;
                    const i128 Lb = L1 > L2 ? L1 : L2;
                    nd.lc = child_cert(S, N);
                    keep = true;
                    if (improvable(Lb, nd.ja, Kinc, jinc)) {
                        sp128(Lb, nd.khi, nd.klo);
                        nd.jb |= kNodeCert;
                        atomicAdd((unsigned long long*)&s_ncert, 1ull);
                    } else {
                        rep = true;
                        nd.khi = kNodeRepair;
                        nd.klo = (unsigned long long)(F + c);
                    }
                } else {
                    atomicAdd(&s_pix, U);
                    atomicAdd((unsigned long long*)&s_nbound, 1ull);
                    const i128 Kb = (i128)M * (i128)S - (i128)N * (i128)N;
                    sp128(Kb, nd.khi, nd.klo);
                    nd.lc = child_cert(U, N);
                    keep = improvable(Kb, nd.ja, Kinc, jinc);
                    if (!keep) atomicAdd((unsigned long long*)&s_pruned, 1ull);
                }
            }
            queue_append(fr, n, CAP, keep, nd, &s_scan, turn, overflow);
            // the children to bound exactly between the phases
            int tot;
            const int r = block_rank(rep, &s_scan, turn, tot);
            if (rep) {
                hy[F + c].kind = HYP_INTERVAL;  // same end rates
                ac[nrep + r] = F + c;
            }
            nrep += tot;
        }
        __syncthreads();
        if (tid == 0) {
            s.bound_evals += s_nbound;
            s.event_hyp += s_nbound * p.n_events;
            s.pixel_updates += (long long)s_pix;
            s.nodes_pruned += s_pruned;
            s.cert_evals += s_ncert;
            s.n_front = n;
            s.n_front0 = n0;
            s.overflow = overflow;
            s.n_repair = nrep;
            if (nrep) st[w] = s;
        }
        if (nrep) {
            emit_items(sp, w, s_tiles, nt, nrep, items, qcap, qf);
            return;
        }
    }
    __syncthreads();
    if (tid == 0) {
        s_pix = 0;
        s_nbound = 0;
        s_pruned = 0;
        s_anycert = 0;
        s_ubmax = 0;  // 0.0f
    }
    for (int b = tid; b < 130; b += NTF) s_hist[b] = 0;
    __syncthreads();

    // (2') the exact bounds of the children whose certificate failed, into
    // their placeholders (this step's children sit at [n_front0, n_front));
    // one that cannot improve is dropped below with the other such nodes
    const int n = s.n_front;
    const int overflow = s.overflow;
    if (repaired) {
        for (int i = s.n_front0 + tid; i < n; i += NTF) {
            Node nd = fr[i];
            if (nd.khi != kNodeRepair) continue;
            unsigned long long S, U;
            long long N;
            slot_sums(pw, (int)nd.klo, T, s_tiles, nt, S, N, U);
            atomicAdd(&s_pix, U);
            atomicAdd((unsigned long long*)&s_nbound, 1ull);
            const i128 Kb = (i128)M * (i128)S - (i128)N * (i128)N;
            sp128(Kb, nd.khi, nd.klo);
            if (!improvable(Kb, nd.ja, Kinc, jinc)) atomicAdd((unsigned long long*)&s_pruned, 1ull);
            fr[i] = nd;
        }
    }
    __syncthreads();

    // (3) which queued nodes can still improve; histogram of their gap
    // sizes; the node Algorithm 1 would pop next (largest bound, ties to the
    // smaller grid index; queued intervals are disjoint, so ja names it).
    // A certificate key is only a lower bound of K_bar: such a node's points
    // are bounded above by its ub (an ancestor's exact bound), and the gap
    // certified while it is queued is taken from that (infinite when some
    // such node has no exactly bounded ancestor).
    i128 best_gap = -1;
    unsigned best_ja = 0xFFFFFFFFu;
    for (int i = tid; i < n; i += NTF) {
        const Node nd = fr[i];
        const i128 k = mk128(nd.khi, nd.klo);
        if (improvable(k, nd.ja, Kinc, jinc)) {
            const i128 gap = k - Kinc;
            atomicAdd(&s_hist[bitlen128(gap)], 1);
            if (nd.jb & kNodeCert) {
                s_anycert = 1;
                atomicMax(&s_ubmax, __float_as_int(nd.ub));  // ub >= 0: int order is float order
            }
            if (gap > best_gap || (gap == best_gap && nd.ja < best_ja)) {
                best_gap = gap;
                best_ja = nd.ja;
            }
        }
    }
    block_argmax(best_gap, best_ja, s_hi, s_lo, s_j);
    // the gap classes from the largest down, one thread each: `before` =
    // improvable nodes in larger classes, n_keep = all of them
    const int hb = tid < 130 ? s_hist[129 - tid] : 0;
    int n_keep = 0;
    const int before = block_scan(hb, &s_scan, turn, n_keep);
    if (tid == 0) {
        s.bound_evals += s_nbound;
        s.event_hyp += s_nbound * p.n_events;
        s.pixel_updates += (long long)s_pix;
        s.nodes_pruned += s_pruned;
        // the gap certified so far (queued and selected nodes), kept for a
        // search that is cut short after this step (-1: none certified)
        i128 gap = best_gap < 0 ? (i128)0 : best_gap;
        bool gap_inf = false;
        if (s_anycert) {
            const float u = __int_as_float(s_ubmax);
            if (!(u < INFINITY)) {
                gap_inf = true;
            } else {
                const i128 g = ceil_i128(u) - Kinc;
                if (g > gap) gap = g;
            }
        }
        sp128(gap_inf ? (i128)-1 : gap, s.gap_hi, s.gap_lo);
        int stop = 0;
        if (overflow) {
            s.status = -5;  // ECMD_EFRONTIER
            sp128((i128)-1, s.gap_hi, s.gap_lo);
            stop = 1;
        } else if (n_keep == 0) {
            s.status = 0;
            s.gap_hi = 0;
            s.gap_lo = 0;
            stop = 1;
        } else if (sp.gamma_key >= 0 && !gap_inf && gap <= (i128)sp.gamma_key) {
            s.status = 0;
            sp128(gap, s.gap_hi, s.gap_lo);
            s.nodes_pruned += n_keep;
            stop = 1;
        }
        int take = min(F, n_keep);
        if (!stop && sp.max_nodes > 0) {
            const long long left = sp.max_nodes - s.nodes_expanded;
            if (left <= 0) {
                s.status = -4;  // ECMD_EBUDGET
                sp128(best_gap, s.gap_hi, s.gap_lo);
                stop = 1;
            } else if (left < take) {
                take = (int)left;
            }
        }
        s_stop = stop;
        s_take = take;
    }
    __syncthreads();
    // take every node of a larger gap class and the first `quota` of class
    // b*, the class where the running count reaches `take`
    if (!s_stop && tid < 130 && before < s_take && s_take <= before + hb) {
        s_bstar = 129 - tid;
        s_quota = s_take - before;
    }
    __syncthreads();
    if (s_stop) {
        if (tid == 0) {
            s.active = 0;
            s.n_sel = 0;
            s.n_front = 0;
            st[w] = s;
            atomicSub(n_active, 1);
        }
        return;
    }

    // (4) split the queue into the nodes expanded now and the rest (in
    // place).  One node: Algorithm 1's pop, the best node found above.
    // More: every node of the larger gap classes and the first `quota`
    // of class b* in queue order.
    const bool pop_one = s_take == 1;
    int out = 0, nsel = 0, inb = 0, nkids = 0;
    for (int base = 0; base < n; base += NTF) {
        const int i = base + tid;
        Node nd = Node{};
        int keep = 0, cand = 0, big = 0;
        if (i < n) {
            nd = fr[i];
            const i128 k = mk128(nd.khi, nd.klo);
            if (improvable(k, nd.ja, Kinc, jinc)) {
                if (pop_one) {
                    big = nd.ja == best_ja;
                    keep = !big;
                } else {
                    const int b = bitlen128(k - Kinc);
                    big = b > s_bstar;
                    cand = b == s_bstar;
                    keep = !big && !cand;
                }
            }
        }
        int tot_c;
        const int rc = block_rank(cand != 0, &s_scan, turn, tot_c);
        const int take = big || (cand && inb + rc < s_quota);
        if (cand && !take) keep = 1;
        inb += tot_c;
        const unsigned jb = nd.jb & ~kNodeCert;
        const int kids = take && jb - nd.ja >= 4;
        int tot_k, tot_t, tot_d;
        const int rk = block_rank(keep != 0, &s_scan, turn, tot_k);
        const int rt = block_rank(take != 0, &s_scan, turn, tot_t);
        block_rank(kids != 0, &s_scan, turn, tot_d);
        if (keep) fr[out + rk] = nd;
        if (take) {
            Sel x;
            x.ja = nd.ja;
            x.jb = jb;
            x.jc = (nd.ja + jb) >> 1;
            x.kids = kids ? 1u : 0u;
            x.lc = nd.lc;
            x.ub = (nd.jb & kNodeCert) ? nd.ub : ub_float(mk128(nd.khi, nd.klo));
            sl[nsel + rt] = x;
        }
        out += tot_k;
        nsel += tot_t;
        nkids += tot_d;
    }
    __syncthreads();
    if (tid == 0) {
        s.n_front = out;
        s.n_sel = nsel;
        s.nodes_expanded += nsel;
        s.steps += 1;
        s.n_repair = 0;
        st[w] = s;
    }
    __syncthreads();
    if (s.steps >= sp.max_steps) return;  // cut short: nothing more is evaluated
    emit_hyps(sp, p, w, T, s_tiles, nt, s_nt[1], sl, nsel, out, nkids, (float)i128_to_double(Kinc), hyps + (long long)w * HS,
              act + (long long)w * HS, items, qcap, qf, &s_scan, turn, true);
}

// Grid range still alive in each active window: the queued nodes and those
// selected for the next step.  Every later hypothesis is a grid interval or
// point inside it and the warp is monotone in d, so events binned with this
// range still reach every tile they can reach for the rest of the search;
// binning again with it drops the guest copies that only the early, wide
// intervals needed.
__global__ __launch_bounds__(NTF) void k_live_range(Search sp, const WinState* __restrict__ st,
                                                    const Node* __restrict__ front, const Sel* __restrict__ sel,
                                                    WinParam* __restrict__ wp) {
    const int w = blockIdx.x, tid = threadIdx.x;
    __shared__ unsigned s_lo, s_hi;
    const WinState s = st[w];
    if (!s.active) return;
    if (tid == 0) {
        s_lo = 0xFFFFFFFFu;
        s_hi = 0u;
    }
    __syncthreads();
    const Node* fr = front + (long long)w * sp.CAP;
    const Sel* sl = sel + (long long)w * sp.F;
    unsigned lo = 0xFFFFFFFFu, hi = 0u;
    for (int i = tid; i < s.n_front; i += NTF) {
        lo = min(lo, fr[i].ja);
        hi = max(hi, fr[i].jb & ~kNodeCert);
    }
    for (int i = tid; i < s.n_sel; i += NTF) {
        lo = min(lo, sl[i].ja);
        hi = max(hi, sl[i].jb);
    }
    atomicMin(&s_lo, lo);
    atomicMax(&s_hi, hi);
    __syncthreads();
    if (tid == 0 && s_lo <= s_hi) {
        WinParam p = wp[w];
        p.r_lo = rate_of(grid_d(sp.d_lo, sp.d_hi, sp.L, s_lo), p.tau);
        p.r_hi = rate_of(grid_d(sp.d_lo, sp.d_hi, sp.L, s_hi), p.tau);
        set_guest_cuts(p);
        wp[w] = p;
    }
}

hipError_t launch_live_range(hipStream_t s, const Search& sp, const WinState* st, const Node* front, const Sel* sel,
                             WinParam* wp, int B) {
    if (B <= 0) return hipSuccess;
    k_live_range<<<B, NTF, 0, s>>>(sp, st, front, sel, wp);
    return hipGetLastError();
}

hipError_t launch_frontier(hipStream_t s, const Search& sp, const WinParam* wp, int B, int T,
                           const long long* seg_off, WinState* st, Node* front, Sel* sel, Hyp* hyps, int* act,
                           const Part* part, Item* items, int qcap, Queue* q_fill, int* n_active, hipEvent_t t0,
                           hipEvent_t t1) {
    if (B <= 0) return hipSuccess;
    hipExtLaunchKernelGGL(k_frontier, dim3(B), dim3(NTF), 0u, s, t0, t1, 0u, sp, wp, B, T, seg_off, st, front, sel,
                          hyps, act, part, items, qcap, q_fill, n_active);
    return hipGetLastError();
}

// ------------------------------------------------------------ asynchronous plan

// The host-side checks of a synchronous call, made on the device for the
// launches of a plan: window w is valid when its offsets are non-negative and
// non-decreasing, it holds fewer than 2^28 events, its exact sums fit 64
// bits, tau > 0 is finite and d_hi * tau < 1 (eq. (11)).  n: its events.
__device__ __forceinline__ bool window_ok(const long long* off, const float* tau, int w, float d_hi, int W, int H,
                                          long long& n) {
    const long long a = off[w], b = off[w + 1];
    n = b - a;
    if (a < 0 || n < 0 || n >= kMaxWindowEvents) return false;
    const double bound = (double)n * (double)n * 2.0 * ((double)W + H + 3.0);
    if (bound >= 9.0e18) return false;
    const float t = tau[w];
    if (!(t > 0.0f) || !isfinite(t)) return false;
    return d_hi * t < 1.0f;
}

constexpr int kCheckThreads = 1024;

// One workgroup: wstat[w] = 0 for a valid window, else ECMD_EINVAL (every
// window when the valid ones hold more than max_events events); blk = the
// exclusive prefix of the prep blocks (`chunk` events each) of the valid
// windows, B + 1 entries; werr, all kQueues queues and n_active cleared.
// Thread k checks the windows [k * per, (k + 1) * per).
__global__ __launch_bounds__(kCheckThreads) void k_plan_check(
    const long long* __restrict__ off, const float* __restrict__ tau, int B, float d_hi, int W, int H,
    long long max_events, int chunk, int* __restrict__ wstat, int* __restrict__ werr, int* __restrict__ blk,
    Queue* __restrict__ q, int* __restrict__ n_active) {
    __shared__ long long s_ev[kCheckThreads / 64];
    __shared__ int s_scan[kCheckThreads];
    const int tid = threadIdx.x;
    if (tid < kQueues) {
        q[tid].n_items = 0;
        q[tid].next = 0;
    }
    if (tid == 0) *n_active = 0;
    const int per = (B + kCheckThreads - 1) / kCheckThreads;
    const int w0 = min(B, tid * per), w1 = min(B, w0 + per);
    long long ev = 0;
    int nb = 0;
    for (int w = w0; w < w1; ++w) {
        long long n;
        if (window_ok(off, tau, w, d_hi, W, H, n)) {
            ev += n;
            nb += (int)((n + chunk - 1) / chunk);
        }
    }
    // events of the valid windows: wave sums, then the workgroup's
    for (int o = 32; o > 0; o >>= 1) ev += __shfl_xor(ev, o);
    if ((tid & 63) == 0) s_ev[tid >> 6] = ev;
    // inclusive scan of the block counts (Hillis-Steele)
    s_scan[tid] = nb;
    __syncthreads();
    for (int o = 1; o < kCheckThreads; o <<= 1) {
        const int a = tid >= o ? s_scan[tid - o] : 0;
        __syncthreads();
        s_scan[tid] += a;
        __syncthreads();
    }
    long long total = 0;
    for (int k = 0; k < kCheckThreads / 64; ++k) total += s_ev[k];
    const bool over = total > max_events;
    int run = over ? 0 : s_scan[tid] - nb;
    for (int w = w0; w < w1; ++w) {
        long long n;
        const bool ok = window_ok(off, tau, w, d_hi, W, H, n) && !over;
        wstat[w] = ok ? 0 : -1;  // ECMD_EINVAL
        werr[w] = 0;
        blk[w] = run;
        if (ok) run += (int)((n + chunk - 1) / chunk);
    }
    if (tid == kCheckThreads - 1) blk[B] = over ? 0 : s_scan[tid];
}

__global__ void k_fill_u32(unsigned* __restrict__ p, long long n, unsigned v) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

// Per-window results of a plan launch, written to `out` (device memory or
// pinned host memory), with the same arithmetic as a synchronous call.
__global__ void k_plan_results(Search sp, int B, const WinState* __restrict__ st, const long long* __restrict__ off,
                               const float* __restrict__ tau, ecmd_result* __restrict__ out) {
    const int w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= B) return;
    const WinState s = st[w];
    ecmd_result r = {};
    r.L = (uint32_t)sp.L;
    if (s.status == -1 || s.status == -2) {  // rejected before the search: only the status
        r.status = s.status;
        out[w] = r;
        return;
    }
    r.status = s.active ? -4 : s.status;  // still running when the steps ran out: ECMD_EBUDGET
    r.j_star = s.j_inc;
    r.d_hat = grid_d(sp.d_lo, sp.d_hi, sp.L, s.j_inc);
    r.K_lo = s.Kinc_lo;
    r.K_hi = s.Kinc_hi;
    const double M2 = (double)sp.M * (double)sp.M;
    r.contrast = i128_to_double(mk128(s.Kinc_hi, s.Kinc_lo)) / M2;
    const double t = (double)tau[w];
    r.d_end = (double)r.d_hat / (1.0 - (double)r.d_hat * t);
    // no finite gap certified: a frontier overflow, or a search cut short
    // while a node kept on its endpoint certificate, with no exactly bounded
    // ancestor, was queued
    r.gap = (s.status == -5 || s.gap_hi < 0) ? (double)INFINITY : i128_to_double(mk128(s.gap_hi, s.gap_lo)) / M2;
    r.n_events = off[w + 1] - off[w];
    r.nodes_expanded = s.nodes_expanded;
    r.nodes_pruned = s.nodes_pruned;
    r.point_evals = s.point_evals;
    r.bound_evals = s.bound_evals;
    r.event_hyp_evals = s.event_hyp;
    r.pixel_updates = s.pixel_updates;
    r.steps = s.steps;
    r.seeded = s.seeded;
    r.bound_certs = s.cert_evals;
    out[w] = r;
}

hipError_t launch_plan_check(hipStream_t s, const long long* off, const float* tau, int B, float d_hi, int W, int H,
                             long long max_events, int chunk, int* wstat, int* werr, int* blk, Queue* q,
                             int* n_active) {
    k_plan_check<<<1, kCheckThreads, 0, s>>>(off, tau, B, d_hi, W, H, max_events, chunk, wstat, werr, blk, q,
                                             n_active);
    return hipGetLastError();
}

hipError_t launch_fill_u32(hipStream_t s, unsigned* p, long long n, unsigned v) {
    if (n <= 0) return hipSuccess;
    const long long nb = (n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192;
    k_fill_u32<<<(int)nb, 256, 0, s>>>(p, n, v);
    return hipGetLastError();
}

hipError_t launch_plan_results(hipStream_t s, const Search& sp, int B, const WinState* st, const long long* off,
                               const float* tau, ecmd_result* out) {
    if (B <= 0) return hipSuccess;
    k_plan_results<<<(B + 255) / 256, 256, 0, s>>>(sp, B, st, off, tau, out);
    return hipGetLastError();
}

// ------------------------------------------------------------ probes

__global__ void k_probe_items(const float* __restrict__ d_a, const float* __restrict__ d_b, int m, float tau, int T,
                              Hyp* __restrict__ hyps, int* __restrict__ act, Item* __restrict__ items,
                              Queue* __restrict__ q) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x, n = (long long)m * T;
    if (i < 2 * kXcd) {
        q[i].n_items = i == 0 ? (int)n : 0;
        q[i].next = 0;
    }
    if (i < m) {
        Hyp h;
        h.ra = rate_of(d_a[i], tau);
        h.rb = d_b ? rate_of(d_b[i], tau) : h.ra;
        h.kind = d_b ? HYP_INTERVAL : HYP_POINT;
        h.pad = 0;
        hyps[i] = h;
        act[i] = (int)i;
    }
    if (i < n) items[i] = Item{0, (int)(i % T), (int)(i / T), 1};
}

hipError_t launch_probe_items(hipStream_t s, const float* d_a, const float* d_b, int m, float tau, int T, Hyp* hyps,
                              int* act, Item* items, Queue* q) {
    const long long n = std::max((long long)m * T, (long long)(2 * kXcd));
    k_probe_items<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(d_a, d_b, m, tau, T, hyps, act, items, q);
    return hipGetLastError();
}

__global__ void k_probe_sums(int m, int T, const long long* __restrict__ seg_off, const Part* __restrict__ part,
                             unsigned long long* __restrict__ S, long long* __restrict__ N) {
    const int h = blockIdx.x * blockDim.x + threadIdx.x;
    if (h >= m) return;
    unsigned long long a = 0, b = 0;
    for (int t = 0; t < T; ++t) {
        if (seg_off[t + 1] == seg_off[t]) continue;  // empty tile: not evaluated, contributes 0
        const Part q = part[(long long)h * T + t];
        a += q.S;
        b += q.N;
    }
    S[h] = a;
    N[h] = (long long)b;
}

hipError_t launch_probe_sums(hipStream_t s, int m, int T, const long long* seg_off, const Part* part,
                             unsigned long long* S, long long* N) {
    k_probe_sums<<<(m + 63) / 64, 64, 0, s>>>(m, T, seg_off, part, S, N);
    return hipGetLastError();
}

__global__ void k_probe_pixels(const float* __restrict__ x, const float* __restrict__ y,
                               const float* __restrict__ t_rel, long long n, float tau, float d, int W,
                               int H, float cx, float cy, int* __restrict__ pix) {
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float r = rate_of(d, tau);
    float ax = (x[i] - cx) * (tau - t_rel[i]);
    float ay = (y[i] - cy) * (tau - t_rel[i]);
    float xw = fmaf(ax, r, x[i]), yw = fmaf(ay, r, y[i]);
    pix[i] = inside(xw, yw, (float)W, (float)H) ? (int)floorf(yw) * W + (int)floorf(xw) : -1;
}

hipError_t launch_probe_pixels(hipStream_t s, const float* x, const float* y, const float* t_rel, long long n,
                               float tau, float d, int W, int H, float cx, float cy, int* pix) {
    if (n <= 0) return hipSuccess;
    k_probe_pixels<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(x, y, t_rel, n, tau, d, W, H, cx, cy, pix);
    return hipGetLastError();
}

// ------------------------------------------------------------ window selection

constexpr int kSelThreads = 1024;

__global__ __launch_bounds__(kSelThreads) void k_select_count(const double* __restrict__ t, long long n, double t0,
                                                              double t1, int* __restrict__ blk_cnt) {
    __shared__ int s_n;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    long long i = (long long)blockIdx.x * kSelThreads + threadIdx.x;
    if (i < n && t[i] >= t0 && t[i] <= t1) atomicAdd(&s_n, 1);
    __syncthreads();
    if (threadIdx.x == 0) blk_cnt[blockIdx.x] = s_n;
}

__global__ __launch_bounds__(1024) void k_select_scan(int nb, int* __restrict__ blk_cnt, long long* __restrict__ total) {
    __shared__ long long s[1024];
    __shared__ long long carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base < nb; base += 1024) {
        int k = base + threadIdx.x;
        long long v = k < nb ? blk_cnt[k] : 0;
        s[threadIdx.x] = v;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            long long a = threadIdx.x >= (unsigned)o ? s[threadIdx.x - o] : 0;
            __syncthreads();
            s[threadIdx.x] += a;
            __syncthreads();
        }
        long long incl = s[threadIdx.x] + carry;
        if (k < nb) blk_cnt[k] = (int)(incl - v);
        __syncthreads();
        if (threadIdx.x == 1023) carry = incl;
        __syncthreads();
    }
    if (threadIdx.x == 0) *total = carry;
}

__global__ __launch_bounds__(kSelThreads) void k_select_write(const float* __restrict__ x, const float* __restrict__ y,
                                                              const double* __restrict__ t,
                                                              const signed char* __restrict__ p, long long n,
                                                              double t0, double t1, const int* __restrict__ blk_off,
                                                              float* __restrict__ xo, float* __restrict__ yo,
                                                              float* __restrict__ to, signed char* __restrict__ po) {
    __shared__ int s[kSelThreads];
    long long i = (long long)blockIdx.x * kSelThreads + threadIdx.x;
    int keep = (i < n && t[i] >= t0 && t[i] <= t1) ? 1 : 0;
    s[threadIdx.x] = keep;
    __syncthreads();
    for (int o = 1; o < kSelThreads; o <<= 1) {
        int a = threadIdx.x >= (unsigned)o ? s[threadIdx.x - o] : 0;
        __syncthreads();
        s[threadIdx.x] += a;
        __syncthreads();
    }
    if (keep) {
        long long k = (long long)blk_off[blockIdx.x] + s[threadIdx.x] - 1;
        xo[k] = x[i];
        yo[k] = y[i];
        to[k] = (float)(t[i] - t0);
        if (p) po[k] = p[i];
    }
}

hipError_t launch_select(hipStream_t s, const float* x, const float* y, const double* t, const signed char* p,
                         long long n, double t0, double t1, float* xo, float* yo, float* to, signed char* po,
                         int* blk_cnt, long long* total) {
    const int nb = (int)((n + kSelThreads - 1) / kSelThreads);
    if (nb > 0) {
        k_select_count<<<nb, kSelThreads, 0, s>>>(t, n, t0, t1, blk_cnt);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    k_select_scan<<<1, 1024, 0, s>>>(nb, blk_cnt, total);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || nb == 0) return e;
    k_select_write<<<nb, kSelThreads, 0, s>>>(x, y, t, p, n, t0, t1, blk_cnt, xo, yo, to, po);
    return hipGetLastError();
}

// ------------------------------------------------------------ learned-incumbent input

__device__ __forceinline__ uint16_t bf16_rne(float v) {
    unsigned u = __float_as_uint(v);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

constexpr int kGrid = 64;

// A workgroup clears and adds up to 4096 counters however few events it bins,
// so with many events its chunk is large; with few it is smaller, or the chip
// stays empty; and for windows that hardly fill a workgroup's counters one of
// 256 threads is started sooner.  us a call with 256 threads and 4096 events,
// 1024 and 8192, 1024 and 32768: one window of 100k events 57.1, 56.0, 62.3, of
// 500k 58.7, 55.5, 62.0; 16 of 300k 73.1, 66.3, 68.5; 64 of 100k 78.7, 69.6,
// 71.3; 16 of 1M 104, 84, 77; 64 of 400k 133, 102, 96; 512 of 5000 73.0, 66.2,
// 66.0; 4096 of 1000 122, 130, 129; 4096 of 100 98, 111, 111.
constexpr int kDownSmall = 4096, kDownMid = 8192, kDownLarge = 32768;
constexpr long long kDownMany = 8000000, kDownPerWindow = 2048;
int down_chunk(long long n_events, int B) {
    return n_events < kDownPerWindow * B ? kDownSmall : n_events < kDownMany ? kDownMid : kDownLarge;
}

__global__ __launch_bounds__(1024) void k_downsample_count(const float* __restrict__ x,
                                                          const float* __restrict__ y,
                                                          const long long* __restrict__ offsets, int B,
                                                          int W, int H, const int* __restrict__ blk_start,
                                                          int chunk, unsigned* __restrict__ counts) {
    __shared__ unsigned s_cnt[kGrid * kGrid];
    for (int k = threadIdx.x; k < kGrid * kGrid; k += blockDim.x) s_cnt[k] = 0;
    __syncthreads();
    const int w = window_of_block(blk_start, B, blockIdx.x);
    const int c = blockIdx.x - blk_start[w];
    const long long beg = offsets[w] + (long long)c * chunk;
    const long long end = min(beg + chunk, offsets[w + 1]);
    const float Wf = (float)W, Hf = (float)H, G = (float)kGrid;
    for (long long i = beg + threadIdx.x; i < end; i += blockDim.x) {
        int bx = (int)floorf((x[i] * G) / Wf);
        int by = (int)floorf((y[i] * G) / Hf);
        bx = min(max(bx, 0), kGrid - 1);
        by = min(max(by, 0), kGrid - 1);
        atomicAdd(&s_cnt[by * kGrid + bx], 1u);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < kGrid * kGrid; k += blockDim.x)
        if (s_cnt[k]) atomicAdd(&counts[(long long)w * kGrid * kGrid + k], s_cnt[k]);
}

__global__ void k_downsample_finish(const unsigned* __restrict__ counts, const long long* __restrict__ offsets,
                                    int B, uint16_t* __restrict__ out) {
    const int w = blockIdx.x;
    const long long n = offsets[w + 1] - offsets[w];
    const float scale = n > 0 ? (float)(kGrid * kGrid) / (float)n : 0.0f;
    for (int k = threadIdx.x; k < kGrid * kGrid; k += blockDim.x)
        out[(long long)w * kGrid * kGrid + k] = bf16_rne((float)counts[(long long)w * kGrid * kGrid + k] * scale);
}

hipError_t launch_downsample(hipStream_t s, const float* x, const float* y, const long long* offsets, int B,
                             int W, int H, const int* blk_start, int nblk, int chunk, unsigned* counts,
                             uint16_t* out) {
    if (B <= 0) return hipSuccess;
    if (nblk > 0) {
        k_downsample_count<<<nblk, chunk == kDownSmall ? 256 : 1024, 0, s>>>(x, y, offsets, B, W, H, blk_start, chunk, counts);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    k_downsample_finish<<<B, 256, 0, s>>>(counts, offsets, B, out);
    return hipGetLastError();
}

}  // namespace ecmd
