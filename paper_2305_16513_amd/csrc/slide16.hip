// sws_slide1d_16 — sliding window sums (Section 2.2, Eq. 3) on bf16 / fp16 storage.
//
// The segment prefix / suffix scheme of the fp32 kernel (the block form of Section 3's
// Algorithm 2): a wavefront owns a tile of 1024 consecutive inputs cut into segments of
// S = w - 1 elements, builds the in-segment prefix sums Pre and suffix sums Suf, and every output
// costs one more (+): y[q] = Suf[q] (+) Pre[q+S].  A lane loads and stores EIGHT elements at a time (128 bits) and scans
// sixteen consecutive ones; scans and the combine are fp32, the results are rounded to nearest even once.  With half the
// bytes per element the kernel is bound by instruction issue and latency rather than by HBM, so LDS carries as little
// as it can: the inputs as they are (16 bits), the prefix sums, the 16-bit results — the suffix sums stay in the registers
// of the lane whose outputs need them.  17 KB of LDS traffic and 4 KB of LDS per 1024 elements; with inputs staged as
// fp32 and both scans in LDS (26 and 8 KB) [900,30000] w = 64 took 28.9 us against 24.0, [186479,422] w = 39 192
// against 151, [8192,16384] w = 64 129.1 against 127.9 (more wavefronts per SIMD than the four that 124 registers
// leave: spills, 365 us).  The next tile is requested before the current one is worked on and staged before its results
// are stored, with no load under a lane's condition on the way: the compiler waited for those at once, and for the stores
// of the tile before, so that nothing was in flight during a tile's arithmetic ([8192,16384] w = 64 128 us, now 93,
// 5.8 TB/s; [186479,422] w = 39 151 / 90, [50000,1000] w = 100 104 / 61).
// Windows up to 33 also have a kernel on shifted loads (eight outputs per lane straight from
// 128-bit loads, no LDS); it serves the windows up to 9 everywhere, and the others on short rows
// and small tensors, where 1024-element wave tiles fit badly.
// Plain rows only (no boundary rules, no chains of windows).
#include "sws_internal.h"

#include <type_traits>

namespace sws {

namespace {

constexpr int kThreads = 256;
constexpr int kWavesPerWg = kThreads / kWave;
constexpr int kC = 16;                               // consecutive elements a lane scans
constexpr int kN = kWave * kC;                       // inputs per wave tile
constexpr int kLine = 32;                            // 16-bit elements per 64-byte line

__device__ __forceinline__ float lane_read(float v, int src_lane)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute((src_lane & 63) << 2, __float_as_int(v)));
}

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS layout of a wave tile of prefix sums: 256 groups of 4 floats, group g stored at
//     g ^ ((g >> 3) & 3) ^ (((g >> 5) & 1) << 3).
// Conflict-free for chunks (lane l writes groups 4l .. 4l+3) and for the shifted groups 4l + S/4 .. of the combine.
__device__ __forceinline__ int lds_group(int g) { return g ^ ((g >> 3) & 3) ^ (((g >> 5) & 1) << 3); }

// 16-bit units (eight elements, 16 bytes) of the same memory: lane l touches units 64 j + l on the way in and out and units
// 2l, 2l + 1 as its chunk; exchanging even and odd units in every other run of sixteen keeps both conflict-free.
__device__ __forceinline__ int lds_unit(int u) { return u ^ ((u >> 4) & 1); }

// In-segment scan step, the reset folded into arithmetic (one VALU op for ADD, two for MAX / MIN).
template <int OP> struct SegStep;
template <> struct SegStep<SWS_OP_ADD> {
    static __device__ __forceinline__ float mask(bool start) { return start ? 0.0f : 1.0f; }
    static __device__ __forceinline__ float f(float acc, float m, float x) { return __builtin_fmaf(acc, m, x); }
};
template <> struct SegStep<SWS_OP_MAX> {
    static __device__ __forceinline__ float mask(bool start) { return start ? -__builtin_huge_valf() : __builtin_huge_valf(); }
    static __device__ __forceinline__ float f(float acc, float m, float x) { return __builtin_fmaxf(__builtin_fminf(acc, m), x); }
};
template <> struct SegStep<SWS_OP_MIN> {
    static __device__ __forceinline__ float mask(bool start) { return start ? __builtin_huge_valf() : -__builtin_huge_valf(); }
    static __device__ __forceinline__ float f(float acc, float m, float x) { return __builtin_fminf(__builtin_fmaxf(acc, m), x); }
};

typedef float v8f __attribute__((ext_vector_type(8)));

// Eight 16-bit elements <-> eight floats.  Widening is exact; narrowing rounds to nearest even.
template <typename T> struct Io {
    typedef T v8 __attribute__((ext_vector_type(8)));
    typedef v8 v8_u __attribute__((aligned(2)));
    static __device__ __forceinline__ v8 load_raw(const T *p) { return *(const v8_u *)p; }
    static __device__ __forceinline__ v8f widen(v8 r) { return __builtin_convertvector(r, v8f); }
    static __device__ __forceinline__ v8f load8(const T *p) { return widen(load_raw(p)); }
    static __device__ __forceinline__ float load1(const T *p) { return (float)*p; }
    static __device__ __forceinline__ void store1(T *p, float v) { *p = (T)v; }
    static __device__ __forceinline__ v8 narrow(v8f o) { return __builtin_convertvector(o, v8); }
    static __device__ __forceinline__ void store_raw(T *p, v8 o) { __builtin_nontemporal_store(o, (v8_u *)p); }
    static __device__ __forceinline__ void store8(T *p, v8f o)
    {
        __builtin_nontemporal_store(__builtin_convertvector(o, v8), (v8_u *)p);
    }
};

template <int OP, typename T>
__global__ __launch_bounds__(kThreads) void slide16_scan_kernel(const T *__restrict__ x, T *__restrict__ y, int len,
                                                                int lo, int S, float scale, int tiles_per_row,
                                                                int tout, int group, int64_t n_tiles,
                                                                int64_t n_units, int remap)
{
    using O = Op<OP>;
    using G = SegStep<OP>;
    using IO = Io<T>;
    constexpr int C = kC, N = kN;
    __shared__ __attribute__((aligned(16))) float lds[kWavesPerWg * N];

    const int64_t unit = remap ? xcd_unit(n_units) : (int64_t)blockIdx.x;
    if (unit < 0) return;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float *A = lds + wave * N;                       // staged 16-bit inputs, then Pre in fp32, then the 16-bit results
    typename IO::v8 *const A16 = (typename IO::v8 *)A;       // ... as units of eight 16-bit elements, unit u at lds_unit(u)
    int64_t gt = unit * group + wave;
    int64_t gt_end = (unit + 1) * group;
    if (gt_end > n_tiles) gt_end = n_tiles;
    int64_t r = gt / tiles_per_row;
    int t = (int)(gt - r * tiles_per_row);

    // Lane constants (as in the fp32 kernel): this lane scans local positions C*lane .. C*lane+C-1;
    // m[k] is the reset mask of element k (a segment of S elements, counted from the tile origin,
    // starts there); m[C] belongs to the first element of the next lane.
    const float inv_s = 1.0f / (float)S;
    const int q0 = (C * lane) - S * (int)(((float)(C * lane) + 0.5f) * inv_s);                // (C*lane) % S
    float m[C + 1];
    if (S > C) {
        const int kb = q0 == 0 ? 0 : S - q0;
#pragma unroll
        for (int k = 0; k <= C; ++k) m[k] = G::mask(k == kb);
    } else {
        int q = q0;
#pragma unroll
        for (int k = 0; k <= C; ++k) {
            m[k] = G::mask(q == 0);
            q = (q + 1 == S) ? 0 : q + 1;
        }
    }
    const int n_pre = (q0 + C - 1) / C;             // earlier lanes holding part of my first segment
    int qe = q0 + C;
    if (S > C) qe = qe >= S ? qe - S : qe;
    else qe -= S * (int)(((float)qe + 0.5f) * inv_s);
    const int rem = qe == 0 ? 0 : S - qe;           // elements of my last segment beyond my chunk
    const int n_suf = (rem + C - 1) / C;
    const int max_reach = (S - 1 + C - 1) / C;
    const int sh = S & 3;                           // misalignment of Pre[q+S] against groups
    const int s4 = (S - sh) >> 2;
    const int chunk_pos = 4 * lds_group(4 * lane);  // my chunk: group u of it sits at chunk_pos ^ (4*u)
    // Pre[q+S] for my 16 outputs: the five aligned groups from element 16*lane + S - sh on (past the tile: wrapped,
    // discarded lanes only)
    int pp[5];
#pragma unroll
    for (int u = 0; u < 5; ++u) pp[u] = 4 * lds_group((4 * lane + s4 + u) & 255);

    // The strips of my next tile are requested before the current tile is worked on, and staged after its results have been
    // read back and before they are stored: 2 KB per tile is too little in flight to wait for at once, or behind stores.
    // A tile that reaches beyond its row is loaded whole too (the neighbouring rows are there), its outside elements are replaced
    // by the identity; only at the ends of x it is loaded element by element.
    const int64_t total = n_tiles / tiles_per_row * (int64_t)len;
    auto origin = [&](int64_t rr, int tt) { return tt * tout - (int)((rr * lo) & (kLine - 1)); };
    typename IO::v8 raw[2];
    auto request = [&](int64_t rr, int tt) -> bool {
        const int64_t e = rr * (int64_t)len + origin(rr, tt);
        const bool whole = e >= 0 && e + N <= total;
        if (whole) {
#pragma unroll
            for (int j = 0; j < 2; ++j) raw[j] = IO::load_raw(x + e + 512 * j + 8 * lane);
        }
        return whole;
    };
    auto stage_element_wise = [&](int64_t rr, int tt) {
        const int t0 = origin(rr, tt);
        const T *xr = x + rr * (int64_t)len;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            typename IO::v8 g;
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int e = t0 + 512 * j + 8 * lane + c;
                g[c] = (e >= 0 && e < len) ? xr[e] : (T)O::id();
            }
            A16[lds_unit(64 * j + lane)] = g;
        }
    };
    auto outside = [&](int64_t rr, int tt) {         // raw: the identity outside the row
        const int t0 = origin(rr, tt);
        if (t0 >= 0 && t0 + N <= len) return;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int c = 0; c < 8; ++c)
                if ((unsigned)(t0 + 512 * j + 8 * lane + c) >= (unsigned)len) raw[j][c] = (T)O::id();
    };
    if (gt >= gt_end) return;                        // (no workgroup barrier below)
    if (request(r, t)) {
        outside(r, t);
#pragma unroll
        for (int j = 0; j < 2; ++j) A16[lds_unit(64 * j + lane)] = raw[j];
    } else {
        stage_element_wise(r, t);
    }
    for (;;) {
        // tile origins pulled back so that (r*lo + t0) is a multiple of 32 elements: every strip
        // store starts on a 64-byte line of y; outputs before the row start are not stored
        const int t0 = origin(r, t);
        const int qlo = t0 < 0 ? -t0 : 0;
        T *yt = y + r * (int64_t)lo + t0;
        gt += kWavesPerWg;
        t += kWavesPerWg;
        while (t >= tiles_per_row) { t -= tiles_per_row; ++r; }
        const bool more = gt < gt_end;
        const bool whole = more && request(r, t);
        wave_lds_sync();
        // ---- my chunk of C consecutive elements
        float v[C];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const v8f g = IO::widen(A16[lds_unit(2 * lane + u)]);
#pragma unroll
            for (int c = 0; c < 8; ++c) v[8 * u + c] = g[c];
        }
        // ---- pass 1: lane totals (tail: my last segment's part, head: my first segment's part)
        float tail = v[0], head = v[C - 1];
#pragma unroll
        for (int k = 1; k < C; ++k) tail = G::f(tail, m[k], v[k]);
#pragma unroll
        for (int k = C - 2; k >= 0; --k) head = G::f(head, m[k + 1], v[k]);
        // ---- cross-lane carries: e from the n_pre lanes before me, g from the n_suf lanes after me
        float e = lane_read(tail, lane - 1);
        float g = lane_read(head, lane + 1);
        for (int d = 1; d < max_reach; d <<= 1) {
            const float te = lane_read(e, lane - d);
            const float tg = lane_read(g, lane + d);
            if (n_pre > d) e = O::f(te, e);
            if (n_suf > d) g = O::f(g, tg);
        }
        // ---- pass 2: the scans seeded with the carries: in-segment prefix sums (over v) and suffix sums
        float suf[C];
        suf[C - 1] = G::f(g, m[C], v[C - 1]);
#pragma unroll
        for (int k = C - 2; k >= 0; --k) suf[k] = G::f(suf[k + 1], m[k + 1], v[k]);
        v[0] = G::f(e, m[0], v[0]);
#pragma unroll
        for (int k = 1; k < C; ++k) v[k] = G::f(v[k - 1], m[k], v[k]);
        wave_lds_sync();                             // (everybody has read the staged inputs)
#pragma unroll
        for (int u = 0; u < 4; ++u)
            *(v4f *)(A + (chunk_pos ^ (4 * u))) = (v4f){v[4 * u], v[4 * u + 1], v[4 * u + 2], v[4 * u + 3]};
        wave_lds_sync();
        // ---- combine: y[q] = Suf[q] (+) Pre[q+S] for my own 16 outputs, one rounding
        {
            float p[20];
#pragma unroll
            for (int u = 0; u < 5; ++u) {
                const v4f q = *(const v4f *)(A + pp[u]);
                p[4 * u] = q.x; p[4 * u + 1] = q.y; p[4 * u + 2] = q.z; p[4 * u + 3] = q.w;
            }
            v8f o[2];
            auto add = [&](auto shift) {
#pragma unroll
                for (int c = 0; c < C; ++c) o[c / 8][c % 8] = O::f(suf[c], p[c + decltype(shift)::value]);
            };
            switch (sh) {                            // wave-uniform
            case 0: add(std::integral_constant<int, 0>{}); break;
            case 1: add(std::integral_constant<int, 1>{}); break;
            case 2: add(std::integral_constant<int, 2>{}); break;
            default: add(std::integral_constant<int, 3>{}); break;
            }
            if (OP == SWS_OP_ADD) {
                o[0] *= scale;
                o[1] *= scale;
            }
            wave_lds_sync();                         // (everybody has read Pre)
#pragma unroll
            for (int u = 0; u < 2; ++u) A16[lds_unit(2 * lane + u)] = IO::narrow(o[u]);
        }
        wave_lds_sync();
        // ---- out: strips of eight results, 128-bit stores; the next tile's strips take their places first
        typename IO::v8 o[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) o[j] = A16[lds_unit(64 * j + lane)];
        wave_lds_sync();
        if (whole) {
            outside(r, t);
#pragma unroll
            for (int j = 0; j < 2; ++j) A16[lds_unit(64 * j + lane)] = raw[j];
        } else if (more) {
            stage_element_wise(r, t);
        }
        int lim = lo - t0;
        if (lim > tout) lim = tout;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int q = 512 * j + 8 * lane;
            if (q >= lim) continue;
            if (q >= qlo && q + 8 <= lim) {
                IO::store_raw(yt + q, o[j]);
            } else {
#pragma unroll
                for (int c = 0; c < 8; ++c)
                    if (q + c >= qlo && q + c < lim) yt[q + c] = o[j][c];
            }
        }
        if (!more) break;
    }
}

// Direct evaluation (windows beyond the scan kernel's reach): one thread per output,
// fp32 accumulation left to right, one rounding at the end.
template <int OP, typename T>
__global__ __launch_bounds__(kThreads) void slide16_naive_kernel(const T *__restrict__ x, T *__restrict__ y,
                                                                 int64_t rows, int len, int lo, int w, float scale)
{
    using O = Op<OP>;
    const int64_t total = rows * (int64_t)lo;
    for (int64_t o = (int64_t)blockIdx.x * kThreads + threadIdx.x; o < total; o += (int64_t)gridDim.x * kThreads) {
        const int64_t r = o / lo;
        const T *xr = x + r * (int64_t)len + (o - r * lo);
        float acc = (float)xr[0];
        for (int j = 1; j < w; ++j) acc = O::f(acc, (float)xr[j]);
        if (OP == SWS_OP_ADD) acc *= scale;
        y[o] = (T)acc;
    }
}

// Small windows on shifted loads: a lane owns eight consecutive outputs and reads the w + 7 inputs
// under them as 128-bit loads.  Up to w = 8 each output combines its inputs left to right (Eq. 3 as
// written).  From w = 9 the eight windows share the inputs 7 .. w-1 of the strip: that core is
// combined once, and output c adds the suffix c .. 6 in front of it and the prefix w .. w+c-1
// behind it (running sums, the register-level form of Section 3's prefix / suffix split), about
// w + 20 operations for the eight outputs instead of 8 (w - 1).  All of it in fp32, one rounding.
// Workgroups are one wavefront and short-lived (512 outputs of a row, or several short rows side
// by side), which streams better than long-lived tiles.
// A 128-bit load may run past the end of its row (those values reach no valid output) but not
// past the ends of x: there it is replaced by element loads.
template <int OP, typename T, int W>
__global__ __launch_bounds__(kWave) void slide16_direct_kernel(const T *__restrict__ x, T *__restrict__ y,
                                                               int64_t rows, int len, int lo, float scale,
                                                               int strips, int wg_per_row, int rows_per_wg, int recip,
                                                               int align)
{
    using O = Op<OP>;
    using IO = Io<T>;
    constexpr int NL = (W + 7 + 7) / 8;              // 128-bit loads per strip
    const int lane = threadIdx.x;
    int64_t r;
    int sidx;
    if (rows_per_wg == 1) {
        const int br = blockIdx.x / (unsigned)wg_per_row;
        r = br;
        sidx = (blockIdx.x - br * wg_per_row) * kWave + lane;
    } else {
        const int lr = (lane * recip) >> 16;         // lane / strips, exact for lane < 64
        if (lr >= rows_per_wg) return;
        r = (int64_t)blockIdx.x * rows_per_wg + lr;
        sidx = lane - lr * strips;
    }
    if (r >= rows || sidx >= strips) return;
    // long rows: strips sit on the 16-byte boundaries of y, so a row that starts between two
    // boundaries has a partial first strip (short rows would spend too many lanes on those)
    T *yrow = y + r * (int64_t)lo;
    const int q = 8 * sidx - (align ? (int)(((uintptr_t)yrow >> 1) & 7) : 0);
    if (q >= lo) return;
    const int64_t g = r * (int64_t)len + q;          // the strip's first input in x
    const int64_t total = rows * (int64_t)len;
    const T *xr = x + g;
    float v[8 * NL];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
        if (g + 8 * k >= 0 && g + 8 * k + 8 <= total) {
            const v8f a = IO::load8(xr + 8 * k);
#pragma unroll
            for (int c = 0; c < 8; ++c) v[8 * k + c] = a[c];
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const int64_t e = g + 8 * k + c;
                v[8 * k + c] = (e >= 0 && e < total) ? IO::load1(xr + 8 * k + c) : 0.0f;
            }
        }
    }
    v8f o;
    if constexpr (W <= 8) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            float acc = v[c];
#pragma unroll
            for (int j = 1; j < W; ++j) acc = O::f(acc, v[c + j]);
            o[c] = acc;
        }
    } else {
        float core = v[7];
#pragma unroll
        for (int j = 8; j < W; ++j) core = O::f(core, v[j]);
        float suf[7], pre[8];
        suf[6] = v[6];
#pragma unroll
        for (int c = 5; c >= 0; --c) suf[c] = O::f(v[c], suf[c + 1]);
        pre[1] = v[W];
#pragma unroll
        for (int c = 2; c < 8; ++c) pre[c] = O::f(pre[c - 1], v[W + c - 1]);
        o[0] = O::f(suf[0], core);
        o[7] = O::f(core, pre[7]);
#pragma unroll
        for (int c = 1; c < 7; ++c) o[c] = O::f(O::f(suf[c], core), pre[c]);
    }
    if (OP == SWS_OP_ADD) o *= scale;
    T *yr = yrow + q;
    if (q >= 0 && q + 8 <= lo) {
        IO::store8(yr, o);
    } else {
#pragma unroll
        for (int c = 0; c < 8; ++c)
            if (q + c >= 0 && q + c < lo) IO::store1(yr + c, o[c]);
    }
}

constexpr int kDirectMaxW = 33;                      // five 128-bit loads per strip of eight outputs

template <int OP, typename T, int W>
hipError_t launch_16_direct_w(const T *x, T *y, int64_t rows, int len, int lo, float scale, hipStream_t s)
{
    // aligned strips pay from about a thousand outputs per row (measured: 4.5 against 4.3 TB/s at
    // 4096, 2.7 against 3.7 at 224); rows of y that all start on a boundary need no shift
    const int align = lo >= 1024 && !(lo % 8 == 0 && (uintptr_t)y % 16 == 0);
    const int strips = (lo + (align ? 14 : 7)) / 8;
    const int wg_per_row = (strips + kWave - 1) / kWave;
    const int rows_per_wg = strips < kWave ? kWave / strips : 1;
    const int recip = 65536 / strips + 1;
    const int64_t grid = rows_per_wg == 1 ? rows * wg_per_row : (rows + rows_per_wg - 1) / rows_per_wg;
    if (grid > 2147483647LL) return kNotTaken;
    hipLaunchKernelGGL((slide16_direct_kernel<OP, T, W>), dim3((unsigned)grid), dim3(kWave), 0, s, x, y, rows, len, lo,
                       scale, strips, wg_per_row, rows_per_wg, recip, align);
    return hipGetLastError();
}

template <int OP, typename T, int W0>
hipError_t launch_16_direct(const T *x, T *y, int64_t rows, int len, int lo, int w, float scale, hipStream_t s)
{
    if constexpr (W0 > kDirectMaxW) {
        return kNotTaken;
    } else {
        if (w == W0) return launch_16_direct_w<OP, T, W0>(x, y, rows, len, lo, scale, s);
        return launch_16_direct<OP, T, W0 + 1>(x, y, rows, len, lo, w, scale, s);
    }
}

constexpr int kScanMaxW = kN - 64 + 1;               // leaves at least 64 outputs per wave tile
constexpr int kLong16MinW = 600;                     // from here the long-window kernel (bf16, 16384-long rows: w = 513 level, 700 1.3 x, 961 5 x the scan)

template <int OP, typename T>
hipError_t launch_16(const T *x, T *y, int64_t rows, int len, int lo, int w, float scale, hipStream_t s)
{
    const int variant = g_opt.slide_variant;
    // Measured on bf16: up to w = 9 (two loads per strip) the shifted loads win at every size (5.2 to
    // 5.8 TB/s against the scan's 4.9 to 5.1 on a 1 GB tensor); beyond that they win where the scan
    // kernel's 1024-element wave tiles fit badly: rows under 2048 outputs (3 to 25 times faster at
    // 56 to 224 elements per row) and tensors under 2^25 elements (2 to 5 times).
    const bool direct_auto = w <= 9 || lo < 2048 || rows * (int64_t)len <= (1LL << 25);
    if (w <= kDirectMaxW && variant != 1 && (variant == 3 || w == 1 || (variant != 2 && direct_auto))) {
        const hipError_t e = launch_16_direct<OP, T, 1>(x, y, rows, len, lo, w, scale, s);
        if (e != kNotTaken) return e;     // a grid beyond the launch limit: the kernels below
    }
    if (w >= 2 && w <= kScanMaxW && variant != 1) {
        const int S = w - 1;
        const int tout = (kN - S) & ~(kLine - 1);    // a multiple of 64 bytes of y (at least 64 outputs)
        const int tiles = (lo + max_origin_shift(lo, kLine) + tout - 1) / tout;
        const int64_t n_tiles = rows * tiles;
        // Four tiles per wavefront (measured, us, 2 / 4 / 8 / 16: [8192,16384] w = 64 101 / 93 / 103 / 113, w = 255 118 / 101 / 101 / 112,
        // [64,1048576] w = 64 48 / 50 / 56 / 65), eight where a row is a tile or two ([186479,422] w = 39 115 / 98 / 90 / 91:
        // the starts of a workgroup weigh more there); workgroups in launch order (dealt to the XCDs in runs: the same).
        int64_t g = (tiles <= 2 ? 8 : 4) * kWavesPerWg;
        int remap = 0;
        // ... halved while that leaves fewer than 2048 workgroups ([3000,5003] w = 40: 17.8 us with 1125, 17.2 with 2250)
        while (g > kWavesPerWg && n_tiles / g < 2048) g /= 2;
        if (g_opt.slide_group > 0) g = (g_opt.slide_group + kWavesPerWg - 1) / kWavesPerWg * kWavesPerWg;
        if (g_opt.slide_chunk & 4) remap = 1;
        if (g_opt.slide_chunk & 8) remap = 0;
        const int64_t n_units = (n_tiles + g - 1) / g;
        const int64_t grid = remap ? xcd_grid(n_units) : n_units;
        if (grid > 2147483647LL) return kNotTaken;
        hipLaunchKernelGGL((slide16_scan_kernel<OP, T>), dim3((unsigned)grid), dim3(kThreads), 0, s, x, y, len, lo, S,
                           scale, tiles, tout, (int)g, n_tiles, n_units, remap);
        return hipGetLastError();
    }
    int64_t grid = (rows * (int64_t)lo + kThreads - 1) / kThreads;
    if (grid > 1048576) grid = 1048576;
    hipLaunchKernelGGL((slide16_naive_kernel<OP, T>), dim3((unsigned)grid), dim3(kThreads), 0, s, x, y, rows, len, lo,
                       w, scale);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_16_op(int op, const void *x, void *y, int64_t rows, int len, int lo, int w, float scale,
                        hipStream_t s)
{
    switch (op) {
    case SWS_OP_ADD: return launch_16<SWS_OP_ADD, T>((const T *)x, (T *)y, rows, len, lo, w, scale, s);
    case SWS_OP_MAX: return launch_16<SWS_OP_MAX, T>((const T *)x, (T *)y, rows, len, lo, w, scale, s);
    default: return launch_16<SWS_OP_MIN, T>((const T *)x, (T *)y, rows, len, lo, w, scale, s);
    }
}

}  // namespace

// 16-bit storage (dtype SWS_DTYPE_BF16 / SWS_DTYPE_F16), fp32 arithmetic, one rounding per output.
hipError_t launch_slide1d_16(int op, int dtype, const void *x, void *y, int64_t rows, int64_t len64, int32_t w,
                             float scale, hipStream_t s)
{
    const int len = (int)len64, lo = len - w + 1;
    // windows longer than a wave tile: the one-pass long-window kernel (slide_long.hip); slide_variant 8 takes it
    // from w = 257, 1 and 5 keep it out
    const int variant = g_opt.slide_variant;
    if ((w >= kLong16MinW || (variant == 8 && w > 256)) && variant != 1 && variant != 5) {
        const hipError_t e = launch_slide1d_long_16(op, dtype, x, y, rows, len, lo, w, scale, s);
        if (e != kNotTaken) return e;
    }
    if (dtype == SWS_DTYPE_BF16) return launch_16_op<__bf16>(op, x, y, rows, len, lo, w, scale, s);
    return launch_16_op<_Float16>(op, x, y, rows, len, lo, w, scale, s);
}

}  // namespace sws
