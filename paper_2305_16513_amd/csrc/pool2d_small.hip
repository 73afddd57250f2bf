// sws_pool2d on small planes — 2-D pooling (Section 2.3) when a plane is a few hundred elements
// (the 7 x 7 and 14 x 14 planes of a network's last stages, with thousands of channels).
//
// The band kernel gives a wavefront to a band of one plane; on a 49-element plane that leaves most
// lanes idle.  Here a workgroup takes G whole planes: they are contiguous in memory, so they are
// staged into LDS as one range of 128-bit loads, and the G * Ho * Wo outputs — contiguous as well —
// are dealt to the threads one by one, each combining its window from LDS (down H, then across W,
// as the direct evaluation does) and stored coalesced.  Window cells outside the plane are skipped
// by clamping the loop bounds, so padding and real-cell averages cost nothing extra.
//
// What bounds it is latency: a workgroup loads, waits, and walks windows through dependent LDS reads.  So a workgroup takes no more planes
// than give every compute unit eight of them, and where it has fewer outputs than threads, 2^ls threads share one, every
// 2^ls-th column each (a global average of 7 x 7 was 49 reads one after the other in 80 of 256 threads).  Average of 7 x 7
// planes, 65536 of them, 6.4 -> 5.2 us (its adjoint is the second kernel's), 3 x 3 on 16384 of them
// 13.5 -> 5.8; four or sixteen workgroups per unit: 5.2 and 5.9 on the first, 9.2 and 9.5 on the second.
#include "sws_internal.h"

namespace sws {

namespace {

constexpr int kThreads = 256;
constexpr int kStage = 4096;                         // floats of LDS per workgroup (16 KB)

typedef float v4f __attribute__((ext_vector_type(4)));

template <int OP, typename T>
__global__ __launch_bounds__(kThreads) void pool2d_small_kernel(const T *__restrict__ x, T *__restrict__ y,
                                                                int64_t planes, int H, int W, int Ho, int Wo, int kh,
                                                                int kw, int sh, int sw, int ph, int pw, float scale,
                                                                int div_valid, int G, int ls, unsigned rcp_q, unsigned rcp_wo)
{
    using O = Op<OP>;
    __shared__ __attribute__((aligned(16))) float lds[kStage];
    const int tid = threadIdx.x;
    const int P = H * W, Q = Ho * Wo;
    const int64_t p0 = (int64_t)blockIdx.x * G;
    const int g = planes - p0 < G ? (int)(planes - p0) : G;
    typedef T v4t __attribute__((ext_vector_type(4)));
    const T *src = x + p0 * P;
    const int n = g * P;
    if (((uintptr_t)src & (4 * sizeof(T) - 1)) == 0) {
        const int n4 = n >> 2;
        for (int i = tid; i < n4; i += kThreads) {
            const v4t q = *(const v4t *)(src + 4 * i);
            *(v4f *)(lds + 4 * i) = (v4f){(float)q[0], (float)q[1], (float)q[2], (float)q[3]};
        }
        for (int i = 4 * n4 + tid; i < n; i += kThreads) lds[i] = (float)src[i];
    } else {
        for (int i = tid; i < n; i += kThreads) lds[i] = (float)src[i];
    }
    __syncthreads();
    T *dst = y + p0 * Q;
    const int m = g * Q;
    const int share = tid & ((1 << ls) - 1);
    for (int i = tid; i < m << ls; i += kThreads) {
        const int o = i >> ls;
        // o = (plane, ho, wo); the quotients by multiplication with 2^32 / d + 1 (exact: o < 2^16, d < 2^12)
        const int pl = Q == 1 ? o : (int)__umulhi((unsigned)o, rcp_q);
        const int cell = o - pl * Q;
        const int ho = Wo == 1 ? cell : (int)__umulhi((unsigned)cell, rcp_wo);
        const int wo = cell - ho * Wo;
        const float *xp = lds + pl * P;
        const int h0 = ho * sh - ph, c0 = wo * sw - pw;
        const int a_lo = h0 < 0 ? -h0 : 0, a_hi = kh < H - h0 ? kh : H - h0;
        const int b_lo = c0 < 0 ? -c0 : 0, b_hi = kw < W - c0 ? kw : W - c0;
        float acc = O::id();
        for (int b = b_lo + share; b < b_hi; b += 1 << ls) {
            float col = O::id();
            for (int a = a_lo; a < a_hi; ++a) col = O::f(col, xp[(h0 + a) * W + c0 + b]);
            acc = O::f(acc, col);
        }
        for (int j = 1; j < 1 << ls; j <<= 1) acc = O::f(acc, __shfl_xor(acc, j, kWave));      // (an output's threads are neighbours: all here)
        if (OP == SWS_OP_ADD) {
            const int cells = (a_hi > a_lo ? a_hi - a_lo : 0) * (b_hi > b_lo ? b_hi - b_lo : 0);
            acc *= div_valid ? scale / (float)cells : scale;
        }
        if (share == 0) dst[o] = (T)acc;
    }
}

// Planes of one element that every window covers (the adjoint of a global average: 1 x 1 -> H x W): an output is its plane's
// element.  Nothing but stores: four outputs a thread, whole planes per workgroup, a multiple of four so that its outputs start on a 16-byte boundary when y
// does.  The kernel above walks a clamped window for every output and stores them one by one: 65536 planes -> 7 x 7 there 8.8 us, here 5.2.
template <int OP, typename T>
__global__ __launch_bounds__(kThreads) void pool2d_spread_kernel(const T *__restrict__ x, T *__restrict__ y, int64_t planes, int Q, float scale, int G,
                                                                 unsigned rcp_q)
{
    using O = Op<OP>;
    typedef T v4t __attribute__((ext_vector_type(4)));
    const int64_t p0 = (int64_t)blockIdx.x * G;
    const int g = planes - p0 < G ? (int)(planes - p0) : G, n = g * Q;
    const T *src = x + p0;
    T *dst = y + p0 * Q;
    auto plane = [&](int o) { return Q == 1 ? o : (int)__umulhi((unsigned)o, rcp_q); };      // (exact: see above)
    auto value = [&](int p) {
        const float v = O::f(O::id(), (float)src[p]);
        return (T)(OP == SWS_OP_ADD ? v * scale : v);
    };
    const bool wide = ((uintptr_t)dst & (4 * sizeof(T) - 1)) == 0;
    const int n4 = wide ? n >> 2 : 0;
    for (int i = threadIdx.x; i < n4; i += kThreads) {
        const int o = 4 * i, a = plane(o);
        v4t q;
        if (Q >= 4) {                                 // at most two planes
            const int b = plane(o + 3), first = (a + 1) * Q - o;
            const T va = value(a), vb = value(b);
            q = (v4t){va, first > 1 ? va : vb, first > 2 ? va : vb, first > 3 ? va : vb};
        } else {
            q = (v4t){value(a), value(plane(o + 1)), value(plane(o + 2)), value(plane(o + 3))};
        }
        *(v4t *)(dst + o) = q;
    }
    for (int o = 4 * n4 + (int)threadIdx.x; o < n; o += kThreads) dst[o] = value(plane(o));
}

}  // namespace

// Planes of at most kStage / 4 elements.  *taken = false: not this kernel's case.
template <typename T>
hipError_t launch_pool2d_small(int op, const T *x, T *y, int64_t planes, int H, int W, int Ho, int Wo, int kh,
                               int kw, int sh, int sw, int ph, int pw, float scale, int div_valid, hipStream_t s,
                               bool *taken)
{
    *taken = false;
    const int64_t P = (int64_t)H * W, Q = (int64_t)Ho * Wo;
    if (P < 1 || P > kStage / 4 || Q < 1 || Q > 4095 || Wo > 4095) return hipSuccess;
    const unsigned rcp_q = (unsigned)(4294967296ULL / (uint64_t)Q + 1), rcp_wo = (unsigned)(4294967296ULL / (uint64_t)Wo + 1);
    if (P == 1 && (int64_t)(Ho - 1) * sh <= ph && (int64_t)(Wo - 1) * sw <= pw && kh > ph && kw > pw) {
        // (one element: its real cells are one.)  One 16-byte store per thread: as many planes as that makes
        const int G = Q <= 256 ? (int)(4 * kThreads / Q) & ~3 : 4;
        const int64_t grid = (planes + G - 1) / G;
        if (grid > 2147483647LL) return hipSuccess;
        *taken = true;
#define SWS_SPREAD(OPV) hipLaunchKernelGGL((pool2d_spread_kernel<OPV, T>), dim3((unsigned)grid), dim3(kThreads), 0, s, x, y, planes, (int)Q, scale, G, rcp_q)
        switch (op) {
        case SWS_OP_ADD: SWS_SPREAD(SWS_OP_ADD); break;
        case SWS_OP_MAX: SWS_SPREAD(SWS_OP_MAX); break;
        default: SWS_SPREAD(SWS_OP_MIN); break;
        }
#undef SWS_SPREAD
        return hipGetLastError();
    }
    // whole planes per workgroup, a multiple of four so that every workgroup's range starts on a
    // 16-byte boundary when x does
    int G = (int)(kStage / P) & ~3;
    // ... and at most 4096 outputs: windows that spread a plane (the adjoint of a global average: 1 x 1 -> 7 x 7, 65536
    // planes) would otherwise leave too few workgroups, or outputs beyond the reach of the quotient below
    if (G * Q > 4096) G = Q < 1024 ? (int)(4096 / Q) & ~3 : 4;
    // ... and no more than leave every compute unit eight workgroups (rounded up: one workgroup over would be a round of its own), but then, where there
    // are only a few passes over the threads, as many as fill the last one (300000 planes, 3 x 3, stride 2: 4 x 4, 576 outputs in three passes
    // 9.5 us, 768 8.4; 5 x 5 16.0 / 14.4)
    const int64_t want = (planes + 8 * device_cus() - 1) / (8 * device_cus());
    if (want < G) {
        const int g = ((int)want + 3) & ~3;
        const int whole = (int)((g * Q + kThreads - 1) / kThreads * kThreads / Q) & ~3;
        const int to = g * Q > kThreads && g * Q <= 6 * kThreads && whole > g ? whole : g;
        if (to < G) G = to;
    }
    int ls = 0;
    while (G * Q << (ls + 1) <= kThreads && 1 << ls < kw && ls < 5) ++ls;
    const int64_t grid = (planes + G - 1) / G;
    if (grid > 2147483647LL) return hipSuccess;
    *taken = true;
#define SWS_PS(OPV)                                                                                                \
    hipLaunchKernelGGL((pool2d_small_kernel<OPV, T>), dim3((unsigned)grid), dim3(kThreads), 0, s, x, y, planes, H, W, Ho, Wo, \
                       kh, kw, sh, sw, ph, pw, scale, div_valid, G, ls, rcp_q, rcp_wo)
    switch (op) {
    case SWS_OP_ADD: SWS_PS(SWS_OP_ADD); break;
    case SWS_OP_MAX: SWS_PS(SWS_OP_MAX); break;
    default: SWS_PS(SWS_OP_MIN); break;
    }
#undef SWS_PS
    return hipGetLastError();
}

template hipError_t launch_pool2d_small<float>(int, const float *, float *, int64_t, int, int, int, int, int, int, int, int, int, int,
                                               float, int, hipStream_t, bool *);
template hipError_t launch_pool2d_small<__bf16>(int, const __bf16 *, __bf16 *, int64_t, int, int, int, int, int, int, int, int, int,
                                                int, float, int, hipStream_t, bool *);
template hipError_t launch_pool2d_small<_Float16>(int, const _Float16 *, _Float16 *, int64_t, int, int, int, int, int, int, int, int,
                                                  int, int, float, int, hipStream_t, bool *);

}  // namespace sws
