// The adjoint of max pooling (Section 2.3) with large windows: every window's gradient goes to the first cell
// (row-major) that holds its maximum.
//
// Scanning kh * kw cells per window costs 2 kh kw vector instructions per cell (13 x 13 windows: 1.0 ms on
// [371,32,37,19], and 26 ms of direct evaluation where the scan's band does not fit LDS).  The maximum with its first
// position is itself associative, so it runs on Section 2's logarithmic scheme: value and position travel in one double —
// a float converted to double leaves 29 zero bits at the bottom, which take the position, reversed for
// positive values (among equals the larger double is then the earlier cell) — and combining two partial windows is one
// v_max_f64.  Windows of kw columns by doubling (ceil(log2 kw) steps over the staged tile in LDS, in place: a wavefront
// walks its rows upwards and reads ahead of what it writes), then of kh rows in the same way; a window's key
// then holds its cell, and the gradient is added there in LDS.  Every wavefront adds into a copy of its own, in
// program order, and the copies are summed in a fixed order: results are reproducible.
//
// -0.0 counts as +0.0 and infinities as the largest finite double, so ties go to the first cell there too.
#include "sws_internal.h"

namespace sws {

namespace {

struct PgLarge {
    int H, W, Ho, Wo, kh, kw, sh, sw, ph, pw;
    int TB, TC, nb, nc;                               // cells of a tile, tiles per plane
    int P, D;                                         // columns of the staged tile; doubles of it, padded
    float inv_P, inv_TC;
};

constexpr unsigned kPosMask = (1u << 27) - 1;         // row << 12 | column inside the tile

// NW wavefronts per tile; U runs of 64 keys in flight: four, but one where the staged tile is no more than four of them
// (7 x 7 on [2000,32,7,7] 56 us against 61; 13 x 13 on [371,32,37,19] 174 against 157).
template <int NW, int U>
__global__ __launch_bounds__(64 * NW) void maxpool_grad_large_kernel(const float *__restrict__ x, const float *__restrict__ gy,
                                                                     float *__restrict__ gx, PgLarge g, int64_t n_units)
{
    constexpr int T = 64 * NW;
    extern __shared__ __attribute__((aligned(16))) double key[];
    float *const acc = (float *)(key + g.D);          // [NW][TB * TC]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t unit = blockIdx.x;
    if (unit >= n_units) return;
    const int per = g.nb * g.nc;
    const int64_t plane = unit / per;
    const int in = (int)(unit - plane * per), ib = in / g.nc, ic = in - ib * g.nc;
    const int r0 = ib * g.TB, c0 = ic * g.TC;
    const int nr = g.H - r0 < g.TB ? g.H - r0 : g.TB, ncol = g.W - c0 < g.TC ? g.W - c0 : g.TC;
    const float *xp = x + plane * (int64_t)g.H * g.W, *gp = gy + plane * (int64_t)g.Ho * g.Wo;
    // windows that cover a cell of the tile, and the cells they see
    int w0 = r0 + g.ph - g.kh + 1, v0 = c0 + g.pw - g.kw + 1;
    w0 = w0 > 0 ? (w0 + g.sh - 1) / g.sh : 0;
    v0 = v0 > 0 ? (v0 + g.sw - 1) / g.sw : 0;
    int w1 = (r0 + nr - 1 + g.ph) / g.sh, v1 = (c0 + ncol - 1 + g.pw) / g.sw;
    w1 = w1 < g.Ho - 1 ? w1 : g.Ho - 1;
    v1 = v1 < g.Wo - 1 ? v1 : g.Wo - 1;
    const int nw = w1 - w0 + 1, nv = v1 - v0 + 1;     // may be 0 or less: no window covers the tile
    const int xr0 = w0 * g.sh - g.ph, xc0 = v0 * g.sw - g.pw;
    const int XR = nw > 0 ? (nw - 1) * g.sh + g.kh : 0, XC = nv > 0 ? (nv - 1) * g.sw + g.kw : 0;
    auto wave_sync = [&]() {                          // what my wavefront's other lanes wrote to LDS
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    auto sync = [&]() {
        if constexpr (NW == 1) wave_sync();
        else __syncthreads();
    };

    for (int e = tid; e < NW * g.TB * g.TC; e += T) acc[e] = 0.0f;
    if (nw > 0 && nv > 0) {
        const int n = XR * g.P;
        for (int e0 = tid; e0 < n; e0 += 4 * T) {     // four loads in flight
            float f[4];
            bool ok[4];
            int pos[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int e = e0 + u * T, i = fdiv(e, g.inv_P), j = e - i * g.P, r = xr0 + i, c = xc0 + j;
                ok[u] = e < n && j < XC && (unsigned)r < (unsigned)g.H && (unsigned)c < (unsigned)g.W;
                pos[u] = i << 12 | j;
                f[u] = xp[ok[u] ? (int64_t)r * g.W + c : 0];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                double d = (double)(f[u] + 0.0f);
                const double top = 0x1p1023;          // (its low bits are zero, like those of every converted float)
                d = d > top ? top : (d < -top ? -top : d);
                unsigned long long b = __builtin_bit_cast(unsigned long long, d);
                b |= (long long)b < 0 ? (unsigned)pos[u] : kPosMask - (unsigned)pos[u];
                if (!ok[u]) b = 0xffefffffffffffffULL;        // the lowest finite double: cells that do not exist
                if (e0 + u * T < n) key[e0 + u * T] = __builtin_bit_cast(double, b);
            }
        }
        sync();
        // ---- kw columns: row by row, in place
        {
            const int rpw = (XR + NW - 1) / NW, i0 = wave * rpw, i1 = i0 + rpw < XR ? i0 + rpw : XR;
            // A step reads what other lanes left in the step before (a row belongs to one wavefront, which waits for itself only),
            // and inside a step everything is read before anything behind it is written.  (Past the end of a wavefront's rows
            // lie another's, or padding: what is read there reaches columns that start no window.)
            const int end = i1 * g.P;
            auto pass = [&](int m) {
                for (int e0 = i0 * g.P + lane; e0 < end; e0 += 64 * U) {
                    double v[U];
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int e = e0 + 64 * u < end ? e0 + 64 * u : e0;
                        v[u] = __builtin_fmax(key[e], key[e + m]);
                    }
                    wave_sync();
#pragma unroll
                    for (int u = 0; u < U; ++u)
                        if (e0 + 64 * u < end) key[e0 + 64 * u] = v[u];
                    wave_sync();
                }
            };
            int m = 1;
            for (; 2 * m <= g.kw; m *= 2) pass(m);
            if (m < g.kw) pass(g.kw - m);
        }
        sync();
        // ---- kh rows: every wavefront its window columns, 64 / cw rows at a time, in place
        {
            const int cpw = (nv + NW - 1) / NW, b0 = wave * cpw, b1 = b0 + cpw < nv ? b0 + cpw : nv;
            for (int b = b0; b < b1; b += 64) {
                const int cw = b1 - b < 64 ? b1 - b : 64, rb = 64 / cw;
                const int rr = fdiv(lane, 1.0f / (float)cw), col = (b + lane - rr * cw) * g.sw;
                const int top = rr < rb ? XR : 0;     // (64 % cw lanes stand by)
                auto pass = [&](int m) {
                    for (int i0 = 0; i0 + m < XR; i0 += U * rb) {
                        double v[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const int i = i0 + u * rb + rr, r = i + m < top ? i : 0;
                            v[u] = __builtin_fmax(key[r * g.P + col], key[(r + m) * g.P + col]);
                        }
                        wave_sync();
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const int i = i0 + u * rb + rr;
                            if (i + m < top) key[i * g.P + col] = v[u];
                        }
                        wave_sync();
                    }
                };
                int m = 1;
                for (; 2 * m <= g.kh; m *= 2) pass(m);
                if (m < g.kh) pass(g.kh - m);
            }
        }
        sync();
        // ---- every window's gradient to its cell
        const float inv_nv = 1.0f / (float)nv;
        float *mine = acc + wave * (g.TB * g.TC);
        for (int q = tid; q < nw * nv; q += T) {
            const int w = fdiv(q, inv_nv), v = q - w * nv;
            const unsigned long long b = __builtin_bit_cast(unsigned long long, key[w * g.sh * g.P + v * g.sw]);
            const unsigned lo = (unsigned)b & kPosMask, pos = (long long)b < 0 ? lo : kPosMask - lo;
            const int r = xr0 + (int)(pos >> 12) - r0, c = xc0 + (int)(pos & 4095) - c0;
            const float d = gp[(int64_t)(w0 + w) * g.Wo + v0 + v];
            if ((unsigned)r < (unsigned)nr && (unsigned)c < (unsigned)ncol)
                __hip_atomic_fetch_add(mine + r * g.TC + c, d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    }
    sync();
    float *out = gx + plane * (int64_t)g.H * g.W;
    for (int e = tid; e < nr * g.TC; e += T) {
        const int r = fdiv(e, g.inv_TC), c = e - r * g.TC;
        float s = acc[e];
#pragma unroll
        for (int k = 1; k < NW; ++k) s += acc[k * g.TB * g.TC + e];
        if (c < ncol) out[(int64_t)(r0 + r) * g.W + c0 + c] = s;
    }
}

}  // namespace

hipError_t launch_maxpool2d_grad_large(const float *x, const float *gy, float *gx, int64_t planes, int64_t H, int64_t W, int64_t Ho,
                                       int64_t Wo, int kh, int kw, int sh, int sw, int ph, int pw, hipStream_t s, bool *taken)
{
    *taken = false;
    if (H >= (1 << 19) || W >= (1 << 19) || kh > 256 || kw > 256 || sh > 256 || sw > 256) return hipSuccess;
    PgLarge g;
    g.H = (int)H; g.W = (int)W; g.Ho = (int)Ho; g.Wo = (int)Wo; g.kh = kh; g.kw = kw; g.sh = sh; g.sw = sw; g.ph = ph; g.pw = pw;
    // Planes of up to two thousand cells: one wavefront per plane (no barriers, many planes per compute unit); larger ones:
    // four per tile.  Tiles: the fewest staged cells per cell with at least two workgroups per compute unit.
    const bool wave = H * W <= 2048;
    const int NW = wave ? 1 : 4;
    // (this runs on every call: only the tile heights and widths that differ are tried, [224,224] 29 x 29 of 64 x 64 cuts)
    struct Cut { int parts, t, span; };               // parts of an axis, cells of one, cells that its windows see
    auto cuts = [](Cut *c, int n, int no, int k, int st) {
        int m = 0;
        for (int parts = 1; parts <= 64 && parts <= n; ++parts) {
            const int t = (int)((unsigned)(n + parts - 1) / (unsigned)parts);
            if (t > 1024 || (m > 0 && t == c[m - 1].t)) continue;
            int win = (int)((unsigned)(t + k - 2) / (unsigned)st) + 1;
            win = win < no ? win : no;
            if ((win - 1) * st + k < 4096) c[m++] = {parts, t, (win - 1) * st + k};
        }
        return m;
    };
    Cut rows[64], cols[64];
    const int nr = cuts(rows, (int)H, (int)(Ho < (1 << 20) ? Ho : 1 << 20), kh, sh), nc = cuts(cols, (int)W, (int)(Wo < (1 << 20) ? Wo : 1 << 20), kw, sw);
    int need = 0;
    int64_t best = 0;
    for (int i = 0; i < nr; ++i)
        for (int j = 0; j < nc; ++j) {
            const int cells = rows[i].span * cols[j].span;
            const int D = cells + kw + 64, bytes = D * 8 + NW * rows[i].t * cols[j].t * 4;
            if (cells > 10240 || bytes > 78 * 1024) continue;
            const int64_t cost = (int64_t)(cells + 512) * (rows[i].parts * cols[j].parts);
            if (need == 0 || cost < best) {
                need = bytes;
                best = cost;
                g.TB = rows[i].t; g.TC = cols[j].t; g.nb = rows[i].parts; g.nc = cols[j].parts; g.P = cols[j].span; g.D = (D + 1) / 2 * 2;
            }
        }
    if (need == 0) return hipSuccess;
    const size_t lds = (size_t)need + 16;
    const int64_t units = planes * g.nb * g.nc;
    if (units > 2147483647LL) return hipSuccess;
    g.inv_P = 1.0f / g.P; g.inv_TC = 1.0f / g.TC;
    *taken = true;
    const auto k = !wave ? maxpool_grad_large_kernel<4, 4> : g.D <= 256 + kw + 64 ? maxpool_grad_large_kernel<1, 1> : maxpool_grad_large_kernel<1, 4>;
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, dim3((unsigned)units), dim3(64 * NW), lds, s, x, gy, gx, g, units);
    return hipGetLastError();
}

}  // namespace sws
