// Dense-channel convolution (Section 2.5) on the bf16 matrix cores with exactly split fp32 operands: any
// kernel of up to 64 taps, stride 1 or 2, any channel counts, one or two dimensions, forward and the adjoint with
// respect to the input.
//
//   y[n][co][p] = sum over taps t, input channels ci of  W_t[co][ci] * X[n][ci][p * s + t]
//
// is a sum of matrix products over shifted views of the same input, the sliding sum over taps.  An fp32 number
// is the exact sum of three bf16 numbers and a product of two bf16 numbers is exact in fp32; of the nine piece
// products of x * w the three smallest are below 2^-22 of the product in all, the other six are accumulated in fp32 by
// v_mfma_f32_32x32x16_bf16: 6 instructions of 32 cycles per 16 channels, tap and 32 x 32 outputs where the fp32
// matrix instruction needs 8 of 64 cycles.
//
// Two launches.  split_weights_kernel writes the weights' pieces into the caller's workspace in the order in which
// the matrix instruction wants them (1 KB per piece of a 32 x 16 block, lane after lane), whatever view they are
// read through (plain, adjoint, output phases of a strided adjoint).  Splitting them inside the main kernel would
// be repeated by every workgroup, and their LDS traffic would double; from the workspace they go
// straight into registers, one 128-bit load per lane and operand, served by L2.
// conv_split_kernel: a workgroup computes 32*MB*WM output channels x 32*NB*WN output positions (each wavefront
// MB x NB blocks of 32 x 32; WK wavefronts share a block's contraction).  Per chunk of 16*NC input
// channels the input lines that the tile's windows meet are loaded once, zero-padded, split and written to LDS as
// 16-byte units of eight channels of one position and piece, positions contiguous; a tap's B operand is that tile
// read at a shifted address, so nothing is staged per tap and no column matrix exists.  Strided layers
// store the columns of a line by residue, so that the positions of a tap are contiguous there too.
//
// Tiles.  Output rows of all images are numbered through (virtual rows) and cut into strips of TW columns; the
// positions of a strip are numbered row after row and a tile is a run of them, so that small planes fill whole
// tiles.  Where runs that start at row ends stage fewer lines, a tile takes whole rows of the strip instead.
//
// Output phases (NPH = 4): the adjoint of a stride-2 layer computes the four cells (2i + er, 2j + ec) of gx from
// the same staged gradients; every tap belongs to one phase, so the work is that of the forward pass, and the two
// cells of a row leave as one store.
//
// Measured, us, with the weights' pass, this kernel / the fp32 matrix kernels: [32,256,14,14] -> 256, 3 x 3 48 / 113, adjoint 47 / 133;
// [32,128,56,56] -> 128, 3 x 3 stride 2 51 / 104, adjoint 62 / 205; [17,128,23,14] -> 104, 5 x 5 43 / 153.
// Staging wavefronts (P), here / without them: [32,256,14,14] 47.8 / 50.2, [32,128,56,56] 51 / 55, [8,256,28,28] -> 512 at stride 2 45 / 56,
// [32,192,19,19] -> 64 at stride 2 32 / 40, [1,416,84,84] -> 232 75 / 83.  What is left of [32,256,14,14], in cycles of a workgroup's 80 k: 7 k until the first
// products, eight chunks of 8.0 k (6.9 k of products), 7 k for the sum over two wavefronts and the stores; 200 workgroups on 256 compute units.  Blocks of one
// wavefront at least two positions wide (NB = 2): with NB = 1 the weights alone saturate the vector cache's 64 bytes
// per cycle.
#include "sws_internal.h"

#include <type_traits>

namespace sws {

namespace {

typedef v2f v2f_u __attribute__((aligned(4)));

constexpr int kMaxSteps = 64;                         // contraction steps per chunk and wavefront (one lane holds one)
constexpr int kStepBytes = 3 * 1024;                  // a step's weights of 32 output channels: 3 pieces x 64 lanes x 16 bytes
constexpr int kPadSteps = 4;                          // steps behind the last one that the prefetch may touch

struct SplitGeom {
    int N, Cin, H, W, HW, Cout, Ho, NR;               // input planes; NR = N * Ho virtual output rows
    int KT, S, NC, nchunk, KS;                        // taps; steps per chunk and wavefront; 16-channel groups, chunks; steps per wavefront
    int ls, LPI, SH, sh, sw, dh0, dw0;                // lines: per output row, per image, per window; strides, first row / column offset
    int CW, LW, TW, TWl, nstrips;                     // columns per residue, positions per line, strip widths
    int bnp, bnpl, tpf, tiles, cot;                   // positions per tile (last strip), tiles per full strip, all tiles, channel tiles
    int PS, bufs;                                     // staged positions; bytes from one LDS buffer to the other
    int yHW, yH, yW, ys;                              // output planes; cells per position and axis (1, or 2 for phases)
    int nt[4];                                        // phases: taps of each
    float inv_tw, inv_twl, inv_Ho, inv_LPI, inv_LW, inv_CW, inv_PS, inv_KT;
    unsigned short tapoff[kMaxSteps];                 // tap -> staged positions from a position's base

    // a chunk is the phases of a 3 x 3 kernel at stride 2 that is padded by one (the usual one): straight-line code
    bool phases9() const { return KT == 9 && nt[0] == 1 && nt[1] == 2 && nt[2] == 2 && nt[3] == 4; }
};

struct PrepGeom {
    int Cin, Cout, KT, G, WK;                         // contraction channels, output channels, taps, 16-channel groups (padded), K split
    int wco, wci;                                     // elements from one output / contraction channel to the next
    unsigned short wtap[kMaxSteps];                   // tap -> element
};

// One wavefront per (32 output channels, 16 contraction channels, tap): lane (l32, half) writes W[co = l32][8 half + e].
// Rounding to nearest in every piece: the pieces sum to the weight exactly and the dropped products are smallest.
__global__ __launch_bounds__(256) void split_weights_kernel(const float *__restrict__ wgt, v4u *__restrict__ ws, PrepGeom g)
{
    fetch_arguments<16 + sizeof(PrepGeom)>();
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const int t = blockIdx.z * 4 + (int)(threadIdx.x >> 6);
    if (t >= g.KT) return;
    const int grp = blockIdx.x, cb = blockIdx.y;
    const int co = cb * 32 + l32, ci0 = grp * 16 + half * 8;
    const float *src = wgt + (int64_t)(co < g.Cout ? co : 0) * g.wco + g.wtap[t];
    unsigned p[3][4];
    float f[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        // an octet that reaches beyond the last channel holds the last eight; those that the octet before it holds
        // too count as zero there (fewer than eight channels in all: the slots behind the last)
        const int cs = ci0 < g.Cin - 8 ? ci0 : (g.Cin > 8 ? g.Cin - 8 : 0), c = cs + e;
        const bool ok = co < g.Cout && c >= ci0 && c < g.Cin;
        const float v = src[(int64_t)(c < g.Cin ? c : 0) * g.wci];
        f[e] = ok ? v : 0.0f;
    }
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        unsigned short h[3][2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            __bf16 f1, f2, f3;
            split_nearest(f[e + u], f1, f2, f3);
            h[0][u] = __builtin_bit_cast(unsigned short, f1);
            h[1][u] = __builtin_bit_cast(unsigned short, f2);
            h[2][u] = __builtin_bit_cast(unsigned short, f3);
        }
#pragma unroll
        for (int q = 0; q < 3; ++q) p[q][e / 2] = (unsigned)h[q][0] | (unsigned)h[q][1] << 16;
    }
    // a wavefront's groups are consecutive: group grp belongs to wavefront grp % WK of the K split
    const int64_t step = ((int64_t)cb * g.G + (grp % g.WK) * (g.G / g.WK) + grp / g.WK) * g.KT + t;
#pragma unroll
    for (int q = 0; q < 3; ++q) ws[step * (kStepBytes / 16) + q * 64 + lane] = (v4u){p[q][0], p[q][1], p[q][2], p[q][3]};
}

// U: staged units (eight channels of one position) per thread.  S: steps per chunk and wavefront when that number is
// compiled in (the chunk is then straight-line code: the next chunk's loads go out between the first products and
// their splitting runs between the last ones; with a loop over the steps the wait counters have to assume
// the worst order of the two kinds of loads), 0: any number.  Straight-line code / the loop, us with the weights' pass, three inputs in
// turn: stride-2 adjoints, 3 x 3, [32,128,56,56] <- 128 67 / 77, [32,256,28,28] <- 256 60 / 89, [8,256,28,28] <- 512 44 / 62, [1,128,56,56] <- 128
// 17 / 22; 5 x 5 [32,256,14,14] -> 256 114 / 120, [8,128,28,28] -> 128 41 / 45.  Five taps of a row at two channel groups came out even: in the loop.  R: steps of weights held, R - 1 of them in flight.
// WPE: wavefronts per SIMD that the registers are meant for.
// P: wavefronts that only stage: they load the input, split it and write it to LDS, the others multiply.  0: every wavefront does both.
template <int MB, int NB, int WM, int WN, int WK, int U, int NPH, int WPE, int P, int S>
__global__ __launch_bounds__(64 * (WM * WN * WK + P)) __attribute__((amdgpu_waves_per_eu(WPE)))
void conv_split_kernel(const float *__restrict__ x, const v4u *__restrict__ ws, float *__restrict__ y, SplitGeom g)
{
    fetch_arguments<24 + sizeof(SplitGeom)>();
    constexpr int T = P ? 64 * P : 64 * WM * WN * WK; // threads that stage
    constexpr int R = S ? (S % 3 == 0 ? 3 : P ? 2 : S % 4 == 0 ? 4 : 5) : 2;
    static_assert(S == 0 || (S % R == 0 && (NPH == 1 || S == 9)), "the ring of weights closes over a chunk");
    static_assert(P == 0 || (S != 0 && NPH == 1), "with wavefronts that only stage: straight-line chunks of one phase");
    constexpr int kPhase9[9] = {0, 1, 1, 2, 2, 3, 3, 3, 3};      // straight-line chunks with phases: a step's phase (see launch_cfg)
    constexpr int NLO = S ? NPH : 1;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const bool stages = P == 0 || wave >= WM * WN * WK;
    const int tid = P ? (int)threadIdx.x - 64 * WM * WN * WK : (int)threadIdx.x;      // (of those that stage)
    const int wk = wave / (WM * WN), wmn = wave - wk * (WM * WN), wn = wmn / WM, wm = wmn - wn * WM;

    // XCD-aware: workgroup b runs on XCD b mod 8; each XCD takes a contiguous run of tiles, the channel tiles of one
    // position tile next to each other (they read the same input lines)
    const int Gx = (int)gridDim.x;                    // a multiple of 8
    const int id = (int)(blockIdx.x & 7) * (Gx >> 3) + (int)(blockIdx.x >> 3);
    if (id >= g.tiles * g.cot) return;
    const int pt = id / g.cot, ct = id - pt * g.cot;
    int strip = pt / g.tpf;
    strip = strip < g.nstrips - 1 ? strip : g.nstrips - 1;
    const bool last = strip == g.nstrips - 1;
    const int tw = last ? g.TWl : g.TW, bnp = last ? g.bnpl : g.bnp;
    const float inv_tw = last ? g.inv_twl : g.inv_tw;
    const int q0 = (pt - strip * g.tpf) * bnp;
    const int R0 = q0 / tw, c_0 = q0 - R0 * tw;
    const int n0 = R0 / g.Ho, oh0 = R0 - n0 * g.Ho;
    const int colbase = strip * g.TW;

    auto barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // ---- where my output positions start in the staged tile
    auto place = [&](int b, int &Rr, int &c, int &dn, int &oh) {
        int me = l32;
        if constexpr (P > 0) asm volatile("" : "+v"(me));      // (worked out twice: kept over the products the places would be spilled)
        const int jj = c_0 + (wn * NB + b) * 32 + me;
        Rr = fdiv(jj, inv_tw);
        c = jj - Rr * tw;
        const int tt = oh0 + Rr;
        dn = fdiv(tt, g.inv_Ho);
        oh = tt - dn * g.Ho;
        return (wn * NB + b) * 32 + me < bnp && R0 + Rr < g.NR;
    };
    int posb[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        int Rr, c, dn, oh;
        posb[b] = place(b, Rr, c, dn, oh) ? ((dn * g.LPI + oh * g.ls - oh0 * g.ls) * g.LW + c) * 16 : 0;
    }

    // ---- my staged units: where they come from, where they go
    const int noct = 2 * g.NC;
    int jl = bnp - 1;                                 // the tile's last position decides how many lines it needs
    {
        const int64_t left = (int64_t)g.NR * tw - q0 - 1;
        if (left < jl) jl = (int)left;
    }
    const int Rl = fdiv(c_0 + jl, inv_tw), tl = oh0 + Rl, dl = fdiv(tl, g.inv_Ho);
    const int nlines = dl * g.LPI + (tl - dl * g.Ho) * g.ls - oh0 * g.ls + g.SH;
    unsigned voff[U];                                 // bytes from image n0 to the position, channel 0; cells that do not exist: kNowhere
    int dst[U], c8[U];                                // place in the staged tile; first channel inside the chunk
    // unit i of the thread: first + i * step
    auto unit = [&](int i, int u) {
        const int oct = fdiv(u, g.inv_PS), pos = u - oct * g.PS;
        const int lr = fdiv(pos, g.inv_LW), cc = pos - lr * g.LW;
        const int cph = fdiv(cc, g.inv_CW), cq = cc - cph * g.CW;
        const int col = (colbase + cq) * g.sw + cph + g.dw0;
        const int l = oh0 * g.ls + lr, dn = fdiv(l, g.inv_LPI), r = l - dn * g.LPI;
        const int row = (g.SH >= g.sh ? r : r * g.sh) + g.dh0;
        const bool in = oct < noct;
        const bool ok = in && lr < nlines && n0 + dn < g.N && (unsigned)row < (unsigned)g.H && (unsigned)col < (unsigned)g.W;
        voff[i] = ok ? 4u * (unsigned)(dn * g.Cin * g.HW + row * g.W + col) : kNowhere;
        c8[i] = oct * 8;
        dst[i] = in ? (oct * 3 * g.PS + pos) * 16 : -1;
    };
    // (P: the first chunk is staged by everybody, U0 units each)
    constexpr int T0 = P ? T + 64 * WM * WN * WK : T, U0 = P ? (U * T + T0 - 1) / T0 : U;
#pragma unroll
    for (int i = 0; i < U0; ++i) unit(i, (int)threadIdx.x + i * T0);
    const int units = noct * g.PS;
    const int64_t x_left = 4 * (int64_t)(g.N - n0) * g.Cin * g.HW;
    const __amdgpu_buffer_rsrc_t xrs = rsrc(x + (int64_t)n0 * g.Cin * g.HW, x_left < 0x7fffffff ? (unsigned)x_left : 0x7fffffffu);
    const int cmax = g.Cin > 8 ? g.Cin - 8 : 0;       // the last eight channels: an octet that reaches beyond them starts there
    float xr[U][8];
    auto issue = [&](int i, int ch) {                 // unit i of chunk ch (no branches: the wait counters stay exact)
        int c = ch * (16 * g.NC) + c8[i];
        c = c < cmax ? c : cmax;
        const unsigned at = voff[i] == kNowhere ? kNowhere : voff[i] + 4u * (unsigned)(c * g.HW);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int se = e < g.Cin ? e : g.Cin - 1;
            xr[i][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xrs, at, 4 * se * g.HW, 0));
        }
    };
    auto commit = [&](int i, char *buf) {
        unsigned p[3][4];
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            float r1[2], r2[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const float v = xr[i][e + u];
                r1[u] = v - __uint_as_float(__float_as_uint(v) & 0xffff0000u);
                r2[u] = r1[u] - __uint_as_float(__float_as_uint(r1[u]) & 0xffff0000u);
            }
            p[0][e / 2] = pack_hi(xr[i][e], xr[i][e + 1]);
            p[1][e / 2] = pack_hi(r1[0], r1[1]);
            p[2][e / 2] = pack_hi(r2[0], r2[1]);
        }
        if (dst[i] >= 0) {
#pragma unroll
            for (int q = 0; q < 3; ++q) *(v4u *)(buf + dst[i] + q * (g.PS * 16)) = (v4u){p[q][0], p[q][1], p[q][2], p[q][3]};
        }
    };
    if constexpr (P > 0) {
#pragma unroll
        for (int i = 0; i < U0; ++i) issue(i, 0);
        if (stages) {
#pragma unroll
            for (int i = 0; i < U0; ++i)
                if (i * T0 < units) commit(i, lds);
            barrier();
            // from here on the chunk that is multiplied is one behind the one written, two behind the one asked for
            if (g.nchunk > 1) {
#pragma unroll
                for (int i = 0; i < U; ++i) unit(i, tid + i * T);
#pragma unroll
                for (int i = 0; i < U; ++i) issue(i, 1);
            }
            char *cur = lds;
            for (int ch = 1; ch < g.nchunk; ++ch) {
                cur = cur == lds ? lds + g.bufs : lds;
#pragma unroll
                for (int i = 0; i < U; ++i)
                    if (i * T < units) commit(i, cur);
                if (ch + 1 < g.nchunk) {
#pragma unroll
                    for (int i = 0; i < U; ++i) issue(i, ch + 1);
                }
                barrier();                            // chunk ch is there; chunk ch - 1 has been multiplied
            }
            for (int k = 0; k < 2 * (WK - 1); ++k) barrier();
            return;
        }
    }

    // ---- my steps' places in the staged tile, one per lane (relative to my wavefront's first channel group)
    int steptab;
    {
        const int s = lane < g.S ? lane : 0;
        const int gl = fdiv(s, g.inv_KT), t = s - gl * g.KT;
        steptab = gl * (WK * 6 * g.PS * 16) + g.tapoff[t] * 16;
    }
    const int bpiece = g.PS * 16;
    const int bbase = (2 * wk + half) * 3 * bpiece;

    // ---- weights: my MB blocks of 32 output channels, steps in order
    const int ncb = (g.Cout + 31) >> 5;
    __amdgpu_buffer_rsrc_t ars[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) {
        int cb = (ct * WM + wm) * MB + m;
        cb = cb < ncb ? cb : ncb - 1;                 // blocks beyond the last are computed from it and not stored
        ars[m] = rsrc((const char *)ws + ((int64_t)cb * WK + wk) * g.KS * kStepBytes, (unsigned)(g.KS * kStepBytes));
    }
    v4u A[R][MB][3];
    auto aload = [&](v4u (&a)[MB][3], int ks) {       // (beyond the last step: zeros that nothing uses)
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int q = 0; q < 3; ++q)
                a[m][q] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(ars[m], lane * 16 + q * 1024, ks * kStepBytes, 0));
    };
    v4u Bq[P ? 1 : 2][NB][3];
    // one piece of a step's inputs
    auto bread = [&](const char *buf, int s, int q) {
        const int off = __builtin_amdgcn_readlane(steptab, s) + bbase;
#pragma unroll
        for (int j = 0; j < NB; ++j) Bq[0][j][q] = *(const v4u *)(buf + (off + posb[j]) + q * bpiece);
    };
    auto bload = [&](v4u (&b)[NB][3], const char *buf, int s) {
        const int off = __builtin_amdgcn_readlane(steptab, s) + bbase;
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int q = 0; q < 3; ++q) b[j][q] = *(const v4u *)(buf + (off + posb[j]) + q * bpiece);
    };

    v16f acc[NPH][MB][NB];
#pragma unroll
    for (int f = 0; f < NPH; ++f)
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[f][m][b][v] = 0.0f;
    // Products of the leading pieces go to one accumulator, the other five (at most 2^-8 of them) to another, added
    // once at the end (phases in a loop over the steps: once per chunk): an output then takes one rounding of its own size per 16 channels and tap
    // instead of six.
    v16f lo[NLO][MB][NB];
    auto clear_lo = [&]() {
#pragma unroll
        for (int f = 0; f < NLO; ++f)
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v) lo[f][m][b][v] = 0.0f;
    };
    auto fold_lo = [&](v16f (&c)[MB][NB], int f) {
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int b = 0; b < NB; ++b) c[m][b] += lo[f][m][b];
    };
    clear_lo();
    auto products = [&](v16f (&c)[MB][NB], v16f (&cl)[MB][NB], const v4u (&a)[MB][3], const v4u (&b)[NB][3]) {
        constexpr int PA[6] = {2, 0, 1, 0, 1, 0}, PB[6] = {0, 0, 1, 2, 0, 1};      // (the leading product second: the chains alternate)
#pragma unroll
        for (int k = 0; k < 6; ++k)
#pragma unroll
            for (int m = 0; m < MB; ++m)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    v16f &d = k == 1 ? c[m][j] : cl[m][j];
                    d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a[m][PA[k]]),
                                                                __builtin_bit_cast(v8bf, b[j][PB[k]]), d, 0, 0, 0);
                }
    };

    if constexpr (P == 0) {
#pragma unroll
        for (int i = 0; i < U; ++i) issue(i, 0);
    }
    // (P: one set of inputs, whose pieces are read again as soon as their last product is out: three wavefronts' registers hold no second one)
    auto products_of = [&](v16f (&c)[MB][NB], v16f (&cl)[MB][NB], const v4u (&a)[MB][3], int qa, int qb) {
#pragma unroll
        for (int m = 0; m < MB; ++m)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                v16f &d = qa + qb == 0 ? c[m][j] : cl[m][j];
                d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, a[m][qa]), __builtin_bit_cast(v8bf, Bq[0][j][qb]), d, 0, 0, 0);
            }
    };

#pragma unroll
    for (int r = 0; r < R - 1; ++r) aload(A[r], r);
#pragma unroll
    for (int i = 0; i < U0; ++i)
        if (i * T0 < units) commit(i, lds);
    barrier();
    int ks = 0;                                       // my step
    char *cur = lds;
    if constexpr (P > 0) {
        for (int ch = 0; ch < g.nchunk; ++ch) {
#pragma unroll
            for (int q = 2; q >= 0; --q) bread(cur, 0, q);
#pragma unroll
            for (int s = 0; s < S; ++s) {
                aload(A[(s + R - 1) % R], ks + s + R - 1);
                __builtin_amdgcn_sched_barrier(0);
                products_of(acc[0], lo[0], A[s % R], 0, 2);
                __builtin_amdgcn_sched_barrier(0);
                if (s + 1 < S) bread(cur, s + 1, 2);
                __builtin_amdgcn_sched_barrier(0);
                products_of(acc[0], lo[0], A[s % R], 1, 1);
                products_of(acc[0], lo[0], A[s % R], 0, 1);
                __builtin_amdgcn_sched_barrier(0);
                if (s + 1 < S) bread(cur, s + 1, 1);
                __builtin_amdgcn_sched_barrier(0);
                products_of(acc[0], lo[0], A[s % R], 2, 0);
                products_of(acc[0], lo[0], A[s % R], 1, 0);
                products_of(acc[0], lo[0], A[s % R], 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (s + 1 < S) bread(cur, s + 1, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            ks += S;
            if (ch + 1 < g.nchunk) {
                cur = cur == lds ? lds + g.bufs : lds;
                barrier();
            }
        }
    } else if constexpr (S != 0) {
        // a chunk: on entry the weights of its first R - 1 steps are in slots 0 .. R - 2, on exit those of the next
        auto chunk = [&](auto more, int ch) {
            char *nxt = cur == lds ? lds + g.bufs : lds;
            bload(Bq[0], cur, 0);
#pragma unroll
            for (int s = 0; s < S; ++s) {
                aload(A[(s + R - 1) % R], ks + s + R - 1);
                if (s + 1 < S) bload(Bq[(s + 1) & 1], cur, s + 1);
                if constexpr (more.value) {
#pragma unroll
                    for (int i = 0; i < U; ++i)
                        if (i * (S / 2) / U == s) issue(i, ch + 1);
                }
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (more.value) {
#pragma unroll
                    for (int i = 0; i < U; ++i)
                        if (S - U + i == s || (S < U && s == S - 1))
                            if (i * T < units) commit(i, nxt);
                }
                constexpr bool kPh = NPH > 1;
                products(acc[kPh ? kPhase9[s % 9] : 0], lo[kPh ? kPhase9[s % 9] : 0], A[s % R], Bq[s & 1]);
                __builtin_amdgcn_sched_barrier(0);
            }
            ks += S;
            if constexpr (more.value) {
                cur = nxt;
                barrier();
            }
        };
        for (int ch = 0; ch + 1 < g.nchunk; ++ch) chunk(std::true_type{}, ch);
        chunk(std::false_type{}, 0);
    } else {
        for (int ch = 0; ch < g.nchunk; ++ch) {
            const bool more = ch + 1 < g.nchunk;
            if (more) {
#pragma unroll
                for (int i = 0; i < U; ++i) issue(i, ch + 1);
            }
            bload(Bq[0], cur, 0);
            // steps s0 .. s1 - 1; on entry the weights of step s0 are in slot 0 and its inputs in Bq[0], on exit likewise
            auto step = [&](v16f (&c)[MB][NB], int r, int s) {
                aload(A[r ^ 1], ks + 1);
                bload(Bq[r ^ 1], cur, s + 1 < g.S ? s + 1 : 0);
                __builtin_amdgcn_sched_barrier(0);
                products(c, lo[0], A[r], Bq[r]);
                __builtin_amdgcn_sched_barrier(0);
                ++ks;
            };
            auto run = [&](v16f (&c)[MB][NB], int s0, int s1) {
                int s = s0;
                for (; s + 2 <= s1; s += 2) {
                    step(c, 0, s);
                    step(c, 1, s + 1);
                }
                if (s < s1) {
                    step(c, 0, s);
#pragma unroll
                    for (int m = 0; m < MB; ++m)
#pragma unroll
                        for (int q = 0; q < 3; ++q) A[0][m][q] = A[1][m][q];
#pragma unroll
                    for (int j = 0; j < NB; ++j)
#pragma unroll
                        for (int q = 0; q < 3; ++q) Bq[0][j][q] = Bq[1][j][q];
                }
            };
            if constexpr (NPH == 1) {
                run(acc[0], 0, g.S);
            } else {
                int s = 0;                            // phases: NC = WK, the chunk's steps are its taps, phase after phase
#pragma unroll
                for (int f = 0; f < NPH; ++f) {
                    if (g.nt[f] == 0) continue;
                    clear_lo();
                    run(acc[f], s, s + g.nt[f]);
                    fold_lo(acc[f], 0);
                    s += g.nt[f];
                }
            }
            if (more) {
                cur = cur == lds ? lds + g.bufs : lds;
#pragma unroll
                for (int i = 0; i < U; ++i)
                    if (i * T < units) commit(i, cur);
                barrier();
            }
        }
    }
    if constexpr (NPH == 1 || S != 0) {
#pragma unroll
        for (int f = 0; f < NLO; ++f) fold_lo(acc[f], f);
    }

    // ---- the wavefronts that share a block add up through LDS
    if constexpr (WK > 1) {
        v4f *red = (v4f *)lds;
        constexpr int BLK = NPH * MB * NB * 4 * 64;   // v4f per wavefront
        for (int k = WK - 1; k >= 1; --k) {
            barrier();
            if (wk == k) {
#pragma unroll
                for (int f = 0; f < NPH; ++f)
#pragma unroll
                    for (int m = 0; m < MB; ++m)
#pragma unroll
                        for (int b = 0; b < NB; ++b)
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                red[wmn * BLK + (((f * MB + m) * NB + b) * 4 + v) * 64 + lane] =
                                    (v4f){acc[f][m][b][4 * v], acc[f][m][b][4 * v + 1], acc[f][m][b][4 * v + 2], acc[f][m][b][4 * v + 3]};
            }
            barrier();
            if (wk == 0) {
#pragma unroll
                for (int f = 0; f < NPH; ++f)
#pragma unroll
                    for (int m = 0; m < MB; ++m)
#pragma unroll
                        for (int b = 0; b < NB; ++b)
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const v4f q = red[wmn * BLK + (((f * MB + m) * NB + b) * 4 + v) * 64 + lane];
#pragma unroll
                                for (int u = 0; u < 4; ++u) acc[f][m][b][4 * v + u] += q[u];
                            }
            }
        }
        if (wk != 0) return;
    }

    // ---- out: register v of lane (l32, half) is output channel 8*(v/4) + 4*half + v%4 of the block, position l32
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        int Rr, c, dn, oh;
        if (!place(b, Rr, c, dn, oh)) continue;
        const int col = colbase + c;
        float *yb = y + (int64_t)(n0 + dn) * g.Cout * g.yHW + (int64_t)(oh * g.ys) * g.yW + col * g.ys;
        const bool pcol1 = 2 * col + 1 < g.yW, prow1 = 2 * oh + 1 < g.yH;      // phases: the second column / row exists
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            const int co0 = ((ct * WM + wm) * MB + m) * 32 + 4 * half;
            float *yp = yb + (int64_t)co0 * g.yHW;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int dc = 8 * (v / 4) + v % 4;
                if (co0 + dc >= g.Cout) continue;
                float *d = yp + (int64_t)dc * g.yHW;
                if constexpr (NPH == 1) {
                    *d = acc[0][m][b][v];
                } else {
                    if (pcol1) *(v2f_u *)d = (v2f){acc[0][m][b][v], acc[1][m][b][v]};
                    else *d = acc[0][m][b][v];
                    if (prow1) {
                        if (pcol1) *(v2f_u *)(d + g.yW) = (v2f){acc[2][m][b][v], acc[3][m][b][v]};
                        else d[g.yW] = acc[2][m][b][v];
                    }
                }
            }
        }
    }
}

struct Cfg {
    int mb, nb, wm, wn, wk, u, nph, wpe;
    // Wavefronts that only stage: one per SIMD beside two that multiply (in chunks of straight-line code).  Loads come back in order, so a
    // wavefront that does both waits at a weight for the input that it asked for before, and its splitting stands between its products: a chunk of
    // [32,256,14,14] -> 256 takes 9.7 k cycles without them and 8.0 k with them (6.9 k of products).  Workgroups of four multiplying wavefronts have none: with
    // six wavefronts only one workgroup finds room on a compute unit ([32,128,56,56] -> 128 at stride 2 60 us for 56).
    constexpr int stagers(int S) const { return nph == 1 && wm * wn * wk == 8 && (S == 6 || S == 8 || S == 9 || S == 12) ? 4 : 0; }
};
// wavefront block x wavefronts x K split; staged units per thread; phases; wavefronts per SIMD
constexpr Cfg kCfg[] = {
    {2, 2, 2, 2, 1, 3, 1, 1},     // 0: 128 x 128
    {2, 2, 1, 4, 1, 4, 1, 1},     // 1:  64 x 256
    {1, 2, 2, 2, 1, 4, 1, 2},     // 2:  64 x 128
    {1, 2, 2, 2, 2, 3, 1, 2},     // 3:  64 x 128, two wavefronts per block
    {1, 2, 1, 4, 1, 4, 1, 2},     // 4:  32 x 256
    {1, 2, 4, 1, 1, 4, 1, 2},     // 5: 128 x 64
    {1, 2, 2, 1, 2, 4, 1, 2},     // 6:  64 x 64, two wavefronts per block
    {1, 2, 1, 2, 2, 4, 1, 2},     // 7:  32 x 128, two wavefronts per block
    {1, 2, 1, 1, 4, 4, 1, 2},     // 8:  32 x 64, four wavefronts per block
    {1, 1, 1, 1, 4, 4, 1, 2},     // 9:  32 x 32, four wavefronts per block
    {1, 2, 2, 2, 1, 3, 4, 1},     // 10: 64 x 128 positions x 4 phases
    {1, 1, 2, 2, 1, 4, 4, 2},     // 11:  64 x 64 x 4
    {1, 1, 2, 2, 2, 3, 4, 2},     // 12:  64 x 64 x 4, two
    {1, 1, 1, 2, 2, 4, 4, 2},     // 13:  32 x 64 x 4, two wavefronts per block
    {1, 2, 4, 2, 1, 3, 1, 2},     // 14: 128 x 128, eight wavefronts
    {1, 2, 2, 4, 1, 3, 1, 2},     // 15:  64 x 256, eight
    {1, 2, 4, 1, 2, 3, 1, 2},     // 16: 128 x 64, two wavefronts per block
};
constexpr int kLargeCfg = 14;
constexpr int kNumCfg = sizeof(kCfg) / sizeof(kCfg[0]);

template <int I, int S>
hipError_t launch_steps(const float *x, const v4u *ws, float *y, const SplitGeom &g, int grid, size_t lds, hipStream_t s)
{
    constexpr Cfg c = kCfg[I];
    constexpr int P = c.stagers(S), U = P ? c.u * c.wm * c.wn * c.wk / P : c.u;
    auto k = conv_split_kernel<c.mb, c.nb, c.wm, c.wn, c.wk, U, c.nph, P ? 3 : c.wpe, P, S>;
    if (lds > 64 * 1024) {
        static std::atomic<uint64_t> raised{0};
        const hipError_t e = raise_lds((const void *)k, 160 * 1024, raised);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, dim3((unsigned)grid), dim3(64 * (c.wm * c.wn * c.wk + P)), lds, s, x, ws, y, g);
    return hipGetLastError();
}

template <int I>
hipError_t launch_cfg(const float *x, const v4u *ws, float *y, const SplitGeom &g, int grid, size_t lds, hipStream_t s)
{
    if constexpr (kCfg[I].nph == 1) {
        switch (g.S) {
        case 6: return launch_steps<I, 6>(x, ws, y, g, grid, lds, s);
        case 8: return launch_steps<I, 8>(x, ws, y, g, grid, lds, s);
        case 9: return launch_steps<I, 9>(x, ws, y, g, grid, lds, s);
        case 12: return launch_steps<I, 12>(x, ws, y, g, grid, lds, s);
        case 25: return launch_steps<I, 25>(x, ws, y, g, grid, lds, s);
        default: break;
        }
    } else if (g.phases9()) {
        return launch_steps<I, 9>(x, ws, y, g, grid, lds, s);
    }
    return launch_steps<I, 0>(x, ws, y, g, grid, lds, s);
}

// A tile's positions; the same for all configurations of as many.
struct Shape {
    int nstrips, TW, TWl, CW, LW, bnp, bnpl, tpf, tiles, PS;
};
constexpr int kMaxShapes = 10;                        // (up to five numbers of strips, each with tiles of whole rows and without)

// A tile geometry for one configuration; cost: estimated cycles of the launch.
struct Tiling : Shape {
    int cot, NC, nchunk, S, KS, bufs, need;
    double cost;
};

// The shapes of tiles of BN positions.  (32-bit divisions: this runs on every call.)
int shapes_of(const SplitGeom &g, int BN, int Wo, int SW, Shape *out)
{
    const int SWc = SW < g.sw ? SW : g.sw;            // column residues that are read
    const int whole = (int)((unsigned)(Wo + BN - 1) / BN);      // strips of at most BN columns
    const int more = (int)((unsigned)(SW - 1) / g.sw);
    int count = 0;
    for (int ns = 1; ns <= Wo; ns = ns < 4 ? ns + 1 : (ns < whole ? whole : Wo + 1)) {
        for (int aligned = 0; aligned < 2; ++aligned) {
            Shape &h = out[count];
            int tw = (int)((unsigned)(Wo + ns - 1) / ns);
            if (ns >= 4 && aligned && tw < BN) tw = BN < Wo ? BN : Wo;
            if (tw > 16384) continue;
            h.nstrips = (int)((unsigned)(Wo + tw - 1) / tw);
            h.TW = tw;
            h.TWl = Wo - (h.nstrips - 1) * tw;
            h.CW = tw + more;
            h.LW = SWc * h.CW;
            int lines = 0;
            unsigned tl[2];
            bool ok = true;
            for (int e = h.nstrips > 1 ? 0 : 1; e < 2; ++e) {       // full strips, last strip
                const int w = e ? h.TWl : h.TW;
                int bnp = BN;
                int rows = (int)((unsigned)(BN + w - 2) / w) + 1;
                const int fit = (int)((unsigned)BN / w);
                if (aligned) {
                    if (fit == 0) { ok = false; break; }
                    rows = fit;
                    bnp = rows * w;
                } else if (fit * w == BN) {
                    rows = fit;
                }
                if (rows > g.NR) rows = g.NR;
                const int crossings = (int)((unsigned)(rows - 1 + g.Ho - 1) / g.Ho);
                const int nl = (rows - 1) * g.ls + g.SH + crossings * (g.SH - g.ls);
                if (nl > lines) lines = nl;
                (e ? h.bnpl : h.bnp) = bnp;
                tl[e] = ((unsigned)g.NR * (unsigned)w + (unsigned)bnp - 1) / (unsigned)bnp;
            }
            if (!ok || lines > 4096 || lines * h.LW > 4096) continue;
            if (h.nstrips == 1) { h.bnp = h.bnpl; tl[0] = tl[1]; }
            h.PS = lines * h.LW;
            const int64_t tiles = (int64_t)tl[0] * (h.nstrips - 1) + tl[1];
            if (tiles > (1 << 30)) continue;
            h.tpf = (int)tl[0];
            h.tiles = (int)tiles;
            ++count;
        }
    }
    return count;
}

// What a launch of n workgroups per compute unit takes at least by plan's formulas: its products and weights (mfma, wld as there).
double plan_least(const Cfg &c, double mfma, double wld, double n)
{
    const double alone = 0.958 * mfma + 0.516 * wld + 6979, all = 1.419 * mfma * n;
    double t = all > alone ? all : alone;
    if (c.nph == 1 && c.wm * c.wn * c.wk == 8) {
        const double staged = 10000 + __builtin_ceil(n) * (1.157 * mfma + 16000);
        t = staged < t ? staged : t;
    }
    return t * (1 - 1e-9);                            // (rounding)
}

// The cheapest tiling of configuration c, of those that cost less than `limit`; false: there is none.  (Nothing is worked out
// for tilings whose products alone take longer than the best so far.)
bool plan(const SplitGeom &g, const Cfg &c, const Shape *shapes, int count, int Wo, int cus, double limit, Tiling *best)
{
    const int BN = 32 * c.nb * c.wn, BM = 32 * c.mb * c.wm, T = 64 * c.wm * c.wn * c.wk;
    const unsigned groups = (unsigned)(g.Cin + 15) / 16;
    bool found = false;
    Tiling h;
    h.cot = (int)((unsigned)(g.Cout + BM - 1) / BM);
    // the fewest steps that the contraction can have (whole rounds of the K split), and the fewest tiles
    const unsigned turns = (groups + c.wk - 1) / (unsigned)c.wk;
    const double steps = (double)(g.KT * (int)turns);
    const double mfma_least = steps * (c.mb * c.nb * 6 * 32) * (T / 256.0) * (c.nph == 1 ? 1.0 : 1.106), wld_least = steps * (T / 64 * c.mb * 48);
    const double per_cu = (double)h.cot / cus;
    if (plan_least(c, mfma_least, wld_least, (double)g.NR * Wo / BN * per_cu) >= limit) return false;
    for (int at = 0; at < count; ++at) {
        static_cast<Shape &>(h) = shapes[at];
        const int64_t tiles = h.tiles;
        if (tiles * h.cot > (1 << 30) || plan_least(c, mfma_least, wld_least, (double)tiles * per_cu) >= limit) continue;
        // channel groups per chunk: enough steps to pass a chunk's loads behind (kernels of few taps), whole rounds of the K split
        int nc = c.wk, per = 1;                   // per = nc / wk
        if (c.nph == 1)
            while (per * g.KT < 8 && (unsigned)(2 * nc) <= turns * c.wk && 2 * per * g.KT <= kMaxSteps &&
                   4 * nc * h.PS <= c.u * T) {
                nc *= 2;
                per *= 2;
            }
        if (2 * nc * h.PS > c.u * T) continue;
        h.NC = nc;
        h.nchunk = (int)((groups + nc - 1) / nc);
        h.S = per * g.KT;
        if (h.S > kMaxSteps) continue;
        h.KS = h.nchunk * h.S;
        const int buf = 2 * nc * 3 * h.PS * 16;
        h.bufs = h.nchunk > 1 ? buf : 0;
        h.need = buf + h.bufs;
        const int red = c.wk > 1 ? c.nph * c.mb * c.nb * 4 * 64 * 16 * c.wm * c.wn : 0;
        if (h.need < red) h.need = red;
        if (h.need > 156 * 1024) continue;
        // Estimated time, in cycles: a workgroup alone takes `alone`, res of them share a compute unit at one per
        // `shared`.  The constants are fitted to 1900 measured launches (104 layers, both directions, configurations
        // 0 - 13): the choice they give is on average 1 % slower than the best configuration of each layer.  Layers that
        // 14, 15 and 16 take by them (and keep_smaller) against those before: with staging wavefronts 9, 14 and 15 % faster on average, without 11, 8 and 8 % (834 layers).
        const double wpw = T / 256.0;             // wavefronts per SIMD and workgroup
        double res = c.wpe / wpw;                 // workgroups per compute unit: registers, 160 KB of LDS
        const int by_lds = 160 * 1024 / h.need;
        if (by_lds < res) res = by_lds;
        if (res < 1) res = 1;
        // (fitted before layers of 25 taps and the usual phases became straight-line chunks: calling them that here chose worse, [32,512,14,14] -> 512
        // 71 us for 65, 5 x 5 on [8,50,40,40] -> 30 21.5 for 19.9)
        const bool line = c.nph == 1 && (h.S == 6 || h.S == 8 || h.S == 9 || h.S == 12);      // straight-line chunks
        const double mfma = (double)h.KS * c.mb * c.nb * 6 * 32 * wpw * (c.nph == 1 ? 1.0 : 1.106);
        const double wld = (double)h.KS * (T / 64) * c.mb * 48;       // weights through the vector cache, 64 bytes per cycle
        const double stage = h.nchunk * (890 + 375 * wpw * ((2 * nc * h.PS + T - 1) / T)) * (line ? 1.0 : 1.105);
        const double m = 1.419 * mfma, l = 0.157 * wld;
        const double shared = (m > l ? m : l) + 0.625 * stage;
        const double alone = 0.958 * mfma + 0.516 * wld + stage + 6979 + (c.wk > 1 ? 466 * c.mb * c.nb * c.nph : 0);
        const double n = (double)tiles * h.cot / cus;
        // Where the staged form's estimate does not hold: 128 channels a tile of which half or more do not exist, in more than one round of one workgroup per unit (3 x 3 at
        // stride 2: [64,200,41,41] -> 32 82 us / 96 with it, [51,224,67,67] -> 32 156 / 167), is left to the others.  The tile of 64 x 128, which was there before that form, is
        // then estimated as it was, also at half a tile of channels ([4,384,90,90] -> 32 70 / 75, [1,200,99,99] -> 495 123 / 126).
        const bool rounds = (int64_t)tiles * h.cot > cus, half = 2 * g.Cout <= BM;
        const bool staged = c.stagers(h.S) > 0;
        if (staged && c.wm == 4 && rounds && half) continue;
        const bool before = c.wm == 2 && c.wn == 2;   // (the tile of 64 x 128)
        if (staged && !(before && (rounds || half))) {
            // one workgroup per compute unit; a chunk takes its products or its staging (1350 cycles per unit of a staging thread), whichever is longer
            const double prod = 1.157 * mfma / h.nchunk, put = 1350.0 * ((2 * nc * h.PS + 255) / 256);
            const double t = 10000 + __builtin_ceil(n) * (h.nchunk * (prod > put ? prod : put) + 16000 + (c.wk > 1 ? 466 * c.mb * c.nb : 0));
            if (t < limit) {
                found = true;
                h.cost = limit = t;
                *best = h;
            }
            if (!before) continue;                    // (that one is never slower than it was: also where its own estimate is the larger one)
        }
        const double full = __builtin_floor(n / res), rem = n - full * res;
        double t = full * (res * shared > alone ? res * shared : alone);
        if (rem > 0) t += __builtin_ceil(rem) * shared > alone ? __builtin_ceil(rem) * shared : alone;
        if (t < limit) {
            found = true;
            h.cost = limit = t;
            *best = h;
        }
    }
    return found;
}

// The largest configurations against the one that the estimate puts just behind: not the estimate but measurements of 5000 layers.  h: the tiling of i, b: that
// of bi.  true: bi stays.
bool keep_smaller(int i, const Tiling &h, int bi, const Tiling &b, int64_t Cout, int cus)
{
    const bool staged = kCfg[i].stagers(h.S) > 0, rounds = (int64_t)h.tiles * h.cot > cus;
    // With staging wavefronts 14 is up to 5 % slower than 6 where a tenth or more of its channels do not exist and 3 - 12 % faster where they do; 15 and 16 are 1 - 13 % slower than 6
    // on nine taps where they fill more than four fifths of the compute units, and 3 - 14 % faster below.
    if (bi == 6 && staged) return i == 14 ? 10 * Cout <= 9 * 128 * h.cot : h.S == 9 && 5LL * h.tiles * h.cot > 4 * cus;
    // Without them 16 is 0 - 15 % slower than 3, 3 % on average, and, in more than one round, 0 - 4 % slower than 5 (in one 3 - 18 % faster); 14 in more than one round, where
    // the estimates differ by less than 1 %, up to 3 % slower than 5; beside 6 it is 1 % faster to 5 % slower.
    if (staged) return false;
    if (i == 16) return bi == 3 || (bi == 5 && rounds);
    return i == 14 && (bi == 6 || (bi == 5 && rounds && h.cost > 0.99 * b.cost));
}

}  // namespace

// One short contraction: the extra launch and the longer start cost more than the products save, the fp32 kernels
// are ahead.  Measured (them / here, us): 1 x 1 of 32 channels [8,32,362] -> 384 6.3 / 9.1, [32,32,40,17] -> 256
// 12.4 / 14.8, but [64,32,29,29] -> 259 35.6 / 29.6; of 64 channels [64,64,8,8] -> 80 7.5 / 8.9, but
// [32,64,26,26] -> 80 13.4 / 11.0.
static bool short_contraction(int64_t Cin, int64_t Cout, int64_t KT, int64_t positions)
{
    const double flop = 2.0 * (double)positions * (double)Cout * (double)Cin;
    return KT == 1 && ((Cin == 32 && flop < 4e8) || (Cin == 64 && flop < 1e8));
}

// Bytes of workspace for a dense layer of Cin contraction channels, Cout result channels and KT taps; 0: not used.
int64_t conv_split_workspace(int64_t Cin, int64_t Cout, int64_t KT, int64_t positions)
{
    if (KT > kMaxSteps || short_contraction(Cin, Cout, KT, positions)) return 0;
    // the contraction is padded to whole chunks, and a chunk is at most the contraction rounded up to four groups
    const int64_t groups = (Cin + 15) / 16, cb = (Cout + 31) / 32;
    const int64_t padded = 2 * groups + 4 < groups + 32 ? 2 * groups + 4 : groups + 32;
    return (cb * padded * KT + kPadSteps) * kStepBytes;
}

// A dense layer given by its taps: tap t reads input row oh*sh + dh[t], column ow*sw + dw[t] with the weights at
// wgt + co*wco + ci*wci + wt[t]; output cell (oh, ow) of Ho x Wo.  phases: ph[t] = 2*er + ec, output cell (2 oh + er,
// 2 ow + ec) of yH x yW, taps in ascending order of phase, sh = sw = 1.
hipError_t launch_conv_split(const float *x, const float *wgt, float *y, int64_t N, int64_t Cin, int64_t H, int64_t W,
                             int64_t Cout, int64_t Ho, int64_t Wo, int64_t yH, int64_t yW, int sh, int sw, int KT,
                             const int *dh, const int *dw, const int *wt, const int *ph, int64_t wco, int64_t wci, Workspace ws,
                             hipStream_t s, bool *taken)
{
    *taken = false;
    if (!ws.p || ((uintptr_t)ws.p & 15) || KT < 1 || KT > kMaxSteps || sh > 2 || sw > 2 || N < 1) return hipSuccess;
    if (N * Ho >= (1LL << 30) || H >= (1 << 18) || Ho >= (1 << 18) || W >= (1LL << 28) || Wo >= (1LL << 28) || Cout * wco >= (1LL << 31) ||
        Cin * wci >= (1LL << 31) || Cin * H * W >= (1LL << 27) || yH * yW >= (1LL << 30) || N * Ho * Wo >= (1LL << 31) - 65536)
        return hipSuccess;
    // ... likewise 1-D of 32 channels, k = 3 (conv1d_split.hip): [32,32,235] -> 64 8.0 / 9.8, but [32,32,283] -> 188 12.9 / 11.8
    const bool forced = g_opt.conv2d_variant >= 100;
    if (!forced && (short_contraction(Cin, Cout, KT, N * Ho * Wo) ||
                    (KT == 3 && Cin == 32 && H == 1 && !ph && wci == KT && sw == 1 && 192.0 * N * Wo * Cout < 1e8)))
        return hipSuccess;
    SplitGeom g;
    g.N = (int)N; g.Cin = (int)Cin; g.H = (int)H; g.W = (int)W; g.HW = (int)(H * W); g.Cout = (int)Cout; g.Ho = (int)Ho;
    g.NR = (int)(N * Ho);
    g.KT = KT; g.sh = sh; g.sw = sw;
    g.yH = (int)yH; g.yW = (int)yW; g.yHW = (int)(yH * yW); g.ys = ph ? 2 : 1;
    int h0 = dh[0], h1 = dh[0], w0 = dw[0], w1 = dw[0];
    for (int t = 1; t < KT; ++t) {
        h0 = dh[t] < h0 ? dh[t] : h0; h1 = dh[t] > h1 ? dh[t] : h1;
        w0 = dw[t] < w0 ? dw[t] : w0; w1 = dw[t] > w1 ? dw[t] : w1;
    }
    g.dh0 = h0; g.dw0 = w0; g.SH = h1 - h0 + 1;
    const int SW = w1 - w0 + 1;
    if (g.SH > 1024 || SW > 4096) return hipSuccess;
    g.ls = g.SH < sh ? g.SH : sh;
    g.LPI = (int)(Ho - 1) * g.ls + g.SH;
    for (int f = 0; f < 4; ++f) g.nt[f] = 0;
    if (ph)
        for (int t = 0; t < KT; ++t) ++g.nt[ph[t]];
    const int cus = device_cus();
    // the configuration whose estimated time is smallest
    int bi = -1;
    Tiling b;
    const int force = forced ? g_opt.conv2d_variant - 100 : -1;       // A/B and tests: this configuration
    bool kept = false;
    Shape shapes[4][kMaxShapes];
    int counts[4] = {-1, -1, -1, -1};
    for (int i = 0; i < kNumCfg; ++i) {
        if ((kCfg[i].nph > 1) != (ph != nullptr) || (force >= 0 && force < kNumCfg && force != i)) continue;
        // (a tile each for a third of the compute units: below that the largest tiles never win, and planning them is host time of every call)
        if (i >= kLargeCfg && force < 0 && 3.0 * N * Ho * Wo * Cout < (double)cus * (1024 * kCfg[i].mb * kCfg[i].nb * kCfg[i].wm * kCfg[i].wn)) continue;
        Tiling h;
        const int nbwn = kCfg[i].nb * kCfg[i].wn, of = nbwn >= 8 ? 3 : nbwn >> 1;      // (1, 2, 4 or 8 blocks of 32 positions)
        if (counts[of] < 0) counts[of] = shapes_of(g, 32 * nbwn, (int)Wo, SW, shapes[of]);
        if (!plan(g, kCfg[i], shapes[of], counts[of], (int)Wo, cus, bi < 0 ? 1e300 : b.cost, &h)) continue;
        if (force < 0 && i >= kLargeCfg && bi >= 0) {
            if (i == 16 && kept) continue;            // (2 - 12 % slower than 6 where 14 or 15 is slower)
            const bool keep = keep_smaller(i, h, bi, b, Cout, cus);
            kept |= keep && bi == 6;
            if (keep) continue;
        }
        // a tile's images, and a wavefront's weights, within 32-bit offsets
        const int64_t imgs = (int64_t)(h.bnp > h.bnpl ? h.bnp : h.bnpl) / (h.TWl * Ho) + 2;
        if (imgs * Cin * H * W >= (1LL << 29) || (int64_t)h.KS * kStepBytes >= (1LL << 31)) continue;
        bi = i;
        b = h;
    }
    if (bi < 0) return hipSuccess;
    const Cfg &c = kCfg[bi];
    const int ncb = (int)((Cout + 31) / 32);
    const int64_t G = (int64_t)b.nchunk * b.NC;
    if (((int64_t)ncb * G * KT + kPadSteps) * kStepBytes > ws.bytes || G > 65535 || ncb > 65535) return hipSuccess;
    g.nstrips = b.nstrips; g.TW = b.TW; g.TWl = b.TWl; g.CW = b.CW; g.LW = b.LW; g.bnp = b.bnp; g.bnpl = b.bnpl; g.tpf = b.tpf;
    g.tiles = b.tiles; g.cot = b.cot; g.PS = b.PS; g.NC = b.NC; g.nchunk = b.nchunk; g.S = b.S; g.KS = b.KS; g.bufs = b.bufs;
    g.inv_tw = 1.0f / g.TW; g.inv_twl = 1.0f / g.TWl; g.inv_Ho = 1.0f / g.Ho; g.inv_LPI = 1.0f / g.LPI;
    g.inv_LW = 1.0f / g.LW; g.inv_CW = 1.0f / g.CW; g.inv_PS = 1.0f / g.PS; g.inv_KT = 1.0f / g.KT;
    for (int t = 0; t < KT; ++t) {
        const int a = dh[t] - h0, b = dw[t] - w0;
        g.tapoff[t] = (unsigned short)(a * g.LW + b % sw * g.CW + b / sw);
    }
    for (int t = KT; t < kMaxSteps; ++t) g.tapoff[t] = 0;
    PrepGeom p;
    p.Cin = (int)Cin; p.Cout = (int)Cout; p.KT = KT; p.G = (int)G; p.WK = c.wk; p.wco = (int)wco; p.wci = (int)wci;
    for (int t = 0; t < kMaxSteps; ++t) p.wtap[t] = (unsigned short)(t < KT ? wt[t] : 0);
    const int grid = (int)xcd_grid((int64_t)g.tiles * g.cot);
    *taken = true;
    hipLaunchKernelGGL(split_weights_kernel, dim3((unsigned)G, (unsigned)ncb, (unsigned)((KT + 3) / 4)), dim3(256), 0, s, wgt,
                       (v4u *)ws.p, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
#define SWS_CFG(I) case I: return launch_cfg<I>(x, (const v4u *)ws.p, y, g, grid, (size_t)b.need, s)
    switch (bi) {
        SWS_CFG(0); SWS_CFG(1); SWS_CFG(2); SWS_CFG(3); SWS_CFG(4); SWS_CFG(5); SWS_CFG(6); SWS_CFG(7); SWS_CFG(8); SWS_CFG(9);
        SWS_CFG(10); SWS_CFG(11); SWS_CFG(12); SWS_CFG(13); SWS_CFG(14); SWS_CFG(15);
    default: return launch_cfg<16>(x, (const v4u *)ws.p, y, g, grid, (size_t)b.need, s);
    }
#undef SWS_CFG
}

}  // namespace sws
