// Thin convolution (one input channel per output channel, Section 2.5) on the bf16 matrix cores with exactly split fp32
// operands: stride 1, taps adjacent or 4, 8, 16, 32 apart, forward and the adjoint with respect to the input (taps last first).
//
// The taps at distance d act on each of the d phases of a row by themselves.  32 consecutive outputs of one phase are
//     out[m + j] = sum over s of  X[m + s] * T[s][j],   T[s][j] = f[s - j] (0 <= s - j < k, else 0),
// and 32 such runs together are the product of a 32 x S by an S x 32 matrix, S = 31 + k rounded up to 16.  Both operands
// are exact sums of three bf16 numbers; six of the nine products of pieces are accumulated in fp32 (the other three are below 2^-21 of
// their term; up to 17 taps, whose sums round so little that this would show, eight) in one accumulator: the lesser ones of all slices first,
// at most 2^-6 of the terms, then the leading ones on top, so that a result takes S / 16 <= 6 roundings of its own size.  A
// tile of 1024 outputs takes 6 S / 16 instructions of 32 cycles (k = 51: 1152 cycles) where one fused multiply-add per tap and output takes
// 64 k (3264).
//
// A workgroup stages the inputs of its NW tiles (one per wavefront) once, split, as three planes of 16-bit numbers in LDS, in the order
// of memory.  T is built once per workgroup and stays in registers.  d = 1: a lane's eight consecutive s are 16
// bytes of a plane.  d >= 4: they lie d apart, and the transposing load ds_read_b64_tr_b16 hands them out: sixteen lanes
// point at four s x sixteen runs (four phases of one s are adjacent).  Every 32 d elements of a plane are followed by a
// gap (d = 1: 16 bytes after every 256), which puts the lanes of a read on different banks.  The rows of the product are the runs, so a
// lane holds four phases of one position: d >= 4 stores whole 16-byte groups, 64 bytes and more side by side; d = 1: 128 bytes.
//
// Loads of the next tile are in flight during a tile's products, and it is split into LDS before the tile's stores, which its loads would
// otherwise be waited for behind; the first tile's go out before T is built.  Bound by HBM up to its workgroups' starts and barriers (three wavefronts
// per SIMD: T takes 72 registers at 51 taps).  Measured, cold inputs, us, the vector-ALU kernels / this one: [1,1024,65536], 51 taps 8 apart
// 168 / 104 (a copy of that size 86; matrix cores 41 % busy), 49 taps 32 apart, which no other kernel but the direct one takes,
// [8,64,65536] 1256 / 82.  Error against 64 bits 4.5e-8 (vector ALU 1.3e-7).
//
// bf16 reaches down to 2^-133: three pieces hold every bit of a number from 2^-110 on.  Inputs are multiplied by 2^40 before they are
// split, so that this is all of them, and taps by 2^-40; a channel with a tap below 2^-70 has its taps multiplied by 2^40
// too, and its results by 2^-80.
//
// An input that is not finite makes every output of its run NaN (zeros of T meet it), and one beyond 2^87 is not finite when multiplied; a
// tile with a result that is not finite is therefore evaluated again, tap by tap from memory.
#include "sws_internal.h"

namespace sws {

namespace {

constexpr int kTile = 1024;                           // outputs per wavefront
constexpr float kUp = 0x1p40f;

// A workgroup takes `rows` rows of one channel (images apart) and `group` tiles of NW * 1024 outputs of each.
struct ToepGeom {
    int B, L, Lo, k, pad, Cin, Cout, cog;
    int tiles, group, chunks, rows;                   // tiles of a row, of a workgroup's row; workgroups per row; rows per workgroup
    int wflip, units;
};

// NCH: slices of 16 s, 31 + k <= 16 NCH.  LD: log2 of the taps' distance (0, 2 .. 5).  NW: wavefronts.
template <int NCH, int LD, int NW>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(NCH <= 3 ? 4 : NCH == 6 && (LD >= 4 || (LD == 3 && NW == 1)) ? 2 : 3)))
void conv1d_toep_kernel(const float *__restrict__ x, const float *__restrict__ wgt, float *__restrict__ y, ToepGeom g)
{
    constexpr int T = 64 * NW, D = 1 << LD, TO = kTile * NW;
    constexpr int NI = TO + (16 * NCH - 32) * D;      // staged inputs
    constexpr int U = (NI + 4 * T - 1) / (4 * T);     // groups of four per thread
    // place of element q in a plane (16-bit elements)
    constexpr int BLK = LD ? 5 + LD : 7, GAP = LD ? 4 * D : 8;
    auto at = [](int q) { return q + GAP * (q >> BLK); };
    constexpr int PLANE = ((NI + GAP * (NI >> BLK)) + 7) / 8 * 8;
    constexpr int TLEN = 16 * NCH + 48;
    __shared__ __attribute__((aligned(16))) unsigned short plane[3 * PLANE];
    __shared__ __attribute__((aligned(16))) unsigned short taps[3][2][TLEN];

    const int unit = xcd_run_unit(g.units);
    if (unit < 0) return;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rc = (unsigned)unit / (unsigned)g.chunks, chunk = unit - rc * g.chunks;
    const int b0 = (unsigned)rc / (unsigned)g.Cout, co = rc - b0 * g.Cout, ci = (unsigned)co / (unsigned)g.cog;
    const float *wr = wgt + (int64_t)co * g.k;
    int b = b0 * g.rows;
    const int b_end = b + g.rows < g.B ? b + g.rows : g.B;
    const int t_first = chunk * g.group, t_end = t_first + g.group < g.tiles ? t_first + g.group : g.tiles;

    v4f in[U];
    // tile origins are pulled back: groups of stores start on 64-byte lines of y
    auto shift = [&](int b) { return ((b * g.Cout + co) & 15) * (g.Lo & 15) & 15; };
    // (no conditional loads: the compiler would wait for them at once)
    auto load = [&](int b, int t) {
        const int p0 = t * TO - shift(b) - g.pad, o = p0 > 0 ? p0 : 0;       // (descriptor from there on: rows of any length)
        const int64_t left = 4 * ((int64_t)g.L - o);
        const __amdgpu_buffer_rsrc_t xrs = rsrc(x + ((int64_t)b * g.Cin + ci) * g.L + o, left < 0 ? 0u : (left < 0x7fffffff ? (unsigned)left : 0x7fffffffu));
        if (p0 >= 0 && p0 + 4 * T * U <= g.L) {
#pragma unroll
            for (int i = 0; i < U; ++i) in[i] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(xrs, 16 * tid, 16 * T * i, 0));
        } else {
#pragma unroll
            for (int i = 0; i < U; ++i) {
                const int p = p0 + 4 * (tid + i * T);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    in[i][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xrs, p + e < 0 ? kNowhere : 4u * (unsigned)(p + e - o), 0, 0));
            }
        }
    };
    auto commit = [&]() {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int q = 4 * (tid + i * T);
            if ((i + 1) * 4 * T > NI && q >= NI) continue;
            float f[4], r1[4], r2[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                f[e] = kUp * in[i][e];
                r1[e] = f[e] - __uint_as_float(__float_as_uint(f[e]) & 0xffff0000u);
                r2[e] = r1[e] - __uint_as_float(__float_as_uint(r1[e]) & 0xffff0000u);
            }
            unsigned short *d = plane + at(q);
            *(v2u *)d = (v2u){pack_hi(f[0], f[1]), pack_hi(f[2], f[3])};
            *(v2u *)(d + PLANE) = (v2u){pack_hi(r1[0], r1[1]), pack_hi(r1[2], r1[3])};
            *(v2u *)(d + 2 * PLANE) = (v2u){pack_hi(r2[0], r2[1]), pack_hi(r2[2], r2[3])};
        }
    };
    auto barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // (lane t of every wavefront holds tap t, k <= 64: one load, and all lanes take part; the first tile's loads go out before it is waited for)
    const float tap = lane < g.k ? wr[g.wflip ? g.k - 1 - lane : lane] : 0.0f;
    int t = t_first;
    load(b, t);
    __builtin_amdgcn_sched_barrier(0);
    const bool tiny = __builtin_amdgcn_ballot_w64(tap != 0.0f && __builtin_fabsf(tap) < 0x1p-70f) != 0;
    const float scaled = tap * (tiny ? kUp : 1.0f / kUp);

    // ---- T: slot p of copy X holds tap p - 32 - X (zero outside [0, k)), so that a lane's eight taps, from tap
    // 16 c + 8 half - j on, start on a dword of copy j & 1
#pragma unroll
    for (int i0 = 0; i0 < 2 * TLEN; i0 += T) {
        const int i = i0 + tid, X = i >= TLEN, p = i - X * TLEN, t = p - 32 - X;
        const float f = __shfl(scaled, t & 63, kWave);
        __bf16 f1, f2, f3;
        split_nearest(t >= 0 && t < g.k ? f : 0.0f, f1, f2, f3);
        if (i < 2 * TLEN) {
            taps[0][X][p] = __builtin_bit_cast(unsigned short, f1);
            taps[1][X][p] = __builtin_bit_cast(unsigned short, f2);
            taps[2][X][p] = __builtin_bit_cast(unsigned short, f3);
        }
    }
    barrier();
    v8bf F[3][NCH];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const int pos = 16 * c + 8 * half - l32 + 32 + (l32 & 1);      // even, >= 2, pos + 7 < TLEN
            const unsigned *src = (const unsigned *)&taps[p][l32 & 1][pos];
            F[p][c] = __builtin_bit_cast(v8bf, (v4u){src[0], src[1], src[2], src[3]});
        }

    // my reads.  d = 1: run l32, s = 16 c + 8 half.  d >= 4: lane 16 a + m of the wavefront points at runs 16 (a & 1) + 4 (m & 3),
    // s = 8 (a >> 1) + m / 4; run r is phase r % d of block r / d of 32 d elements
    int base;
    if constexpr (LD == 0) {
        base = kTile * wave + 32 * l32 + 8 * half;
    } else {
        const int a = lane >> 4, m = lane & 15, r = 16 * (a & 1) + 4 * (m & 3), s = 8 * (a >> 1) + (m >> 2);
        base = kTile * wave + ((r >> LD) << (5 + LD)) + (s << LD) + (r & (D - 1));
    }
    auto operand = [&](int base, int p, int c) -> v8bf {
        if constexpr (LD == 0) {
            return __builtin_bit_cast(v8bf, *(const v4u *)(plane + p * PLANE + at(base + 16 * c)));
        } else {
            // (16 c d is a multiple of half a block, s and r stay inside a half)
            const unsigned short *q = plane + p * PLANE + at(base + ((16 * c) << LD));
            return tr8((const char *)q, (const char *)(q + (4 << LD)));
        }
    };

    commit();
    for (bool more = true; more;) {
        barrier();
        const int q0 = t * TO - shift(b) + kTile * wave, b_now = b;
        if (++t == t_end) {
            t = t_first;
            ++b;
        }
        more = b < b_end;
        if (more) load(b, t);
        const bool mine = q0 < g.Lo && q0 + kTile > 0;                // (the last tiles of a row may lie behind it)
        v16f hi = {0.0f};
        if (mine) {
            // the five lesser products first, the leading ones on top of their sum
            v8bf x0[NCH];
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                const v8bf x2 = operand(base, 2, c), x1 = operand(base, 1, c);
                x0[c] = operand(base, 0, c);
                if constexpr (NCH < 4) {              // (eight products: see conv1d_toep_takes)
                    hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x2, F[1][c], hi, 0, 0, 0);
                    hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x1, F[2][c], hi, 0, 0, 0);
                }
                hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x2, F[0][c], hi, 0, 0, 0);
                hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x1, F[1][c], hi, 0, 0, 0);
                hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x0[c], F[2][c], hi, 0, 0, 0);
                hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x1, F[0][c], hi, 0, 0, 0);
                hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x0[c], F[1][c], hi, 0, 0, 0);
            }
            if constexpr (NCH > 5) {                  // (the leading pieces read again, or their registers would be spilled)
                int again = base;
                asm volatile("" : "+v"(again));
#pragma unroll
                for (int c = 0; c < NCH; ++c) x0[c] = operand(again, 0, c);
            }
#pragma unroll
            for (int c = 0; c < NCH; ++c) hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x0[c], F[0][c], hi, 0, 0, 0);
        }
        // (the next tile goes to LDS before the stores: its loads are then not waited for behind them)
        if (more) {
            barrier();                                // everybody has read the tile
            commit();
        }
        // ---- out: register v is run 8 (v / 4) + 4 half + v % 4, position l32
        if (!mine) continue;
        float *yr = y + ((int64_t)b_now * g.Cout + co) * g.Lo;
        if (tiny) {
#pragma unroll
            for (int v = 0; v < 16; ++v) hi[v] *= 1.0f / (kUp * kUp);
        }
        float s = 0.0f;
#pragma unroll
        for (int v = 0; v < 16; ++v) s += hi[v];
        const bool again = __builtin_amdgcn_ballot_w64(!__builtin_isfinite(s)) != 0;
        if (!again && q0 >= 0 && q0 + kTile <= g.Lo) {
            if constexpr (LD == 0) {
                float *d = yr + q0 + 128 * half + l32;
#pragma unroll
                for (int v = 0; v < 16; ++v) __builtin_nontemporal_store(hi[v], d + 32 * (8 * (v / 4) + v % 4));
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int r = 8 * u + 4 * half;
                    const v4f o = {hi[4 * u], hi[4 * u + 1], hi[4 * u + 2], hi[4 * u + 3]};
                    __builtin_nontemporal_store(o, (v4f_u *)(yr + q0 + ((r >> LD) << (5 + LD)) + (l32 << LD) + (r & (D - 1))));
                }
            }
        } else if (!again) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int r = 8 * (v / 4) + 4 * half + v % 4, q = q0 + ((r >> LD) << (5 + LD)) + (l32 << LD) + (r & (D - 1));
                if (q >= 0 && q < g.Lo) yr[q] = hi[v];
            }
        } else {
            // Eight outputs per lane at a time, 64 apart (one at a time, each load waited for: 2930 us for the dilated layer above with a NaN in
            // every tile, now 1300; bound by L2).  Loads outside the row return zero, which is no term where the tap is not finite.
            const int p0 = q0 - g.pad, o = p0 > 0 ? p0 : 0;
            const int64_t left = 4 * ((int64_t)g.L - o);
            const __amdgpu_buffer_rsrc_t xrs = rsrc(x + ((int64_t)b_now * g.Cin + ci) * g.L + o, left < 0 ? 0u : (left < 0x7fffffff ? (unsigned)left : 0x7fffffffu));
#pragma unroll 1
            for (int h = lane; h < kTile; h += 512) {
                float acc[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) acc[i] = 0.0f;
                float next = wr[g.wflip ? g.k - 1 : 0];
#pragma unroll 1
                for (int u = 0; u < g.k; ++u) {
                    const float f = next;
                    const int un = u + 1 < g.k ? u + 1 : u, p = p0 + u * D + h;
                    next = wr[g.wflip ? g.k - 1 - un : un];
                    float e[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        e[i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xrs, p + 64 * i < 0 ? kNowhere : 4u * (unsigned)(p + 64 * i - o), 0, 0));
                    const bool finite = __builtin_isfinite(f);
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        if (finite || (p + 64 * i >= 0 && p + 64 * i < g.L)) acc[i] = __builtin_fmaf(f, e[i], acc[i]);
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int q = q0 + h + 64 * i;
                    if (q >= 0 && q < g.Lo) yr[q] = acc[i];
                }
            }
            // (no load is left when the next tile's are in flight: the compiler would wait for both)
            __builtin_amdgcn_s_waitcnt(0x0f70);       // vmcnt(0)
        }
    }
}

template <int NCH, int LD, int NW>
hipError_t launch(const float *x, const float *wgt, float *y, ToepGeom g, hipStream_t s)
{
    constexpr int TO = kTile * NW;
    g.tiles = (g.Lo + max_origin_shift(g.Lo, 16) + TO - 1) / TO;
    // Tiles of a row per workgroup, one to four: T is built once for them, in about a tile's time, and a compute unit holds twelve wavefronts.
    // The fewest rounds of workgroups times tiles; with one tile each wherever that fills the device ([16,64,4000], 33 taps, 1.3
    // rounds) 12.2 us, now 9.9.
    const int64_t places = 12 * (int64_t)device_cus() / NW, rows_out = (int64_t)g.B * g.Cout;
    const int per = g_opt.slide_group > 0 ? (int)g_opt.slide_group : 4;
    int64_t best = 0;
    for (int t = g_opt.slide_group > 0 && per < g.tiles ? per : 1; t <= per && t <= g.tiles; ++t) {
        const int chunks = (g.tiles + t - 1) / t;
        const int64_t cost = (rows_out * chunks + places - 1) / places * (t + 1);
        if (best == 0 || cost <= best) {
            best = cost;
            g.chunks = chunks;
        }
    }
    g.group = (g.tiles + g.chunks - 1) / g.chunks;
    g.chunks = (g.tiles + g.group - 1) / g.group;
    g.rows = 1;
    while (g.chunks == 1 && (g.rows + 1) * g.tiles <= per && (int64_t)((g.B + g.rows) / (g.rows + 1)) * g.Cout >= 4 * places) ++g.rows;
    const int64_t units = (int64_t)((g.B + g.rows - 1) / g.rows) * g.Cout * g.chunks, grid = xcd_run_grid(units);
    if (grid > 2147483647LL - 64) return kNotTaken;
    g.units = (int)units;
    hipLaunchKernelGGL((conv1d_toep_kernel<NCH, LD, NW>), dim3((unsigned)grid), dim3(64 * NW), 0, s, x, wgt, y, g);
    return hipGetLastError();
}

// Two wavefronts per workgroup, or three where that leaves fewer of them without outputs; one for rows of a few tiles, if a tile's halo is short
// ([40,128,3000], 41 taps 32.5 us with three, 30 with one; [32,64,4000], 33 taps 4 apart 18.7 with two, 17.4).
template <int NCH, int LD>
hipError_t launch_waves(const float *x, const float *wgt, float *y, const ToepGeom &g, hipStream_t s)
{
    const int n = (g.Lo + max_origin_shift(g.Lo, 16) + kTile - 1) / kTile;
    if constexpr (NCH < 4) {                          // (few taps: only rows of one tile come here, see conv1d_toep_wanted)
        if constexpr (LD >= 2 && LD <= 4)
            if (n == 1) return launch<NCH, LD, 1>(x, wgt, y, g, s);
        return kNotTaken;
    } else if constexpr (LD < 5) {
        if (n == 1 || (n <= 4 && LD <= 2)) return launch<NCH, LD, 1>(x, wgt, y, g, s);
        if ((n + 2) / 3 * 3 < (n + 1) / 2 * 2) return launch<NCH, LD, 3>(x, wgt, y, g, s);
        return launch<NCH, LD, 2>(x, wgt, y, g, s);
    } else {
        return launch<NCH, LD, 2>(x, wgt, y, g, s);
    }
}

template <int LD>
hipError_t launch_taps(const float *x, const float *wgt, float *y, const ToepGeom &g, hipStream_t s)
{
    switch ((31 + g.k + 15) / 16) {
    case 3: return launch_waves<3, LD>(x, wgt, y, g, s);
    case 4: return launch_waves<4, LD>(x, wgt, y, g, s);
    case 5: return launch_waves<5, LD>(x, wgt, y, g, s);
    case 6: return launch_waves<6, LD>(x, wgt, y, g, s);
    default: return kNotTaken;
    }
}

}  // namespace

// One and two taps keep their fp32 kernels, whose few roundings are less than the matrix cores'.  Error against 64 bits, 2-norm of normal
// numbers and of numbers in 0 .. 1 (multiply-adds / here, 1e-8): k = 1 2.5, 2.5 / 3.4, 3.3, k = 2 3.1, 3.0 / 3.3, 3.0, k = 3 3.6, 3.3 / 3.2, 2.8,
// k = 5 4.1, 3.9 / 3.2, 2.8, k = 17 7.5, 6.4 / 3.4, 3.1, k = 33 10, 8.5 / 4.2, 3.4.
bool conv1d_toep_takes(int32_t k, int32_t dilation)
{
    return k >= 3 && k <= 64 && (dilation == 1 || dilation == 4 || dilation == 8 || dilation == 16 || dilation == 32);
}

// More than 32 taps: the vector-ALU kernels are bound by their multiply-adds.  Measured (them / here, us, cold inputs): dilation 1, [1,512,65536]
// k = 25 48 / 56, 33 53 / 54, 37 63 / 55, 49 73 / 56, [40,128,3000] 49 39 / 28; dilation 8, [1,512,65536] k = 25 61 / 55, 33 67 / 57,
// 49 90 / 57, [16,128,2095] k = 25 14.7 / 17.4, 33 16.5 / 17.1, 49 21 / 16.5; dilation 32, [1,512,65536] k = 17 61 / 61, 33
// 96 / 74.  Rows of one tile with taps 4, 8 or 16 apart (their scatter table is built for one tile): [64,45,900], dilation 4, k = 5 13.4 / 9.7, dilation
// 16, k = 5 14.1 / 12.6; 16 apart rows that fill a tile are behind where there are few of them and ahead where there are many: [32,64,1000], k = 5
// 9.9 / 10.9, [400,100,1000] 178 / 135.
//
// 33 - 36 adjacent taps on up to 8192 tiles, two to eight in a row, stay on the vector ALU: it spares their many starts (conv1d_thin_kernel /
// here, us, 36 taps; rows x length): 1024 x 2000 6.6 / 8.3, 2048 x 3000 13.0 / 14.4, 819 x 4100 10.5 / 13.5, 877 x 7000 12.5 / 14.7, but 4096 x 1000
// 13.9 / 12.7, 6144 x 2000 26.4 / 24.7, 8192 x 3000 51.4 / 45.0, 10922 x 5200 107 / 105, 1445 x 16384 42.3 / 40.4.
bool conv1d_toep_wanted(int64_t rows, int64_t Lo, int32_t k, int32_t dilation)
{
    const int64_t tiles = (Lo + max_origin_shift(Lo, 16) + kTile - 1) / kTile;
    if (dilation == 1 && k <= 36 && tiles >= 2 && tiles <= 8 && rows * tiles <= 8192) return false;
    return k > 32 || (dilation >= 4 && dilation <= 16 && tiles == 1);
}

hipError_t launch_conv1d_toep(const float *x, const float *wgt, float *y, int64_t B, int64_t Cin, int64_t L, int64_t Cout, int64_t Lo,
                              int32_t k, int32_t pad, int32_t dilation, int32_t groups, hipStream_t s, int wadj)
{
    if (B * Cout >= (1LL << 31)) return kNotTaken;
    ToepGeom g;
    g.B = (int)B; g.L = (int)L; g.Lo = (int)Lo; g.k = k; g.pad = pad; g.Cin = (int)Cin; g.Cout = (int)Cout; g.cog = (int)(Cout / groups);
    g.wflip = wadj;
    switch (dilation) {
    case 1: return launch_taps<0>(x, wgt, y, g, s);
    case 4: return launch_taps<2>(x, wgt, y, g, s);
    case 8: return launch_taps<3>(x, wgt, y, g, s);
    case 16: return launch_taps<4>(x, wgt, y, g, s);
    case 32: return launch_taps<5>(x, wgt, y, g, s);
    default: return kNotTaken;
    }
}

}  // namespace sws
