// The adjoint of a dense convolution with respect to its weights, any kernel of up to 64 taps, strides 1 and 2, any channel
// counts, one or two dimensions, on the bf16 matrix cores with exactly split fp32 operands:
//
//   gw[co][ci][t] = sum over positions p of  gy[n][co][p] * x[n][ci][p * s + t]
//
// is, per tap, a matrix product whose contraction index is the position.  v_mfma_f32_32x32x16_bf16 wants eight
// consecutive contraction indices of one channel per lane, while one staged tile of x should serve every tap, i.e. be read at
// any shift of the position.  Both hold with the tile stored position by position (16-byte units of eight channels of
// one position and bf16 piece) and read with the transposing LDS load ds_read_b64_tr_b16: sixteen lanes point at four
// positions x sixteen channels and receive four positions of one channel each.  The positions of a read are arbitrary
// addresses, so strides, odd shifts and rows that end inside a run cost nothing; no column matrix, no permutes.
//
// A workgroup owns 64 output x 64 input channels x up to nine taps (whole kernel rows, or a run of one) and a run of
// tiles of up to 128 positions: eight wavefronts, 32 x 32 channels x all its taps each, two wavefronts per block that take
// alternate groups of 16 positions.  A tile is rpt whole rows of a strip of TW columns; rows are numbered through all
// images, so small planes fill it.  The next tile's lines of x and gy are loaded into registers before the products of
// the current one and split into LDS after them.  Both operands' pieces are cut, not rounded, so a dropped product may reach
// 2^-22 of its term and the three of them 2^-21 (on average 2^-25).
//
// Sums.  The matrix instruction adds its products in two halves of eight, each cut at 2^-24 of its largest product, and each half to
// the accumulator with one rounding; an accumulator that is small beside the products is cut like one of them.  Six
// products per 16 positions into the run's sum are twelve roundings of its own size, and a sum that starts with the small products
// is cut by the large ones every time (a bias: 6.8e-7 on [32,64,56,56] -> 64, 3 x 3).  So the leading products and the
// other five go to accumulators of their own.  Up to three taps: per tile from zero, added to the run's sum at its end.  Four to eight: per 16 positions
// from zero.  Nine: the leading ones on the run's sum, the others per 16 positions (registers).  Layers whose kernel without a workspace is a
// split-operand one too (FAST, five and nine taps): all six on the run's sum, still more exact than that kernel (but not in conv_gw_staged_kernel).  Error of gw against
// 64 bits, fp32 kernels / all six on the run's sum / now: [1,168,84,84] -> 200, 5 x 5 1.6e-7 / 3.3e-7 / 1.6e-7, [16,500,28,28] -> 500,
// 3 x 3 1.7e-7 / 6.1e-7 / 1.4e-7, [32,61,14,14] -> 32 1.45e-7 / 2.1e-7 / 1.1e-7, [16,24,5574] -> 32, k = 1 3.7e-7 / 6.2e-7 / 1.2e-7.
// Operands of one tap at a time, a piece of the next read as soon as the last product with the present one is out: with two sets the nine-tap
// instance spills, whose reloads wait for the loads in flight ([32,64,56,56] -> 64 93 us, now 75).
//
// Sums leave as partial blocks in the caller's workspace, lane after lane, and gw_reduce_kernel or gw_reduce_few_kernel adds them in a fixed order:
// the result does not depend on the order in which workgroups end (5 - 10 us; the atomic adds of conv_gw_split.hip, 36864 per
// workgroup, take 27 us on 64 x 64 channels, 3 x 3).
//
// Measured, us, this kernel with its second pass / the kernels without a workspace: [17,128,23,14] -> 104, 5 x 5 55 / 313,
// [1,96,65,65] -> 484, 3 x 3 49 / 208, [32,256,14,14] -> 256, 3 x 3 56 / 87, [32,64,56,56] -> 64 53 / 74, [16,64,4096] -> 64, k = 3
// 24 / 31.  Two LDS buffers with tiles of 64 positions, one wavefront of a SIMD splitting while the other multiplies, came out even at nine
// taps and behind at one (174 against 127 us on [19,96,87,87] -> 256): not taken.
#include "sws_internal.h"

#include <type_traits>

namespace sws {

namespace {

typedef short v8s __attribute__((ext_vector_type(8)));

constexpr int kThreads = 512;
constexpr int kMaxTaps = 64, kMaxGroups = 64;
constexpr int kBN = 128;                              // positions per tile
constexpr int kMaxAdds = 64;                          // see plan_gw
constexpr int kPG = 140;                              // positions per staged plane of gy: >= kBN, = 12 mod 16 (see PS below)
constexpr int kOctG = 3 * kPG * 16;                   // bytes from one octet of gy's channels to the next

struct GwTile {
    int N, Cin, H, W, HW, Cout, Ho, Wo, HoWo, NR;     // NR = N * Ho virtual rows of gy
    int KT, ls, LPI, SH, sh, sw;                      // taps; lines per output row, per image, per window; strides
    int CW, LW, TW, nstrips, rpt, tps, tiles;         // columns per residue, positions per line, strip width; rows per tile, tiles per strip
    int PS;                                           // positions per staged plane of x, = 12 mod 16: the octets' planes
                                                      // then start 16 banks apart, and a transposing read of four of them meets each bank twice
    int ksteps, per, nsplit, cob, cib, ng;            // groups of 16 positions per tile; tiles per workgroup, runs; channel blocks, tap groups
    int lines, nq, group, rows;                             // conv_gw_staged_kernel: lines of x per tile, groups of four columns of a line, rows of a group, of a run (0: not its)
    float inv_TW, inv_Ho, inv_LPI, inv_LW, inv_CW, inv_PS, inv_nq, inv_lines;
    short gdh[kMaxGroups], gdw[kMaxGroups];           // tap group: row and column of its first tap, relative to the position
    unsigned char gt0[kMaxGroups], gnt[kMaxGroups];   // first tap, taps
    unsigned short tapoff[kMaxTaps];                  // tap -> staged positions from a position's base
};

// a 16-byte unit: eight channels' values, split into three pieces, to dst, dst + step, dst + 2 step
__device__ __forceinline__ void put_unit(char *dst, int step, const float (&v)[8])
{
    unsigned p[3][4];
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
        float r1[2], r2[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            r1[u] = v[e + u] - __uint_as_float(__float_as_uint(v[e + u]) & 0xffff0000u);
            r2[u] = r1[u] - __uint_as_float(__float_as_uint(r1[u]) & 0xffff0000u);
        }
        p[0][e / 2] = pack_hi(v[e], v[e + 1]);
        p[1][e / 2] = pack_hi(r1[0], r1[1]);
        p[2][e / 2] = pack_hi(r2[0], r2[1]);
    }
#pragma unroll
    for (int q = 0; q < 3; ++q) *(v4u *)(dst + q * step) = (v4u){p[q][0], p[q][1], p[q][2], p[q][3]};
}

// TB: taps per group at most (a shorter last group computes its last tap again); WM x WN blocks of 32 x 32 channels, WK
// wavefronts each; UX: staged units of x per thread (gy has WM).  The places of a thread's units are worked out anew for every
// tile (opaque): kept in registers they push the accumulators into scratch memory, whose reloads would wait for the loads in flight.
template <int TB, int WM, int WN, int UX, bool FAST>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2)))
void conv_gw_tile_kernel(const float *__restrict__ x, const float *__restrict__ gy, float *__restrict__ ws, GwTile g)
{
    fetch_arguments<24 + sizeof(GwTile)>();
    constexpr int WK = 8 / (WM * WN), OG = 4 * WM, OX = 4 * WN;      // octets of channels
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char *const G = lds, *const X = lds + OG * kOctG;
    const int pieceX = g.PS * 16, octX = 3 * pieceX;
    int *const tab = (int *)(X + OX * octX);          // position -> byte offset of its base in a plane of x
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM % WN, wk = wave / (WM * WN);

    const int Gx = (int)gridDim.x;                    // a multiple of 8: each XCD takes a contiguous run
    const int id = (int)(blockIdx.x & 7) * (Gx >> 3) + (int)(blockIdx.x >> 3);
    const int nblk = g.cob * g.cib * g.ng;
    if (id >= g.nsplit * nblk) return;
    const int split = id / nblk, blk = id - split * nblk;
    const int grp = blk % g.ng, cb = blk / g.ng, cob = cb / g.cib, cib = cb - cob * g.cib;
    const int nt = g.gnt[grp], t0 = g.gt0[grp], dh = g.gdh[grp], dw = g.gdw[grp];
    const int co0 = cob * (32 * WM), ci0 = cib * (32 * WN);
    const int first = split * g.per, end = first + g.per < g.tiles ? first + g.per : g.tiles;

    // ---- staged units.  gy: octet of channels, position; x: octet, line and column of the tile
    const int gmax = g.Cout > 8 ? g.Cout - 8 : 0, xmax = g.Cin > 8 ? g.Cin - 8 : 0;
    const int units = OX * g.PS;
    float gr[WM][8], xr[UX][8];
    int tabv = 0;
    auto issue = [&](int tile) {
        const int strip = tile / g.tps, R0 = (tile - strip * g.tps) * g.rpt, cb0 = strip * g.TW;
        const int n0 = R0 / g.Ho, oh0 = R0 - n0 * g.Ho;
        const int64_t xl_ = 4 * (int64_t)(g.N - n0) * g.Cin * g.HW, gl_ = 4 * (int64_t)(g.N - n0) * g.Cout * g.HoWo;
        const __amdgpu_buffer_rsrc_t xs = rsrc(x + (int64_t)n0 * g.Cin * g.HW, xl_ < 0x7fffffff ? (unsigned)xl_ : 0x7fffffffu);
        const __amdgpu_buffer_rsrc_t gs = rsrc(gy + (int64_t)n0 * g.Cout * g.HoWo, gl_ < 0x7fffffff ? (unsigned)gl_ : 0x7fffffffu);
        int me = tid;
        asm volatile("" : "+v"(me));
        {
            const int R = fdiv(me & 127, g.inv_TW), c = (me & 127) - R * g.TW;
            const int t = oh0 + R, dn = fdiv(t, g.inv_Ho), oh = t - dn * g.Ho;
            const bool in = R < g.rpt, ok = in && R0 + R < g.NR && cb0 + c < g.Wo;
            tabv = in ? ((dn * g.LPI + (oh - oh0) * g.ls) * g.LW + c) * 16 : 0;
#pragma unroll
            for (int i = 0; i < WM; ++i) {
                const int ch = co0 + 8 * ((me >> 7) + 4 * i), cc = ch < gmax ? ch : gmax;
                const unsigned at = ok && ch < g.Cout ? 4u * (unsigned)((dn * g.Cout + cc) * g.HoWo + oh * g.Wo + cb0 + c) : kNowhere;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int se = e < g.Cout ? e : g.Cout - 1;
                    gr[i][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(gs, at, 4 * se * g.HoWo, 0));
                }
            }
        }
#pragma unroll
        for (int i = 0; i < UX; ++i) {
            if (i * kThreads >= units) continue;
            const int u = me + i * kThreads, oct = fdiv(u, g.inv_PS), pos = u - oct * g.PS;
            const int ln = fdiv(pos, g.inv_LW), c0 = pos - ln * g.LW, cph = fdiv(c0, g.inv_CW);
            const int col = (cb0 + c0 - cph * g.CW) * g.sw + cph + dw;
            const int l = oh0 * g.ls + ln, dn = fdiv(l, g.inv_LPI), r = l - dn * g.LPI;
            const int row = (g.SH >= g.sh ? r : r * g.sh) + dh;
            const int ch = ci0 + oct * 8, cc = ch < xmax ? ch : xmax;
            const bool ok = oct < OX && ch < g.Cin && n0 + dn < g.N && (unsigned)row < (unsigned)g.H && (unsigned)col < (unsigned)g.W;
            const unsigned at = ok ? 4u * (unsigned)((dn * g.Cin + cc) * g.HW + row * g.W + col) : kNowhere;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int se = e < g.Cin ? e : g.Cin - 1;
                xr[i][e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(xs, at, 4 * se * g.HW, 0));
            }
        }
    };
    auto commit = [&]() {
        int me = tid;
        asm volatile("" : "+v"(me));
#pragma unroll
        for (int i = 0; i < WM; ++i) put_unit(G + ((me >> 7) + 4 * i) * kOctG + (me & 127) * 16, kPG * 16, gr[i]);
#pragma unroll
        for (int i = 0; i < UX; ++i) {
            if (i * kThreads >= units) continue;
            const int u = me + i * kThreads, oct = fdiv(u, g.inv_PS), pos = u - oct * g.PS;
            if (oct < OX) put_unit(X + oct * octX + pos * 16, pieceX, xr[i]);
        }
        if (me < kBN) tab[me] = tabv;
    };
    auto barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    // ---- operand reads: lane 16 b + m points at octet 2 (b & 1) + (m & 3) / 2, half (m & 1), position 8 (b >> 1) + m / 4
    const int b = lane >> 4, m = lane & 15;
    const int oct = 2 * (b & 1) + ((m & 3) >> 1), pj = 8 * (b >> 1) + (m >> 2);
    const char *const Ga = G + (4 * wm + oct) * kOctG + (m & 1) * 8 + pj * 16;
    const char *const Xa = X + (4 * wn + oct) * octX + (m & 1) * 8;
    unsigned off2[(TB + 1) / 2];                      // two taps' offsets (below 2^14 bytes) per scalar register
#pragma unroll
    for (int j = 0; j < TB; j += 2) {
        const unsigned a = g.tapoff[t0 + (j < nt ? j : nt - 1)], b = g.tapoff[t0 + (j + 1 < nt ? j + 1 : nt - 1)];
        off2[j / 2] = __builtin_amdgcn_readfirstlane((a | b << 16) << 4);
    }
    constexpr bool TILE_SUM = TB <= 3, ON_RUN = TB == 9 || FAST;
    v16f acc[TB];
#pragma unroll
    for (int t = 0; t < TB; ++t) acc[t] = (v16f){0.0f};

    if (first < end) issue(first);
    for (int tile = first; tile < end; ++tile) {
        commit();
        barrier();
        if (tile + 1 < end) issue(tile + 1);
        v16f hi[TILE_SUM ? TB : 1], lo[TILE_SUM ? TB : 1];
        if constexpr (TILE_SUM) {
#pragma unroll
            for (int t = 0; t < TB; ++t) hi[t] = lo[t] = (v16f){0.0f};
        }
        for (int s = wk; s < g.ksteps; s += WK) {
            const int p0 = tab[16 * s + pj], p1 = tab[16 * s + pj + 4];
            v8bf a[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) a[q] = tr8(Ga + s * 256 + q * (kPG * 16), Ga + s * 256 + 64 + q * (kPG * 16));
            auto xread = [&](int t, int q) {
                const int off = (int)(t & 1 ? off2[t / 2] >> 16 : off2[t / 2] & 0xffff) + q * pieceX;
                return tr8(Xa + p0 + off, Xa + p1 + off);
            };
            v8bf b2 = xread(0, 2), b1 = xread(0, 1), b0 = xread(0, 0);
#pragma unroll
            for (int t = 0; t < TB; ++t) {
                // (a piece of the next tap is read as soon as this tap's last product of it is out: twelve registers less
                // than with two sets)
                v16f l = {0.0f};
                if constexpr (TILE_SUM) l = lo[t];
                else if constexpr (FAST) l = acc[t];
                __builtin_amdgcn_sched_barrier(0);
                l = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b2, l, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (t + 1 < TB) b2 = xread(t + 1, 2);
                __builtin_amdgcn_sched_barrier(0);
                l = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b1, l, 0, 0, 0);
                l = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b1, l, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (t + 1 < TB) b1 = xread(t + 1, 1);
                __builtin_amdgcn_sched_barrier(0);
                l = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], b0, l, 0, 0, 0);
                l = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b0, l, 0, 0, 0);
                v16f h = {0.0f};
                if constexpr (TILE_SUM) h = hi[t];
                else if constexpr (FAST) h = l;
                else if constexpr (ON_RUN) h = acc[t];
                h = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b0, h, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (t + 1 < TB) b0 = xread(t + 1, 0);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (TILE_SUM) {
                    lo[t] = l;
                    hi[t] = h;
                } else if constexpr (FAST) {
                    acc[t] = h;
                } else if constexpr (ON_RUN) {
                    acc[t] = h + l;
                } else {
                    acc[t] += h + l;
                }
            }
        }
        if constexpr (TILE_SUM) {
#pragma unroll
            for (int t = 0; t < TB; ++t) acc[t] += hi[t] + lo[t];
        }
        barrier();                                    // everybody has read the tile
    }

    // ---- the wavefronts of a block add up through LDS, three taps at a time; then to the workspace:
    //      ws[split][block][tap][wm, wn][register / 4][lane][register % 4]
    constexpr int BLK = WM * WN, ROWS = TB < 3 ? TB : 3;
    v4f *const out = (v4f *)ws + ((int64_t)split * nblk + blk) * (TB * BLK * 256) + (wave % BLK) * 256 + lane;
    v4f *const red = (v4f *)lds + lane;
#pragma unroll
    for (int q = 0; q < TB; q += 3) {
        if (wk > 0) {
#pragma unroll
            for (int t = q; t < q + 3 && t < TB; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    red[((wave - BLK) * (4 * ROWS) + (t - q) * 4 + v) * 64] =
                        (v4f){acc[t][4 * v], acc[t][4 * v + 1], acc[t][4 * v + 2], acc[t][4 * v + 3]};
        }
        barrier();
        if (wk == 0) {
#pragma unroll
            for (int t = q; t < q + 3 && t < TB; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    v4f r = {acc[t][4 * v], acc[t][4 * v + 1], acc[t][4 * v + 2], acc[t][4 * v + 3]};
                    for (int k = 0; k < WK - 1; ++k) r += red[((k * BLK + wave) * (4 * ROWS) + (t - q) * 4 + v) * 64];
                    if (t < nt) out[t * (BLK * 256) + v * 64] = r;
                }
        }
        barrier();
    }
}

// The same for 3 x 3 at stride 1 (nine taps, 32 WM x 32 channels, whole blocks) with wavefronts that only stage: four of them (one per SIMD) load,
// split and write tiles, eight multiply.  A multiplying wavefront holds one block of 32 x 32 channels, five or four of the taps (two wavefronts of a SIMD:
// one of each) and every WK-th group of 16 positions: 80 accumulators instead of 144, so that three wavefronts per SIMD find registers.  x has two
// buffers; gy has one, which is free as soon as everybody has read its last group's operand, and is written while that group is multiplied.
//   What bounds the kernel above is that all its wavefronts stage at once (4.5 k cycles of a tile's 14 k in addresses and loads, 3 k in splitting and writing, 6.9 k
// of products) while none multiplies.  One-dword loads alone would keep the staging wavefronts longer than the products take: a load occupies the address unit
// for 16 cycles whatever its width.  So a thread stages eight channels of four consecutive columns (x) or two consecutive positions (gy) by eight 16- or 8-byte loads.
//   Runs are rows, not whole tiles, so that the runs of a round end together (seven tiles where 6.2 are due, before), and go through the strips of a group of
// images before the next one: strips share cache lines, and runs side by side an XCD's cache (without it [32,64,56,56] -> 64 165 us for a
// training step, with it 156).
//   Second pass included, us, kernel above / here: [32,256,14,14] -> 256 65.0 / 56.4, [32,64,56,56] -> 64 65.6 / 52.6, [32,128,28,28] -> 128 60.6 / 51.3,
// [64,160,12,12] -> 160 50.0 / 41.4, [4,256,56,56] -> 128 64.5 / 54.0.  The bound is now the products, 2.1 k cycles per 16 positions and SIMD of which 1.7 k are theirs,
// and what a run has besides: its first tile's staging and the sums at its end, a fifth of these layers.
// Sums: the leading products on the run's sum, the other five per 16 positions from zero (as the kernel above without FAST): error of
// gw against 64 bits on the two layers of 56 x 56 and 14 x 14 3.4e-7 and 2.4e-7 above, 1.9e-7 here.
template <int WM>
__global__ __launch_bounds__(768) __attribute__((amdgpu_waves_per_eu(3)))
void conv_gw_staged_kernel(const float *__restrict__ x, const float *__restrict__ gy, float *__restrict__ ws, GwTile g)
{
    fetch_arguments<24 + sizeof(GwTile)>();
    constexpr int WK = 4 / WM, OG = 4 * WM, OX = 4, T = 256, TB = 9, TW = 5;      // octets of channels; staging threads; TW: taps of a wavefront
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int pieceX = g.PS * 16, octX = 3 * pieceX, bufX = OX * octX;
    char *const G = lds, *const X = lds + OG * kOctG;
    int *const tab = (int *)(X + 2 * bufX);           // position -> byte offset of its base in a plane of x; two of them
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wm = wave % WM, wk = wave / WM % WK, th = wave >> 2;

    const int Gx = (int)gridDim.x;                    // a multiple of 8: each XCD takes a contiguous run
    const int id = (int)(blockIdx.x & 7) * (Gx >> 3) + (int)(blockIdx.x >> 3);
    const int nblk = g.cob * g.cib * g.ng;
    if (id >= g.nsplit * nblk) return;
    const int split = id / nblk, blk = id - split * nblk;
    const int grp = blk % g.ng, cb = blk / g.ng, cob = cb / g.cib, cib = cb - cob * g.cib;
    const int nt = g.gnt[grp], t0 = g.gt0[grp], dh = g.gdh[grp], dw = g.gdw[grp];
    const int co0 = cob * (32 * WM), ci0 = cib * 32;
    // A run is g.rows rows in the order (group of whole images, strip, row); its tiles have rpt of them, the last one of a run and of a group what is left.
    struct Place { int at, R, gs, ge, strip; };       // rows before it; its row; first row and last + 1 of its group; its strip
    const int begin = split * g.rows, all = g.nstrips * g.NR, end = begin + g.rows < all ? begin + g.rows : all;
    Place now;
    {
        const int full = g.nstrips * g.group, grp0 = begin / full, gs = grp0 * g.group, ge = gs + g.group < g.NR ? gs + g.group : g.NR;
        const int rest = begin - grp0 * full, strip = rest / (ge - gs);
        now = {begin, gs + rest - strip * (ge - gs), gs, ge, strip};
    }
    auto rows_of = [&](const Place &p) {
        const int r = end - p.at < g.rpt ? end - p.at : g.rpt;
        return r < p.ge - p.R ? r : p.ge - p.R;
    };
    auto after_of = [&](Place p) {
        const int rows = rows_of(p);
        p.at += rows;
        p.R += rows;
        if (p.R == p.ge) {
            p.R = p.gs;
            if (++p.strip == g.nstrips) {
                p.R = p.gs = p.ge;
                p.ge = p.ge + g.group < g.NR ? p.ge + g.group : g.NR;
                p.strip = 0;
            }
        }
        return p;
    };
    auto barrier = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };

    if (wave >= 8) {
        const int tid = (int)threadIdx.x - 512;
        struct Tile { int n0, oh0, cb0, rows; };      // its first row's image and row there, first column, rows
        auto tile_of = [&](const Place &p) {
            const int n0 = p.R / g.Ho;
            return Tile{n0, p.R - n0 * g.Ho, p.strip * g.TW, rows_of(p)};
        };
        struct Cols { int clo, lo, hi; };             // first staged column of x; first and last + 1 that exist
        auto cols = [&](const Tile &t) {
            Cols c;
            c.clo = t.cb0 + dw;
            c.lo = c.clo > 0 ? c.clo : 0;
            c.hi = c.clo + g.LW < g.W ? c.clo + g.LW : g.W;
            if (c.hi <= c.lo) c.lo = c.hi = c.clo;    // (all of them padding)
            return c;
        };
        // my unit of x: four columns of a line; of gy: pairs of positions 2 (tid % 64), octets tid / 64 and four further
        const int xrow = fdiv(tid, g.inv_nq), q4 = 4 * (tid - xrow * g.nq), xoct = fdiv(xrow, g.inv_lines), ln = xrow - xoct * g.lines;
        const int xat = (ci0 + 8 * xoct) * g.HW + q4, xdst = xoct * octX + (ln * g.LW + q4) * 16;
        const int gpos = 2 * (tid & 63), goct = tid >> 6, gR = fdiv(gpos, g.inv_TW), gc = gpos - gR * g.TW;
        v4f xr[8];
        v2f gr[WM][8];
        auto issue_x = [&](const Tile &t) {
            const int64_t xl_ = 4 * (int64_t)(g.N - t.n0) * g.Cin * g.HW;
            const __amdgpu_buffer_rsrc_t xs = rsrc(x + (int64_t)t.n0 * g.Cin * g.HW, xl_ < 0x7fffffff ? (unsigned)xl_ : 0x7fffffffu);
            const Cols k = cols(t);
            const int l = t.oh0 + ln, dn = fdiv(l, g.inv_LPI), row = l - dn * g.LPI + dh;
            const bool ok = xoct < OX && t.n0 + dn < g.N && (unsigned)row < (unsigned)g.H;
            const unsigned at = ok ? 4u * (unsigned)(dn * g.Cin * g.HW + row * g.W + k.lo + xat) : kNowhere;
#pragma unroll
            for (int e = 0; e < 8; ++e) xr[e] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(xs, at, 4 * e * g.HW, 0));
        };
        auto issue_g = [&](const Tile &t) {
            const int64_t gl_ = 4 * (int64_t)(g.N - t.n0) * g.Cout * g.HoWo;
            const __amdgpu_buffer_rsrc_t gs = rsrc(gy + (int64_t)t.n0 * g.Cout * g.HoWo, gl_ < 0x7fffffff ? (unsigned)gl_ : 0x7fffffffu);
            const int r = t.oh0 + gR, dn = fdiv(r, g.inv_Ho), oh = r - dn * g.Ho;
            const bool ok = gR < t.rows && t.cb0 + gc < g.Wo;      // (even columns of rows of even length: both positions or none)
#pragma unroll
            for (int i = 0; i < WM; ++i) {
                const unsigned at = ok ? 4u * (unsigned)((dn * g.Cout + co0 + 8 * (goct + 4 * i)) * g.HoWo + oh * g.Wo + t.cb0 + gc) : kNowhere;
#pragma unroll
                for (int e = 0; e < 8; ++e) gr[i][e] = __builtin_bit_cast(v2f, __builtin_amdgcn_raw_buffer_load_b64(gs, at, 4 * e * g.HoWo, 0));
            }
        };
        // (the columns that a row lacks on either side are zeros)
        auto commit_x = [&](const Tile &t, char *Xb) {
            const Cols k = cols(t);
            const int left = xoct < OX ? k.hi - k.lo - q4 : 0, front = k.lo - k.clo;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float v[8] = {xr[0][c], xr[1][c], xr[2][c], xr[3][c], xr[4][c], xr[5][c], xr[6][c], xr[7][c]};
                if (c < left) put_unit(Xb + xdst + (front + c) * 16, pieceX, v);
            }
            const int pads = g.LW - (k.hi - k.lo);
            if (pads > 0) {
                const float inv = 1.0f / (float)pads;
                for (int u = tid; u < pads * OX * g.lines; u += T) {
                    const int r = fdiv(u, inv), j = u - r * pads, o = fdiv(r, g.inv_lines);
                    char *const d = Xb + o * octX + ((r - o * g.lines) * g.LW + (j < front ? j : j + k.hi - k.lo)) * 16;
#pragma unroll
                    for (int p = 0; p < 3; ++p) *(v4u *)(d + p * pieceX) = (v4u){0, 0, 0, 0};
                }
            }
        };
        auto commit_g = [&](const Tile &t, int *tb) {
            if (tid < kBN) {
                const int R = fdiv(tid, g.inv_TW), c = tid - R * g.TW, r = t.oh0 + R, dn = fdiv(r, g.inv_Ho), oh = r - dn * g.Ho;
                tb[tid] = R < g.rpt ? ((dn * g.LPI + oh - t.oh0) * g.LW + c) * 16 : 0;
            }
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const float v[8] = {gr[i][0][c], gr[i][1][c], gr[i][2][c], gr[i][3][c], gr[i][4][c], gr[i][5][c], gr[i][6][c], gr[i][7][c]};
                    put_unit(G + (goct + 4 * i) * kOctG + (gpos + c) * 16, kPG * 16, v);
                }
        };
        // Between two tiles stands only the splitting of gy; its loads go out behind the barrier, those of x a tile further ahead
        Tile tile = tile_of(now);
        issue_x(tile);
        issue_g(tile);
        commit_x(tile, X);
        commit_g(tile, tab);
        Place next = after_of(now);
        if (next.at < end) issue_x(tile = tile_of(next));
        barrier();                                    // the first tile is there
        int cur = 0;
        for (bool more = next.at < end;; ) {
            cur ^= 1;
            Tile ahead = tile;
            if (more) {
                issue_g(tile);
                commit_x(tile, X + cur * bufX);
                next = after_of(next);
                if (next.at < end) issue_x(ahead = tile_of(next));
            }
            barrier();                                // the tile's operands of gy have been read
            if (!more) break;
            commit_g(tile, tab + cur * kBN);
            barrier();                                // the next tile is there, this one has been multiplied
            tile = ahead;
            more = next.at < end;
        }
        barrier();
        barrier();
        return;
    }

    // ---- operand reads: lane 16 b + m points at octet 2 (b & 1) + (m & 3) / 2, half (m & 1), position 8 (b >> 1) + m / 4
    const int b = lane >> 4, m = lane & 15;
    const int oct = 2 * (b & 1) + ((m & 3) >> 1), pj = 8 * (b >> 1) + (m >> 2);
    const char *const Ga = G + (4 * wm + oct) * kOctG + (m & 1) * 8 + pj * 16;
    const char *const Xa = X + oct * octX + (m & 1) * 8;
    int off[TW];                                      // my taps' offsets (the fifth of the second wavefront: its fourth again, not stored)
#pragma unroll
    for (int j = 0; j < TW; ++j) {
        const int t = TW * th + j, tt = t < nt && t < TB ? t : nt - 1;
        off[j] = __builtin_amdgcn_readfirstlane((int)g.tapoff[t0 + tt]) * 16;
    }
    v16f acc[TW];
#pragma unroll
    for (int t = 0; t < TW; ++t) acc[t] = (v16f){0.0f};

    auto run = [&](auto mine) {
        constexpr int NT = mine.value;                // taps
        barrier();                                    // the first tile is there
        int cur = 0;
        Place p = now;
        while (p.at < end) {
            const int ksteps = (rows_of(p) * g.TW + 15) >> 4;
            p = after_of(p);
            const char *const Xc = Xa + cur * bufX;
            const int *const tc = tab + cur * kBN;
            auto xread = [&](int p0, int p1, int t, int q) { return tr8(Xc + p0 + off[t] + q * pieceX, Xc + p1 + off[t] + q * pieceX); };
            auto gread = [&](v8bf (&a)[3], int s) {
#pragma unroll
                for (int q = 0; q < 3; ++q) a[q] = tr8(Ga + s * 256 + q * (kPG * 16), Ga + s * 256 + 64 + q * (kPG * 16));
            };
            v8bf a[3], an[3], b2, b1, b0;
            int p0 = 0, p1 = 0;
            if (wk < ksteps) {
                gread(an, wk);
                p0 = tc[16 * wk + pj];
                p1 = tc[16 * wk + pj + 4];
                b2 = xread(p0, p1, 0, 2);
                b1 = xread(p0, p1, 0, 1);
                b0 = xread(p0, p1, 0, 0);
            } else {
                barrier();
            }
            for (int s = wk; s < ksteps; s += WK) { // sixteen positions
                const bool last = s + WK >= ksteps;
                const int c0 = p0, c1 = p1, sn = last ? s : s + WK;
#pragma unroll
                for (int q = 0; q < 3; ++q) a[q] = an[q];
                if (last) barrier();                  // everybody has its last operands of gy
                else gread(an, sn);
                p0 = tc[16 * sn + pj];
                p1 = tc[16 * sn + pj + 4];
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    // (a piece of the next tap is read as soon as this tap's last product of it is out)
                    const int n0 = t + 1 < NT ? c0 : p0, n1 = t + 1 < NT ? c1 : p1, tn = t + 1 < NT ? t + 1 : 0;
                    v16f l = {0.0f};
                    __builtin_amdgcn_sched_barrier(0);
                    l = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b2, l, 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    b2 = xread(n0, n1, tn, 2);
                    __builtin_amdgcn_sched_barrier(0);
                    l = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b1, l, 0, 0, 0);
                    l = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b1, l, 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    b1 = xread(n0, n1, tn, 1);
                    __builtin_amdgcn_sched_barrier(0);
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], b0, acc[t], 0, 0, 0);
                    l = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], b0, l, 0, 0, 0);
                    l = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], b0, l, 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    b0 = xread(n0, n1, tn, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    acc[t] += l;
                }
            }
            cur ^= 1;
            if (p.at < end) barrier();           // the next tile is there, this one has been multiplied
        }
    };
    if (th == 0) run(std::integral_constant<int, TW>{});
    else run(std::integral_constant<int, TB - TW>{});

    // ---- the WK wavefronts of a block's taps add up through LDS, 4 / WK of four groups of registers each; then to the workspace, as above
    v4f *const red = (v4f *)lds + lane;
    barrier();
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (v % WK != wk) red[(wave * (4 * TW) + t * 4 + v) * 64] = (v4f){acc[t][4 * v], acc[t][4 * v + 1], acc[t][4 * v + 2], acc[t][4 * v + 3]};
    barrier();
    v4f *const out = (v4f *)ws + ((int64_t)split * nblk + blk) * (TB * WM * 256) + wm * 256 + lane;
#pragma unroll
    for (int t = 0; t < TW; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (v % WK != wk) continue;
            v4f r = {acc[t][4 * v], acc[t][4 * v + 1], acc[t][4 * v + 2], acc[t][4 * v + 3]};
#pragma unroll
            for (int k = 1; k < WK; ++k) {
                const int other = 4 * th + wm + WM * ((wk + k) % WK);
                r += red[(other * (4 * TW) + t * 4 + v) * 64];
            }
            const int tt = TW * th + t;
            if (tt < nt && (th == 0 || t < TB - TW)) out[tt * (WM * 256) + v * 64] = r;
        }
}

// The channel that a slot of a block holds; -1: none, or one that another slot holds (an octet of channels that reached beyond the last
// one held the last eight, see the staging).
__device__ __forceinline__ int slot_channel(int slot, int n)
{
    const int o = slot & ~7, c0 = o < n - 8 ? o : (n > 8 ? n - 8 : 0), c = c0 + (slot & 7);
    return o < n && c >= o && c < n ? c : -1;
}

// gw from the partial blocks: a workgroup adds 64 elements of one (block, tap, wavefront), its four wavefronts
// every fourth run; element 256 q + 4 (32 half + l32) + r of a block of 32 x 32 is output channel 8 q + 4 half + r, input channel l32.
// DEEP: sixteen runs in flight a wavefront.  A second pass of few workgroups or of little to add waits for memory and back; a larger one is bound by bytes, and
// four runs in flight with nothing in front of them get more of those.  (wave: not made uniform.  With a scalar loop the last runs wait for the others:
// 128 x 416 channels, 9 taps, 18 runs 12.6 us / 16.3, and DEEP 14.7.)  us, four in flight / DEEP, both measured: 64 x 64, 3 taps, 256 runs 6.8 / 4.9, 24 x 18, 3 taps 6.8 / 4.5;
// 192 x 57, 9 taps, 80 runs 7.4 / 8.2, 320 x 288, 3 taps, 9 runs 8.2 / 8.9, 241 x 352, 9 taps, 9 runs 18.7 / 21.5.  Two elements a lane and eight wavefronts:
// 6.2 on the first.
template <bool DEEP>
__global__ __launch_bounds__(256) void gw_reduce_kernel(const float *__restrict__ ws, float *__restrict__ gw, GwTile g, int TB, int WM, int WN)
{
    if constexpr (DEEP) fetch_arguments<28 + sizeof(GwTile)>();
    __shared__ float part[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nblk = g.cob * g.cib * g.ng, BLK = WM * WN;
    const int v = blockIdx.x & 15, rest = (int)(blockIdx.x >> 4), w = rest % BLK, t = rest / BLK % TB, blk = rest / (BLK * TB);
    const int grp = blk % g.ng, cb = blk / g.ng, cob = cb / g.cib, cib = cb - cob * g.cib;
    if (t >= g.gnt[grp]) return;
    const int64_t step = (int64_t)nblk * (TB * BLK * 1024);
    const float *p = ws + (int64_t)blk * (TB * BLK * 1024) + t * (BLK * 1024) + w * 1024 + v * 64 + lane;
    constexpr int M = DEEP ? 16 : 4;
    float s[M];
#pragma unroll
    for (int u = 0; u < M; ++u) s[u] = 0.0f;
    int k = wave;
    auto batch = [&](auto many) {
        constexpr int n = many.value;
#pragma unroll
        for (int u = 0; u < n; ++u) s[u] += p[(k + 4 * u) * step];
        k += 4 * n;
    };
    if constexpr (DEEP) {
        while (k + 60 < g.nsplit) batch(std::integral_constant<int, 16>{});
        if (k + 28 < g.nsplit) batch(std::integral_constant<int, 8>{});
        if (k + 12 < g.nsplit) batch(std::integral_constant<int, 4>{});
        if (k < g.nsplit) {
            float f[3];
#pragma unroll
            for (int u = 0; u < 3; ++u) f[u] = p[(k + 4 * u < g.nsplit ? k + 4 * u : k) * step];
#pragma unroll
            for (int u = 0; u < 3; ++u) s[u] += k + 4 * u < g.nsplit ? f[u] : 0.0f;       // (beyond the last run: not counted)
        }
#pragma unroll
        for (int u = 4; u < M; ++u) s[u & 3] += s[u];
    } else {
        while (k + 12 < g.nsplit) batch(std::integral_constant<int, 4>{});
        for (; k < g.nsplit; k += 4) s[0] += p[k * step];
    }
    part[wave][lane] = (s[0] + s[1]) + (s[2] + s[3]);
    __syncthreads();
    if (wave != 0) return;
    const float sum = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
    const int from = 16 * (v & 3) + (lane >> 2);      // the lane that summed it
    const int co = slot_channel(cob * (32 * WM) + w % WM * 32 + 8 * (v >> 2) + 4 * (from >> 5) + (lane & 3), g.Cout);
    const int ci = slot_channel(cib * (32 * WN) + w / WM * 32 + (from & 31), g.Cin);
    if (co >= 0 && ci >= 0) gw[((int64_t)co * g.Cin + ci) * g.KT + g.gt0[grp] + t] = sum;
}

// The same where few runs are to be added, at most kFewRuns: a workgroup takes a quarter (registers 4 q .. 4 q + 3, eight output channels x 32 input
// channels) of one (block, wavefront) and all its taps, a wavefront each, so that what it stores is contiguous; 128-bit loads, all of a
// wavefront's in flight at once, which is what limits the runs.  A tap and 64 elements per workgroup, as above, leave a channel's taps to as many workgroups
// of different XCDs.  Durations, us, gw_reduce_kernel<false> / here: 256 x 256 channels, 3 x 3, 8 runs 13.0 / 6.6, 3 runs 12.3 / 5.3; 512 x 480, 2 runs, 1 x 1 6.5 / 4.9 (512 x 512),
// 1 x 3 15.7 / 5.8, 2 x 2 19.8 / 6.9, 1 x 5 24.2 / 7.3, 3 x 3, 4 runs 40.8 / 13.8; one block of one run 2.9 / 4.1.
constexpr int kFewRuns = 8;
__global__ __launch_bounds__(576) void gw_reduce_few_kernel(const float *__restrict__ ws, float *__restrict__ gw, GwTile g, int TB, int WM, int WN)
{
    fetch_arguments<28 + sizeof(GwTile)>();
    __shared__ v4f part[9][64];
    const int lane = threadIdx.x & 63, t = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int BLK = WM * WN;
    const unsigned rest = blockIdx.x >> 2, blk = rest / (unsigned)BLK, cb = blk / (unsigned)g.ng;
    const int qr = blockIdx.x & 3, w = (int)(rest - blk * BLK), grp = (int)(blk - cb * g.ng);
    const int cob = (int)(cb / (unsigned)g.cib), cib = (int)cb - cob * g.cib;
    const int nt = g.gnt[grp];
    if (t < nt) {
        const int64_t step = (int64_t)g.cob * g.cib * g.ng * (TB * BLK * 256);
        const v4f *p = (const v4f *)ws + ((int64_t)blk * TB + t) * (BLK * 256) + w * 256 + qr * 64 + lane;
        v4f f[kFewRuns];
#pragma unroll
        for (int u = 0; u < kFewRuns; ++u) f[u] = p[(u < g.nsplit ? u : 0) * step];
#pragma unroll
        for (int u = 1; u < kFewRuns; ++u) f[u] = u < g.nsplit ? f[u] : (v4f){0.0f, 0.0f, 0.0f, 0.0f};       // (beyond the last run: not counted)
        part[t][lane] = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
    }
    __syncthreads();
    // (consecutive threads: consecutive taps of an input channel, then the next one, then the next output channel)
    const float inv_nt = 1.0f / (float)nt;
    for (int i = threadIdx.x; i < 256 * nt; i += 64 * TB) {
        const int e = fdiv(i, inv_nt), tt = i - e * nt, c8 = e >> 5, l32 = e & 31;
        const float sum = ((const float *)part[tt])[((c8 >> 2) * 32 + l32) * 4 + (c8 & 3)];
        const int co = slot_channel(cob * (32 * WM) + w % WM * 32 + 8 * qr + c8, g.Cout);
        const int ci = slot_channel(cib * (32 * WN) + w / WM * 32 + l32, g.Cin);
        if (co >= 0 && ci >= 0) gw[((int64_t)co * g.Cin + ci) * g.KT + g.gt0[grp] + tt] = sum;
    }
}

template <int WM>
hipError_t launch_staged(const float *x, const float *gy, float *ws, const GwTile &g, size_t lds, hipStream_t s)
{
    if (lds > 64 * 1024) {
        static std::atomic<uint64_t> raised{0};
        const hipError_t e = raise_lds((const void *)conv_gw_staged_kernel<WM>, 160 * 1024, raised);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(conv_gw_staged_kernel<WM>, dim3((unsigned)xcd_grid((int64_t)g.nsplit * g.cob * g.cib * g.ng)), dim3(768), lds, s, x, gy, ws, g);
    return hipGetLastError();
}

template <int TB, int WM, int WN, bool FAST, int UX>
hipError_t launch_all(const float *x, const float *gy, float *ws, const GwTile &g, size_t lds, hipStream_t s)
{
    if (lds > 64 * 1024) {
        static std::atomic<uint64_t> raised{0};
        const hipError_t e = raise_lds((const void *)conv_gw_tile_kernel<TB, WM, WN, UX, FAST>, 160 * 1024, raised);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((conv_gw_tile_kernel<TB, WM, WN, UX, FAST>), dim3((unsigned)xcd_grid((int64_t)g.nsplit * g.cob * g.cib * g.ng)), dim3(kThreads), lds,
                       s, x, gy, ws, g);
    return hipGetLastError();
}

template <int TB, int WM, int WN, bool FAST, int UX = 4>
hipError_t launch_gw1(const float *x, const float *gy, float *gw, float *ws, const GwTile &g, size_t lds, hipStream_t s)
{
    const int nblk = g.cob * g.cib * g.ng;
    hipError_t e;
    if constexpr (TB == 9 && WN == 1 && UX == 4 && FAST)
        e = g.rows ? launch_staged<WM>(x, gy, ws, g, lds, s) : launch_all<TB, WM, WN, FAST, UX>(x, gy, ws, g, lds, s);
    else
        e = launch_all<TB, WM, WN, FAST, UX>(x, gy, ws, g, lds, s);
    if (e != hipSuccess) return e;
    if (g.nsplit <= kFewRuns)
        hipLaunchKernelGGL(gw_reduce_few_kernel, dim3((unsigned)(nblk * WM * WN * 4)), dim3(64 * TB), 0, s, ws, gw, g, TB, WM, WN);
    else {
        // (300 layers: with DEEP everywhere up to 3 us longer, with it nowhere up to 3.3; above this line it takes 0.3 - 2 us more on most, below it 0.3 - 3.3 less)
        const int64_t wgs = (int64_t)nblk * TB * WM * WN * 16;
        const int cus = device_cus();
        auto k = wgs <= 2 * cus || wgs * g.nsplit <= 96 * cus ? gw_reduce_kernel<true> : gw_reduce_kernel<false>;
        hipLaunchKernelGGL(k, dim3((unsigned)wgs), dim3(256), 0, s, ws, gw, g, TB, WM, WN);
    }
    return hipGetLastError();
}

template <int TB, bool FAST>
hipError_t launch_gw2(const float *x, const float *gy, float *gw, float *ws, const GwTile &g, int WM, int WN, size_t lds, hipStream_t s)
{
    if (WM == 2 && WN == 2) return launch_gw1<TB, 2, 2, FAST>(x, gy, gw, ws, g, lds, s);
    if constexpr (TB == 9)
        if (WN == 1 && 4 * g.PS > 4 * kThreads)
            return WM == 2 ? launch_gw1<TB, 2, 1, FAST, 5>(x, gy, gw, ws, g, lds, s) : launch_gw1<TB, 1, 1, FAST, 5>(x, gy, gw, ws, g, lds, s);
    if (WM == 2) return launch_gw1<TB, 2, 1, FAST>(x, gy, gw, ws, g, lds, s);
    if (WN == 2) return launch_gw1<TB, 1, 2, FAST>(x, gy, gw, ws, g, lds, s);
    return launch_gw1<TB, 1, 1, FAST>(x, gy, gw, ws, g, lds, s);
}

template <int TB>
hipError_t launch_gw(const float *x, const float *gy, float *gw, float *ws, const GwTile &g, bool exact, int WM, int WN, size_t lds, hipStream_t s)
{
    if constexpr (TB == 5 || TB == 9)                 // (the taps of the layers whose runs need not be exact)
        if (!exact) return launch_gw2<TB, true>(x, gy, gw, ws, g, WM, WN, lds, s);
    return launch_gw2<TB, false>(x, gy, gw, ws, g, WM, WN, lds, s);
}

struct Groups { int rows, taps, ng, tb; };            // kernel rows and taps per row of a group; groups; taps of a group

Groups tap_groups(int kh, int kw)
{
    Groups q;
    q.taps = (kw + (kw + 8) / 9 - 1) / ((kw + 8) / 9);        // a row of more than nine taps: runs of it, evenly
    q.rows = kw <= 9 ? 9 / kw : 1;
    if (q.rows > kh) q.rows = kh;
    q.rows = (kh + (kh + q.rows - 1) / q.rows - 1) / ((kh + q.rows - 1) / q.rows);      // evenly
    q.ng = (kh + q.rows - 1) / q.rows * ((kw + q.taps - 1) / q.taps);
    q.tb = q.rows * q.taps;
    return q;
}

// A layer's plan: the geometry but for its taps' offsets; channel blocks of a workgroup; LDS and workspace bytes; estimated us.
struct GwPlan {
    GwTile g;
    int WM, WN;
    size_t lds;
    int64_t bytes;
    double us;
};

// The cheapest plan of at most `limit` bytes of workspace; false: the layer is not this kernel's.
// exact: see the dispatch (conv_grad.hip); no run then adds more than kMaxAdds times to a wavefront's sums.
bool plan_gw(const GwLayer &l, bool exact, int64_t limit, GwPlan *best)
{
    const int64_t N = l.N, Cin = l.Cin, H = l.H, W = l.W, Cout = l.Cout, Ho = l.Ho, Wo = l.Wo;
    const int kh = l.kh, kw = l.kw, sh = l.sh, sw = l.sw, dil = l.dil;
    if ((int64_t)kh * kw > kMaxTaps || sh > 2 || sw > 2 || N < 1) return false;
    if (N * Ho >= (1LL << 30) || H >= (1 << 18) || Ho >= (1 << 18) || W >= (1LL << 27) || Wo >= (1LL << 27) || Cin * H * W >= (1LL << 27) ||
        Cout * Ho * Wo >= (1LL << 27))
        return false;
    if (l.ph > 16384 || l.pw > 16384 || kw * (int64_t)dil > 16384) return false;
    const Groups q = tap_groups(kh, kw);
    GwTile &g = best->g;
    g.N = (int)N; g.Cin = (int)Cin; g.H = (int)H; g.W = (int)W; g.HW = (int)(H * W); g.Cout = (int)Cout; g.Ho = (int)Ho; g.Wo = (int)Wo;
    g.HoWo = (int)(Ho * Wo); g.NR = (int)(N * Ho); g.KT = kh * kw; g.sh = sh; g.sw = sw;
    g.SH = q.rows; g.ls = g.SH < sh ? g.SH : sh;
    if (g.SH < sh && g.SH != 1) return false;
    g.LPI = (int)(Ho - 1) * g.ls + g.SH;
    const int SW = (q.taps - 1) * dil + 1, SWc = SW < sw ? SW : sw, cus = device_cus();
    g.ng = q.ng;
    // Layers of conv_gw_staged_kernel: 3 x 3 at stride 1, channels in whole blocks, rows and strips of even length (pairs of positions lie side by side), one
    // unit of x per staging thread.
    const bool whole_blocks = kh == 3 && kw == 3 && sh == 1 && sw == 1 && Cin % 32 == 0 && Cout % 32 == 0 && Wo % 2 == 0;
    // The shapes of tiles: strip width and rows.  They are the same whatever the channel blocks.
    struct Shape { int TW, nstrips, CW, LW, rpt, period, lines, PS, tps, tiles, ksteps, nq; };
    Shape shapes[4 * 16];                             // (rows: 128, 96, 72 ... 4, 3, 2, 1 at most)
    int count = 0;
    for (int ns = (int)((Wo + kBN - 1) / kBN), last = ns + 3; ns <= last && ns <= Wo; ++ns) {
        Shape h;
        h.TW = (int)((unsigned)(Wo + ns - 1) / ns); h.nstrips = (int)((unsigned)(Wo + h.TW - 1) / h.TW);
        h.CW = h.TW + (int)((unsigned)(SW - 1) / sw); h.LW = SWc * h.CW;
        h.nq = ((h.LW < g.W ? h.LW : g.W) + 3) / 4;
        for (int rpt = kBN / h.TW < g.NR ? kBN / h.TW : g.NR; rpt >= 1; rpt = rpt > 4 ? rpt * 3 / 4 : rpt - 1) {
            // (tiles start at multiples of rpt, so at most this far down an image: where rpt divides Ho no tile meets two)
            int start = rpt, mod = g.Ho;
            while (mod) { const int r = (int)((unsigned)start % (unsigned)mod); start = mod; mod = r; }
            const int crossings = (int)((unsigned)(g.Ho - start + rpt - 1) / (unsigned)g.Ho);
            const int64_t lines = (int64_t)(rpt - 1) * g.ls + g.SH + crossings * (g.SH - g.ls);
            if (lines * h.LW > 1024) continue;
            const int64_t imgs = (unsigned)rpt / (unsigned)g.Ho + 2;      // a tile's images within 32-bit offsets
            if (imgs * Cin * H * W >= (1LL << 29) || imgs * Cout * Ho * Wo >= (1LL << 29)) continue;
            h.rpt = rpt; h.period = start; h.lines = (int)lines;
            h.PS = ((int)(lines * h.LW) + 3) / 16 * 16 + 12;
            h.tps = (int)((unsigned)(g.NR + rpt - 1) / rpt); h.ksteps = (rpt * h.TW + 15) / 16;
            if ((int64_t)h.tps * h.nstrips >= (1LL << 30)) continue;
            h.tiles = h.tps * h.nstrips;
            shapes[count++] = h;
        }
    }
    // Channel blocks of a workgroup, tile and runs: the smallest estimated time of the longest run (products
    // on two wavefronts per SIMD, staging per unit, a run's end), in cycles.  (The second pass is in `end` as it was before
    // there were two of them: it weighs channel blocks against runs, and takes 3 - 14 us either way.  This runs on every call: a form whose tiles alone, dealt to all compute units
    // evenly, take longer than the best so far is left at that.)
    bool found = false;
    double cost = 1e300;
    for (int wmn = 0; wmn < 4; ++wmn) {
        const int wm = 1 + (wmn & 1), wn = 1 + (wmn >> 1), wk = 8 / (wm * wn);
        if ((wm == 2 && Cout <= 32) || (wn == 2 && Cin <= 32)) continue;
        const int64_t cob = (Cout + 32 * wm - 1) / (32 * wm), cib = (Cin + 32 * wn - 1) / (32 * wn), nblk = cob * cib * g.ng;
        if (nblk * 16 * wm * wn * q.tb >= (1LL << 30)) continue;
        const double once = (4000 + 6.0 / 64 * q.tb * wm * wn * (double)nblk) * (1 - 1e-9), each = (double)nblk / cus * (1 - 1e-9);      // (rounding)
        for (int at = 0; at < count; ++at) {
            const Shape &h = shapes[at];
            const int TW = h.TW, rpt = h.rpt, tiles = h.tiles;
            const size_t stage = (size_t)4 * 3 * 16 * (wn * h.PS + wm * kPG) + kBN * 4;
            const size_t red = (size_t)(8 - wm * wn) * 4 * (q.tb < 3 ? q.tb : 3) * 1024;
            // (3 x 3 at stride 2 on one block of input channels: a fifth unit a thread lets a tile hold 112 positions instead of 84, whose four
            // wavefronts per block then take seven groups of 16 in the time of six: [32,64,56,56] -> 64, taken here for comparison, 34 us -> 26)
            if (4 * wn * h.PS > (wn == 1 && q.tb == 9 && sh == 2 && sw == 2 ? 5 : 4) * kThreads || stage > 158 * 1024) continue;
            const int steps = (h.ksteps + wk - 1) / wk, units = (4 * wn * h.PS + kThreads - 1) / kThreads + wm;
            const double tile = steps * (double)q.tb * 6 * 32 * 2 * 1.2 + 1200 + 500.0 * units;
            const size_t two = (size_t)4 * 3 * 16 * (2 * h.PS + wm * kPG) + 2 * kBN * 4, sums = (size_t)8 * 4 * 5 * 1024;
            const int64_t all = (int64_t)g.NR * h.nstrips;
            // conv_gw_staged_kernel: a multiplying wavefront's 16 positions and what a tile takes besides
            constexpr double kStep = 9 * 6 * 32 * 1.25, kTile = 1500;
            const bool one = once + each * tiles * tile < cost;
            const bool both = !exact && wn == 1 && whole_blocks && TW % 2 == 0 && 4 * h.lines * h.nq <= 256 && two <= 160 * 1024 && all < (1LL << 30) &&
                              once + 8000 + each * (double)all * TW / (8 * wk) * kStep < cost;
            if (!one && !both) continue;
            // Runs per block of gw: a workgroup fills a compute unit (LDS), so as many as there are units, or twice as many,
            // and never a few more: those would be a round of their own ([4,288,4658] -> 448, k = 1, 18 runs of 15 blocks: 132 us,
            // 17 runs: 66).
            for (int r = 1; r <= 2; ++r) {
                int64_t least = 1, whole = r;         // rounds
                if (exact) {
                    const int adds = q.tb <= 3 ? 1 : steps * (q.tb < 9 ? 1 : 3), most = kMaxAdds / adds > 1 ? kMaxAdds / adds : 1;
                    least = (int)((unsigned)(tiles + most - 1) / (unsigned)most);
                    const int64_t needs = (least * nblk + cus - 1) / cus;
                    if (whole < needs) whole = needs;
                }
                int64_t n = whole * cus / nblk;
                if (n < least) n = least;
                if (n > tiles) n = tiles;
                auto better = [&](double run, int nsplit, double rounds, double end) {
                    const double c = rounds * (run + 4000 + 6.0 * end / 64);
                    if (!(c < cost)) return false;
                    found = true;
                    cost = c;
                    best->WM = wm; best->WN = wn;
                    best->bytes = nblk * nsplit * q.tb * wm * wn * 4096;
                    g.TW = TW; g.nstrips = h.nstrips; g.CW = h.CW; g.LW = h.LW; g.rpt = rpt; g.PS = h.PS; g.tps = h.tps; g.tiles = tiles;
                    g.ksteps = h.ksteps; g.lines = h.lines; g.nq = h.nq; g.nsplit = nsplit; g.cob = (int)cob; g.cib = (int)cib;
                    return true;
                };
                auto fits = [&](int nsplit) { return nblk * nsplit * q.tb * wm * wn * 4096 <= limit && nblk * nsplit < (1LL << 30); };
                const int per = (int)((unsigned)(tiles + n - 1) / (unsigned)n), few = (int)((unsigned)(tiles + per - 1) / per);
                const double full = 0.269 * steps * q.tb + 1.67 + 0.09 * units;
                if (one && fits(few)) {
                    const double rounds = (double)(int)((unsigned)(nblk * few + cus - 1) / (unsigned)cus), end = q.tb * wm * wn * (double)(nblk * few);
                    if (better(per * tile, few, rounds, end)) {
                        best->lds = stage > red ? stage : red;
                        best->us = 6.9 + rounds * (per * full + 0.75) + 0.0026 * end;
                        g.per = per; g.rows = g.group = 0;
                    }
                }
                // A staged run costs its first tile's staging by half as many wavefronts and 160 KB of sums at its end, and saves the staging of every further
                // tile.  8000 cycles is on the safe side, long runs only: with 3500 [8,96,30,30] -> 160, four tiles a run, would come here too, 33 us -> 26.
                if (both) {
                    // (a staged run is rows: the runs of a round end together)
                    const int rows = (int)((unsigned)((all + n - 1) / n + h.period - 1) / (unsigned)h.period) * h.period;
                    const int nsplit = (int)((unsigned)(all + rows - 1) / (unsigned)rows);
                    if (!fits(nsplit)) continue;
                    // (runs of one image's strips side by side, i.e. in the same XCD's cache: a row's strips share cache lines)
                    const int group = h.nstrips == 1 || rows >= g.NR ? g.NR : rows < g.Ho ? g.Ho : (int)((unsigned)(rows + g.Ho / 2) / (unsigned)g.Ho) * g.Ho;
                    const double rounds = (double)(int)((unsigned)(nblk * nsplit + cus - 1) / (unsigned)cus), end = q.tb * wm * wn * (double)(nblk * nsplit);
                    auto part = [&](int of) { return ((of * TW + 15) / 16 + wk / 2 - 1) / (wk / 2) * kStep + kTile; };
                    const int whole_tiles = (int)((unsigned)rows / (unsigned)rpt), rest = rows - whole_tiles * rpt;
                    const double run = whole_tiles * part(rpt) + (rest ? part(rest) : 0) + ((unsigned)group % (unsigned)rows ? 3000 : 0) + 8000;
                    if (better(run, nsplit, rounds, end)) {
                        best->lds = two > sums ? two : sums;
                        best->us = 6.9 + rounds * (per * full + 0.75) + 0.0026 * end;
                        g.per = per; g.rows = rows; g.group = group;
                    }
                }
            }
        }
    }
    if (found) best->us += 12e-8 * (double)(N * (Cin * H * W + Cout * Ho * Wo));
    return found;
}

}  // namespace

// Bytes that suffice for a layer of these channels and taps whatever its planes: two rounds of runs on every compute unit.
int64_t conv_gw_tile_most(int64_t Cin, int64_t Cout, int kh, int kw)
{
    if ((int64_t)kh * kw > kMaxTaps || kh > 64 || kw > 64) return 0;
    const Groups q = tap_groups(kh, kw);
    int64_t most = 0;
    for (int wmn = 0; wmn < 4; ++wmn) {
        const int wm = 1 + (wmn & 1), wn = 1 + (wmn >> 1);
        if ((wm == 2 && Cout <= 32) || (wn == 2 && Cin <= 32)) continue;
        const int64_t nblk = ((Cout + 32 * wm - 1) / (32 * wm)) * ((Cin + 32 * wn - 1) / (32 * wn)) * q.ng;
        const int64_t bytes = (nblk > 2 * device_cus() ? nblk : 2 * device_cus()) * q.tb * wm * wn * 4096;
        most = bytes > most ? bytes : most;
    }
    return most;
}

// Bytes of workspace of a layer; 0: not this kernel's, or estimated to take longer than other_us.
int64_t conv_gw_tile_workspace(const GwLayer &l, bool exact, double other_us)
{
    GwPlan p;
    return plan_gw(l, exact, INT64_MAX, &p) && p.us <= other_us ? p.bytes : 0;
}

hipError_t launch_conv_gw_tile(const float *x, const float *gy, float *gw, const GwLayer &l, bool exact, double other_us, Workspace ws,
                               hipStream_t s, bool *taken)
{
    *taken = false;
    if (!ws.p || ((uintptr_t)ws.p & 15)) return hipSuccess;
    GwPlan p;
    if (!plan_gw(l, exact, ws.bytes, &p) || p.us > other_us) return hipSuccess;
    GwTile &g = p.g;
    const int WM = p.WM, WN = p.WN;
    const size_t lds = p.lds;
    const Groups q = tap_groups(l.kh, l.kw);
    const int runs = (l.kw + q.taps - 1) / q.taps;
    for (int k = 0; k < q.ng; ++k) {
        const int a0 = k / runs * q.rows, b0 = k % runs * q.taps;
        const int na = l.kh - a0 < q.rows ? l.kh - a0 : q.rows, nb = l.kw - b0 < q.taps ? l.kw - b0 : q.taps;
        g.gdh[k] = (short)(a0 - l.ph); g.gdw[k] = (short)(b0 * l.dil - l.pw);
        g.gt0[k] = (unsigned char)(a0 * l.kw + b0); g.gnt[k] = (unsigned char)(na * nb);
    }
    for (int t = 0; t < g.KT; ++t) {
        const int a = t / l.kw % q.rows, bcol = t % l.kw % q.taps * l.dil;
        g.tapoff[t] = (unsigned short)(a * g.LW + bcol % l.sw * g.CW + bcol / l.sw);
    }
    for (int t = g.KT; t < kMaxTaps; ++t) g.tapoff[t] = 0;
    g.inv_TW = 1.0f / g.TW; g.inv_Ho = 1.0f / g.Ho; g.inv_LPI = 1.0f / g.LPI; g.inv_LW = 1.0f / g.LW; g.inv_CW = 1.0f / g.CW;
    g.inv_PS = 1.0f / g.PS;
    g.inv_nq = 1.0f / g.nq; g.inv_lines = 1.0f / g.lines;
    float *w = (float *)ws.p;
    *taken = true;
#define SWS_GW_TB(T) case T: return launch_gw<T>(x, gy, gw, w, g, exact, WM, WN, lds, s)
    switch (q.tb) {
        SWS_GW_TB(1); SWS_GW_TB(2); SWS_GW_TB(3); SWS_GW_TB(4); SWS_GW_TB(5); SWS_GW_TB(6); SWS_GW_TB(7); SWS_GW_TB(8);
    default: return launch_gw<9>(x, gy, gw, w, g, exact, WM, WN, lds, s);
    }
#undef SWS_GW_TB
}

}  // namespace sws
