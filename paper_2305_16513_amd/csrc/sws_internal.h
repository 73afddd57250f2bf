// Internal declarations shared by the libsws translation units (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "sws.h"
#include "sws_dev.h"

namespace sws {

// Measurement knobs set through sws_set_option(); 0 means "choose automatically".  Host-side only;
// every launcher reads a knob once (relaxed atomic load through Knob's conversion).
struct Knob {
    std::atomic<int> v{0};
    operator int() const { return v.load(std::memory_order_relaxed); }
    Knob &operator=(int x) { v.store(x, std::memory_order_relaxed); return *this; }
};
struct Options {
    Knob slide_variant;
    Knob slide_chunk;
    Knob slide_group;
    Knob pool2d_variant;
    Knob conv1d_variant;
    Knob conv2d_variant;
    Knob copy_variant;
};
extern Options g_opt;

// A launcher's answer when its kernel does not cover the request (the caller then tries the next
// kernel); never a code the HIP runtime returns.
constexpr hipError_t kNotTaken = (hipError_t)2047;

constexpr int kWave = 64;    // CDNA wavefront width
constexpr int kXcd = 8;      // XCDs (separate L2s) on MI355X

typedef float v4f __attribute__((ext_vector_type(4)));
typedef v4f v4f_u __attribute__((aligned(4)));     // 16-byte access at 4-byte alignment
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef short v4s __attribute__((ext_vector_type(4)));

// The operator (+) of the sliding window sum, with its identity element.  `a` is always
// the older (left) operand so the kernels stay valid for non-commutative operators.
template <int OP> struct Op;
template <> struct Op<SWS_OP_ADD> {
    static __device__ __forceinline__ float id() { return 0.0f; }
    static __device__ __forceinline__ float f(float a, float b) { return a + b; }
};
template <> struct Op<SWS_OP_MAX> {
    static __device__ __forceinline__ float id() { return -__builtin_huge_valf(); }
    static __device__ __forceinline__ float f(float a, float b) { return __builtin_fmaxf(a, b); }
};
template <> struct Op<SWS_OP_MIN> {
    static __device__ __forceinline__ float id() { return __builtin_huge_valf(); }
    static __device__ __forceinline__ float f(float a, float b) { return __builtin_fminf(a, b); }
};

// x / d for 0 <= x < 2^20, inv_d = 1.0f / d, exact (the margin 0.5 / d is larger than the rounding of the product: x / d < 2^20)
__device__ __forceinline__ int fdiv(int x, float inv_d) { return (int)(((float)x + 0.5f) * inv_d); }

// the upper halves of two floats as one register of two bf16 (lo in the low half)
__device__ __forceinline__ unsigned pack_hi(float lo, float hi)
{
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}

// f as three bf16 numbers whose sum it is, each rounded to nearest (but cut where that would be infinity): the products of pieces
// that are left out are then smallest.
__device__ __forceinline__ void split_nearest(float f, __bf16 &f1, __bf16 &f2, __bf16 &f3)
{
    f1 = (__bf16)(__builtin_fabsf(f) < 0x1.ffp127f ? f : __uint_as_float(__float_as_uint(f) & 0xffff0000u));
    const float r1 = f - (float)f1;
    f2 = (__bf16)r1;
    f3 = (__bf16)(r1 - (float)f2);
}

// Eight 16-bit elements of a lane by two transposing LDS reads of four.
__device__ __forceinline__ v8bf tr8(const char *p0, const char *p1)
{
    typedef __attribute__((address_space(3))) v4s lds_v4s;
    const v4s a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s *)p0);
    const v4s b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s *)p1);
    return __builtin_bit_cast(v8bf, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
}

// The lines of a kernel's arguments (BYTES of them) fetched side by side, as the first thing that it does.  A launch's arguments are cold: a 64-byte line takes a wavefront
// 700 cycles, from the scalar cache 84, and the compiler reads the fields of a large structure one after the other, where they are used.
// (Waited for in here: the registers hold nothing that anybody reads.)
template <int BYTES>
__device__ __forceinline__ void fetch_arguments()
{
    constexpr int n = (BYTES + 63) / 64, last = (BYTES - 4) / 4 * 4;
    static_assert(n <= 12, "more lines than loads below");
    const auto *p = __builtin_amdgcn_kernarg_segment_ptr();
    unsigned t0, t1, t2, t3, t4, t5, t6, t7, t8, t9, t10, t11;
#define SWS_LINE(I) "i"(64 * I < last ? 64 * I : last)
    if constexpr (n <= 4)
        asm volatile("s_load_dword %0, %4, %5\n\ts_load_dword %1, %4, %6\n\ts_load_dword %2, %4, %7\n\ts_load_dword %3, %4, %8\n\ts_waitcnt lgkmcnt(0)"
                     : "=&s"(t0), "=&s"(t1), "=&s"(t2), "=&s"(t3) : "s"(p), SWS_LINE(0), SWS_LINE(1), SWS_LINE(2), SWS_LINE(3));
    else
        asm volatile("s_load_dword %0, %12, %13\n\ts_load_dword %1, %12, %14\n\ts_load_dword %2, %12, %15\n\ts_load_dword %3, %12, %16\n\t"
                     "s_load_dword %4, %12, %17\n\ts_load_dword %5, %12, %18\n\ts_load_dword %6, %12, %19\n\ts_load_dword %7, %12, %20\n\t"
                     "s_load_dword %8, %12, %21\n\ts_load_dword %9, %12, %22\n\ts_load_dword %10, %12, %23\n\ts_load_dword %11, %12, %24\n\ts_waitcnt lgkmcnt(0)"
                     : "=&s"(t0), "=&s"(t1), "=&s"(t2), "=&s"(t3), "=&s"(t4), "=&s"(t5), "=&s"(t6), "=&s"(t7), "=&s"(t8), "=&s"(t9), "=&s"(t10), "=&s"(t11)
                     : "s"(p), SWS_LINE(0), SWS_LINE(1), SWS_LINE(2), SWS_LINE(3), SWS_LINE(4), SWS_LINE(5), SWS_LINE(6), SWS_LINE(7), SWS_LINE(8),
                       SWS_LINE(9), SWS_LINE(10), SWS_LINE(11));
#undef SWS_LINE
}

// One buffer descriptor: loads beyond `bytes` return zero; kNowhere lies beyond every descriptor.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(const void *p, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000);
}
constexpr unsigned kNowhere = 0x80000000u;

// N sliding windows of K consecutive elements at stride 1, out[j] = in[j] (+) ... (+) in[j + K - 1], from what they
// share: the elements N - 1 .. K - 1 lie in all of them and are combined once; window j puts the rest of the head
// in front (in[j] .. in[N - 2]) and the start of the tail behind (in[K] .. in[K + j - 1]) — Section 3's suffix /
// prefix split between registers.  K + 3N - 6 operations instead of N (K - 1); operand order is kept.
// F(a, b) combines two elements (floats, or vectors of columns).
template <int K, int N, typename E, typename F>
__device__ __forceinline__ void windows_shared(const E *in, E *out, F f)
{
    // (windows of fewer than five elements are combined left to right as Eq. 3 writes them: nothing to gain, and the
    // strided kernels, which share nothing, then give the same bits)
    if constexpr (N < 2 || K < N || K < 5 || K + 3 * N - 6 >= N * (K - 1)) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            E acc = in[j];
#pragma unroll
            for (int b = 1; b < K; ++b) acc = f(acc, in[j + b]);
            out[j] = acc;
        }
    } else {
        E core = in[N - 1];
#pragma unroll
        for (int b = N; b < K; ++b) core = f(core, in[b]);
        E head[N - 1], tail[N - 1];                  // head[j] = in[j] .. in[N-2];  tail[j] = in[K] .. in[K+j]
        head[N - 2] = in[N - 2];
#pragma unroll
        for (int j = N - 3; j >= 0; --j) head[j] = f(in[j], head[j + 1]);
        tail[0] = in[K];
#pragma unroll
        for (int j = 1; j < N - 1; ++j) tail[j] = f(tail[j - 1], in[K + j]);
#pragma unroll
        for (int j = 0; j < N; ++j) {
            E acc = j < N - 1 ? f(head[j], core) : core;
            out[j] = j > 0 ? f(acc, tail[j - 1]) : acc;
        }
    }
}

// Boundary conditions of a row extended by pad_left virtual elements in front (and more behind):
// the physical index that virtual element e stands for, or -1 for the operator's identity.
// mode: SWS_PAD_IDENTITY, SWS_PAD_MIRROR (x[-i] = x[i]), SWS_PAD_PERIODIC (x[-i] = x[len-i]),
// SWS_PAD_EDGE (the end element repeated), SWS_PAD_SHRINK (identity; the caller rescales ADD results).
// The caller keeps e inside the extended row.
__device__ __forceinline__ int pad_src(int e, int len, int pad_left, int mode)
{
    const int p = e - pad_left;
    if (p >= 0 && p < len) return p;
    if (mode == SWS_PAD_IDENTITY || mode == SWS_PAD_SHRINK) return -1;
    if (mode == SWS_PAD_MIRROR) return p < 0 ? -p : 2 * (len - 1) - p;
    if (mode == SWS_PAD_PERIODIC) return p < 0 ? p + len : p - len;
    return p < 0 ? 0 : len - 1;
}

// Workgroups are dealt round-robin to the 8 XCDs.  This maps blockIdx so that each XCD
// (one L2) walks a contiguous range of work units, keeping a tile's halo re-read in the
// L2 that fetched it.  Returns an id in [0, n_units) or -1 for the padding blocks.
__device__ __forceinline__ int64_t xcd_unit(int64_t n_units)
{
    const int64_t b = blockIdx.x;
    const int64_t per = (n_units + kXcd - 1) / kXcd;
    const int64_t u = (b % kXcd) * per + b / kXcd;
    return (b / kXcd < per && u < n_units) ? u : -1;
}
// The same in runs of kXcdRun units, for kernels that stream through memory once: the eight XCDs then walk through one window
// together instead of eight windows an eighth of the input apart, and all but one halo in kXcdRun still stay in one L2
// ([8,64,65536] depthwise, k = 13: 48 us against 55; runs of 4, 8 and 16 alike, of one 5 % behind with wide halos).  32-bit arithmetic: a 64-bit division costs a wavefront
// about a hundred vector instructions.
constexpr int kXcdRun = 8;
__device__ __forceinline__ int xcd_run_unit(int n_units)
{
    const int b = blockIdx.x, in = b % (kXcd * kXcdRun), u = b - in + in % kXcd * kXcdRun + in / kXcd;
    return u < n_units ? u : -1;
}
inline int64_t xcd_run_grid(int64_t n_units) { return (n_units + kXcd * kXcdRun - 1) / (kXcd * kXcdRun) * (kXcd * kXcdRun); }
// Kernels pull every row's tile origins back by (r * lo) mod line elements so that stores start on
// 64-byte lines.  The largest such shift over all rows r: line - gcd(lo mod line, line), i.e. 0 when
// lo is a multiple of the line (then no row needs an extra tile).
inline int max_origin_shift(int64_t lo, int line)
{
    int a = (int)(lo % line), b = line;
    while (a) { const int t = b % a; b = a; a = t; }
    return line - b;
}

// A kernel's limit of dynamic LDS raised to `bytes`, once per device (`done`: the caller's, one bit a device; raising it twice does no harm).
inline hipError_t raise_lds(const void *kernel, int bytes, std::atomic<uint64_t> &done)
{
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev < 64 ? 1ull << dev : 0;
    if (done.load(std::memory_order_relaxed) & bit) return hipSuccess;
    const hipError_t a = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (a == hipSuccess) done.fetch_or(bit, std::memory_order_relaxed);
    return a;
}

// Device memory a caller lends a dense convolution for the duration of the call (stream-ordered); empty: none.
struct Workspace {
    void *p = nullptr;
    int64_t bytes = 0;
};

// Compute units of the current device (256 on MI355X), asked once.
int device_cus();

inline int64_t xcd_grid(int64_t n_units) { return ((n_units + kXcd - 1) / kXcd) * kXcd; }

hipError_t launch_copy(const float *src, float *dst, int64_t n, hipStream_t s);
hipError_t launch_slide1d(int op, const float *x, float *y, int64_t rows, int64_t len, int32_t w,
                          int32_t pad_left, int32_t pad_right, int pad_mode, float scale, hipStream_t s);
hipError_t launch_slide1d_16(int op, int dtype, const void *x, void *y, int64_t rows, int64_t len, int32_t w,
                             float scale, hipStream_t s);
// Generic-operator kernels (slide_generic.hip): the pair operator, and +, max, min as a cross-check.
hipError_t launch_slide1d_pair(const float *u, const float *v, float *yu, float *yv, int64_t rows, int64_t len,
                               int32_t w, hipStream_t s);
// Medium windows (slide1d_reg_min_w() .. slide1d_reg_max_w()) on plain rows: one 256-element strip per
// single-wavefront workgroup, held in registers, whole lanes summed across the wavefront (slide_reg.hip).
// kNotTaken: not its case, nothing launched.
int slide1d_reg_min_w();
int slide1d_reg_max_w();
hipError_t launch_slide1d_reg(int op, const float *x, float *y, int64_t rows, int len, int lo, int w, float scale,
                              hipStream_t s);

// Short rows, windows up to slide1d_rows_max_w(): four outputs per lane from shifted 128-bit loads,
// several rows per wavefront.  hipErrorInvalidValue: not taken (w or grid beyond its reach).
// 2-D pooling on planes of a few hundred elements: several whole planes per workgroup through LDS.
// *taken = false: not its case (the caller goes on to the other kernels).
// (T: float, or 16-bit storage with fp32 arithmetic)
template <typename T>
hipError_t launch_pool2d_small(int op, const T *x, T *y, int64_t planes, int H, int W, int Ho, int Wo, int kh,
                               int kw, int sh, int sw, int ph, int pw, float scale, int div_valid, hipStream_t s,
                               bool *taken);
int slide1d_rows_max_w();
hipError_t launch_slide1d_rows(int op, const float *x, float *y, int64_t rows, int len, int lo, int32_t w, float scale,
                               bool padded, int pad_left, int pad_mode, hipStream_t s);
// Windows longer than a wave tile in one pass (slide_long.hip): w > 256, plain rows or rows extended by a boundary
// rule other than the shrinking window; kNotTaken otherwise.
hipError_t launch_slide1d_long(int op, const float *x, float *y, int64_t rows, int len, int lo, int w, float scale,
                               bool padded, int pad_left, int pad_mode, int lv, hipStream_t s);
hipError_t launch_slide1d_long_16(int op, int dtype, const void *x, void *y, int64_t rows, int len, int lo, int w,
                                  float scale, hipStream_t s);
hipError_t launch_slide1d_generic(int op, const float *x, float *y, int64_t rows, int64_t len, int32_t w, float scale,
                                  hipStream_t s);
hipError_t launch_pool2d(int op, const float *x, float *y, int64_t planes, int64_t H, int64_t W,
                         int64_t Ho, int64_t Wo, int32_t kh, int32_t kw, int32_t sh, int32_t sw,
                         int32_t ph, int32_t pw, float scale, int div_valid, hipStream_t s);
// Pooling over planes extended by a boundary rule on four sides (pool2d_padded.hip).
hipError_t launch_pool2d_padded(int op, const float *x, float *y, int64_t planes, int64_t H, int64_t W, int64_t Ho,
                                int64_t Wo, int32_t kh, int32_t kw, int32_t sh, int32_t sw, int32_t pt, int32_t pl,
                                int32_t pb, int32_t pr, int mode, float scale, hipStream_t s);
hipError_t launch_maxpool2d_grad(const float *x, const float *gy, float *gx, int64_t planes, int64_t H, int64_t W,
                                 int64_t Ho, int64_t Wo, int32_t kh, int32_t kw, int32_t sh, int32_t sw, int32_t ph,
                                 int32_t pw, hipStream_t s);
hipError_t launch_avgpool2d_grad(const float *gy, float *gx, int64_t planes, int64_t H, int64_t W, int64_t Ho, int64_t Wo,
                                 int32_t kh, int32_t kw, int32_t sh, int32_t sw, int32_t ph, int32_t pw, int div_real,
                                 float scale, hipStream_t s);
// Row-streaming adjoints of 3 x 3 pooling (pool_grad_rows.hip); *taken = false: shape not covered, nothing launched.
hipError_t launch_maxpool2d_grad_rows(const float *x, const float *gy, float *gx, int64_t planes, int H, int W, int Ho,
                                      int Wo, int kh, int kw, int sh, int sw, int ph, int pw, hipStream_t s, bool *taken);
// Large windows (pool_grad_large.hip); *taken = false: not its case, nothing launched.
hipError_t launch_maxpool2d_grad_large(const float *x, const float *gy, float *gx, int64_t planes, int64_t H, int64_t W, int64_t Ho,
                                       int64_t Wo, int kh, int kw, int sh, int sw, int ph, int pw, hipStream_t s, bool *taken);
hipError_t launch_avgpool2d_grad_rows(const float *gy, float *gx, int64_t planes, int H, int W, int Ho, int Wo, int kh,
                                      int kw, int sh, int sw, int ph, int pw, float scale, hipStream_t s, bool *taken);
hipError_t launch_pool2d_16(int op, int dtype, const void *x, void *y, int64_t planes, int64_t H, int64_t W, int64_t Ho,
                            int64_t Wo, int32_t kh, int32_t kw, int32_t sh, int32_t sw, int32_t ph, int32_t pw,
                            float scale, hipStream_t s);
hipError_t launch_conv1d(const float *x, const float *wgt, float *y, int64_t B, int64_t Cin, int64_t L,
                         int64_t Cout, int64_t Lo, int32_t k, int32_t stride, int32_t pad,
                         int32_t dilation, int32_t groups, hipStream_t s, int wadj = 0, bool *taken = nullptr, Workspace ws = {});
// Rows extended by pad_left / pad_right elements under a boundary rule (mirror, periodic, edge; conv1d.hip).
hipError_t launch_conv1d_padded(const float *x, const float *wgt, float *y, int64_t B, int64_t Cin, int64_t L,
                                int64_t Cout, int64_t Lo, int32_t k, int32_t stride, int32_t pad_left, int32_t pad_right,
                                int32_t dilation, int32_t groups, int mode, hipStream_t s, Workspace ws = {});
// Thin layers (one input channel per output channel) on the bf16 matrix cores (conv1d_toep.hip); wadj: the taps run
// backwards.  toep_wanted: the layers that run there by themselves; kNotTaken: not its case, nothing launched.
bool conv1d_toep_takes(int32_t k, int32_t dilation);
bool conv1d_toep_wanted(int64_t rows, int64_t Lo, int32_t k, int32_t dilation);
hipError_t launch_conv1d_toep(const float *x, const float *wgt, float *y, int64_t B, int64_t Cin, int64_t L, int64_t Cout, int64_t Lo,
                              int32_t k, int32_t pad, int32_t dilation, int32_t groups, hipStream_t s, int wadj);
// Dense 1-D layers of 32 / 64 input channels on the bf16 matrix cores with split fp32 operands (conv1d_split.hip);
// *taken = false: not one of its shapes, nothing launched.
hipError_t launch_conv1d_split(const float *x, const float *wgt, float *y, int64_t B, int64_t Cin, int64_t L, int64_t Cout,
                               int64_t Lo, int32_t k, int32_t pad, hipStream_t s, bool *taken);
// 16-bit storage (conv1d16.hip): x, y bf16 / fp16, taps fp32.
hipError_t launch_conv1d_16(int dtype, const void *x, const float *wgt, void *y, int64_t B, int64_t Cin, int64_t L,
                            int64_t Cout, int64_t Lo, int32_t k, int32_t stride, int32_t pad, int32_t dilation,
                            int32_t groups, hipStream_t s);
// Adjoints of the 1-D convolution (conv_grad.hip).
hipError_t launch_conv1d_grad_input(const float *gy, const float *wgt, float *gx, int64_t B, int64_t Cin, int64_t L,
                                    int64_t Cout, int64_t Lo, int32_t k, int32_t stride, int32_t pad,
                                    int32_t dilation, int32_t groups, hipStream_t s, Workspace ws = {});
hipError_t launch_conv1d_grad_weight(const float *x, const float *gy, float *gw, int64_t B, int64_t Cin, int64_t L,
                                     int64_t Cout, int64_t Lo, int32_t k, int32_t stride, int32_t pad,
                                     int32_t dilation, int32_t groups, hipStream_t s, Workspace ws = {});
hipError_t launch_conv2d_grad_input(const float *gy, const float *wgt, float *gx, int64_t N, int64_t Cin, int64_t H,
                                    int64_t W, int64_t Cout, int64_t Ho, int64_t Wo, int32_t kh, int32_t kw, int32_t sh,
                                    int32_t sw, int32_t ph, int32_t pw, hipStream_t s, Workspace ws = {});
hipError_t launch_conv2d_grad_weight(const float *x, const float *gy, float *gw, int64_t N, int64_t Cin, int64_t H,
                                     int64_t W, int64_t Cout, int64_t Ho, int64_t Wo, int32_t kh, int32_t kw, int32_t sh,
                                     int32_t sw, int32_t ph, int32_t pw, hipStream_t s, Workspace ws = {});
hipError_t launch_conv2d(const float *x, const float *wgt, float *y, int64_t N, int64_t Cin, int64_t H,
                         int64_t W, int64_t Cout, int64_t Ho, int64_t Wo, int32_t kh, int32_t kw,
                         int32_t sh, int32_t sw, int32_t ph, int32_t pw, hipStream_t s, Workspace ws = {});

// Planes extended on four sides under a boundary rule (conv2d_padded.hip).
hipError_t launch_conv2d_padded(const float *x, const float *wgt, float *y, int64_t N, int64_t Cin, int64_t H, int64_t W,
                                int64_t Cout, int64_t Ho, int64_t Wo, int32_t kh, int32_t kw, int32_t sh, int32_t sw,
                                int32_t pt, int32_t pl, int32_t pb, int32_t pr, int mode, hipStream_t s, Workspace ws = {});

// Dense grad-weight on the bf16 matrix cores with split fp32 operands (conv_gw_split.hip): 3 x 3, horizontal
// stride 1, channel counts in multiples of 32; gw must hold zeros; *taken = false: not its case, nothing launched.
hipError_t launch_conv2d_gw_split(const float *x, const float *gy, float *gw, int64_t N, int64_t Cin, int64_t H, int64_t W,
                                  int64_t Cout, int64_t Ho, int64_t Wo, int32_t kh, int32_t kw, int32_t sh, int32_t sw,
                                  int32_t ph, int32_t pw, hipStream_t s, bool *taken);

// The same for kernels one row high (the 1-D convolution; 1 x k layers): rows = images * RH rows of L inputs / Lo outputs.
hipError_t launch_conv1d_gw_split(const float *x, const float *gy, float *gw, int64_t rows, int RH, int64_t Cin, int64_t L,
                                  int64_t Cout, int64_t Lo, int32_t k, int32_t pad, int64_t x_cs, int64_t gy_cs, hipStream_t s,
                                  bool *taken);

// Matrix-core convolution (conv_mfma.hip); *taken = false: shape not covered, nothing launched.
bool conv2d_gw_split_takes(int64_t Cin, int64_t W, int64_t Cout, int32_t kh, int32_t kw, int32_t sh, int32_t sw, int32_t pw);
double conv1d_gw_split_us(int64_t rows, int64_t Cin, int64_t L, int64_t Cout, int64_t Lo, int32_t k, int32_t pad);
hipError_t launch_conv2d_mfma(const float *x, const float *wgt, float *y, int64_t N, int64_t Cin, int64_t H,
                              int64_t W, int64_t Cout, int64_t Ho, int64_t Wo, int32_t kh, int32_t kw, int32_t sh,
                              int32_t sw, int32_t ph, int32_t pw, int32_t dh, int32_t dw, hipStream_t s,
                              bool *taken, int wadj = 0, Workspace ws = {});
// Dense layers on the bf16 matrix cores with split fp32 operands, weights split into the caller's workspace first
// (conv_split.hip); *taken = false: not its case or the workspace is too small, nothing launched.
int64_t conv_split_workspace(int64_t Cin, int64_t Cout, int64_t KT, int64_t positions);
hipError_t launch_conv_split(const float *x, const float *wgt, float *y, int64_t N, int64_t Cin, int64_t H, int64_t W,
                             int64_t Cout, int64_t Ho, int64_t Wo, int64_t yH, int64_t yW, int sh, int sw, int KT,
                             const int *dh, const int *dw, const int *wt, const int *ph, int64_t wco, int64_t wci, Workspace ws,
                             hipStream_t s, bool *taken);
hipError_t launch_conv2d_split(const float *x, const float *wgt, float *y, int64_t N, int64_t Cin, int64_t H, int64_t W,
                               int64_t Cout, int64_t Ho, int64_t Wo, int32_t kh, int32_t kw, int32_t sh, int32_t sw,
                               int32_t ph, int32_t pw, int32_t dh, int32_t dw, hipStream_t s, bool *taken, int wadj, Workspace ws);
// Dense grad-weight on the bf16 matrix cores through transposing LDS reads, partial sums in the caller's workspace (conv_gw_tile.hip);
// gw need not hold zeros; *taken = false: not its case or the workspace is too small, nothing launched.
struct GwLayer {
    int64_t N, Cin, H, W, Cout, Ho, Wo;
    int kh, kw, sh, sw, ph, pw, dil;                  // (dil: along rows)
};
int64_t conv_gw_tile_most(int64_t Cin, int64_t Cout, int kh, int kw);
int64_t conv_gw_tile_workspace(const GwLayer &l, bool exact, double other_us);
hipError_t launch_conv_gw_tile(const float *x, const float *gy, float *gw, const GwLayer &l, bool exact, double other_us, Workspace ws,
                               hipStream_t s, bool *taken);
// Bytes that the adjoints with respect to the weights use, 0: none (conv_grad.hip).
int64_t conv2d_gw_workspace(int64_t N, int64_t Cin, int64_t H, int64_t W, int64_t Cout, int64_t Ho, int64_t Wo, int32_t kh, int32_t kw, int32_t sh,
                            int32_t sw, int32_t ph, int32_t pw);
int64_t conv1d_gw_workspace(int64_t B, int64_t Cin, int64_t L, int64_t Cout, int64_t Lo, int32_t k, int32_t stride, int32_t pad, int32_t dilation,
                            int32_t groups);
// Weight-stationary streaming kernel (conv_stream.hip): 64 input channels, 3 x 3 on narrow images and
// 1 x 3 on 1-D rows, stride 1; *taken = false: not its case, nothing launched.
hipError_t launch_conv2d_stream(const float *x, const float *wgt, float *y, int64_t N, int64_t Cin, int64_t H, int64_t W,
                                int64_t Cout, int64_t Ho, int64_t Wo, int32_t kh, int32_t kw, int32_t ph, int32_t pw,
                                hipStream_t s, bool *taken, int wadj, bool split_only = false);
// Strided adjoint with respect to the input, one stride-1 launch chain per output phase; phases no
// tap reaches are NOT written (the caller clears gx first when kh < sh or kw < sw).
hipError_t launch_conv2d_grad_input_phases(const float *gy, const float *wgt, float *gx, int64_t N, int64_t Cin,
                                           int64_t H, int64_t W, int64_t Cout, int64_t Ho, int64_t Wo, int32_t kh,
                                           int32_t kw, int32_t sh, int32_t sw, int32_t ph, int32_t pw, hipStream_t s,
                                           bool *taken, Workspace ws = {});

// Direct-evaluation fallbacks (naive_kernels.hip).
hipError_t launch_slide1d_naive(int op, const float *x, float *y, int64_t rows, int64_t len, int32_t w,
                                int32_t pad_left, int32_t pad_right, int pad_mode, float scale, hipStream_t s);
hipError_t launch_pool2d_naive(int op, const float *x, float *y, int64_t planes, int64_t H, int64_t W,
                               int64_t Ho, int64_t Wo, int32_t kh, int32_t kw, int32_t sh, int32_t sw,
                               int32_t ph, int32_t pw, float scale, int div_valid, hipStream_t s);
hipError_t launch_conv1d_naive(const float *x, const float *wgt, float *y, int64_t B, int64_t Cin,
                               int64_t L, int64_t Cout, int64_t Lo, int32_t k, int32_t stride, int32_t pad,
                               int32_t dilation, int32_t groups, hipStream_t s, int mode = SWS_PAD_IDENTITY);
hipError_t launch_conv2d_naive(const float *x, const float *wgt, float *y, int64_t N, int64_t Cin,
                               int64_t H, int64_t W, int64_t Cout, int64_t Ho, int64_t Wo, int32_t kh,
                               int32_t kw, int32_t sh, int32_t sw, int32_t ph, int32_t pw, hipStream_t s);

}  // namespace sws
