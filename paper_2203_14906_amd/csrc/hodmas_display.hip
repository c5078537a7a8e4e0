// Display chain of a beamformed image (Sec. III): band-pass along depth,
// envelope by the Hilbert transform, log compression.
//
// Kernel 1 (envelope_kernel) takes pairs of neighbouring depth columns.  The
// columns are read row by row into LDS and band-passed with the centred FIR,
// eight outputs of both columns per lane from a sliding register window.  The
// analytic signal of a real column x is x + i h with h the Hilbert transform
// over bins 1..nz/2-1, and h is real, so one complex FFT of (x_a + i x_b) and
// back, with the bins turned by -i and +i between, gives h_a + i h_b: half the
// transforms, and x itself is never rounded by them.  The transform runs in
// registers, eight points per lane: radix-8 decimation-in-frequency stages
// (natural order in, digit-reversed out) and their mirror images back, in place
// through LDS, the innermost stage and its inverse with no exchange between.
// It writes the envelope sqrt(x^2 + h^2) and one maximum per workgroup.
// Kernel 2 reduces those maxima and writes 20 log10(envelope / max), clipped
// at the dynamic range.
//
// Kernel 1 is bound by VALU issue where the launch fills the device (63 taps:
// 68 of its 120 VALU instructions per pixel are the filter's) and by one wave's latency where
// it does not.  16 images of 1024 x 1024, 63 taps: 71 us, and kernel 2 24 us
// (5.4 TB/s of reads and writes), together 98 us a pass; a radix-2 transform
// per column with every pass through LDS took 407 + 57 us.  One 512 x 512
// image: 8.6 + 2.5 us, was 20.9 + 3.5.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <new>
#include <vector>

#include "hodmas.h"

namespace {

constexpr int kDispBlock = 256;
constexpr int kMaxNz = 8192;
constexpr int kMaxLog2Nz = 13;
constexpr int kMaxTaps = 255;
constexpr int kTapFloats = 256;          // taps on the device: zeros to a multiple of 16
constexpr uint32_t kDisplayMagic = 0x44495350u;  // "DISP"
constexpr int kXcds = 8;                 // workgroup b runs on XCD b mod 8
// Word 3 of a raw (stride 0) buffer resource on gfx950: 32-bit data format, an
// access is in range iff its byte offset is below the resource's size.
constexpr int kBufferFlags = 0x00020000;

// Images of one launch: the envelope kernel and the log compression take
// image blockIdx.y (up to kDisplayBatch per launch pair).
constexpr int kDisplayBatch = 16;
struct DisplayImages {
    const float* image[kDisplayBatch];
    float* env[kDisplayBatch];        // envelope out (the dB buffer when no envelope is wanted)
    float* db[kDisplayBatch];
};

struct Complex {
    float x, y;
};
__device__ __forceinline__ Complex operator+(Complex a, Complex b) { return {a.x + b.x, a.y + b.y}; }
__device__ __forceinline__ Complex operator-(Complex a, Complex b) { return {a.x - b.x, a.y - b.y}; }
// a exp(-i t) forward, a exp(+i t) back, w = exp(-i t)
template <bool BACK>
__device__ __forceinline__ Complex turn(Complex a, float2 w)
{
    const float s = BACK ? -w.y : w.y;
    return {a.x * w.x - a.y * s, a.x * s + a.y * w.x};
}
// a times -i forward, +i back
template <bool BACK>
__device__ __forceinline__ Complex quarter(Complex a)
{
    return BACK ? Complex{-a.y, a.x} : Complex{a.y, -a.x};
}

// DFT of R points a[0], a[S], a[2 S], .., in place and in order.
template <int R, int S, bool BACK>
__device__ __forceinline__ void dft(Complex* a)
{
    if constexpr (R == 2) {
        const Complex t = a[0] - a[S];
        a[0] = a[0] + a[S];
        a[S] = t;
    } else if constexpr (R == 4) {
        const Complex s0 = a[0] + a[2 * S], s1 = a[0] - a[2 * S];
        const Complex s2 = a[S] + a[3 * S], s3 = quarter<BACK>(a[S] - a[3 * S]);
        a[0] = s0 + s2;
        a[S] = s1 + s3;
        a[2 * S] = s0 - s2;
        a[3 * S] = s1 - s3;
    } else if constexpr (R == 8) {
        constexpr float c = 0.70710678118654752f;
        Complex u[4], v[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            u[m] = a[m * S] + a[(m + 4) * S];
            v[m] = a[m * S] - a[(m + 4) * S];
        }
        const Complex q1 = quarter<BACK>(v[1]), q3 = quarter<BACK>(v[3]);
        v[1] = {(v[1].x + q1.x) * c, (v[1].y + q1.y) * c};
        v[2] = quarter<BACK>(v[2]);
        v[3] = {(q3.x - v[3].x) * c, (q3.y - v[3].y) * c};
        dft<4, 1, BACK>(u);
        dft<4, 1, BACK>(v);
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            a[2 * m * S] = u[m];
            a[(2 * m + 1) * S] = v[m];
        }
    }
}

// LDS place of point i of a transform: one float of padding every eight, so
// that the lanes of every stage -- eight points apart in the innermost, runs of
// eight further out -- fall in different banks.
__device__ __forceinline__ int fft_at(int i) { return i + (i >> 3); }
// fft_at(i + m STEP), with the step's share a constant where it is one: for
// steps of whole blocks of eight, and for a step of 1 from a block's start.
template <int STEP>
__device__ __forceinline__ int fft_step(int at_i, int i, int m)
{
    if constexpr (STEP % 8 == 0)
        return at_i + m * (STEP / 8 * 9);
    else if constexpr (STEP == 1)
        return at_i + m;
    else
        return fft_at(i + m * STEP);
}
// LDS place of raw sample i of a column: blocks of eight, twelve floats apart,
// which keeps the FIR's four-float reads aligned and lanes eight samples apart
// in different banks.
__device__ __forceinline__ int raw_at(int i) { return i + (i >> 3) * 4; }

// Lanes that exchange data through LDS: within one wave its LDS instructions
// complete in order, so it is enough to keep the compiler from moving them.
template <bool WAVE>
__device__ __forceinline__ void exchange()
{
    if constexpr (WAVE) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

// exp(-2 pi i m t / N), m t < N, for one of a stage's R points: t is below N / R,
// so from m = R / 2 + 1 on the angle may pass the table's half circle.
template <int N, int R>
__device__ __forceinline__ float2 twiddle(const float2* __restrict__ tw, unsigned t, int m)
{
    unsigned i = t;
    for (int k = 1; k < m; ++k)      // sums: an integer product issues at a quarter of the rate
        i += t;
    if (m <= R / 2)
        return tw[i];
    const float2 w = tw[i & (N / 2 - 1)];
    const unsigned s = (i & (N / 2)) ? 0x80000000u : 0u;
    return make_float2(__builtin_bit_cast(float, __builtin_bit_cast(unsigned, w.x) ^ s),
                       __builtin_bit_cast(float, __builtin_bit_cast(unsigned, w.y) ^ s));
}

// The Hilbert transform's bins on the innermost stage: point m of `first`'s
// lane is bin m N/8 exactly, of the others a bin between m N/8 and
// (m + 1) N/8.  Bins below N/2 are turned by -i, above by +i; 0 and N/2 go.
template <int R>
__device__ __forceinline__ void hilbert_bins(Complex* a, bool first)
{
#pragma unroll
    for (int m = 0; m < R; ++m) {
        const Complex t = m < R / 2 ? quarter<false>(a[m]) : quarter<true>(a[m]);
        const bool drop = first && (m == 0 || m == R / 2);
        a[m] = {drop ? 0.f : t.x, drop ? 0.f : t.y};
    }
}

// The stages inside blocks of B points of an N-point transform and back: the
// points stand in LDS (re, im) on entry and on return.
template <int N, int B, bool WAVE>
__device__ __forceinline__ void inner_stages(float* re, float* im, int j, const float2* __restrict__ tw)
{
    constexpr int span = B / 8;
    const int pos = j % span, base = (j / span) * B + pos, at = fft_at(base);
    Complex a[8];
#pragma unroll
    for (int m = 0; m < 8; ++m)
        a[m] = {re[fft_step<span>(at, base, m)], im[fft_step<span>(at, base, m)]};
    dft<8, 1, false>(a);
    if constexpr (B == 8) {
        hilbert_bins<8>(a, j == 0);
    } else {
        float2 w[8];
#pragma unroll
        for (int m = 1; m < 8; ++m)
            w[m] = twiddle<N, 8>(tw, pos * (N / B), m);
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            if (m)
                a[m] = turn<false>(a[m], w[m]);
            re[fft_step<span>(at, base, m)] = a[m].x;
            im[fft_step<span>(at, base, m)] = a[m].y;
        }
        exchange<WAVE>();
        inner_stages<N, B / 8, WAVE>(re, im, j, tw);
        exchange<WAVE>();
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            a[m] = {re[fft_step<span>(at, base, m)], im[fft_step<span>(at, base, m)]};
            if (m)
                a[m] = turn<true>(a[m], w[m]);
        }
    }
    dft<8, 1, true>(a);
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        re[fft_step<span>(at, base, m)] = a[m].x;
        im[fft_step<span>(at, base, m)] = a[m].y;
    }
}

// Shape of the kernel for nz = 2^L: P points per lane, T lanes per pair of
// columns, the outermost stage of radix R0 (the others are of radix 8).
template <int L>
struct Shape {
    static constexpr int N = 1 << L;
    static constexpr int P = N < 8 ? N : 8;
    static constexpr int T = N / P;
    static constexpr int R0 = L <= 3 ? N : L % 3 == 0 ? 8 : 1 << (L % 3);
    // 256 threads: three to five workgroups per CU, so one's barriers pass under
    // another's arithmetic (512 threads, one per CU at its registers: 151 us a
    // pass of 16 images of 1024 x 1024 where 256 took 118)
    static constexpr int kMaxPairs = T >= 256 ? 1 : T > 16 ? 256 / T : 16;   // pairs per workgroup
    static constexpr int kMinPairs = T >= 64 ? 1 : 64 / T < 16 ? 64 / T : 16;
    static constexpr int kThreads = T * kMaxPairs < 64 ? 64 : T * kMaxPairs;
};

// LDS floats: one raw column, one transform's real or imaginary part, one
// output column; the three uses follow one another in the same memory.
constexpr int raw_floats(int n, int taps16) { return (((n + taps16) * 3 / 2 + 19) / 32) * 32 + 12; }
constexpr int fft_floats(int n) { return n + n / 8 + 1; }
constexpr int out_floats(int n, int cols) { return n + (cols < 64 ? 64 / cols : 1); }
constexpr size_t envelope_lds(int n, int taps16, int pairs)
{
    const int c = 2 * pairs;
    const int most = raw_floats(n, taps16) > fft_floats(n) ? raw_floats(n, taps16) : fft_floats(n);
    return sizeof(float) * (size_t)c * (most > out_floats(n, c) ? most : out_floats(n, c));
}

template <int L>
__global__ __launch_bounds__(Shape<L>::kThreads) void envelope_kernel(DisplayImages ims, int nx, int pairs,
                                                                     const float* __restrict__ taps, int numtaps,
                                                                     const float2* __restrict__ tw,
                                                                     float* __restrict__ block_max)
{
    using S = Shape<L>;
    constexpr int N = S::N, P = S::P, T = S::T, R0 = S::R0;
    constexpr bool kWave = T <= 64;        // a transform's lanes sit in one wave
    extern __shared__ __align__(16) float lds[];
    __shared__ float wave_max[(S::kThreads + 63) / 64];
    __shared__ int col_bits[T > 64 ? 2 * S::kMaxPairs * (T / 64) : 1];
    const float* __restrict__ image = ims.image[blockIdx.y];
    float* __restrict__ env = ims.env[blockIdx.y];
    const int tid = threadIdx.x, threads = T * pairs;      // blockDim.x, at least a wave
    // neighbouring groups of columns share memory lines: a contiguous run of
    // groups per XCD reads each line into one L2
    const int nb = gridDim.x, q0 = nb / kXcds, rem = nb % kXcds;
    const int xcd = blockIdx.x % kXcds;
    const int group = xcd * q0 + min(xcd, rem) + (int)blockIdx.x / kXcds;
    const int cols = 2 * pairs, lcols = 31 - __builtin_clz(cols);
    const int x0 = group * cols;
    const int nc = min(cols, nx - x0);     // columns of this group inside the image
    const int taps16 = (numtaps + 15) / 16 * 16, half = (numtaps - 1) / 2;
    const int rl = raw_floats(N, taps16);
    // the lane's pixels of a pass over the group's rows: its i-th is i * threads
    // on.  Images are read and written through buffer resources of their size,
    // so that columns past the image read as zero and are not written.
    auto row = [&](int i) { return (tid + i * threads) >> lcols; };
    auto col = [&](int i) { return (tid + i * threads) & (cols - 1); };
    const unsigned bytes = (unsigned)nx * N * 4u, past = 0xffffffffu;
    auto pixel = [&](int i) -> unsigned {
        return tid < threads && col(i) < nc ? ((unsigned)row(i) * (unsigned)nx + (unsigned)(x0 + col(i))) * 4u : past;
    };
    // with two lanes or more per pair a lane stays in its column, T / 2 rows
    // further on each time: one offset, and a scalar step
    const unsigned pixel0 = pixel(0), step = (unsigned)(T / 2) * (unsigned)nx * 4u;

    // 1. raw samples, row by row (the group's columns of a row are adjacent):
    //    sample z of a column at z + half, zeros before and after
    const int block = blockDim.x;
    for (int q = tid; q < taps16 << lcols; q += block) {
        const int i = q >> lcols, c = q & (cols - 1);
        lds[c * rl + raw_at(i < half ? i : i + N)] = 0.f;
    }
    {
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(image), (short)0, (int)bytes, kBufferFlags);
        float v[2 * P];
#pragma unroll
        for (int i = 0; i < 2 * P; ++i)
            v[i] = __builtin_bit_cast(float, T >= 2 ? __builtin_amdgcn_raw_buffer_load_b32(rs, (int)pixel0, (int)(i * step), 0)
                                                    : __builtin_amdgcn_raw_buffer_load_b32(rs, (int)pixel(i), 0, 0));
        const int at0 = col(0) * rl + raw_at(row(0) + half);
#pragma unroll
        for (int i = 0; i < 2 * P; ++i) {
            if (tid < threads)
                lds[T >= 16 ? at0 + i * (T / 2 * 3 / 2) : col(i) * rl + raw_at(row(i) + half)] = v[i];
        }
    }
    __syncthreads();
    // 2. centred FIR along depth: lane j of a pair forms samples P j .. P j + P - 1
    //    of both columns
    const int g = min(tid / T, pairs - 1), j = tid % T;
    Complex a[P];
    {
        // the taps that meet a sample: in a column shorter than the filter, not all
        // (one column of 8 samples, 255 taps: 22.6 us a pass with all of them, 13.3 so)
        const int first = N <= kMaxTaps / 2 ? max(0, half - N + 1) : 0;
        const int last = N <= kMaxTaps / 2 ? min(numtaps, half + N) : numtaps;
        const float* ra = lds + 2 * g * rl;
        const float* rb = ra + rl;
#pragma unroll
        for (int r = 0; r < P; ++r)
            a[r] = {0.f, 0.f};
        if constexpr (P == 8) {
            float wa[2][8], wb[2][8];      // the window: two blocks of eight samples
            auto load8 = [](float (&w)[8], const float* r) {
                const float4 lo = *reinterpret_cast<const float4*>(r), hi = *reinterpret_cast<const float4*>(r + 4);
                w[0] = lo.x, w[1] = lo.y, w[2] = lo.z, w[3] = lo.w;
                w[4] = hi.x, w[5] = hi.y, w[6] = hi.z, w[7] = hi.w;
            };
            const int b0 = first / 16 * 16;
            ra += 12 * j + b0 / 8 * 12;
            rb += 12 * j + b0 / 8 * 12;
            load8(wa[0], ra);
            load8(wb[0], rb);
            for (int b = b0; b < last; b += 16) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    ra += 12;
                    rb += 12;
                    load8(wa[1 - h], ra);
                    load8(wb[1 - h], rb);
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        // in a vector register: an FMA that reads a scalar one
                        // issues at half the rate
                        float t;
                        asm("v_mov_b32 %0, %1" : "=v"(t) : "s"(taps[b + 8 * h + k]));
#pragma unroll
                        for (int r = 0; r < 8; ++r) {
                            a[r].x = __builtin_fmaf(t, r + k < 8 ? wa[h][r + k] : wa[1 - h][r + k - 8], a[r].x);
                            a[r].y = __builtin_fmaf(t, r + k < 8 ? wb[h][r + k] : wb[1 - h][r + k - 8], a[r].y);
                        }
                    }
                }
            }
        } else {
            for (int k = first; k < last; ++k) {
#pragma unroll
                for (int r = 0; r < P; ++r) {
                    a[r].x = __builtin_fmaf(taps[k], ra[raw_at(P * j + r + k)], a[r].x);
                    a[r].y = __builtin_fmaf(taps[k], rb[raw_at(P * j + r + k)], a[r].y);
                }
            }
        }
    }
    // 3. each column scaled by a power of two to about 1 for the transform, so
    //    that one column's rounding stays below its neighbour's own however
    //    much brighter it is; a column of zeros stays one; a column that is not
    //    finite goes in as zeros (and comes out as NaN) and leaves its
    //    neighbour alone
    int ma = 0, mb = 0;
#pragma unroll
    for (int r = 0; r < P; ++r) {
        ma = max(ma, __builtin_bit_cast(int, __builtin_fabsf(a[r].x)));
        mb = max(mb, __builtin_bit_cast(int, __builtin_fabsf(a[r].y)));
    }
#pragma unroll
    for (int off = (T < 64 ? T : 64) / 2; off >= 1; off >>= 1) {
        ma = max(ma, __shfl_xor(ma, off));
        mb = max(mb, __shfl_xor(mb, off));
    }
    if constexpr (T > 64) {
        constexpr int W = T / 64;          // waves of a transform
        if (tid % 64 == 0) {
            col_bits[2 * (tid / 64)] = ma;
            col_bits[2 * (tid / 64) + 1] = mb;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < W; ++w) {
            ma = max(ma, col_bits[2 * (g * W + w)]);
            mb = max(mb, col_bits[2 * (g * W + w) + 1]);
        }
    }
    const bool na = ma >= 0x7f800000, nb_ = mb >= 0x7f800000;
    const int ea = min(max(ma >> 23, 1), 253), eb = min(max(mb >> 23, 1), 253);
    const float sa = na ? 0.f : __builtin_bit_cast(float, (254 - ea) << 23);
    const float sb = nb_ ? 0.f : __builtin_bit_cast(float, (254 - eb) << 23);
    const float ua = na ? __builtin_nanf("") : ma ? __builtin_bit_cast(float, ea << 23) : 0.f;
    const float ub = nb_ ? __builtin_nanf("") : mb ? __builtin_bit_cast(float, eb << 23) : 0.f;
    float* re = lds + 2 * g * fft_floats(N);
    float* im = re + fft_floats(N);
    const int at = fft_at(j), at8 = fft_at(P * j);
    __syncthreads();                       // the raw samples are read
#pragma unroll
    for (int r = 0; r < P; ++r) {
        re[P == 8 ? at8 + r : fft_at(P * j + r)] = na ? 0.f : a[r].x * sa;
        im[P == 8 ? at8 + r : fft_at(P * j + r)] = nb_ ? 0.f : a[r].y * sb;
    }
    exchange<kWave>();
    // 4. Hilbert transform of both columns: lane j holds points j, j + T, ..
    Complex x[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
        x[i] = {re[fft_step<T>(at, j, i)], im[fft_step<T>(at, j, i)]};
        a[i] = x[i];
    }
    if constexpr (R0 == N) {
        dft<R0, 1, false>(a);
        hilbert_bins<R0>(a, true);
        dft<R0, 1, true>(a);
    } else {
        constexpr int Q = P / R0;          // butterflies of the outermost stage per lane
        float2 w[P];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            dft<R0, Q, false>(a + q);
#pragma unroll
            for (int m = 1; m < R0; ++m) {
                w[q + m * Q] = twiddle<N, R0>(tw, j + q * T, m);
                a[q + m * Q] = turn<false>(a[q + m * Q], w[q + m * Q]);
            }
        }
#pragma unroll
        for (int i = 0; i < P; ++i) {
            re[fft_step<T>(at, j, i)] = a[i].x;
            im[fft_step<T>(at, j, i)] = a[i].y;
        }
        exchange<kWave>();
        inner_stages<N, N / R0, kWave>(re, im, j, tw);
        exchange<kWave>();
#pragma unroll
        for (int q = 0; q < Q; ++q) {
#pragma unroll
            for (int m = 0; m < R0; ++m) {
                const int i = q + m * Q;
                a[i] = {re[fft_step<T>(at, j, i)], im[fft_step<T>(at, j, i)]};
                if (m)
                    a[i] = turn<true>(a[i], w[i]);
            }
            dft<R0, Q, true>(a + q);
        }
    }
    // 5. envelope, back to rows through LDS, and this workgroup's maximum
    const int ol = out_floats(N, cols);
    constexpr float inv_n = 1.f / N;
    float m = 0.f;
    __syncthreads();                       // the transforms are read
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const float ha = a[i].x * inv_n, hb = a[i].y * inv_n;
        const float va = ua * __builtin_amdgcn_sqrtf(__builtin_fmaf(x[i].x, x[i].x, ha * ha));
        const float vb = ub * __builtin_amdgcn_sqrtf(__builtin_fmaf(x[i].y, x[i].y, hb * hb));
        if (tid < threads) {
            lds[2 * g * ol + j + i * T] = va;
            lds[(2 * g + 1) * ol + j + i * T] = vb;
            m = fmaxf(m, fmaxf(va, vb));   // columns past the image are zeros
        }
    }
    __syncthreads();
    const __amdgpu_buffer_rsrc_t out =
        __builtin_amdgcn_make_buffer_rsrc(env, (short)0, (int)bytes, kBufferFlags);
#pragma unroll
    for (int i = 0; i < 2 * P; ++i) {
        if constexpr (T >= 2)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, lds[col(0) * ol + row(0) + i * (T / 2)]),
                                                  out, (int)pixel0, (int)(i * step), 0);
        else if (tid < threads)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, lds[col(i) * ol + row(i)]), out,
                                                  (int)pixel(i), 0, 0);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        m = fmaxf(m, __shfl_xor(m, off));
    if ((tid & 63) == 0)
        wave_max[tid >> 6] = m;
    __syncthreads();
    if (tid == 0) {
        float bm = 0.f;
        for (int w = 0; w < (block + 63) / 64; ++w)
            bm = fmaxf(bm, wave_max[w]);
        block_max[(int64_t)blockIdx.y * nb + blockIdx.x] = bm;
    }
}

using EnvelopeFn = void (*)(DisplayImages, int, int, const float*, int, const float2*, float*);

template <int L>
constexpr void fill_envelopes(EnvelopeFn* fn, int* lanes, int* most, int* least)
{
    fn[L] = envelope_kernel<L>;
    lanes[L] = Shape<L>::T;
    most[L] = Shape<L>::kMaxPairs;
    least[L] = Shape<L>::kMinPairs;
    if constexpr (L < kMaxLog2Nz)
        fill_envelopes<L + 1>(fn, lanes, most, least);
}

// The envelope kernels by log2 nz, with their lanes per pair and the range of
// pairs per workgroup.
struct Envelopes {
    EnvelopeFn fn[kMaxLog2Nz + 1] = {};
    int lanes[kMaxLog2Nz + 1] = {}, most[kMaxLog2Nz + 1] = {}, least[kMaxLog2Nz + 1] = {};
    Envelopes() { fill_envelopes<1>(fn, lanes, most, least); }
};
const Envelopes& envelopes()
{
    static const Envelopes e;
    return e;
}

// 20 log10 r = (20 log10 2) log2 r, the hardware's log2 and the product in two
// parts of the constant.
__device__ __forceinline__ float decibels(float e, float inv_peak, float floor_db)
{
    constexpr float hi = 6.02059991f, lo = (float)(6.0205999132796239 - (double)6.02059991f);
    const float r = e * inv_peak;
    const bool tiny = r < 1.17549435e-38f;       // the hardware's log2 takes no denormals
    const float l = __builtin_amdgcn_logf(tiny ? r * 0x1p32f : r) - (tiny ? 32.f : 0.f);
    const float v = __builtin_fmaf(hi, l, lo * l);
    return r > 0.f ? fmaxf(v, floor_db) : floor_db;
}

__global__ __launch_bounds__(kDispBlock) void log_compress_kernel(DisplayImages ims, int64_t count,
                                                                  const float* __restrict__ block_max,
                                                                  int n_blocks, float dyn_range_db)
{
    __shared__ float part[kDispBlock / 64];
    const float* env = ims.env[blockIdx.y];
    float* db = ims.db[blockIdx.y];
    block_max += (int64_t)blockIdx.y * n_blocks;
    float m = 0.f;
    for (int i = threadIdx.x; i < n_blocks; i += kDispBlock)
        m = fmaxf(m, block_max[i]);
    for (int off = 32; off >= 1; off >>= 1)
        m = fmaxf(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0)
        part[threadIdx.x >> 6] = m;
    __syncthreads();
    float peak = 0.f;
    for (int w = 0; w < kDispBlock / 64; ++w)
        peak = fmaxf(peak, part[w]);
    const float floor_db = -dyn_range_db;
    // a peak below the normal numbers, whose reciprocal may overflow, and its
    // pixels are scaled by a power of two first
    const float up = peak < 0x1p-126f ? 0x1p100f : 1.f;
    const float inv_peak = peak > 0.f ? 1.f / (peak * up) : 0.f;
    // four pixels per lane where both buffers are aligned for it
    const bool wide = ((reinterpret_cast<uintptr_t>(env) | reinterpret_cast<uintptr_t>(db)) & 15) == 0;
    const int64_t step = (int64_t)gridDim.x * kDispBlock;
    const int64_t first = (int64_t)blockIdx.x * kDispBlock + threadIdx.x;
    const int64_t quads = wide ? count / 4 : 0;
    for (int64_t i = first; i < quads; i += step) {
        const float4 e = reinterpret_cast<const float4*>(env)[i];
        reinterpret_cast<float4*>(db)[i] =
            make_float4(decibels(e.x * up, inv_peak, floor_db), decibels(e.y * up, inv_peak, floor_db),
                        decibels(e.z * up, inv_peak, floor_db), decibels(e.w * up, inv_peak, floor_db));
    }
    for (int64_t i = 4 * quads + first; i < count; i += step)
        db[i] = decibels(env[i] * up, inv_peak, floor_db);
}

// ---------------------------------------------------------------------------
// Allocation-free form (hodmas_display_run_static).  Its band-pass taps, FFT
// twiddles and per-workgroup envelope maxima live in this file-scope device
// array instead of buffers a plan allocates.  Every GPU the library runs on
// holds its own copy until the process ends; host code reaches it only
// through the address hipGetSymbolAddress returns for that device.
constexpr int kStaticTapFloats = kTapFloats;            // taps (numtaps <= 255), zeros after them
constexpr int kStaticTwiddles = kMaxNz / 2;             // float2 twiddles
constexpr int kStaticMaxBlocks = 65536;                 // one maximum per workgroup (nx <= 65536)
constexpr size_t kStaticTwiddleOffset = sizeof(float) * kStaticTapFloats;
constexpr size_t kStaticBlockMaxOffset = kStaticTwiddleOffset + sizeof(float2) * kStaticTwiddles;
constexpr size_t kStaticScratchBytes = kStaticBlockMaxOffset + sizeof(float) * kStaticMaxBlocks;
static_assert(kStaticTwiddleOffset % 8 == 0 && kStaticBlockMaxOffset % 4 == 0, "scratch regions aligned");

__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// Pairs of columns per envelope workgroup: as many as a workgroup takes --
// whole memory lines of a row, few maxima -- but few enough that the launch
// gives every CU a workgroup.
int display_pairs(int nx, int log2n, int images, int cus)
{
    const Envelopes& e = envelopes();
    int p = e.most[log2n];
    while (p > e.least[log2n] && (int64_t)((nx + 2 * p - 1) / (2 * p)) * images < cus)
        p /= 2;
    return p;
}
// The most workgroups of a launch (their maxima).
int display_blocks(int nx, int log2n)
{
    const int least = envelopes().least[log2n];
    return (nx + 2 * least - 1) / (2 * least);
}
// Lets the kernel of log2 nz use the LDS its largest workgroup needs.
bool allow_lds(int log2n)
{
    const Envelopes& e = envelopes();
    const size_t most = envelope_lds(1 << log2n, kTapFloats, e.most[log2n]);
    return most <= 64 * 1024 || hipFuncSetAttribute((const void*)e.fn[log2n],
                                                    hipFuncAttributeMaxDynamicSharedMemorySize,
                                                    (int)most) == hipSuccess;
}

struct StaticTaps {
    float v[kMaxTaps];
};

// The taps (from the kernel arguments) and the twiddles exp(-2 pi i t / nz),
// t < nz / 2, evaluated in float64 and rounded to float as the plan does.
__global__ __launch_bounds__(kDispBlock) void static_tables_kernel(StaticTaps taps, int numtaps, int nz,
                                                                   float* __restrict__ d_taps,
                                                                   float2* __restrict__ d_tw)
{
    const int i = blockIdx.x * kDispBlock + threadIdx.x;
    if (i < kStaticTapFloats)
        d_taps[i] = i < numtaps ? taps.v[i] : 0.f;
    if (i < nz / 2) {
        double sn, cs;
        sincospi(-2.0 * double(i) / double(nz), &sn, &cs);
        d_tw[i] = make_float2((float)cs, (float)sn);
    }
}

}  // namespace

struct hodmas_display_s {
    uint32_t magic = kDisplayMagic;
    hodmas_display_desc desc{};
    int log2n = 0, cus = 256, device = -1;
    float* d_taps = nullptr;
    float2* d_tw = nullptr;
    float* d_block_max = nullptr;
};

extern "C" {

hodmas_status hodmas_display_taps(const hodmas_display_desc* d, double* taps)
{
    if (!d || !taps)
        return HODMAS_EINVAL;
    const int nt = d->numtaps;
    if (nt < 1 || nt > kMaxTaps || nt % 2 == 0 || !(d->dz_m > 0.0) || !(d->sound_speed_m_s > 0.0))
        return HODMAS_EINVAL;
    const double fs = d->sound_speed_m_s / d->dz_m;     // one-way flight: dz is dz/c seconds
    if (!(d->f_lo_hz > 0.0 && d->f_lo_hz < d->f_hi_hz && d->f_hi_hz < 0.5 * fs))
        return HODMAS_EINVAL;
    // difference of two Hamming-windowed ideal low-pass responses, scaled to
    // unit gain at the centre of the pass band
    const double lo = d->f_lo_hz / fs, hi = d->f_hi_hz / fs, mid = 0.5 * (nt - 1);
    const double pi = 3.14159265358979323846;
    auto sinc = [pi](double x) { return x == 0.0 ? 1.0 : std::sin(pi * x) / (pi * x); };
    double gain = 0.0;
    for (int k = 0; k < nt; ++k) {
        const double m = k - mid;
        double h = 2.0 * hi * sinc(2.0 * hi * m) - 2.0 * lo * sinc(2.0 * lo * m);
        if (nt > 1)
            h *= 0.54 - 0.46 * std::cos(2.0 * pi * k / (nt - 1));
        taps[k] = h;
        gain += h * std::cos(pi * (lo + hi) * m);
    }
    for (int k = 0; k < nt; ++k)
        taps[k] /= gain;
    return HODMAS_OK;
}

hodmas_status hodmas_display_plan(const hodmas_display_desc* d, hodmas_display_t* out)
{
    if (!d || !out)
        return HODMAS_EINVAL;
    *out = nullptr;
    if (d->nx < 1 || d->nz < 2 || d->nz > kMaxNz || (d->nz & (d->nz - 1)) != 0 || d->nx > 65536 ||
        !(d->dynamic_range_db > 0.f))
        return HODMAS_EINVAL;
    std::vector<double> taps(kMaxTaps);
    hodmas_status st = hodmas_display_taps(d, taps.data());
    if (st != HODMAS_OK)
        return st;
    hodmas_display_s* p = new (std::nothrow) hodmas_display_s;
    if (!p)
        return HODMAS_ENOMEM;
    p->desc = *d;
    while ((1 << p->log2n) < d->nz)
        ++p->log2n;
    {
        int dev = 0;
        hipDeviceProp_t prop;
        if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess)
            p->cus = prop.multiProcessorCount;
    }
    std::vector<float> ft(kTapFloats, 0.f);
    for (int k = 0; k < d->numtaps; ++k)
        ft[k] = (float)taps[k];
    std::vector<float2> tw(d->nz / 2);
    for (int t = 0; t < d->nz / 2; ++t) {
        const double a = -2.0 * 3.14159265358979323846 * t / d->nz;
        tw[t] = make_float2((float)std::cos(a), (float)std::sin(a));
    }
    const size_t maxima = sizeof(float) * (size_t)display_blocks(d->nx, p->log2n) * kDisplayBatch;
    bool ok = hipGetDevice(&p->device) == hipSuccess && allow_lds(p->log2n) &&
              hipMalloc((void**)&p->d_taps, sizeof(float) * ft.size()) == hipSuccess &&
              hipMalloc((void**)&p->d_tw, sizeof(float2) * tw.size()) == hipSuccess &&
              hipMalloc((void**)&p->d_block_max, maxima) == hipSuccess &&
              hipMemcpy(p->d_taps, ft.data(), sizeof(float) * ft.size(), hipMemcpyHostToDevice) == hipSuccess &&
              hipMemcpy(p->d_tw, tw.data(), sizeof(float2) * tw.size(), hipMemcpyHostToDevice) == hipSuccess;
    if (!ok) {
        (void)hipGetLastError();
        hodmas_display_destroy(p);
        return HODMAS_ENOMEM;
    }
    *out = p;
    return HODMAS_OK;
}

}  // extern "C"

namespace {

// Launch the chain for n <= kDisplayBatch images of one shape.
hipError_t launch_display(const hodmas_display_desc& d, int log2n, int cus, const float* taps, const float2* tw,
                          float* block_max, const DisplayImages& ims, int n, hipStream_t st)
{
    const int pairs = display_pairs(d.nx, log2n, n, cus);
    const int n_blocks = (d.nx + 2 * pairs - 1) / (2 * pairs);
    const int threads = std::max(64, envelopes().lanes[log2n] * pairs);
    const size_t lds = envelope_lds(d.nz, (d.numtaps + 15) / 16 * 16, pairs);
    hipLaunchKernelGGL(envelopes().fn[log2n], dim3(n_blocks, n), dim3(threads), lds, st, ims, d.nx, pairs, taps,
                       d.numtaps, tw, block_max);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        const int64_t count = (int64_t)d.nx * d.nz;
        const int grid = (int)std::min<int64_t>((count + 4 * kDispBlock - 1) / (4 * kDispBlock), 4096);
        hipLaunchKernelGGL(log_compress_kernel, dim3(grid, n), dim3(kDispBlock), 0, st, ims, count, block_max,
                           n_blocks, d.dynamic_range_db);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace

extern "C" {

hodmas_status hodmas_display_run_batch(hodmas_display_t p, const float* const* images_dev,
                                       float* const* envelopes_dev, float* const* dbs_dev, int32_t n,
                                       void* stream)
{
    if (!p || p->magic != kDisplayMagic || !images_dev || !dbs_dev || n < 1)
        return HODMAS_EINVAL;
    for (int32_t i = 0; i < n; ++i) {
        const float* env = envelopes_dev ? envelopes_dev[i] : nullptr;
        if (!images_dev[i] || !dbs_dev[i] || images_dev[i] == dbs_dev[i] || images_dev[i] == env)
            return HODMAS_EINVAL;
    }
    int cur = -1;
    if (hipGetDevice(&cur) != hipSuccess)
        return HODMAS_EDEVICE;
    if (cur != p->device && hipSetDevice(p->device) != hipSuccess)
        return HODMAS_EDEVICE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t e = hipSuccess;
    for (int32_t i0 = 0; i0 < n && e == hipSuccess; i0 += kDisplayBatch) {
        const int m = std::min<int32_t>(kDisplayBatch, n - i0);
        DisplayImages ims{};
        for (int j = 0; j < m; ++j) {
            float* env = envelopes_dev ? envelopes_dev[i0 + j] : nullptr;
            ims.image[j] = images_dev[i0 + j];
            ims.db[j] = dbs_dev[i0 + j];
            ims.env[j] = env ? env : dbs_dev[i0 + j];     // the dB pass then works in place
        }
        e = launch_display(p->desc, p->log2n, p->cus, p->d_taps, p->d_tw, p->d_block_max, ims, m, st);
    }
    if (cur != p->device)
        (void)hipSetDevice(cur);
    return e == hipSuccess ? HODMAS_OK : HODMAS_EDEVICE;
}

hodmas_status hodmas_display_run(hodmas_display_t p, const float* image_dev, float* envelope_dev, float* db_dev,
                                 void* stream)
{
    return hodmas_display_run_batch(p, &image_dev, envelope_dev ? &envelope_dev : nullptr, &db_dev, 1, stream);
}

}  // extern "C"

namespace {

constexpr int kMaxDevices = 64;

struct StaticDevice {
    bool ready = false;
    void* scratch = nullptr;      // device address of `scratch` on this device
    int cus = 256;
};

std::mutex g_static_mu;
StaticDevice g_static[kMaxDevices];

// First call on a device: the device address of its scratch array, its CU
// count, and the LDS limit of the envelope kernel.  Returns null on failure.
const StaticDevice* static_device(int dev)
{
    if (dev < 0 || dev >= kMaxDevices)
        return nullptr;
    std::lock_guard<std::mutex> lock(g_static_mu);
    StaticDevice& sd = g_static[dev];
    if (!sd.ready) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return nullptr;
        }
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
        for (int l = 1; l <= kMaxLog2Nz; ++l) {
            if (!allow_lds(l)) {
                (void)hipGetLastError();
                return nullptr;
            }
        }
        sd.scratch = ptr;
        sd.cus = prop.multiProcessorCount;
        sd.ready = true;
    }
    return &sd;
}

}  // namespace

extern "C" {

hodmas_status hodmas_display_run_static(const hodmas_display_desc* d, const float* image_dev, float* envelope_dev,
                                        float* db_dev, void* stream)
{
    if (!d || !image_dev || !db_dev || image_dev == db_dev || image_dev == envelope_dev)
        return HODMAS_EINVAL;
    if (d->nx < 1 || d->nz < 2 || d->nz > kMaxNz || (d->nz & (d->nz - 1)) != 0 || !(d->dynamic_range_db > 0.f))
        return HODMAS_EINVAL;
    if (d->nx > kStaticMaxBlocks)
        return HODMAS_EUNSUPPORTED;             // more workgroup maxima than the scratch array holds
    double taps[kMaxTaps];
    const hodmas_status tst = hodmas_display_taps(d, taps);
    if (tst != HODMAS_OK)
        return tst;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess)
        return HODMAS_EDEVICE;
    const StaticDevice* sd = static_device(dev);
    if (!sd)
        return HODMAS_EDEVICE;
    int log2n = 0;
    while ((1 << log2n) < d->nz)
        ++log2n;
    if (display_blocks(d->nx, log2n) > kStaticMaxBlocks)
        return HODMAS_EUNSUPPORTED;
    StaticTaps ft;
    for (int k = 0; k < kMaxTaps; ++k)
        ft.v[k] = k < d->numtaps ? (float)taps[k] : 0.f;
    unsigned char* base = static_cast<unsigned char*>(sd->scratch);
    float* d_taps = reinterpret_cast<float*>(base);
    float2* d_tw = reinterpret_cast<float2*>(base + kStaticTwiddleOffset);
    float* d_block_max = reinterpret_cast<float*>(base + kStaticBlockMaxOffset);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int n_tab = std::max(kStaticTapFloats, d->nz / 2);
    hipLaunchKernelGGL(static_tables_kernel, dim3((n_tab + kDispBlock - 1) / kDispBlock), dim3(kDispBlock), 0, st,
                       ft, d->numtaps, d->nz, d_taps, d_tw);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        DisplayImages ims{};
        ims.image[0] = image_dev;
        ims.db[0] = db_dev;
        ims.env[0] = envelope_dev ? envelope_dev : db_dev;
        e = launch_display(*d, log2n, sd->cus, d_taps, d_tw, d_block_max, ims, 1, st);
    }
    return e == hipSuccess ? HODMAS_OK : HODMAS_EDEVICE;
}

hodmas_status hodmas_display_destroy(hodmas_display_t p)
{
    if (!p)
        return HODMAS_OK;
    if (p->magic != kDisplayMagic)
        return HODMAS_EINVAL;
    if (p->d_taps) (void)hipFree(p->d_taps);
    if (p->d_tw) (void)hipFree(p->d_tw);
    if (p->d_block_max) (void)hipFree(p->d_block_max);
    p->magic = 0;
    delete p;
    return HODMAS_OK;
}

}  // extern "C"
