// Fused HO-DMAS beamforming kernel for gfx950 (MI355X).
//
// One workgroup (4 wave64) forms one pixel tile.  Per pixel and element it
//   1. rebuilds the one-way delay from the tile's float64 anchor (registers),
//   2. gathers the two neighbouring samples from an LDS window that the
//      workgroup staged with coalesced channel-major loads, and interpolates,
//   3. takes the signed k-th root y = sign(s)|s|^(1/k)       (Eq. 2, Eqs. 4-6),
//   4. accumulates the power sums p_j = sum y^j, j = 1..k, with compensated
//      float32 summation (groups of four, Kahan steps per 32 elements),
// and per pixel recovers the order-k symmetric sum e_k from p_1..p_k with
// Newton's identities (the general form of Eqs. 3, 7, 8 and 9):
//   e_0 = 1,  m e_m = sum_{j=1..m} (-1)^(j-1) e_{m-j} p_j.
// The recovery runs in float32 for k <= 4 and in float64 for k >= 5, where the
// alternating terms cancel more.  y^k is taken as the sample itself (odd k) or
// its magnitude (even k), exactly as the paper's forms use sum s and sum |s|.
//
// Per-element constants are wave-uniform (every lane of a wave works on the same
// element at the same time), so they live in SGPRs via scalar loads; the
// per-pixel state lives in VGPRs.  No MFMA: this is gather + VALU work.
// Template parameter M = 2 pairs each pixel with its mirror image about x = 0
// (one delay serves both; see process_tile).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "hodmas_internal.h"

namespace hodmas {
namespace {

// Read-only tables; wave-uniform indices let the compiler use scalar loads.
using ConstTile = const hodmas_tile_desc* __restrict__;
using ConstEntry = const hodmas_chan_entry* __restrict__;
using ConstStage = const hodmas_stage_entry* __restrict__;

// The tables and work lists are never written by a kernel.  Their elements
// are read through the constant address space, which says so: loads at
// wave-uniform addresses then become scalar loads even after the kernel has
// stored to global memory (the batch kernels store a tile's pixels before
// reading the next tile's entries), and pointers that were themselves read
// from memory are not left as flat pointers.  The copy goes dword by dword
// (every table record is a whole number of dwords).
template <class T>
__device__ __forceinline__ T load_const(const T* base, int64_t index)
{
    static_assert(sizeof(T) % 4 == 0, "table records are whole dwords");
    using CP = const __attribute__((address_space(4))) int*;
    const CP p = (CP)(const void*)(base + index);
    T out;
    int* o = reinterpret_cast<int*>(&out);
#pragma unroll
    for (int i = 0; i < int(sizeof(T) / 4); ++i)
        o[i] = p[i];
    return out;
}

// RF records and images live in global memory; saying so keeps accesses
// through pointers read from a work list global rather than flat (flat loads
// also count against the LDS wait counter).
template <class T>
using Global = __attribute__((address_space(1))) T*;
template <class T>
__device__ __forceinline__ Global<T> global_ptr(T* p)
{
    return (Global<T>)p;
}

// Word 3 of a raw (stride 0) buffer resource on gfx950: 32-bit data format,
// no swizzle; with stride 0 an access is in range iff its byte offset is below
// the resource's size.
constexpr int kBufferFlags = 0x00020000;

// Kahan step: s + x with the running compensation c (true sum ~ s - c).
__device__ __forceinline__ void kahan_add(float& s, float& c, float x)
{
    float y = x - c;
    float t = s + y;
    c = (t - s) - y;
    s = t;
}

// Where one element's delayed sample sits in the LDS window for this lane's
// pixel: t = delay - floor(anchor delay), its fraction f and the LDS index.
// d^2 - d0^2 comes from one FMA on per-pixel terms; d - d0 = (d^2 - d0^2)/(d + d0).
struct Tap {
    float t, f;
    int addr;    // LDS byte address of the sample before the delay
};

__device__ __forceinline__ Tap locate_at(const hodmas_chan_entry& e, float u2, float q, int off)
{
    Tap p;
    const float num = __builtin_fmaf(u2, e.a, q);
    const float d = __builtin_amdgcn_sqrtf(__builtin_fabsf(e.d0sq + num));
    const float r = __builtin_amdgcn_rcpf(d + e.d0);
    p.t = __builtin_fmaf(num, r, e.frac0);
    // floor(t) as an integer in one instruction (the compiler emits a floor and
    // a conversion), and t - floor(t), which is exact in float32, so fract
    // returns it unchanged
    int fl;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(fl) : "v"(p.t));
    p.f = __builtin_amdgcn_fractf(p.t);
    p.addr = (fl << 2) + off;
    return p;
}

__device__ __forceinline__ Tap locate(const hodmas_chan_entry& e, float u2, float q)
{
    return locate_at(e, u2, q, e.off);
}

// Delays shared along translated pixels.  When the element pitch of a uniform
// linear array is SH pixel columns, the pixel in column x sees element i + 1
// at exactly the delay at which the pixel in column x - SH sees element i
// (Eq. 1 depends on the pixel's x minus the element's x only).  The 16 lanes
// of a tile row are 16 neighbouring columns, so for elements i + s, s = 1..3,
// a lane takes element i's delay from the lane s*SH columns to its left -- or,
// in the row's first s*SH lanes, from F: element i + 3's delay at the pixel
// 16 - 3*SH columns to the left, which is also element i + 4's at the lane's
// own pixel (the next group's first element).  A group of four elements then
// computes one delay per lane instead of four, and passes the others between
// the lanes of a row through 32 entries of an LDS buffer: F in entries [0, 16),
// element i's own delays in [16, 32), so element i + s of lane j is entry
// 16 + j - s*SH.  The shared quantities are 4 floor(delay) as an absolute
// sample index and the fraction; each element adds the byte offset that its
// LDS row gives sample 0.
// Rows' buffers are 48 entries apart: a 64-bit LDS access serves 32 lanes --
// two rows -- at once, and 16 entries of one row fill half the banks, so the
// neighbouring row's entries start half the banks (128 bytes) further on.
constexpr int kRowEntries = 48;

struct alignas(8) XF {     // one 64-bit LDS access per entry
    int x;      // 4 floor(delay), absolute sample index
    float f;    // fraction of the delay
};

struct Shared {
    int x;      // the group's first element at the lane's pixel
    float f;
    int fx;     // F: the next group's first element at the lane's pixel
    float ff;
    XF* buf;    // the lane's entry j of its row's buffer
};

// Orders the LDS accesses of one wave that exchange data between its lanes:
// a wave's LDS instructions complete in issue order, so keeping the compiler
// from moving them across this point is all that is needed.
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Byte offset of sample 0 in the LDS rows of four consecutive staged slots
// (slot, ..., slot + 3 of the chunk whose staging entries start at S): the
// sample at absolute index j of slot m sits at 4 j + ro[m].
__device__ __forceinline__ void load_rowoff(ConstStage S, int slot, int stride, int (&ro)[4])
{
#pragma unroll
    for (int m = 0; m < 4; ++m)
        ro[m] = 4 * ((slot + m) * stride - load_const(S, slot + m).first_sample);
}

// Tiles whose delays may leave the record (CHECK): a delay outside [lo, hi]
// -- before the first sample or past the last -- contributes nothing, so its
// address is pointed at a pair of zeros the staging keeps after the rows
// (`zero`, bytes) and the interpolation yields exactly 0.
__device__ __forceinline__ void redirect(Tap& p, const hodmas_chan_entry& e, int zero)
{
    p.addr = (p.t >= e.lo && p.t <= e.hi) ? p.addr : zero;
}

__device__ __forceinline__ float lds_at(const float* __restrict__ lds, int addr)
{
    return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(lds) + addr);
}

// Linear interpolation between the two staged samples.  HALF: the LDS words
// hold FP16 samples in their low halves (rows copied straight from an FP16
// record); the mixed-precision FMA widens them, exactly, as it interpolates,
// in the same two instructions.
template <bool HALF = false>
__device__ __forceinline__ float interp(const Tap& p, float s0, float s1)
{
    if constexpr (HALF) {
        const float h0 = (float)__builtin_bit_cast(_Float16, (unsigned short)__builtin_bit_cast(unsigned, s0));
        const float h1 = (float)__builtin_bit_cast(_Float16, (unsigned short)__builtin_bit_cast(unsigned, s1));
        return __builtin_fmaf(p.f, h1, __builtin_fmaf(-p.f, h0, h0));
    } else {
        return __builtin_fmaf(p.f, s1 - s0, s0);
    }
}

// The K-th root of a = |v|: square roots for K = 2 and 4, else 2^(log2 a / K),
// where a = 0 gives 2^-inf = 0; and its square.
template <int K>
__device__ __forceinline__ float root(float a)
{
    if constexpr (K == 1)
        return a;
    else if constexpr (K == 2)
        return __builtin_amdgcn_sqrtf(a);
    else if constexpr (K == 4)
        return __builtin_amdgcn_sqrtf(__builtin_amdgcn_sqrtf(a));
    else
        return __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(a) * (1.0f / K));
}
template <int K>
__device__ __forceinline__ float root_squared(float a, float r)
{
    if constexpr (K == 2)
        return a;
    else if constexpr (K == 4)
        return __builtin_amdgcn_sqrtf(a);
    else
        return r * r;
}

// y^1 .. y^K of the signed K-th root of v.
template <int K>
__device__ __forceinline__ void powers(float v, float (&T)[K])
{
    const float a = __builtin_fabsf(v);
    const float r = root<K>(a), r2 = root_squared<K>(a, r);
    T[0] = __builtin_copysignf(r, v);
    if constexpr (K > 1)
        T[1] = r2;
    if constexpr (K > 2)
        T[2] = T[0] * r2;
    if constexpr (K > 3)
        T[3] = r2 * r2;
    if constexpr (K > 4)
        T[4] = T[2] * r2;
    if constexpr (K > 2)
        T[K - 1] = K % 2 ? v : a;      // y^K is the sample itself, or its magnitude
}

// LDS layout of a staged chunk: rows of window + 2 floats.  Rows [0, nch) hold
// the chunk's slots (row r: slot r's element over its sample window), and the
// two floats after row 0's window are zeros, the target of out-of-record
// delays.  With M == 2 (mirror pairing) rows [nch, 2 nch) hold the mirrored
// elements, n_elements - 1 - element, over the same sample windows: the mirror
// pixel reads them at the same delays, mirror_offset bytes on -- which also
// takes the zeros' address to the same two floats of row nch.
__device__ __forceinline__ int row_stride(int window) { return window + 2; }
__device__ __forceinline__ int zero_offset(int window) { return window * 4; }
__device__ __forceinline__ int mirror_offset(int nch, int window) { return nch * row_stride(window) * 4; }

// The rows a wave stages are a contiguous run of the chunk's; lane j holds the
// table entry of the run's row c + j, so one vector load brings 64 rows'
// entries.  (Requesting a chunk's entries with the rows of the chunk before
// gained nothing and cost short units 2 %.)
// A row inside the record needs the byte offset in the frame of LDS window
// position 0, in `at`; others (CHECK) its index in the record, and the record.
struct Rows {
    int at, channel;
};

struct RowRun {
    int s0, s1;               // the wave's rows
};
template <int M>
__device__ __forceinline__ RowRun row_run(int nch, int wave, int nwaves)
{
    const int rows = M * nch;
    const int per_wave = (rows + nwaves - 1) / nwaves;
    const int s0 = wave * per_wave;
    return {s0, min(rows, s0 + per_wave)};
}

template <int DT, int M, bool CHECK>
__device__ __forceinline__ Rows load_rows(const FrameArgs& A, ConstStage st, int nch, RowRun run, int c, int lane)
{
    const Global<const int> ent = global_ptr(reinterpret_cast<const int*>(st));
    const int j = min(c + lane, run.s1 - 1);
    const bool mirrored = M == 2 && j >= nch;
    const int src = mirrored ? j - nch : j;
    const int elem = ent[2 * src];
    const int channel = mirrored ? A.n_elements - 1 - elem : elem, first = ent[2 * src + 1];
    if constexpr (!CHECK)
        return {int(((unsigned)channel * (unsigned)A.stride + (unsigned)first) * (DT == HODMAS_F32 ? 4u : 2u)), 0};
    else
        return {first, channel};
}

// Rows are copied from memory straight into LDS: buffer loads that write LDS,
// one per 64 samples, so a row costs a lane read or two, scalar work and one
// load per wave -- no vector registers in flight and one wait for all of them.
// A 2-byte sample lands, zero-extended, in the low half of its LDS word (the
// layout of FP32 rows); FP16 is widened by the interpolation, int16 codes by a
// pass of each wave over its own rows (widen_codes).
// Rows inside the record (CHECK false) are read through one buffer resource
// over the whole frame, the row's start in the scalar offset.  Rows of tiles
// that reach the record ends are read through a resource of their own record,
// each lane's sample index clamped into it: a delay inside the record meets a
// clamped sample only as the neighbour of the record's last one, with weight
// zero, and every other delay is pointed at the zero pair (redirect).
// Measured against int16 rows, and rows at the record ends, through registers
// (sixteen loads, a wait, conversions and LDS stores at a time): int16, 256 elements, 4096 samples,
// mirror pairs at order 1, 256 x 256 60 -> 42 us, 512 x 512 62 -> 53 us; 1024 x
// 1024, 2048 samples, order 6 225 -> 220 us; a 331 x 203 image of 96 elements
// whose far half runs past the record 14.7 -> 13.3 us; 16 mixed frames as one
// batch 473 -> 434 us.
template <int DT, int M, bool CHECK>
__device__ __forceinline__ void stage_direct(const FrameArgs& A, ConstStage st, int nch, RowRun run, int window,
                                             float* __restrict__ lds, int lane)
{
    constexpr int esz = DT == HODMAS_F32 ? 4 : 2;
    using LdsPtr = __attribute__((address_space(3))) void*;
    const int stride = row_stride(window);
    auto copy = [&](__amdgpu_buffer_rsrc_t rs, int row, int b, int voff, int soff) {
        // the builtin takes the size as a constant
        if constexpr (DT == HODMAS_F32)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (LdsPtr)(lds + row * stride + b), 4, voff, soff, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (LdsPtr)(lds + row * stride + b), 2, voff, soff, 0, 0);
    };
    for (int c = run.s0; c < run.s1; c += 64) {
        const Rows r = load_rows<DT, M, CHECK>(A, st, nch, run, c, lane);
        const int cend = __builtin_amdgcn_readfirstlane(min(run.s1 - c, 64));
        if constexpr (CHECK) {
            const char* rf = static_cast<const char*>(A.rf);
            const int64_t row_bytes = int64_t(A.stride) * esz;
            for (int b = 0; b < window; b += 64) {
                if (b + lane < window) {
                    for (int m = 0; m < cend; ++m) {
                        const int ch = __builtin_amdgcn_readlane(r.channel, m);
                        const int first = __builtin_amdgcn_readlane(r.at, m);
                        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                            const_cast<char*>(rf + ch * row_bytes), (short)0, A.n_samples * esz, kBufferFlags);
                        copy(rs, c + m, b, max(0, min(first + b + lane, A.n_samples - 1)) * esz, 0);
                    }
                }
            }
        } else {
            // below 2^32 (the plan tests every tile otherwise), as are the row starts: both unsigned
            const unsigned bytes = (unsigned)A.n_elements * (unsigned)A.stride * esz;
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(A.rf), (short)0, (int)bytes, kBufferFlags);
            for (int b = 0; b < window; b += 64) {
                if (b + lane < window) {
                    for (int m = 0; m < cend; ++m)
                        copy(rs, c + m, b, (b + lane) * esz, __builtin_amdgcn_readlane(r.at, m));
                }
            }
        }
    }
}

// int16 codes in a wave's own rows dequantised and scaled in place, the pads
// between rows with them (the zero pair stays zero); eight times 64 words at a
// time, so the reads of one wave overlap.
__device__ __forceinline__ void widen_codes(float* __restrict__ lds, int begin, int end, float scale, int lane)
{
    constexpr int kAhead = 8;
    for (int b = begin; b < end; b += 64 * kAhead) {
        int w[kAhead];
#pragma unroll
        for (int m = 0; m < kAhead; ++m)
            w[m] = __builtin_bit_cast(int, lds[min(b + m * 64 + lane, end - 1)]);
#pragma unroll
        for (int m = 0; m < kAhead; ++m)
            if (b + m * 64 + lane < end)
                lds[b + m * 64 + lane] = (float)(short)w[m] * scale;
    }
}

// One chunk's rows into LDS.
template <int DT, int M, bool CHECK>
__device__ __forceinline__ void stage_chunk(const FrameArgs& A, ConstStage st, int nch, int window,
                                            float* __restrict__ lds, int wave, int nwaves, int lane)
{
    const RowRun run = row_run<M>(nch, wave, nwaves);
    const int stride = row_stride(window);
    // the zero pairs; with codes each by the wave whose row it follows, since
    // widen_codes runs over a wave's rows and their pads
    if constexpr (DT != HODMAS_I16) {
        if (wave == 0 && lane < 2 * M)
            lds[(lane >> 1) * nch * stride + window + (lane & 1)] = 0.f;
    } else {
#pragma unroll
        for (int mm = 0; mm < M; ++mm) {
            const int row = mm * nch;
            if (row >= run.s0 && row < run.s1 && lane < 2)
                lds[row * stride + window + lane] = 0.f;
        }
    }
    stage_direct<DT, M, CHECK>(A, st, nch, run, window, lds, lane);
    __builtin_amdgcn_s_waitcnt(0);   // the copies are in LDS before the caller's barrier
    if constexpr (DT == HODMAS_I16)
        widen_codes(lds, run.s0 * stride, run.s1 * stride, A.in_scale, lane);
}

// Workgroups are dealt to the eight XCDs round-robin (workgroup b runs on XCD
// b mod 8).  Give each XCD a contiguous run of tiles -- a band of tile rows --
// so the RF samples an XCD stages come from a narrow range of delays and its
// own L2 holds them, instead of every XCD fetching the whole frame.
__device__ __forceinline__ int xcd_tile(int b, int n)
{
    const int q = n / kXcds, r = n % kXcds;
    const int x = b % kXcds, l = b / kXcds;
    return x * q + min(x, r) + l;
}

// Power-sum accumulation.  Compensated mode: the terms of four elements are
// summed by themselves (PixelSums::add_group), eight such groups (32 elements)
// accumulate in a plain float32 partial, and the partial enters the running
// sum with one Kahan step.  The rounding error then stays at a few units of
// the partials' magnitude instead of growing with N.
template <int N, bool COMP>
struct PowerSums {
    float s[N], c[N];     // running sums, compensations
    float P[N];           // the current block's partials
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            s[j] = 0.f;
            c[j] = 0.f;
        }
    }
    // at each chunk's start: the partials need no registers while rows are staged
    __device__ __forceinline__ void start_block()
    {
#pragma unroll
        for (int j = 0; j < N; ++j)
            P[j] = 0.f;
    }
    __device__ __forceinline__ void add(int j, float a)
    {
        if (COMP)
            P[j] += a;
        else
            s[j] += a;
    }
    __device__ __forceinline__ void flush()
    {
        if (COMP) {
#pragma unroll
            for (int j = 0; j < N; ++j)
                kahan_add(s[j], c[j], P[j]);
            start_block();
        }
    }
    // the split groups' combination: (sum, compensation) pairs through LDS
    static constexpr int kFloats = 2 * N;
    __device__ __forceinline__ void put(float* red) const
    {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            red[2 * j] = s[j];
            red[2 * j + 1] = c[j];
        }
    }
    __device__ __forceinline__ void take(const float* red)
    {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const float so = red[2 * j], co = red[2 * j + 1];
            if (COMP) {
                kahan_add(s[j], c[j], so);
                kahan_add(s[j], c[j], -co);
            } else {
                s[j] += so;
            }
        }
    }
    template <class R>
    __device__ __forceinline__ R value(int j) const { return COMP ? R(s[j]) - R(c[j]) : R(s[j]); }
};

// a_0 + .. + a_3, and a_0 b_0 + .. + a_3 b_3 without rounding the products but
// the first: four instructions, where forming the products first takes seven.
__device__ __forceinline__ float sum4(const float (&a)[4]) { return (a[0] + a[1]) + (a[2] + a[3]); }
__device__ __forceinline__ float dot4(const float (&a)[4], const float (&b)[4])
{
    return __builtin_fmaf(a[3], b[3], __builtin_fmaf(a[2], b[2], __builtin_fmaf(a[1], b[1], a[0] * b[0])));
}

// y^1 .. y^K of four elements' signed K-th roots, each power summed over the
// four.  Bound by VALU issue, so every power that no later power needs is formed
// inside its sum (dot4): counted per element over the whole paired kernels 22.4
// instead of 23.3 instructions at K = 6, 20.1 instead of 20.8 at K = 5, 0.3 to 0.4
// fewer at K = 3 and 4 (unpaired 0.2 to 0.6 fewer).  Measured: int16, 256
// elements, 1024 x 1024, order 6 231.3 -> 225.3 us; float32 mirror pairs, 128
// elements, 2048 x 2048, order 5 300.6 -> 289.6 us; the six orders of eight
// 512 x 512 frames 823 -> 802 us.  (Carrying the symmetric sums themselves,
// e_m += y e_{m-1}, takes fewer instructions still, but where the array's
// halves cancel their partial sums exceed the result a thousandfold, and a
// float32 rounding of one with it.)
template <int K>
__device__ __forceinline__ void power_sums4(const float (&v)[4], float (&S)[K])
{
    float r[4], y[4], a[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        a[m] = __builtin_fabsf(v[m]);
        r[m] = root<K>(a[m]);
        y[m] = __builtin_copysignf(r[m], v[m]);
    }
    S[0] = sum4(y);
    if constexpr (K == 2) {
        S[1] = sum4(a);
    } else if constexpr (K == 3) {
        S[1] = dot4(r, r);
        S[2] = sum4(v);
    } else if constexpr (K > 3) {
        float r2[4];
#pragma unroll
        for (int m = 0; m < 4; ++m)
            r2[m] = root_squared<K>(a[m], r[m]);
        S[1] = sum4(r2);
        S[2] = dot4(y, r2);
        if constexpr (K == 4) {
            S[3] = sum4(a);
        } else if constexpr (K == 5) {
            S[3] = dot4(r2, r2);
            S[4] = sum4(v);
        } else {
            float r4[4];
#pragma unroll
            for (int m = 0; m < 4; ++m)
                r4[m] = r2[m] * r2[m];
            S[3] = sum4(r4);
            S[4] = dot4(y, r4);
            S[5] = sum4(a);
        }
    }
}

// What one pixel accumulates: its order's power sums and -- with
// coherence-factor weighting -- the sums of the samples and of their squares.
template <int K, bool CF, bool COMP>
struct PixelSums : PowerSums<K + (CF ? 2 : 0), COMP> {
    // A chunk whose last group has ended a block needs no flush after it.  Whether
    // to test for that is the loop's scheduling: with the test the orders from 5 on
    // take 2 to 3 % less, unpaired order 3 and weighted ones up to 3 %, but paired
    // order 2 (float16, 512 x 512 19.8 -> 20.4 us) and 4 (float32 23.7 -> 24.4) 3 % more.
    static constexpr bool kEndsBlock = !CF && (K <= 2 || K == 4);
    __device__ __forceinline__ void add_group(const float (&v)[4])
    {
        if constexpr (COMP) {
            float S[K];
            power_sums4<K>(v, S);
#pragma unroll
            for (int j = 0; j < K; ++j)
                this->add(j, S[j]);
            if constexpr (CF) {
                this->add(K, sum4(v));
                this->add(K + 1, dot4(v, v));
            }
        } else {
#pragma unroll
            for (int m = 0; m < 4; ++m)
                add_one(v[m]);
        }
    }
    __device__ __forceinline__ void add_one(float v)
    {
        float T[K];
        powers<K>(v, T);
#pragma unroll
        for (int j = 0; j < K; ++j)
            this->add(j, T[j]);
        if constexpr (CF) {
            this->add(K, v);
            this->add(K + 1, v * v);
        }
    }
};

__device__ __forceinline__ void load_group(ConstEntry E, hodmas_chan_entry (&e)[4])
{
#pragma unroll
    for (int m = 0; m < 4; ++m)
        e[m] = load_const(E, m);
}

// One group of four elements: delays and LDS addresses, the four gathers
// issued together, the interpolations, then -- once this group's LDS data is
// in -- the scalar loads of the next group's constants (the LDS/scalar wait
// counter does not order scalar loads, so issuing them earlier would make
// this group's waits also wait for them), then roots, powers and the sums.
// With M == 2 each delay also serves the lane's mirror pixel, whose samples
// sit `moff` bytes further on in the LDS (the mirrored rows).  `zero`: the
// LDS byte address of the zero pair (CHECK).  SH > 0: delays shared along
// translated pixels (see Shared): `sh` holds the group's first element's delay
// on entry and the next group's on return; (u2f, qf) are the lane's pixel
// moved 16 - 3*SH columns to the left; ro / ron: the LDS row offsets of this
// group's slots and, loaded with the next group's constants, of the next.
template <class Sums, bool CHECK, bool HALF, int M, int SH>
__device__ __forceinline__ void process_group(const hodmas_chan_entry (&e)[4], float u2, float q,
                                              const float* __restrict__ lds, int moff, int zero, Sums (&acc)[M],
                                              bool more, ConstEntry En,
                                              hodmas_chan_entry (&en)[4], Shared& sh, float u2f, float qf,
                                              const int (&ro)[4], ConstStage Sn, int slot_n, int stride,
                                              int (&ron)[4])
{
    Tap tp[4];
    float s0[M][4], s1[M][4], v[M][4];
    if constexpr (SH > 0) {
        static_assert(!CHECK && M == 1, "shared delays: untested tiles, one pixel per lane");
        static_assert(4 * SH == 16, "a group of four elements spans one row of 16 lanes");
        // the buffer holds this group's F and first element (written at the
        // end of the previous group, or before the first)
        const XF* b = sh.buf;
        wave_lds_order();
        const XF d1 = b[16 - SH], d2 = b[16 - 2 * SH], d3 = b[16 - 3 * SH];
        tp[0] = Tap{0.f, sh.f, sh.x + ro[0]};
        tp[1] = Tap{0.f, d1.f, d1.x + ro[1]};
        tp[2] = Tap{0.f, d2.f, d2.x + ro[2]};
        tp[3] = Tap{0.f, d3.f, d3.x + ro[3]};
    } else {
#pragma unroll
        for (int m = 0; m < 4; ++m)
            tp[m] = locate(e[m], u2, q);
    }
    if (CHECK) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
            redirect(tp[m], e[m], zero);
    }
#pragma unroll
    for (int mm = 0; mm < M; ++mm) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            s0[mm][m] = lds_at(lds, tp[m].addr + mm * moff);
            s1[mm][m] = lds_at(lds, tp[m].addr + mm * moff + 4);
        }
    }
#pragma unroll
    for (int mm = 0; mm < M; ++mm) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
            v[mm][m] = interp<HALF>(tp[m], s0[mm][m], s1[mm][m]);
    }
    // emits nothing: makes the samples (hence this group's LDS waits)
    // complete before the scalar loads below are issued
#pragma unroll
    for (int mm = 0; mm < M; ++mm)
        asm volatile("" ::"v"(v[mm][0]), "v"(v[mm][1]), "v"(v[mm][2]), "v"(v[mm][3]) : "memory");
    if (more) {
        load_group(En, en);
        if constexpr (SH > 0)
            load_rowoff(Sn, slot_n, stride, ron);
    }
#pragma unroll
    for (int mm = 0; mm < M; ++mm)
        acc[mm].add_group(v[mm]);
    if constexpr (SH > 0) {
        if (more) {
            // the next group's F -- its last element at the moved pixel --
            // formed here, after this group's arithmetic has been issued, so
            // its latency and that of the next group's constants overlap it;
            // written over this group's entries, whose reads came first
            const Tap tf = locate_at(en[3], u2f, qf, en[3].off - ron[3]);
            XF* b = sh.buf;
            wave_lds_order();
            b[0] = XF{tf.addr, tf.f};
            b[16] = XF{sh.fx, sh.ff};
            sh.x = sh.fx;
            sh.f = sh.ff;
            sh.fx = tf.addr;
            sh.ff = tf.f;
        }
    }
}

// The n elements of this wave's split group in one staged chunk (their
// constants stored contiguously), four at a time; two constant sets alternate
// so nothing is copied between them.
template <class Sums, bool CHECK, bool HALF, int M, int SH>
__device__ __forceinline__ void accumulate_chunk(ConstEntry E, int n, float u2, float q,
                                                 const float* __restrict__ lds, int moff, int zero, Sums (&acc)[M],
                                                 ConstStage St, int stride, float u2f, float qf, XF* shbuf)
{
    auto flush = [&]() {
#pragma unroll
        for (int mm = 0; mm < M; ++mm)
            acc[mm].flush();
    };
#pragma unroll
    for (int mm = 0; mm < M; ++mm)
        acc[mm].start_block();
    int sl = 0;
    if (n >= 4) {
        hodmas_chan_entry ea[4], eb[4];
        int ra[4] = {0, 0, 0, 0}, rb[4] = {0, 0, 0, 0};
        Shared sh{0, 0.f, 0, 0.f, shbuf};
        load_group(E, ea);
        if constexpr (SH > 0) {
            // slots 0..3 of the chunk: the first element's delay computed in
            // full, and the first group's F
            load_rowoff(St, 0, stride, ra);
            const Tap t0 = locate_at(ea[0], u2, q, ea[0].off - ra[0]);
            const Tap tf = locate_at(ea[3], u2f, qf, ea[3].off - ra[3]);
            sh.x = t0.addr;
            sh.f = t0.f;
            sh.fx = tf.addr;
            sh.ff = tf.f;
            wave_lds_order();
            sh.buf[0] = XF{tf.addr, tf.f};
            sh.buf[16] = XF{t0.addr, t0.f};
        }
        int groups = 0;
        while (true) {
            const bool more_a = sl + 8 <= n;
            process_group<Sums, CHECK, HALF, M, SH>(ea, u2, q, lds, moff, zero, acc, more_a, E + sl + 4, eb, sh, u2f,
                                                    qf, ra, St, sl + 4, stride, rb);
            if ((++groups & 7) == 0)
                flush();
            sl += 4;
            if (!more_a)
                break;
            const bool more_b = sl + 8 <= n;
            process_group<Sums, CHECK, HALF, M, SH>(eb, u2, q, lds, moff, zero, acc, more_b, E + sl + 4, ea, sh, u2f,
                                                    qf, rb, St, sl + 4, stride, ra);
            if ((++groups & 7) == 0)
                flush();
            sl += 4;
            if (!more_b)
                break;
        }
    }
    for (; sl < n; ++sl) {
        const hodmas_chan_entry e = load_const(E, sl);
        Tap tp = locate(e, u2, q);
        if (CHECK)
            redirect(tp, e, zero);
#pragma unroll
        for (int mm = 0; mm < M; ++mm) {
            const int addr = tp.addr + mm * moff;
            acc[mm].add_one(interp<HALF>(tp, lds_at(lds, addr), lds_at(lds, addr + 4)));
        }
    }
    if (Sums::kEndsBlock || (n & 31))
        flush();
}

// Newton's identities: e_m = (1/m) sum_{j=1..m} (-1)^(j-1) e_{m-j} p_j.
template <int K, typename R>
__device__ __forceinline__ R newton(const R (&p)[K])
{
    R e[K + 1];
    e[0] = R(1);
#pragma unroll
    for (int m = 1; m <= K; ++m) {
        R acc = R(0);
#pragma unroll
        for (int j = 1; j <= m; ++j) {
            R term = e[m - j] * p[j - 1];
            acc = (j & 1) ? acc + term : acc - term;
        }
        e[m] = acc * (R(1) / R(m));
    }
    return e[K];
}

// One pixel tile of one frame: stage, accumulate, combine, recover, store.
// Every thread of the workgroup calls this with the same (A, tile); all
// branches on tile data are workgroup-uniform, so the barriers inside match.
// With M == 2 the workgroup also forms the mirror tile: the pixel at column
// nx-1-ix of each lane's own pixel at ix.  When the array and the grid are
// symmetric about x = 0 (checked on the host), that pixel's delay to element
// n-1-i equals this pixel's delay to element i, so one delay serves both and
// the mirror pixel gathers from the mirrored rows the staging fills.
// `staged` is called once, when the first chunk's rows are in LDS: a request to
// memory made there is not waited for with them.
template <int K, int DT, bool COMP, bool CF, int M, bool CHECK, int SH, class Staged>
__device__ __forceinline__ void process_tile(const FrameArgs& A, const hodmas_tile_desc& td,
                                             float* __restrict__ lds, Staged staged)
{
    using Sums = PixelSums<K, CF, COMP>;
    constexpr bool kHalf = DT == HODMAS_F16;
    const int tid = threadIdx.x;
    const int npix = A.block / A.split;
    const int nwaves = A.block >> 6;
    const int g = __builtin_amdgcn_readfirstlane(tid / npix);   // npix is a multiple of 64
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int pl = tid - g * npix;
    const int lx = pl % A.tile_x, lz = pl / A.tile_x;
    const bool valid = lx < td.nx && lz < td.nz;
    const int ix = td.ix0 + min(lx, td.nx - 1);
    const int iz = td.iz0 + min(lz, td.nz - 1);
    // the lane's pixel (mm = 0) and, with M == 2, its mirror image; formed
    // where it is stored, so no 64-bit address stays live through the loops
    auto dst = [&](int mm) {
        return global_ptr(A.image + (int64_t)iz * A.nx + (mm == 0 ? ix : A.nx - 1 - ix));
    };

    if (td.n_active < K) {
        staged();
        // fewer contributing elements than the order: no K-subset exists, e_K = 0 exactly
        if (g == 0 && valid) {
#pragma unroll
            for (int mm = 0; mm < M; ++mm)
                *dst(mm) = 0.f;
        }
        return;
    }

    // pixel offset from the anchor, in float64 once per pixel
    const double u = A.x0s + ix * A.dxs - td.xa;
    const double w = A.z0s + iz * A.dzs - td.za;
    const float u2 = (float)(2.0 * u);
    const float q = (float)(u * u + w * (w + 2.0 * td.za));
    // SH > 0: the same pixel moved 16 - 3*SH columns to the left (the plan
    // keeps every tile 16 columns wide, so no lane's column was clamped)
    float u2f = 0.f, qf = 0.f;
    XF* shbuf = nullptr;
    if constexpr (SH > 0) {
        const double uf = u + (3 * SH - 16) * A.dxs;
        u2f = (float)(2.0 * uf);
        qf = (float)(uf * uf + w * (w + 2.0 * td.za));
        // the row's buffer after the staged rows (pixel row pl / 16 of
        // the workgroup; no lane's column was clamped, see above)
        shbuf = reinterpret_cast<XF*>(reinterpret_cast<char*>(lds) + A.shift_off) + (pl >> 4) * kRowEntries + lx;
    }

    Sums acc[M];
#pragma unroll
    for (int mm = 0; mm < M; ++mm)
        acc[mm].clear();
    ConstEntry E = A.entries + td.first_entry;
    ConstStage St = A.stage + td.first_entry;
    for (int c0 = 0; c0 < td.n_active; c0 += A.chunk) {
        const int nch = min(A.chunk, td.n_active - c0);
        __syncthreads();                       // previous readers of the LDS are done
        stage_chunk<DT, M, CHECK>(A, St + c0, nch, td.window, lds, wave, nwaves, lane);
        __syncthreads();
        if (c0 == 0)
            staged();
        const int moff = mirror_offset(nch, td.window);  // bytes from a slot's row to its mirrored row
        const int zero = zero_offset(td.window);
        // this group's elements of the chunk: slots g, g+split, ..., stored together
        int goff = 0;
        for (int h = 0; h < g; ++h)
            goff += (nch - h + A.split - 1) / A.split;
        const int ng = nch > g ? (nch - g + A.split - 1) / A.split : 0;
        accumulate_chunk<Sums, CHECK, kHalf, M, SH>(E + c0 + goff, ng, u2, q, lds, moff, zero, acc, St + c0,
                                                    row_stride(td.window), u2f, qf, shbuf);
    }

    if (A.split > 1) {
        // fixed-order combination of the groups' partial sums through LDS
        // floats per pixel and group: two per sum, padded to an odd stride so
        // consecutive lanes fall in different LDS banks
        constexpr int W = M * Sums::kFloats + 1;
        __syncthreads();
        float* red = lds;
        if (g > 0) {
#pragma unroll
            for (int mm = 0; mm < M; ++mm)
                acc[mm].put(red + ((g - 1) * npix + pl) * W + mm * Sums::kFloats);
        }
        __syncthreads();
        if (g == 0) {
            for (int gg = 1; gg < A.split; ++gg) {
#pragma unroll
                for (int mm = 0; mm < M; ++mm)
                    acc[mm].take(red + ((gg - 1) * npix + pl) * W + mm * Sums::kFloats);
            }
        }
    }
    if (g != 0 || !valid)
        return;
    using R = typename std::conditional<(K >= 5), double, float>::type;
#pragma unroll
    for (int mm = 0; mm < M; ++mm) {
        R p[K];
#pragma unroll
        for (int j = 0; j < K; ++j)
            p[j] = acc[mm].template value<R>(j);
        const R ek = newton<K, R>(p);
        if constexpr (CF) {
            // coherence factor (sum v)^2 / (N sum v^2) of the normalised samples
            const double s1 = acc[mm].template value<double>(K);
            const double s2 = acc[mm].template value<double>(K + 1);
            const double cf = s2 > 0.0 ? (s1 * s1) / (double(A.n_elements) * s2) : 0.0;
            *dst(mm) = (float)(double(ek) * cf * double(A.out_scale));
        } else {
            *dst(mm) = (float)(ek * R(A.out_scale));
        }
    }
}

// Tiles that reach the record ends take the body with the range test, the
// others the body without it.  The choice is made once per tile, so each body
// is a whole of its own: with the test inside the element loop, or with both
// loop variants in one body, the paired kernels' sums no longer fit their
// registers and the loop's scheduling suffers.
struct Nothing {
    __device__ __forceinline__ void operator()() const {}
};
template <int K, int DT, bool COMP, bool CF, int M, class Staged = Nothing>
__device__ __forceinline__ void form_tile(const FrameArgs& A, int tile, float* __restrict__ lds, Staged staged = {})
{
    const hodmas_tile_desc td = load_const(A.tiles, tile);
    if (td.check) {
        process_tile<K, DT, COMP, CF, M, true, 0>(A, td, lds, staged);
    } else {
        if constexpr (M == 1 && !CF && K >= 2) {
            if (A.shift == 4 && td.iz0 >= A.shift_iz0) {
                process_tile<K, DT, COMP, CF, M, false, 4>(A, td, lds, staged);
                return;
            }
        }
        process_tile<K, DT, COMP, CF, M, false, 0>(A, td, lds, staged);
    }
}

// M == 1: workgroup b forms tile xcd_tile(b).  M == 2: workgroup b forms pair
// p = xcd_tile(b) of the n_tiles / 2 pairs -- the p-th tile of the grid's
// left half (row-major over its tile rows) and that tile's mirror image.
template <int K, int DT, bool COMP, bool CF, int M>
__global__ __launch_bounds__(kMaxBlock) void hodmas_frame_kernel(FrameArgs A)
{
    extern __shared__ float lds[];
    if constexpr (M == 1) {
        form_tile<K, DT, COMP, CF, 1>(A, xcd_tile(blockIdx.x, A.n_tiles), lds);
    } else {
        const int half = A.nx / A.tile_x / 2;     // tile columns left of the centre
        const int p = xcd_tile(blockIdx.x, A.n_tiles / 2);
        const int bz = p / half;
        form_tile<K, DT, COMP, CF, 2>(A, bz * 2 * half + (p - bz * half), lds);
    }
}

// Batched form: one kernel per (order, storage type, pairing, coherence
// weighting).  Its grid walks that kind's slice of the batch's work
// list -- (frame, tile) units of many frames with their own plans.  The slice
// is cut into one run per XCD (neighbouring tiles of one or a few frames, of
// about equal estimated cost, each sorted by cost); the g workgroups on XCD x
// (workgroups x, x+8, ...) walk run x, the l-th of them taking unit l.  A grid
// has one workgroup per unit of the longest run; only in lists beyond the
// largest grid, or beyond the list a captured launch was made for, does the l-th
// go on to units 2g-1-l, 2g+l, ... (a snake, which evens out the per-workgroup
// cost).  With
// M == 2 a unit is a mirror pair, named by its left tile.  Each unit runs
// exactly the code of the per-frame kernel, so a frame's image does not depend
// on what else is in the batch.
// Mirror pairs keep two pixels' sums per lane.  At order 6 that takes a paired
// kernel a little above 80 VGPRs (five waves per SIMD), while a 64-element
// chunk's LDS leaves room for six workgroups per CU; asking for six waves
// costs a few dwords of spill per tile (values kept for the final store), none
// in the loops.  Lower orders fit six or seven waves without asking; with
// coherence weighting (two more sums per pixel) six waves would spill inside
// the loops, so those kernels are left at the four or five they fit.
constexpr int batch_min_waves(int K, int M, bool CF) { return M == 2 && K == 6 && !CF ? 6 : 1; }

// This workgroup among those of one XCD, and the XCD's run of the kind's units.
struct UnitRun {
    int l, g;             // this workgroup, of so many on the XCD
    int first, n;         // the run's units in the list
    // the workgroup's unit of round r, below n while it has one
    __device__ __forceinline__ int unit(int r) const { return (r & 1) ? (r + 1) * g - 1 - l : r * g + l; }
};
__device__ __forceinline__ UnitRun unit_run(const BatchHeader* __restrict__ hdr, int kind)
{
    const int x = (int)blockIdx.x % kXcds;
    const int lo = load_const(&hdr->xcd[kind][0], x);
    return {(int)blockIdx.x / kXcds, ((int)gridDim.x - x + kXcds - 1) / kXcds, load_const(&hdr->begin[0], kind) + lo,
            load_const(&hdr->xcd[kind][0], x + 1) - lo};
}

template <int K, int DT, bool COMP, bool CF, int M>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(batch_min_waves(K, M, CF))))
void hodmas_batch_kernel(const BatchHeader* __restrict__ hdr, const BatchFrame* __restrict__ frames,
                         const BatchUnit* __restrict__ units)
{
    extern __shared__ float lds[];
    const UnitRun run = unit_run(hdr, batch_kind(K, DT, M, CF ? 1 : 0));
    for (int r = 0; r * run.g < run.n; ++r) {
        const int u = run.unit(r);
        if (u >= run.n)
            continue;
        const BatchUnit un = load_const(units, run.first + u);
        const BatchFrame fr = load_const(frames, un.frame);
        form_tile<K, DT, COMP, CF, M>(fr.args, un.tile, lds);
    }
}

// Units of any order and pairing, each formed by the code of its own kind in
// the registers of the largest (six waves, as the paired order 6 asks for), so
// that one launch, and one tail, serves a work list whose kinds would each
// leave the device half empty.  Units of several orders differ too much for equal
// shares of a grid that fills the device (24 FP16 frames of 17 shapes, mirror
// pairs: 862 us).  Without counts (null) the grid has a workgroup per unit (697 us).
// With them it fills the device and workgroups draw: after units l and 2g - 1 - l
// of its XCD's run (heaviest first) a workgroup asks for its next one while it
// forms the last in hand (679 us).  counts belongs to this launch alone until it
// ends, so launches of one list may overlap.  The workgroups of a run draw until
// they fail, one failure each, and whoever makes the last draw sets the count back
// to zero.  Counts of different XCDs stand in lines of their own: in one line, the
// draws of all XCDs waited for each other (36 frames of 128 x 128 at six orders 103
// us, 54 apart).  The number passes through the first word of the LDS, which is
// free between units.
template <int DT>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6)))
void hodmas_mixed_kernel(const BatchHeader* __restrict__ hdr, const BatchFrame* __restrict__ frames,
                         const BatchUnit* __restrict__ units, DrawCount* counts)
{
    extern __shared__ float lds[];
    const UnitRun run = unit_run(hdr, mixed_kind(DT));
    const int fixed = 2 * run.g;                     // units taken without drawing
    const bool draws = counts != nullptr && run.n > fixed;
    int* const count = draws ? &counts[DT * kXcds + blockIdx.x % kXcds].n : nullptr;
    int* const number = reinterpret_cast<int*>(lds);
    for (int r = 0, u = run.l; u < run.n;) {
        int drawn = 0;
        auto draw = [&] {
            if (draws && r > 0 && threadIdx.x == 0)
                drawn = __hip_atomic_fetch_add(count, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        const BatchUnit un = load_const(units, run.first + u);
        const BatchFrame fr = load_const(frames, un.frame);
        switch (2 * fr.order + fr.pairing) {
        case 3: form_tile<1, DT, true, false, 1>(fr.args, un.tile, lds, draw); break;
        case 4: form_tile<1, DT, true, false, 2>(fr.args, un.tile, lds, draw); break;
        case 5: form_tile<2, DT, true, false, 1>(fr.args, un.tile, lds, draw); break;
        case 6: form_tile<2, DT, true, false, 2>(fr.args, un.tile, lds, draw); break;
        case 7: form_tile<3, DT, true, false, 1>(fr.args, un.tile, lds, draw); break;
        case 8: form_tile<3, DT, true, false, 2>(fr.args, un.tile, lds, draw); break;
        case 9: form_tile<4, DT, true, false, 1>(fr.args, un.tile, lds, draw); break;
        case 10: form_tile<4, DT, true, false, 2>(fr.args, un.tile, lds, draw); break;
        case 11: form_tile<5, DT, true, false, 1>(fr.args, un.tile, lds, draw); break;
        case 12: form_tile<5, DT, true, false, 2>(fr.args, un.tile, lds, draw); break;
        case 13: form_tile<6, DT, true, false, 1>(fr.args, un.tile, lds, draw); break;
        case 14: form_tile<6, DT, true, false, 2>(fr.args, un.tile, lds, draw); break;
        }
        if (!draws || r == 0) {
            u = run.unit(++r);
            continue;
        }
        __syncthreads();                   // the unit's readers of the LDS are done
        if (threadIdx.x == 0) {
            *number = drawn;
            if (drawn == run.n - fixed + run.g - 1)   // every unit drawn, and g failures
                __hip_atomic_store(count, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        u = fixed + __builtin_amdgcn_readfirstlane(*number);
        __syncthreads();                   // and the number is read
    }
}

// ---------------------------------------------------------------------------
// Every order 1..KMAX in one pass.  The delay, gather and interpolation are
// the same for all orders; the roots share their transcendentals
// (|v|^(1/4) = sqrt(|v|^(1/2)), |v|^(1/6) = sqrt(|v|^(1/3)), one log2 serves
// the cube and fifth roots); and many power sums coincide across orders,
// since y_k^j = sign(v)^j |v|^(j/k) depends only on j/k and the parity of j:
// orders 1..6 need 15 distinct sums instead of 21.
//
//   sum   exponent  signed   used as p_j of order k
//    0      1        yes     k1 p1, k3 p3, k5 p5
//    1      1        no      k2 p2, k4 p4, k6 p6
//    2      1/2      yes     k2 p1, k6 p3
//    3      1/2      no      k4 p2
//    4      1/3      yes     k3 p1
//    5      1/3      no      k6 p2
//    6      2/3      no      k3 p2, k6 p4
//    7      1/4      yes     k4 p1
//    8      3/4      yes     k4 p3
//    9..12  j/5      j odd   k5 p1..p4
//   13      1/6      yes     k6 p1
//   14      5/6      yes     k6 p5
constexpr int kSums = kOrderSums;
constexpr int kSumOf[HODMAS_MAX_ORDER + 1][HODMAS_MAX_ORDER] = {
    {0, 0, 0, 0, 0, 0},
    {0, 0, 0, 0, 0, 0},
    {2, 1, 0, 0, 0, 0},
    {4, 6, 0, 0, 0, 0},
    {7, 3, 8, 1, 0, 0},
    {9, 10, 11, 12, 0, 0},
    {13, 5, 2, 6, 14, 1},
};

// Is sum i needed by some order <= KMAX?
constexpr bool sum_needed(int i, int kmax)
{
    for (int k = 1; k <= kmax; ++k)
        for (int j = 0; j < k; ++j)
            if (kSumOf[k][j] == i)
                return true;
    return false;
}

template <int KMAX>
__device__ __forceinline__ void terms_all(float v, float (&T)[kSums])
{
    const float a = __builtin_fabsf(v);
    T[0] = v;
    T[1] = a;
    if constexpr (KMAX >= 2) {
        const float r2 = __builtin_amdgcn_sqrtf(a);
        T[2] = __builtin_copysignf(r2, v);
        T[3] = r2;
        if constexpr (KMAX >= 3) {
            const float L = __builtin_amdgcn_logf(a);
            const float r3 = __builtin_amdgcn_exp2f(L * (1.0f / 3));
            T[4] = __builtin_copysignf(r3, v);
            T[5] = r3;
            T[6] = r3 * r3;
            if constexpr (KMAX >= 4) {
                const float y4 = __builtin_copysignf(__builtin_amdgcn_sqrtf(r2), v);
                T[7] = y4;
                T[8] = y4 * r2;
                if constexpr (KMAX >= 5) {
                    const float r5 = __builtin_amdgcn_exp2f(L * 0.2f);
                    const float y5 = __builtin_copysignf(r5, v);
                    const float q5 = r5 * r5;
                    T[9] = y5;
                    T[10] = q5;
                    T[11] = y5 * q5;
                    T[12] = q5 * q5;
                    if constexpr (KMAX >= 6) {
                        const float y6 = __builtin_copysignf(__builtin_amdgcn_sqrtf(r3), v);
                        T[13] = y6;
                        T[14] = y6 * T[6];
                    }
                }
            }
        }
    }
}

// One element's terms added to S (FIRST: begin S with them), the products that
// nothing else needs inside the addition: four instructions fewer per element
// at KMAX = 6 than terms_all and 15 additions (128 elements, 512 x 512, orders
// 1..6 in one pass: 53.2 -> 52.5 us; four waves per SIMD, so latency more than
// issue holds it).
template <int KMAX, bool FIRST>
__device__ __forceinline__ void add_terms(float v, float (&S)[kSums])
{
    auto sum = [&](int j, float t) { S[j] = FIRST ? t : S[j] + t; };
    auto product = [&](int j, float a, float b) { S[j] = FIRST ? a * b : __builtin_fmaf(a, b, S[j]); };
    const float a = __builtin_fabsf(v);
    sum(0, v);
    sum(1, a);
    if constexpr (KMAX >= 2) {
        const float r2 = __builtin_amdgcn_sqrtf(a);
        sum(2, __builtin_copysignf(r2, v));
        sum(3, r2);
        if constexpr (KMAX >= 3) {
            const float L = __builtin_amdgcn_logf(a);
            const float r3 = __builtin_amdgcn_exp2f(L * (1.0f / 3));
            const float q3 = r3 * r3;
            sum(4, __builtin_copysignf(r3, v));
            sum(5, r3);
            sum(6, q3);
            if constexpr (KMAX >= 4) {
                const float y4 = __builtin_copysignf(__builtin_amdgcn_sqrtf(r2), v);
                sum(7, y4);
                product(8, y4, r2);
                if constexpr (KMAX >= 5) {
                    const float r5 = __builtin_amdgcn_exp2f(L * 0.2f);
                    const float y5 = __builtin_copysignf(r5, v);
                    const float q5 = r5 * r5;
                    sum(9, y5);
                    sum(10, q5);
                    product(11, y5, q5);
                    product(12, q5, q5);
                    if constexpr (KMAX >= 6) {
                        const float y6 = __builtin_copysignf(__builtin_amdgcn_sqrtf(r3), v);
                        sum(13, y6);
                        product(14, y6, q3);
                    }
                }
            }
        }
    }
}

template <int KMAX, bool COMP, bool CHECK, bool HALF>
__device__ __forceinline__ void process_group_all(const hodmas_chan_entry (&e)[4], float u2, float q,
                                                  const float* __restrict__ lds, int zero, float (&s)[kSums],
                                                  float (&P)[kSums], bool more, ConstEntry En,
                                                  hodmas_chan_entry (&en)[4])
{
    Tap tp[4];
    float s0[4], s1[4], v[4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
        tp[m] = locate(e[m], u2, q);
    if (CHECK) {
#pragma unroll
        for (int m = 0; m < 4; ++m)
            redirect(tp[m], e[m], zero);
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        s0[m] = lds_at(lds, tp[m].addr);
        s1[m] = lds_at(lds, tp[m].addr + 4);
    }
#pragma unroll
    for (int m = 0; m < 4; ++m)
        v[m] = interp<HALF>(tp[m], s0[m], s1[m]);
    asm volatile("" ::"v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]) : "memory");
    if (more)
        load_group(En, en);
    if constexpr (COMP) {
        float S[kSums];
        add_terms<KMAX, true>(v[0], S);
#pragma unroll
        for (int m = 1; m < 4; ++m)
            add_terms<KMAX, false>(v[m], S);
#pragma unroll
        for (int j = 0; j < kSums; ++j)
            if (sum_needed(j, KMAX))
                P[j] += S[j];
    } else {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            float T[kSums];
            terms_all<KMAX>(v[m], T);
#pragma unroll
            for (int j = 0; j < kSums; ++j)
                if (sum_needed(j, KMAX))
                    s[j] += T[j];
        }
    }
}

template <int KMAX, bool COMP>
__device__ __forceinline__ void flush_all(float (&s)[kSums], float (&c)[kSums], float (&P)[kSums])
{
#pragma unroll
    for (int j = 0; j < kSums; ++j) {
        if (!sum_needed(j, KMAX))
            continue;
        kahan_add(s[j], c[j], P[j]);
        P[j] = 0.f;
    }
}

template <int KMAX, bool COMP, bool CHECK, bool HALF>
__device__ __forceinline__ void accumulate_chunk_all(ConstEntry E, int n, float u2, float q,
                                                     const float* __restrict__ lds, int zero, float (&s)[kSums],
                                                     float (&c)[kSums])
{
    float P[kSums];
#pragma unroll
    for (int j = 0; j < kSums; ++j)
        P[j] = 0.f;
    int sl = 0;
    if (n >= 4) {
        hodmas_chan_entry ea[4], eb[4];
        load_group(E, ea);
        int groups = 0;
        while (true) {
            const bool more_a = sl + 8 <= n;
            process_group_all<KMAX, COMP, CHECK, HALF>(ea, u2, q, lds, zero, s, P, more_a, E + sl + 4, eb);
            if (COMP && (++groups & 7) == 0)
                flush_all<KMAX, COMP>(s, c, P);
            sl += 4;
            if (!more_a)
                break;
            const bool more_b = sl + 8 <= n;
            process_group_all<KMAX, COMP, CHECK, HALF>(eb, u2, q, lds, zero, s, P, more_b, E + sl + 4, ea);
            if (COMP && (++groups & 7) == 0)
                flush_all<KMAX, COMP>(s, c, P);
            sl += 4;
            if (!more_b)
                break;
        }
    }
    for (; sl < n; ++sl) {
        const hodmas_chan_entry e = load_const(E, sl);
        Tap tp = locate(e, u2, q);
        if (CHECK)
            redirect(tp, e, zero);
        float T[kSums];
        terms_all<KMAX>(interp<HALF>(tp, lds_at(lds, tp.addr), lds_at(lds, tp.addr + 4)), T);
#pragma unroll
        for (int j = 0; j < kSums; ++j) {
            if (!sum_needed(j, KMAX))
                continue;
            if (COMP)
                P[j] += T[j];
            else
                s[j] += T[j];
        }
    }
    if (COMP)
        flush_all<KMAX, COMP>(s, c, P);
}

template <int K, bool COMP>
__device__ __forceinline__ void store_order(const float (&s)[kSums], const float (&c)[kSums], float out_scale,
                                            float* __restrict__ dst)
{
    using R = typename std::conditional<(K >= 5), double, float>::type;
    R p[K];
#pragma unroll
    for (int j = 0; j < K; ++j)
        p[j] = COMP ? R(s[kSumOf[K][j]]) - R(c[kSumOf[K][j]]) : R(s[kSumOf[K][j]]);
    *dst = (float)(newton<K, R>(p) * R(out_scale));
}

template <int KMAX, int DT, bool COMP, bool CHECK>
__device__ __forceinline__ void orders_tile(const FrameArgs& A, const OrderImages& out, const hodmas_tile_desc& td,
                                            float* __restrict__ lds)
{
    constexpr int NT = kSums;
    constexpr bool kHalf = DT == HODMAS_F16;
    const int tid = threadIdx.x;
    const int npix = A.block / A.split;
    const int nwaves = A.block >> 6;
    const int g = __builtin_amdgcn_readfirstlane(tid / npix);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int pl = tid - g * npix;
    const int lx = pl % A.tile_x, lz = pl / A.tile_x;
    const bool valid = lx < td.nx && lz < td.nz;
    const int ix = td.ix0 + min(lx, td.nx - 1);
    const int iz = td.iz0 + min(lz, td.nz - 1);
    const int64_t pix = (int64_t)iz * A.nx + ix;

    const double u = A.x0s + ix * A.dxs - td.xa;
    const double w = A.z0s + iz * A.dzs - td.za;
    const float u2 = (float)(2.0 * u);
    const float q = (float)(u * u + w * (w + 2.0 * td.za));

    float s[NT], c[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        // unneeded sums stay zero and are never read
        s[j] = 0.f;
        c[j] = 0.f;
    }
    ConstEntry E = A.entries + td.first_entry;
    ConstStage St = A.stage + td.first_entry;
    for (int c0 = 0; c0 < td.n_active; c0 += A.chunk) {
        const int nch = min(A.chunk, td.n_active - c0);
        __syncthreads();
        stage_chunk<DT, 1, CHECK>(A, St + c0, nch, td.window, lds, wave, nwaves, lane);
        __syncthreads();
        int goff = 0;
        for (int h = 0; h < g; ++h)
            goff += (nch - h + A.split - 1) / A.split;
        const int ng = nch > g ? (nch - g + A.split - 1) / A.split : 0;
        accumulate_chunk_all<KMAX, COMP, CHECK, kHalf>(E + c0 + goff, ng, u2, q, lds, zero_offset(td.window), s, c);
    }
    if (A.split > 1) {
        __syncthreads();
        float* red = lds;
        if (g > 0) {
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                if (!sum_needed(j, KMAX))
                    continue;
                red[((g - 1) * npix + pl) * (2 * NT + 1) + 2 * j] = s[j];
                red[((g - 1) * npix + pl) * (2 * NT + 1) + 2 * j + 1] = c[j];
            }
        }
        __syncthreads();
        if (g == 0) {
            for (int gg = 1; gg < A.split; ++gg) {
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    if (!sum_needed(j, KMAX))
                        continue;
                    const float so = red[((gg - 1) * npix + pl) * (2 * NT + 1) + 2 * j];
                    const float co = red[((gg - 1) * npix + pl) * (2 * NT + 1) + 2 * j + 1];
                    if (COMP) {
                        kahan_add(s[j], c[j], so);
                        kahan_add(s[j], c[j], -co);
                    } else {
                        s[j] += so;
                    }
                }
            }
        }
    }
    if (g != 0 || !valid)
        return;
    // orders with fewer contributing elements than k are exactly 0
    const int na = td.n_active;
    if (na >= 1) store_order<1, COMP>(s, c, A.out_scale, out.img[0] + pix); else out.img[0][pix] = 0.f;
    if constexpr (KMAX >= 2) { if (na >= 2) store_order<2, COMP>(s, c, A.out_scale, out.img[1] + pix); else out.img[1][pix] = 0.f; }
    if constexpr (KMAX >= 3) { if (na >= 3) store_order<3, COMP>(s, c, A.out_scale, out.img[2] + pix); else out.img[2][pix] = 0.f; }
    if constexpr (KMAX >= 4) { if (na >= 4) store_order<4, COMP>(s, c, A.out_scale, out.img[3] + pix); else out.img[3][pix] = 0.f; }
    if constexpr (KMAX >= 5) { if (na >= 5) store_order<5, COMP>(s, c, A.out_scale, out.img[4] + pix); else out.img[4][pix] = 0.f; }
    if constexpr (KMAX >= 6) { if (na >= 6) store_order<6, COMP>(s, c, A.out_scale, out.img[5] + pix); else out.img[5][pix] = 0.f; }
}

template <int KMAX, int DT, bool COMP>
__global__ __launch_bounds__(kMaxBlock) void hodmas_orders_kernel(FrameArgs A, OrderImages out)
{
    extern __shared__ float lds[];
    const hodmas_tile_desc td = load_const(A.tiles, xcd_tile(blockIdx.x, A.n_tiles));
    if (td.check)
        orders_tile<KMAX, DT, COMP, true>(A, out, td, lds);
    else
        orders_tile<KMAX, DT, COMP, false>(A, out, td, lds);
}

template <int KMAX, int DT>
int launch_orders_k(const FrameArgs& a, const OrderImages& out, bool comp, int64_t lds_bytes, hipStream_t st)
{
    dim3 grid(a.n_tiles), block(a.block);
    if (comp)
        hipLaunchKernelGGL((hodmas_orders_kernel<KMAX, DT, true>), grid, block, (size_t)lds_bytes, st, a, out);
    else
        hipLaunchKernelGGL((hodmas_orders_kernel<KMAX, DT, false>), grid, block, (size_t)lds_bytes, st, a, out);
    return (int)hipGetLastError();
}

template <int DT>
int launch_orders_dt(const FrameArgs& a, const OrderImages& out, int kmax, bool comp, int64_t lds_bytes,
                     hipStream_t st)
{
    switch (kmax) {
    case 1: return launch_orders_k<1, DT>(a, out, comp, lds_bytes, st);
    case 2: return launch_orders_k<2, DT>(a, out, comp, lds_bytes, st);
    case 3: return launch_orders_k<3, DT>(a, out, comp, lds_bytes, st);
    case 4: return launch_orders_k<4, DT>(a, out, comp, lds_bytes, st);
    case 5: return launch_orders_k<5, DT>(a, out, comp, lds_bytes, st);
    case 6: return launch_orders_k<6, DT>(a, out, comp, lds_bytes, st);
    }
    return (int)hipErrorInvalidValue;
}

// A workgroup may hold more than 64 KB of LDS only once the kernel says so.
int launch_one(void (*fn)(FrameArgs), dim3 grid, dim3 block, int64_t lds_bytes, hipStream_t st,
               const FrameArgs& a)
{
    if (lds_bytes > 64 * 1024 &&
        hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds_bytes) != hipSuccess)
        return (int)hipGetLastError();
    hipLaunchKernelGGL(fn, grid, block, (size_t)lds_bytes, st, a);
    return (int)hipGetLastError();
}

template <int K, int DT, int M>
int launch_km(const FrameArgs& a, bool comp, bool cf, int64_t lds_bytes, hipStream_t st)
{
    const dim3 grid(a.n_tiles / M), block(a.block);
    if (comp && cf)
        return launch_one(hodmas_frame_kernel<K, DT, true, true, M>, grid, block, lds_bytes, st, a);
    if (comp)
        return launch_one(hodmas_frame_kernel<K, DT, true, false, M>, grid, block, lds_bytes, st, a);
    if (cf)
        return launch_one(hodmas_frame_kernel<K, DT, false, true, M>, grid, block, lds_bytes, st, a);
    return launch_one(hodmas_frame_kernel<K, DT, false, false, M>, grid, block, lds_bytes, st, a);
}

template <int K, int DT>
int launch_k(const FrameArgs& a, bool comp, bool cf, bool mirror, int64_t lds_bytes, hipStream_t st)
{
    return mirror ? launch_km<K, DT, 2>(a, comp, cf, lds_bytes, st) : launch_km<K, DT, 1>(a, comp, cf, lds_bytes, st);
}

template <int DT>
int launch_dt(const FrameArgs& a, int order, bool comp, bool cf, bool mirror, int64_t lds_bytes,
              hipStream_t st)
{
    switch (order) {
    case 1: return launch_k<1, DT>(a, comp, cf, mirror, lds_bytes, st);
    case 2: return launch_k<2, DT>(a, comp, cf, mirror, lds_bytes, st);
    case 3: return launch_k<3, DT>(a, comp, cf, mirror, lds_bytes, st);
    case 4: return launch_k<4, DT>(a, comp, cf, mirror, lds_bytes, st);
    case 5: return launch_k<5, DT>(a, comp, cf, mirror, lds_bytes, st);
    case 6: return launch_k<6, DT>(a, comp, cf, mirror, lds_bytes, st);
    }
    return (int)hipErrorInvalidValue;
}

}  // namespace

int launch_frame(const FrameArgs& a, int order, int dtype, bool compensated, bool coherence,
                 bool mirror, int64_t lds_bytes, void* stream)
{
    hipStream_t st = static_cast<hipStream_t>(stream);
    switch (dtype) {
    case HODMAS_F32: return launch_dt<HODMAS_F32>(a, order, compensated, coherence, mirror, lds_bytes, st);
    case HODMAS_F16: return launch_dt<HODMAS_F16>(a, order, compensated, coherence, mirror, lds_bytes, st);
    case HODMAS_I16: return launch_dt<HODMAS_I16>(a, order, compensated, coherence, mirror, lds_bytes, st);
    }
    return (int)hipErrorInvalidValue;
}

// coherence-weighted kinds exist for compensated accumulation only
template <int K, int DT, int M>
const void* batch_fn(bool comp, bool cf)
{
    if (cf)
        return comp ? reinterpret_cast<const void*>(&hodmas_batch_kernel<K, DT, true, true, M>) : nullptr;
    return comp ? reinterpret_cast<const void*>(&hodmas_batch_kernel<K, DT, true, false, M>)
                : reinterpret_cast<const void*>(&hodmas_batch_kernel<K, DT, false, false, M>);
}

template <int DT, int M>
const void* batch_fn_dt(int order, bool comp, bool cf)
{
    switch (order) {
    case 1: return batch_fn<1, DT, M>(comp, cf);
    case 2: return batch_fn<2, DT, M>(comp, cf);
    case 3: return batch_fn<3, DT, M>(comp, cf);
    case 4: return batch_fn<4, DT, M>(comp, cf);
    case 5: return batch_fn<5, DT, M>(comp, cf);
    case 6: return batch_fn<6, DT, M>(comp, cf);
    }
    return nullptr;
}

template <int M>
const void* batch_fn_m(int order, int dtype, bool comp, bool cf)
{
    switch (dtype) {
    case HODMAS_F32: return batch_fn_dt<HODMAS_F32, M>(order, comp, cf);
    case HODMAS_F16: return batch_fn_dt<HODMAS_F16, M>(order, comp, cf);
    case HODMAS_I16: return batch_fn_dt<HODMAS_I16, M>(order, comp, cf);
    }
    return nullptr;
}

int launch_orders(const FrameArgs& a, const OrderImages& out, int kmax, int dtype, bool compensated,
                  int64_t lds_bytes, void* stream)
{
    hipStream_t st = static_cast<hipStream_t>(stream);
    switch (dtype) {
    case HODMAS_F32: return launch_orders_dt<HODMAS_F32>(a, out, kmax, compensated, lds_bytes, st);
    case HODMAS_F16: return launch_orders_dt<HODMAS_F16>(a, out, kmax, compensated, lds_bytes, st);
    case HODMAS_I16: return launch_orders_dt<HODMAS_I16>(a, out, kmax, compensated, lds_bytes, st);
    }
    return (int)hipErrorInvalidValue;
}

const void* batch_kernel(int kind, bool compensated)
{
    if (kind < 0 || kind >= kBatchKinds)
        return nullptr;
    if (kind >= kOrderKinds) {             // mixed orders: compensated only
        const void* const fn[3] = {reinterpret_cast<const void*>(&hodmas_mixed_kernel<HODMAS_F32>),
                                   reinterpret_cast<const void*>(&hodmas_mixed_kernel<HODMAS_F16>),
                                   reinterpret_cast<const void*>(&hodmas_mixed_kernel<HODMAS_I16>)};
        static_assert(HODMAS_F32 == 0 && HODMAS_F16 == 1 && HODMAS_I16 == 2, "by storage type");
        return compensated ? fn[kind - kOrderKinds] : nullptr;
    }
    const int order = kind_order(kind), dtype = kind_dtype(kind);
    const bool cf = kind_cf(kind) != 0;
    switch (kind_pairing(kind)) {
    case 1: return batch_fn_m<1>(order, dtype, compensated, cf);
    case 2: return batch_fn_m<2>(order, dtype, compensated, cf);
    }
    return nullptr;
}

int launch_batch(int kind, const BatchHeader* hdr, const BatchFrame* frames, const BatchUnit* units, int grid,
                 bool compensated, int64_t lds_bytes, void* stream)
{
    const void* fn = batch_kernel(kind, compensated);
    if (!fn || kind >= kOrderKinds)
        return (int)hipErrorInvalidValue;
    void* args[] = {(void*)&hdr, (void*)&frames, (void*)&units};
    return (int)hipLaunchKernel(fn, dim3(grid), dim3(kBlock), args, (size_t)lds_bytes,
                                static_cast<hipStream_t>(stream));
}

}  // namespace hodmas
