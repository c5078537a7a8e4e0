// Image-quality metrics of a beamformed (envelope) image (Sec. IV): SNR
// (Eq. 10), CR (Eq. 11), gCNR (Eq. 12) over a target and a background
// rectangle, and the FWHM of the target's lateral profile.
//
// The statistics need each other in sequence -- means and maxima, then the
// deviations and the amplitude histograms, then the overlap and the
// half-maximum walk -- so there are two kernels over both regions and one
// workgroup for the rest.  (The rest in the last workgroup of the second kernel
// to finish would save a launch, but the fences and tickets that takes cost
// more: that kernel took 17 us with 40 workgroups and 30 with 157.)  Sums are
// float64 and formed in a fixed order; the amplitude bins use a float64
// division, so a pixel lands in the same bin as in a float64 reference.
//
// Bound by latency, not by rate (a few hundred thousand pixels): a 160 x 160
// target and a 400 x 400 background take 5, 5 and 6 us in the three kernels
// and 34 us a call; one workgroup for everything took 157 us, and 183 us a call
// with an allocation, a copy and a free.  (1024 or 4096 pixels per workgroup
// instead of 2048: 34.3 and 35.4 us a call.)
#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstring>
#include <mutex>

#include "hodmas.h"

namespace {

constexpr int kMetBlock = 512;
constexpr int kMetPixels = 2048;     // pixels per workgroup ...
constexpr int kMetBlocks = 256;      // ... and the most workgroups
constexpr int kMaxBins = 4096;

struct Rect {
    int ix0, ix1, iz0, iz1;
    __host__ __device__ int count() const { return (ix1 - ix0) * (iz1 - iz0); }
    __device__ int64_t at(int q, int nx) const   // q-th pixel in row-major order
    {
        const int w = ix1 - ix0;
        return (int64_t)(iz0 + q / w) * nx + ix0 + q % w;
    }
};

// Sums and maxima of the regions, and the target's first maximum (its pixel
// number, or the target's pixel count where no pixel equals the maximum).
struct Extent {
    double sum_t, sum_b, max_t, max_b;
    int first, pad;
};

// What one call keeps on the device.  The first kernel clears hist.
struct Scratch {
    Extent part[kMetBlocks];
    double dev[kMetBlocks];
    unsigned hist[2][kMaxBins];
};

__device__ __forceinline__ Extent joined(const Extent& a, const Extent& b)
{
    Extent r;
    r.sum_t = a.sum_t + b.sum_t;
    r.sum_b = a.sum_b + b.sum_b;
    r.max_t = fmax(a.max_t, b.max_t);
    r.max_b = fmax(a.max_b, b.max_b);
    r.first = a.max_t > b.max_t ? a.first : b.max_t > a.max_t ? b.first : min(a.first, b.first);
    r.pad = 0;
    return r;
}

// What the last kernel joins: deviations, histogram overlap, and the steps
// from the maximum to the nearest sample at or below half of it on either side.
struct Tail {
    double sq, overlap;
    int left, right;
};
__device__ __forceinline__ Tail joined(const Tail& a, const Tail& b)
{
    return {a.sq + b.sq, a.overlap + b.overlap, min(a.left, b.left), min(a.right, b.right)};
}
__device__ __forceinline__ double joined(double a, double b) { return a + b; }

// The block's values joined, in a fixed order; every thread gets the result.
template <class V>
__device__ V block_join(V v, V* sh)
{
    static_assert(sizeof(V) % 4 == 0, "whole dwords");
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        int w[sizeof(V) / 4];
        __builtin_memcpy(w, &v, sizeof(V));
#pragma unroll
        for (int i = 0; i < int(sizeof(V) / 4); ++i)
            w[i] = __shfl_xor(w[i], off);
        V o;
        __builtin_memcpy(&o, w, sizeof(V));
        v = joined(v, o);
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0)
        sh[threadIdx.x >> 6] = v;
    __syncthreads();
    V r = sh[0];
    for (int i = 1; i < kMetBlock / 64; ++i)
        r = joined(r, sh[i]);
    return r;
}

__device__ __forceinline__ Extent nothing(int nt) { return {0.0, 0.0, -HUGE_VAL, -HUGE_VAL, nt, 0}; }

// Means and maxima: one Extent per workgroup.
__global__ __launch_bounds__(kMetBlock) void metrics_extent_kernel(const float* __restrict__ img, int nx, Rect tr,
                                                                   Rect br, int bins, Scratch* __restrict__ s)
{
    __shared__ Extent sh[kMetBlock / 64];
    const int nt = tr.count(), nb = br.count();
    const int first = blockIdx.x * kMetBlock + threadIdx.x, step = gridDim.x * kMetBlock;
    for (int i = first; i < 2 * bins; i += step)
        s->hist[i / bins][i % bins] = 0u;
    Extent e = nothing(nt);
    // 64 bits: a step past the last pixel of a large region passes 2^31
    for (int64_t q = first; q < nt; q += step) {
        const double v = img[tr.at((int)q, nx)];
        e.sum_t += v;
        if (v > e.max_t || (v == e.max_t && e.first == nt)) {
            e.max_t = v;
            e.first = (int)q;
        }
    }
    for (int64_t q = first; q < nb; q += step) {
        const double v = img[br.at((int)q, nx)];
        e.sum_b += v;
        e.max_b = fmax(e.max_b, v);
    }
    e = block_join(e, sh);
    if (threadIdx.x == 0)
        s->part[blockIdx.x] = e;
}

// Deviations from the background's mean, and histograms of the normalised
// amplitude.
__global__ __launch_bounds__(kMetBlock) void metrics_histogram_kernel(const float* __restrict__ img, int nx, Rect tr,
                                                                      Rect br, int bins, Scratch* __restrict__ s)
{
    __shared__ Extent she[kMetBlock / 64];
    __shared__ double sh[kMetBlock / 64];
    __shared__ unsigned hist[2][kMaxBins];
    const int tid = threadIdx.x, blocks = gridDim.x;
    const int nt = tr.count(), nb = br.count();
    const int first = blockIdx.x * kMetBlock + tid, step = blocks * kMetBlock;
    static_assert(kMetBlocks <= kMetBlock, "one Extent per thread");
    const Extent e = block_join(tid < blocks ? s->part[tid] : nothing(nt), she);
    const double mu_out = e.sum_b / nb;
    const double peak = fmax(e.max_t, e.max_b);
    for (int i = tid; i < bins; i += kMetBlock) {
        hist[0][i] = 0u;
        hist[1][i] = 0u;
    }
    __syncthreads();
    auto bin = [&](double v) { return min(max((int)(v / peak * bins), 0), bins - 1); };
    if (peak > 0.0)
        for (int64_t q = first; q < nt; q += step)
            atomicAdd(&hist[0][bin(img[tr.at((int)q, nx)])], 1u);
    double dev = 0.0;
    for (int64_t q = first; q < nb; q += step) {
        const double v = img[br.at((int)q, nx)], d = v - mu_out;
        dev += d * d;
        if (peak > 0.0)
            atomicAdd(&hist[1][bin(v)], 1u);
    }
    dev = block_join(dev, sh);             // its barriers also end the histograms
    for (int i = tid; i < bins; i += kMetBlock) {
#pragma unroll
        for (int r = 0; r < 2; ++r)
            if (hist[r][i])
                atomicAdd(&s->hist[r][i], hist[r][i]);
    }
    if (tid == 0)
        s->dev[blockIdx.x] = dev;
}

// One workgroup: the results.
__global__ __launch_bounds__(kMetBlock) void metrics_result_kernel(const float* __restrict__ img, int nx, Rect tr,
                                                                   Rect br, int bins, double dx, int blocks,
                                                                   const Scratch* __restrict__ s,
                                                                   hodmas_metrics* __restrict__ out)
{
    __shared__ Extent she[kMetBlock / 64];
    __shared__ Tail sht[kMetBlock / 64];
    const int tid = threadIdx.x;
    const int nt = tr.count(), nb = br.count();
    const Extent e = block_join(tid < blocks ? s->part[tid] : nothing(nt), she);
    const double mu_in = e.sum_t / nt, mu_out = e.sum_b / nb;
    const double peak = fmax(e.max_t, e.max_b);
    Tail t{tid < blocks ? s->dev[tid] : 0.0, 0.0, nx, nx};
    for (int i = tid; i < bins; i += kMetBlock)
        t.overlap += fmin((double)s->hist[0][i] / nt, (double)s->hist[1][i] / nb);
    // FWHM along the row through the target's first maximum (the region's first
    // pixel where none equals it: NaNs): the nearest sample at or below half
    // of it to either side
    const int64_t p = tr.at(e.first < nt ? e.first : 0, nx);
    const int iz = (int)(p / nx), ix = (int)(p - (int64_t)iz * nx);
    const float* row = img + (int64_t)iz * nx;
    const double half = 0.5 * (double)row[ix];
    for (int x = tid; x < nx; x += kMetBlock) {
        if ((double)row[x] <= half) {
            if (x < ix)
                t.left = min(t.left, ix - x);
            else if (x > ix)
                t.right = min(t.right, x - ix);
        }
    }
    t = block_join(t, sht);
    const double sigma_out = sqrt(t.sq / nb);
    if (tid == 0) {
        auto edge = [&](int steps, int dir) {
            if (steps == nx)
                return dir > 0 ? (double)(nx - 1) : 0.0;   // the image's edge
            const int j = ix + dir * (steps - 1);
            const double a = row[j], b = row[j + dir];
            return j + dir * (a - half) / (a - b);
        };
        hodmas_metrics m;
        m.mu_in = mu_in;
        m.mu_out = mu_out;
        m.sigma_out = sigma_out;
        m.snr_db = 20.0 * log10(mu_in / sigma_out);
        m.cr_db = 20.0 * log10(mu_in / mu_out);
        m.gcnr = peak > 0.0 ? 1.0 - t.overlap : 0.0;
        m.fwhm_m = (edge(t.right, 1) - edge(t.left, -1)) * dx;
        *out = m;
    }
}

bool rect_ok(const hodmas_rect* r, int nx, int nz)
{
    return r && r->ix0 >= 0 && r->ix0 < r->ix1 && r->ix1 <= nx && r->iz0 >= 0 && r->iz0 < r->iz1 &&
           r->iz1 <= nz;
}

// A call's scratch and the pinned host memory its result arrives in.  Each
// device holds kSlots of them in a file-scope array, taken for the length of
// one call, so up to kSlots host threads evaluate at once with no allocation;
// one more allocates its own and frees it.
constexpr int kSlots = 8;
constexpr int kMaxDevices = 64;
__device__ Scratch slots[kSlots];

struct Device {
    Scratch* scratch = nullptr;            // `slots` on this device
    hodmas_metrics* result = nullptr;      // pinned, kSlots
};
std::mutex g_mu;
Device g_device[kMaxDevices];
unsigned g_taken[kMaxDevices];             // bit i: slot i is in use

class Workspace {
  public:
    explicit Workspace(int dev) : dev_(dev)
    {
        if (dev >= 0 && dev < kMaxDevices) {
            std::lock_guard<std::mutex> lock(g_mu);
            Device& d = g_device[dev];
            if (!d.scratch) {
                void* ptr = nullptr;
                hodmas_metrics* host = nullptr;
                if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(slots)) == hipSuccess && ptr &&
                    hipHostMalloc((void**)&host, sizeof(hodmas_metrics) * kSlots, hipHostMallocPortable) == hipSuccess) {
                    d.scratch = static_cast<Scratch*>(ptr);
                    d.result = host;
                } else {
                    (void)hipGetLastError();   // the call's own launches are checked with it
                }
            }
            for (int i = 0; d.scratch && i < kSlots && slot_ < 0; ++i) {
                if (!(g_taken[dev] & (1u << i))) {
                    g_taken[dev] |= 1u << i;
                    slot_ = i;
                    scratch = d.scratch + i;
                    result = d.result + i;
                }
            }
        }
        if (slot_ < 0 && (hipMalloc((void**)&scratch, sizeof(Scratch)) != hipSuccess ||
                          hipHostMalloc((void**)&result, sizeof(hodmas_metrics), hipHostMallocPortable) != hipSuccess)) {
            (void)hipGetLastError();
            if (scratch)
                (void)hipFree(scratch);
            scratch = nullptr;
        }
    }
    ~Workspace()
    {
        if (slot_ >= 0) {
            std::lock_guard<std::mutex> lock(g_mu);
            g_taken[dev_] &= ~(1u << slot_);
        } else if (scratch) {
            (void)hipFree(scratch);
            (void)hipHostFree(result);
        }
    }
    Workspace(const Workspace&) = delete;
    Workspace& operator=(const Workspace&) = delete;
    Scratch* scratch = nullptr;            // null: no memory
    hodmas_metrics* result = nullptr;

  private:
    int dev_, slot_ = -1;
};

}  // namespace

extern "C" hodmas_status hodmas_image_metrics(const float* image_dev, int32_t nx, int32_t nz, double dx_m,
                                              const hodmas_rect* target, const hodmas_rect* background,
                                              int32_t bins, void* stream, hodmas_metrics* out)
{
    if (!image_dev || !out || nx < 1 || nz < 1 || !(dx_m > 0.0) || bins < 2 || bins > kMaxBins ||
        !rect_ok(target, nx, nz) || !rect_ok(background, nx, nz))
        return HODMAS_EINVAL;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess)
        return HODMAS_EDEVICE;
    Workspace ws(dev);
    if (!ws.scratch)
        return HODMAS_ENOMEM;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const Rect tr{target->ix0, target->ix1, target->iz0, target->iz1};
    const Rect br{background->ix0, background->ix1, background->iz0, background->iz1};
    const int64_t most = tr.count() > br.count() ? tr.count() : br.count();
    const int64_t want = (most + kMetPixels - 1) / kMetPixels;
    const dim3 grid((unsigned)(want < 1 ? 1 : want > kMetBlocks ? kMetBlocks : want));
    hipLaunchKernelGGL(metrics_extent_kernel, grid, dim3(kMetBlock), 0, st, image_dev, nx, tr, br, bins, ws.scratch);
    bool ok = hipGetLastError() == hipSuccess;
    if (ok) {
        hipLaunchKernelGGL(metrics_histogram_kernel, grid, dim3(kMetBlock), 0, st, image_dev, nx, tr, br, bins,
                           ws.scratch);
        ok = hipGetLastError() == hipSuccess;
    }
    if (ok) {
        hipLaunchKernelGGL(metrics_result_kernel, dim3(1), dim3(kMetBlock), 0, st, image_dev, nx, tr, br, bins, dx_m,
                           (int)grid.x, ws.scratch, ws.result);
        ok = hipGetLastError() == hipSuccess;
    }
    // the slot is given back only once nothing can still be writing to it
    ok = hipStreamSynchronize(st) == hipSuccess && ok;
    if (!ok) {
        (void)hipGetLastError();
        return HODMAS_EDEVICE;
    }
    std::memcpy(out, ws.result, sizeof(*out));
    return HODMAS_OK;
}
