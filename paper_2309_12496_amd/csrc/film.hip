// Film read-out emulation (Section 4.4): the paper images the detector plane
// with a pinhole camera and a film, and counts pixels above an intensity
// threshold as hits.  Detected photons are projected onto the film and
// splatted with a Gaussian reconstruction filter; a second pass thresholds.
#include <hip/hip_runtime.h>

#include "kernels.h"
#include "rich_dev.h"

namespace rich {

namespace {

constexpr int kFilmBlock = 256;
constexpr uint64_t kStripMin = uint64_t(1) << 15;   // photons from which the film is splatted by strips

// The film pixels [i0, i1] x [j0, j1] whose centres lie within 4 sigma of
// (x, y) in x and in y; false for a hit that reaches none (NaN, far outside).
struct Window {
    int i0, i1, j0, j1;
};
__device__ __forceinline__ bool film_window(const FilmArgs &a, float x, float y, Window &w) {
    if (!(fabsf(x) < 1e9f && fabsf(y) < 1e9f)) return false;
    w.i0 = max((int)ceilf(x - a.radius - 0.5f), 0);
    w.i1 = min((int)floorf(x + a.radius - 0.5f), a.width - 1);
    w.j0 = max((int)ceilf(y - a.radius - 0.5f), 0);
    w.j1 = min((int)floorf(y + a.radius - 0.5f), a.height - 1);
    return true;
}

// Adds 255 exp(-r^2 / 2 sigma^2) to the pixels of a window's rows [j0, j1].
template <class Add>
__device__ __forceinline__ void splat(const FilmArgs &a, float x, float y, int i0, int i1, int j0, int j1, Add &&add) {
    for (int j = j0; j <= j1; ++j) {
        const float dy = (float)j + 0.5f - y;
        for (int i = i0; i <= i1; ++i) {
            const float dx = (float)i + 0.5f - x;
            add(j, i, 255.0f * __expf(-(dx * dx + dy * dy) * a.inv_2s2));
        }
    }
}

// One thread per photon, straight into the image.
__global__ __launch_bounds__(kFilmBlock) void film_splat_kernel(FilmArgs a, const uint8_t *fate, const float *uv,
                                                                uint64_t n, float *image) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += stride) {
        if (fate[p] != 0) continue;   // DETECTED only
        const float x = fmaf(a.scale, uv[2 * p], a.cx), y = fmaf(a.scale, uv[2 * p + 1], a.cy);
        Window w;
        if (!film_window(a, x, y, w)) continue;
        splat(a, x, y, w.i0, w.i1, w.j0, w.j1,
              [&](int j, int i, float v) { atomicAdd(image + (size_t)j * a.width + i, v); });
    }
}

// The same for many photons, which one atomic on the image per photon and
// pixel binds (25 a photon; 13e9 a second on a ring, 33e9 spread out).  The image
// is cut into strips of whole rows that fit a block's LDS and the photons into
// slices; a block goes through one slice, keeps what falls into its strip in
// LDS, and adds each pixel it touched to the image once.  Every photon is read
// once per strip, so the blocks of a slice follow each other on one XCD (block
// b runs on XCD b mod 8), whose L2 serves all but the first.  Few photons of a
// slice lie in the strip: a wave queues them and splats 64 at a time.  What
// binds now is that search, a photon per thread and strip, and for a film full
// of hits the additions in LDS.
// With the threshold pass, 2,000,003 photons on 1320 x 620 pixels: 11 %
// detected on a ring 499 -> 83 us, all detected, spread out 1510 -> 184 us.
constexpr int kStripBlock = 1024, kStripWords = 36000, kStripQueue = 128, kStripUnroll = 8;
constexpr int kStripBlocks = 256;   // one a CU
constexpr size_t kStripLds = kStripWords * sizeof(float) + (size_t)(kStripBlock / 64) * kStripQueue * sizeof(float2);

__global__ __launch_bounds__(kStripBlock) void film_strip_kernel(FilmArgs a, const uint8_t *fate, const float *uv,
                                                                 uint64_t n, float *image, int rows, int strips,
                                                                 int slices) {
    extern __shared__ float strip[];
    float2 *const queue = reinterpret_cast<float2 *>(strip + kStripWords) + (threadIdx.x >> 6) * kStripQueue;
    const int lane = threadIdx.x & 63;
    const int job = (int)(blockIdx.x % 8 * (gridDim.x / 8) + blockIdx.x / 8);
    const int slice = job / strips;
    if (slice >= slices) return;
    const int r0 = job % strips * rows, r1 = min(r0 + rows, a.height) - 1;   // rows r0..r1
    const int words = (r1 - r0 + 1) * a.width;
    for (int k = threadIdx.x; k < words; k += kStripBlock) strip[k] = 0.0f;
    __syncthreads();
    // hits further than this from the strip's middle row have no pixel in it
    // (a pixel more than the window's reach for the roundings)
    const float mid = 0.5f * (float)(r0 + r1 + 1), reach = 0.5f * (float)(r1 - r0 + 1) + a.radius + 1.0f;
    int queued = 0;   // of this wave (uniform)
    auto flush = [&](int count) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        if (lane < count) {
            const float2 h = queue[queued - count + lane];
            Window w;
            if (film_window(a, h.x, h.y, w))
                splat(a, h.x, h.y, w.i0, w.i1, max(w.j0, r0), min(w.j1, r1),
                      [&](int j, int i, float v) { atomicAdd(strip + (j - r0) * a.width + i, v); });
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        queued -= count;
    };
    const uint64_t lo = n / slices * slice + min((uint64_t)slice, n % slices);
    const uint64_t hi = lo + n / slices + ((uint64_t)slice < n % slices ? 1 : 0);
    // a round's positions are fetched while the round before it is searched,
    // and its fates a round earlier still
    constexpr uint64_t kRound = (uint64_t)kStripBlock * kStripUnroll;
    uint8_t fates[kStripUnroll];
    bool on[kStripUnroll], next_on[kStripUnroll];
    float u[kStripUnroll], v[kStripUnroll], next_u[kStripUnroll], next_v[kStripUnroll];
    auto fetch_fates = [&](uint64_t base) {
#pragma unroll
        for (int k = 0; k < kStripUnroll; ++k) {
            const uint64_t p = base + (uint64_t)(k * kStripBlock) + threadIdx.x;
            fates[k] = p < hi ? fate[p] : 255;
        }
    };
    auto fetch = [&](uint64_t base) {
#pragma unroll
        for (int k = 0; k < kStripUnroll; ++k) {
            const uint64_t p = base + (uint64_t)(k * kStripBlock) + threadIdx.x;
            next_on[k] = fates[k] == 0;   // DETECTED only
            if (next_on[k]) {
                next_u[k] = uv[2 * p];
                next_v[k] = uv[2 * p + 1];
            }
        }
        fetch_fates(base + kRound);
    };
    fetch_fates(lo);
    fetch(lo);
    for (uint64_t base = lo; base < hi; base += kRound) {
#pragma unroll
        for (int k = 0; k < kStripUnroll; ++k) {
            on[k] = next_on[k];
            u[k] = next_u[k];
            v[k] = next_v[k];
        }
        fetch(base + kRound);
#pragma unroll
        for (int k = 0; k < kStripUnroll; ++k) {
            const float x = fmaf(a.scale, u[k], a.cx), y = fmaf(a.scale, v[k], a.cy);
            const bool in = on[k] && fabsf(y - mid) <= reach;   // the window itself is cut to the strip later
            const unsigned long long m = __ballot(in);
            if (in) queue[queued + (int)__popcll(m & ((1ull << lane) - 1ull))] = make_float2(x, y);
            queued += (int)__popcll(m);
            if (queued >= 64) flush(64);
        }
    }
    if (queued > 0) flush(queued);
    __syncthreads();
    float *const out = image + (size_t)r0 * a.width;
    for (int k = threadIdx.x; k < words; k += kStripBlock) {
        const float s = strip[k];
        if (s != 0.0f) atomicAdd(out + k, s);
    }
}

__global__ __launch_bounds__(kFilmBlock) void film_threshold_kernel(const float *image, uint64_t n_pix, float threshold,
                                                                    uint8_t *hits) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n_pix; k += stride)
        hits[k] = fminf(image[k], 255.0f) >= threshold ? 1 : 0;
}

}  // namespace

hipError_t launch_film(const FilmArgs &a, const uint8_t *fate, const float *uv, uint64_t n, float *image,
                       uint8_t *hits, hipStream_t st) {
    // Strips for 2^15 photons or more: 32,768 on a ring take 10.1 us against 9.9
    // straight, spread out 14 against 27; 16,384 on a ring 9.5 against 8.6; 65,536
    // 11 against 17 and 20 against 52.  At most 32 strips, since each reads all
    // photons: the search costs up to 3 us per strip and 2e6 photons, which at
    // 128 strips would be what the image atomics take.
    const int rows = kStripWords / a.width;
    const int strips = rows > 0 ? (a.height + rows - 1) / rows : 0;
    if (n >= kStripMin && strips >= 1 && strips <= 32) {
        const int slices = kStripBlocks / strips;
        hipLaunchKernelGGL(film_strip_kernel, dim3(kStripBlocks), dim3(kStripBlock), kStripLds, st, a,
                           fate, uv, n, image, rows, strips, slices);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    } else if (n > 0) {
        uint64_t blocks = (n + kFilmBlock - 1) / kFilmBlock;
        if (blocks > 4096) blocks = 4096;
        hipLaunchKernelGGL(film_splat_kernel, dim3((unsigned)blocks), dim3(kFilmBlock), 0, st, a, fate, uv, n, image);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (hits) {
        const uint64_t n_pix = (uint64_t)a.width * a.height;
        uint64_t blocks = (n_pix + kFilmBlock - 1) / kFilmBlock;
        if (blocks > 4096) blocks = 4096;
        hipLaunchKernelGGL(film_threshold_kernel, dim3((unsigned)blocks), dim3(kFilmBlock), 0, st, image, n_pix,
                           a.threshold, hits);
        return hipGetLastError();
    }
    return hipSuccess;
}

}  // namespace rich
