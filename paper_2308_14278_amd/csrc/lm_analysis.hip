// lm_analysis.hip -- light-curve peak identification on a count map (Sec. 4.2).
//
// A light curve is row i of the row-major map counts[i][j] (fixed source index
// along the caustic, j across it).  Candidate peak: N_ij > max(N_i,j-1, N_i,j+1)
// and h_ij > k sigma_ij with h_ij = N_ij - <N>, <N> the mean of the three
// counts and sigma_ij = sqrt(<N>); with S the sum of the three counts this is
// (3 N_ij - S)^2 > 3 k^2 S, decided exactly in integers.  True peak: a
// candidate with a candidate among (i-1, j-1..j+1) and among (i+1, j-1..j+1).
//
// k_peak_stats gathers the statistics of Sec. 4.2 (Figs. 4 and 5): the true
// peaks of the listed light curves per bin of distance to the caustic and the
// sum of their counts, both exact integers.
//
// Both kernels are latency-bound (ten curves of a 3694-pixel map read 0.9 MB):
// what a call costs is its copies, launches and waits.  Each call is one launch
// that takes short lists by value and writes its results to the caller's
// (pinned) memory.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <mutex>

#include "lm_internal.h"

namespace {

// Scratch memory of the allocation-free peak statistics: the listed rows, the
// first pixel column of every bin and the two histograms, at fixed offsets.  Each
// device holds its own copy; host code reaches it only through the address
// hipGetSymbolAddress returns on that device.
static __device__ __align__(256) unsigned char scratch[LM_SCRATCH_BYTES];

std::mutex g_scratch_mu;
void* g_scratch_ptr[LM_MAX_DEVICES] = {};

__device__ __forceinline__ bool candidate(const unsigned long long* __restrict__ c, int64_t nx,
                                          int64_t i, int64_t j, unsigned k2x3)
{
    if (j <= 0 || j >= nx - 1) return false;
    const unsigned long long* row = c + i * nx;
    const unsigned long long a = row[j - 1], n = row[j], b = row[j + 1];
    if (!(n > a && n > b)) return false;
    const unsigned __int128 s = (unsigned __int128)a + n + b;
    const unsigned __int128 n3 = (unsigned __int128)n * 3u;
    if (n3 <= s) return false;
    const unsigned __int128 t = n3 - s;
    // 3 k^2 S < 2^90 for k <= 1000, so any t >= 2^64 passes
    if ((unsigned long long)(t >> 64) != 0ull) return true;
    const unsigned long long tl = (unsigned long long)t;
    return (unsigned __int128)tl * tl > (unsigned __int128)k2x3 * s;
}

__device__ __forceinline__ bool true_peak(const unsigned long long* __restrict__ c, int64_t nx,
                                          int64_t ny, int64_t i, int64_t j, unsigned k2x3)
{
    if (!(i > 0 && i < ny - 1) || !candidate(c, nx, i, j, k2x3)) return false;
    const bool left = candidate(c, nx, i - 1, j - 1, k2x3) || candidate(c, nx, i - 1, j, k2x3) ||
                      candidate(c, nx, i - 1, j + 1, k2x3);
    return left && (candidate(c, nx, i + 1, j - 1, k2x3) || candidate(c, nx, i + 1, j, k2x3) ||
                    candidate(c, nx, i + 1, j + 1, k2x3));
}

// Flags of pixels j of the listed rows: one light curve per grid row (more than
// 65535 in turns), the rows from `tracks` or, if null, from the argument.
__global__ __launch_bounds__(256) void k_peaks(const unsigned long long* __restrict__ counts,
                                               int64_t nx, int64_t ny, LmTracks rows,
                                               const int32_t* __restrict__ tracks, int64_t nt,
                                               unsigned k2x3, uint8_t* __restrict__ flags)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j >= nx) return;
    for (int64_t t = blockIdx.y; t < nt; t += gridDim.y) {
        const int64_t i = tracks ? tracks[t] : rows.row[t];
        uint8_t f = 0;
        if (candidate(counts, nx, i, j, k2x3)) f = true_peak(counts, nx, ny, i, j, k2x3) ? 3 : 1;
        flags[t * nx + j] = f;
    }
}

// Statistics of the listed rows over the pixel columns [col[0], col[nb]); column
// p belongs to the last bin b with col[b] <= p.  True peaks are rare, so they
// search their bin and add to hist (peaks[nb], heights[nb]) with global atomics.
// With `done`, the last workgroup to finish moves the sums to out, leaving hist and
// *done zero as it found them; without (more bins than one workgroup moves in a few
// steps), k_peak_out does.
__global__ __launch_bounds__(256) void k_peak_stats(const unsigned long long* __restrict__ counts,
                                                    int64_t nx, int64_t ny, LmTracks rows,
                                                    const int32_t* __restrict__ tracks, int64_t nt,
                                                    unsigned k2x3, LmBins bins,
                                                    const int32_t* __restrict__ cols, int c0, int c1,
                                                    int nb, unsigned long long* hist,
                                                    unsigned* done, unsigned long long* out)
{
    __shared__ bool last;
    const int64_t j = c0 + (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (j < c1) {
        for (int64_t t = blockIdx.y; t < nt; t += gridDim.y) {
            const int64_t i = tracks ? tracks[t] : rows.row[t];
            if (!true_peak(counts, nx, ny, i, j, k2x3)) continue;
            int lo = 0, hi = nb - 1;  // the last b with col[b] <= j (col[0] <= j < col[nb])
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if ((cols ? cols[mid] : bins.col[mid]) <= j)
                    lo = mid;
                else
                    hi = mid - 1;
            }
            atomicAdd(&hist[lo], 1ull);
            atomicAdd(&hist[nb + lo], counts[i * nx + j]);
            // a wave waits for its own additions: the barrier does not, and the fence
            // before the count below waits for the first wave's alone.  Here, where
            // additions are rare, it costs nothing measurable (flags and statistics
            // of ten curves 58.6 us; with every wave's fence at the barrier 60.3)
            __threadfence();
        }
    }
    if (!done) return;
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        last = atomicAdd(done, 1u) == gridDim.x * gridDim.y - 1u;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();
    for (int b = threadIdx.x; b < 2 * nb; b += 256) out[b] = atomicExch(&hist[b], 0ull);
    if (threadIdx.x == 0) atomicExch(done, 0u);
}

// The sums of k_peak_stats to out, hist left zero.
__global__ __launch_bounds__(256) void k_peak_out(unsigned long long* __restrict__ hist, int n,
                                                  unsigned long long* __restrict__ out)
{
    const int i = (int)(blockIdx.x * 256 + threadIdx.x);
    if (i >= n) return;
    out[i] = hist[i];
    hist[i] = 0;
}

__global__ __launch_bounds__(256) void k_copy_i32(const int32_t* __restrict__ src, int64_t n,
                                                  int32_t* __restrict__ dst)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

}  // namespace

int lm_launch_peak_stats(const unsigned long long* counts, int64_t nx, int64_t ny,
                         const LmTracks& rows, const int32_t* tracks, int64_t nt, int k,
                         const LmBins& bins, const int32_t* cols, int c0, int c1, int nb,
                         unsigned long long* hist, unsigned* done, unsigned long long* out,
                         void* stream)
{
    if (nt <= 0) return 0;
    // At most 512 workgroups, each with every few-th row: their counts of `done` wait
    // for one another (us a call, 300 rows of 4000 pixels: 132 with a workgroup to
    // every 256 pixels, 42.5 so).  Up to kHandOff bins the last of them moves the
    // sums (a launch less), more take a kernel of their own (us a call, 64 x 64 pixels,
    // 20000 bins: 174 and 72).
    constexpr int kHandOff = 1024;
    const int64_t gx = ((c1 > c0 ? c1 - c0 : 1) + 255) / 256;
    int64_t gy = gx < 512 ? 512 / gx : 1;
    if (gy > nt) gy = nt;
    const dim3 grid((unsigned)gx, (unsigned)gy);
    hipStream_t s = (hipStream_t)stream;
    const bool hand = nb <= kHandOff;
    hipLaunchKernelGGL(k_peak_stats, grid, dim3(256), 0, s, counts, nx, ny, rows, tracks, nt,
                       (unsigned)(3 * k * k), bins, cols, c0, c1, nb, hist, hand ? done : nullptr,
                       out);
    if (hand) return (int)hipGetLastError();
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
    hipLaunchKernelGGL(k_peak_out, dim3((unsigned)((2 * nb + 255) / 256)), dim3(256), 0, s, hist,
                       2 * nb, out);
    return (int)hipGetLastError();
}

int lm_launch_copy_i32(const int32_t* src, int64_t n, int32_t* dst, void* stream)
{
    if (n <= 0) return 0;
    hipLaunchKernelGGL(k_copy_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0,
                       (hipStream_t)stream, src, n, dst);
    return (int)hipGetLastError();
}

int lm_launch_peaks(const unsigned long long* counts, int64_t nx, int64_t ny, const LmTracks& rows,
                    const int32_t* tracks, int64_t nt, int k, uint8_t* flags, void* stream)
{
    if (nt <= 0 || nx <= 0) return 0;
    const dim3 grid((unsigned)((nx + 255) / 256), (unsigned)(nt < 65535 ? nt : 65535));
    hipLaunchKernelGGL(k_peaks, grid, dim3(256), 0, (hipStream_t)stream, counts, nx, ny, rows,
                       tracks, nt, (unsigned)(3 * k * k), flags);
    return (int)hipGetLastError();
}

int lm_scratch_address(void** out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev < 0 || dev >= LM_MAX_DEVICES) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return (int)e;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return 0;
}
