// State copies (checkpoints) and the window-mean score of the drag series.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "../../include/lbm.h"
#include "api_internal.hpp"

using namespace lbm;

extern "C" int lbm_copy_state_out(const lbm_ctx* c, int32_t m, float* dst_dev) {
    if (!c || !dst_dev) return lbm_fail(LBM_EINVAL, "NULL argument");
    if (m < 0 || m >= c->n) return lbm_fail(LBM_EINVAL, "member %d out of range", m);
    const MemberDev& md = c->h_members[m];
    const size_t bytes = sizeof(float) * 9 * (size_t)md.nx * md.ny;
    hipError_t e = hipMemcpyAsync(dst_dev, c->pop[c->h_parity[m]] + md.off, bytes, hipMemcpyDeviceToDevice, c->stream);
    return e == hipSuccess ? LBM_OK : lbm_hip_fail(e, "state copy out");
}

extern "C" int lbm_copy_state_in(lbm_ctx* c, int32_t m, const float* src_dev, int32_t t) {
    if (!c || !src_dev) return lbm_fail(LBM_EINVAL, "NULL argument");
    if (m < 0 || m >= c->n) return lbm_fail(LBM_EINVAL, "member %d out of range", m);
    if (t < 0 || t > c->cap) return lbm_fail(LBM_EINVAL, "time %d outside [0, %d]", t, c->cap);
    const MemberDev& md = c->h_members[m];
    const size_t bytes = sizeof(float) * 9 * (size_t)md.nx * md.ny;
    hipError_t e = hipMemcpyAsync(c->pop[c->h_parity[m]] + md.off, src_dev, bytes, hipMemcpyDeviceToDevice, c->stream);
    if (e != hipSuccess) return lbm_hip_fail(e, "state copy in");
    if ((e = set_int(c->d_cursor + m, t, c->stream)) != hipSuccess) return lbm_hip_fail(e, "cursor set");
    c->h_cursor[m] = t;
    return LBM_OK;
}

namespace lbm {

// Each thread owns WM_RUN consecutive outputs: the first window is summed in
// FP64, the others slide (+ the new sample, - the oldest); the FP64 sliding
// error (a few ulps of the running sum) is far below the FP32 output rounding,
// and a sample that is not finite reaches only the runs whose windows hold it.
constexpr int WM_RUN = 16;
constexpr int WM_OUT = 256 * WM_RUN;      // outputs of a workgroup
constexpr int WM_SPAN = 13 * 1024;        // samples a workgroup holds in LDS at most (63 KB with the run sums)

// LDS form: a workgroup brings the samples of its outputs' windows into LDS
// (sample p at p + p / 16, so that threads 16 samples apart use different
// banks) with the sums of aligned runs of 16, and a first window is its head,
// the runs inside it and its tail: window / 16 + 30 additions at most, from
// LDS, instead of `window` dependent ones from memory.  512 rows of 2560
// samples, window 512: 103 -> 15 us.
__global__ __launch_bounds__(256) void window_mean_lds_kernel(const float* series, int n, int ld, int t_len, int window,
                                                              float* out) {
    extern __shared__ double seg[];  // run sums, then the samples
    const int t_first = (int)blockIdx.x * WM_OUT, nt = (int)blockDim.x, t = (int)threadIdx.x;
    const int t_end = t_first + min(t_len - t_first, WM_OUT);
    const int base = max(0, t_first - window + 1);
    const int span = t_end - base, nseg = (span + 15) / 16;
    float* const v = (float*)(seg + nseg);
    auto at = [](int p) { return p + (p >> 4); };
    const double inv = 1.0 / (double)window;
    for (int m = (int)blockIdx.y; m < n; m += (int)gridDim.y) {  // rows beyond the grid's height
        const float* row = series + (long long)m * ld + base;
        float* orow = out + (long long)m * t_len;
        for (int p = t; p < span; p += nt) v[at(p)] = row[p];
        __syncthreads();
        for (int s = t; s < span / 16; s += nt) {
            double acc = 0.0;
#pragma unroll
            for (int k = 0; k < 16; ++k) acc += (double)v[17 * s + k];
            seg[s] = acc;
        }
        __syncthreads();
        const int t0 = t_first + t * WM_RUN, t1 = min(t_end, t0 + WM_RUN);
        double acc = 0.0;
        bool have = false;
        for (int q = t0; q < t1; ++q) {
            if (q < window - 1) {
                orow[q] = -INFINITY;
                continue;
            }
            const int p = q - base;  // the newest sample of the window
            if (!have) {
                int lo = p - window + 1;
                const int hi = p + 1;  // [lo, hi)
                for (; lo < hi && (lo & 15); ++lo) acc += (double)v[at(lo)];
                for (; lo + 16 <= hi; lo += 16) acc += seg[lo >> 4];
                for (; lo < hi; ++lo) acc += (double)v[at(lo)];
                have = true;
            } else {
                acc += (double)v[at(p)] - (double)v[at(p - window)];
            }
            orow[q] = (float)(acc * inv);
        }
        __syncthreads();  // the next row overwrites the samples
    }
}

// From memory: windows too long for LDS.
__global__ __launch_bounds__(256) void window_mean_kernel(const float* series, int n, int ld, int t_len, int window,
                                                          float* out) {
    const long long t0 = ((long long)blockIdx.x * blockDim.x + threadIdx.x) * WM_RUN;
    if (t0 >= t_len) return;
    const int t1 = (int)min((long long)t_len, t0 + WM_RUN);
    const double inv = 1.0 / (double)window;
    for (int m = (int)blockIdx.y; m < n; m += (int)gridDim.y) {  // rows beyond the grid's height
        const float* row = series + (long long)m * ld;
        float* orow = out + (long long)m * t_len;
        double acc = 0.0;
        bool have = false;
        for (int t = (int)t0; t < t1; ++t) {
            if (t < window - 1) {
                orow[t] = -INFINITY;
                continue;
            }
            if (!have) {
                for (int k = t - window + 1; k <= t; ++k) acc += (double)row[k];
                have = true;
            } else {
                acc += (double)row[t] - (double)row[t - window];
            }
            orow[t] = (float)(acc * inv);
        }
    }
}

}  // namespace lbm

extern "C" int lbm_window_mean(const float* series_dev, int32_t n, int32_t ld, int32_t t_len, int32_t window,
                               float* out_dev, void* hip_stream) {
    if (!series_dev || !out_dev) return lbm_fail(LBM_EINVAL, "NULL argument");
    if (n < 0 || t_len < 0 || ld < t_len || window < 1) return lbm_fail(LBM_EINVAL, "bad sizes");
    if (n == 0 || t_len == 0) return LBM_OK;
    const unsigned runs = (unsigned)((t_len + WM_RUN - 1) / WM_RUN);
    // the samples a workgroup needs: its outputs and the window before the first of them
    const long long span = std::min<long long>(t_len, (long long)std::min(t_len, WM_OUT) + window - 1);
    if (span <= WM_SPAN) {
        const size_t lds = sizeof(double) * (size_t)((span + 15) / 16) + sizeof(float) * (size_t)(span + span / 16 + 1);
        const unsigned threads = std::min(256u, (runs + 63) / 64 * 64);
        hipLaunchKernelGGL(window_mean_lds_kernel, dim3((unsigned)((t_len + WM_OUT - 1) / WM_OUT), (unsigned)std::min(n, 65535)),
                           dim3(threads), lds, (hipStream_t)hip_stream, series_dev, n, ld, t_len, window, out_dev);
        hipError_t e = hipGetLastError();
        return e == hipSuccess ? LBM_OK : lbm_hip_fail(e, "window mean kernel");
    }
    hipLaunchKernelGGL(window_mean_kernel, dim3((runs + 255) / 256, (unsigned)std::min(n, 65535)), dim3(256), 0,
                       (hipStream_t)hip_stream, series_dev, n, ld, t_len, window, out_dev);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? LBM_OK : lbm_hip_fail(e, "window mean kernel");
}
