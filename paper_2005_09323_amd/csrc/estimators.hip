// GKTL estimators on the device (paper Appendix C.1-C.2), in FP64.
//
// After a GKTL run the drag series of every slot is a patchwork of the
// trajectories that occupied the slot in each period.  The final ensemble's
// trajectories are rebuilt by walking the ancestors back; each carries the
// time integral of the observable along its lineage and the maximum of its
// window-averaged drag; the unbiased tail probability is the sum of
// exp(sum_i ln R_i - k int A) over trajectories above each level.
#include "estimators.hpp"

namespace lbm {

// Block = final trajectory j.  Lineage slot of each period, the rebuilt drag
// series and the integral of A along the lineage (added in period order).
// The walk back is a chain of dependent reads, one per period: the ancestors
// are brought into LDS first where they fit (a step of the chain then takes
// an LDS read instead of a memory read), and the lineage's integrals are read
// side by side and added by one thread.  24 periods of 256 members: 12.6 ->
// 10.3 us.
constexpr int REBUILD_LDS = 8 * 1024;  // ancestors held in LDS (32 KB)

__global__ __launch_bounds__(256) void gktl_rebuild_kernel(RebuildArgs a, int in_lds) {
    __shared__ int slot[MAX_PERIODS];
    __shared__ double part[256], part_r[256];
    extern __shared__ int anc[];
    const int j = (int)blockIdx.x, t = (int)threadIdx.x;
    if (in_lds) {
#pragma unroll 8
        for (int i = t; i < a.n_periods * a.n; i += 256) anc[i] = a.ancestors[i];
        __syncthreads();
    }
    if (t == 0) {
        int s = j;
        for (int i = a.n_periods - 1; i >= 0; --i) {
            s = in_lds ? anc[i * a.n + s] : a.ancestors[(long long)i * a.n + s];
            slot[i] = s;
        }
    }
    __syncthreads();
    double integ = 0.0, lz = 0.0;
    for (int i0 = 0; i0 < a.n_periods; i0 += 256) {
        const int i = i0 + t, cnt = min(256, a.n_periods - i0);
        if (i < a.n_periods) {
            part[t] = a.integrals[(long long)i * a.n + slot[i]];
            part_r[t] = a.ln_r[i];
        }
        __syncthreads();
        if (t == 0)
#pragma unroll 8
            for (int q = 0; q < cnt; ++q) {
                integ += part[q];
                lz += part_r[q];
            }
        __syncthreads();
    }
    if (t == 0) {
        a.log_weight[j] = lz - a.k * integ;
        a.traj_integral[j] = integ;
    }
    const int len = a.n_periods * a.tau;
#pragma unroll 8
    for (int q = t; q < len; q += 256) {
        const int i = q / a.tau;
        a.traj[(long long)j * len + q] = a.series[(long long)slot[i] * a.ld + a.col0 + q];
    }
}

// Block = trajectory: FP64 running sums, then the largest window mean
// (1/T) (S_t - S_{t-T}) over the windows inside [0, len).  The running sums
// are a block-wide scan over tiles of 4096 samples (eight neighbouring samples
// per thread, added in order; then the threads' totals), which replaces one
// thread adding the row sample by sample: 256 rows of 6144 samples, 302 -> 17 us.
constexpr int WMAX_THREADS = 512, WMAX_RUN = 8, WMAX_TILE = WMAX_THREADS * WMAX_RUN;

__global__ __launch_bounds__(WMAX_THREADS) void window_max_kernel(WindowMaxArgs a) {
    const int j = (int)blockIdx.x, t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
    const float* row = a.series + (long long)j * a.len;
    double* pre = a.prefix + (long long)j * ((long long)a.len + 1);
    __shared__ float tile[WMAX_TILE + WMAX_THREADS];  // sample i at i + i / 8: a thread's eight lie nine words apart
    __shared__ double wsum[WMAX_THREADS / 64];
    double carry = 0.0;
    if (t == 0) pre[0] = 0.0;
    for (long long base = 0; base < a.len; base += WMAX_TILE) {
#pragma unroll
        for (int q = 0; q < WMAX_RUN; ++q) {
            const int i = q * WMAX_THREADS + t;
            tile[i + i / WMAX_RUN] = base + i < a.len ? row[base + i] : 0.0f;
        }
        __syncthreads();
        double s[WMAX_RUN], tot = 0.0;
#pragma unroll
        for (int q = 0; q < WMAX_RUN; ++q) {
            tot += (double)tile[t * (WMAX_RUN + 1) + q];
            s[q] = tot;
        }
        double inc = tot;  // inclusive scan of the threads' totals: within the wave, then over the waves
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const double v = __shfl_up(inc, off, 64);
            if (lane >= off) inc += v;
        }
        if (lane == 63) wsum[wave] = inc;
        const double up = __shfl_up(inc, 1, 64);
        __syncthreads();
        double before = carry, all = carry;
#pragma unroll
        for (int w = 0; w < WMAX_THREADS / 64; ++w) {
            if (w < wave) before += wsum[w];
            all += wsum[w];
        }
        if (lane > 0) before += up;
        const long long i0 = base + t * WMAX_RUN;
#pragma unroll
        for (int q = 0; q < WMAX_RUN; ++q)
            if (i0 + q < a.len) pre[i0 + q + 1] = before + s[q];
        carry = all;
        __syncthreads();  // the next tile overwrites the samples and the wave totals
    }
    __syncthreads();
    __shared__ double sh[WMAX_THREADS];
    double best = -INFINITY;
#pragma unroll 4
    for (long long i = (long long)a.window + t; i <= a.len; i += WMAX_THREADS) {
        const double v = (pre[i] - pre[i - a.window]) / (double)a.window;
        best = fmax(best, v);
    }
    sh[t] = best;
    __syncthreads();
    for (int s = WMAX_THREADS / 2; s > 0; s >>= 1) {
        if (t < s) sh[t] = fmax(sh[t], sh[t + s]);
        __syncthreads();
    }
    if (t == 0) a.fmax[j] = sh[0];
}

// Block = level: (1/N) sum_j exp(log_weight_j) [fmax_j >= a], j in order.  The
// terms are formed side by side, a chunk of them in LDS at a time, and added
// in order by one thread (members below the level add zero, which changes
// nothing).  24 levels of 256 members: 53 us with one thread per level, 5.3 here.
constexpr int TAIL_CHUNK = 1024;

__global__ __launch_bounds__(256) void tail_probability_kernel(TailArgs a) {
    const int q = (int)blockIdx.x, t = (int)threadIdx.x;
    const double lev = a.levels[q];
    __shared__ double term[TAIL_CHUNK];
    double s = 0.0;
    for (int j0 = 0; j0 < a.n; j0 += TAIL_CHUNK) {
        const int cnt = min(TAIL_CHUNK, a.n - j0);
        for (int i = t; i < cnt; i += 256) term[i] = a.fmax[j0 + i] >= lev ? exp(a.log_weight[j0 + i]) : 0.0;
        __syncthreads();
        if (t == 0) {
            int i = 0;
            for (; i + 8 <= cnt; i += 8) {
                double v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = term[i + k];
#pragma unroll
                for (int k = 0; k < 8; ++k) s += v[k];
            }
            for (; i < cnt; ++i) s += term[i];
        }
        __syncthreads();
    }
    if (t == 0) a.prob[q] = s / (double)a.n;
}

// SCGF estimate (paper Appendix C.1): lambda(k) = (1/T_a) sum_i ln R_i, the
// sum in period order (one thread).
__global__ void scgf_kernel(const double* ln_r, int n_periods, double t_a, double* out) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    double s = 0.0;
    for (int i = 0; i < n_periods; ++i) s += ln_r[i];
    out[0] = s / t_a;
}

// Return time of a level from the probability p that a block of length T_a
// holds a window of length T above it (paper Appendix C.2):
// r = -(T_a - T) / ln(1 - p); +inf where p = 0 (0 where p = 1).
__global__ void return_times_kernel(const double* prob, int n, double t_a, double window, double* r) {
    const int q = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (q >= n) return;
    const double p = prob[q];
    r[q] = p == 0.0 ? INFINITY : -(t_a - window) / log1p(-p);
}

// Unbiased AMS estimate of P(max >= a) (paper Appendix B): the product over
// the iterations of (1 - K_j / N), in order, times the fraction of the final
// ensemble whose maximum reaches a.  Thread = level.
__global__ void ams_probability_kernel(AmsProbArgs a) {
    const int q = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (q >= a.n_levels) return;
    double f = 1.0;
    for (int j = 0; j < a.n_iter; ++j) f *= 1.0 - (double)a.k_history[j] / (double)a.n;
    const double lev = a.levels[q];
    int c = 0;
    for (int m = 0; m < a.n; ++m) c += a.final_max[m] >= lev ? 1 : 0;
    a.prob[q] = f * (double)c / (double)a.n;
}

// AMS score from a learned predictor, kept consistent with the target event
// {max_t F_T(t) >= a}: the score is a once the time-averaged drag has reached a;
// before that the prediction g is mapped strictly increasingly into (-inf, a),
// a - w ln(1 + exp((a - g)/w)), so that max_t score >= a exactly when the event
// happened while over-predictions keep their order.  Evaluated in FP64 in the
// form whose exponential cannot overflow, rounded to FP32 (a monotone rounding)
// and held at or below the float just under a.
__global__ void learned_score_kernel(const float* ghat, const float* ft, long long count, float a, float w,
                                     float* out) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const float g = ghat[i];
    float s;
    if (ft[i] >= a) {
        s = a;
    } else if (!isfinite(g)) {
        s = -INFINITY;
    } else {
        const double x = ((double)a - (double)g) / (double)w;
        const double v = x > 0.0 ? (double)g - (double)w * log1p(exp(-x)) : (double)a - (double)w * log1p(exp(x));
        s = fminf((float)v, nextafterf(a, -INFINITY));
    }
    out[i] = s;
}

hipError_t launch_learned_score(const float* ghat, const float* ft, long long count, float a, float w, float* out,
                                hipStream_t st) {
    hipLaunchKernelGGL(learned_score_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, ghat, ft,
                       count, a, w, out);
    return hipGetLastError();
}

hipError_t launch_rebuild(const RebuildArgs& a, hipStream_t st) {
    const long long anc = (long long)a.n_periods * a.n;
    const int in_lds = anc <= REBUILD_LDS ? 1 : 0;
    hipLaunchKernelGGL(gktl_rebuild_kernel, dim3(a.n), dim3(256), in_lds ? sizeof(int) * (size_t)anc : 0, st, a, in_lds);
    return hipGetLastError();
}
hipError_t launch_window_max(const WindowMaxArgs& a, int rows, hipStream_t st) {
    hipLaunchKernelGGL(window_max_kernel, dim3(rows), dim3(WMAX_THREADS), 0, st, a);
    return hipGetLastError();
}
hipError_t launch_scgf(const double* ln_r, int n_periods, double t_a, double* out, hipStream_t st) {
    hipLaunchKernelGGL(scgf_kernel, dim3(1), dim3(64), 0, st, ln_r, n_periods, t_a, out);
    return hipGetLastError();
}
hipError_t launch_return_times(const double* prob, int n, double t_a, double window, double* r, hipStream_t st) {
    hipLaunchKernelGGL(return_times_kernel, dim3((n + 255) / 256), dim3(256), 0, st, prob, n, t_a, window, r);
    return hipGetLastError();
}
hipError_t launch_ams_probability(const AmsProbArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(ams_probability_kernel, dim3((a.n_levels + 255) / 256), dim3(256), 0, st, a);
    return hipGetLastError();
}
hipError_t launch_tail(const TailArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(tail_probability_kernel, dim3(a.n_levels), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace lbm
