// GKTL cloning (paper Appendix C.1) and the branching perturbation with mass
// rescaling (paper Appendix D), on the device.
//
// Selection runs in one workgroup: the weights are FP64, the running sum that
// the multinomial draw inverts is formed sequentially in slot order (so the
// decisions are a fixed function of the inputs), and the uniforms come from
// the counter-based Philox stream.  Cloning is a gather over the ensemble:
// every member's new state is its ancestor's, perturbed for all but the
// first copy of each ancestor.
#include "rare_kernels.hpp"

namespace lbm {

typedef float f4g __attribute__((ext_vector_type(4)));

// The perturbation coefficients of member m and their sum (four words per
// Philox block).
__device__ __forceinline__ double draw_alphas(double* __restrict__ alpha, int m, int period, uint64_t key, int n_snap) {
    double psum = 0.0;
    for (int q0 = 0; q0 < n_snap; q0 += 4) {
        const U64x4 w = philox4x64_10((uint64_t)m, (uint64_t)period, (uint64_t)(q0 / 4), 0, key, PURPOSE_PRTB);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (q0 + j >= n_snap) break;
            const double al = uniform53(w.v[j]);
            alpha[(long long)m * MAX_SNAP + q0 + j] = al;
            psum += al;
        }
    }
    return psum;
}

// One workgroup of 1024 threads; N <= MAX_SELECT.  The weights, the running
// sum and every table the decisions need sit in LDS; one thread forms the
// running sum in slot order, eight slots at a time (from memory, 256 members
// took 50 of the kernel's 65 us; the kernel takes 17 now).  What the host needs of the result
// goes straight to its pinned tables.
__global__ __launch_bounds__(1024) void gktl_select_kernel(SelectArgs a) {
    __shared__ double prefix[MAX_SELECT];
    __shared__ int first_slot[MAX_SELECT];
    __shared__ int anc_of[MAX_SELECT];
    __shared__ int dead_state[MAX_SELECT];
    __shared__ double wave_max[16];
    __shared__ int wave_live[16], wave_dead[16], wave_extra[16];
    const int t = (int)threadIdx.x, nt = (int)blockDim.x, n = a.n, lane = t & 63, wave = t >> 6;
    double mx = -INFINITY;
    int live = 0;  // the last slot with a finite weight: the ancestor if u * total rounds up to total
    for (int m = t; m < n; m += nt) {
        const double s = a.k * a.accum[m];
        if (isfinite(s)) {
            mx = fmax(mx, s);
            live = m;
        }
        prefix[m] = s;
        first_slot[m] = 0x7fffffff;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {  // maxima are exact and order-free
        mx = fmax(mx, __shfl_xor(mx, off, 64));
        live = max(live, __shfl_xor(live, off, 64));
    }
    if (lane == 0) {
        wave_max[wave] = mx;
        wave_live[wave] = live;
    }
    __syncthreads();
    for (int w = 0; w < 16; ++w) {
        mx = fmax(mx, wave_max[w]);
        live = max(live, wave_live[w]);
    }
    if (!isfinite(mx)) {  // every weight non-finite: report and change nothing
        if (t == 0) {
            *a.status = 1;
            *a.status_host = 1;
            if (a.relabel) *a.n_extra = 0;
        }
        return;
    }
    // weights relative to the largest, then the running sum in slot order
    for (int m = t; m < n; m += nt) {
        const double s = prefix[m];
        prefix[m] = isfinite(s) ? exp(s - mx) : 0.0;
    }
    __syncthreads();
    if (t == 0) {
        double acc = 0.0;
        int m = 0;
        for (; m + 8 <= n; m += 8) {
            double v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = prefix[m + j];
#pragma unroll
            for (int j = 0; j < 8; ++j) prefix[m + j] = acc += v[j];
        }
        for (; m < n; ++m) prefix[m] = acc += prefix[m];
        *a.ln_r = mx + log(acc) - log((double)n);
        *a.status = 0;
        *a.status_host = 0;
    }
    __syncthreads();
    const double total = prefix[n - 1];
    for (int m = t; m < n; m += nt) {
        const U64x4 w = philox4x64_10((uint64_t)m, (uint64_t)a.period, 0, 0, a.key, PURPOSE_GKTS);
        const double target = uniform53(w.v[0]) * total;
        // first n with prefix[n] > target (prefix is non-decreasing)
        int lo = 0, hi = n;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (prefix[mid] > target) hi = mid; else lo = mid + 1;
        }
        const int anc = lo < n ? lo : live;
        a.ancestors[m] = anc;
        anc_of[m] = anc;
        a.need_mass[m] = 0;
        atomicMin(&first_slot[anc], m);  // lowest slot taking each ancestor: order-free
    }
    __syncthreads();
    for (int m = t; m < n; m += nt) {
        const int anc = anc_of[m];
        const int pert = (a.n_snap > 0 && a.eps != 0.0 && first_slot[anc] != m) ? 1 : 0;
        a.mode[m] = pert ? MODE_PERTURB : MODE_COPY;
        a.src[m] = anc;
        if (pert) {
            a.need_mass[anc] = 1;  // parents of perturbed copies need their mass
            a.alpha_sum[m] = draw_alphas(a.alpha, m, a.period, a.key, a.n_snap);
        }
    }
    if (!a.relabel) return;
    // Relabelling: the first copy of each ancestor keeps the ancestor's block
    // and buffer; the k-th further copy (in slot order) takes the block of the
    // k-th state (in slot order) that left no descendant.  There are as many
    // such states as further copies, and no copy reads them.  Ranks by a
    // block-wide exclusive prefix count over slot order (each thread counts
    // PER consecutive slots, then scans within and over the waves).
    constexpr int PER = MAX_SELECT / 1024;
    const int b0 = t * PER;
    int cd = 0, ce = 0;
    for (int j = 0; j < PER; ++j) {
        const int m = b0 + j;
        if (m < n) {
            cd += first_slot[m] == 0x7fffffff ? 1 : 0;
            ce += first_slot[anc_of[m]] != m ? 1 : 0;
        }
    }
    int rd = cd, re = ce;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int vd = __shfl_up(rd, off, 64), ve = __shfl_up(re, off, 64);
        if (lane >= off) {
            rd += vd;
            re += ve;
        }
    }
    if (lane == 63) {
        wave_dead[wave] = rd;
        wave_extra[wave] = re;
    }
    __syncthreads();
    rd -= cd;
    re -= ce;  // exclusive ranks of this thread's first slot
    int total_extra = 0;
    for (int w = 0; w < 16; ++w) {
        if (w < wave) {
            rd += wave_dead[w];
            re += wave_extra[w];
        }
        total_extra += wave_extra[w];
    }
    for (int j = 0; j < PER; ++j) {
        const int m = b0 + j;
        if (m < n && first_slot[m] == 0x7fffffff) dead_state[rd++] = m;
    }
    __syncthreads();
    for (int j = 0; j < PER; ++j) {
        const int m = b0 + j;
        if (m >= n) break;
        const int anc = anc_of[m], par = a.parity[anc];
        long long off = a.members[anc].off;
        if (first_slot[anc] != m) {
            off = a.members[dead_state[re]].off;
            a.extra[re++] = m;
        }
        a.new_parity[m] = par;
        a.new_off[m] = off;
        a.new_parity_host[m] = par;
        a.new_off_host[m] = off;
    }
    if (t == 0) *a.n_extra = total_extra;
}

// Host-chosen modes (in-place perturbation of selected members): fill the
// same tables the selection kernel fills.
__global__ void perturb_plan_kernel(PlanArgs a) {
    const int m = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (m >= a.n) return;
    const int pert = (a.mask.w[m >> 5] >> (m & 31)) & 1u;
    a.mode[m] = pert ? MODE_PERTURB : MODE_SKIP;
    a.src[m] = m;
    a.need_mass[m] = pert;
    if (pert) a.alpha_sum[m] = draw_alphas(a.alpha, m, a.period, a.key, a.n_snap);
}

// Sum of deviations over the fluid cells of one state, as fixed per-block
// partials (block b covers elements [b*chunk, (b+1)*chunk) of the 9*nx*ny
// floats); the partials are added in block order afterwards.
// blockIdx.y: member index (< n) or snapshot index (n + q).
__global__ __launch_bounds__(256) void mass_partial_kernel(MassArgs a) {
    const int j = (int)blockIdx.y;
    const bool snap = j >= a.n;
    if (a.status && *a.status) return;  // the selection changed nothing
    if (!snap && !a.need_mass[j]) return;
    const MemberDev m = a.members[snap ? 0 : j];
    const long long plane = (long long)m.nx * m.ny;
    const long long total = 9 * plane;
    const float* base = snap ? a.snapshots + (long long)(j - a.n) * total
                             : (a.parity[j] ? a.pop1 : a.pop0) + m.off;
    __shared__ double sh[256];
    const long long b0 = (long long)blockIdx.x * MASS_CHUNK;
    double acc = 0.0;
    if (b0 < total) {
        const long long e1 = min(b0 + MASS_CHUNK, total);
        if ((m.nx & 3) == 0) {
            // four cells of one row per thread and load (a row never splits a vector)
            for (long long e = b0 + 4 * threadIdx.x; e < e1; e += 1024) {
                const f4g v = *(const f4g*)(base + e);
                const long long cell = e % plane;
                const int y = (int)(cell / m.nx), x = (int)(cell - (long long)y * m.nx);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (!in_solid(m, x + k, y)) acc += (double)v[k];
            }
        } else {
            long long e = b0 + threadIdx.x;
            // the cell of the first element by division, the next ones by stepping 256 cells on
            const long long cell = e % plane;
            int y = (int)(cell / m.nx), x = (int)(cell - (long long)y * m.nx);
            for (; e < e1; e += 256) {
                if (!in_solid(m, x, y)) acc += (double)base[e];
                x += 256;
                while (x >= m.nx) {
                    x -= m.nx;
                    if (++y == m.ny) y = 0;
                }
            }
        }
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) a.partial[(long long)j * a.blocks_per_state + blockIdx.x] = sh[0];
}

// Per perturbed member: scale s restoring the parent's mass and the
// coefficient of the rest weights, c_w = s (1 + eps sum alpha) - 1.
//   M_parent = N_fluid + sum d_parent,  M_n = N_fluid + sum d^(n),
//   M_after = M_parent + eps sum_n alpha_n M_n,  s = M_parent / M_after.
// One wave per member: lane 0 adds the parent's partials, lane 1 + q those of
// snapshot q, each in block order (one thread doing all of it took 25 us for
// 10 snapshots of 36 partials, 6 so).
__global__ __launch_bounds__(64) void mass_scale_kernel(ScaleArgs a) {
    const int m = (int)blockIdx.x, lane = (int)threadIdx.x;
    if (a.status && *a.status) return;
    if (a.mode[m] != MODE_PERTURB) return;
    double mass = 0.0, al = 0.0;
    if (lane <= a.n_snap) {
        const double* p = a.partial + (long long)(lane == 0 ? a.src[m] : a.n + lane - 1) * a.blocks_per_state;
        double s = 0.0;
#pragma unroll 12
        for (int b = 0; b < a.blocks_per_state; ++b) s += p[b];
        mass = a.n_fluid + s;
        if (lane > 0) al = a.alpha[(long long)m * MAX_SNAP + lane - 1];
    }
    const double mp = __shfl(mass, 0, 64);
    double add = 0.0;
    for (int q = 0; q < a.n_snap; ++q) add += __shfl(al, q + 1, 64) * __shfl(mass, q + 1, 64);
    if (lane == 0) {
        const double s = mp / (mp + a.eps * add);
        a.scale[m] = s;
        a.coef_w[m] = s * (1.0 + a.eps * a.alpha_sum[m]) - 1.0;
    }
}

// New state of every member with mode != SKIP, written to the buffer that
// does not hold its current state:
//   copy:    d_new = d_src
//   perturb: d_new = s (d_src + eps sum_n alpha_n d^(n)) + c_w w_i
// (full populations: f_new = s (f_src + eps sum_n alpha_n f^(n)), f = w + d).
// blockIdx.y = member; each thread moves 4 consecutive floats with 16-byte
// accesses when the member block allows it (a plane of a multiple-of-4
// width never splits a vector between two directions).
// The perturbation's arithmetic, shared by every kernel that writes a
// perturbed copy (so that all of them give the same bits):
//   ad += alpha_q d^(q) (snapshots in order q = 0, 1, ...), then
//   d_new = s (d_src + eps ad) + c_w w_i, with explicit FMAs.
__device__ __forceinline__ double perturb_acc(double ad, double al, float sv) { return fma(al, (double)sv, ad); }
__device__ __forceinline__ float perturb_out(float v, double ad, double s, double eps, double cw) {
    return (float)fma(s, fma(eps, ad, (double)v), cw);
}

__global__ __launch_bounds__(256) void clone_gather_kernel(GatherArgs a) {
    const int m = (int)blockIdx.y;
    const int mode = a.mode[m];
    if (mode == MODE_SKIP) return;
    const MemberDev md = a.members[m];
    const long long plane = (long long)md.nx * md.ny;
    const long long total = 9 * plane;
    const long long e0 = 4 * ((long long)blockIdx.x * 256 + threadIdx.x);
    if (e0 >= total) return;
    const int src = a.src[m];
    const float* sp = (a.parity[src] ? a.pop1 : a.pop0) + a.members[src].off;
    float* dp = (a.parity[m] ? a.pop0 : a.pop1) + md.off;
    const bool vec = (plane & 3) == 0;
    if (vec) {
        const f4g v = *(const f4g*)(sp + e0);
        if (mode == MODE_COPY) {
            __builtin_nontemporal_store(v, (f4g*)(dp + e0));
            return;
        }
        const int i = (int)(e0 / plane);
        f4g acc = {0.0f, 0.0f, 0.0f, 0.0f};
        double ad[4] = {0.0, 0.0, 0.0, 0.0};
        for (int q = 0; q < a.n_snap; ++q) {
            const double al = a.alpha[(long long)m * MAX_SNAP + q];
            const f4g sv = *(const f4g*)(a.snapshots + (long long)q * total + e0);
#pragma unroll
            for (int k = 0; k < 4; ++k) ad[k] = perturb_acc(ad[k], al, sv[k]);
        }
        const double s = a.scale[m], cw = a.coef_w[m] * WD[i], eps = a.eps;
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[k] = perturb_out(v[k], ad[k], s, eps, cw);
        *(f4g*)(dp + e0) = acc;
        return;
    }
    const int cnt = (int)min((long long)4, total - e0);
    if (mode == MODE_COPY) {
        for (int k = 0; k < cnt; ++k) dp[e0 + k] = sp[e0 + k];
        return;
    }
    const double s = a.scale[m], eps = a.eps;
    for (int k = 0; k < cnt; ++k) {
        const long long e = e0 + k;
        const int i = (int)(e / plane);
        double ad = 0.0;
        for (int q = 0; q < a.n_snap; ++q)
            ad = perturb_acc(ad, a.alpha[(long long)m * MAX_SNAP + q], a.snapshots[(long long)q * total + e]);
        dp[e] = perturb_out(sp[e], ad, s, eps, a.coef_w[m] * WD[i]);
    }
}

// Bookkeeping after a gather: members that received a new state flip parity;
// the GKTL period restarts (accum = 0) and the non-finite flag follows the state.
__global__ void clone_finish_kernel(FinishArgs a) {
    const int m = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (m >= a.n) return;
    const int mode = a.mode[m];
    if (mode == MODE_SKIP) return;
    if (a.reset_accum) {
        a.accum[m] = 0.0;
        a.flags_new[m] = a.flags[a.src[m]];
    }
}
__global__ void clone_commit_kernel(FinishArgs a) {
    const int m = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (m >= a.n || a.mode[m] == MODE_SKIP) return;
    a.parity[m] ^= 1;
    if (a.reset_accum) a.flags[m] = a.flags_new[m];
}

// Relabelling clone: the further copies extra[PLACE_GROUP * blockIdx.y + g]
// get their ancestor's state (copy) or its perturbation (the arithmetic of
// clone_gather_kernel), written into their new blocks in the ancestor's
// buffer.  Sources are blocks of ancestors, destinations blocks of states
// without descendant: never the same block.
//
// Bound by memory: a workgroup takes one stretch of 1024 values, holds it of
// every snapshot in registers (FP64, NS >= n_snap of them, zeros beyond), and
// runs through up to 32 copies, the next copy's source in flight while one is
// formed; the copies' pointers and coefficients are gathered into LDS first.
// 92 copies of 1024 x 256 from 10 snapshots: 756 us with groups of 8 copies
// (the snapshots then cross the fabric 12 times, 1.1 of 2.8 GB, and every
// stretch waited for the chain of small reads that gives a copy's pointers),
// 468 us here (1.7 GB in and out: 3.7 TB/s).
constexpr int PLACE_GROUP = 32;

template <int NS>
__global__ __launch_bounds__(256) void clone_place_kernel(PlaceArgs a) {
    const int g0 = (int)blockIdx.y * PLACE_GROUP;
    const int ng = min(PLACE_GROUP, *a.n_extra - g0);  // the count is 0 where the selection changed nothing
    if (ng <= 0) return;
    const int t = (int)threadIdx.x;
    __shared__ const float* from[PLACE_GROUP];
    __shared__ float* to[PLACE_GROUP];
    __shared__ double al[PLACE_GROUP][NS > 0 ? NS : 1], sc[PLACE_GROUP], cw[PLACE_GROUP];
    if (t < ng) {
        const int m = a.extra[g0 + t], src = a.src[m];
        float* const buf = a.parity[src] ? a.pop1 : a.pop0;
        from[t] = buf + a.members[src].off;
        to[t] = buf + a.new_off[m];
        if (NS > 0) {
            sc[t] = a.scale[m];
            cw[t] = a.coef_w[m];
        }
    }
    if constexpr (NS > 0)
        for (int i = t; i < ng * NS; i += 256) {
            const int g = i / NS, q = i - g * NS;
            al[g][q] = q < a.n_snap ? a.alpha[(long long)a.extra[g0 + g] * MAX_SNAP + q] : 0.0;
        }
    const MemberDev& m0 = a.members[0];  // every member has one lattice shape
    const long long plane = (long long)m0.nx * m0.ny;
    const long long total = 9 * plane;
    const long long e0 = 4 * ((long long)blockIdx.x * 256 + t);
    __syncthreads();
    if (e0 >= total) return;
    const double eps = a.eps;
    if ((plane & 3) == 0) {
        double sn[NS > 0 ? NS : 1][4];
        if constexpr (NS > 0)
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                const f4g v = q < a.n_snap ? *(const f4g*)(a.snapshots + (long long)q * total + e0) : f4g{0, 0, 0, 0};
#pragma unroll
                for (int k = 0; k < 4; ++k) sn[q][k] = (double)v[k];
            }
        const double wi = WD[(int)(e0 / plane)];
        f4g next = *(const f4g*)(from[0] + e0);
#pragma unroll 1
        for (int g = 0; g < ng; ++g) {
            const f4g v = next;
            if (g + 1 < ng) next = *(const f4g*)(from[g + 1] + e0);
            f4g out = v;
            if constexpr (NS > 0) {
                double ad[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int q = 0; q < NS; ++q)
#pragma unroll
                    for (int k = 0; k < 4; ++k) ad[k] = fma(al[g][q], sn[q][k], ad[k]);
                const double s = sc[g], c = cw[g] * wi;
#pragma unroll
                for (int k = 0; k < 4; ++k) out[k] = perturb_out(v[k], ad[k], s, eps, c);
            }
            __builtin_nontemporal_store(out, (f4g*)(to[g] + e0));
        }
        return;
    }
    const int cnt = (int)min((long long)4, total - e0);
    for (int g = 0; g < ng; ++g)
        for (int k = 0; k < cnt; ++k) {
            const long long e = e0 + k;
            if constexpr (NS == 0) {
                to[g][e] = from[g][e];
            } else {
                double ad = 0.0;
                for (int q = 0; q < a.n_snap; ++q) ad = perturb_acc(ad, al[g][q], a.snapshots[(long long)q * total + e]);
                to[g][e] = perturb_out(from[g][e], ad, sc[g], eps, cw[g] * WD[(int)(e / plane)]);
            }
        }
}

// After the relabelling clone: every slot's block, buffer and flag (its
// ancestor's, read before any is written: one workgroup).
__global__ __launch_bounds__(1024) void clone_relabel_commit_kernel(CommitArgs a) {
    if (*a.status) return;
    constexpr int PER = MAX_SELECT / 1024;
    const int t = (int)threadIdx.x;
    int flag[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int m = t + 1024 * j;
        flag[j] = m < a.n ? a.flags[a.src[m]] : 0;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int m = t + 1024 * j;
        if (m >= a.n) break;
        a.members[m].off = a.new_off[m];
        a.parity[m] = a.new_parity[m];
        a.accum[m] = 0.0;
        a.flags[m] = flag[j];
    }
}

hipError_t launch_place(const PlaceArgs& a, int n, long long floats_per_member, hipStream_t st) {
    if (n < 2) return hipSuccess;  // at most n - 1 further copies
    const dim3 grid((unsigned)((floats_per_member + 1023) / 1024), (n - 1 + PLACE_GROUP - 1) / PLACE_GROUP), block(256);
    if (a.n_snap == 0) hipLaunchKernelGGL(clone_place_kernel<0>, grid, block, 0, st, a);
    else if (a.n_snap <= 4) hipLaunchKernelGGL(clone_place_kernel<4>, grid, block, 0, st, a);
    else if (a.n_snap <= 10) hipLaunchKernelGGL(clone_place_kernel<10>, grid, block, 0, st, a);
    else hipLaunchKernelGGL(clone_place_kernel<MAX_SNAP>, grid, block, 0, st, a);
    return hipGetLastError();
}

hipError_t launch_relabel_commit(const CommitArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(clone_relabel_commit_kernel, dim3(1), dim3(1024), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_select(const SelectArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(gktl_select_kernel, dim3(1), dim3(1024), 0, st, a);
    return hipGetLastError();
}
hipError_t launch_plan(const PlanArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(perturb_plan_kernel, dim3((a.n + 255) / 256), dim3(256), 0, st, a);
    return hipGetLastError();
}
hipError_t launch_mass(const MassArgs& a, int n_states, hipStream_t st) {
    hipLaunchKernelGGL(mass_partial_kernel, dim3(a.blocks_per_state, n_states), dim3(256), 0, st, a);
    return hipGetLastError();
}
hipError_t launch_scale(const ScaleArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(mass_scale_kernel, dim3(a.n), dim3(64), 0, st, a);
    return hipGetLastError();
}
hipError_t launch_gather(const GatherArgs& a, long long floats_per_member, hipStream_t st) {
    const unsigned gx = (unsigned)((floats_per_member / 4 + 255) / 256 + 1);
    hipLaunchKernelGGL(clone_gather_kernel, dim3(gx, a.n), dim3(256), 0, st, a);
    return hipGetLastError();
}
hipError_t launch_finish(const FinishArgs& a, hipStream_t st) {
    hipLaunchKernelGGL(clone_finish_kernel, dim3((a.n + 255) / 256), dim3(256), 0, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(clone_commit_kernel, dim3((a.n + 255) / 256), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace lbm
