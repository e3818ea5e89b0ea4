// C-ABI layer: context lifetime, argument validation, chunked stepping and
// the bookkeeping mirrors the host keeps of per-member device state.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <fstream>
#include <mutex>
#include <sstream>
#include <string>
#include <vector>

#include "../../include/lbm.h"
#include "api_internal.hpp"

using namespace lbm;

static thread_local std::string g_last_error;

int lbm_fail(int code, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}

int lbm_hip_fail(hipError_t e, const char* what) {
    return lbm_fail(LBM_EHIP, "%s: %s", what, hipGetErrorString(e));
}

extern "C" const char* lbm_last_error(void) { return g_last_error.c_str(); }

// ---------------------------------------------------------------------------
// small device utilities

namespace lbm {

__global__ void fill_int_kernel(int* p, int n, int v) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) p[i] = v;
}
__global__ void fill_double_kernel(double* p, int n, double v) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) p[i] = v;
}
__global__ void set_int_kernel(int* p, int v) { *p = v; }
__global__ void iota_kernel(int* p, int n) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i < n) p[i] = i;
}
__global__ void set_bits_kernel(int* p, int* list, int n, MaskBits bits) {
    const int i = (int)(blockIdx.x * blockDim.x + threadIdx.x);
    if (i >= n) return;
    const unsigned on = (bits.w[i >> 5] >> (i & 31)) & 1u;
    p[i] = (int)on;
    if (list && on) {  // position = set bits below i
        int pos = __popc(bits.w[i >> 5] & ((1u << (i & 31)) - 1u));
        for (int w = 0; w < (i >> 5); ++w) pos += __popc(bits.w[w]);
        list[pos] = i;
    }
}

hipError_t fill_int(int* p, int n, int v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_int_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}
hipError_t fill_double(double* p, int n, double v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_double_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}
hipError_t fill_iota(int* p, int n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(iota_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, n);
    return hipGetLastError();
}
hipError_t set_int(int* p, int v, hipStream_t st) {
    hipLaunchKernelGGL(set_int_kernel, dim3(1), dim3(1), 0, st, p, v);
    return hipGetLastError();
}
hipError_t set_bits(int* p, int* list, int n, const MaskBits& bits, hipStream_t st) {
    hipLaunchKernelGGL(set_bits_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, list, n, bits);
    return hipGetLastError();
}

}  // namespace lbm

// ---------------------------------------------------------------------------

static long long member_floats(const lbm_member_desc& d) { return 9LL * d.nx * d.ny; }

extern "C" size_t lbm_state_floats(const lbm_member_desc* members, int32_t n) {
    if (!members || n <= 0) return 0;
    size_t tot = 0;
    for (int i = 0; i < n; ++i) tot += (size_t)member_floats(members[i]);
    return tot;
}

static int validate_member(const lbm_member_desc& d, int i) {
    if (d.nx < 4 || d.ny < 4) return lbm_fail(LBM_EINVAL, "member %d: nx, ny must be >= 4", i);
    // the kernels index a member's 9 planes with 32-bit element offsets
    if (9LL * d.nx * d.ny > 0xFFFFFFFFLL)
        return lbm_fail(LBM_EINVAL, "member %d: lattice too large (at most %lld cells)", i, 0xFFFFFFFFLL / 9);
    if (d.reserved != 0) return lbm_fail(LBM_EINVAL, "member %d: reserved field must be 0", i);
    if (!(d.tau > 0.5) || !std::isfinite(d.tau)) return lbm_fail(LBM_EINVAL, "member %d: tau must be > 1/2", i);
    if (!std::isfinite(d.force_x)) return lbm_fail(LBM_EINVAL, "member %d: force must be finite", i);
    if (d.sq_side < 0) return lbm_fail(LBM_EINVAL, "member %d: negative square side", i);
    if (d.sq_side > 0) {
        if (d.sq_x0 < 1 || d.sq_x0 + d.sq_side > d.nx - 1 || d.sq_y0 < 1 || d.sq_y0 + d.sq_side > d.ny - 1)
            return lbm_fail(LBM_EINVAL, "member %d: square must keep one fluid cell on every side", i);
    }
    return LBM_OK;
}

// Rows per workgroup of a two-step shape's strips (0: whole strips).  The
// adaptive shape keeps whole strips when there are at least as many as
// workgroup slots (two per compute unit); otherwise it cuts them into the
// tallest row ranges (128, 64 or 32 rows) that give two workgroups per slot,
// or 32 rows when none does.  A few tall strips leave most slots idle, and a
// cut costs only the rows that both neighbours collide at phase A.  Measured
// on 16 to 96 members of 1024 x 256 and 64 to 128 of 512 x 128, this comes
// within 5 % of the best row range, at 1.2 to 1.9 x the speed of whole strips.
static int strip_rows(const lbm_ctx* c, const TileShape& ts) {
    if (ts.seg_rows >= 0) return ts.seg_rows;
    const long long slots = 2LL * c->cu_count;
    auto groups = [&](int h) {
        long long g = 0;
        for (int m = 0; m < c->n; ++m) {
            const auto& d = c->desc[m];
            const int rows = h > 0 ? std::min(h, d.ny) : d.ny;
            g += (long long)(d.nx / 256) * ((d.ny + rows - 1) / rows);
        }
        return g;
    };
    if (groups(0) >= slots) return 0;
    for (int h : {128, 64})
        if (groups(h) >= 2 * slots) return h;
    return 32;
}

// Segment table of one tiling: runs of consecutive members with the same
// lattice shape share it.  strips: the two-step kernel's tiling (one
// workgroup per 256-column strip, or per row range of one: Segment::rows).
static int build_table(lbm_ctx* c, const TileShape& ts, bool strips, Segment* seg, int& nseg, int& total) {
    const int rows = ts.tyt * ts.r;
    const int shape_split = strips ? strip_rows(c, ts) : 0;
    nseg = 0;
    int blocks = 0;
    for (int m = 0; m < c->n; ++m) {
        const auto& d = c->desc[m];
        const bool same = nseg > 0 && c->desc[seg[nseg - 1].member_begin].nx == d.nx &&
                          c->desc[seg[nseg - 1].member_begin].ny == d.ny;
        // strips: rows per workgroup, the run's own choice if it has one
        const int run = same ? nseg - 1 : nseg;
        const int split = strips && run < (int)c->run_rows.size() && c->run_rows[run] >= 0 ? c->run_rows[run]
                                                                                           : shape_split;
        const int hseg = split > 0 ? std::min(split, d.ny) : d.ny;
        const int tx = (d.nx + 255) / 256, ty = strips ? (d.ny + hseg - 1) / hseg : (d.ny + rows - 1) / rows;
        if (!same) {
            if (nseg == MAX_SEGMENTS)
                return lbm_fail(LBM_EUNSUPPORTED, "more than %d runs of distinct lattice shapes; group members by shape",
                                MAX_SEGMENTS);
            Segment s;
            s.block_begin = blocks;
            s.member_begin = m;
            s.tiles_per_member = tx * ty;
            s.tiles_x = tx;
            // four cells per lane needs 16-byte rows, and 32-bit byte offsets over the member's block
            s.vec = (d.nx % 4 == 0 && 36LL * d.nx * d.ny < (1LL << 31)) ? 1 : 0;
            s.rows = strips ? hseg : 0;
            seg[nseg++] = s;
        }
        if ((long long)blocks + (long long)tx * ty > (1LL << 31) - 1)
            return lbm_fail(LBM_EUNSUPPORTED, "ensemble needs more than 2^31 workgroups");
        blocks += tx * ty;
    }
    total = blocks;
    return LBM_OK;
}

// Whether the next batch makes two steps per launch.  The two-step kernel
// gives one workgroup per strip (or row range of a strip): with few active
// members (an AMS branch re-simulates a handful) that leaves most compute
// units idle, and one-step launches (many small tiles, the same results bit
// for bit) are faster.  The adaptive shape uses it once the active members
// give 1.5 workgroups per compute unit (measured with split strips: 0.8 x the
// one-step speed at 1 workgroup per CU, 1.1 x at 1.5, 1.2 to 1.5 x at 2).
static bool two_step_now(const lbm_ctx* c) {
    if (!c->two_step) return false;
    if (!TILE_SHAPES[c->tile_id].adaptive) return true;
    long long groups = 0;  // workgroups of the active members
    for (int s = 0; s < c->nseg2; ++s) {
        const int end = s + 1 < c->nseg2 ? c->seg2[s + 1].member_begin : c->n;
        for (int m = c->seg2[s].member_begin; m < end; ++m)
            if (c->h_active[m]) groups += c->seg2[s].tiles_per_member;
    }
    return 2 * groups >= 3LL * c->cu_count;
}

// The resident kernel's cuts, with the us of a step of a full launch: BGK and
// unit-rate central moments with the waves alone on their SIMD and two on each,
// and in open channels, whose outlet's waves first wait for the last columns
// beside them (BGK there forms its coefficients in each cell); and how many times
// as long central moments with three rates take, whose larger cuts spill.
// Measured, MI355X, us per
// step: 1 x 256 x 64 with two columns per lane and 1, 2, 3, 4, 6 rows 2.2, 3.0,
// 3.9, 4.5, 6.0 (lone waves); 64 x 512 x 128, per launch, in workgroups of eight
// waves, with 2, 3, 4, 6 rows 4.0, 5.2, 6.6, 8.9, and with three columns and 2,
// 3, 4 rows 5.0, 6.3, 7.8.  Two columns fill eight waves in lattices of 113-128,
// 225-256, 449-512 or 897-1024 columns, three in 169-192, 337-384 or 673-768:
// 24 x 330 x 110 8.4 with two columns, 6.8 with three, open 64 x 513 x 129 71 and
// 46.  (One column per lane: 2.4 for 1 x 256 x 64; five: 21 for 24 x 330 x 110,
// its registers spill.)  Open: 8 x 512 x 128 with 2, 3, 4, 6 rows 5.4, 6.1, 7.2,
// 10.5, 10 x 640 x 100 with three columns and 2, 3 rows 6.6, 7.6.  Three rates:
// 1500 x 292 x 50 with three columns and four rows 14.0 per launch, 14 x 768 x 146
// with three 9.0, 88 x 512 x 165 with two columns and six rows 12.5, open 415 x
// 768 x 39 with three columns and rows 12.9.
struct ResidentCut {
    int cells, rows;                     // columns per lane, rows per wave
    double lone, both;                   // us per step
    double opened, opened_bgk;           // (0: not made)
    double rates, opened_rates;          // three rates: times as long
};
constexpr ResidentCut RESIDENT_CUTS[] = {
    {2, 1, 2.2, 3.0, 0.0, 0.0, 1.2, 0.0},   {2, 2, 3.1, 3.8, 4.8, 4.8, 1.3, 1.2},  {2, 3, 4.1, 5.0, 5.8, 5.8, 1.25, 1.25},
    {2, 4, 4.9, 6.2, 7.1, 7.1, 1.3, 1.3},   {2, 6, 6.5, 8.2, 11.0, 13.3, 1.5, 1.6}, {3, 2, 4.5, 5.0, 6.1, 6.1, 1.3, 1.25},
    {3, 3, 5.8, 6.5, 7.7, 8.6, 1.35, 1.65}, {3, 4, 7.0, 7.8, 0.0, 0.0, 2.0, 0.0},
};
// One step: the rows' time, or that of the words between workgroups (`sides`
// rows of a wave handed to another workgroup) if they take longer (4 x 512 x
// 128, one row of two columns per lane: 4096 sides 6.3 us, 2048 sides 3.6).
static double resident_cost(const ResidentCut& cut, bool two, bool open, int model, double sides) {
    const double rows = open ? (model == 0 ? cut.opened_bgk : cut.opened) : two ? cut.both : cut.lone;
    const double rates = model != 1 ? 1.0 : open ? cut.opened_rates : cut.rates;
    return rates * (std::max(rows, 0.75e-3 * cut.cells * sides) + 0.75e-4 * cut.cells * sides);
}

// The resident launches of a batch, if the adaptive shape may have any: a
// whole chunk of steps per launch with the populations in registers (channels
// of up to 1024 columns, all workgroups of a launch side by side on
// the device: two waves per SIMD at most), as many launches as the members
// need.  The cut, and the waves per workgroup (four, two of them on a compute
// unit, or eight), with the least estimated time: more rows per wave are fewer
// launches, fewer rows a shorter step; eight waves hand half as many rows to
// other workgroups as two times four (16 x 512 x 128: 7.0 us per step instead
// of 7.7), four leave small ensembles a SIMD per wave (1 x 256 x 64: 2.3
// instead of 2.5).
static bool plan_resident(const lbm_ctx* c, ResidentPlan& p, bool every_member) {
    if (!TILE_SHAPES[c->tile_id].adaptive) return false;
    for (int r : c->run_rows)
        if (r >= 0) return false;  // row ranges given by the caller: for the kernels that have such
    const bool listed = !every_member && c->n_active < c->n && c->uniform_shape;
    double cells = 0.0;
    int widest = 0;
    for (int s = 0; s < c->nseg; ++s) {
        const lbm_member_desc& d = c->desc[c->seg[s].member_begin];
        if (36LL * d.nx * d.ny >= (1LL << 31)) return false;
        widest = std::max(widest, d.nx);
        const int end = s + 1 < c->nseg ? c->seg[s + 1].member_begin : c->n;
        cells += (double)(listed ? c->n_active : end - c->seg[s].member_begin) * d.nx * d.ny;
    }
    if (widest > RESIDENT_WIDEST || cells > RESIDENT_PASSES * 1.6e6) return false;
    // adds the launches of the runs s0 .. s1 - 1 with a cut and workgroups of `waves` waves (or one row of the lattice,
    // if wider) to a plan
    auto cut = [&](const ResidentCut& rc, int waves, int s0, int s1, ResidentPlan& q) {
        int block_waves = 1;
        for (int s = s0; s < s1; ++s) {
            const int w = (c->desc[c->seg[s].member_begin].nx + 64 * rc.cells - 1) / (64 * rc.cells);
            if (w > SWEEP_WAVES) return false;
            block_waves = std::max(block_waves, w * std::max(1, waves / w));
        }
        const long long slots = (long long)c->cu_count * (SWEEP_WAVES / block_waves);
        const int first = q.passes;
        long long blocks = slots, sides = 0, words = 0;  // (no pass yet)
        auto close = [&] {
            if (q.passes == first) return;
            q.pass[q.passes - 1].args.total_blocks = (int)blocks;
            q.us += resident_cost(rc, blocks * block_waves > 4LL * c->cu_count, c->open, c->model, (double)sides);
        };
        for (int s = s0; s < s1; ++s) {
            const lbm_member_desc& d = c->desc[c->seg[s].member_begin];
            ResidentSegment g;
            const int lanes = (d.nx + rc.cells - 1) / rc.cells;
            g.waves = (lanes + 63) / 64;
            g.lanes = (lanes + g.waves - 1) / g.waves;
            g.groups = std::max(1, waves / g.waves);
            g.ranges = (d.ny + g.groups * rc.rows - 1) / (g.groups * rc.rows);
            if (g.ranges > slots) return false;
            int m = listed ? 0 : c->seg[s].member_begin;
            const int end = listed ? c->n_active : s + 1 < c->nseg ? c->seg[s + 1].member_begin : c->n;
            while (m < end) {
                if (slots - blocks < g.ranges) {  // another pass
                    close();
                    if (q.passes == RESIDENT_PASSES) return false;
                    ResidentPass& p = q.pass[q.passes++];
                    p.cells = rc.cells;
                    p.rows = rc.rows;
                    p.args.nseg = 0;
                    p.args.block_waves = block_waves;
                    p.args.full = 1;
                    blocks = sides = words = 0;
                }
                ResidentArgs& a = q.pass[q.passes - 1].args;
                const int here = (int)std::min<long long>(end - m, (slots - blocks) / g.ranges);
                g.block_begin = (int)blocks;
                g.member_begin = m;
                g.halo_begin = words;
                a.seg[a.nseg++] = g;
                if (d.nx % (64 * rc.cells)) a.full = 0;
                blocks += (long long)here * g.ranges;
                sides += 2LL * here * (g.ranges - 1) * g.waves;
                words += (long long)here * g.ranges * (12LL * rc.cells * lanes + (c->open ? 4 * RESIDENT_OUTLET_WORDS : 0));
                q.halo_words = std::max(q.halo_words, (size_t)words);
                m += here;
            }
        }
        close();
        return q.passes > first;
    };
    // the best cut of the runs s0 .. s1 - 1 (null: none fits); us: its estimate
    ResidentPlan q;
    auto best_cut = [&](int s0, int s1, int& best_waves, double& us) {
        const ResidentCut* best = nullptr;
        for (int waves : {4, 8})
            for (const ResidentCut& rc : RESIDENT_CUTS) {
                if (c->open ? waves < 8 || rc.opened == 0.0 : waves < 8 && rc.cells > 2) continue;  // (their LDS fits once on a compute unit)
                q.passes = 0;
                q.us = 0.0;
                if (cut(rc, waves, s0, s1, q) && (!best || q.us < us)) {
                    us = q.us;
                    best = &rc;
                    best_waves = waves;
                }
            }
        return best;
    };
    // all runs with one cut, or each run with its own (24 x 330 x 110 with 40 x 201 x 75: 14.0 and 11.8 us per step)
    int waves[MAX_SEGMENTS + 1];
    const ResidentCut* own[MAX_SEGMENTS + 1];
    double all = 1e300, each = 0.0, us = 0.0;
    own[c->nseg] = best_cut(0, c->nseg, waves[c->nseg], us);
    if (own[c->nseg]) all = us;
    for (int s = 0; s < c->nseg && c->nseg > 1 && each < all; ++s) {
        own[s] = best_cut(s, s + 1, waves[s], us);
        each += own[s] ? us : 1e300;
    }
    p.passes = 0;
    p.us = 0.0;
    p.halo_words = 0;
    p.listed = listed;
    p.slots = listed ? c->n_active : c->n;
    if (c->nseg > 1 && each < all) {
        for (int s = 0; s < c->nseg; ++s)
            if (!cut(*own[s], waves[s], s, s + 1, p)) return false;
    } else if (!own[c->nseg] || !cut(*own[c->nseg], waves[c->nseg], 0, c->nseg, p)) {
        return false;
    }
    if (p.halo_words > c->halo_words) return false;  // (no memory for them: allocate_resident)
    for (int k = 0; k < p.passes; ++k) {
        ResidentArgs& a = p.pass[k].args;
        a.members = c->d_members;
        a.parity = c->d_parity;
        a.active = c->d_active;
        a.active_list = listed ? c->d_active_list : nullptr;
        a.pop0 = c->pop[0];
        a.pop1 = c->pop[1];
        a.partial = c->d_partial;
        a.halo = c->d_halo;
        a.given_up = c->d_given_up;
        a.n_members = c->n;
        a.pass = k;
    }
    return true;
}

// The most words between workgroups that a plan for any of the context's members can need (at most some
// 26 MB, 51 for several widths): for each cut the workgroups that the device or all members have, whichever are
// fewer, of the widest member.  0: no plan.
static size_t resident_words(const lbm_ctx* c) {
    size_t most = 0;
    for (int waves : {4, 8})
        for (const ResidentCut& rc : RESIDENT_CUTS) {
            long long units = 0, words = 0;
            int block_waves = SWEEP_WAVES;  // the fewest
            for (const lbm_member_desc& d : c->desc) {
                if (d.nx > RESIDENT_WIDEST) return 0;
                const int lanes = (d.nx + rc.cells - 1) / rc.cells, w = (lanes + 63) / 64, groups = std::max(1, waves / w);
                if (w > SWEEP_WAVES) continue;
                block_waves = std::min(block_waves, w * groups);
                units += (d.ny + groups * rc.rows - 1) / (groups * rc.rows);
                words = std::max(words, 12LL * rc.cells * lanes + 4 * RESIDENT_OUTLET_WORDS);
            }
            const long long places = (long long)c->cu_count * (SWEEP_WAVES / block_waves);
            most = std::max(most, (size_t)(std::min(units, places) * words));
        }
    return most;
}

// The words between workgroups, cleared (no launch's), for every plan to come: a batch allocates nothing.  Later
// launches find older launches' words, whoever wrote them: each chunk has its own number, so no old word
// passes for a new one.  Without memory for them there is no plan (another kernel steps the batches then).
static void allocate_resident(lbm_ctx* c) {
    const size_t words = resident_words(c);
    if (words == 0) return;
    if (hipHostMalloc(&c->gave_up, sizeof(int)) == hipSuccess &&
        hipEventCreateWithFlags(&c->resident_done, hipEventDisableTiming) == hipSuccess &&
        hipMalloc(&c->d_halo, sizeof(unsigned long long) * words) == hipSuccess &&
        fill_int((int*)c->d_halo, (int)(2 * words), 0, c->stream) == hipSuccess) {
        *c->gave_up = 0;
        c->halo_words = words;
    }
    (void)hipGetLastError();
}

static hipError_t clear_redo(const lbm_ctx* c, hipStream_t st) {
    return fill_int(c->d_redo, std::max(c->n, REDO_TASKS) + 2, 0, st);
}

static hipError_t launch_resident_passes(lbm_ctx* c, ResidentPlan& p, int steps, int flip, hipStream_t st) {
    if (++c->resident_launch >= RESIDENT_LAUNCHES) {  // the words' tags would repeat: from the start again
        hipError_t e;
        if ((e = fill_int(c->d_given_up, c->n + 1, 0, st)) != hipSuccess || (e = clear_redo(c, st)) != hipSuccess ||
            (e = fill_int((int*)c->d_halo, (int)(2 * c->halo_words), 0, st)) != hipSuccess)
            return e;
        c->resident_launch = c->resident_first = 1;
    }
    for (int k = 0; k < p.passes; ++k) {
        ResidentArgs& a = p.pass[k].args;
        a.launch = c->resident_launch;
        a.first = c->resident_first;
        a.wait_ticks = c->wait_ticks;
        a.n_steps = steps;
        a.flip = flip;
        const hipError_t e = launch_resident(p.pass[k].cells, p.pass[k].rows, c->open, a, c->model, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Another thread may be capturing a stream of its own: allocations and event
// queries here are no part of that.
struct OutsideCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    OutsideCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~OutsideCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// The contexts of this process that have made resident launches.  Workgroups
// of a resident launch wait for one another, so two launches that do not fit
// on the device together must not run together: each could hold the places
// that the other's missing workgroups need, until a wait reaches its limit.
struct ResidentUsers {
    std::mutex lock;
    std::vector<lbm_ctx*> users;
};
static ResidentUsers& resident_users() {
    static ResidentUsers* const u = new ResidentUsers;  // (contexts may outlive static destructors)
    return *u;
}

// Before resident launches of `c` (under the lock, until leave_resident): its stream waits for the other
// contexts' launches that are still running, if all of them together are more than the device holds.
static hipError_t admit_resident(lbm_ctx* c, ResidentUsers& u, const ResidentPlan& p) {
    const OutsideCapture outside;
    hipError_t e;
    if (std::find(u.users.begin(), u.users.end(), c) == u.users.end()) u.users.push_back(c);
    ResidentUse now;
    for (int k = 0; k < p.passes; ++k) {
        const ResidentArgs& a = p.pass[k].args;
        const ResidentUse one{a.total_blocks, SWEEP_WAVES / a.block_waves};
        now = k == 0 ? one : either_of(now, one);
    }
    auto running = [](const lbm_ctx* o) { return hipEventQuery(o->resident_done) == hipErrorNotReady; };
    c->resident_use = running(c) ? either_of(c->resident_use, now) : now;
    std::vector<ResidentUse> uses{c->resident_use};
    for (const lbm_ctx* o : u.users)
        if (o != c && o->device == c->device && running(o)) uses.push_back(o->resident_use);
    (void)hipGetLastError();  // (not ready)
    if (side_by_side(uses, c->cu_count)) return hipSuccess;
    for (const lbm_ctx* o : u.users)
        if (o != c && o->device == c->device && (e = hipStreamWaitEvent(c->stream, o->resident_done, 0)) != hipSuccess) return e;
    return hipSuccess;
}

// After them: where the other contexts' launches would wait.
static hipError_t leave_resident(lbm_ctx* c, std::unique_lock<std::mutex>& hold) {
    const hipError_t e = hipEventRecord(c->resident_done, c->stream);
    hold.unlock();
    return e;
}

// Rows per unit of a sweep: the run's own choice (lbm_set_run_rows) or `rows`.
static int sweep_rows(const lbm_ctx* c, int run, int ny, int rows) {
    const int own = run < (int)c->run_rows.size() ? c->run_rows[run] : -1;
    return std::max(1, std::min(own < 0 ? rows : own == 0 ? ny : own, ny));
}

// Estimated us of one sweep launch of `steps` steps with about `rows` rows per
// unit.  A unit takes rows + 2 (steps - 1) iterations (the rows beside its own
// that the later stages pull from, and the pipeline's fill) and about three
// iterations' time to start; a memory pass is bounded by 4.8 TB/s.
// For the choice of the rows: with two waves per SIMD (the registers allow no
// more) an iteration takes 1.2 us plus 0.8 us per stage, alone on its SIMD
// 0.6 of that (measured, MI355X: 1 x 128 x 512 for a lone wave, 256 x 1024 x 128 for a full device); units of
// fewer than 32 rows take longer (us per launch of four steps, 12, 20
// and 32 x 1024 x 256 in units of 13, 22 and 32 rows: 148, 194 and 204, without
// the last factor 92, 130 and 184).
// `chosen`: of the rows chosen, for the choice of the kernel.  Us of an iteration of four steps, over 160 lattices of
// 1.5 M to 40 M cells: 3.5 to 4.6 in whole strips whatever the share of the device that the workgroups fill, in ranges
// up to 5.9 where a unit has seven or eight waves; central moments 1.15 times, with three rates 1.6 times as long.
static double sweep_cost(const lbm_ctx* c, const SweepPlan& p, int steps, int rows, const int* members, bool chosen) {
    const double slots = (double)c->cu_count * (SWEEP_WAVES / p.args.block_waves);
    double load = 0.0, longest = 0.0, blocks = 0.0, bytes = 0.0;
    bool cut = false;
    for (int s = 0; s < c->nseg; ++s) {
        const lbm_member_desc& d = c->desc[c->seg[s].member_begin];
        const int h = sweep_rows(c, s, d.ny, rows), ranges = (d.ny + h - 1) / h;
        const double len = h + 2.0 * (steps - 1) + 3.0;
        const int per = p.args.block_waves / p.args.seg[s].waves;
        const double nb = std::ceil((double)members[s] * ranges / per);
        blocks += nb;
        load += nb * len;
        longest = std::max(longest, len);
        bytes += (double)members[s] * d.nx * (72.0 * d.ny + 72.0 * (steps - 1) * (ranges - 1));
        cut = cut || ranges > 1;
    }
    const double rounds = c->nseg == 1 ? std::ceil(blocks / slots) * longest : std::max(longest, load / slots + 0.5 * longest);
    double iteration = 1.2 + 0.8 * steps;
    if (chosen) {
        iteration *= (c->model == 1 ? 1.5 : c->model == 2 ? 1.1 : 0.95) * (cut ? (p.args.block_waves > 6 ? 1.2 : 1.08) : 1.0);
        return std::max(rounds * iteration, bytes / 4.8e6) + 4.0;
    }
    const double fill = std::min(1.0, blocks / slots);
    iteration *= fill > 0.5 ? 0.2 + 0.8 * fill : 0.6;
    return std::max(rounds * iteration, bytes / 4.8e6) * (1.0 + 0.03 * std::max(0, 32 - rows)) + 4.0;
}

// Estimated us per step of the one- and two-step kernels.  Two steps: workgroups, two on a compute unit, of so many rows each,
// us per row 1.75, 1.7 (central moments) and 2.2 (three rates), in open channels 2.2, 2.15 and 2.5, and 4 us per launch
// (open: 7 more for the outlet's).  One step: 6 us (open 13, three rates 1.5 more) and in rows of four cells per lane 80 G
// updates/s, or 58 to 78 by how much of the waves' 256 columns a row fills (open 68 by that); one cell per lane 78, 52 beyond 2.6 M
// cells (190 MB), open 48.  Over 500 lattices of 0.1 M to 40 M cells these are within a quarter of the time nine times in ten.
static double others_cost(const lbm_ctx* c, double cells) {
    if (two_step_now(c)) {
        double load = 0.0, groups = 0.0, tallest = 0.0;
        for (int s = 0; s < c->nseg2; ++s) {
            const int end = s + 1 < c->nseg2 ? c->seg2[s + 1].member_begin : c->n;
            double g = 0.0;
            for (int m = c->seg2[s].member_begin; m < end; ++m)
                if (c->h_active[m]) g += c->seg2[s].tiles_per_member;
            groups += g;
            load += g * (c->seg2[s].rows + 3);
            tallest = std::max(tallest, (double)c->seg2[s].rows + 3);
        }
        const double slots = 2.0 * c->cu_count;
        const double rounds = c->nseg2 == 1 ? std::ceil(groups / slots) * tallest : std::max(tallest, load / slots);
        const double row = c->open ? (c->model == 1 ? 2.5 : c->model == 2 ? 2.15 : 2.2) : c->model == 1 ? 2.2 : c->model == 2 ? 1.7 : 1.75;
        return (4.0 + (c->open ? 7.0 : 0.0) + rounds * row) / 2.0 + (c->model == 1 ? 1.5 : 0.0);
    }
    bool four = true;
    double filled = 1.0;  // the share of the waves' columns that the rows fill, at the worst
    for (int s = 0; s < c->nseg; ++s) {
        const int nx = c->desc[c->seg[s].member_begin].nx;
        four = four && c->seg[s].vec;
        filled = std::min(filled, nx / (256.0 * ((nx + 255) / 256)));
    }
    double rate;
    if (four) rate = c->open ? 68e3 * filled : std::min(80e3, std::max(78e3 * filled, 58e3));
    else rate = c->open ? 48e3 : cells < 2.6e6 ? 78e3 : 52e3;
    return cells / rate + (c->open ? 13.0 : 6.0) + (c->model == 1 ? 1.5 : 0.0);
}

// The sweep takes lattices of up to 64 SWEEP_WAVES SWEEP_CELLS = 1024 columns in periodic channels, with the
// adaptive shape.
static bool sweep_takes(const lbm_ctx* c) {
    if (!TILE_SHAPES[c->tile_id].adaptive || c->open) return false;
    for (int s = 0; s < c->nseg; ++s) {
        const lbm_member_desc& d = c->desc[c->seg[s].member_begin];
        if (36LL * d.nx * d.ny >= (1LL << 31) || d.nx > 64 * SWEEP_WAVES * SWEEP_CELLS) return false;
    }
    return true;
}

// The sweep launch of a batch (steps per launch and the table of units) with its estimated time per step, for
// ensembles of 3 M cells or more; false if another kernel should step it.
static bool plan_sweep(const lbm_ctx* c, SweepPlan& p, bool every_member) {
    if (!sweep_takes(c)) return false;
    const bool listed = !every_member && c->n_active < c->n && c->uniform_shape;
    p = SweepPlan();
    SweepArgs& a = p.args;
    a.nseg = c->nseg;
    a.full = 1;
    a.block_waves = 1;
    int members[MAX_SEGMENTS], tallest = 0;
    double cells = 0.0;
    for (int s = 0; s < c->nseg; ++s) {
        const lbm_member_desc& d = c->desc[c->seg[s].member_begin];
        const int end = s + 1 < c->nseg ? c->seg[s + 1].member_begin : c->n;
        const int lanes = (d.nx + SWEEP_CELLS - 1) / SWEEP_CELLS;
        SweepSegment& g = a.seg[s];
        g.member_begin = c->seg[s].member_begin;
        g.waves = (lanes + 63) / 64;
        g.lanes = (lanes + g.waves - 1) / g.waves;
        a.block_waves = std::max(a.block_waves, g.waves);
        if (d.nx % (64 * SWEEP_CELLS)) a.full = 0;
        members[s] = listed ? c->n_active : end - g.member_begin;
        tallest = std::max(tallest, d.ny);
        cells += (double)members[s] * d.nx * d.ny;
    }
    double best = 1e300;
    int rows = tallest;
    // every height that cuts the tallest lattice into equal parts, from the whole of it down (some 2 sqrt(ny) of them)
    for (int steps : {4, 2})
        for (int h = tallest;;) {
            const double t = sweep_cost(c, p, steps, h, members, false) / steps;
            if (t < best) {
                best = t;
                rows = h;
                p.steps = steps;
            }
            if (h == 1) break;
            const int parts = (tallest + h - 2) / (h - 1);  // the fewest that are lower
            h = (tallest + parts - 1) / parts;
        }
    p.us = sweep_cost(c, p, p.steps, rows, members, true) / p.steps;
    if (cells < 3e6 && c->batch_kernel != LBM_KERNEL_SWEEP) return false;
    int blocks = 0;
    for (int s = 0; s < c->nseg; ++s) {
        const int ny = c->desc[c->seg[s].member_begin].ny;
        SweepSegment& g = a.seg[s];
        g.rows = sweep_rows(c, s, ny, rows);
        g.ranges = (ny + g.rows - 1) / g.rows;
        g.units_per_block = a.block_waves / g.waves;
        if ((long long)members[s] * g.ranges + blocks > (1LL << 30)) return false;
        g.units = members[s] * g.ranges;
        g.block_begin = blocks;
        blocks += (g.units + g.units_per_block - 1) / g.units_per_block;
    }
    a.total_blocks = blocks;
    a.members = c->d_members;
    a.parity = c->d_parity;
    a.active = c->d_active;
    a.active_list = listed ? c->d_active_list : nullptr;
    a.pop0 = c->pop[0];
    a.pop1 = c->pop[1];
    a.partial = c->d_partial;
    return true;
}

// Which kernel steps the next batch of n_steps with the adaptive shape
// (LBM_KERNEL_*): the one asked for (lbm_set_batch_kernel), or by the estimated
// times.  us per step in long batches, resident launches and the others:
// 1 x 256 x 64 2.1 and 6.8, 16 x 512 x 128 6.7 and 15.6, 64 x 512 x 128 26.5 and
// 44, 20 x 1024 x 256 31.6 and 48.5, 32 x 1024 x 256 52.1 and 51.0, 256 x 512 x
// 128 106 and 80; open
// channels of 16, 64 and 512 x 512 x 128 7.4 and 25.4, 28.5 and 51, 226 and 321.
// Resident launches also load and store the state: 13 us (open 15) and 11 for each launch after the first, and
// the copy's time (500 lattices: 11 to 20, and 5 to 15 per launch), which is part of their us per step in whole
// chunks.  Short of eight steps that decides: two steps of 1 x 768 x 94 21.3 us and 19.7 with one step per launch,
// of 97 x 399 x 68 111 and 79, three of open 437 x 601 x 58 1144 and 949; four of 11 x 256 x 47 27 and 42.  A sweep
// of fewer steps than a launch makes takes about 0.45 of the launch; batches of one to three steps are never swept.
// Of 500 lattices of 0.1 M to 40 M cells with every collision, in batches of 1, 2, 3, 4, 5, 8, 16 and 64 steps, 1 % take more than
// 3 % longer than with the one- or two-step kernel (1.25 times at most), and all together 2.5 % longer than with the best of the three.
// resting: no resident launches now.
static int plan_batch(const lbm_ctx* c, int n_steps, BatchPlans& p, bool every_member, bool resting) {
    const int asked = c->batch_kernel;
    if (asked == LBM_KERNEL_PLAIN) return LBM_KERNEL_PLAIN;
    if (!p.resident_known) {
        p.resident_found = plan_resident(c, p.resident, every_member);
        p.cells = 0.0;  // those the launches cover
        for (int m = 0; m < c->n; ++m)
            if (every_member || !c->uniform_shape || c->h_active[m]) p.cells += (double)c->desc[m].nx * c->desc[m].ny;
    }
    p.resident_known = true;
    const ResidentPlan& resident = p.resident;
    bool stays = p.resident_found && !resting && asked != LBM_KERNEL_SWEEP;
    if (stays) {
        hipStreamCaptureStatus captured;  // a replay would not be known to the other contexts' launches
        if (hipStreamIsCapturing(c->stream, &captured) != hipSuccess) {
            (void)hipGetLastError();
            stays = false;
        } else if (captured != hipStreamCaptureStatusNone) {
            stays = false;
        }
    }
    if (stays && ((resident.passes == 1 && n_steps >= 8) || asked == LBM_KERNEL_RESIDENT)) return LBM_KERNEL_RESIDENT;
    if (!p.sweep_known) p.sweep_found = plan_sweep(c, p.sweep, every_member);
    p.sweep_known = true;
    if (asked == LBM_KERNEL_SWEEP) return p.sweep_found ? LBM_KERNEL_SWEEP : LBM_KERNEL_PLAIN;
    if (!stays && !p.sweep_found) return LBM_KERNEL_PLAIN;
    if (!p.others_known) p.others_us = others_cost(c, p.cells);
    p.others_known = true;
    int kernel = LBM_KERNEL_PLAIN;
    double us = p.others_us * n_steps;
    if (p.sweep_found && n_steps >= 4) {
        const int left = n_steps < c->chunk ? n_steps % p.sweep.steps : 0;
        const double swept = p.sweep.us * (n_steps - left + (left ? 0.45 * p.sweep.steps : 0.0));
        if (swept < us) {
            us = swept;
            kernel = LBM_KERNEL_SWEEP;
        }
    }
    if (stays) {
        const double start = n_steps < c->chunk ? (c->open ? 15.0 : 13.0) + 11.0 * (resident.passes - 1) + 72.0 * p.cells / 5.2e6 : 0.0;
        if (start + resident.us * n_steps < (n_steps < 4 ? 0.95 : 1.0) * us) kernel = LBM_KERNEL_RESIDENT;
    }
    return kernel;
}

// The tables, the collision, the channel or the active members have changed.
static void forget_plans(lbm_ctx* c) { c->plans.resident_known = c->plans.sweep_known = c->plans.others_known = false; }

// Tables of the current tile shape.  A two-step shape applies when every
// member's width is a multiple of 256 and its block fits 32-bit byte
// offsets; otherwise (and for the last step of an odd chunk) the library
// steps with the one-step shape 0, which gives the same results.
static int build_segments(lbm_ctx* c) {
    const TileShape ts = TILE_SHAPES[c->tile_id];
    ++c->table_gen;
    forget_plans(c);
    c->two_step = false;
    c->one_tile = c->tile_id;
    if (ts.steps == 2) {
        c->one_tile = 0;
        bool ok = true;
        for (int m = 0; m < c->n; ++m)
            ok = ok && c->desc[m].nx % 256 == 0 && 36LL * c->desc[m].nx * c->desc[m].ny < (1LL << 31);
        if (ok) {
            int rc = build_table(c, ts, true, c->seg2, c->nseg2, c->total_blocks2);
            if (rc) return rc;
            c->two_step = true;
            c->split2 = false;
            for (int s = 0; s < c->nseg2; ++s)
                c->split2 = c->split2 || c->seg2[s].rows < c->desc[c->seg2[s].member_begin].ny;
        }
    }
    return build_table(c, TILE_SHAPES[c->one_tile], false, c->seg, c->nseg, c->total_blocks);
}

extern "C" int lbm_create(lbm_ctx** out, const lbm_member_desc* members, int32_t n_members, float* pop_a,
                          float* pop_b, size_t pop_floats, float* drag_series, int32_t series_capacity,
                          double* accum, void* hip_stream) {
    if (!out) return lbm_fail(LBM_EINVAL, "out is NULL");
    *out = nullptr;
    if (!members || n_members <= 0) return lbm_fail(LBM_EINVAL, "need at least one member");
    if (n_members > MAX_MEMBERS) return lbm_fail(LBM_EINVAL, "at most %d members", MAX_MEMBERS);
    if (!pop_a || !pop_b || !drag_series || !accum) return lbm_fail(LBM_EINVAL, "NULL device buffer");
    if (pop_a == pop_b) return lbm_fail(LBM_EINVAL, "pop_a and pop_b must be distinct buffers");
    if (((uintptr_t)pop_a | (uintptr_t)pop_b) & 15) return lbm_fail(LBM_EINVAL, "population buffers must be 16-byte aligned");
    if (series_capacity < 1) return lbm_fail(LBM_EINVAL, "series_capacity must be >= 1");
    for (int i = 0; i < n_members; ++i) {
        int rc = validate_member(members[i], i);
        if (rc) return rc;
    }
    const size_t need = lbm_state_floats(members, n_members);
    if (pop_floats < need) return lbm_fail(LBM_EINVAL, "population buffers hold %zu floats, need %zu", pop_floats, need);

    lbm_ctx* c = new lbm_ctx();
    c->n = n_members;
    c->desc.assign(members, members + n_members);
    c->pop[0] = pop_a;
    c->pop[1] = pop_b;
    c->pop_floats = pop_floats;
    c->series = drag_series;
    c->cap = series_capacity;
    c->accum = accum;
    c->stream = (hipStream_t)hip_stream;
    c->h_parity.assign(n_members, 0);
    c->h_cursor.assign(n_members, 0);
    c->h_active.assign(n_members, 1);

    long long off = 0, part = 0;
    c->h_members.resize(n_members);
    c->uniform_shape = true;
    for (int i = 0; i < n_members; ++i) {
        const auto& d = members[i];
        MemberDev& m = c->h_members[i];
        m.nx = d.nx;
        m.ny = d.ny;
        m.sx0 = d.sq_x0;
        m.sy0 = d.sq_y0;
        m.ss = d.sq_side;
        m.ring = d.sq_side > 0 ? 4 * d.sq_side + 4 : 0;
        const double omega = 1.0 / d.tau;
        m.omega = omega;
        m.half_fx = 0.5 * d.force_x;
        m.force = d.force_x;
        bgk_coefficients(m);
        m.sb = m.s3 = m.s4 = 1.0;
        m.model = 0;
        m.open = 0;
        m.gx0 = m.bar = 0;
        m.sp_x0 = d.nx;
        m.out_rho = 0;
        m.tau = m.tau_sp = d.tau;
        m.sp_inv = 0.0;
        m.u_c = 0.0;
        m.ghost_off = 0;
        m.off = off;
        m.part_off = part;
        off += member_floats(d);
        part += (long long)m.ring * MAX_CHUNK;
        c->max_cells = std::max<long long>(c->max_cells, (long long)d.nx * d.ny);
        c->max_ny = std::max(c->max_ny, d.ny);
        if (d.nx != members[0].nx || d.ny != members[0].ny) c->uniform_shape = false;
    }
    c->partial_floats = std::max<long long>(part, 1);
    c->tile_id = DEFAULT_TILE;
    {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && cus > 0)
            c->cu_count = cus;
        c->device = dev;
    }
    int rc = build_segments(c);
    if (rc) {
        delete c;
        return rc;
    }

    hipError_t e;
    if ((e = hipMalloc(&c->d_members, sizeof(MemberDev) * n_members)) != hipSuccess ||
        (e = hipMalloc(&c->d_parity, sizeof(int) * n_members)) != hipSuccess ||
        (e = hipMalloc(&c->d_cursor, sizeof(int) * n_members)) != hipSuccess ||
        (e = hipMalloc(&c->d_active, sizeof(int) * n_members)) != hipSuccess ||
        (e = hipMalloc(&c->d_active_list, sizeof(int) * n_members)) != hipSuccess ||
        (e = hipMalloc(&c->d_flags, sizeof(int) * n_members)) != hipSuccess ||
        (e = hipMalloc(&c->d_given_up, sizeof(int) * (n_members + 1))) != hipSuccess ||
        (e = hipMalloc(&c->d_redo, sizeof(int) * (std::max(n_members, REDO_TASKS) + 2))) != hipSuccess ||
        (e = hipMalloc(&c->d_partial, sizeof(double) * c->partial_floats)) != hipSuccess ||
        (e = hipMalloc(&c->d_scratch, sizeof(double) * (4 * (size_t)n_members + 64))) != hipSuccess ||
        (e = hipMalloc(&c->d_iscratch, sizeof(int) * (4 * (size_t)n_members + 64))) != hipSuccess) {
        lbm_destroy(c);
        return lbm_hip_fail(e, "hipMalloc of library scratch");
    }
    if ((e = hipMemcpy(c->d_members, c->h_members.data(), sizeof(MemberDev) * n_members, hipMemcpyHostToDevice)) !=
        hipSuccess) {
        lbm_destroy(c);
        return lbm_hip_fail(e, "upload of member table");
    }
    if ((e = fill_int(c->d_parity, n_members, 0, c->stream)) != hipSuccess ||
        (e = fill_int(c->d_cursor, n_members, 0, c->stream)) != hipSuccess ||
        (e = fill_int(c->d_active, n_members, 1, c->stream)) != hipSuccess ||
        (e = fill_iota(c->d_active_list, n_members, c->stream)) != hipSuccess ||
        (e = fill_int(c->d_given_up, n_members + 1, 0, c->stream)) != hipSuccess ||
        (e = clear_redo(c, c->stream)) != hipSuccess ||
        (e = fill_int(c->d_flags, n_members, 0, c->stream)) != hipSuccess) {
        lbm_destroy(c);
        return lbm_hip_fail(e, "initialising bookkeeping");
    }
    allocate_resident(c);
    c->n_active = n_members;
    *out = c;
    return LBM_OK;
}

extern "C" int lbm_destroy(lbm_ctx* c) {
    if (!c) return LBM_OK;
    if (c->stream) hipStreamSynchronize(c->stream); else hipDeviceSynchronize();
    hipFree(c->d_members);
    hipFree(c->d_parity);
    hipFree(c->d_cursor);
    hipFree(c->d_active);
    hipFree(c->d_active_list);
    hipFree(c->d_flags);
    hipFree(c->d_given_up);
    hipFree(c->d_redo);
    hipFree(c->d_halo);
    if (c->gave_up) hipHostFree(c->gave_up);
    if (c->resident_done) {
        ResidentUsers& u = resident_users();
        const std::lock_guard<std::mutex> hold(u.lock);
        const auto at = std::find(u.users.begin(), u.users.end(), c);
        if (at != u.users.end()) u.users.erase(at);
        hipEventDestroy(c->resident_done);
    }
    hipFree(c->d_partial);
    hipFree(c->d_scratch);
    hipFree(c->d_iscratch);
    hipFree(c->d_ghost);
    free_chunk_graph(c);
    if (c->cap_stream) hipStreamDestroy(c->cap_stream);
    free_rare_scratch(c);
    delete c;
    return LBM_OK;
}

static FinalizeArgs finalize_args(lbm_ctx* c, int n, int accumulate, int swap_parity) {
    FinalizeArgs f;
    f.members = c->d_members;
    f.active = c->d_active;
    f.parity = c->d_parity;
    f.cursor = c->d_cursor;
    f.flags = c->d_flags;
    f.partial = c->d_partial;
    f.series = c->series;
    f.accum = c->accum;
    f.ld = c->cap;
    f.n = n;
    f.accumulate = accumulate;
    f.swap_parity = swap_parity;
    f.mu = c->mu;
    f.inv_sigma_dt = c->dt / c->sigma;
    return f;
}

// The reduction of the last chunk of resident launches (states_only: an untracked one, of `flip`).
static hipError_t finalize_resident(lbm_ctx* c, const ResidentPlan& p, int n, int flip, bool states_only, hipStream_t st) {
    RedoArgs r;
    r.launch = c->resident_launch;
    r.given_up = c->d_given_up;
    r.n_members = c->n;
    r.active_list = p.listed ? c->d_active_list : nullptr;
    r.slots = p.slots;
    r.bands = std::max(1, std::min(REDO_TASKS / p.slots, (c->max_ny + 3) / 4));
    r.flip = flip;
    r.states_only = states_only ? 1 : 0;
    r.done = c->d_redo;
    r.ticket = c->d_redo + std::max(c->n, REDO_TASKS);
    r.gave_up_host = c->gave_up;
    r.pop0 = c->pop[0];
    r.pop1 = c->pop[1];
    r.partial = c->d_partial;
    r.ghost = c->d_ghost;
    return launch_finalize_resident(finalize_args(c, n, 1, 1), r, st);
}

extern "C" int lbm_init(lbm_ctx* c, uint64_t seed, double noise_amp) { return lbm_init_flow(c, seed, noise_amp, 0.0); }

extern "C" int lbm_init_flow(lbm_ctx* c, uint64_t seed, double noise_amp, double ux0) {
    if (!c) return lbm_fail(LBM_EINVAL, "NULL context");
    if (!std::isfinite(noise_amp) || noise_amp < 0 || noise_amp >= 0.5)
        return lbm_fail(LBM_EINVAL, "noise_amp must be in [0, 0.5)");
    if (!std::isfinite(ux0) || std::fabs(ux0) > 0.3) return lbm_fail(LBM_EINVAL, "|ux0| must be <= 0.3");
    if (c->open && ux0 != 0.0) return lbm_fail(LBM_EINVAL, "an open channel starts from its inlet profile: ux0 must be 0");
    hipError_t e;
    if ((e = fill_int(c->d_parity, c->n, 0, c->stream)) != hipSuccess ||
        (e = fill_int(c->d_cursor, c->n, 0, c->stream)) != hipSuccess ||
        (e = fill_int(c->d_active, c->n, 1, c->stream)) != hipSuccess ||
        (e = fill_iota(c->d_active_list, c->n, c->stream)) != hipSuccess ||
        (e = fill_int(c->d_flags, c->n, 0, c->stream)) != hipSuccess ||
        (e = fill_double(c->accum, c->n, 0.0, c->stream)) != hipSuccess)
        return lbm_hip_fail(e, "lbm_init bookkeeping");
    std::fill(c->h_parity.begin(), c->h_parity.end(), 0);
    std::fill(c->h_active.begin(), c->h_active.end(), 1);
    c->n_active = c->n;
    forget_plans(c);
    InitArgs a;
    a.members = c->d_members;
    a.pop0 = c->pop[0];
    a.partial = c->d_partial;
    a.seed = seed;
    a.noise_amp = noise_amp;
    a.ux0 = ux0;
    if ((e = launch_init(a, c->n, c->max_cells, c->stream)) != hipSuccess) return lbm_hip_fail(e, "init kernel");
    if ((e = launch_finalize(finalize_args(c, 1, 0, 0), c->n, c->stream)) != hipSuccess)
        return lbm_hip_fail(e, "drag reduction");
    std::fill(c->h_cursor.begin(), c->h_cursor.end(), 1);
    return LBM_OK;
}

extern "C" int lbm_set_observable(lbm_ctx* c, double mu, double sigma, double dt) {
    if (!c) return lbm_fail(LBM_EINVAL, "NULL context");
    if (!std::isfinite(mu) || !(sigma > 0) || !std::isfinite(sigma) || !(dt > 0) || !std::isfinite(dt))
        return lbm_fail(LBM_EINVAL, "need finite mu, sigma > 0, dt > 0");
    c->mu = mu;
    c->sigma = sigma;
    c->dt = dt;
    return LBM_OK;
}

extern "C" int lbm_set_active(lbm_ctx* c, const int32_t* active_host) {
    if (!c) return lbm_fail(LBM_EINVAL, "NULL context");
    MaskBits bits{};
    c->n_active = 0;
    for (int m = 0; m < c->n; ++m) {
        const int on = active_host ? (active_host[m] != 0) : 1;
        c->h_active[m] = on;
        c->n_active += on;
        if (on) bits.w[m >> 5] |= 1u << (m & 31);
    }
    forget_plans(c);
    hipError_t e = set_bits(c->d_active, c->d_active_list, c->n, bits, c->stream);
    return e == hipSuccess ? LBM_OK : lbm_hip_fail(e, "active mask upload");
}

extern "C" int lbm_step_batch(lbm_ctx* c, int32_t n_steps) {
    if (!c) return lbm_fail(LBM_EINVAL, "NULL context");
    if (n_steps < 0) return lbm_fail(LBM_EINVAL, "n_steps must be >= 0");
    if (n_steps == 0) return LBM_OK;
    for (int m = 0; m < c->n; ++m)
        if (c->h_active[m] && (long long)c->h_cursor[m] + n_steps > c->cap)
            return lbm_fail(LBM_ERANGE, "member %d: drag column %d + %d steps exceeds capacity %d", m,
                            c->h_cursor[m], n_steps, c->cap);
    StepArgs a;
    a.members = c->d_members;
    a.parity = c->d_parity;
    a.active = c->d_active;
    a.pop0 = c->pop[0];
    a.pop1 = c->pop[1];
    a.partial = c->d_partial;
    a.xcd = TILE_SHAPES[c->one_tile].xcd;
    a.split = 0;
    a.total_blocks = c->total_blocks;
    a.nseg = c->nseg;
    for (int s = 0; s < c->nseg; ++s) a.seg[s] = c->seg[s];
    StepArgs a2 = a;
    if (c->two_step) {
        a2.xcd = TILE_SHAPES[c->tile_id].xcd;
        a2.split = c->split2 ? 1 : 0;
        a2.total_blocks = c->total_blocks2;
        a2.nseg = c->nseg2;
        for (int s = 0; s < c->nseg2; ++s) a2.seg[s] = c->seg2[s];
    }
    const int waves2 = TILE_SHAPES[c->tile_id].tyt;
    const bool two = two_step_now(c);
    ResidentPlan& resident = c->plans.resident;
    SweepPlan& sweep = c->plans.sweep;
    // A chunk was given up: something else keeps holding part of the device (another process, long
    // kernels of other streams), and a chunk stepped again costs several times a good one.
    if (c->gave_up && *(volatile int*)c->gave_up && c->wait_ticks >= 0) {
        *(volatile int*)c->gave_up = 0;
        c->resident_rest = RESIDENT_REST;
    }
    c->resident_first = c->resident_launch + 1;
    int kernel = plan_batch(c, n_steps, c->plans, false, false);
    if (kernel == LBM_KERNEL_RESIDENT && c->resident_rest > 0 && c->batch_kernel != LBM_KERNEL_RESIDENT) {
        --c->resident_rest;
        kernel = plan_batch(c, n_steps, c->plans, false, true);
    }
    const bool stays = kernel == LBM_KERNEL_RESIDENT, swept = kernel == LBM_KERNEL_SWEEP;
    a.active_list = nullptr;
    a2.active_list = nullptr;
    a.ghost = c->open ? c->d_ghost : nullptr;
    a2.ghost = a.ghost;
    GhostArgs g;
    g.members = c->d_members;
    g.parity = c->d_parity;
    g.active = c->d_active;
    g.pop0 = c->pop[0];
    g.pop1 = c->pop[1];
    g.ghost = c->d_ghost;
    if (c->n_active == 0) return LBM_OK;  // nothing steps (no drag column either)
    if (c->n_active < c->n && c->uniform_shape) {
        // launch the active members' tiles only: the inactive ones would cost a
        // workgroup dispatch each (the grid of a full ensemble) for no work
        a.active_list = c->d_active_list;
        a.total_blocks = c->n_active * c->seg[0].tiles_per_member;
        if (c->two_step) {
            a2.active_list = c->d_active_list;
            a2.total_blocks = c->n_active * c->seg2[0].tiles_per_member;
        }
    }
    // the launches of one chunk of steps on stream st; `launches` counts them
    // (every launch swaps the buffers once, whether it makes one step or two)
    auto enqueue = [&](int chunk, hipStream_t st, int& launches) -> hipError_t {
        hipError_t e;
        int s = 0;
        launches = 0;
        if (stays) {
            launches = 1;  // every member's buffers swap once
            if ((e = launch_resident_passes(c, resident, chunk, 0, st)) != hipSuccess) return e;
            return finalize_resident(c, resident, chunk, 0, false, st);
        }
        if (swept)
            for (int t; s < chunk; s += t, ++launches) {
                t = std::min(sweep.steps, chunk - s);
                sweep.args.slot = s;
                sweep.args.flip = launches & 1;
                if ((e = launch_sweep(t, sweep.args, c->model, st)) != hipSuccess) return e;
            }
        if (two)
            for (; s + 1 < chunk; s += 2, ++launches) {
                a2.slot = s;
                a2.flip = launches & 1;
                if (c->open) {  // the inlet's values and the outlet ghost column of the first of the two steps
                    g.flip = a2.flip;
                    if ((e = launch_outlet_ghost(g, c->n, c->max_ny, st)) != hipSuccess) return e;
                }
                if ((e = launch_step2(waves2, a2, c->model, st)) != hipSuccess) return e;
            }
        for (; s < chunk; ++s, ++launches) {
            a.slot = s;
            a.flip = launches & 1;
            if (c->open) {
                g.flip = a.flip;
                if ((e = launch_outlet_ghost(g, c->n, c->max_ny, st)) != hipSuccess) return e;
            }
            if ((e = launch_step(c->one_tile, a, c->model, st)) != hipSuccess) return e;
        }
        return launch_finalize(finalize_args(c, chunk, 1, launches & 1), c->n, st);
    };
    hipError_t e;
    int done = 0;
    // Resident chunks are enqueued a few at a time under the users' lock, so that another thread's context waits for
    // these at most and not for a whole long batch.
    constexpr int CHUNKS_HELD = 8;
    ResidentUsers* const users = stays ? &resident_users() : nullptr;
    std::unique_lock<std::mutex> hold;
    while (done < n_steps) {
        const int chunk = std::min(n_steps - done, c->chunk);
        int launches = 0;
        if (stays && !hold.owns_lock()) {
            hold = std::unique_lock<std::mutex>(users->lock);
            if ((e = admit_resident(c, *users, resident)) != hipSuccess) return lbm_hip_fail(e, "resident launch");
        }
        if (c->graphs && chunk == c->chunk && !stays) {  // (a resident chunk is two launches)
            ChunkGraphKey key{c->tile_id, c->one_tile, two ? 1 : 0, waves2, c->model, c->open ? 1 : 0, chunk,
                              c->table_gen, a.total_blocks, a2.total_blocks, a.active_list ? 1 : 0, c->mu, c->dt / c->sigma,
                              (const void*)c->d_ghost};
            if (swept) {
                sweep.args.slot = sweep.args.flip = 0;
                key.sweep = sweep;
            }
            if (!c->graph_exec || !(key == c->graph_key)) {
                free_chunk_graph(c);
                if (!c->cap_stream && (e = hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking)) != hipSuccess)
                    return lbm_hip_fail(e, "capture stream");
                if ((e = hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeThreadLocal)) != hipSuccess)
                    return lbm_hip_fail(e, "begin capture");
                int l = 0;
                const hipError_t ce = enqueue(chunk, c->cap_stream, l);
                hipGraph_t gr = nullptr;
                const hipError_t ee = hipStreamEndCapture(c->cap_stream, &gr);
                if (ce != hipSuccess || ee != hipSuccess) {
                    if (gr) hipGraphDestroy(gr);
                    return lbm_hip_fail(ce != hipSuccess ? ce : ee, "capture of a chunk of steps");
                }
                if ((e = hipGraphInstantiateWithFlags(&c->graph_exec, gr, 0)) != hipSuccess) {
                    hipGraphDestroy(gr);
                    c->graph_exec = nullptr;
                    return lbm_hip_fail(e, "graph instantiation");
                }
                c->graph = gr;
                c->graph_key = key;
                c->graph_launches = l;
            }
            if ((e = hipGraphLaunch(c->graph_exec, c->stream)) != hipSuccess) return lbm_hip_fail(e, "graph launch");
            launches = c->graph_launches;
        } else if ((e = enqueue(chunk, c->stream, launches)) != hipSuccess) {
            if (stays) (void)leave_resident(c, hold);  // (what was launched still runs)
            return lbm_hip_fail(e, "lattice step launches");
        }
        for (int m = 0; m < c->n; ++m)
            if (c->h_active[m]) {
                c->h_parity[m] ^= (launches & 1);
                c->h_cursor[m] += chunk;
            }
        done += chunk;
        if (stays && (done == n_steps || done % (CHUNKS_HELD * c->chunk) == 0) && (e = leave_resident(c, hold)) != hipSuccess)
            return lbm_hip_fail(e, "resident launch");
    }
    return LBM_OK;
}

void free_chunk_graph(lbm_ctx* c) {
    if (c->graph_exec) hipGraphExecDestroy(c->graph_exec);
    if (c->graph) hipGraphDestroy(c->graph);
    c->graph_exec = nullptr;
    c->graph = nullptr;
}

extern "C" int lbm_set_batch_kernel(lbm_ctx* c, int32_t kernel) {
    if (!c) return lbm_fail(LBM_EINVAL, "NULL context");
    if (kernel < LBM_KERNEL_ESTIMATED || kernel > LBM_KERNEL_RESIDENT) return lbm_fail(LBM_EINVAL, "kernel %d: -1 to 2", kernel);
    c->batch_kernel = kernel;
    forget_plans(c);
    return LBM_OK;
}

extern "C" int lbm_batch_kernel(lbm_ctx* c, int32_t n_steps, int32_t* out) {
    if (!c || !out) return lbm_fail(LBM_EINVAL, "NULL argument");
    if (n_steps < 1) return lbm_fail(LBM_EINVAL, "n_steps must be >= 1");
    const bool resting = c->resident_rest > 0 && c->batch_kernel != LBM_KERNEL_RESIDENT;
    out[0] = plan_batch(c, n_steps, c->plans, false, resting);
    if (out[0] == LBM_KERNEL_RESIDENT) {
        const ResidentPlan& p = c->plans.resident;
        out[1] = std::min(n_steps, c->chunk);
        out[2] = p.passes;
        out[3] = p.pass[0].cells;
        out[4] = p.pass[0].rows;
    } else if (out[0] == LBM_KERNEL_SWEEP) {
        out[1] = c->plans.sweep.steps;
        out[2] = 1;
        out[3] = SWEEP_CELLS;
        out[4] = c->plans.sweep.args.seg[0].rows;
    } else {
        out[1] = two_step_now(c) ? 2 : 1;
        out[2] = 1;
        out[3] = out[1] == 2 || c->seg[0].vec ? 4 : 1;
        out[4] = out[1] == 2 ? c->seg2[0].rows : TILE_SHAPES[c->one_tile].r;
    }
    return LBM_OK;
}

extern "C" int lbm_set_graphs(lbm_ctx* c, int32_t on) {
    if (!c) return lbm_fail(LBM_EINVAL, "NULL context");
    c->graphs = on != 0;
    return LBM_OK;
}

extern "C" int lbm_set_wait_limit(lbm_ctx* c, int32_t us) {
    if (!c) return lbm_fail(LBM_EINVAL, "NULL context");
    c->wait_ticks = us < 0 ? -1 : 100LL * us;
    return LBM_OK;
}

extern "C" int lbm_drag(const lbm_ctx* c, int32_t t0, int32_t t1, float* out_dev) {
    if (!c) return lbm_fail(LBM_EINVAL, "NULL context");
    if (t0 < 0 || t1 < t0 || t1 > c->cap) return lbm_fail(LBM_EINVAL, "bad column range [%d, %d)", t0, t1);
    if (t1 == t0) return LBM_OK;
    if (!out_dev) return lbm_fail(LBM_EINVAL, "NULL output");
    hipError_t e = hipMemcpy2DAsync(out_dev, sizeof(float) * (t1 - t0), c->series + t0, sizeof(float) * c->cap,
                                    sizeof(float) * (t1 - t0), c->n, hipMemcpyDeviceToDevice, c->stream);
    return e == hipSuccess ? LBM_OK : lbm_hip_fail(e, "drag copy");
}

extern "C" int lbm_member_state(const lbm_ctx* c, int32_t m, float** state_dev) {
    if (!c || !state_dev) return lbm_fail(LBM_EINVAL, "NULL argument");
    if (m < 0 || m >= c->n) return lbm_fail(LBM_EINVAL, "member %d out of range", m);
    *state_dev = c->pop[c->h_parity[m]] + c->h_members[m].off;
    return LBM_OK;
}

extern "C" int lbm_member_time(const lbm_ctx* c, int32_t m, int32_t* t) {
    if (!c || !t) return lbm_fail(LBM_EINVAL, "NULL argument");
    if (m < 0 || m >= c->n) return lbm_fail(LBM_EINVAL, "member %d out of range", m);
    *t = c->h_cursor[m];
    return LBM_OK;
}

extern "C" int lbm_set_time(lbm_ctx* c, int32_t t) {
    if (!c) return lbm_fail(LBM_EINVAL, "NULL context");
    if (t < 0 || t > c->cap) return lbm_fail(LBM_EINVAL, "time %d outside [0, %d]", t, c->cap);
    hipError_t e = fill_int(c->d_cursor, c->n, t, c->stream);
    if (e != hipSuccess) return lbm_hip_fail(e, "cursor reset");
    std::fill(c->h_cursor.begin(), c->h_cursor.end(), t);
    return LBM_OK;
}

extern "C" int lbm_flags(const lbm_ctx* c, int32_t* out_dev) {
    if (!c || !out_dev) return lbm_fail(LBM_EINVAL, "NULL argument");
    hipError_t e = hipMemcpyAsync(out_dev, c->d_flags, sizeof(int) * c->n, hipMemcpyDeviceToDevice, c->stream);
    return e == hipSuccess ? LBM_OK : lbm_hip_fail(e, "flags copy");
}

extern "C" int lbm_set_flags(lbm_ctx* c, const int32_t* flags_dev) {
    if (!c || !flags_dev) return lbm_fail(LBM_EINVAL, "NULL argument");
    hipError_t e = hipMemcpyAsync(c->d_flags, flags_dev, sizeof(int) * c->n, hipMemcpyDeviceToDevice, c->stream);
    return e == hipSuccess ? LBM_OK : lbm_hip_fail(e, "flags copy");
}

extern "C" int lbm_set_collision(lbm_ctx* c, int32_t model, double s_bulk, double s_third, double s_fourth) {
    if (!c) return lbm_fail(LBM_EINVAL, "NULL context");
    if (model != 0 && model != 1) return lbm_fail(LBM_EINVAL, "collision model %d: 0 (BGK) or 1 (central moments)", model);
    if (model == 1)
        for (double s : {s_bulk, s_third, s_fourth})
            if (!(s > 0.0 && s < 2.0)) return lbm_fail(LBM_EINVAL, "relaxation rate %g outside (0, 2)", s);
    // unit bulk, third- and fourth-order rates: the shorter evaluation of the same collision
    const int internal = model == 1 && s_bulk == 1.0 && s_third == 1.0 && s_fourth == 1.0 ? 2 : model;
    c->model = internal;
    forget_plans(c);
    for (auto& m : c->h_members) {
        m.model = internal;
        if (model == 1) {
            m.sb = s_bulk;
            m.s3 = s_third;
            m.s4 = s_fourth;
        }
    }
    hipError_t e = hipMemcpyAsync(c->d_members, c->h_members.data(), sizeof(MemberDev) * c->n, hipMemcpyHostToDevice,
                                  c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    return e == hipSuccess ? LBM_OK : lbm_hip_fail(e, "member table upload");
}

static int validate_open(const lbm_member_desc& d, int i, const lbm_open_channel& o) {
    if (d.ny > 2048) return lbm_fail(LBM_EUNSUPPORTED, "member %d: open channels support ny <= 2048", i);
    if (o.grid_bar > 0) {
        if (o.grid_x0 < 1 || o.grid_x0 + o.grid_bar > d.nx - 2)
            return lbm_fail(LBM_EINVAL, "member %d: the grid must lie within columns 1 .. nx - 3", i);
        if (d.sq_side > 0 && o.grid_x0 + o.grid_bar > d.sq_x0 - 2)
            return lbm_fail(LBM_EINVAL, "member %d: the grid must end at least two columns before the square", i);
    }
    if (d.sq_side > 0 && (d.sq_x0 < 2 || d.sq_x0 + d.sq_side > d.nx - 3))
        return lbm_fail(LBM_EINVAL, "member %d: an open channel needs two fluid columns before and three after the square", i);
    return LBM_OK;
}

extern "C" int lbm_set_open_channel(lbm_ctx* c, const lbm_open_channel* oc) {
    if (!c) return lbm_fail(LBM_EINVAL, "NULL context");
    if (oc) {
        if (oc->outlet_density != 0 && oc->outlet_density != 1)
            return lbm_fail(LBM_EINVAL, "outlet_density must be 0 (held at 1) or 1 (extrapolated)");
        if (!std::isfinite(oc->u_c) || oc->u_c < 0.0 || oc->u_c > 0.3)
            return lbm_fail(LBM_EINVAL, "inlet centre-line velocity must be in [0, 0.3]");
        if (oc->grid_bar < 0) return lbm_fail(LBM_EINVAL, "negative grid bar size");
        if (oc->sponge_x0 < 0) return lbm_fail(LBM_EINVAL, "negative sponge start");
        if (!(oc->sponge_tau > 0.5) || !std::isfinite(oc->sponge_tau))
            return lbm_fail(LBM_EINVAL, "sponge relaxation time must be > 1/2");
        for (int m = 0; m < c->n; ++m) {
            int rc = validate_open(c->desc[m], m, *oc);
            if (rc) return rc;
        }
    }
    hipError_t e = hipStreamSynchronize(c->stream);  // no launch may still read the table or the ghost columns
    if (e != hipSuccess) return lbm_hip_fail(e, "stream synchronisation");
    free_chunk_graph(c);  // it holds the old ghost pointer
    hipFree(c->d_ghost);
    c->d_ghost = nullptr;
    long long goff = 0;
    for (int m = 0; m < c->n; ++m) {
        MemberDev& md = c->h_members[m];
        const auto& d = c->desc[m];
        md.open = oc ? 1 : 0;
        md.gx0 = oc && oc->grid_bar > 0 ? oc->grid_x0 : 0;
        md.bar = oc ? oc->grid_bar : 0;
        md.sp_x0 = oc ? std::min(oc->sponge_x0, d.nx) : d.nx;
        md.tau_sp = oc ? oc->sponge_tau : d.tau;
        md.sp_inv = md.sp_x0 < d.nx - 1 ? 1.0 / (double)(d.nx - 1 - md.sp_x0) : 0.0;
        md.u_c = oc ? oc->u_c : 0.0;
        md.out_rho = oc ? oc->outlet_density : 0;
        md.ghost_off = goff;
        goff += 9LL * d.ny;
    }
    c->open = oc != nullptr;
    if (c->open && (e = hipMalloc(&c->d_ghost, sizeof(float) * (size_t)goff)) != hipSuccess) {
        c->open = false;
        for (auto& md : c->h_members) md.open = md.bar = 0;
        hipMemcpy(c->d_members, c->h_members.data(), sizeof(MemberDev) * c->n, hipMemcpyHostToDevice);
        build_segments(c);
        return lbm_hip_fail(e, "hipMalloc of outlet ghost columns");
    }
    e = hipMemcpy(c->d_members, c->h_members.data(), sizeof(MemberDev) * c->n, hipMemcpyHostToDevice);
    if (e != hipSuccess) return lbm_hip_fail(e, "member table upload");
    return build_segments(c);
}

extern "C" int32_t lbm_tile_count(void) { return N_TILE_SHAPES; }

extern "C" int lbm_launch_steps(const lbm_ctx* c, int32_t* steps) {
    if (!c || !steps) return lbm_fail(LBM_EINVAL, "NULL argument");
    *steps = two_step_now(c) ? 2 : 1;
    return LBM_OK;
}

extern "C" int lbm_set_tile(lbm_ctx* c, int32_t tile_id) {
    if (!c) return lbm_fail(LBM_EINVAL, "NULL context");
    if (tile_id < 0 || tile_id >= N_TILE_SHAPES) return lbm_fail(LBM_EINVAL, "tile id %d out of range", tile_id);
    const int old = c->tile_id;
    c->tile_id = tile_id;
    int rc = build_segments(c);
    if (rc) {
        c->tile_id = old;
        build_segments(c);
    }
    return rc;
}

// Runs of consecutive members with one lattice shape (the segments of the tables).
static int count_runs(const lbm_ctx* c) {
    int runs = 0;
    for (int m = 0; m < c->n; ++m)
        if (m == 0 || c->desc[m].nx != c->desc[m - 1].nx || c->desc[m].ny != c->desc[m - 1].ny) ++runs;
    return runs;
}

extern "C" int lbm_run_count(const lbm_ctx* c, int32_t* n_runs) {
    if (!c || !n_runs) return lbm_fail(LBM_EINVAL, "NULL argument");
    *n_runs = count_runs(c);
    return LBM_OK;
}

extern "C" int lbm_set_run_rows(lbm_ctx* c, const int32_t* rows, int32_t n_runs) {
    if (!c) return lbm_fail(LBM_EINVAL, "NULL context");
    if (n_runs == 0) {
        c->run_rows.clear();
        return build_segments(c);
    }
    if (!rows) return lbm_fail(LBM_EINVAL, "NULL rows");
    if (n_runs != count_runs(c))
        return lbm_fail(LBM_EINVAL, "%d row ranges for %d runs of lattice shapes", n_runs, count_runs(c));
    for (int r = 0; r < n_runs; ++r)
        if (rows[r] < -1) return lbm_fail(LBM_EINVAL, "run %d: rows %d (-1 by the shape, 0 whole strips, >= 1)", r, rows[r]);
    const std::vector<int> old = c->run_rows;
    c->run_rows.assign(rows, rows + n_runs);
    int rc = build_segments(c);
    if (rc) {
        c->run_rows = old;
        build_segments(c);
    }
    return rc;
}

extern "C" int lbm_get_run_rows(const lbm_ctx* c, int32_t* rows, int32_t max_runs, int32_t* n_runs) {
    if (!c || !n_runs) return lbm_fail(LBM_EINVAL, "NULL argument");
    *n_runs = c->two_step ? c->nseg2 : count_runs(c);
    if (rows && max_runs < *n_runs) return lbm_fail(LBM_EINVAL, "room for %d runs, need %d", max_runs, *n_runs);
    if (rows)
        for (int s = 0; s < *n_runs; ++s) {
            // one step per launch: no ranges, but those given for the sweep, which takes any width
            const int ny = c->desc[(c->two_step ? c->seg2[s] : c->seg[s]).member_begin].ny;
            const int given = s < (int)c->run_rows.size() && sweep_takes(c) ? c->run_rows[s] : -1;
            const int used = c->two_step ? c->seg2[s].rows : given;
            rows[s] = used >= ny ? 0 : used;
        }
    return LBM_OK;
}

extern "C" int lbm_autotune(lbm_ctx* c, int32_t n_steps, int32_t* best_tile) {
    if (!c || !best_tile) return lbm_fail(LBM_EINVAL, "NULL argument");
    if (n_steps < 1) return lbm_fail(LBM_EINVAL, "n_steps must be >= 1");
    StepArgs a;
    a.members = c->d_members;
    a.parity = c->d_parity;
    a.active = c->d_active;
    a.pop0 = c->pop[0];
    a.pop1 = c->pop[1];
    a.partial = c->d_partial;
    a.active_list = nullptr;  // every member, whatever the mask
    a.ghost = c->open ? c->d_ghost : nullptr;
    GhostArgs g;
    g.members = c->d_members;
    g.parity = c->d_parity;
    g.active = c->d_active;
    g.pop0 = c->pop[0];
    g.pop1 = c->pop[1];
    g.ghost = c->d_ghost;
    // Launches are timed in pairs so every state ends in the buffer it
    // started in; the states do advance (untracked: no drag, no cursor), so
    // callers tune before lbm_init, which rebuilds step 0.
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
        return lbm_fail(LBM_EHIP, "event creation failed");
    float best_ms = 1e30f;  // per step
    int best = c->tile_id;
    c->run_rows.clear();  // the shapes first, each with its own row policy
    // time the current tables with shape t; ms per step, or a negative value
    // if the shape does not apply
    auto time_shape = [&](int t, float& ms) -> int {
        ms = -1.0f;
        if (build_segments(c) != LBM_OK) return LBM_OK;
        const TileShape ts = TILE_SHAPES[t];
        if (ts.steps == 2 && !ts.adaptive && !c->two_step) return LBM_OK;  // it would run shape 0
        // the adaptive shape: where it stays in registers or sweeps (it runs shape 16 or 0 otherwise)
        BatchPlans plans;
        ResidentPlan& resident = plans.resident;
        SweepPlan& sweep = plans.sweep;
        const int kernel = ts.adaptive ? plan_batch(c, c->chunk, plans, true, false) : LBM_KERNEL_PLAIN;
        const bool stays = kernel == LBM_KERNEL_RESIDENT;
        if (ts.adaptive && kernel == LBM_KERNEL_PLAIN) return LBM_OK;
        const bool two = ts.steps == 2;
        a.total_blocks = two ? c->total_blocks2 : c->total_blocks;
        a.split = two && c->split2 ? 1 : 0;
        a.xcd = ts.xcd;
        a.nseg = two ? c->nseg2 : c->nseg;
        for (int s = 0; s < a.nseg; ++s) a.seg[s] = two ? c->seg2[s] : c->seg[s];
        a.slot = 0;
        auto launch = [&](int flip) {
            a.flip = flip;
            if (c->open) {  // the outlet ghost column the launch's first step pulls
                g.flip = flip;
                hipError_t ge = launch_outlet_ghost(g, c->n, c->max_ny, c->stream);
                if (ge != hipSuccess) return ge;
            }
            if (stays) {
                const hipError_t re = launch_resident_passes(c, resident, c->chunk, flip, c->stream);
                return re == hipSuccess ? finalize_resident(c, resident, c->chunk, flip, true, c->stream) : re;
            }
            if (ts.adaptive) {
                sweep.args.flip = flip;
                return launch_sweep(sweep.steps, sweep.args, c->model, c->stream);
            }
            return two ? launch_step2(ts.tyt, a, c->model, c->stream) : launch_step(t, a, c->model, c->stream);
        };
        std::unique_lock<std::mutex> hold;  // until the timing has ended
        if (stays) {
            ResidentUsers& u = resident_users();
            hold = std::unique_lock<std::mutex>(u.lock);
            if (admit_resident(c, u, resident) != hipSuccess) return lbm_fail(LBM_EHIP, "resident launch");
        }
        c->resident_first = c->resident_launch + 1;
        const int steps_per_launch = stays ? c->chunk : ts.adaptive ? sweep.steps : ts.steps;
        const int pairs = std::max(1, n_steps / (ts.adaptive ? 2 * steps_per_launch : 2));
        // warm-up pair
        launch(0);
        launch(1);
        hipEventRecord(e0, c->stream);
        for (int p = 0; p < pairs; ++p) {
            launch(0);
            launch(1);
        }
        hipEventRecord(e1, c->stream);
        hipError_t err = hipEventSynchronize(e1);
        if (err != hipSuccess) return lbm_hip_fail(err, "autotune timing");
        float t_ms = 0;
        hipEventElapsedTime(&t_ms, e0, e1);
        ms = t_ms / (float)(2 * pairs * steps_per_launch);
        return LBM_OK;
    };
    int rc = LBM_OK;
    for (int t = 0; t < N_TILE_SHAPES && rc == LBM_OK; ++t) {
        c->tile_id = t;
        float ms;
        rc = time_shape(t, ms);
        if (rc == LBM_OK && ms >= 0.0f && ms < best_ms) {
            best_ms = ms;
            best = t;
        }
    }
    // Runs of different lattice sizes (an uneven batch): each run's row range
    // on its own, one run at a time (whole strips, 128, 64 or 32 rows per
    // workgroup), keeping whatever times best for the whole ensemble.
    c->tile_id = best;
    const int runs = count_runs(c);
    if (rc == LBM_OK && TILE_SHAPES[best].steps == 2 && !TILE_SHAPES[best].adaptive && runs > 1 && build_segments(c) == LBM_OK && c->two_step) {
        c->run_rows.assign(runs, -1);
        for (int r = 0; r < runs; ++r) c->run_rows[r] = c->seg2[r].rows >= c->desc[c->seg2[r].member_begin].ny ? 0 : c->seg2[r].rows;
        rc = time_shape(best, best_ms);  // the reference, timed next to the variants
        for (int r = 0; r < runs && rc == LBM_OK; ++r) {
            const int ny = c->desc[c->seg2[r].member_begin].ny;
            int keep = c->run_rows[r];
            for (int h : {0, 128, 64, 32}) {
                if (h == keep || (h > 0 && h >= ny)) continue;
                c->run_rows[r] = h;
                float ms;
                rc = time_shape(best, ms);
                if (rc != LBM_OK) break;
                if (ms >= 0.0f && ms < 0.99f * best_ms) {  // a clear gain only
                    best_ms = ms;
                    keep = h;
                }
            }
            c->run_rows[r] = keep;
        }
    }
    hipEventDestroy(e0);
    hipEventDestroy(e1);
    c->tile_id = best;
    build_segments(c);
    *best_tile = best;
    return rc;
}

// What a tuned launch shape depends on: the runs of lattice shapes, the
// collision and whether the channels are open.
static std::string tune_key(const lbm_ctx* c) {
    std::ostringstream k;
    k << "model=" << c->model << " open=" << (c->open ? 1 : 0) << " shapes=";
    int run = 0;
    for (int m = 0; m < c->n; ++m) {
        ++run;
        if (m + 1 == c->n || c->desc[m + 1].nx != c->desc[m].nx || c->desc[m + 1].ny != c->desc[m].ny) {
            k << c->desc[m].nx << "x" << c->desc[m].ny << "*" << run << ";";
            run = 0;
        }
    }
    return k.str();
}

extern "C" int lbm_autotune_cached(lbm_ctx* c, int32_t n_steps, const char* path, int32_t* best_tile) {
    if (!c || !path || !best_tile) return lbm_fail(LBM_EINVAL, "NULL argument");
    const std::string key = tune_key(c);
    {
        std::ifstream in(path);
        std::string line;
        while (in && std::getline(in, line)) {
            const size_t tab = line.rfind('\t');
            if (tab == std::string::npos || line.compare(0, tab, key) != 0 || tab != key.size()) continue;
            // "<tile>" or "<tile> <rows of run 0>,<rows of run 1>,..."
            std::istringstream val(line.substr(tab + 1));
            int tile = -1;
            val >> tile;
            if (!val && !val.eof()) continue;
            if (tile < 0 || tile >= N_TILE_SHAPES) continue;  // a table from another build: tune again
            std::vector<int32_t> rows;
            std::string list;
            if (val >> list) {
                std::istringstream ls(list);
                std::string item;
                while (std::getline(ls, item, ',')) rows.push_back((int32_t)std::atoi(item.c_str()));
            }
            c->run_rows.clear();
            int rc = lbm_set_tile(c, tile);
            if (rc) return rc;
            if (!rows.empty() && (rc = lbm_set_run_rows(c, rows.data(), (int32_t)rows.size())) != LBM_OK) return rc;
            *best_tile = tile;
            return LBM_OK;
        }
    }
    const int rc = lbm_autotune(c, n_steps, best_tile);
    if (rc) return rc;
    std::ofstream out(path, std::ios::app);
    out << key << '\t' << *best_tile;
    for (size_t r = 0; r < c->run_rows.size(); ++r) out << (r ? ',' : ' ') << c->run_rows[r];
    out << '\n';
    if (!out) return lbm_fail(LBM_EINVAL, "cannot append the tuned shape to %s", path);
    return LBM_OK;
}
