// Lattice-Boltzmann kernels: initial state, fused pull-stream + BGK collide
// step with momentum-exchange drag partials, and the per-chunk drag
// reduction with the FP64 observable integral.
//
// Paper Appendix A gives the scheme (exact streaming, BGK relaxation to the
// second-order equilibrium); Section 2 the halfway bounce-back on walls and
// obstacle; Section 2.1 the drag.  Populations are FP32 deviations
// d_i = f_i - w_i so that the O(1) rest weights never enter FP32 sums.
#include "lbm_device.hpp"

namespace lbm {

// One fluid-or-solid cell, one population per lane access: used for lattices
// whose width is not a multiple of 4.  OPEN: x is not periodic; populations
// entering at x = 0 come from the inlet ghost column, those entering at
// x = nx - 1 from the outlet ghost column (ghost: the member's [9][ny] block,
// +x movers from the inlet, -x movers from the outlet).
template <int MODEL, bool OPEN>
__device__ __forceinline__ void scalar_cell(const MemberDev& m, const float* __restrict__ src, float* __restrict__ dst,
                                            double* __restrict__ part, const float* __restrict__ ghost, int x, int y) {
    const int nx = m.nx, ny = m.ny;
    const long long plane = (long long)nx * ny;
    if (solid_at<OPEN>(m, x, y)) return;
    float dl[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        int xs = x - CX[i];
        if (!OPEN) xs = xs < 0 ? xs + nx : (xs >= nx ? xs - nx : xs);
        const int ys = y - CY[i];
        const bool wall = (ys < 0) | (ys >= ny);
        const bool inside = (unsigned)xs < (unsigned)nx;
        const bool bounce = wall || (inside && solid_at<OPEN>(m, xs, ys));
        if (bounce)
            dl[i] = src[(long long)OPP[i] * plane + (long long)y * nx + x];
        else if (OPEN && (xs < 0 || xs >= nx))
            dl[i] = ghost[(long long)i * ny + ys];
        else
            dl[i] = src[(long long)i * plane + (long long)ys * nx + xs];
    }
    const int ri = ring_index(m, x, y);
    const unsigned links = ri >= 0 ? square_links(m, x, y) : 0u;
    double drag;
    if (OPEN) {
        drag = collide_cell<MODEL, true>(at_column<MODEL>(m, x, true), dl, links, ri >= 0);
    } else {
        drag = collide_cell<MODEL, true>(m, dl, links, ri >= 0);
    }
    const long long cell = (long long)y * nx + x;
#pragma unroll
    for (int i = 0; i < 9; ++i) dst[(long long)i * plane + cell] = dl[i];
    if (ri >= 0) part[ri] = drag;
}

// One row segment of up to 256 cells per wave, four consecutive cells per
// lane, 16-byte loads and stores.  A population moving along +x (c_x = 1) is
// pulled from x - 1: the lane's aligned float4 supplies three of its four
// cells and the fourth comes from the neighbouring lane through a wave
// shift; the first lane of the wave takes it from one wave-uniform load,
// which also carries the periodic wrap at x = 0 (OPEN: the inlet ghost
// column).  Likewise for c_x = -1 at the right end (OPEN: the outlet ghost
// column).
// Rows next to a wall are wave-uniform (the whole row bounces back); only
// waves touching a solid cell decide per cell.  OPEN also sets the
// relaxation rates per cell (sponge zone).
template <int MODEL, bool OPEN>
__device__ __forceinline__ void vec_row(const MemberDev& m, const float* __restrict__ src, float* __restrict__ dst,
                                        double* __restrict__ part, const float* __restrict__ ghost, int base, int y,
                                        int lane) {
    const int nx = m.nx, ny = m.ny;
    const unsigned plane = (unsigned)nx * (unsigned)ny;
    const int nvalid = min(256, nx - base);  // a multiple of 4
    const int last = nvalid / 4 - 1;         // last lane holding cells
    const bool live = lane <= last;
    const int x0 = base + 4 * min(lane, last);
    const unsigned voff = 4u * (unsigned)x0;  // per-lane byte offset within a row
    const unsigned rowoff = (unsigned)y * (unsigned)nx;
    const bool left_end = base == 0, right_end = base + nvalid == nx;
    const int xl = (left_end ? nx : base) - 1;
    const int xr = right_end ? 0 : base + nvalid;
    const bool near_sq = m.ss > 0 && y >= m.sy0 - 1 && y <= m.sy0 + m.ss && base <= m.sx0 + m.ss &&
                         base + nvalid - 1 >= m.sx0 - 1;
    // which of the rows y - 1, y, y + 1 cross the grid's bars (wave-uniform)
    bool grow[3] = {false, false, false};
    if (OPEN) {
#pragma unroll
        for (int j = 0; j < 3; ++j) grow[j] = y - 1 + j >= 0 && y - 1 + j < ny && grid_row(m, y - 1 + j);
    }
    const bool near_grid = OPEN && (grow[0] || grow[1] || grow[2]) && base <= m.gx0 + m.bar &&
                           base + nvalid - 1 >= m.gx0 - 1;
    const bool near = near_sq || near_grid;
    // bit j: column x0 - 1 + j (j = 0..5, the lane's cells and their neighbours) holds grid bars
    unsigned gcols = 0;
    if (near_grid)
#pragma unroll
        for (int j = 0; j < 6; ++j) gcols |= ((unsigned)(x0 - 1 + j - m.gx0) < (unsigned)m.bar ? 1u : 0u) << j;
    // solid test of column x0 + dx (dx = -1 .. 4) in row y - 1 + j
    auto solid = [&](int dx, int j) {
        return (near_sq && in_square(m, x0 + dx, y - 1 + j)) || (OPEN && grow[j] && ((gcols >> (dx + 1)) & 1u));
    };
    // open channel: the columns of this segment reach the sponge zone (wave-uniform)
    const bool sponge_wave = OPEN && base + nvalid - 1 > m.sp_x0;
    // buffer resources over the member's whole block (range-checked by the hardware);
    // row offsets are wave-uniform (scalar), the lane offset is the only vector operand
    const unsigned bytes = 36u * plane;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)src, (short)0, (int)bytes, BUFFER_RSRC_WORD3);
    const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc((void*)dst, (short)0, (int)bytes, BUFFER_RSRC_WORD3);
    // load phase: nine 16-byte non-temporal loads and the edge elements, no
    // branches in between (row choice by wave-uniform selects), so all are in
    // flight at once
    f4 v[9];
    float e[9];
    bool wall[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const int ys = y - CY[i];
        wall[i] = ys < 0 || ys >= ny;  // the whole row takes its own opposite population
        const unsigned row = wall[i] ? (unsigned)OPP[i] * plane + rowoff : (unsigned)i * plane + (unsigned)ys * (unsigned)nx;
        v[i] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff, 4u * row, BUFFER_NT);
        // the edge element goes through the vector memory pipe like the rest
        // (every lane asks for the same word)
        if (CX[i] == 1) {
            if (OPEN && left_end) e[i] = ghost[(unsigned)i * (unsigned)ny + (unsigned)(wall[i] ? y : ys)];
            else e[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, 4u * (unsigned)xl, 4u * row, 0));
        } else if (CX[i] == -1) {
            if (OPEN && right_end) e[i] = ghost[(unsigned)i * (unsigned)ny + (unsigned)(wall[i] ? y : ys)];
            else e[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, 4u * (unsigned)xr, 4u * row, 0));
        } else {
            e[i] = 0.0f;
        }
    }
    // shift phase: +x movers take x - 1 from the left neighbour lane, -x movers x + 1 from the right
    f4 p[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        if (CX[i] == 1) {
            const float sh = wave_shr1(v[i].w);
            const f4 s4 = f4{lane == 0 ? e[i] : sh, v[i].x, v[i].y, v[i].z};
            p[i] = wall[i] ? v[i] : s4;
        } else if (CX[i] == -1) {
            const float sh = wave_shl1(v[i].x);
            const f4 s4 = f4{v[i].y, v[i].z, v[i].w, lane == last ? e[i] : sh};
            p[i] = wall[i] ? v[i] : s4;
        } else {
            p[i] = v[i];
        }
    }
    if (near) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (solid(k, 1)) continue;  // a solid cell's results are never stored
#pragma unroll
            for (int i = 1; i < 9; ++i) {
                const int ys = y - CY[i];
                if (ys < 0 || ys >= ny) continue;
                if (solid(k - CX[i], 1 - CY[i])) p[i][k] = src[(unsigned)OPP[i] * plane + rowoff + (unsigned)(x0 + k)];
            }
        }
    }
    // collide the four cells one after the other, in place
#pragma unroll 1
    for (int k = 0; k < 4; ++k) {
        float dl[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) dl[i] = p[i][k];
        const int ri = (near_sq && live && !in_square(m, x0 + k, y)) ? ring_index(m, x0 + k, y) : -1;
        const unsigned links = ri >= 0 ? square_links(m, x0 + k, y) : 0u;
        double drag;
        if (OPEN) {
            drag = collide_cell<MODEL, true>(at_column<MODEL>(m, x0 + k, sponge_wave), dl, links, near_sq);
        } else {
            drag = collide_cell<MODEL, true>(m, dl, links, near_sq);
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) p[i][k] = dl[i];
        if (ri >= 0) part[ri] = drag;
    }
    if (!live) return;
    // lanes whose four cells are all fluid store 16 bytes at a time, lanes
    // with only solid cells store nothing, and the rare mixed ones store cell
    // by cell, leaving the solid cells untouched
    unsigned smask = 0;  // bit k: cell x0 + k is solid
    if (near)
#pragma unroll
        for (int k = 0; k < 4; ++k) smask |= (solid(k, 1) ? 1u : 0u) << k;
    if (smask == 0) {
#pragma unroll
        for (int i = 0; i < 9; ++i)
            __builtin_amdgcn_raw_buffer_store_b128(p[i], rd, voff, 4u * ((unsigned)i * plane + rowoff), BUFFER_NT);
    } else if (smask != 0xFu) {
#pragma unroll 1
        for (int k = 0; k < 4; ++k) {
            if (solid(k, 1)) continue;
#pragma unroll
            for (int i = 0; i < 9; ++i) dst[(unsigned)i * plane + rowoff + (unsigned)(x0 + k)] = p[i][k];
        }
    }
}

// Fused pull-stream + collide step over the whole ensemble.  Workgroup =
// TYT waves; a tile is 256 columns by TYT*R rows; wave w handles rows
// w, w + TYT, ... of the tile.
// One-row shapes are held to 96 VGPRs (5 waves per SIMD): the memory-bound
// step needs the waves in flight more than the registers.  OPEN: the
// open-channel instantiation (inlet, grid, sponge, outlet ghost column).
template <int TYT, int R, int MODEL, bool OPEN>
__global__ __launch_bounds__(64 * TYT) __attribute__((amdgpu_waves_per_eu(R == 1 && MODEL == 0 && !OPEN ? 5 : 4))) void step_kernel(StepArgs a) {
    const int b = a.xcd ? xcd_remap((int)blockIdx.x, a.total_blocks) : (int)blockIdx.x;
    int tx, ty, vec, seg_rows;
    const int mi = block_to_member(a, b, tx, ty, vec, seg_rows);
    // the three bookkeeping reads are independent: issue them together
    const int on = a.active[mi];
    MemberDev m = a.members[mi];
    const int par = a.parity[mi] ^ a.flip;
    if (!on) return;
    // Few coefficients (bgk_guo), and three of them in vector registers: an instruction takes one scalar operand only,
    // and nine coefficients in scalar registers spill 34 of these (1 x 256 x 64, 64 launches: 441 -> 423 us; open
    // 16 x 512 x 128 1641 -> 1586).
    if constexpr (MODEL == 0 && !OPEN)
        for (double* c : {&m.q9, &m.qg, &m.keep}) __asm__ volatile("" : "+v"(*c));
    const float* __restrict__ src = (par ? a.pop1 : a.pop0) + m.off;
    float* __restrict__ dst = (par ? a.pop0 : a.pop1) + m.off;
    double* __restrict__ part = a.partial + m.part_off + (long long)a.slot * m.ring;
    const float* __restrict__ ghost = OPEN ? a.ghost + m.ghost_off : nullptr;
    const int lane = (int)(threadIdx.x & 63);
    // the wave index is uniform across the wave: say so, so that all row logic stays scalar
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int base = tx * 256;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = ty * (TYT * R) + r * TYT + wv;
        if (y >= m.ny) break;
        if (vec) {
            vec_row<MODEL, OPEN>(m, src, dst, part, ghost, base, y, lane);
        } else {
#pragma unroll 1
            for (int k = 0; k < 4; ++k) {
                const int x = base + 64 * k + lane;
                if (x < m.nx) scalar_cell<MODEL, OPEN>(m, src, dst, part, ghost, x, y);
            }
        }
    }
}

// Open channel boundaries (paper Section 2), rebuilt before every step into
// the member's [9][ny] ghost block: the +x movers (i = 1, 5, 8) of the inlet
// column x = -1, which the cells of column 0 pull, and the -x movers
// (i = 3, 6, 7) of the outlet column x = nx, which the cells of column nx - 1
// pull.  The inlet is the equilibrium of the parabolic profile (inlet_dev);
// the outlet is outlet_ghost_value of the post-collision state about to be
// streamed.
// One workgroup per member: each thread takes rows t, t + 256, ... and puts
// the velocities of the last two columns into LDS ([4][ny] doubles); after a
// barrier every thread rebuilds the ghost populations of its rows from its
// own and its neighbours' entries.
__global__ __launch_bounds__(256) void outlet_ghost_kernel(GhostArgs a) {
    const int mi = (int)blockIdx.x;
    const MemberDev m = a.members[mi];
    if (!m.open || !a.active[mi]) return;  // the whole workgroup
    extern __shared__ OutletVel vel[];      // [ny]
    const int par = a.parity[mi] ^ a.flip;
    const float* __restrict__ src = (par ? a.pop1 : a.pop0) + m.off;
    const int nx = m.nx, ny = m.ny;
    const unsigned plane = (unsigned)nx * (unsigned)ny;
    for (int y = (int)threadIdx.x; y < ny; y += 256) {
        float d1[9], d2[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const unsigned row = (unsigned)i * plane + (unsigned)y * (unsigned)nx;
            d1[i] = src[row + (unsigned)(nx - 1)];
            d2[i] = src[row + (unsigned)(nx - 2)];
        }
        OutletVel v;
        stored_velocity(d1, v.ux1, v.uy1);
        stored_velocity(d2, v.ux2, v.uy2);
        vel[y] = v;
    }
    __syncthreads();
    float* __restrict__ g = a.ghost + m.ghost_off;
    for (int y = (int)threadIdx.x; y < ny; y += 256) {
        const OutletVel va = vel[y > 0 ? y - 1 : 0], v0 = vel[y], vb = vel[y + 1 < ny ? y + 1 : ny - 1];
        double rho_g = 1.0;
        if (m.out_rho) {  // the row's two cells again (the LDS table keeps velocities only)
            float d1[9], d2[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const unsigned row = (unsigned)i * plane + (unsigned)y * (unsigned)nx;
                d1[i] = src[row + (unsigned)(nx - 1)];
                d2[i] = src[row + (unsigned)(nx - 2)];
            }
            rho_g = outlet_density(m, d1, d2);
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            if (CX[i] == 1) g[i * ny + y] = inlet_dev(m, i, y);
            else if (CX[i] == -1) g[i * ny + y] = outlet_ghost_value(m, CX[i], CY[i], WD[i], y, va, v0, vb, rho_g);
        }
    }
}

// Step 0: equilibrium with the seeded density and a uniform velocity
// (u_x0, 0) (at rest for u_x0 = 0; an open channel's inlet profile
// (u_in(y), 0) instead), relaxed once.
__global__ __launch_bounds__(256) void init_kernel(InitArgs a) {
    const int mi = (int)blockIdx.y;
    const MemberDev m = a.members[mi];
    const long long plane = (long long)m.nx * m.ny;
    const long long cell = (long long)blockIdx.x * 256 + threadIdx.x;
    if (cell >= plane) return;
    const int y = (int)(cell / m.nx), x = (int)(cell - (long long)y * m.nx);
    if (in_solid(m, x, y)) return;
    double drho = 0.0;
    if (a.noise_amp != 0.0) {
        const U64x4 w = philox4x64_10((uint64_t)cell, (uint64_t)mi, 0, 0, a.seed, PURPOSE_INIT);
        drho = a.noise_amp * (2.0 * uniform53(w.v[0]) - 1.0);
    }
    // f_i = f_i^eq(rho, u0) - w_i = w_i [drho + rho (3 c.u + 4.5 (c.u)^2 - 1.5 u^2)]
    double u0 = a.ux0;
    if (m.open) {
        const double yc = (double)y + 0.5;
        u0 = 4.0 * m.u_c * yc * ((double)m.ny - yc) / ((double)m.ny * (double)m.ny);
    }
    const double rho = 1.0 + drho;
    float d[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const double cu = (double)CX[i] * u0;
        d[i] = (float)(WD[i] * (drho + rho * (3.0 * cu + 4.5 * cu * cu - 1.5 * u0 * u0)));
    }
    const int ri = ring_index(m, x, y);
    MemberDev mc = m;
    if (m.open) {
        sponge_at(mc, x);
        bgk_coefficients(mc);
    }
    const double drag = collide_member(mc, d, ri >= 0 ? square_links(m, x, y) : 0u);
    float* dst = a.pop0 + m.off;  // step 0 lives in buffer 0 (parity 0)
#pragma unroll
    for (int i = 0; i < 9; ++i) dst[(long long)i * plane + cell] = d[i];
    if (ri >= 0) a.partial[m.part_off + ri] = drag;
}

// The velocities of the last two columns of row y.
__device__ __forceinline__ OutletVel outlet_velocities(const MemberDev& m, const float* __restrict__ src, int y, float d1[9], float d2[9]) {
    const unsigned plane = (unsigned)m.nx * (unsigned)m.ny;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        const unsigned row = (unsigned)i * plane + (unsigned)y * (unsigned)m.nx;
        d1[i] = src[row + (unsigned)(m.nx - 1)];
        d2[i] = src[row + (unsigned)(m.nx - 2)];
    }
    OutletVel v;
    stored_velocity(d1, v.ux1, v.uy1);
    stored_velocity(d2, v.ux2, v.uy2);
    return v;
}

// Rows y0 .. y1 - 1 of one step of a member, cell by cell.
template <bool OPEN>
__device__ __forceinline__ void redo_rows(const MemberDev& m, const float* src, float* dst, double* part, float* g, int y0, int y1) {
    if (OPEN) {  // the ghost columns that the rows pull first (every row's neighbours anew: no table of rows)
        for (int y = max(y0 - 1, 0) + (int)threadIdx.x; y < min(y1 + 1, m.ny); y += (int)blockDim.x) {
            float d1[9], d2[9];
            const OutletVel va = outlet_velocities(m, src, y > 0 ? y - 1 : 0, d1, d2);
            const OutletVel vb = outlet_velocities(m, src, y + 1 < m.ny ? y + 1 : m.ny - 1, d1, d2);
            const OutletVel v0 = outlet_velocities(m, src, y, d1, d2);
            const double rho_g = outlet_density(m, d1, d2);
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                if (CX[i] == 1) g[i * m.ny + y] = inlet_dev(m, i, y);
                else if (CX[i] == -1) g[i * m.ny + y] = outlet_ghost_value(m, CX[i], CY[i], WD[i], y, va, v0, vb, rho_g);
            }
        }
        __syncthreads();
    }
    for (int c = y0 * m.nx + (int)threadIdx.x; c < y1 * m.nx; c += (int)blockDim.x) {
        const int y = c / m.nx, x = c - y * m.nx;
        if (m.model == 2) scalar_cell<2, OPEN>(m, src, dst, part, g, x, y);
        else if (m.model == 1) scalar_cell<1, OPEN>(m, src, dst, part, g, x, y);
        else scalar_cell<0, OPEN>(m, src, dst, part, g, x, y);
    }
}

// Resident chunks that were given up (lbm_resident.hip), stepped again from the
// source buffers, which the resident kernel only read; the last step's state
// ends in the other buffer.
//
// A step of a member is cut into bands of rows (four at least).  The tasks
// (step, member, band) are taken in this order from a counter by whichever
// blocks run, and a task waits for the step before of its own band and of those
// beside it: all that its rows pull, the outlet's rows two further on included,
// and all that still pulls what it overwrites.  Those were taken earlier, by
// blocks that run, so the earliest unfinished task never waits and every wait
// ends, however few blocks the device holds at a time.  Bands beside each other
// are at most one step apart: a ghost row that both form is formed for the same
// step, to the same values.
__device__ __forceinline__ void resident_redo(const FinalizeArgs& a, const RedoArgs& r) {
    __shared__ int taken;
    const int t0 = (int)threadIdx.x;
    const int per = r.slots * r.bands, base = r.launch * REDO_STEPS;
    const int steps = a.n + (a.n % 2 == 0 ? 1 : 0);  // an even number of steps ends in the source buffer: then a copy
    auto seen = [&](int at) { return __hip_atomic_load(r.done + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    if (blockIdx.x == 0 && t0 == 0 && !r.states_only) *r.gave_up_host = 1;
    // The last task's end and the next one's taking are one block of thread 0's between two barriers: with such a
    // block at either end of the loop the compiler joins them across it, and the other lanes of the wave meet the
    // barriers without lane 0.
    int ended = -1, made = 0;
#pragma unroll 1
    for (;;) {
        __syncthreads();  // (the last task's rows are written, and its number read by all)
        if (t0 == 0) {
            if (ended >= 0) __hip_atomic_store(r.done + ended, made, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            taken = atomicAdd(r.ticket, 1);
        }
        __syncthreads();
        const int k = __builtin_amdgcn_readfirstlane(taken);
        ended = -1;
        if (k >= per * steps) break;
        const int t = k / per, slot = (k - t * per) / r.bands, band = k - t * per - slot * r.bands;
        const int mi = __builtin_amdgcn_readfirstlane(r.active_list ? r.active_list[slot] : slot);
        if (!a.active[mi] || r.given_up[mi] != r.launch) continue;
        const MemberDev m = a.members[mi];
        const int high = max((m.ny + r.bands - 1) / r.bands, 4), y0 = band * high, y1 = min(y0 + high, m.ny);
        if (y0 >= m.ny) continue;
        const int at = slot * r.bands + band;
        if (t > 0) {
            if (t0 < 3 && (t0 > 0 || band > 0) && (t0 < 2 || y1 < m.ny))
                while (seen(at - 1 + t0) < base + t) __builtin_amdgcn_s_sleep(2);
            __syncthreads();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        const int par = a.parity[mi] ^ r.flip;
        float* const from = (par ? r.pop1 : r.pop0) + m.off;
        float* const to = (par ? r.pop0 : r.pop1) + m.off;
        const float* const src = t & 1 ? to : from;
        float* const dst = t & 1 ? from : to;
        if (t < a.n) {
            double* const part = r.partial + m.part_off + (long long)t * m.ring;
            if (m.open) redo_rows<true>(m, src, dst, part, r.ghost + m.ghost_off, y0, y1);
            else redo_rows<false>(m, src, dst, part, nullptr, y0, y1);
        } else {
            const int cells = m.nx * m.ny;
            for (int c = y0 * m.nx + t0; c < y1 * m.nx; c += (int)blockDim.x) {
                const int y = c / m.nx, x = c - y * m.nx;
                if (in_solid(m, x, y)) continue;
                for (int i = 0; i < 9; ++i) dst[(long long)i * cells + c] = src[(long long)i * cells + c];
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        ended = at;
        made = base + t + 1;
    }
    if (t0 == 0 && atomicAdd(r.ticket + 1, 1) == (int)gridDim.x - 1) {  // no block takes a task any more
        r.ticket[0] = 0;
        r.ticket[1] = 0;
    }
    // this block's own member, wherever its bands were made
    const int slot = (int)blockIdx.x;
    if (slot < r.slots) {
        const int mi = r.active_list ? r.active_list[slot] : slot;
        if (a.active[mi] && r.given_up[mi] == r.launch) {
            const int ny = a.members[mi].ny, high = max((ny + r.bands - 1) / r.bands, 4);
            for (int band = t0; band * high < ny; band += (int)blockDim.x)
                while (seen(slot * r.bands + band) < base + steps) __builtin_amdgcn_s_sleep(2);
        }
    }
    __syncthreads();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// Reduce the drag partials of a chunk of n steps for one member per block:
// f_d(s) = sum of ring partials in ring order (FP64), written to the series at
// the member's cursor; then, in step order, accum += (f_d - mu)/sigma * dt.
// The member's parity flips n times (not for step 0, which init wrote in
// place) and its cursor advances by n.
__device__ __forceinline__ void finalize_member(const FinalizeArgs& a, int mi) {
    const int s = (int)threadIdx.x;
    const bool on = a.active[mi];
    const MemberDev m = a.members[mi];
    __shared__ double fd[256];
    if (!on) return;
    const int cur = a.cursor[mi];
    if (s < a.n) {
        double acc = 0.0;
        const double* p = a.partial + m.part_off + (long long)s * m.ring;
#pragma unroll 16
        for (int r = 0; r < m.ring; ++r) acc += p[r];  // loads in flight, sums in order
        fd[s] = acc;
        a.series[(long long)mi * a.ld + cur + s] = (float)acc;
    }
    __syncthreads();
    if (s == 0) {
        bool bad = false;
        if (a.accumulate) {
            double tot = a.accum[mi];
            for (int t = 0; t < a.n; ++t) {
                tot += (fd[t] - a.mu) * a.inv_sigma_dt;
                bad |= !isfinite(fd[t]);
            }
            a.accum[mi] = tot;
        } else {
            for (int t = 0; t < a.n; ++t) bad |= !isfinite(fd[t]);
        }
        if (bad) a.flags[mi] = 1;
        a.parity[mi] ^= a.swap_parity;
        a.cursor[mi] = cur + a.n;
    }
}

__global__ __launch_bounds__(256) void finalize_kernel(FinalizeArgs a) { finalize_member(a, (int)blockIdx.x); }

__global__ __launch_bounds__(256) void finalize_resident_kernel(FinalizeArgs a, RedoArgs r) {
    if (r.given_up[r.n_members] == r.launch) resident_redo(a, r);
    const int slot = (int)blockIdx.x;
    if (r.states_only || slot >= r.slots) return;
    finalize_member(a, r.active_list ? r.active_list[slot] : slot);
}

// ---------------------------------------------------------------------------
// launchers

template <int TYT, int R>
static hipError_t launch_step_t(const StepArgs& a, int model, hipStream_t st) {
    const dim3 grid(a.total_blocks), block(64 * TYT);
    if (a.ghost) {
        if (model == 2) hipLaunchKernelGGL((step_kernel<TYT, R, 2, true>), grid, block, 0, st, a);
        else if (model == 1) hipLaunchKernelGGL((step_kernel<TYT, R, 1, true>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((step_kernel<TYT, R, 0, true>), grid, block, 0, st, a);
    } else {
        if (model == 2) hipLaunchKernelGGL((step_kernel<TYT, R, 2, false>), grid, block, 0, st, a);
        else if (model == 1) hipLaunchKernelGGL((step_kernel<TYT, R, 1, false>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((step_kernel<TYT, R, 0, false>), grid, block, 0, st, a);
    }
    return hipGetLastError();
}

// Table of step-kernel launch shapes: TYT waves per workgroup, R rows per
// wave, whether workgroups are remapped so each XCD gets contiguous tiles,
// and steps per launch.  Ids 0-15 are one-step shapes (launch_step switches
// on id % 8); ids 16-19 are the two-step kernel with TYT rows per iteration;
// ids 21-23 are shape 16 with shorter strips, and id 20 takes the resident kernel (a chunk of steps
// per launch), the sweep kernel (up to four), shape 16 or shape 0, by estimated times of the active members.
const TileShape TILE_SHAPES[] = {
    {4, 1, 1, 1, 0}, {4, 2, 1, 1, 0}, {8, 1, 1, 1, 0}, {2, 2, 1, 1, 0},
    {16, 1, 1, 1, 0}, {1, 4, 1, 1, 0}, {4, 4, 1, 1, 0}, {8, 2, 1, 1, 0},
    {4, 1, 0, 1, 0}, {4, 2, 0, 1, 0}, {8, 1, 0, 1, 0}, {2, 2, 0, 1, 0},
    {16, 1, 0, 1, 0}, {1, 4, 0, 1, 0}, {4, 4, 0, 1, 0}, {8, 2, 0, 1, 0},
    {4, 1, 1, 2, 0}, {2, 1, 1, 2, 0}, {8, 1, 1, 2, 0}, {4, 1, 0, 2, 0},
    {4, 1, 1, 2, 1, -1}, {4, 1, 1, 2, 0, 128}, {4, 1, 1, 2, 0, 64}, {4, 1, 1, 2, 0, 32},
};
const int N_TILE_SHAPES = (int)(sizeof(TILE_SHAPES) / sizeof(TILE_SHAPES[0]));

hipError_t launch_step(int tile_id, const StepArgs& a, int model, hipStream_t st) {
    switch (tile_id % 8) {
        case 0: return launch_step_t<4, 1>(a, model, st);
        case 1: return launch_step_t<4, 2>(a, model, st);
        case 2: return launch_step_t<8, 1>(a, model, st);
        case 3: return launch_step_t<2, 2>(a, model, st);
        case 4: return launch_step_t<16, 1>(a, model, st);
        case 5: return launch_step_t<1, 4>(a, model, st);
        case 6: return launch_step_t<4, 4>(a, model, st);
        case 7: return launch_step_t<8, 2>(a, model, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_outlet_ghost(const GhostArgs& a, int n_members, int max_ny, hipStream_t st) {
    hipLaunchKernelGGL(outlet_ghost_kernel, dim3(n_members), dim3(256), sizeof(double) * 4 * max_ny, st, a);
    return hipGetLastError();
}

hipError_t launch_init(const InitArgs& a, int n_members, long long max_cells, hipStream_t st) {
    const unsigned gx = (unsigned)((max_cells + 255) / 256);
    hipLaunchKernelGGL(init_kernel, dim3(gx, n_members), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_finalize(const FinalizeArgs& a, int n_members, hipStream_t st) {
    hipLaunchKernelGGL(finalize_kernel, dim3(n_members), dim3(256), 0, st, a);
    return hipGetLastError();
}

// (blocks beyond the members' have nothing to do unless a chunk is stepped again)
hipError_t launch_finalize_resident(const FinalizeArgs& a, const RedoArgs& r, hipStream_t st) {
    hipLaunchKernelGGL(finalize_resident_kernel, dim3(max(r.slots, min(r.slots * r.bands, 256))), dim3(256), 0, st, a, r);
    return hipGetLastError();
}

}  // namespace lbm
