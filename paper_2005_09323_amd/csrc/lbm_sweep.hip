// Several lattice steps per pass over the populations (temporal blocking of
// the fused pull-stream + collide step of paper Appendix A), with the steps
// in between held in registers.
//
// The waves of a unit span one member's whole width, C neighbouring cells per
// lane, and sweep a range of its rows from the bottom up, one row per
// iteration.  Stage 1 of an iteration pulls row y of the state at t from
// memory and collides it (step t+1); stage 2 collides row y - 1 at step t+2,
// ..., stage T row y - T + 1 at step t+T, which is written to the other
// buffer.  A lane's cells never move: what stage b + 1 pulls from stage b
// differs from the lane's own results by one row (a delay of one or two
// iterations, kept in registers: 9 C floats per stage boundary) and one
// column (a shift by one cell: C - 1 of the C values are the lane's own, one
// comes from the lane beside it, and at the ends of a wave from the
// neighbouring wave through LDS, one 3-value exchange per side and stage).
// So the populations cross memory once per T steps and nothing else of them
// is written anywhere.
//
// Rows ya .. yb - 1 are the unit's to write; stage b also collides the T - b
// rows on either side that the later stages pull from, which the neighbouring
// units collide too, bit for bit the same (the arithmetic of every cell is
// collide_cell's on FP32 inputs, as in the one-step kernel).
//
// Halfway bounce-back between the stages is done where the values are
// produced: a population that leaves row r towards a solid cell or a wall
// comes back to its own cell reversed, so it replaces what the solid cell
// would have sent there.  Towards a solid cell in the same row or the row
// below, the lane overwrites its own delayed values; towards the row above,
// the solid cell itself, when its row is produced, sends back what arrived
// at it (its delayed values), and a wall above the last row is one more
// produced row of solid cells.
//
// What bounds it: the FP64 units.  128 x 1024 x 256, 64 BGK steps: 15.9 ms with
// the two-step kernel (32 passes over 2.4 GB of HBM at 4.85 TB/s, 94 % of a
// device copy), 10.0 ms here (16 passes, 3.9 TB/s); an iteration of the four
// stages takes 4.4 us with two waves per SIMD, and its 890 instructions (656
// of them FP64, which issue at 5.2 cycles of 2.4 GHz each) account for 4.0.
// Two cells per lane and four stages: 243 registers, the most that two waves
// per SIMD can hold; four cells per lane spill 172 and take 21.7 ms, three
// stages take 11.8 ms, two 16.1.  Shorter row ranges collide more rows twice
// (64 rows instead of 128: 10.8 ms).
#include "lbm_device.hpp"

#include <type_traits>

namespace lbm {

static_assert(SWEEP_CELLS == 2, "cells are stored in pairs");
__device__ __forceinline__ void store_cells(__amdgpu_buffer_rsrc_t rd, unsigned voff, unsigned soff, const float v[SWEEP_CELLS]) {
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(u2{__float_as_uint(v[0]), __float_as_uint(v[1])}, rd, voff, soff, BUFFER_NT);
}

// FULL: a width that is a multiple of 64 SWEEP_CELLS (every lane has its cells); else any (lanes beyond
// the width, and the row's last lane may have fewer cells).
// An iteration has two forms: `plain` while no row of the wave touches a wall
// or the square, and `special` with all the tests otherwise (registers and scalars of the tests would
// otherwise be live through every row: 68 scalar spills and their reloads).
template <int T, int MODEL, bool FULL>
__global__ __launch_bounds__(64 * SWEEP_WAVES) __attribute__((amdgpu_waves_per_eu(2))) void sweep_kernel(SweepArgs a) {
    constexpr int C = SWEEP_CELLS;
    // [parity][boundary][wave][side]: side 0 the wave's first cell (3, 6, 7), side 1 its last (1, 5, 8)
    __shared__ f4 edge[2][T > 1 ? T - 1 : 1][SWEEP_WAVES][2];
    const int b = xcd_remap((int)blockIdx.x, a.total_blocks);
    int s = 0;
#pragma unroll 1
    while (s + 1 < a.nseg && b >= a.seg[s + 1].block_begin) ++s;
    const SweepSegment sg = a.seg[s];
    const int lane = (int)(threadIdx.x & 63);
    const int wg_wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int W = sg.waves;
    const int slot = wg_wave / W, w = wg_wave - slot * W;  // unit of the workgroup, wave of the unit
    const int unit = (b - sg.block_begin) * sg.units_per_block + slot;
    // every wave of a unit leaves here or none does (a barrier waits for the waves that remain)
    if (slot >= sg.units_per_block || unit >= sg.units) return;
    const int mloc = unit / sg.ranges;
    const int range = unit - mloc * sg.ranges;
    const int mi = a.active_list ? a.active_list[mloc] : sg.member_begin + mloc;
    const int on = a.active[mi];
    MemberDev m = a.members[mi];
    const int par = a.parity[mi] ^ a.flip;
    if (!on) return;
    // the update's coefficients in vector registers: an instruction takes one scalar operand only
    if constexpr (MODEL == 0)
        for (double* c : {&m.keep, &m.a45, &m.a3, &m.a9, &m.ag, &m.q45, &m.q3, &m.q9, &m.qg}) __asm__ volatile("" : "+v"(*c));
    const float* __restrict__ src = (par ? a.pop1 : a.pop0) + m.off;
    float* __restrict__ dst = (par ? a.pop0 : a.pop1) + m.off;
    double* const part = a.partial + m.part_off + (long long)a.slot * m.ring;
    const int nx = m.nx, ny = m.ny;
    const unsigned plane = (unsigned)nx * (unsigned)ny;
    const unsigned bytes = 36u * plane;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)src, (short)0, (int)bytes, BUFFER_RSRC_WORD3);
    const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc((void*)dst, (short)0, (int)bytes, BUFFER_RSRC_WORD3);
    const int base = w * sg.lanes * C;               // the wave's first column
    const int x0 = base + C * lane;                  // the lane's first column
    const bool last_wave = w == W - 1;
    // the wave's last lane with cells, and how many of its cells exist
    const int lastl = FULL ? 63 : last_wave ? (nx - base + C - 1) / C - 1 : sg.lanes - 1;
    const int rem = !FULL && last_wave ? nx - base - C * lastl : C;
    // A wave of fewer than 64 lanes works out some columns of the next wave too, the last of them wrongly (nothing
    // enters beside lane 63; one column more with each stage): its surplus lanes write no cell and no drag.
    const bool owns = FULL || lane <= lastl;
    // a short last lane loads the row's last C cells and moves them down
    const unsigned voff = 4u * (unsigned)min(x0, nx - C);
    const unsigned vl = 4u * (unsigned)((w == 0 ? nx : base) - 1);     // the column left of the wave (periodic)
    const unsigned vr = 4u * (unsigned)(last_wave ? 0 : base + sg.lanes * C);  // the column right of it
    // stores of the lanes beyond the row go beyond the buffer, which the hardware drops
    const unsigned vstore = !owns || (!FULL && lane == lastl && rem != C) ? 0x80000000u : voff;
    const bool sq_cols = m.ss > 0 && base <= m.sx0 + m.ss && base + sg.lanes * C - 1 >= m.sx0 - 1;
    unsigned sqc = 0;                                // bit j: column x0 - 1 + j crosses the square
    if (sq_cols)
#pragma unroll
        for (int j = 0; j < C + 2; ++j) sqc |= ((unsigned)(x0 - 1 + j - m.sx0) < (unsigned)m.ss ? 1u : 0u) << j;
    const int ya = range * sg.rows, yb = min(ya + sg.rows, ny);
    const int y0 = max(ya - (T - 1), 0);
    const int y1 = min(yb + (T - 1), ny);            // stage 1's rows: [y0, y1)
    const int yend = yb + T - 1;                     // stage T writes row yb - 1 in iteration yend - 1
    // plain iterations: y in [p0, p1) but not in [q0, q1)
    //  no wall: stage 1 and stage T - 1 in rows above 0, stage 1's row and the next one (load_own) below ny - 1
    //  no stage in a row beside or in the square, nor stage 1 in the row before
    // (a stage outside its row range computes values that nothing reads)
    const int p0 = y0 == 0 ? (T > 1 ? T - 1 : 1) : y0, p1 = min(yend, ny - 2);
    const int q0 = sq_cols ? m.sy0 - 2 : 0, q1 = sq_cols ? m.sy0 + m.ss + T : 0;
    // the neighbouring waves' edge slots
    const int wl = wg_wave + (w == 0 ? W - 1 : -1), wr = wg_wave + (last_wave ? 1 - W : 1);

    float cur[9][C], e[9], own[6][C];
    auto load_row = [&](int y) {
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            // (rows beyond a wall: any row, its values are replaced)
            const int ys = CY[i] == 0 ? y : CY[i] == 1 ? max(y - 1, 0) : min(y + 1, ny - 1);
            const unsigned row = 4u * ((unsigned)i * plane + (unsigned)ys * (unsigned)nx);
            load_cells<C>(rs, voff, row, cur[i]);
            if (CX[i] != 0) e[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, CX[i] == 1 ? vl : vr, row, 0));
        }
    };
    // the row's own populations that leave it up (2, 5, 6) and down (4, 7, 8), for its bounce-back:
    // needed where the row touches a wall or the square, loaded with the row before
    auto load_own = [&](int y) {
        constexpr int UD[6] = {2, 5, 6, 4, 7, 8};
#pragma unroll
        for (int i = 0; i < 6; ++i) load_cells<C>(rs, voff, 4u * ((unsigned)UD[i] * plane + (unsigned)y * (unsigned)nx), own[i]);
    };
    // cells of a short last lane: those loaded are the row's last C, move them to its first places
    auto settle = [&](float v[C]) {
        if constexpr (!FULL)
#pragma unroll
            for (int sh = 1; sh < C; ++sh)
#pragma unroll
                for (int k = 0; k + sh < C; ++k) v[k] = lane == lastl && C - rem == sh ? v[k + sh] : v[k];
    };
    // one cell to the right (+x movers) or left (-x movers); `in` enters at the row end of the wave
    auto shift_right = [&](float v[C], float in) {
        const float sh = wave_shr1_in(v[C - 1], in);
#pragma unroll
        for (int k = C - 1; k > 0; --k) v[k] = v[k - 1];
        v[0] = sh;
    };
    auto shift_left = [&](float v[C], float in) {
        const float sh = wave_shl1_in(v[0], in);
#pragma unroll
        for (int k = 0; k + 1 < C; ++k) v[k] = !FULL && lane == lastl && rem == k + 1 ? in : v[k + 1];
        v[C - 1] = FULL ? sh : (lane == lastl ? in : sh);
    };
    auto last_cell = [&](const float v[C]) {
        float r = v[C - 1];
        if constexpr (!FULL)
#pragma unroll
            for (int k = 1; k < C; ++k) r = rem == k ? v[k - 1] : r;
        return r;
    };
    // what stage b + 1 pulls from stage b: populations moving up that wait for the next row (A) and the
    // one before (O), those moving along the row (M)
    constexpr int NB = T > 1 ? T - 1 : 1;
    float A[NB][3][C], O[NB][3][C], M[NB][3][C];
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < C; ++k) A[q][i][k] = O[q][i][k] = M[q][i][k] = 0.0f;

    auto iteration = [&](int y, auto special_form) {
        constexpr bool SP = decltype(special_form)::value;
        auto solid_row = [&](int r) { return sq_cols && (unsigned)(r - m.sy0) < (unsigned)m.ss; };
        float p[9][C];
        // stage 1 pulls row y: the +-x movers one cell over, bounce-back next to solid cells
#pragma unroll
        for (int i = 0; i < 9; ++i) settle(cur[i]);
        if constexpr (SP) {
            const bool near = y == 0 || y >= ny - 1 || solid_row(y - 1) || solid_row(y) || solid_row(y + 1);
            float back[9][C];  // what bounces back into each direction: the row's own opposite population
            if (near) {
                constexpr int AT[9] = {0, 0, 3, 0, 0, 4, 5, 1, 2};  // own[] of the opposite of 2, 4, 5, 6, 7, 8
#pragma unroll
                for (int i = 0; i < 6; ++i) settle(own[i]);
#pragma unroll
                for (int i = 1; i < 9; ++i)
#pragma unroll
                    for (int k = 0; k < C; ++k) back[i][k] = CY[i] == 0 ? cur[OPP[i]][k] : own[AT[i]][k];
            }
#pragma unroll
            for (int i = 0; i < 9; ++i) {
#pragma unroll
                for (int k = 0; k < C; ++k) p[i][k] = cur[i][k];
                if (CX[i] == 1) shift_right(p[i], e[i]);
                else if (CX[i] == -1) shift_left(p[i], e[i]);
            }
            if (near) {
#pragma unroll
                for (int i = 1; i < 9; ++i) {
                    const int ys = y - CY[i];
                    // bit k: the cell pulled from is solid, or beyond a wall
                    const unsigned mk = ys < 0 || ys >= ny ? ~0u : solid_row(ys) ? sqc >> (1 - CX[i]) : 0u;
#pragma unroll
                    for (int k = 0; k < C; ++k) p[i][k] = (mk >> k) & 1u ? back[i][k] : p[i][k];
                }
            }
            load_own(min(y + 1, y1 - 1));
        } else {
#pragma unroll
            for (int i = 0; i < 9; ++i) {
#pragma unroll
                for (int k = 0; k < C; ++k) p[i][k] = cur[i][k];
                if (CX[i] == 1) shift_right(p[i], e[i]);
                else if (CX[i] == -1) shift_left(p[i], e[i]);
            }
        }
        // the next row, in flight until the next iteration (on every path, so that the compiler can
        // count the loads and waits for nothing else)
        load_row(min(y + 1, y1 - 1));
#pragma unroll
        for (int st = 1; st <= T; ++st) {
            const int r = y - (st - 1);  // the stage's row
            const bool real = !SP || (r >= max(ya - (T - st), 0) && r < min(yb + (T - st), ny));
            if constexpr (SP) {
                if (real) {
                    const bool ring_row = sq_cols && r >= m.sy0 - 1 && r <= m.sy0 + m.ss;
                    double* const ps = part + (long long)(st - 1) * m.ring;
#pragma unroll
                    for (int k = 0; k < C; ++k) {
                        float dl[9];
#pragma unroll
                        for (int i = 0; i < 9; ++i) dl[i] = pinned(p[i][k]);
                        const int ri = ring_row && owns && !in_square(m, x0 + k, r) ? ring_index(m, x0 + k, r) : -1;
                        const unsigned links = ri >= 0 ? square_links(m, x0 + k, r) : 0u;
                        const double drag = collide_cell<MODEL>(m, dl, links, ring_row);
#pragma unroll
                        for (int i = 0; i < 9; ++i) p[i][k] = pinned(dl[i]);
                        if (ri >= 0) ps[ri] = drag;
                    }
                }
            } else {
#pragma unroll
                for (int k = 0; k < C; ++k) {
                    float dl[9];
#pragma unroll
                    for (int i = 0; i < 9; ++i) dl[i] = pinned(p[i][k]);
                    collide_cell<MODEL>(m, dl, 0u, false);
#pragma unroll
                    for (int i = 0; i < 9; ++i) p[i][k] = pinned(dl[i]);
                }
            }
            if (st == T) {
                const bool mine = SP ? real : r >= ya && r < yb;
                const unsigned rowoff = (unsigned)(mine ? r : ya) * (unsigned)nx;
                // stores that must not happen get an offset beyond the buffer too: they are issued on
                // every path, so that the compiler can count them behind the prefetch
                const unsigned vs = mine ? vstore : 0x80000000u;
                if constexpr (SP) {
                    // lanes with a solid cell store cell by cell, the others all C at once
                    const unsigned skip = solid_row(r) ? (sqc >> 1) & ((1u << C) - 1u) : 0u;
                    const unsigned so = skip == 0u ? vs : 0x80000000u;
#pragma unroll
                    for (int i = 0; i < 9; ++i) store_cells(rd, so, 4u * ((unsigned)i * plane + rowoff), p[i]);
                    if (mine && owns && skip != 0u && skip != (1u << C) - 1u) {
#pragma unroll
                        for (int k = 0; k < C; ++k)
                            if (!((skip >> k) & 1u) && x0 + k < nx) {
#pragma unroll
                                for (int i = 0; i < 9; ++i) dst[(unsigned)i * plane + rowoff + (unsigned)(x0 + k)] = p[i][k];
                            }
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 9; ++i) store_cells(rd, vs, 4u * ((unsigned)i * plane + rowoff), p[i]);
                }
                if constexpr (!FULL) {  // the short last lane (never next to the square: a fluid column is between)
#pragma unroll
                    for (int k = 0; k < C - 1; ++k) {
                        const unsigned so = mine && lane == lastl && rem != C && k < rem ? 4u * (unsigned)(x0 + k) : 0x80000000u;
#pragma unroll
                        for (int i = 0; i < 9; ++i)
                            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(p[i][k]), rd, so, 4u * ((unsigned)i * plane + rowoff), 0);
                    }
                }
            } else {
                const int q = st - 1 < NB ? st - 1 : 0;
                const bool near = SP && (solid_row(r) || solid_row(r - 1));
                if constexpr (SP) {
                    if (r == ny) {  // the wall above the last row sends back what arrived at it
#pragma unroll
                        for (int k = 0; k < C; ++k) {
                            p[4][k] = A[q][0][k];
                            p[7][k] = A[q][1][k];
                            p[8][k] = A[q][2][k];
                        }
                    }
                    if (near) {
                        const unsigned here = solid_row(r) ? sqc : 0u, below = solid_row(r - 1) ? sqc : 0u;
#pragma unroll
                        for (int k = 0; k < C; ++k) {
                            // solid cells of this row send back what came up to them
                            const bool in = (here >> (k + 1)) & 1u;
                            p[4][k] = in ? A[q][0][k] : p[4][k];
                            p[7][k] = in ? A[q][1][k] : p[7][k];
                            p[8][k] = in ? A[q][2][k] : p[8][k];
                            // towards solid cells in the row below: back up in this row
                            A[q][0][k] = (below >> (k + 1)) & 1u ? p[4][k] : A[q][0][k];
                            A[q][1][k] = (below >> k) & 1u ? p[7][k] : A[q][1][k];
                            A[q][2][k] = (below >> (k + 2)) & 1u ? p[8][k] : A[q][2][k];
                        }
                    }
                    if (r == 0) {  // the wall below the first row
#pragma unroll
                        for (int k = 0; k < C; ++k) {
                            A[q][0][k] = p[4][k];
                            A[q][1][k] = p[7][k];
                            A[q][2][k] = p[8][k];
                        }
                    }
                }
                f4* const ed = &edge[y & 1][q][0][0];
                if (lane == 0) ed[2 * wg_wave] = f4{p[3][0], p[6][0], p[7][0], 0.0f};
                if (lane == lastl) ed[2 * wg_wave + 1] = f4{last_cell(p[1]), last_cell(p[5]), last_cell(p[8]), 0.0f};
                if (W > 1) lds_barrier();
                else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
                const f4 el = ed[2 * wl + 1], er = ed[2 * wr];
                float n1[C], n3[C], n5[C], n6[C], n7[C], n8[C];
#pragma unroll
                for (int k = 0; k < C; ++k) {
                    n1[k] = p[1][k];
                    n3[k] = p[3][k];
                    n5[k] = p[5][k];
                    n6[k] = p[6][k];
                    n7[k] = p[7][k];
                    n8[k] = p[8][k];
                }
                shift_right(n1, el.x);
                shift_right(n5, el.y);
                shift_right(n8, el.z);
                shift_left(n3, er.x);
                shift_left(n6, er.y);
                shift_left(n7, er.z);
                if (SP && near) {  // towards solid cells beside: back the other way
                    const unsigned here = solid_row(r) ? sqc : 0u;
#pragma unroll
                    for (int k = 0; k < C; ++k) {
                        n3[k] = (here >> (k + 2)) & 1u ? p[1][k] : n3[k];
                        n1[k] = (here >> k) & 1u ? p[3][k] : n1[k];
                    }
                }
                // stage st + 1 pulls row r - 1
#pragma unroll
                for (int k = 0; k < C; ++k) {
                    const float t0 = p[0][k], t2 = p[2][k];
                    p[0][k] = M[q][0][k];
                    p[1][k] = M[q][1][k];
                    p[3][k] = M[q][2][k];
                    p[2][k] = O[q][0][k];
                    p[5][k] = O[q][1][k];
                    p[6][k] = O[q][2][k];
                    p[7][k] = n7[k];
                    p[8][k] = n8[k];
                    O[q][0][k] = A[q][0][k];
                    O[q][1][k] = A[q][1][k];
                    O[q][2][k] = A[q][2][k];
                    A[q][0][k] = t2;
                    A[q][1][k] = n5[k];
                    A[q][2][k] = n6[k];
                    M[q][0][k] = t0;
                    M[q][1][k] = n1[k];
                    M[q][2][k] = n3[k];
                }
            }
        }
    };
    load_row(y0);
    load_own(y0);
#pragma unroll 1
    for (int y = y0; y < yend; ++y) {
        if (y >= p0 && y < p1 && !(y >= q0 && y < q1)) iteration(y, std::false_type{});
        else iteration(y, std::true_type{});
    }
}

template <int T, bool FULL>
static hipError_t launch_sweep_w(const SweepArgs& a, int model, hipStream_t st) {
    const dim3 grid(a.total_blocks), block(64 * a.block_waves);
    if (model == 2) hipLaunchKernelGGL((sweep_kernel<T, 2, FULL>), grid, block, 0, st, a);
    else if (model == 1) hipLaunchKernelGGL((sweep_kernel<T, 1, FULL>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((sweep_kernel<T, 0, FULL>), grid, block, 0, st, a);
    return hipGetLastError();
}

template <int T>
static hipError_t launch_sweep_t(const SweepArgs& a, int model, hipStream_t st) {
    return a.full ? launch_sweep_w<T, true>(a, model, st) : launch_sweep_w<T, false>(a, model, st);
}

hipError_t launch_sweep(int steps, const SweepArgs& a, int model, hipStream_t st) {
    switch (steps) {
        case 1: return launch_sweep_t<1>(a, model, st);
        case 2: return launch_sweep_t<2>(a, model, st);
        case 3: return launch_sweep_t<3>(a, model, st);
        case 4: return launch_sweep_t<4>(a, model, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm
