// A whole chunk of lattice steps in one launch, with the populations in the
// registers of the device.
//
// A wave holds R rows of up to 64 C columns (C cells per lane), all nine
// populations, from the first step of the chunk to the last; the waves of a
// workgroup span one member's width and a few groups of R rows, and the
// workgroups of a member share its height.  In a step a row pulls from the
// rows and columns around it and is collided in place.  What leaves a wave
// sideways passes through LDS (one 3-value exchange per row and side), what
// leaves it up or down through LDS within the workgroup and through memory
// between workgroups, as 8-byte words that carry their step beside the value:
// a reader takes a word once its step is the one it waits for, so there is no
// flag to order and no fence.  Two slots alternate; a workgroup can be at most
// one step ahead of its neighbour.  The rows inside a wave come first in a
// step, the lowest and the highest last: the words travel meanwhile.
//
// Open channels: what enters from the inlet is constant; what enters from the
// outlet is formed by the waves of the last columns before each step
// (outlet_ghost_value), from the last two columns of their rows and of two rows
// on either side, which their neighbours hand out beside the rows above.
//
// The wait for a neighbour is bounded: workgroups of a member run side by side
// when the device is free (the host launches at most as many as fit), but
// kernels of other streams may hold part of it.  A wave that waits longer than
// its limit (lbm_set_wait_limit; a short one once a chunk of the same batch was
// given up) gives the member's chunk up: it marks it and
// leaves, every other wave of the member that waits leaves too, and the
// chunk's drag reduction steps the member again from the untouched source
// buffer (resident_redo).  So every wave ends, and the result never
// depends on what ran beside.
//
// What bounds it: with few waves, a step's chain: a row's collision by a lone
// wave (0.8 us) and the words' way to memory and back (1 x 256 x 64: 2.1 us
// per step, 6.8 with one launch per step); with the registers full, the FP64
// units (16 x 512 x 128, four rows per wave, two waves per SIMD: 6.7 us, 3.5 of
// them the 204 FP64 instructions of a wave's row at 5.2 cycles of 2.4 GHz; 15.6
// us with one launch per step).  Six rows of two cells per lane, or four
// of three, are the most that 256 registers hold (eight spill 73, two of five
// 20).  Rows in the order from the bottom up, waiting first: 9.3 us;
// walls and square links worked out in each step instead of once: 8.7.
#include "lbm_device.hpp"

namespace lbm {

typedef float f2 __attribute__((ext_vector_type(2)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));

// (by value: a choice between two places would keep the populations in memory)
__device__ __forceinline__ float pick(bool c, float a, float b) { return c ? a : b; }

__device__ __forceinline__ void put_word(unsigned long long* p, float v, unsigned tag) {
    __hip_atomic_store(p, ((unsigned long long)tag << 32) | __float_as_uint(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long get_word(const unsigned long long* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void give_up(int* given_up, int mi, int n_members, int launch) {
    __hip_atomic_store(given_up + mi, launch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(given_up + n_members, launch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The kernel's arguments by their address: what only a long wait reads is loaded there and holds no scalar
// registers in the rows' loop, which spills them (us, 64 steps: 512 x 512 x 128 open 13.94 -> 13.86 ms, 64 x 513 x 129
// open 2849 -> 2839, 1 x 256 x 64 142.8 -> 137.5).
typedef const __attribute__((address_space(4))) ResidentArgs* KernelArgs;
__device__ __forceinline__ KernelArgs kernel_args() { return (KernelArgs)__builtin_amdgcn_kernarg_segment_ptr(); }

// FULL: every member's width is a multiple of 64 C (no lane or cell of a wave is beyond it, and no choice of its end
// is made in each row: us per step 1 x 256 x 64 2.2 -> 2.1, 16 x 512 x 128 7.2 -> 7.0, 4 x 1024 x 256 7.0 -> 6.7).
template <int C, int R, int MODEL, bool OPEN, bool FULL>
__global__ __launch_bounds__(64 * SWEEP_WAVES) __attribute__((amdgpu_waves_per_eu(2))) void resident_kernel(ResidentArgs a) {
    // columns beside a wave: [slot][wave][row][side]: side 0 its first cell (3, 6, 7), side 1 its last (1, 5, 8)
    __shared__ f4 xe[2][SWEEP_WAVES][R][2];
    // rows beside a wave of the workgroup: [slot][side][direction x cell of the lane][row group x lanes]:
    // side 0 the group's lowest row (4, 7, 8), side 1 its highest (2, 5, 6)
    __shared__ float yh[2][2][3 * C * 512];
    // the lane's cells of a row beside a wall or the square: bits 0-7 the directions 1-8 that come from a wall or
    // the square, bits 8-15 those that go to the square, from bit 16 the cell's place in the ring + 1
    __shared__ __attribute__((aligned(16))) unsigned marks[SWEEP_WAVES][R][64][C];
    // open channels: what enters from the inlet (1, 5, 8) and the outlet (3, 6, 7) column, rows -1 .. R of a row
    // group; the last two columns (nx - 1 and nx - 2, nine populations each) of rows -2 .. groups R + 1 of the
    // workgroup, [slot]; their velocities, rows -2 .. R + 1 of a row group
    constexpr int OG = OPEN ? SWEEP_WAVES : 1;
    __shared__ f4 inlet[OG][R + 2], outlet[OG][R + 2];
    __shared__ __attribute__((aligned(16))) float last2[OPEN ? 2 : 1][OG * R + 4][24];
    __shared__ OutletVel vel[OG][R + 4];
    const int b = (int)blockIdx.x;
    int s = 0;
#pragma unroll 1
    while (s + 1 < a.nseg && b >= a.seg[s + 1].block_begin) ++s;
    const ResidentSegment sg = a.seg[s];
    const int lane = (int)(threadIdx.x & 63);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // row group and column wave; every other group from the right, so that a SIMD's two waves (four apart) are not
    // both at one end of their rows
    const int W = sg.waves, g = wave / W, wn = wave - g * W, w = g & 1 ? W - 1 - wn : wn;
    auto wave_at = [&](int cw) { return g * W + (g & 1 ? W - 1 - cw : cw); };
    if (g >= sg.groups) return;
    const int unit = b - sg.block_begin;
    const int mloc = unit / sg.ranges, range = unit - mloc * sg.ranges;
    const int mi = a.active_list ? a.active_list[sg.member_begin + mloc] : sg.member_begin + mloc;
    const int on = a.active[mi];
    const MemberDev m = a.members[mi];
    const int par = a.parity[mi] ^ a.flip;
    const unsigned tag0 = ((unsigned)a.launch << RESIDENT_PASS_BITS | (unsigned)a.pass) << RESIDENT_STEP_BITS;  // tag of step t: + t + 1
    if (!on) return;
    const float* __restrict__ src = (par ? a.pop1 : a.pop0) + m.off;
    float* __restrict__ dst = (par ? a.pop0 : a.pop1) + m.off;
    const int nx = m.nx, ny = m.ny;
    const unsigned plane = (unsigned)nx * (unsigned)ny;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)src, (short)0, (int)(36u * plane), BUFFER_RSRC_WORD3);
    const int base = w * sg.lanes * C;
    const int x0 = base + C * lane;
    const bool last_wave = w == W - 1;
    const int lastl = FULL ? 63 : last_wave ? (nx - base + C - 1) / C - 1 : sg.lanes - 1;
    const int lastk = FULL ? C - 1 : last_wave ? nx - base - C * lastl - 1 : C - 1;  // the last cell of the wave's last lane
    auto last_cell = [&](const float (&v)[C]) {
        float e = v[C - 1];
#pragma unroll
        for (int k = 0; k < C - 1; ++k) e = pick(lastk == k, v[k], e);
        return e;
    };
    const int ys = (range * sg.groups + g) * R;                 // the wave's lowest row
    const int rows = min(R, ny - ys);                           // <= 0: no row (it only meets the barriers)
    const bool below = rows > 0 && ys > 0, above = rows == R && ys + R < ny;
    const bool low_mem = below && g == 0, high_mem = above && g == sg.groups - 1;
    const bool outlet_wave = OPEN && last_wave, inlet_wave = OPEN && w == 0;
    const bool sq_cols = m.ss > 0 && base <= m.sx0 + m.ss && base + sg.lanes * C - 1 >= m.sx0 - 1;
    unsigned sqc = 0;  // bit j: column x0 - 1 + j crosses the square
    if (sq_cols)
#pragma unroll
        for (int j = 0; j < C + 2; ++j) sqc |= ((unsigned)(x0 - 1 + j - m.sx0) < (unsigned)m.ss ? 1u : 0u) << j;
    const bool grid_cols = OPEN && m.bar > 0 && base <= m.gx0 + m.bar && base + sg.lanes * C - 1 >= m.gx0 - 1;
    unsigned gridc = 0;  // likewise for the grid's columns
    if (grid_cols)
#pragma unroll
        for (int j = 0; j < C + 2; ++j) gridc |= ((unsigned)(x0 - 1 + j - m.gx0) < (unsigned)m.bar ? 1u : 0u) << j;
    // bit j: row ys - 1 + j is a wall, or crosses the square or the grid's bars in the wave's columns; bit r: row
    // ys + r is beside such a row, or may hold cells beside the square
    unsigned wall_rows = 0, solid_rows = 0, grid_rows = 0, near_rows = 0, ring_rows = 0;
#pragma unroll
    for (int j = 0; j < R + 2; ++j) {
        const int y = ys - 1 + j;
        wall_rows |= (y < 0 || y >= ny ? 1u : 0u) << j;
        solid_rows |= (sq_cols && (unsigned)(y - m.sy0) < (unsigned)m.ss ? 1u : 0u) << j;
        if (OPEN) grid_rows |= (grid_cols && y >= 0 && y < ny && grid_row(m, y) ? 1u : 0u) << j;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = ys + r;
        near_rows |= (((wall_rows | solid_rows | grid_rows) >> r) & 7u ? 1u : 0u) << r;
        ring_rows |= (r < rows && sq_cols && y >= m.sy0 - 1 && y <= m.sy0 + m.ss ? 1u : 0u) << r;
    }
#pragma unroll 1
    for (int r = 0; r < R; ++r) {
        if (!((near_rows >> r) & 1u)) continue;
        const int y = ys + r;
        unsigned word[C];
#pragma unroll
        for (int k = 0; k < C; ++k) {
            word[k] = 0;
#pragma unroll
            for (int i = 1; i < 9; ++i) {
                const int j = r + 1 - CY[i];
                const bool back = ((wall_rows >> j) & 1u) || (((solid_rows >> j) & 1u) && ((sqc >> (1 - CX[i] + k)) & 1u)) ||
                                  (OPEN && ((grid_rows >> j) & 1u) && ((gridc >> (1 - CX[i] + k)) & 1u));
                word[k] |= (back ? 1u : 0u) << (i - 1);
            }
            // (a lane beyond the wave's columns is in no ring)
            if (((ring_rows >> r) & 1u) && lane <= lastl && !in_square(m, x0 + k, y) && ring_index(m, x0 + k, y) >= 0)
                word[k] |= square_links(m, x0 + k, y) << 7 | (unsigned)(ring_index(m, x0 + k, y) + 1) << 16;
        }
#pragma unroll
        for (int k = 0; k < C; ++k) marks[wave][r][lane][k] = word[k];
    }
    // Words and floats of a row beside a wave are laid out [direction 3][cell of the lane C][lane of the
    // member's width]; a lane reads its own columns and shifts, and the first and the last lane read the column beside the
    // wave: of the direction that moves right (d 1 from below: 5, d 2 from above: 8), and left (6 and 7).
    const int hp = (nx + C - 1) / C;
    const int lc = min(w * sg.lanes + lane, hp - 1);
    const int left_k = w == 0 ? (nx - 1) % C : C - 1;
    const int beside = lane == 0 ? (w == 0 ? hp - 1 : w * sg.lanes - 1) : lane == lastl ? (last_wave ? 0 : (w + 1) * sg.lanes) : lc;
    const int beside_low = lane == 0 ? C + left_k : lane == lastl ? 2 * C : 0;
    const int beside_high = lane == 0 ? 2 * C + left_k : lane == lastl ? C : 0;
    const long long hs = 3LL * C * hp;  // words of a row: [unit][side][slot]; then, in open channels, of the last columns
    const long long unit_words = 4 * hs + (OPEN ? 4 * RESIDENT_OUTLET_WORDS : 0);
    unsigned long long* const mine = a.halo + sg.halo_begin + unit * unit_words;
    const int wl = wave_at(w == 0 ? W - 1 : w - 1), wr = wave_at(last_wave ? 0 : w + 1);
    double om[C];  // open channels: the relaxation rate of the lane's columns (the sponge's rises to the outlet)
    if constexpr (OPEN) {
#pragma unroll
        for (int k = 0; k < C; ++k) {
            MemberDev mc = m;
            sponge_at(mc, x0 + k);
            om[k] = mc.omega;
        }
        if (inlet_wave && lane < R + 2) {
            const int y = ys - 1 + lane;
            inlet[g][lane] = f4{inlet_dev(m, 1, y), inlet_dev(m, 5, y), inlet_dev(m, 8, y), 0.0f};
        }
    }

    float f[R][9][C];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const unsigned row = (unsigned)max(min(ys + r, ny - 1), 0) * (unsigned)nx;
#pragma unroll
        for (int i = 0; i < 9; ++i) load_cells<C>(rs, 4u * (unsigned)x0, 4u * ((unsigned)i * plane + row), f[r][i]);  // (dead cells: any value)
    }

    // hand out the populations of row r that leave the wave sideways, for the step with slot n
    auto publish_row = [&](int r, int n) {
        if (lane == 0) xe[n][wave][r][0] = f4{f[r][3][0], f[r][6][0], f[r][7][0], 0.0f};
        if (lane == lastl) xe[n][wave][r][1] = f4{last_cell(f[r][1]), last_cell(f[r][5]), last_cell(f[r][8]), 0.0f};
        if (OPEN && outlet_wave) {
            float* const q = last2[n][g * R + r + 2];
            if (lane == lastl)
#pragma unroll
                for (int i = 0; i < 9; ++i) q[i] = last_cell(f[r][i]);
            if (lane == (lastk ? lastl : lastl - 1))
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    float e = f[r][i][C - 1];
#pragma unroll
                    for (int k = 0; k < C - 1; ++k) e = pick(lastk == k + 1, f[r][i][k], e);
                    q[12 + i] = e;
                }
        }
    };
    // a word of the last columns: lane 0-17 the first of two rows, 18-35 the second
    const int last_row = lane < 18 ? 0 : 1, last_at = lane - 18 * last_row < 9 ? lane - 18 * last_row : lane - 18 * last_row + 3;
    auto publish_outlet = [&](int n, unsigned tag) {
        if (!OPEN || !outlet_wave) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup", "local");  // (written by other lanes of the wave)
        if (lane < RESIDENT_OUTLET_WORDS) {
            unsigned long long* const p = mine + 4 * hs + lane;
            if (low_mem) put_word(p + n * RESIDENT_OUTLET_WORDS, last2[n][2 + last_row][last_at], tag);
            if (high_mem) put_word(p + (2 + n) * RESIDENT_OUTLET_WORDS, last2[n][g * R + R + last_row][last_at], tag);
        }
    };
    // those of the lowest (side 0: 4, 7, 8) or highest row (side 1: 2, 5, 6); tag: the step they are for
    auto publish_side = [&](int side, int r, int i0, int i1, int i2, int n, unsigned tag) {
        if (!(side ? above : below)) return;
        float v[3 * C];
#pragma unroll
        for (int k = 0; k < C; ++k) {
            v[k] = f[r][i0][k];
            v[C + k] = f[r][i1][k];
            v[2 * C + k] = f[r][i2][k];
        }
        if (side ? high_mem : low_mem) {
            if (lane <= lastl) {
                unsigned long long* const p = mine + (side * 2 + n) * hs;
#pragma unroll
                for (int q = 0; q < 3 * C; ++q) put_word(p + (q * hp + lc), v[q], tag);
            }
        } else if (lane <= lastl) {
#pragma unroll
            for (int q = 0; q < 3 * C; ++q) yh[n][side][q * 512 + g * hp + lc] = v[q];
        }
    };
#pragma unroll
    for (int r = 0; r < R; ++r) publish_row(r, 0);
    publish_side(0, 0, 4, 7, 8, 0, tag0 + 1u);
    publish_side(1, R - 1, 2, 5, 6, 0, tag0 + 1u);
    publish_outlet(0, tag0 + 1u);
    if (a.wait_ticks < 0 && (low_mem || high_mem)) {  // no wait at all (the giving up is tested so)
        give_up(a.given_up, mi, a.n_members, a.launch);
        return;
    }
    lds_barrier();

    auto right = [&](const float (&v)[C], float in, float (&o)[C]) {  // +x movers: one cell to the right
        const float sh = wave_shr1_in(v[C - 1], in);
#pragma unroll
        for (int k = C - 1; k > 0; --k) o[k] = v[k - 1];
        o[0] = sh;
    };
    auto left = [&](const float (&v)[C], float in, float (&o)[C]) {  // -x movers
        const float sh = wave_shl1_in(v[0], in);
#pragma unroll
        for (int k = 0; k < C; ++k) {
            const float e = k + 1 < C ? v[k + 1 < C ? k + 1 : k] : sh;
            o[k] = FULL ? e : pick(lane == lastl && lastk == k, in, e);  // (lane 63's shifted value is `in`)
        }
    };
#pragma unroll 1
    for (int t = 0; t < a.n_steps; ++t) {
        // looked at afresh each step: the tests made from these are the same in every step, and the compiler would
        // keep all of them (two scalars each) through the loop
        unsigned nears = (unsigned)__builtin_amdgcn_readfirstlane((int)near_rows);
        unsigned rings = (unsigned)__builtin_amdgcn_readfirstlane((int)ring_rows);
        int hq = __builtin_amdgcn_readfirstlane(hp);
        __asm__ volatile("" : "+s"(nears), "+s"(rings), "+s"(hq));
        const int n = t & 1;
        const unsigned tag = tag0 + (unsigned)t + 1u;
        double* const ps = a.partial + m.part_off + (long long)t * m.ring;

        auto collide = [&](float (&dl)[9], int k, unsigned links, bool ring) -> double {
            if constexpr (OPEN) {
                MemberDev mc = m;
                mc.omega = om[k];
                __asm__ volatile("" : "+v"(mc.omega));  // (what follows from it would fill the registers otherwise)
                if (MODEL == 0) bgk_coefficients(mc);
                return collide_cell<MODEL>(mc, dl, links, ring);
            } else {
                return collide_cell<MODEL>(m, dl, links, ring);
            }
        };
        // row r of the step, given what arrives from the rows below (2, 5, 6) and above (4, 7, 8) and the columns beside
        auto collide_row = [&](int r, const float (&up)[3][C], const float (&dn)[3][C], float el, float er) {
            float p[9][C];
#pragma unroll
            for (int k = 0; k < C; ++k) {
                p[0][k] = f[r][0][k];
                p[2][k] = up[0][k];
                p[5][k] = up[1][k];
                p[6][k] = up[2][k];
                p[4][k] = dn[0][k];
                p[7][k] = dn[1][k];
                p[8][k] = dn[2][k];
            }
            right(f[r][1], el, p[1]);
            left(f[r][3], er, p[3]);
            unsigned mark[C] = {};
            if ((nears >> r) & 1u) {  // halfway bounce-back: the cell's own opposite population
#pragma unroll
                for (int k = 0; k < C; ++k) mark[k] = marks[wave][r][lane][k];
#pragma unroll
                for (int i = 1; i < 9; ++i)
#pragma unroll
                    for (int k = 0; k < C; ++k) {
                        unsigned back;  // all ones or zero (the compiler would make a comparison and a choice of it)
                        __asm__("v_bfe_i32 %0, %1, %2, 1" : "=v"(back) : "v"(mark[k]), "n"(i - 1));
                        p[i][k] = pinned(__uint_as_float((back & __float_as_uint(f[r][OPP[i]][k])) | (~back & __float_as_uint(p[i][k]))));
                    }
            }
            if ((rings >> r) & 1u) {
#pragma unroll
                for (int k = 0; k < C; ++k) {
                    float dl[9];
#pragma unroll
                    for (int i = 0; i < 9; ++i) dl[i] = pinned(p[i][k]);
                    const double drag = collide(dl, k, mark[k] >> 7 & 0x1FEu, true);
#pragma unroll
                    for (int i = 0; i < 9; ++i) f[r][i][k] = pinned(dl[i]);
                    if (mark[k] >> 16) ps[(int)(mark[k] >> 16) - 1] = drag;
                }
            } else {
#pragma unroll
                for (int k = 0; k < C; ++k) {
                    float dl[9];
#pragma unroll
                    for (int i = 0; i < 9; ++i) dl[i] = pinned(p[i][k]);
                    collide(dl, k, 0u, false);
#pragma unroll
                    for (int i = 0; i < 9; ++i) f[r][i][k] = pinned(dl[i]);
                }
            }
            publish_row(r, n ^ 1);
        };
        // what row r sends to the row above it, and to the row below
        auto send_up = [&](int r, const f4& el, const f4& er, float (&o)[3][C]) {
#pragma unroll
            for (int k = 0; k < C; ++k) o[0][k] = f[r][2][k];
            right(f[r][5], el.y, o[1]);
            left(f[r][6], er.y, o[2]);
        };
        auto send_down = [&](int r, const f4& el, const f4& er, float (&o)[3][C]) {
#pragma unroll
            for (int k = 0; k < C; ++k) o[0][k] = f[r][4][k];
            left(f[r][7], er.z, o[1]);
            right(f[r][8], el.z, o[2]);
        };
        // until every lane's words are there; false: given up (bounded: see the top of the file)
        auto wait = [&](auto&& words) -> bool {
            long long began = 0;
            for (int spin = 0;; ++spin) {
                const bool ok = words();
                if (__all(ok)) return true;
                if ((spin & 63) == 63) {
                    const long long now = wall_clock64();
                    if (!began) began = now;
                    const KernelArgs k = kernel_args();
                    int* const up = k->given_up;
                    const int any = __hip_atomic_load(up + k->n_members, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const long long limit = any >= k->first ? min(k->wait_ticks, RESIDENT_SHORT_WAIT) : k->wait_ticks;
                    const bool late = now - began > limit;
                    if (late) give_up(up, mi, k->n_members, k->launch);
                    if (late || __hip_atomic_load(up + mi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == k->launch) return false;
                }
            }
        };
        // what arrives from the row below the wave (side 0) or above it; false: given up
        auto arrive = [&](int side, float (&o)[3][C]) -> bool {
            float v[3][C], e = 0.0f;
#pragma unroll
            for (int q = 0; q < 3 * C; ++q) v[q / C][q % C] = 0.0f;
            if (side ? high_mem : low_mem) {
                // the unit below's side 1, or the unit above's side 0
                const unsigned long long* const p = mine + (side ? unit_words + n * hs : (2 + n) * hs - unit_words);
                unsigned long long u[3 * C + 1];
                if (!wait([&] {
#pragma unroll
                        for (int q = 0; q < 3 * C; ++q) u[q] = get_word(p + (q * hq + lc));
                        u[3 * C] = get_word(p + ((side ? beside_high : beside_low) * hq + beside));
                        bool ok = true;
#pragma unroll
                        for (int q = 0; q <= 3 * C; ++q) ok = ok && (unsigned)(u[q] >> 32) == tag;
                        return ok;
                    }))
                    return false;
#pragma unroll
                for (int q = 0; q < 3 * C; ++q) v[q / C][q % C] = __uint_as_float((unsigned)u[q]);
                e = __uint_as_float((unsigned)u[3 * C]);
            } else if (side ? above : below) {
                const float* const q = &yh[n][side ^ 1][(side ? g + 1 : g - 1) * hp];
#pragma unroll
                for (int j = 0; j < 3 * C; ++j) v[j / C][j % C] = q[j * 512 + lc];
                e = q[(side ? beside_high : beside_low) * 512 + beside];
            }
            if (OPEN) {  // beside the first and the last column
                if (inlet_wave) e = pick(lane == 0, side ? inlet[g][R + 1].z : inlet[g][0].y, e);
                if (outlet_wave) e = pick(lane == lastl, side ? outlet[g][R + 1].z : outlet[g][0].y, e);
            }
#pragma unroll
            for (int k = 0; k < C; ++k) o[0][k] = v[0][k];
            if (side) {
                left(v[1], e, o[1]);
                right(v[2], e, o[2]);
            } else {
                right(v[1], e, o[1]);
                left(v[2], e, o[2]);
            }
            return true;
        };

        // Open channels: what enters from the outlet column (outlet_ghost_value) needs the last two columns of the
        // rows up to two above and below: lanes form the velocities, then the populations, one each.
        if (OPEN && outlet_wave) {
            if (low_mem || high_mem) {
                const unsigned long long* const pl = mine - unit_words + 4 * hs + (2 + n) * RESIDENT_OUTLET_WORDS + lane;
                const unsigned long long* const ph = mine + unit_words + 4 * hs + n * RESIDENT_OUTLET_WORDS + lane;
                unsigned long long ul = 0, uh = 0;
                if (!wait([&] {
                        bool ok = true;
                        if (lane < RESIDENT_OUTLET_WORDS) {
                            if (low_mem) ul = get_word(pl);
                            if (high_mem) uh = get_word(ph);
                            ok = (!low_mem || (unsigned)(ul >> 32) == tag) && (!high_mem || (unsigned)(uh >> 32) == tag);
                        }
                        return ok;
                    }))
                    return;
                if (lane < RESIDENT_OUTLET_WORDS) {
                    if (low_mem) last2[n][last_row][last_at] = __uint_as_float((unsigned)ul);
                    if (high_mem) last2[n][g * R + R + 2 + last_row][last_at] = __uint_as_float((unsigned)uh);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup", "local");
            }
            if (lane < 2 * (R + 4)) {
                float dl[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) dl[i] = last2[n][g * R + (lane >> 1)][12 * (lane & 1) + i];
                double ux, uy;
                stored_velocity(dl, ux, uy);
                double* const q = &vel[g][lane >> 1].ux1 + 2 * (lane & 1);
                q[0] = ux;
                q[1] = uy;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup", "local");
            if (lane < 3 * (R + 2)) {
                const int r = lane / 3, d = lane - 3 * r, y = ys - 1 + r;  // directions 3, 6, 7
                const OutletVel va = vel[g][y > 0 ? r : r + 1], v0 = vel[g][r + 1], vb = vel[g][y + 1 < ny ? r + 2 : r + 1];
                double rho_g = 1.0;
                if (m.out_rho) {
                    float d1[9], d2[9];
#pragma unroll
                    for (int i = 0; i < 9; ++i) {
                        d1[i] = last2[n][g * R + r + 1][i];
                        d2[i] = last2[n][g * R + r + 1][12 + i];
                    }
                    rho_g = outlet_density(m, d1, d2);
                }
                ((float*)&outlet[g][r])[d] =
                    outlet_ghost_value(m, -1.0, d == 0 ? 0.0 : d == 1 ? 1.0 : -1.0, d == 0 ? WD[3] : WD[6], y, va, v0, vb, rho_g);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup", "local");
        }
        auto beside_left = [&](int r) { return OPEN && inlet_wave ? inlet[g][r + 1] : xe[n][wl][r][1]; };
        auto beside_right = [&](int r) { return OPEN && outlet_wave ? outlet[g][r + 1] : xe[n][wr][r][0]; };

        if constexpr (R == 1) {
            const f4 el = beside_left(0), er = beside_right(0);
            float up[3][C], dn[3][C];
            if (!arrive(0, up) || !arrive(1, dn)) return;
            collide_row(0, up, dn, el.x, er.x);
            publish_side(0, 0, 4, 7, 8, n ^ 1, tag + 1u);
            publish_side(1, 0, 2, 5, 6, n ^ 1, tag + 1u);
        } else {
            // the rows that wait for nothing first: the words from the workgroups beside travel meanwhile
            float below0[3][C], nu[3][C];  // what row 1 sends down to row 0; what arrives at the next row from below
            f4 el = beside_left(0), er = beside_right(0);
            send_up(0, el, er, nu);
            el = beside_left(1);
            er = beside_right(1);
            send_down(1, el, er, below0);
#pragma unroll
            for (int r = 1; r + 1 < R; ++r) {
                const f4 eln = beside_left(r + 1), ern = beside_right(r + 1);
                float nn[3][C], dn[3][C];
                send_up(r, el, er, nn);
                send_down(r + 1, eln, ern, dn);
                collide_row(r, nu, dn, el.x, er.x);
#pragma unroll
                for (int q = 0; q < 3 * C; ++q) nu[q / C][q % C] = nn[q / C][q % C];
                el = eln;
                er = ern;
            }
            {
                float up[3][C];
                if (!arrive(0, up)) return;
                collide_row(0, up, below0, beside_left(0).x, beside_right(0).x);
                publish_side(0, 0, 4, 7, 8, n ^ 1, tag + 1u);
            }
            {
                float dn[3][C];
                if (!arrive(1, dn)) return;
                collide_row(R - 1, nu, dn, el.x, er.x);
                publish_side(1, R - 1, 2, 5, 6, n ^ 1, tag + 1u);
            }
        }
        publish_outlet(n ^ 1, tag + 1u);
        lds_barrier();
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r < rows) {
            unsigned skip = (solid_rows >> (r + 1)) & 1u ? sqc >> 1 : 0u;  // bit k: not written
            if (OPEN && ((grid_rows >> (r + 1)) & 1u)) skip |= gridc >> 1;
            if (lane >= lastl) skip |= lane > lastl ? ~0u : ~0u << (lastk + 1);
            const unsigned cell = (unsigned)(ys + r) * (unsigned)nx + (unsigned)x0;
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                float* const q = dst + ((unsigned)i * plane + cell);
#pragma unroll
                for (int k = 0; k < C; ++k)
                    if (!((skip >> k) & 1u)) q[k] = f[r][i][k];
            }
        }
    }
}

template <int C, int R, bool OPEN, bool FULL>
static hipError_t launch_resident_f(const ResidentArgs& a, int model, hipStream_t st) {
    const dim3 grid(a.total_blocks), block(64 * a.block_waves);
    if (model == 2) hipLaunchKernelGGL((resident_kernel<C, R, 2, OPEN, FULL>), grid, block, 0, st, a);
    else if (model == 1) hipLaunchKernelGGL((resident_kernel<C, R, 1, OPEN, FULL>), grid, block, 0, st, a);
    else hipLaunchKernelGGL((resident_kernel<C, R, 0, OPEN, FULL>), grid, block, 0, st, a);
    return hipGetLastError();
}

template <int C, int R, bool OPEN>
static hipError_t launch_resident_r(const ResidentArgs& a, int model, hipStream_t st) {
    if constexpr (C == 2)
        if (a.full) return launch_resident_f<C, R, OPEN, true>(a, model, st);
    return launch_resident_f<C, R, OPEN, false>(a, model, st);
}

hipError_t launch_resident(int cells, int rows, bool open, const ResidentArgs& a, int model, hipStream_t st) {
    switch (10 * cells + rows) {
        case 21: return open ? hipErrorInvalidValue : launch_resident_r<2, 1, false>(a, model, st);
        case 22: return open ? launch_resident_r<2, 2, true>(a, model, st) : launch_resident_r<2, 2, false>(a, model, st);
        case 23: return open ? launch_resident_r<2, 3, true>(a, model, st) : launch_resident_r<2, 3, false>(a, model, st);
        case 24: return open ? launch_resident_r<2, 4, true>(a, model, st) : launch_resident_r<2, 4, false>(a, model, st);
        case 26: return open ? launch_resident_r<2, 6, true>(a, model, st) : launch_resident_r<2, 6, false>(a, model, st);
        case 32: return open ? launch_resident_r<3, 2, true>(a, model, st) : launch_resident_r<3, 2, false>(a, model, st);
        case 33: return open ? launch_resident_r<3, 3, true>(a, model, st) : launch_resident_r<3, 3, false>(a, model, st);
        case 34: return open ? hipErrorInvalidValue : launch_resident_r<3, 4, false>(a, model, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm
