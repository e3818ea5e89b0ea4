// Kernel argument blocks and launchers shared between the kernel sources and
// the C-ABI layer.
#pragma once

#include "common.hpp"

namespace lbm {

constexpr int MAX_SEGMENTS = 32;  // runs of consecutive members with one lattice shape
constexpr int MAX_CHUNK = 256;    // steps per drag-reduction chunk

struct Segment {
    int block_begin;       // first workgroup of the segment
    int member_begin;      // first member
    int tiles_per_member;  // tiles_x * tiles_y
    int tiles_x;           // tiles of 256 columns
    int vec;               // 1: width a multiple of 4, rows handled four cells per lane
    int rows;              // two-step strips: rows per workgroup (the lattice height when not split)
};

struct StepArgs {
    const MemberDev* members;
    const int* parity;   // per member: which buffer holds its state before this chunk
    const int* active;
    float* pop0;
    float* pop1;
    double* partial;     // drag partials [member][slot][ring]
    int slot;            // step index within the chunk
    int flip;            // slot & 1: parity of this step relative to the chunk start
    int xcd;             // remap workgroups so each XCD gets contiguous tiles
    int total_blocks;
    int nseg;
    Segment seg[MAX_SEGMENTS];
    // non-null: the launch covers only these members (all of seg[0]'s shape),
    // tiles_per_member workgroups each, in list order
    const int* active_list;
    // two-step launches: 1 when some strip is split into row ranges (Segment::rows)
    int split;
    // non-null: open channels; the outlet ghost columns [member][9][ny]
    // (MemberDev::ghost_off), filled for this step by the ghost kernel
    const float* ghost;
};

constexpr int SWEEP_WAVES = 8;  // waves of a sweep workgroup at most
constexpr int SWEEP_CELLS = 2;  // cells per lane (four: 172 registers of the four-step kernel spill, 2.2 x the time)

// Members of one lattice shape in a sweep launch: a unit is the row range
// `rows` of one member, `waves` waves wide; a workgroup holds units_per_block.
struct SweepSegment {
    int block_begin;
    int member_begin;
    int units;            // members x ranges
    int ranges;           // row ranges per member
    int rows;             // rows per range (the last may be shorter)
    int waves;            // waves per unit, spanning the width
    int lanes;            // lanes used of each wave (the last wave: what is left)
    int units_per_block;
};

struct SweepArgs {
    const MemberDev* members;
    const int* parity;
    const int* active;
    const int* active_list;  // as StepArgs::active_list
    float* pop0;
    float* pop1;
    double* partial;
    int slot;                // chunk step of the launch's first step
    int flip;
    int full;                // every width is a multiple of 64 SWEEP_CELLS
    int total_blocks;
    int block_waves;         // waves per workgroup
    int nseg;
    SweepSegment seg[MAX_SEGMENTS];
};

// Members of one lattice shape in a resident launch: a workgroup (unit) holds
// `groups` groups of the launch's rows per wave of one member, `waves` waves
// wide; `ranges` workgroups share a member.
struct ResidentSegment {
    int block_begin;
    int member_begin;
    int ranges;
    int waves, lanes;      // as SweepSegment
    int groups;
    long long halo_begin;  // first halo word of the segment: [unit]{[side 2][slot 2][3 cells][lanes of the width], open: [side][slot][36]}
};

// A word's tag: the chunk's number, its pass and the step it is for.
constexpr int RESIDENT_STEP_BITS = 7, RESIDENT_PASS_BITS = 6;
constexpr int RESIDENT_LAUNCHES = 1 << (32 - RESIDENT_STEP_BITS - RESIDENT_PASS_BITS);
// Bound of a wait in the chunks of a batch after one was given up in it (0.2 ms: some 30 steps).
constexpr long long RESIDENT_SHORT_WAIT = 20000;

constexpr int RESIDENT_WIDEST = 1024;         // columns
constexpr int RESIDENT_OUTLET_WORDS = 36;  // open channels: two rows of the last two columns

struct ResidentArgs {
    const MemberDev* members;
    const int* parity;
    const int* active;
    const int* active_list;  // as StepArgs::active_list (member_begin counts in it then)
    float* pop0;
    float* pop1;
    double* partial;
    unsigned long long* halo;
    int launch;              // the chunk's number (1 .. RESIDENT_LAUNCHES - 1)
    int first;               // that of the batch's first chunk
    int* given_up;           // per member: the number of the chunk given up; then that of the last one of any member
    int n_members;
    long long wait_ticks;    // bound of a wait (100 MHz clock); below 0: give up at the first
    int n_steps;
    int flip;                // as StepArgs::flip
    int pass;
    int full;                // every member's width is a multiple of 64 cells per lane
    int total_blocks;
    int block_waves;
    int nseg;
    ResidentSegment seg[MAX_SEGMENTS];
};

struct GhostArgs {
    const MemberDev* members;
    const int* parity;
    const int* active;
    const float* pop0;
    const float* pop1;
    float* ghost;
    int flip;            // parity of the step's source buffer relative to the chunk start
};

struct InitArgs {
    const MemberDev* members;
    float* pop0;
    double* partial;
    uint64_t seed;
    double noise_amp;
    double ux0;  // initial uniform x-velocity
};

struct FinalizeArgs {
    const MemberDev* members;
    const int* active;
    int* parity;
    int* cursor;
    int* flags;
    const double* partial;
    float* series;
    double* accum;
    long long ld;        // row stride of the drag series
    int n;               // steps in this chunk
    int accumulate;      // add the observable to accum (0 for step 0)
    int swap_parity;     // parity of the number of buffer swaps in this chunk (one per kernel launch)
    double mu;
    double inv_sigma_dt; // dt / sigma
};

// The reduction of a resident chunk: block b's member is active_list[b], or b.
// Members whose chunk was given up are stepped again first, by every block of
// the launch (lbm_kernels.hip).
constexpr int REDO_TASKS = 512;   // bands of rows, of all members together, that a step is cut into
constexpr int REDO_STEPS = 1 << 9;  // above every chunk's steps: the counts of launch n start at n REDO_STEPS
struct RedoArgs {
    int launch;              // as ResidentArgs
    const int* given_up;
    int n_members;
    const int* active_list;
    int slots;               // members of the launch, active or not
    int bands;               // per member
    int flip;                // as ResidentArgs
    int states_only;         // 1: no reduction (an untracked chunk)
    int* done;               // [slots][bands]: launch REDO_STEPS + steps made
    int* ticket;             // [2]: tasks taken, blocks that have found none left (both 0 between launches)
    int* gave_up_host;       // pinned: set when a chunk is stepped again
    float* pop0;
    float* pop1;
    double* partial;
    float* ghost;            // open channels, as GhostArgs::ghost
};

struct TileShape {
    int tyt;    // waves per workgroup
    int r;      // rows per wave (a tile is 256 columns by tyt * r rows); 1 for two-step shapes
    int xcd;    // 1: remap workgroups so each XCD gets a contiguous range of tiles
    int steps;  // lattice steps per launch: 1, or 2 (a strip of 256 columns swept bottom to top)
    int adaptive;  // chooses between the resident kernel, the sweep, the two-step kernel and shape 0 by the active members
    int seg_rows;  // two-step shapes: rows per workgroup (0: whole strips; -1: split only when
                   // the strips alone leave workgroup slots empty)
};

extern const TileShape TILE_SHAPES[];
extern const int N_TILE_SHAPES;

// model: 0 BGK, 1 central moments (every member of the launch uses it)
hipError_t launch_step(int tile_id, const StepArgs& a, int model, hipStream_t st);
// two steps per launch, `waves` rows per iteration; the segment table must
// describe strips of 256 columns (tiles_per_member = tiles_x = nx / 256)
hipError_t launch_step2(int waves, const StepArgs& a, int model, hipStream_t st);
// up to four steps per launch
hipError_t launch_sweep(int steps, const SweepArgs& a, int model, hipStream_t st);
// a chunk of steps in one launch, `cells` columns per lane and `rows` rows per wave (the host's table of cuts)
hipError_t launch_resident(int cells, int rows, bool open, const ResidentArgs& a, int model, hipStream_t st);
hipError_t launch_init(const InitArgs& a, int n_members, long long max_cells, hipStream_t st);
// the outlet ghost columns of the open-channel members for the next one-step launch
hipError_t launch_outlet_ghost(const GhostArgs& a, int n_members, int max_ny, hipStream_t st);
hipError_t launch_finalize(const FinalizeArgs& a, int n_members, hipStream_t st);
hipError_t launch_finalize_resident(const FinalizeArgs& a, const RedoArgs& r, hipStream_t st);

}  // namespace lbm
