// Internal declarations shared by the device kernels and the host runtime.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace omap {

constexpr int kLanes = 64;                          // CDNA wavefront
constexpr int kWavesPerBlock = 4;
constexpr int kBlockThreads = kLanes * kWavesPerBlock;
constexpr uint32_t kObstacleBit = 0x80000000u;      // in-register obstacle marker
// Visit counters are kept in kSpread copies (a block adds to copy blockIdx mod
// kSpread) so that concurrent waves do not serialise on one address; readers
// sum the copies.
constexpr int kSpread = 16;
// Rounds whose scheduled counts the host can look at (a ring by round).
constexpr int kPosted = 64;
// Bit-packed front propagation (omap_front.h): layers per tile visit, in steps
// of 16, and the tile.
constexpr int kFrontSteps = 4;
constexpr int kFrontLayers = 16 * kFrontSteps;
constexpr int kFrontTileRows = 64;
constexpr int kFrontCols = 64;

// Maze state on the device.  Activity rows are `pitch` int32 apart (pitch a
// multiple of 64, so rows are 256-byte aligned); the obstacle mask has one bit
// per cell (bit c&31 of word c>>5 of the row, 1 = obstacle), `mpitch` words per
// row, and the bits of columns >= W are set (guard bits).  Word j of row r lies
// at r * mrow + j * mcol: row by row (mrow = mpitch, mcol = 1) for the integer
// sweeps, strip by strip (mrow = 1, mcol >= H) for the front propagation.
struct MazeDev {
    int32_t H, W;
    int32_t pitch;
    int32_t mpitch;
    int32_t mrow, mcol;
    int32_t tiles_x, tiles_y;
    int32_t tile_base;      // global id of tile (0, 0)
    int32_t K;              // source level of the encoding
    int32_t* V[2];          // activity ping-pong (front propagation: V[0] alone)
    const uint32_t* mask;
    uint32_t* R[2];         // front propagation: reached-set planes (mask layout), else null
    int32_t round0;         // front propagation: index of the maze's first round
    uint32_t tiles_x_inv;   // front propagation: min(2^32 / tiles_x, 2^32 - 1) (see front_tile_row)
};

// Arguments of round r of the tile schedule.  The tile lists and their dedup
// flags alternate by r mod 2; the list counts, the per-maze scheduled counts
// and the dense schedule's "changed" flags rotate over three buffers by r mod
// 3, so that round r can clear the buffer round r+1 will fill without racing
// with anything that reads or writes during round r.
struct RoundArgs {
    const MazeDev* mazes;
    const int32_t* tile_maze;     // global tile id -> maze slot (-1 = unused id)
    int32_t n_tile_ids;           // size of the tile id space
    const int32_t* list_in;       // (tile id, slot) pairs of round r (active schedule)
    const int32_t* count_in;      // their number
    int32_t* flags_in;            // cleared as the tiles of round r are visited
    int32_t* list_out;            // (tile id, slot) pairs scheduled for round r+1
    int32_t* count_out;           // their number (dense: 1 = some tile changed)
    int32_t* flags_out;           // 1 = already scheduled for round r+1
    int32_t* count_clear;         // count of round r+2, zeroed by round r
    const int32_t* sched_in;      // per slot: tiles scheduled for round r (more than one slot)
    int32_t* sched_out;           // per slot: tiles scheduled for round r+1 (kept only with
                                  // more than one slot; with one slot it equals *count_out)
    int32_t* sched_clear;         // per slot: scheduled counts of round r+2, zeroed by round r
    int32_t* dchg_prev;           // dense, per slot: changed in round r-1 (visit in round r)
    int32_t* dchg_cur;            // dense, per slot: changed in round r
    int32_t* dchg_clear;          // dense, per slot: flags of round r+1, zeroed by round r
    int32_t* maze_last_round;     // per slot: last round with a tile visited
    uint8_t* touched;             // per tile id: written since its maze's buffers were last cleared
    int64_t* maze_visits;         // [slot][kSpread]: tile visits
    unsigned long long* total_cells;  // [kSpread], all slots: interior cells of visited tiles (front
                                  // propagation: once per step of 16 layers)
    unsigned long long* maze_reached; // front propagation, [slot][kSpread]: cells reached
    int32_t* maze_layer;          // front propagation, [slot][kSpread]: last layer that reached a cell
    int32_t n_slots;
    int32_t round_id;             // r (wraps; only differences are used); in a graph replay
                                  // the round's offset in the captured group
    const int32_t* round_base;    // graph replays: device counter holding the group's first
                                  // round, added to round_id by the kernels (else null)
    int32_t parity;               // activity buffer read in round r (r mod 2)
    int32_t tile_rows;            // interior rows per tile
    int32_t tile_cols;            // interior columns per tile (64*C - 2T)
    int32_t dense;                // 1 = dense schedule
    uint64_t* posted;             // pinned host memory, [kPosted] by round: round << 32 | count (or null)
    int32_t wave_stride;          // waves in the launch (set by the launch wrapper)
    MazeDev md0;                  // copy of mazes[0] when n_slots == 1 (saves a dependent load)
};

// Sweep variants (layers per visit T, columns per lane C); each is compiled in
// its own translation unit (omap_sweep_variant.hip with OMAP_T, OMAP_C).
#define OMAP_SWEEP_VARIANTS(X) \
    X(4, 4) X(8, 4) X(12, 4) X(16, 4) X(4, 2) X(8, 2) X(12, 2) X(16, 2) X(24, 2) X(32, 2) \
    X(4, 1) X(8, 1) X(12, 1) X(16, 1)

#define X(t, c)                                                                                       \
    hipError_t launch_sweep_T##t##_C##c(const RoundArgs& a, int32_t grid, hipStream_t s, hipEvent_t e0, \
                                        hipEvent_t e1);                                               \
    int sweep_blocks_per_cu_T##t##_C##c();
OMAP_SWEEP_VARIANTS(X)
#undef X

// A round of the front propagation (omap_front.hip), `grid` visiting blocks.
hipError_t launch_front(const RoundArgs& a, int32_t grid, hipStream_t s, hipEvent_t e0 = nullptr,
                        hipEvent_t e1 = nullptr);
int front_blocks_per_cu();

// ---- launch wrappers (omap_kernels.hip) -------------------------------------
hipError_t launch_pack_mask(const uint8_t* occ, const MazeDev& md, uint32_t* mask, hipStream_t s);
hipError_t launch_fill(int32_t* p, int64_t n_elems, int32_t value, hipStream_t s);
// Seed slot's sources (V := K) and schedule their tiles into a.list_out /
// a.count_out / a.flags_out / a.sched_out (the runtime points these at the
// round about to run).
// (src_slot: per-source slots, or nullptr for `slot`)
hipError_t launch_seed(const RoundArgs& a, int32_t slot, const int32_t* src_rc, const int32_t* src_slot,
                       int32_t n_src, int32_t* bad_count, hipStream_t s);
// posted (a word of pinned host memory, or null): the number of sources on
// obstacles, with the tag in the upper 16 bits.  sum: two words, zero before and after.
hipError_t launch_check_sources(const MazeDev& md, const int32_t* src_rc, int32_t n_src, int32_t* sum,
                                uint64_t* posted, uint32_t tag, hipStream_t s);
bool sweep_supported(int T, int C);
// e0 / e1 (optional, both or neither): events that record the kernel's own
// start and end (hipExtLaunchKernel), for profiling.
hipError_t launch_sweep(int T, int C, const RoundArgs& a, int32_t grid, hipStream_t s,
                        hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);

// What a start does before its seeds (k_start).
struct StartArgs {
    const MazeDev* staged;        // descriptors of every slot, copied to mazes_out
    MazeDev* mazes_out;
    const int32_t* sel;           // per slot: 1 = zero its written tiles, 2 = all its tiles
    int32_t tile_begin, n_tiles;  // tile ids to look at
    int32_t* zero;                // words to zero (the schedule's tables)
    int64_t n_zero;
    int32_t n_zero_blocks;        // set by the launch wrapper
    const int32_t* started;       // slots whose counters are reset
    int32_t n_started;
};
hipError_t launch_start(const RoundArgs& a, StartArgs st, hipStream_t s);

// Packing of several mazes' occupancy in one launch.
struct PackJob {
    const uint8_t* occ;
    uint32_t* mask;
    int32_t H, W, mpitch, mrow, mcol;
    int64_t block_begin;   // blocks of the jobs before this one
};
int64_t pack_blocks(int32_t H, int32_t mpitch);   // blocks of a maze's packing
hipError_t launch_pack_mask_many(const PackJob& first, const PackJob* jobs, int32_t n_jobs, int64_t blocks,
                                 hipStream_t s);
hipError_t launch_check_sources_many(const MazeDev* mazes, const int32_t* src_rc, const int32_t* src_slot,
                                     int32_t n, int32_t* bad, hipStream_t s);
// Smallest positive activity and reached count of the touched tiles in
// [tile_begin, tile_end) of the selected slots.
hipError_t launch_reduce(const MazeDev* mazes, const int32_t* tile_maze, const uint8_t* touched,
                         int32_t tile_begin, int32_t tile_end, const int32_t* slot_select, int32_t tile_rows,
                         int32_t tile_cols, int32_t parity, int32_t* maze_min,
                         unsigned long long* maze_reached, hipStream_t s);
hipError_t launch_front_report(const MazeDev* mazes, const unsigned long long* reached, const int32_t* layer,
                               const int32_t* last_round, const int64_t* visits, int32_t n_slots, int32_t* maze_min,
                               unsigned long long* maze_reached, int32_t* last_out, int64_t* visits_out,
                               hipStream_t s);
// Lengths (mazes null: len holds them already) and offsets of the paths.  order
// (optional) receives the targets by path length, longest first; posted (a word
// of pinned host memory, or null) the number of path cells, tagged as above.
// Up to kScanLengths targets the scan's one block computes the lengths too, at
// most four gathers per thread in place of a launch and its gap (5 us).  Above
// kScanOneBlock targets are scanned by many blocks if there is `work`
// (scan_work_bytes(n), 8-byte aligned): the extraction of 4,096 targets takes 9 us
// less (the one block 23 us), of 2,048 10 us, but of 512 3 us more.
constexpr int kScanLengths = 4096, kScanOneBlock = 1024;
size_t scan_work_bytes(int32_t n);
hipError_t launch_lengths_offsets(const MazeDev* mazes, const int32_t* tgt_slot, const int32_t* tgt_rc, int32_t n_tgt,
                                  int32_t parity, int32_t* len, int64_t* offsets, int32_t* order, void* work,
                                  uint64_t* posted, uint32_t tag, hipStream_t s);
// Caller's arrays that a walk copies lengths and offsets to (null: none).
struct WalkOut {
    int32_t* len = nullptr;
    int64_t* off = nullptr;
};
// order (optional): the walk's order of the targets (from launch_lengths_offsets)
// (total: cells of all the paths)
hipError_t launch_walk(const MazeDev* mazes, const int32_t* tgt_slot, const int32_t* tgt_rc,
                       int32_t n_tgt, int32_t parity, const int32_t* len, const int64_t* offsets,
                       int32_t* cells, int64_t total, hipStream_t s, const int32_t* order = nullptr, const WalkOut& out = {});
hipError_t launch_walk_random(const MazeDev* mazes, const int32_t* tgt_slot, const int32_t* tgt_rc,
                              const int32_t* tgt_local, int32_t n_tgt, int32_t parity, uint64_t seed,
                              const int32_t* len, const int64_t* offsets, int32_t* cells, hipStream_t s,
                              const int32_t* order, const WalkOut& out);
// Above these numbers of targets the random-tie and the Euclidean walks take a
// lane per target, below a wave.  The wave's time grows with all the moves, the
// lanes' stays that of the longest path until they fill the chip.  Both forms, us
// for asking and taking the paths of a plan, lane / wave:
//   random     49,152  950 / 863 (empty 1000^2, 227 moves)  861 / 507 (2048^2, 96)
//             131,072 1610 / 2138                          1317 / 1202
//           1,048,576 10.8 / 16.1 ms                        7.4 / 8.7 ms
//   Euclidean  16,384 1887 / 1622                          1665 / 640
//              24,000 1969 / 2190                          1723 / 1129
//              65,536 2328 / 5344                          2150 / 2718
//           1,048,576 19.4 / 80.1 ms                       14.1 / 39.5 ms
// The lines lie where the wave form first loses to a lane per target on either.
constexpr int kRandomLaneTargets = 65536, kEuclidLaneTargets = 20480;
// offsets: cells are written there (the lengths are known); none: the lengths are
// counted, and with cells (stride apart per target) the paths written as well.
hipError_t launch_walk_euclid(const MazeDev* mazes, const int32_t* tgt_slot, const int32_t* tgt_rc, int32_t n_tgt,
                              int32_t parity, int32_t* len, const int64_t* offsets, int32_t* cells, int64_t stride,
                              hipStream_t s, const WalkOut& out);
hipError_t launch_gather_paths(const int32_t* points, int64_t stride, int32_t n_tgt, const int32_t* len,
                               const int64_t* offsets, int32_t* cells, hipStream_t s, const WalkOut& out);
hipError_t launch_source_index(const MazeDev* mazes, const int32_t* tgt_slot, int32_t n_tgt,
                               const int32_t* len, const int64_t* offsets, const int32_t* cells,
                               const int32_t* src_sorted, const int32_t* src_base, const int32_t* src_n,
                               int32_t* out, hipStream_t s);
hipError_t launch_activity(const MazeDev& md, int32_t parity, int32_t offset, int32_t* dst, int64_t dpitch,
                           hipStream_t s);
hipError_t launch_selftest(int32_t* out, hipStream_t s);
// *counter += add (one thread): advances the round counter of graph replays.
hipError_t launch_round_advance(int32_t* counter, int32_t add, hipStream_t s);
int sweep_max_waves_per_cu(int T, int C);

}  // namespace omap

#include "omap.h"

namespace omap {

// Records `message` as the thread's last error (omap_last_error) and returns st.
omap_status_t report_error(omap_status_t st, const char* message);

}  // namespace omap
