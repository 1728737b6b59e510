// Bit-packed front propagation: the layers of the paper on a reached set of
// one bit per cell, kFrontSteps x 16 layers per tile visit.
//
// With d(x) the 8-neighbour step distance from the nearest source, the layer
// output of the paper is A_L(x) = max(0, L + 1 - d(x)) (Sec. Methods; the
// closed form is what the tests pin), and the integer sweeps hold it as
// V = K - d.  Here the state is the reached set R_n = {x : d(x) <= n}:
// R_0 = sources and R_{n+1} = free AND dilate3x3(R_n).  A cell entering R at
// layer n gets V = K - n written once (activity buffer 0), so V is exactly
// what the integer sweeps produce and everything after propagation is shared.
//
// Layer numbers must be exact, so every visited tile of a maze advances the
// same T layers per round (round r of a maze covers layers (r - round0) T + 1
// .. + T) from ping-pong bit planes.
//
// Layout.  Planes and masks are strip-major: the 32-cell words of one 32-column
// strip are contiguous down the rows (word (r, j) at j * mcol + r), so that a
// wave whose lanes are rows loads 64 words with one contiguous access.  A
// lane holds one row of the tile's region, its words in registers: horizontal
// neighbours are funnel shifts between a lane's words, vertical ones DPP moves
// between lanes, and a layer costs 6 VALU operations per word of 32 cells.
//
// A visit.  The block loads the tile's region (64 x 64 cells and a halo of T
// on every side) into LDS once and runs kFrontSteps steps of 16 layers on it.
// In step k wave g takes the 64 rows from 16 k + 32 g, applies 16 layers in
// registers and returns the middle 32 rows, which are exact, to the other LDS
// buffer; after the last step exactly the tile's 64 rows are left.  A wave whose
// rows gain no cell in the first layer has nothing to do in any (its rows are
// settled, and nothing outside them comes near its middle rows in 16 layers);
// if no wave gains a cell the visit is over.  A wave that gains cells in some of
// its words only advances those and the words beside them: three, four or six of
// the six (26,000^2 with 5000 sources 8.49 -> 8.23 ms of propagation, 512 mazes
// 3.62 -> 3.30, 2000^2 dense 0.665 -> 0.613, 23170^2 1.62 -> 1.525).
//
// The registers of the 16 layers of the tile's own words form a unary code of
// each cell's arrival, turned into 4 bit planes by 11 selects per word; the
// planes and arrivals of the visit are kept in LDS, and at the end the waves
// write the activity from them, four columns a lane.
//
// Dense schedule: every tile of a maze that changed in the round before, no
// lists and no claims; a tile that gained a cell flags its maze.
//
// Scheduling.  A cell reached before the last layer of a round has all its free
// neighbours reached by the end of the round, so only cells reached in
// the last layer are a front that moves on: a tile with such a cell schedules
// its 3 x 3 tiles (T <= 64 layers reach no further).  A tile that gained any cell
// schedules itself: its next visit brings the other plane up to date, so
// that both planes of an unvisited tile are equal.
//
// What bounds it: on one large maze the chain of rounds (launch gap, list and
// region loads, four steps, claims), 64 layers per round instead of 16 of the
// two-wave integer visit it replaced: 12 us a round; a pass over a 23170^2 map
// (load, propagate with L* = 7124, 4096 paths) 6.4 -> 2.3 ms, over 4096^2 corridors
// (L* = 11,178) 12.4 -> 2.9, of which propagation 1.53 and 2.19.
// With fronts everywhere (26,000^2, 5000 sources, 650 layers) VALU issue, 51 % of
// the cycles: 485,000 visits of 5,000 VALU and 1,900 scalar instructions; the
// whole pass 67.7 -> 9.7 ms.  The dense schedule on 2000^2 (1,024 tiles a round on
// 768 resident blocks: two visits one after another) is latency again, 16 to 21 us
// a round with VALU issue in 13 % of the cycles.  A lone visit takes 10 us: list
// entry 0.9, region 0.6, steps 2.1 + 1.7 + 1.3 + 1.2, claims and activity 1.3, and
// 1.6 us pass before the next round's first wave.  Tiles of 64 x 128 cells take a third fewer operations
// per cell but 3 us longer per visit: 26,000^2 propagation 9.0 against 8.6 ms at the
// time, corridors 2.85 against 2.30; 32 layers a round take half the operations per
// layer but twice the visits: 11.3 against 8.5, corridors 2.79 against 2.21, and
// only 512 mazes gain, 3.41 against 3.55.  Against the earlier bit-sliced sweep (one
// row of 1984 columns per wave, 8 layers per visit, a per-lane loop to write
// activity) a batch of 512 mazes takes 7.7 instead of 21.6 ms.
#pragma once

#include <type_traits>

#include "omap_sweep.h"

namespace omap {

constexpr int kFrontRows = 64;                       // tile rows
constexpr int kFrontWords = kFrontCols / 32;         // tile words per row
constexpr int kFrontHaloRows = kFrontLayers;
constexpr int kFrontHaloWords = (kFrontLayers + 31) / 32;
constexpr int kFrontRegionRows = kFrontRows + 2 * kFrontHaloRows;
constexpr int kFrontRegionWords = kFrontWords + 2 * kFrontHaloWords;
constexpr int kFrontGroups = (kFrontRegionRows - 32) / 32;   // waves with rows in step 0
// (4096^2 corridors, propagation: 8 waves 2.55 ms, 6: 2.77, 5: 3.03)
constexpr int kFrontWaves = 8;
constexpr int kFrontThreads = kFrontWaves * kLanes;
static_assert(kFrontRows == kFrontTileRows && kFrontRegionRows % 64 == 0 && kFrontGroups <= kFrontWaves, "front tile");
static_assert(kFrontLayers <= kFrontRows && kFrontLayers <= kFrontCols, "a front reaches the next tiles only");

struct FrontShared {
    uint32_t r[2][kFrontRegionWords][kFrontRegionRows];   // reached, double-buffered over the steps
    uint32_t f[kFrontRegionWords][kFrontRegionRows];      // free
    // per word of the tile: the layer of arrival within the visit as 6 bit planes
    // (lo: the 4 within a step, hi.x, hi.y: the step's) and the cells that
    // arrived in the visit (hi.z)
    uint4 lo[kFrontRows][kFrontWords], hi[kFrontRows][kFrontWords];
    int32_t active[kFrontSteps];                          // some wave gained a cell in step k
    int32_t last;                                         // a cell of the tile arrived in the last layer
};

// Keeps the compiler's scheduler from moving instructions across this point.
// A dependent VALU instruction issues 8 cycles after the one before it, an
// independent one after 4 (measured, one wave on its SIMD), so a layer is
// written as runs of independent instructions and kept that way: left to
// itself the scheduler puts each funnel shift next to the OR that uses it.
__device__ __forceinline__ void keep_order() { __builtin_amdgcn_sched_barrier(0); }

// One layer of NW words per lane: r = free AND dilate(r).
template <int NW>
__device__ __forceinline__ void front_layer(uint32_t (&r)[NW], const uint32_t (&f)[NW]) {
    uint32_t left[NW], right[NW], up[NW], h[NW];
    keep_order();
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        // column c sees c-1 (bit c-1, or bit 31 of the word to the left) and c+1
        left[w] = w > 0 ? __builtin_amdgcn_alignbit(r[w], r[w > 0 ? w - 1 : 0], 31) : r[w] << 1;
        right[w] = w + 1 < NW ? __builtin_amdgcn_alignbit(r[w + 1 < NW ? w + 1 : w], r[w], 1) : r[w] >> 1;
    }
    keep_order();
#pragma unroll
    for (int w = 0; w < NW; ++w) h[w] = r[w] | left[w] | right[w];
    keep_order();
#pragma unroll
    for (int w = 0; w < NW; ++w) up[w] = (uint32_t)from_left_lane((int)h[w]);   // the row above is the lane below
    keep_order();
#pragma unroll
    for (int w = 0; w < NW; ++w) up[w] |= (uint32_t)from_right_lane((int)h[w]);
    keep_order();
#pragma unroll
    for (int w = 0; w < NW; ++w) r[w] = (h[w] | up[w]) & f[w];
    keep_order();
}

// m ? a : b, bit by bit.
__device__ __forceinline__ uint32_t bit_select(uint32_t m, uint32_t a, uint32_t b) { return (a & m) | (b & ~m); }

template <int N>
constexpr std::integral_constant<int, N> at{};

// Step k of a visit, rows 16 k + 32 g .. + 63 and words W0 .. W0 + NW - 1 of
// the region (one wave).  Of the tile's words it takes OWN from T0 on (their
// arrivals, and in the last step their sets alone).
template <int W0, int NW, int T0, int OWN, bool LAST>
__device__ __forceinline__ void front_step(FrontShared& sh, int k, int g, int lane) {
    constexpr int C0 = kFrontHaloWords + T0 - W0;   // the first of them among the lane's
    constexpr int S0 = LAST ? C0 : 0, S1 = LAST ? C0 + OWN : NW;   // words stored
    const int row = 16 * k + 32 * g + lane;
    const int cur = k & 1;
    uint32_t r[NW], f[NW], first[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        first[w] = r[w] = sh.r[cur][W0 + w][row];
        f[w] = sh.f[W0 + w][row];
    }
    front_layer<NW>(r, f);
    uint32_t gain = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) gain |= r[w] ^ first[w];
    const bool mid = lane >= 16 && lane < 48;
    if (__ballot(gain != 0) == 0) {
        if (mid) {
#pragma unroll
            for (int w = S0; w < S1; ++w) sh.r[cur ^ 1][W0 + w][row] = r[w];
        }
        return;
    }
    if (lane == 0) sh.active[k] = 1;
    // The arrivals of 8 layers are coded at a time (fewer registers): after
    // layers 1 .. 8 of a half, in4 = in the set after 4, in2 = after 2 or 6 by
    // in4, in1 = after 1, 3, 5 or 7 by both.
    uint32_t in8[OWN], in4[2][OWN] = {}, in2[2][OWN] = {}, in1[2][OWN] = {}, before[OWN];
    // layers 2 .. 16 on words S .. S + N - 1 of the wave's (rolled over the halves:
    // the code is two thirds as long, and a short propagation fetches it cold)
    auto layers = [&](auto s_, auto n_) {
        constexpr int S = decltype(s_)::value, N = decltype(n_)::value;
        uint32_t q[N], e[N];
#pragma unroll
        for (int w = 0; w < N; ++w) {
            q[w] = r[S + w];
            e[w] = f[S + w];
        }
        // (a word of the tile outside S .. keeps its cells)
        auto own_word = [&](int c) {
            return C0 + c >= S && C0 + c < S + N ? q[C0 + c >= S && C0 + c < S + N ? C0 + c - S : 0] : r[C0 + c];
        };
#pragma unroll 1
        for (int half = 0; half < 2; ++half) {
#pragma unroll
            for (int c = 0; c < OWN; ++c) {
                in8[c] = own_word(c);
                in4[0][c] = in4[1][c];
                in2[0][c] = in2[1][c];
                in1[0][c] = in1[1][c];
            }
            uint32_t h[7][OWN];
#pragma unroll
            for (int j = 0; j < 7; ++j) {
                if (j != 0 || half != 0) front_layer<N>(q, e);
#pragma unroll
                for (int c = 0; c < OWN; ++c) h[j][c] = own_word(c);
            }
            front_layer<N>(q, e);
#pragma unroll
            for (int c = 0; c < OWN; ++c) {
                in4[1][c] = h[3][c];
                in2[1][c] = bit_select(h[3][c], h[1][c], h[5][c]);
                in1[1][c] = bit_select(in2[1][c], bit_select(h[3][c], h[0][c], h[4][c]),
                                       bit_select(h[3][c], h[2][c], h[6][c]));
                before[c] = h[6][c];
                // (or the compiler moves the selects down to their use and keeps every h)
                asm volatile("" : "+v"(in4[1][c]), "+v"(in2[1][c]), "+v"(in1[1][c]));
            }
        }
#pragma unroll
        for (int w = 0; w < N; ++w) r[S + w] = q[w];
    };
    // A cell that arrives in these layers lies within 15 columns of one that
    // arrived in the first, so only the words that gained a cell and the next ones
    // are advanced (the others hold what the layers would leave).
    if constexpr (NW == 6) {
        const uint32_t g01 = (r[0] ^ first[0]) | (r[1] ^ first[1]), g45 = (r[4] ^ first[4]) | (r[5] ^ first[5]);
        const uint32_t g2 = r[2] ^ first[2], g3 = r[3] ^ first[3];
        if (__ballot((g45 | g3) != 0) == 0) {
            if (__ballot(g2 != 0) == 0) layers(at<0>, at<3>);
            else layers(at<0>, at<4>);
        } else if (__ballot((g01 | g2) != 0) == 0) {
            if (__ballot(g3 != 0) == 0) layers(at<3>, at<3>);
            else layers(at<2>, at<4>);
        } else if (__ballot((g01 | g45) != 0) == 0) {
            layers(at<1>, at<4>);
        } else {
            layers(at<0>, at<6>);
        }
    } else if constexpr (NW == 4) {
        if (__ballot(((r[2] ^ first[2]) | (r[3] ^ first[3])) != 0) == 0) layers(at<0>, at<3>);
        else if (__ballot(((r[0] ^ first[0]) | (r[1] ^ first[1])) != 0) == 0) layers(at<1>, at<3>);
        else layers(at<0>, at<4>);
    } else {
        layers(at<0>, at<NW>);
    }
    if (mid) {
#pragma unroll
        for (int w = S0; w < S1; ++w) sh.r[cur ^ 1][W0 + w][row] = r[w];
    }
    const int ti = row - kFrontHaloRows;   // row of the tile
    const bool own = mid && ti >= 0 && ti < kFrontRows;
    uint32_t fresh[OWN], any = 0, lastb = 0;
#pragma unroll
    for (int c = 0; c < OWN; ++c) {
        fresh[c] = own ? r[C0 + c] & ~first[C0 + c] : 0u;
        any |= fresh[c];
        lastb |= fresh[c] & ~before[c];
    }
    if (__ballot(any != 0) == 0) return;
    if (LAST && __ballot(lastb != 0) != 0 && lane == 0) sh.last = 1;
    if (!own) return;
    // (one lane owns each word; the steps are separated by barriers)
#pragma unroll
    for (int c = 0; c < OWN; ++c) {
        uint4 lo = sh.lo[ti][T0 + c], hi = sh.hi[ti][T0 + c];
        lo.x |= fresh[c] & ~bit_select(in8[c], in1[0][c], in1[1][c]);
        lo.y |= fresh[c] & ~bit_select(in8[c], in2[0][c], in2[1][c]);
        lo.z |= fresh[c] & ~bit_select(in8[c], in4[0][c], in4[1][c]);
        lo.w |= fresh[c] & ~in8[c];
        hi.x |= k & 1 ? fresh[c] : 0u;
        hi.y |= k & 2 ? fresh[c] : 0u;
        hi.z |= fresh[c];
        sh.lo[ti][T0 + c] = lo;
        sh.hi[ti][T0 + c] = hi;
    }
}

// lt / tiles_x for 0 <= lt < 2^31: the product with the rounded-down reciprocal
// is the quotient or one less.
__device__ __forceinline__ int front_tile_row(const MazeDev& md, int lt) {
    const int q = (int)(((uint64_t)(uint32_t)lt * md.tiles_x_inv) >> 32);
    return q + (lt - q * md.tiles_x >= md.tiles_x);
}

// One round: T = kFrontLayers layers of every listed tile.  ONE: a single maze,
// described in the arguments (copying either description into one variable
// kept both in scalar registers, and their spills cost 0.9 us of a round).
// (6 waves per SIMD: at most 80 registers, three blocks to a CU instead of two;
// 512-maze batch 9.55 -> 9.15 ms, 23170^2 propagation 1.76 -> 1.67)
template <bool ONE, bool DENSE>
__global__ __launch_bounds__(kFrontThreads) __attribute__((amdgpu_waves_per_eu(6))) void k_front(RoundArgs a) {
    // first list entry and count issued before anything else (see k_sweep)
    int i = (int)blockIdx.x - 1;   // block 0: the accounting block
    const int ie = i >= 0 && i < a.n_tile_ids ? i : 0;
    uint64_t e = __hip_atomic_load(reinterpret_cast<const uint64_t*>(a.list_in + 2 * ie), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
    const int cnt = __hip_atomic_load(a.count_in, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    // the arguments are read while those loads are in flight, all together (left
    // to the compiler, their loads are issued and waited for in four groups
    // after the list entry arrived: 0.7 us)
    if (ONE)
        asm volatile("" ::"s"(a.md0.mask), "s"(a.md0.R[0]), "s"(a.md0.R[1]), "s"(a.md0.H), "s"(a.md0.mpitch),
                     "s"(a.md0.mcol), "s"(a.md0.tiles_x), "s"(a.md0.tiles_x_inv), "s"(a.md0.tile_base), "s"(a.md0.K),
                     "s"(a.md0.round0), "s"(a.parity), "s"(a.round_id), "s"(a.flags_in), "s"(a.maze_last_round),
                     "s"(a.wave_stride), "s"(a.md0.V[0]), "s"(a.md0.pitch), "s"(a.md0.W), "s"(a.total_cells),
                     "s"(a.maze_reached), "s"(a.maze_layer), "s"(a.touched));
    else
        asm volatile("" ::"s"(a.mazes), "s"(a.parity), "s"(a.round_id), "s"(a.flags_in), "s"(a.maze_last_round),
                     "s"(a.wave_stride));
    if (a.round_base) a.round_id += *a.round_base;
    if (blockIdx.x == 0) {
        round_accounting<kFrontLayers, kFrontThreads>(a);
        return;
    }
    __shared__ FrontShared sh;
    constexpr int RR = kFrontRegionRows, RW = kFrontRegionWords;
    const int stride = a.wave_stride;
    const int n = DENSE ? a.n_tile_ids : __builtin_amdgcn_readfirstlane(cnt);
    for (; i < n; i += stride) {
        if (DENSE) {
            const int s = a.tile_maze[i];
            if (s < 0 || __builtin_amdgcn_readfirstlane(a.dchg_prev[s]) == 0) continue;
            e = (uint64_t)(uint32_t)s << 32 | (uint32_t)i;
        }
        // (opaque to the compiler, which would otherwise compute everything that
        // depends on these alone before the loop, ahead of the first visit's loads)
        int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = lane_id(), round = a.round_id;
        asm volatile("" : "+s"(wave), "+v"(lane), "+s"(round));
        const int tid = wave * kLanes + lane;
        const int g = __builtin_amdgcn_readfirstlane((int)(uint32_t)e);
        const int slot = __builtin_amdgcn_readfirstlane((int)(uint32_t)(e >> 32));
        const MazeDev& md = ONE ? a.md0 : a.mazes[slot];
        const int lt = g - md.tile_base;
        const int ty = front_tile_row(md, lt), tx = lt - ty * md.tiles_x;
        const int r0 = ty * kFrontRows, j0 = tx * kFrontWords;
        const uint32_t* Rin = a.parity ? md.R[1] : md.R[0];
        uint32_t* Rout = a.parity ? md.R[0] : md.R[1];
        // ---- load the region: wave w takes word w, every row; all loads are issued
        // before the first is used.  A strip is addressed through a buffer resource
        // over its rows near the tile: rows outside the maze (a negative offset is a
        // large unsigned one) and words outside it (an empty resource) read 0.
        static_assert(RW < kFrontWaves && RR % kLanes == 0, "a wave per word of the region");
        constexpr int kPer = RR / kLanes;
        uint32_t vr[kPer], vm[kPer];
        const int row0 = max(r0 - kFrontHaloRows, 0), row_off = r0 - kFrontHaloRows - row0 + lane;
        const int j = j0 - kFrontHaloWords + wave;
        const bool word_ok = wave < RW && j >= 0 && j < md.mpitch;
        if (wave < RW) {
            const int64_t x = word_ok ? (int64_t)j * md.mcol + row0 : 0;
            const int bytes = word_ok ? 4 * min(md.H - row0, RR) : 0;
            const __amdgpu_buffer_rsrc_t br = raw_rsrc(Rin + x, bytes), bm = raw_rsrc(md.mask + x, bytes);
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                vr[q] = (uint32_t)bload<1>(br, 4 * (row_off + q * kLanes), 0)[0];
                vm[q] = (uint32_t)bload<1>(bm, 4 * (row_off + q * kLanes), 0)[0];
            }
        }
        if (!DENSE && i + stride < n) e = *reinterpret_cast<const uint64_t*>(a.list_in + 2 * (i + stride));
        const int64_t n0 = (int64_t)(round - md.round0) * kFrontLayers;   // layers done before this round
        const int64_t left = (int64_t)md.K - 1 - n0;                      // layers the maze still has
        if (left <= 0) {   // every layer below K is done
            if (!DENSE && tid == 0) a.flags_in[g] = 0;
            continue;
        }
        if (tid == 0) {   // (the touched flag is set by a tile that gained a cell)
            if (DENSE)
                atomicAdd(reinterpret_cast<unsigned long long*>(
                              &a.maze_visits[slot * kSpread + (blockIdx.x & (kSpread - 1))]), 1ull);
            else
                a.flags_in[g] = 0;
            a.maze_last_round[slot] = round;
        }
        for (int t = tid; t < kFrontWords * kFrontRows; t += kFrontThreads)
            (&sh.lo[0][0])[t] = (&sh.hi[0][0])[t] = make_uint4(0, 0, 0, 0);
        if (tid < kFrontSteps) sh.active[tid] = 0;
        if (tid == 0) sh.last = 0;
        if (wave < RW) {
#pragma unroll
            for (int q = 0; q < kPer; ++q) {
                const int row = row_off + row0 + q * kLanes;
                sh.r[0][wave][q * kLanes + lane] = vr[q];
                // guard bits (columns >= W) are obstacles, so is all outside the maze
                sh.f[wave][q * kLanes + lane] = word_ok && row >= 0 && row < md.H ? ~vm[q] : 0u;
            }
        }
        lds_barrier();
        // ---- the steps
        int fin = 0;   // buffer holding the tile's reached set
        int k = 0;
        for (; k < kFrontSteps; ++k) {
            // the last 32 layers need the words next to the tile only; the last step
            // is split by the tile's words too (its rows take two waves, the
            // block's other SIMDs would idle)
            constexpr int H = kFrontHaloWords, NW = kFrontWords, HALF = NW / 2;
            static_assert(H == 2 && NW % 2 == 0 && kFrontSteps == 4, "words of a step");
            if (k < kFrontSteps - 2) {
                if (wave < kFrontGroups - k) front_step<0, RW, 0, NW, false>(sh, k, wave, lane);
            } else if (k < kFrontSteps - 1) {
                if (wave < kFrontGroups - k) front_step<H - 1, NW + 2, 0, NW, false>(sh, k, wave, lane);
            } else {
                if (wave < 2) front_step<H - 1, HALF + 2, 0, HALF, true>(sh, k, wave, lane);
                else if (wave < 4) front_step<H - 1 + HALF, HALF + 2, HALF, HALF, true>(sh, k, wave - 2, lane);
            }
            lds_barrier();
            if (sh.active[k] == 0) break;   // nothing moves any more
            fin ^= 1;
        }
        // ---- the last wave schedules the next round (a chain of two atomics, so
        // that is all it does), waves 0 .. kFrontWords-1 store the reached set
        // and count, and they and the others write activity rows
        const int base_v = md.K - 1 - (int)n0;
        const int limit = left < kFrontLayers ? (int)left : kFrontLayers;
        if (wave < kFrontWords) {
            const uint32_t rf = sh.r[fin][kFrontHaloWords + wave][kFrontHaloRows + lane];
            const uint4 lo = sh.lo[lane][wave], hi = sh.hi[lane][wave];
            const uint32_t plane[6] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y};
            uint32_t fr = hi.z;
            if (limit < kFrontLayers) {   // cells past the maze's last layer do not count
                uint32_t less = 0, same = fr;
#pragma unroll
                for (int b = 5; b >= 0; --b) {
                    if ((limit >> b) & 1) {
                        less |= same & ~plane[b];
                        same &= plane[b];
                    } else {
                        same &= ~plane[b];
                    }
                }
                fr = less;
            }
            if (r0 + lane < md.H && j0 + wave < md.mpitch)
                Rout[(int64_t)(j0 + wave) * md.mcol + r0 + lane] = rf & ~(hi.z & ~fr);
            const int sp = blockIdx.x & (kSpread - 1);
            if (wave == 0 && lane == 0 && k > 0)   // 16 layers of the tile's cells per step that moved
                atomicAdd(a.total_cells + sp, (unsigned long long)(k * tile_cells(md, ty, tx, kFrontRows, kFrontCols)));
            if (__ballot(fr != 0) != 0) {
                int top = 0;   // the latest arrival among the counted cells
                uint32_t m = fr;
#pragma unroll
                for (int b = 5; b >= 0; --b) {
                    if (__ballot((m & plane[b]) != 0) != 0) {
                        top |= 1 << b;
                        m &= plane[b];
                    }
                }
                int count = __popc(fr);
                for (int o = kLanes / 2; o > 0; o >>= 1) count += __shfl_xor(count, o);
                if (lane == 0) {
                    atomicAdd(&a.maze_reached[slot * kSpread + sp], (unsigned long long)count);
                    atomicMax(&a.maze_layer[slot * kSpread + sp], (int)n0 + top + 1);
                    a.touched[g] = 1;
                }
            }
        }
        if (wave == kFrontWaves - 1) {
            if (left > kFrontLayers) {
                uint32_t fr = 0;
#pragma unroll
                for (int c = 0; c < kFrontWords; ++c) fr |= sh.hi[lane][c].z;
                const bool last = sh.last != 0;
                if (DENSE) {
                    if (__ballot(fr != 0) != 0 && lane == 0) {
                        a.dchg_cur[slot] = 1;
                        *a.count_out = 1;
                    }
                } else if (__ballot(fr != 0) != 0) {
                    const int ny = ty + lane / 3 - 1, nx = tx + lane % 3 - 1;
                    const int gn = md.tile_base + ny * md.tiles_x + nx;
                    bool won = false;
                    if ((lane == 4 || (last && lane < 9)) && ny >= 0 && ny < md.tiles_y && nx >= 0 && nx < md.tiles_x)
                        won = atomicExch(&a.flags_out[gn], 1) == 0;
                    const uint64_t wmask = __ballot(won);
                    const int nwon = __popcll(wmask);
                    if (nwon > 0) {
                        int base = 0;
                        if (lane == 0) base = atomicAdd(a.count_out, nwon);
                        base = __builtin_amdgcn_readfirstlane(base);
                        if (won) {
                            const int q = base + __popcll(wmask & ((1ull << lane) - 1));
                            a.list_out[2 * q] = gn;
                            a.list_out[2 * q + 1] = slot;
                        }
                        if (!ONE && lane == 0) atomicAdd(&a.sched_out[slot], nwon);
                    }
                }
            }
            lds_barrier();   // the block's LDS is reused by the next tile
            continue;
        }
        // activity: 4 columns a lane.  A nibble of each plane is spread to a bit per
        // byte by a multiplication, so the 4 arrivals are the bytes of one word.
        constexpr int kQuads = kFrontCols / 4, kRowsAtOnce = kLanes / kQuads, kTimes = kFrontRows / kRowsAtOnce;
        const int c = (lane % kQuads) >> 3, b = 4 * (lane & 7);
        int32_t* const V = md.V[0] + (int64_t)r0 * md.pitch + j0 * 32 + 4 * (lane % kQuads);
        // (waves 0 .. kFrontWords-1 have had their part: they take the last rows)
        constexpr int kHelp = kFrontWords, kWriters = kFrontWaves - 1 - kHelp, kRest = kTimes * kHelp / (kHelp + 2 * kWriters);
        const bool helper = wave < kHelp;
        int it = helper ? kTimes - kRest + wave : wave - kHelp;
        const int it_end = helper ? kTimes : kTimes - kRest, it_step = helper ? kHelp : kWriters;
        for (; it < it_end; it += it_step) {
            const int row = it * kRowsAtOnce + lane / kQuads;
            const uint4 hi = sh.hi[row][c];
            uint32_t here = (hi.z >> b) & 15u;
            if (__ballot(here != 0) == 0) continue;
            const uint4 lo = sh.lo[row][c];
            auto spread = [&](uint32_t plane) { return __umul24((plane >> b) & 15u, 0x204081u) & 0x01010101u; };
            const uint32_t t = spread(lo.x) | spread(lo.y) << 1 | spread(lo.z) << 2 | spread(lo.w) << 3 |
                               spread(hi.x) << 4 | spread(hi.y) << 5;
            const int t0 = (int)(t & 0xff), t1 = (int)(t >> 8 & 0xff), t2 = (int)(t >> 16 & 0xff), t3 = (int)(t >> 24);
            if (limit < kFrontLayers)
                here &= (uint32_t)(t0 < limit) | (uint32_t)(t1 < limit) << 1 | (uint32_t)(t2 < limit) << 2 |
                        (uint32_t)(t3 < limit) << 3;
            int32_t* const q = V + (int64_t)row * md.pitch;
            if (here == 15u) {
                *(__attribute__((address_space(1))) v4i32*)q = v4i32{base_v - t0, base_v - t1, base_v - t2, base_v - t3};
            } else {
                if (here & 1u) q[0] = base_v - t0;
                if (here & 2u) q[1] = base_v - t1;
                if (here & 4u) q[2] = base_v - t2;
                if (here & 8u) q[3] = base_v - t3;
            }
        }
        lds_barrier();   // the block's LDS is reused by the next tile
    }
}

}  // namespace omap
