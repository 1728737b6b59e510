// Device kernels of the oMAP planner for gfx950 (CDNA4, wave64) other than
// the tile sweeps (omap_sweep.h): ingest, seeding, reset, the run-time layer
// count, path lengths and walks, copy-out; and the launch wrappers, which
// dispatch the sweeps to the per-variant launch functions.

#include "omap_sweep.h"

namespace omap {

// ---------------------------------------------------------------------------
// ingest: occupancy bytes -> obstacle bit mask
// ---------------------------------------------------------------------------

// A block packs 1,024 words, as many rows as the maze's width and height make
// sensible (pack_rows: 32 rows x 1024 columns of most mazes).  A lane reads 16 bytes
// with every load issued before the first is used, turns each byte into a bit
// (nonzero bytes to 0x01, four of them to a nibble by a dot product with 1, 2, 4, 8)
// and two lanes' bits into a word; the block's words go through LDS to the mask's
// layout, contiguous down a strip or along a row.  One job per maze, blocks in job
// order.  Bound by the read of the occupancy: 3.8 TB/s on 26,000^2 cells (0.179 ms)
// and 4.0 on 23,170^2 (0.133); a thread per word, 32 byte loads each, took 0.19 ms.
// 512 mazes of up to 2,048^2 cells take 0.095 ms; with a thread per word, each
// searching its job, 0.46.
constexpr int kPackWords = 1024, kPackThreads = 256, kPackGrid = 65536;
typedef uint32_t v4u32_bytes __attribute__((ext_vector_type(4), aligned(1)));

// Log2 of the rows a block packs: its 1,024 words are as wide as the maze up to 32
// words, and wider only where the maze has fewer than 32 rows (blocks of 32 x 32
// words left most lanes without a column: loading 4,000,000 x 8 cells 196 us, now 74;
// with a thread per word 100).
__host__ __device__ __forceinline__ int pack_rows_log2(int32_t H, int32_t mpitch) {
    int rows = 10;
    while (rows > 5 && mpitch > kPackWords >> rows) --rows;
    while (rows > 0 && H <= 1 << (rows - 1)) --rows;
    return rows;
}

// SQUARE: 32 rows x 32 words, known when compiled (2,048^2 cells 3.8 us, else 4.4).
template <bool SQUARE>
__global__ __launch_bounds__(kPackThreads) void k_pack_mask(PackJob one, const PackJob* __restrict__ jobs,
                                                            int32_t n_jobs, int64_t blocks) {
    __shared__ uint32_t tile[2 * kPackWords];   // word w of row r at w * (rows + 1) + r
    const int t = threadIdx.x, wave = t >> 6, lane = lane_id();
    for (int64_t q = blockIdx.x; q < blocks; q += gridDim.x) {
        PackJob jb = one;
        if (n_jobs > 1) {
            int lo = 0, hi = n_jobs;   // the last job with block_begin <= q, 64 looked at at a time
            while (hi - lo > 1) {
                const int step = (hi - lo + kLanes - 1) / kLanes, j = lo + lane_id() * step;
                const int below = __popcll(__ballot(j < hi && jobs[min(j, n_jobs - 1)].block_begin <= q));
                lo += (below - 1) * step;
                hi = min(hi, lo + step);
            }
            jb = jobs[lo];
        }
        const int log_rows = SQUARE ? 5 : pack_rows_log2(jb.H, jb.mpitch), log_words = 10 - log_rows;
        const int rows = 1 << log_rows, words = 1 << log_words;
        const int32_t col_tiles = (jb.mpitch + words - 1) >> log_words;
        const int64_t b = q - jb.block_begin;
        const int32_t rt = (int32_t)(b / col_tiles), ct = (int32_t)(b - (int64_t)rt * col_tiles);
        const int64_t row0 = (int64_t)rt << log_rows;
        const int32_t w0 = ct << log_words;
        const auto occ = (const __attribute__((address_space(1))) uint8_t*)jb.occ;
        if (jb.W < 16) {   // narrower than a lane's load; columns past the row are obstacles
            for (int u = t; u < kPackWords; u += kPackThreads) {
                const int w = u >> log_rows, r = u & (rows - 1);
                uint32_t word = ~0u;
                if (w0 + w == 0) {
                    const int64_t at = min(row0 + r, (int64_t)jb.H - 1) * jb.W;
                    for (int e = 0; e < jb.W; ++e)
                        if (occ[at + e] == 0) word &= ~(1u << e);
                }
                tile[w * (rows + 1) + r] = word;
            }
        } else {
            // half words of the tile, row by row, 512 a wave (a lane past the row's last 16
            // bytes reads those and shifts its bits)
            constexpr int kPer = 2 * kPackWords / kPackThreads;
            v4u32_bytes v[kPer];
            int32_t past[kPer];
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int u = kLanes * (kPer * wave + k) + lane;
                const int32_t c = 16 * min(2 * w0 + (u & (2 * words - 1)), 2 * jb.mpitch - 1), at = min(c, jb.W - 16);
                const int64_t r = min(row0 + (u >> (log_words + 1)), (int64_t)jb.H - 1);
                past[k] = min(c - at, 16);
                v[k] = *(const __attribute__((address_space(1))) v4u32_bytes*)(occ + r * jb.W + at);
            }
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                uint32_t bits = 0;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    uint32_t y[2];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const uint32_t x = v[k][2 * h + e];
                        y[e] = ((((x & 0x7f7f7f7fu) + 0x7f7f7f7fu) | x) >> 7) & 0x01010101u;
                    }
                    const uint32_t low = __builtin_amdgcn_udot4(y[0], 0x08040201u, 0, false);
                    bits |= __builtin_amdgcn_udot4(y[1], 0x80402010u, low, false) << (8 * h);
                }
                bits = (bits | 0xffff0000u) >> past[k] & 0xffffu;
                const uint32_t next = (uint32_t)__builtin_amdgcn_mov_dpp((int)bits, 0xF5, 0xF, 0xF, true);   // quad_perm [1, 1, 3, 3]
                const int u = kLanes * (kPer * wave + k) + lane;
                if ((t & 1) == 0) tile[((u & (2 * words - 1)) >> 1) * (rows + 1) + (u >> (log_words + 1))] = bits | next << 16;
            }
        }
        __syncthreads();
        const bool strips = jb.mrow == 1;
        for (int u = t; u < kPackWords; u += kPackThreads) {
            const int w = strips ? u >> log_rows : u & (words - 1), r = strips ? u & (rows - 1) : u >> log_words;
            if (w0 + w < jb.mpitch && row0 + r < jb.H)
                jb.mask[(row0 + r) * jb.mrow + (int64_t)(w0 + w) * jb.mcol] = tile[w * (rows + 1) + r];
        }
        __syncthreads();   // the next tile overwrites the words
    }
}

// p[0 .. n) := value (int4 stores, then the last n mod 4 elements).
__global__ void k_fill(int32_t* __restrict__ p, int64_t n, int32_t value) {
    const int64_t n4 = n / 4;
    int4 v = make_int4(value, value, value, value);
    int4* q = reinterpret_cast<int4*>(p);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4;
         i += (int64_t)gridDim.x * blockDim.x)
        q[i] = v;
    if (blockIdx.x == 0 && threadIdx.x < (unsigned)(n - 4 * n4)) p[4 * n4 + threadIdx.x] = value;
}

// Index of the mask (or plane) word holding cell (r, c).
__device__ __forceinline__ int64_t mask_word(const MazeDev& md, int32_t r, int32_t c) {
    return (int64_t)r * md.mrow + (int64_t)(c >> 5) * md.mcol;
}

// Stores a value below 2^48 with its tag in one word of pinned host memory (one
// thread; `posted` null: nothing).  What was enqueued before this kernel is done
// by then.
__device__ __forceinline__ void post(uint64_t* posted, uint64_t value, uint32_t tag) {
    if (posted != nullptr)
        __hip_atomic_store(posted, (uint64_t)tag << 48 | value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Posts the number of sources on obstacles.  Each block counts its sources; of
// several, the last to finish posts the sum and leaves sum[0] (bad sources) and
// sum[1] (blocks done) zero for the next time (one check at a time per handle).
// One block for any number took 0.28 ms for 200,000 sources; a block per 1,024 of
// 2,000,000 took 48 us, most of it their additions to the same words (13 ns each), now 23.
constexpr int kCheckBlock = 1024, kCheckGrid = 256;

__global__ __launch_bounds__(kCheckBlock) void k_check_sources(MazeDev md, const int32_t* __restrict__ src, int32_t n,
                                                               int32_t* sum, uint64_t* posted, uint32_t tag) {
    __shared__ int bad;
    if (threadIdx.x == 0) bad = 0;
    __syncthreads();
    int mine = 0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t r = src[2 * i], c = src[2 * i + 1];
        mine += (md.mask[mask_word(md, r, c)] >> (c & 31)) & 1u;
    }
    if (mine) atomicAdd(&bad, mine);
    __syncthreads();
    if (threadIdx.x != 0) return;
    int total = bad;
    if (gridDim.x > 1) {
        if (total != 0) atomicAdd(&sum[0], total);
        __threadfence();
        if (atomicAdd(&sum[1], 1) != (int)gridDim.x - 1) return;
        total = atomicExch(&sum[0], 0);
        atomicExch(&sum[1], 0);
    }
    post(posted, (uint64_t)(uint32_t)total, tag);
}

// Seed V := K at the sources (both buffers) and, when `schedule` is set,
// schedule the tiles whose interior or halo holds a source.  Bound by the chain of a
// source's nine exchanges (10 us), with many sources to a tile by atomics on the same
// addresses: 2,000,000 on 4096^2 took 3.0 ms with an exchange per tile and an addition
// per source, 0.39 with the flags read first and an addition per wave.  Reading the
// flags makes the chain 3 to 7 us longer, so few sources do without: 5,000 on 4096^2
// 10.7 us (16.3 with), 20,000 on 1000^2 23 us with (87 without).
constexpr int kSeedMany = 8192;

__global__ void k_seed(RoundArgs a, int32_t slot0, const int32_t* __restrict__ src,
                       const int32_t* __restrict__ src_slot, int32_t n, int32_t schedule,
                       int32_t* __restrict__ bad) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int slot = src_slot != nullptr ? src_slot[i] : slot0;
    const MazeDev md = a.mazes[slot];
    const int32_t r = src[2 * i], c = src[2 * i + 1];
    const uint32_t w = md.mask[mask_word(md, r, c)];
    if ((w >> (c & 31)) & 1u) {
        atomicAdd(bad, 1);
        return;
    }
    const int64_t x = (int64_t)r * md.pitch + c;
    md.V[0][x] = md.K;
    if (md.R[0] != nullptr) {   // front propagation: the source is in R_0 (both planes), counted once
        const int64_t wx = mask_word(md, r, c);
        const uint32_t bit = 1u << (c & 31);
        atomicOr(&md.R[1][wx], bit);
        const bool first = !(atomicOr(&md.R[0][wx], bit) & bit);
        // one addition for all lanes of the first lane's maze (most often the wave), by the last of them
        const bool same = slot == __builtin_amdgcn_readfirstlane(slot);
        const uint64_t group = __ballot(same);
        const int together = __popcll(__ballot(first) & group);
        const int add = !same ? (int)first : (group >> lane_id() == 1 ? together : 0);
        const int copy = (int)(blockIdx.x * (blockDim.x / kLanes) + threadIdx.x / kLanes) % kSpread;
        if (add > 0) atomicAdd(&a.maze_reached[slot * kSpread + copy], (unsigned long long)add);
    } else {
        md.V[1][x] = md.K;
    }
    const int ty = r / a.tile_rows, tx = c / a.tile_cols;
    a.touched[md.tile_base + ty * md.tiles_x + tx] = 1;
    if (!schedule) {   // dense: the maze counts as changed, so the first round visits it
        a.dchg_prev[slot] = 1;
        return;
    }
    for (int dy = -1; dy <= 1; ++dy)
        for (int dx = -1; dx <= 1; ++dx) {
            const int ny = ty + dy, nx = tx + dx;
            if (ny < 0 || ny >= md.tiles_y || nx < 0 || nx >= md.tiles_x) continue;
            // (a tile that is flagged already needs no exchange)
            const int g = md.tile_base + ny * md.tiles_x + nx;
            if (n <= kSeedMany || __hip_atomic_load(&a.flags_out[g], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)
                schedule_tile(a, md, slot, ny, nx);
        }
}

// Zeroes the interior of tile (ty, tx): both activity buffers, or the front
// propagation's one buffer and both reached-set planes (one wave).
__device__ __forceinline__ void clear_tile(const MazeDev& md, int ty, int tx, int tile_rows, int tile_cols) {
    const int r0 = ty * tile_rows, c0 = tx * tile_cols;
    const int rows = min(tile_rows, md.H - r0), cols = min(tile_cols, md.W - c0);
    if (md.R[0] != nullptr) {   // front tiles: whole words and rows up to the pitch, 16 bytes a lane
        constexpr int kQuads = kFrontCols / 4;
        static_assert(kLanes % kQuads == 0 && kFrontTileRows == kLanes, "front tile");
        const int4 zero = make_int4(0, 0, 0, 0);
        const int c = c0 + 4 * (lane_id() % kQuads);
        if (c < md.pitch)
            for (int k = lane_id() / kQuads; k < rows; k += kLanes / kQuads)
                *reinterpret_cast<int4*>(md.V[0] + (int64_t)(r0 + k) * md.pitch + c) = zero;
        if (lane_id() < rows) {
            for (int j = 0; j < kFrontCols / 32 && c0 + 32 * j < md.pitch; ++j) {
                const int64_t x = mask_word(md, r0 + lane_id(), c0 + 32 * j);
                md.R[0][x] = 0;
                md.R[1][x] = 0;
            }
        }
        return;
    }
    for (int k = lane_id(); k < rows * cols; k += kLanes) {
        const int64_t x = (int64_t)(r0 + k / cols) * md.pitch + c0 + k % cols;
        md.V[0][x] = 0;
        md.V[1][x] = 0;
    }
}

// What a start needs before its seeds, in one launch.  The first blocks take a
// tile id in [tile_begin, + n_tiles) per wave: the tile of a selected maze is
// zeroed if it was written since the last time (select 2: always).  The next
// n_zero_blocks blocks zero n_zero words (the schedule's tables), the others copy
// the descriptors to their table and reset the started slots' counters (last round
// = r - 1): 1,024 words a block, since one block took 0.9 ms for 20,000 mazes.
constexpr int kStartWords = 1024;

__global__ __launch_bounds__(kBlockThreads) void k_start(RoundArgs a, StartArgs st) {
    const int nb = (st.n_tiles + kWavesPerBlock - 1) / kWavesPerBlock;
    int b = blockIdx.x;
    if (b < nb) {
        const int t = b * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        if (t >= st.n_tiles) return;
        const int g = st.tile_begin + t;
        const int slot = a.tile_maze[g];
        if (slot < 0 || st.sel[slot] == 0 || (st.sel[slot] == 1 && !a.touched[g])) return;
        const MazeDev& md = st.staged[slot];
        const int lt = g - md.tile_base;
        const int ty = lt / md.tiles_x;
        clear_tile(md, ty, lt - ty * md.tiles_x, a.tile_rows, a.tile_cols);
        if (lane_id() == 0) a.touched[g] = 0;
        return;
    }
    b -= nb;
    if (b < st.n_zero_blocks) {
        for (int64_t i = (int64_t)b * kBlockThreads + threadIdx.x; i < st.n_zero; i += (int64_t)st.n_zero_blocks * kBlockThreads)
            st.zero[i] = 0;
        return;
    }
    b -= st.n_zero_blocks;
    const int64_t first = (int64_t)b * kBlockThreads + threadIdx.x;
    const int64_t step = ((int64_t)gridDim.x - nb - st.n_zero_blocks) * kBlockThreads;
    const uint32_t* from = reinterpret_cast<const uint32_t*>(st.staged);
    uint32_t* to = reinterpret_cast<uint32_t*>(st.mazes_out);
    for (int64_t i = first; i < (int64_t)(sizeof(MazeDev) / 4) * a.n_slots; i += step) to[i] = from[i];
    for (int64_t i = first; i < (int64_t)st.n_started * kSpread; i += step) {
        const int slot = st.started[i / kSpread];
        const int64_t x = (int64_t)slot * kSpread + i % kSpread;
        if (i % kSpread == 0) a.maze_last_round[slot] = a.round_id - 1;
        a.maze_visits[x] = 0;
        a.maze_reached[x] = 0;
        a.maze_layer[x] = 0;
    }
}

// Sources of several mazes on obstacles: bad[slot] counts them.
__global__ void k_check_sources_many(const MazeDev* __restrict__ mazes, const int32_t* __restrict__ src,
                                     const int32_t* __restrict__ src_slot, int32_t n, int32_t* __restrict__ bad) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int slot = src_slot[i];
    const MazeDev md = mazes[slot];
    const int32_t r = src[2 * i], c = src[2 * i + 1];
    const uint32_t w = md.mask[mask_word(md, r, c)];
    if ((w >> (c & 31)) & 1u) atomicAdd(&bad[slot], 1);
}

// ---------------------------------------------------------------------------
// finalize: smallest positive activity and reached-cell count per maze
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_reduce(const MazeDev* __restrict__ mazes,
                                                const int32_t* __restrict__ tile_maze,
                                                const uint8_t* __restrict__ touched,
                                                int32_t tile_begin, const int32_t* __restrict__ sel,
                                                int32_t tile_rows, int32_t tile_cols, int32_t parity,
                                                int32_t* __restrict__ maze_min,
                                                unsigned long long* __restrict__ maze_reached) {
    const int g = tile_begin + blockIdx.x;
    const int slot = tile_maze[g];
    // tiles never written since the last clear hold only zeros
    if (slot < 0 || (sel != nullptr && sel[slot] == 0) || !touched[g]) return;
    const MazeDev md = mazes[slot];
    const int lt = g - md.tile_base;
    const int ty = lt / md.tiles_x, tx = lt - ty * md.tiles_x;
    const int r0 = ty * tile_rows, c0 = tx * tile_cols;
    const int rows = min(tile_rows, md.H - r0), cols = min(tile_cols, md.W - c0);
    const int32_t* V = parity ? md.V[1] : md.V[0];
    int vmin = 0x7fffffff;
    int cnt = 0;
    for (int k = threadIdx.x; k < rows * cols; k += blockDim.x) {
        const int r = r0 + k / cols, c = c0 + k % cols;
        const int v = V[(int64_t)r * md.pitch + c];
        if (v > 0) {
            vmin = min(vmin, v);
            ++cnt;
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        vmin = min(vmin, __shfl_xor(vmin, off));
        cnt += __shfl_xor(cnt, off);
    }
    __shared__ int smin[4], scnt[4];
    const int w = threadIdx.x >> 6;
    if (lane_id() == 0) {
        smin[w] = vmin;
        scnt[w] = cnt;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int m = smin[0], n = scnt[0];
        for (int k = 1; k < (int)(blockDim.x >> 6); ++k) {
            m = min(m, smin[k]);
            n += scnt[k];
        }
        if (n > 0) {
            atomicMin(&maze_min[slot], m);
            atomicAdd(&maze_reached[slot], (unsigned long long)n);
        }
    }
}

// The same from the counts the front propagation's visits keep: per slot, the
// cells reached and K minus the last layer that reached one, and if asked for
// the last round and the tile visits (the results may be in host memory).
__global__ void k_front_report(const MazeDev* __restrict__ mazes, const unsigned long long* __restrict__ reached,
                               const int32_t* __restrict__ layer, const int32_t* __restrict__ last_round,
                               const int64_t* __restrict__ visits, int32_t n_slots, int32_t* __restrict__ maze_min,
                               unsigned long long* __restrict__ maze_reached, int32_t* __restrict__ last_out,
                               int64_t* __restrict__ visits_out) {
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= n_slots) return;
    unsigned long long n = 0;
    int64_t v = 0;
    int last = 0;
    for (int k = 0; k < kSpread; ++k) {
        n += reached[s * kSpread + k];
        v += visits[s * kSpread + k];
        last = max(last, layer[s * kSpread + k]);
    }
    maze_min[s] = mazes[s].K - last;
    maze_reached[s] = n;
    if (last_out != nullptr) {
        last_out[s] = last_round[s];
        visits_out[s] = v;
    }
}

// ---------------------------------------------------------------------------
// paths: lengths, offsets, gradient walk
// ---------------------------------------------------------------------------

__device__ __forceinline__ int path_length(const MazeDev& md, int r, int c, int parity) {
    const int v = (parity ? md.V[1] : md.V[0])[(int64_t)r * md.pitch + c];
    return v > 0 ? md.K - v : -1;
}

__global__ void k_path_lengths(const MazeDev* __restrict__ mazes, const int32_t* __restrict__ tslot,
                               const int32_t* __restrict__ trc, int32_t n, int32_t parity,
                               int32_t* __restrict__ len) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) len[i] = path_length(mazes[tslot[i]], trc[2 * i], trc[2 * i + 1], parity);
}

// Takes a slot in bucket k for every lane with k >= 0 (wave-uniform call):
// one LDS atomic per distinct key in the wave, the lanes of a key numbered in
// lane order.  Returns the lane's slot, or -1 for k < 0.
__device__ __forceinline__ int wave_bucket_slot(int* bucket, int k) {
    const int lane = lane_id();
    int slot = -1;
    uint64_t todo = __ballot(k >= 0);
    while (todo != 0) {
        const int leader = __builtin_ctzll(todo);
        const int kk = __shfl(k, leader);
        const uint64_t same = __ballot(k == kk);
        int base = 0;
        if (lane == leader) base = atomicAdd(&bucket[kk], __popcll(same));
        base = __shfl(base, leader);
        if (k == kk) slot = base + __popcll(same & ((1ull << lane) - 1));
        todo &= ~same;
    }
    return slot;
}

// Offsets of the paths (exclusive scan of length + 1 over reached targets),
// and optionally an order of the targets by path length, longest first (by
// the length's bit width: a bucket order, not a full sort), so that the walk
// starts the paths that take longest before the others.
// (lengths: computed here first, for up to kScanLengths targets; posted: the
// number of path cells goes to the host as soon as it is known)
__global__ __launch_bounds__(1024) void k_scan(const MazeDev* __restrict__ mazes, const int32_t* __restrict__ tslot,
                                               const int32_t* __restrict__ trc, int32_t parity,
                                               int32_t* __restrict__ len, int32_t n, int64_t* __restrict__ off,
                                               int32_t* __restrict__ order, uint64_t* posted, uint32_t tag) {
    __shared__ int64_t part[1024];
    const int t = threadIdx.x;
    if (mazes != nullptr) {
        for (int i = t; i < n; i += 1024) len[i] = path_length(mazes[tslot[i]], trc[2 * i], trc[2 * i + 1], parity);
        __syncthreads();
    }
    const int chunk = (n + 1023) / 1024;
    const int b = min(n, t * chunk), e = min(n, b + chunk);
    int64_t s = 0;
#pragma unroll 8
    for (int i = b; i < e; ++i) s += len[i] >= 0 ? (int64_t)len[i] + 1 : 0;
    part[t] = s;
    __syncthreads();
    for (int d = 1; d < 1024; d <<= 1) {
        const int64_t v = t >= d ? part[t - d] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int64_t base = t ? part[t - 1] : 0;
    if (t == 0) {
        off[0] = 0;
        post(posted, (uint64_t)part[1023], tag);
    }
#pragma unroll 8
    for (int i = b; i < e; ++i) {
        base += len[i] >= 0 ? (int64_t)len[i] + 1 : 0;
        off[i + 1] = base;
    }
    if (order == nullptr) return;
    __shared__ int bucket[33];
    if (t < 33) bucket[t] = 0;
    __syncthreads();
    // key 0 = the longest lengths (32 - bit width of len + 1; unreached last);
    // elements in rows of 1024 (every thread runs the same number of rounds,
    // -1: past the end), eight rows' keys loaded together, one LDS atomic per
    // distinct key of a wave
    auto key = [&](int i) { return i >= n ? -1 : (len[i] < 0 ? 32 : __clz(len[i] + 1)); };
    constexpr int kRows = 8;
    const int rows = (n + 1023) / 1024;
    for (int j0 = 0; j0 < rows; j0 += kRows) {
        int kb[kRows];
#pragma unroll
        for (int u = 0; u < kRows; ++u) kb[u] = key((j0 + u) * 1024 + t);
#pragma unroll
        for (int u = 0; u < kRows; ++u) (void)wave_bucket_slot(bucket, kb[u]);
    }
    __syncthreads();
    if (t == 0) {
        int acc = 0;
        for (int k = 0; k < 33; ++k) {
            const int c = bucket[k];
            bucket[k] = acc;
            acc += c;
        }
    }
    __syncthreads();
    for (int j0 = 0; j0 < rows; j0 += kRows) {
        int kb[kRows];
#pragma unroll
        for (int u = 0; u < kRows; ++u) kb[u] = key((j0 + u) * 1024 + t);
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            const int slot = wave_bucket_slot(bucket, kb[u]);
            if (slot >= 0) order[slot] = (j0 + u) * 1024 + t;
        }
    }
}

// The same over many blocks, for more targets than one block does quickly
// (136,824 targets: 24 us in three launches against 295): lengths with the sum
// and the bucket counts of each block's 256 targets, a scan of the blocks' sums
// and the buckets' first places, then offsets and places.
constexpr int kScanBlock = 256, kBuckets = 33;

// Bucket of a length: 0 = the longest lengths (32 - bit width of length + 1),
// unreached last.
__device__ __forceinline__ int length_bucket(int len) { return len < 0 ? kBuckets - 1 : __clz(len + 1); }

// Inclusive scan over the block's threads.
template <int WAVES>
__device__ __forceinline__ int64_t block_scan(int64_t v, int64_t (&wave_sum)[WAVES]) {
    const int lane = lane_id(), wave = threadIdx.x >> 6;
    for (int d = 1; d < kLanes; d <<= 1) {
        const int64_t u = __shfl_up(v, d);
        if (lane >= d) v += u;
    }
    if (lane == kLanes - 1) wave_sum[wave] = v;
    __syncthreads();
    for (int w = 0; w < wave; ++w) v += wave_sum[w];
    return v;
}

__global__ __launch_bounds__(kScanBlock) void k_block_sums(const MazeDev* __restrict__ mazes,
                                                           const int32_t* __restrict__ tslot,
                                                           const int32_t* __restrict__ trc, int32_t parity,
                                                           int32_t* __restrict__ len, int32_t n,
                                                           int64_t* __restrict__ sums, int32_t* __restrict__ counts) {
    __shared__ int bucket[kBuckets];
    __shared__ int64_t wave_sum[4];
    const int i = blockIdx.x * kScanBlock + threadIdx.x;
    if (threadIdx.x < kBuckets) bucket[threadIdx.x] = 0;
    __syncthreads();
    int l = -1;
    if (i < n) {
        if (mazes != nullptr) {
            l = path_length(mazes[tslot[i]], trc[2 * i], trc[2 * i + 1], parity);
            len[i] = l;
        } else {
            l = len[i];
        }
    }
    (void)wave_bucket_slot(bucket, i < n ? length_bucket(l) : -1);
    const int64_t sum = block_scan(l >= 0 ? (int64_t)l + 1 : 0, wave_sum);   // (also waits for the buckets)
    if (threadIdx.x == kScanBlock - 1) sums[blockIdx.x] = sum;
    if (threadIdx.x < kBuckets) counts[(int64_t)blockIdx.x * kBuckets + threadIdx.x] = bucket[threadIdx.x];
}

// sums[0 .. nb) := their exclusive scan; place[k] := first place of bucket k.
__global__ __launch_bounds__(1024) void k_scan_sums(int64_t* __restrict__ sums, const int32_t* __restrict__ counts,
                                                          int32_t nb, int32_t* __restrict__ place, uint64_t* posted,
                                                          uint32_t tag) {
    __shared__ int64_t wave_sum[16];
    __shared__ int64_t run;
    __shared__ int bucket[kBuckets];
    if (threadIdx.x == 0) run = 0;
    if (threadIdx.x < kBuckets) bucket[threadIdx.x] = 0;
    __syncthreads();
    for (int b0 = 0; b0 < nb; b0 += 1024) {
        const int b = b0 + threadIdx.x;
        const int64_t v = b < nb ? sums[b] : 0;
        const int64_t incl = block_scan(v, wave_sum) + run;
        if (b < nb) sums[b] = incl - v;
        __syncthreads();
        if (threadIdx.x == 1023) run = incl;
        __syncthreads();
    }
    if (threadIdx.x == 0) post(posted, (uint64_t)run, tag);
    // (31 threads to a bucket)
    constexpr int kPer = 1024 / kBuckets;
    if (threadIdx.x < kPer * kBuckets) {
        int m = 0;
#pragma unroll 8
        for (int b = threadIdx.x / kBuckets; b < nb; b += kPer) m += counts[(int64_t)b * kBuckets + threadIdx.x % kBuckets];
        if (m) atomicAdd(&bucket[threadIdx.x % kBuckets], m);
    }
    __syncthreads();
    if (threadIdx.x < kBuckets) {
        int at = 0;
        for (int k = 0; k < (int)threadIdx.x; ++k) at += bucket[k];
        place[threadIdx.x] = at;
    }
}

__global__ __launch_bounds__(kScanBlock) void k_block_offsets(const int32_t* __restrict__ len, int32_t n,
                                                              const int64_t* __restrict__ sums,
                                                              int32_t* __restrict__ place, int64_t* __restrict__ off,
                                                              int32_t* __restrict__ order) {
    __shared__ int bucket[kBuckets], base[kBuckets];
    __shared__ int64_t wave_sum[4];
    const int i = blockIdx.x * kScanBlock + threadIdx.x;
    if (threadIdx.x < kBuckets) bucket[threadIdx.x] = 0;
    __syncthreads();
    const int l = i < n ? len[i] : -1;
    const int k = i < n ? length_bucket(l) : -1;
    const int slot = wave_bucket_slot(bucket, k);
    const int64_t end = block_scan(l >= 0 ? (int64_t)l + 1 : 0, wave_sum) + sums[blockIdx.x];
    if (i < n) off[i + 1] = end;
    if (i == 0) off[0] = 0;
    if (order == nullptr) return;
    if (threadIdx.x < kBuckets && bucket[threadIdx.x] > 0)
        base[threadIdx.x] = atomicAdd(&place[threadIdx.x], bucket[threadIdx.x]);
    __syncthreads();
    if (i < n) order[base[k] + slot] = i;
}

// The walk is a chain of dependent steps, so its time is the longest path
// times the latency of one step.  One wave follows one target through the
// activity map from a window of kWinRows x 64 cells held in LDS (one global
// round trip per window, 16-byte loads).
//
// A step from a reached non-source cell with activity v0 goes to its first
// neighbour (fixed order: row-major over the 3 x 3 block, centre skipped)
// whose activity is v0 + 1: the map's largest neighbour value is exactly
// v0 + 1 there (activity drops by one per move away from the sources), so
// this is the first maximal neighbour.  Three steps are resolved per LDS
// read: lane l reads the cell at (l / 8 - 3, l % 8 - 3) from the current
// cell, i.e. the 8 x 8 block around it, and three ballots mark the block's
// cells holding v0 + 1, v0 + 2 and v0 + 3.  Block cells are numbered
// row-major, so the 8 neighbours of block cell q, in the fixed order, are the
// set bits of kNbr << (q - 9), and step j moves to the lowest set bit of
// ballot j among the neighbours of the cell step j - 1 reached (a cell at
// most j - 1 from the centre, whose neighbours stay inside the block for
// j <= 3).  Window cells outside the grid read -1 and obstacles 0, so neither
// ever matches.  The window is placed so that the path's direction over the
// previous window has the most room ahead; it is reloaded when the 8 x 8
// block around the current cell no longer fits.
constexpr int kWinRows = 48;
constexpr int kWinCols = 64;                       // window row: 64 cells = 16 chunks of 4
constexpr int kWinChunks = kWinRows * kWinCols / 4;
static_assert(kWinRows >= 16 && kWinChunks % kLanes == 0, "walk window");
constexpr int kWalkWaves = 4;
// neighbours of block cell 9 (row 1, column 1): cells 0, 1, 2, 8, 10, 16, 17, 18
constexpr uint64_t kNbr = 0x70507ull;

// A wave reads what its lanes wrote, and writes the next window after every
// lane's reads: LDS operations of a wave complete in order; the wave barrier
// keeps the compiler from moving them past each other.
__device__ __forceinline__ void walk_window_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Loads the window with corner (R0, C0), C0 a multiple of 4, into a wave's LDS;
// cells outside the grid read -1.  Every chunk's load is issued before the
// first is used, so the window costs one global round trip.
// A window inside the grid needs no masks, which were most of its instructions
// (4096 paths of a 23,170^2 map 0.674 -> 0.636 ms, 512 of 1021 x 1533 84.5 -> 79.1
// us, Euclidean walks 0.910 -> 0.866 ms).
__device__ __forceinline__ void walk_window(const MazeDev& md, const int32_t* V, int R0, int C0, int32_t* win) {
    const int lane = lane_id();
    v4i32 ld[kWinChunks / kLanes];
    if (R0 >= 0 && R0 + kWinRows <= md.H && C0 >= 0 && C0 + kWinCols <= md.W) {   // (uniform)
        const char* base = reinterpret_cast<const char*>(V + (int64_t)R0 * md.pitch + C0);
        const uint32_t off = 4 * ((uint32_t)(lane >> 4) * (uint32_t)md.pitch + 4 * (lane & 15));
#pragma unroll
        for (int k = 0; k < kWinChunks / kLanes; ++k)
            ld[k] = *(const __attribute__((address_space(1))) v4i32*)(base + (int64_t)k * (16 * (int64_t)md.pitch) + off);
#pragma unroll
        for (int k = 0; k < kWinChunks / kLanes; ++k)
            *(__attribute__((address_space(3))) v4i32*)(win + 4 * (lane + kLanes * k)) = ld[k];
        walk_window_sync();
        return;
    }
#pragma unroll
    for (int k = 0; k < kWinChunks / kLanes; ++k) {
        const int q = lane + kLanes * k;
        const int wr = q >> 4, wc = 4 * (q & 15);
        const int R = R0 + wr, cs = C0 + wc;
        const bool rok = R >= 0 && R < md.H;
        const bool cok = cs >= 0 && cs < md.pitch;   // a chunk lies wholly inside or outside a row
        ld[k] = *(const __attribute__((address_space(1))) v4i32*)(V + (int64_t)(rok ? R : 0) * md.pitch +
                                                                  (cok ? cs : 0));
    }
#pragma unroll
    for (int k = 0; k < kWinChunks / kLanes; ++k) {
        const int q = lane + kLanes * k;
        const int wr = q >> 4, wc = 4 * (q & 15);
        const int R = R0 + wr, cs = C0 + wc;
        const bool rok = R >= 0 && R < md.H;
        v4i32 m;
#pragma unroll
        for (int e = 0; e < 4; ++e) m[e] = (rok && cs + e >= 0 && cs + e < md.W) ? ld[k][e] : -1;
        *(__attribute__((address_space(3))) v4i32*)(win + wr * kWinCols + wc) = m;
    }
    walk_window_sync();
}

// Row and column of the current cell in its next window: the most room in the
// direction the path last went.
__device__ __forceinline__ int walk_row(int dr) { return dr < 0 ? kWinRows - 5 : (dr > 0 ? 3 : kWinRows / 2); }
__device__ __forceinline__ int walk_col(int dc) { return dc < 0 ? 56 : (dc > 0 ? 3 : 30); }

// Moves left before the 8 x 8 block around (lr, lc) could leave the window.
__device__ __forceinline__ int walk_room(int lr, int lc) {
    return min(min(lr - 3, kWinRows - 5 - lr), min(lc - 3, kWinCols - 5 - lc));
}

// The random numbers of 64 consecutive moves, lane l those of move s + l: the
// hash modulo 1 .. 8, three bits each (modulo c at bit 3 (c - 1)).
__device__ __forceinline__ uint32_t tie_remainders(uint64_t seed, uint64_t target, uint64_t step);

// Position of the j-th set bit of m.
__device__ __forceinline__ int nth_bit(uint64_t m, int j) {
    for (; j > 0; --j) m &= m - 1;
    return __builtin_ctzll(m);
}

// Copies target i's length and offset to the caller's arrays (null: they are the
// caller's already), and after target 0's the end of the last path.
__device__ __forceinline__ void walk_results(const WalkOut& out, int i, int n, const int32_t* len, const int64_t* off) {
    if (out.len == nullptr || lane_id() != 0) return;
    out.len[i] = len[i];
    out.off[i] = off[i];
    if (i == 0) out.off[n] = off[n];
}

// RANDOM: among a cell's maximal neighbours, those holding v0 + 1, the one at
// position hash mod count in the fixed order is taken, not the first; the
// hashes of 64 moves are computed together, one per lane.
template <bool RANDOM>
__global__ __launch_bounds__(kLanes * kWalkWaves) void k_walk(
    const MazeDev* __restrict__ mazes, const int32_t* __restrict__ tslot, const int32_t* __restrict__ trc,
    int32_t n, int32_t parity, const int32_t* __restrict__ len, const int64_t* __restrict__ off,
    int32_t* __restrict__ cells, const int32_t* __restrict__ order, const int32_t* __restrict__ tlocal,
    uint64_t seed, WalkOut out) {
    __shared__ __attribute__((aligned(16))) int32_t win_all[kWalkWaves][kWinRows * kWinCols];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = lane_id();
    const int w = blockIdx.x * kWalkWaves + wave;
    if (w >= n) return;
    // (order: longest paths first, see k_scan)
    const int i = order ? __builtin_amdgcn_readfirstlane(order[w]) : w;
    const int steps = __builtin_amdgcn_readfirstlane(len[i]);
    walk_results(out, i, n, len, off);
    if (steps < 0) return;
    const int slot = __builtin_amdgcn_readfirstlane(tslot[i]);
    const MazeDev md = mazes[slot];
    const int32_t* __restrict__ V = parity ? md.V[1] : md.V[0];
    int32_t* win = win_all[wave];
    // this lane's cell of the 8 x 8 block, relative to the current cell
    const int my_off = ((lane >> 3) - 3) * kWinCols + ((lane & 7) - 3);
    int r = __builtin_amdgcn_readfirstlane(trc[2 * i]);
    int c = __builtin_amdgcn_readfirstlane(trc[2 * i + 1]);
    int64_t o = off[i];
    if (lane == 0) cells[o] = r * md.W + c;
    ++o;
    const uint64_t target = RANDOM ? (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(tlocal[i]) : 0;
    // the set bit of m that the path's next move takes (k: moves since the
    // remainders were computed)
    auto choose = [&](uint64_t m, uint32_t ties, int k) {
        if (!RANDOM) return __builtin_ctzll(m);
        const uint32_t rem = (uint32_t)__builtin_amdgcn_readlane((int)ties, k);
        return nth_bit(m, (int)((rem >> (3 * (__popcll(m) - 1))) & 7u));
    };
    // the cells of a window's steps are logged one iteration (three steps)
    // per lane (lane k: iteration k of the window) as (window position of the
    // iteration's 8 x 8 block centre) << 18 | q1 << 12 | q2 << 6 | q3 (the
    // cells reached, numbered in the block), and stored when the window is left
    int log = 0, it = 0;
    int dr_prev = 0, dc_prev = 0;   // displacement over the previous window
    int v0 = 0;
    for (int s = 0; s < steps;) {
        const int R0 = r - walk_row(dr_prev), C0 = (c - walk_col(dc_prev)) & ~3;
        walk_window(md, V, R0, C0, win);
        int lr = r - R0, lc = c - C0;
        if (s == 0) v0 = __builtin_amdgcn_readfirstlane(win[lr * kWinCols + lc]);
        const int s_start = s;
        // Whole iterations of three steps.  An iteration moves at most three
        // rows and three columns, so from the current cell the next n
        // iterations all start with their 8 x 8 block inside the window; the
        // bounds are checked once per such run.
        for (;;) {
            const int room = walk_room(lr, lc);
            int n = room < 0 ? 0 : room / 3 + 1;
            n = min(n, min((steps - s) / 3, kLanes - it));
            if (RANDOM) n = min(n, kLanes / 3);
            if (n <= 0) break;
            const uint32_t ties = RANDOM ? tie_remainders(seed, target, (uint64_t)s) : 0;
            for (int k = 0; k < n; ++k) {
                const int pos = lr * kWinCols + lc;
                const int d = win[pos + my_off] - v0;
                const uint64_t m1 = __ballot(d == 1);
                const uint64_t m2 = __ballot(d == 2);
                const uint64_t m3 = __ballot(d == 3);
                const int q1 = choose(m1 & (kNbr << 18), ties, 3 * k);   // neighbours of the centre, cell 27
                const int q2 = choose(m2 & (kNbr << (q1 - 9)), ties, 3 * k + 1);
                const int q3 = choose(m3 & (kNbr << (q2 - 9)), ties, 3 * k + 2);
                const int e = (pos << 18) | (q1 << 12) | (q2 << 6) | q3;
                log = lane == it + k ? e : log;
                lr += (q3 >> 3) - 3;
                lc += (q3 & 7) - 3;
                v0 += 3;
            }
            it += n;
            s += 3 * n;
        }
        // the path's last one or two steps, once their block fits
        if (s < steps && steps - s < 3 && it < kLanes && walk_room(lr, lc) >= 0) {
            const uint32_t ties = RANDOM ? tie_remainders(seed, target, (uint64_t)s) : 0;
            const int pos = lr * kWinCols + lc;
            const int d = win[pos + my_off] - v0;
            const uint64_t m1 = __ballot(d == 1);
            const uint64_t m2 = __ballot(d == 2);
            const int todo = steps - s;
            const int q1 = choose(m1 & (kNbr << 18), ties, 0);
            const int q2 = todo > 1 ? choose(m2 & (kNbr << (q1 - 9)), ties, 1) : 0;
            const int q = todo > 1 ? q2 : q1;
            log = lane == it ? (pos << 18) | (q1 << 12) | (q2 << 6) : log;
            ++it;
            lr += (q >> 3) - 3;
            lc += (q & 7) - 3;
            v0 += todo;
            s += todo;
        }
        const int nst = s - s_start;   // steps taken in this window
        if (lane < it) {
            const int pos = log >> 18, pr = pos >> 6, pc = pos & 63;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                if (3 * lane + j < nst) {
                    const int q = (log >> (12 - 6 * j)) & 63;
                    cells[o + 3 * lane + j] = (R0 + pr - 3 + (q >> 3)) * md.W + (C0 + pc - 3 + (q & 7));
                }
            }
        }
        o += nst;
        it = 0;
        dr_prev = lr - (r - R0);
        dc_prev = lc - (c - C0);
        // a move of less than a third of the steps counts as no direction
        if (3 * abs(dr_prev) < nst) dr_prev = 0;
        if (3 * abs(dc_prev) < nst) dc_prev = 0;
        r = R0 + lr;
        c = C0 + lc;
        walk_window_sync();
    }
}

// A few targets with long paths: a block per target, which spends its threads on
// shortening the chain.  For every cell of a 64 x 64 window the next cell of its
// path is worked out (bytes of one-hot activity modulo 3, four cells a register:
// adjacent reached cells differ by at most one, so a neighbour with one more is
// one whose class follows), then the cell 2, 4 and 8 moves on by pointer doubling
// in LDS.  The chain is one LDS read per 8 moves; the moves between are filled in
// by all threads, move k of the window from the chain's read k / 8 by the pointers
// of k's bits.  A cell on the window's border, a source and a cell without a path
// point to themselves.
//
// Bound by a window's latency, 3.3 us (about 1 us the load, the rest the steps
// between barriers), whatever its moves: about 60 straight on.  The wave's three
// moves per LDS read take 0.23 us and its window 1.5.  Extraction of one path of
// 9,125 moves in corridors 0.757 -> 0.550 ms, of 64 of up to 10,164 0.837 -> 0.578.
// 16 moves a hop, 1,024 threads, or loading the window that lies ahead meanwhile
// measured no better (0.560, 0.557, 0.654 ms), 256 threads 0.692.
//
// Taken by the number of targets and their moves on average (of reached targets
// and others): 160 targets of 37 moves 39.7 us with a wave each, 43.4 with a block;
// 64 of 162 62 and 56; 256 of 1,263 182 and 138.  Where two blocks share a CU a
// window takes longer: 512 targets of 261 moves 85 and 93, of 1,256 185 and 174, of
// 5,547 928 and 700; 1,024 of 5,364 942 and 1,040.
constexpr int kWalkTileTargets = 256, kWalkTileMoves = 64;          // a block per CU
constexpr int kWalkTileTargetsLong = 512, kWalkTileMovesLong = 1024;   // two
constexpr int kTileWalkThreads = 512;
constexpr int kTileWalkLevels = 3;   // the longest hop is 2^3 moves
constexpr int kTileWalkPitch = 18;   // dwords of a row of classes: 16 and one of none on either side

struct TileWalkShared {
    int32_t v[64 * 64];
    uint32_t cls[66 * kTileWalkPitch];
    uint16_t next[kTileWalkLevels + 1][64 * 64];   // the cell 1, 2, 4, 8 moves on
};

__global__ __launch_bounds__(kTileWalkThreads) void k_walk_tile(
    const MazeDev* __restrict__ mazes, const int32_t* __restrict__ tslot, const int32_t* __restrict__ trc,
    int32_t n, int32_t parity, const int32_t* __restrict__ len, const int64_t* __restrict__ off,
    int32_t* __restrict__ cells, const int32_t* __restrict__ order, WalkOut out) {
    __shared__ __attribute__((aligned(16))) TileWalkShared sh;
    typedef uint16_t v4u16 __attribute__((ext_vector_type(4)));
    constexpr int kGroups = 64 * 64 / 4 / kTileWalkThreads;   // groups of four cells a thread
    constexpr int kRowStep = kTileWalkThreads / 16;
    const int t = threadIdx.x, lane = lane_id();
    const int i = order ? __builtin_amdgcn_readfirstlane(order[blockIdx.x]) : (int)blockIdx.x;
    const int steps = __builtin_amdgcn_readfirstlane(len[i]);
    if (t < kLanes) walk_results(out, i, n, len, off);
    if (steps < 0) return;
    const MazeDev md = mazes[__builtin_amdgcn_readfirstlane(tslot[i])];
    const int32_t* __restrict__ V = parity ? md.V[1] : md.V[0];
    int r = __builtin_amdgcn_readfirstlane(trc[2 * i]), c = __builtin_amdgcn_readfirstlane(trc[2 * i + 1]);
    int32_t* __restrict__ to = cells + off[i];
    for (int q = t; q < 66 * kTileWalkPitch; q += kTileWalkThreads) sh.cls[q] = 0;   // (the frame stays 0)
    const int row = t >> 4, col = 4 * (t & 15);
    v4i32 ld[kGroups];
    auto load = [&](int R0, int C0) {
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const int R = R0 + row + g * kRowStep, cs = C0 + col;
            const bool ok = R >= 0 && R < md.H && cs >= 0 && cs < md.pitch;   // a chunk lies inside or outside a row
            ld[g] = *(const __attribute__((address_space(1))) v4i32*)(V + (ok ? (int64_t)R * md.pitch + cs : 0));
        }
    };
    int R0 = r - 32, C0 = (c - 30) & ~3;
    load(R0, C0);
    for (int s = 0, v0 = md.K - steps; s < steps;) {   // v0: activity of the current cell
        lds_barrier();   // the last window's tables are no longer read
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const int wr = row + g * kRowStep, R = R0 + wr, cs = C0 + col;
            const bool rok = R >= 0 && R < md.H && cs >= 0;
            uint32_t cls = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int v = rok && cs + e < md.W ? ld[g][e] : 0;
                cls |= (v > 0 ? 1u << ((uint32_t)v % 3u) : 0u) << (8 * e);
            }
            *(__attribute__((address_space(3))) v4i32*)(sh.v + 64 * wr + col) = ld[g];
            sh.cls[(wr + 1) * kTileWalkPitch + 1 + (t & 15)] = cls;
        }
        lds_barrier();
        v4u16 own[kGroups];
#pragma unroll
        for (int g = 0; g < kGroups; ++g) {
            const int wr = row + g * kRowStep;
            const uint32_t* p = sh.cls + (wr + 1) * kTileWalkPitch + 1 + (t & 15);
            const uint32_t own_cls = p[0];
            const uint32_t want = ((own_cls << 1) & 0x06060606u) | ((own_cls >> 2) & 0x01010101u);
            // the first neighbour wanted, as (row + 1) << 2 | column + 1; 5: none
            uint32_t code = 0x05050505u;
#pragma unroll
            for (int d = 8; d >= 0; --d) {
                if (d == 4) continue;
                const uint32_t* q = p + (d / 3 - 1) * kTileWalkPitch;
                const uint32_t nb = d % 3 == 0   ? __builtin_amdgcn_alignbyte(q[0], q[-1], 3)
                                    : d % 3 == 1 ? q[0]
                                                 : __builtin_amdgcn_alignbyte(q[1], q[0], 1);
                uint32_t m = nb & want;
                m = (m | m >> 1 | m >> 2) & 0x01010101u;
                m = (m << 8) - m;
                code = (code & ~m) | ((uint32_t)(((d / 3) << 2 | d % 3) * 0x01010101u) & m);
            }
            if (wr == 0 || wr == 63) code = 0x05050505u;
            if (col == 0) code = (code & ~0xffu) | 5u;
            if (col == 60) code = (code & 0x00ffffffu) | 5u << 24;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t k = (code >> (8 * e)) & 0xfu;
                own[g][e] = (uint16_t)(64 * wr + col + e + (k >> 2) * 64 + (k & 3) - 65);
            }
            *(__attribute__((address_space(3))) v4u16*)(sh.next[0] + 64 * wr + col) = own[g];
        }
        lds_barrier();
#pragma unroll
        for (int l = 1; l <= kTileWalkLevels; ++l) {
#pragma unroll
            for (int g = 0; g < kGroups; ++g) {
#pragma unroll
                for (int e = 0; e < 4; ++e) own[g][e] = sh.next[l - 1][own[g][e]];
                *(__attribute__((address_space(3))) v4u16*)(sh.next[l] + 64 * (row + g * kRowStep) + col) = own[g];
            }
            lds_barrier();
        }
        // the chain, by every wave for itself; lane h keeps the cell after 8 h moves
        const int entry = (r - R0) * 64 + (c - C0);
        int at = entry, log = 0;
        for (int h = 0; h < kLanes; ++h) {
            log = lane == h ? at : log;
            const int to_cell = __builtin_amdgcn_readfirstlane((int)sh.next[kTileWalkLevels][at]);
            if (to_cell == at) break;
            at = to_cell;
        }
        const int moves = min(__builtin_amdgcn_readfirstlane(sh.v[at]) - v0, steps - s);
        const int from_r = R0, from_c = C0;
        const int dr = (at >> 6) - (entry >> 6), dc = (at & 63) - (entry & 63);
        r = R0 + (at >> 6);
        c = C0 + (at & 63);
        if (moves <= 0) return;   // (a map that is not an activity map: no move)
        if (s + moves < steps) {
            // the most room in the direction the path went; less than a third of
            // the moves counts as none
            R0 = r - (3 * abs(dr) < moves ? 32 : (dr < 0 ? 62 : 1));
            C0 = (c - (3 * abs(dc) < moves ? 30 : (dc < 0 ? 59 : 1))) & ~3;
            load(R0, C0);
        }
        for (int k0 = t - lane; k0 < moves; k0 += kTileWalkThreads) {
            const int k = k0 + lane;
            int q = __shfl(log, min(k >> kTileWalkLevels, kLanes - 1));   // (every lane takes part)
#pragma unroll
            for (int b = 0; b < kTileWalkLevels; ++b)
                if (k >> b & 1) q = sh.next[b][q];
            if (k < moves) to[s + k] = (from_r + (q >> 6)) * md.W + from_c + (q & 63);
        }
        s += moves;
        v0 += moves;
    }
    if (t == 0) to[steps] = r * md.W + c;
}

// ---- random ties and Euclidean reconstruction ------------------------------

// SplitMix64 output function on seed ^ (target << 32) ^ step: the counter-based
// random number of the random tie-break (Steele, Lea, Flood 2014).
__device__ __forceinline__ uint64_t tie_hash(uint64_t seed, uint64_t target, uint64_t step) {
    uint64_t z = seed ^ (target << 32) ^ step;
    z += 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ uint32_t tie_remainders(uint64_t seed, uint64_t target, uint64_t step) {
    const uint64_t z = tie_hash(seed, target, step + (uint64_t)lane_id());
    const uint32_t lo = (uint32_t)z, hi = (uint32_t)(z >> 32);
    // 2^32 is 1 modulo 3 and 5, and 4 modulo 7
    const uint32_t m3 = (lo % 3 + hi % 3) % 3, m5 = (lo % 5 + hi % 5) % 5, m7 = (lo % 7 + 4 * (hi % 7)) % 7;
    const uint32_t m6 = m3 + 3 * ((m3 ^ lo) & 1);   // m3 or m3 + 3, whichever has the parity of z
    return (lo & 1) << 3 | m3 << 6 | (lo & 3) << 9 | m5 << 12 | m6 << 15 | m7 << 18 | (lo & 7) << 21;
}

// Euclidean reconstruction (Eq. 1 and straightening).  The walk climbs through
// 4-neighbours (first maximum in the order up, left, right, down), allows one
// sideways move to an equal 4-neighbour per activity level, and otherwise
// takes the first maximal 8-neighbour; the straightening pass (drop a point
// whose predecessor and successor are diagonal neighbours) runs on the fly.
//
// One wave per target, from the same windows and 8 x 8 blocks as k_walk: a
// block serves three moves, with ballots of the cells holding v .. v + 3 (a
// cell's maximal 4-neighbour holds v + 1, v or less, its maximal 8-neighbour
// v + 1); choosing them is a scalar chain.  Moves are logged three to a lane,
// and when the window is left its points are straightened together: point x is
// dropped if x - 1 and x + 1 are diagonal neighbours and x - 1 was kept (after
// a drop the next point is kept in any case: no move from one diagonal
// neighbour of a cell reaches another), so in a run of candidates every other
// one goes, beginning with the first.  2048 targets on 2048 x 2048, one pass: a
// lane per target reading its neighbours from memory 2.2 ms, straightening
// move by move in this kernel 0.37 ms.
constexpr uint64_t kNbr4 = 0x20502ull;   // up, left, right, down of block cell 9: cells 1, 8, 10, 17

// Whether two cells of a window (row * kWinCols + column) are diagonal neighbours.
__device__ __forceinline__ bool diagonal(int a, int b) {
    const int dr = (a >> 6) - (b >> 6), dc = (a & 63) - (b & 63);
    return dr * dr == 1 && dc * dc == 1;
}

// Every other bit of each run of ones in m, beginning with the run's first (or,
// for a run that begins at bit 0 after a dropped point, with its second).
__device__ __forceinline__ uint64_t every_other(uint64_t m, bool after_drop) {
    const uint64_t even = 0x5555555555555555ull;
    uint64_t begin = m & ~(m << 1) & even;
    if (after_drop) begin &= ~1ull;
    const uint64_t on_even = m & ~(m + begin);   // the runs that take their even bits
    return (on_even & even) | (m & ~on_even & ~even);
}

// COUNT: the path's length (its points less one, -1 for no path) goes to len.
// WRITE: its cells go to cells, from off[i] on or, where they are counted as well,
// from i * stride on (at most stride of them); k_gather_paths moves them once the
// offsets are known, in place of a second walk: 2,048 paths of a 2,048^2 map, asked for and taken, 0.867 -> 0.635 ms.
template <bool WRITE, bool COUNT>
__global__ __launch_bounds__(kLanes * kWalkWaves) void k_walk_euclid(
    const MazeDev* __restrict__ mazes, const int32_t* __restrict__ tslot, const int32_t* __restrict__ trc, int32_t n,
    int32_t parity, int32_t* __restrict__ len, const int64_t* __restrict__ off, int32_t* __restrict__ cells,
    int64_t stride, WalkOut out) {
    __shared__ __attribute__((aligned(16))) int32_t win_all[kWalkWaves][kWinRows * kWinCols];
    __shared__ uint16_t seq_all[kWalkWaves][3 * kLanes + 8];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = lane_id();
    const int i = blockIdx.x * kWalkWaves + wave;
    if (i >= n) return;
    if (!COUNT) walk_results(out, i, n, len, off);
    const int slot = __builtin_amdgcn_readfirstlane(tslot[i]);
    const MazeDev md = mazes[slot];
    const int32_t* __restrict__ V = parity ? md.V[1] : md.V[0];
    int32_t* win = win_all[wave];
    uint16_t* seq = seq_all[wave];   // window positions: last decided point, pending point, the moves
    const int my_off = ((lane >> 3) - 3) * kWinCols + ((lane & 7) - 3);
    int r = __builtin_amdgcn_readfirstlane(trc[2 * i]);
    int c = __builtin_amdgcn_readfirstlane(trc[2 * i + 1]);
    int v = __builtin_amdgcn_readfirstlane(V[(int64_t)r * md.pitch + c]);
    if (v <= 0) {
        if (COUNT && lane == 0) len[i] = -1;
        return;
    }
    const int K = md.K, W = md.W;
    int64_t o = COUNT ? (WRITE ? i * stride : 0) : off[i];
    const int64_t o_end = COUNT ? o + stride : INT64_MAX;
    int count = 1;   // points kept
    if (WRITE && lane == 0) cells[o] = r * W + c;
    ++o;
    int kr = r, kc = c;              // last decided point, and whether it was dropped
    bool dropped = false;
    int pr = 0, pc = 0;              // pending point (decided by the move after it)
    bool pending = false;
    bool sideways_before = false;
    int dr_prev = 0, dc_prev = 0;
    while (v != K) {
        const int R0 = r - walk_row(dr_prev), C0 = (c - walk_col(dc_prev)) & ~3;
        walk_window(md, V, R0, C0, win);
        int lr = r - R0, lc = c - C0;
        const int lr_in = lr, lc_in = lc;
        int log = 0, it = 0, moves = 0;
        while (v != K && it < kLanes && walk_room(lr, lc) >= 0) {
            const int pos = lr * kWinCols + lc;
            const int d = win[pos + my_off] - v;
            uint64_t m0 = __ballot(d == 0), m1 = __ballot(d == 1), m2 = __ballot(d == 2), m3 = __ballot(d == 3);
            int q = 27, e = pos, done = 0;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                if (j == 0 || v != K) {
                    const uint64_t up = m1 & (kNbr4 << (q - 9));
                    uint64_t to = up;
                    if (__builtin_expect(up == 0, 0)) {
                        const uint64_t side = m0 & (kNbr4 << (q - 9));
                        const bool sideways = side != 0 && !sideways_before;
                        to = sideways ? side : m1 & (kNbr << (q - 9));
                        sideways_before = sideways;
                    } else {
                        sideways_before = false;
                    }
                    q = __builtin_ctzll(to);
                    if (!sideways_before) {
                        m0 = m1;
                        m1 = m2;
                        m2 = m3;
                        ++v;
                    }
                    ++done;
                }
                e = e << 6 | q;
            }
            log = lane == it ? e : log;
            ++it;
            moves += done;
            lr += (q >> 3) - 3;
            lc += (q & 7) - 3;
        }
        r = R0 + lr;
        c = C0 + lc;
        // ---- straighten what the window gave
        const int first = pending ? 2 : 1;   // index of the first move in seq
        if (lane == 0) {
            seq[0] = (uint16_t)((kr - R0) * kWinCols + (kc - C0));
            if (pending) seq[1] = (uint16_t)((pr - R0) * kWinCols + (pc - C0));
        }
        if (lane < it) {
            const int pos = log >> 18;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const int q = (log >> (12 - 6 * j)) & 63;
                if (3 * lane + j < moves)
                    seq[first + 3 * lane + j] = (uint16_t)(pos + ((q >> 3) - 3) * kWinCols + ((q & 7) - 3));
            }
        }
        walk_window_sync();
        const int end = first + moves - 1;   // the last point stays pending
        for (int x0 = 1; x0 < end; x0 += kLanes) {
            const int x = x0 + lane;
            const bool valid = x < end;
            const int here = valid ? seq[x] : 0;
            const uint64_t cand = __ballot(valid && diagonal(seq[valid ? x - 1 : 0], seq[valid ? x + 1 : 0]));
            const uint64_t drop = every_other(cand, dropped);
            const uint64_t keep = __ballot(valid) & ~drop;
            const int64_t to = o + __popcll(keep & ((1ull << lane) - 1));
            if (WRITE && (keep >> lane & 1) && to < o_end) cells[to] = (R0 + (here >> 6)) * W + C0 + (here & 63);
            o += __popcll(keep);
            count += __popcll(keep);
            dropped = (drop >> (min(end - x0, kLanes) - 1)) & 1;
        }
        if (end > 1) {
            const int k = __builtin_amdgcn_readfirstlane(seq[end - 1]);
            kr = R0 + (k >> 6);
            kc = C0 + (k & 63);
        }
        pr = r;
        pc = c;
        pending = true;
        dr_prev = lr - lr_in;
        dc_prev = lc - lc_in;
        // a move of less than a third of the moves counts as no direction
        if (3 * abs(dr_prev) < moves) dr_prev = 0;
        if (3 * abs(dc_prev) < moves) dc_prev = 0;
        walk_window_sync();
    }
    if (pending) {
        if (WRITE && lane == 0 && o < o_end) cells[o] = pr * W + pc;
        ++count;
    }
    if (COUNT && lane == 0) len[i] = count - 1;
}

// Both for very many targets (see kRandomLaneTargets): a lane per target, its
// neighbours read from memory.  A wave per target issues about as much for one path
// as a wave of these does for 64 (choosing a move is a scalar chain, a window 12 KB),
// which pays while the chip would otherwise be idle.  2^20 targets on 2048^2, of 307
// moves on average: random ties 17 ms against 21, Euclidean 37 against 117.
__device__ __forceinline__ int dir_dr(int k) { return k < 3 ? -1 : (k < 5 ? 0 : 1); }
__device__ __forceinline__ int dir_dc(int k) { return k < 3 ? k - 1 : (k < 5 ? 2 * k - 7 : k - 6); }

__device__ __forceinline__ int read_or(const int32_t* V, const MazeDev& md, int r, int c, int outside) {
    return (r >= 0 && r < md.H && c >= 0 && c < md.W) ? V[(int64_t)r * md.pitch + c] : outside;
}

// walk_results of a lane's target.
__device__ __forceinline__ void lane_results(const WalkOut& out, int i, int n, const int32_t* len, const int64_t* off) {
    if (out.len == nullptr) return;
    out.len[i] = len[i];
    out.off[i] = off[i];
    if (i == 0) out.off[n] = off[n];
}

__global__ __launch_bounds__(kLanes) void k_walk_random_lanes(
    const MazeDev* __restrict__ mazes, const int32_t* __restrict__ tslot, const int32_t* __restrict__ trc,
    const int32_t* __restrict__ tlocal, int32_t n, int32_t parity, uint64_t seed, const int32_t* __restrict__ len,
    const int64_t* __restrict__ off, int32_t* __restrict__ cells, WalkOut out) {
    const int i = blockIdx.x * kLanes + threadIdx.x;
    if (i >= n) return;
    lane_results(out, i, n, len, off);
    const int steps = len[i];
    if (steps < 0) return;
    const MazeDev md = mazes[tslot[i]];
    const int32_t* __restrict__ V = parity ? md.V[1] : md.V[0];
    int r = trc[2 * i], c = trc[2 * i + 1];
    int64_t o = off[i];
    cells[o++] = r * md.W + c;
    const uint64_t t = (uint64_t)(uint32_t)tlocal[i];
    for (int s = 0; s < steps; ++s) {
        int nv[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) nv[k] = read_or(V, md, r + dir_dr(k), c + dir_dc(k), -1);
        int best = nv[0];
#pragma unroll
        for (int k = 1; k < 8; ++k) best = max(best, nv[k]);
        int left = 0;   // maxima from direction k on
#pragma unroll
        for (int k = 0; k < 8; ++k) left += nv[k] == best;
        const int j = (int)(tie_hash(seed, t, (uint64_t)s) % (uint64_t)left);
        int pick = 0;
#pragma unroll
        for (int k = 7; k >= 0; --k)
            if (nv[k] == best && --left == j) pick = k;
        r += dir_dr(pick);
        c += dir_dc(pick);
        cells[o++] = r * md.W + c;
    }
}

// WRITE: the path's cells go to cells from off[i] on; else its length to len.
template <bool WRITE>
__global__ __launch_bounds__(kLanes) void k_walk_euclid_lanes(const MazeDev* __restrict__ mazes,
                                                              const int32_t* __restrict__ tslot,
                                                              const int32_t* __restrict__ trc, int32_t n,
                                                              int32_t parity, int32_t* __restrict__ len,
                                                              const int64_t* __restrict__ off,
                                                              int32_t* __restrict__ cells, WalkOut out) {
    const int i = blockIdx.x * kLanes + threadIdx.x;
    if (i >= n) return;
    if (WRITE) lane_results(out, i, n, len, off);
    const MazeDev md = mazes[tslot[i]];
    const int32_t* __restrict__ V = parity ? md.V[1] : md.V[0];
    int r = trc[2 * i], c = trc[2 * i + 1];
    int v = V[(int64_t)r * md.pitch + c];
    if (v <= 0) {
        if (!WRITE) len[i] = -1;
        return;
    }
    int64_t o = WRITE ? off[i] : 0;
    int count = 1;                 // points kept
    if (WRITE) cells[o++] = r * md.W + c;
    int kr = r, kc = c;            // last kept point
    int pr = -1, pc = -1;          // pending point (decided by the move after it)
    bool sideways_before = false;
    while (v != md.K) {
        const int up = read_or(V, md, r - 1, c, -1), lt = read_or(V, md, r, c - 1, -1);
        const int rt = read_or(V, md, r, c + 1, -1), dn = read_or(V, md, r + 1, c, -1);
        int to = up, dr = -1, dc = 0;
        if (lt > to) { to = lt; dr = 0; dc = -1; }
        if (rt > to) { to = rt; dr = 0; dc = 1; }
        if (dn > to) { to = dn; dr = 1; dc = 0; }
        if (to > v) {
            sideways_before = false;
        } else if (to == v && !sideways_before) {
            sideways_before = true;
        } else {
            int best = 0;
            to = read_or(V, md, r + dir_dr(0), c + dir_dc(0), -1);
#pragma unroll
            for (int k = 1; k < 8; ++k) {
                const int x = read_or(V, md, r + dir_dr(k), c + dir_dc(k), -1);
                if (x > to) {
                    to = x;
                    best = k;
                }
            }
            dr = dir_dr(best);
            dc = dir_dc(best);
            sideways_before = false;
        }
        r += dr;
        c += dc;
        v = to;
        if (pr >= 0 && !(abs(kr - r) == 1 && abs(kc - c) == 1)) {
            if (WRITE) cells[o++] = pr * md.W + pc;
            ++count;
            kr = pr;
            kc = pc;
        }
        pr = r;
        pc = c;
    }
    if (pr >= 0) {
        if (WRITE) cells[o++] = pr * md.W + pc;
        ++count;
    }
    if (!WRITE) len[i] = count - 1;
}

// Path i from points[i * stride] on to cells[off[i]] on, a wave each.
__global__ void k_gather_paths(const int32_t* __restrict__ points, int64_t stride, int32_t n,
                               const int32_t* __restrict__ len, const int64_t* __restrict__ off,
                               int32_t* __restrict__ cells, WalkOut out) {
    const int i = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    if (i >= n) return;
    walk_results(out, i, n, len, off);
    const int m = len[i] + 1;
    const int64_t o = off[i];
    for (int j = lane_id(); j < m; j += kLanes) cells[o + j] = points[i * stride + j];
}

// Index (in its maze's source list) of the source each path ends on; -1 if no
// path.  src_sorted holds per-maze (linear cell, first list index) pairs sorted
// by cell, src_base[t] / src_n[t] the target's maze's range.
__global__ void k_source_index(const MazeDev* __restrict__ mazes, const int32_t* __restrict__ tslot,
                               int32_t n, const int32_t* __restrict__ len,
                               const int64_t* __restrict__ off, const int32_t* __restrict__ cells,
                               const int32_t* __restrict__ src_sorted,
                               const int32_t* __restrict__ src_base,
                               const int32_t* __restrict__ src_n, int32_t* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (len[i] < 0) {
        out[i] = -1;
        return;
    }
    const int32_t end = cells[off[i + 1] - 1];
    const int32_t* p = src_sorted + 2 * (int64_t)src_base[i];
    int lo = 0, hi = src_n[i] - 1, found = -1;
    while (lo <= hi) {
        const int mid = (lo + hi) >> 1;
        const int32_t key = p[2 * mid];
        if (key == end) {
            found = p[2 * mid + 1];
            break;
        }
        if (key < end) lo = mid + 1; else hi = mid - 1;
    }
    out[i] = found;
}

// O = V - offset where V > 0, else 0 (offset = K - L - 1 maps the encoding back
// to the paper's activity values).
//
// Bound by memory (4 B read and 4 B written per cell): a wave takes 256 columns
// of kCopyRows rows, 16 bytes a lane and row with every load issued before the
// first store (one cell a lane reached 2.8 TB/s on 26,000^2 cells).  The caller's
// rows need no alignment beyond that of int32.
constexpr int kCopyRows = 4;
typedef int v4i32_any __attribute__((ext_vector_type(4), aligned(4)));

__global__ __launch_bounds__(kBlockThreads) void k_activity(MazeDev md, int32_t parity, int32_t offset,
                                                            int32_t* __restrict__ dst, int64_t dpitch,
                                                            int32_t col_blocks) {
    const int64_t b = blockIdx.x;
    const int64_t rb = b / col_blocks;
    const int32_t c = (int32_t)(b - rb * col_blocks) * (4 * kLanes) + 4 * lane_id();
    const int64_t r0 = (rb * kWavesPerBlock + (threadIdx.x >> 6)) * kCopyRows;
    if (c >= md.W) return;
    const int32_t* V = parity ? md.V[1] : md.V[0];
    v4i32 v[kCopyRows];
#pragma unroll
    for (int k = 0; k < kCopyRows; ++k)   // (c is below the pitch, a multiple of 64)
        v[k] = *(const __attribute__((address_space(1))) v4i32*)(V + min(r0 + k, (int64_t)md.H - 1) * md.pitch + c);
#pragma unroll
    for (int k = 0; k < kCopyRows; ++k) {
        if (r0 + k >= md.H) break;
        int32_t* const q = dst + (r0 + k) * dpitch + c;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[k][e] = v[k][e] > 0 ? v[k][e] - offset : 0;
        if (c + 4 <= md.W) {
            *reinterpret_cast<v4i32_any*>(q) = v[k];
        } else {
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (c + e < md.W) q[e] = v[k][e];
        }
    }
}

// Device self-check of the cross-lane moves and the saturating decrement.
__global__ void k_selftest(int32_t* out) {
    const int l = lane_id();
    out[l] = from_left_lane(l + 100);
    out[64 + l] = from_right_lane(l + 100);
    if (l == 0) {
        out[128] = (int32_t)sat_dec(0u);
        out[129] = (int32_t)sat_dec(5u);
        out[130] = (int32_t)sat_dec(kObstacleBit);
        out[131] = (int32_t)max(kObstacleBit, sat_dec(0x7fffffffu));
        out[132] = max3i((int)kObstacleBit, 3, -5);
    }
}

// ---------------------------------------------------------------------------
// launch wrappers
// ---------------------------------------------------------------------------

static int grid_for(int64_t n, int block, int cap = 1 << 20) {
    int64_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

int64_t pack_blocks(int32_t H, int32_t mpitch) {
    const int log_rows = pack_rows_log2(H, mpitch), log_words = 10 - log_rows;
    return (((int64_t)H + (1 << log_rows) - 1) >> log_rows) * (((int64_t)mpitch + (1 << log_words) - 1) >> log_words);
}

hipError_t launch_pack_mask(const uint8_t* occ, const MazeDev& md, uint32_t* mask, hipStream_t s) {
    const PackJob jb{occ, mask, md.H, md.W, md.mpitch, md.mrow, md.mcol, 0};
    const int64_t blocks = pack_blocks(md.H, md.mpitch);
    const auto kernel = pack_rows_log2(md.H, md.mpitch) == 5 ? k_pack_mask<true> : k_pack_mask<false>;
    hipLaunchKernelGGL(kernel, dim3(grid_for(blocks, 1, kPackGrid)), dim3(kPackThreads), 0, s, jb, nullptr, 1, blocks);
    return hipGetLastError();
}

hipError_t launch_fill(int32_t* p, int64_t n_elems, int32_t value, hipStream_t s) {
    if (n_elems <= 0) return hipSuccess;
    const int64_t n4 = n_elems / 4;
    hipLaunchKernelGGL(k_fill, dim3(grid_for(n4 > 0 ? n4 : 1, 256, 65536)), dim3(256), 0, s, p, n_elems, value);
    return hipGetLastError();
}

hipError_t launch_check_sources(const MazeDev& md, const int32_t* src_rc, int32_t n_src, int32_t* sum,
                                uint64_t* posted, uint32_t tag, hipStream_t s) {
    hipLaunchKernelGGL(k_check_sources, dim3(grid_for(n_src, kCheckBlock, kCheckGrid)),
                       dim3(n_src > 256 ? kCheckBlock : 64), 0, s, md, src_rc, n_src, sum, posted, tag);
    return hipGetLastError();
}

hipError_t launch_seed(const RoundArgs& a, int32_t slot, const int32_t* src_rc, const int32_t* src_slot,
                       int32_t n_src, int32_t* bad_count, hipStream_t s) {
    if (n_src <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_seed, dim3(grid_for(n_src, 256)), dim3(256), 0, s, a, slot, src_rc, src_slot, n_src,
                       a.dense ? 0 : 1, bad_count);
    return hipGetLastError();
}

hipError_t launch_start(const RoundArgs& a, StartArgs st, hipStream_t s) {
    const int64_t zero_blocks = (st.n_zero + 4 * kBlockThreads - 1) / (4 * kBlockThreads);
    st.n_zero_blocks = (int32_t)(zero_blocks < 1024 ? zero_blocks : 1024);
    const int64_t words = (int64_t)(sizeof(MazeDev) / 4) * a.n_slots + (int64_t)st.n_started * kSpread;
    const int blocks = (st.n_tiles + kWavesPerBlock - 1) / kWavesPerBlock + st.n_zero_blocks +
                       grid_for(words, kStartWords, 1024);
    hipLaunchKernelGGL(k_start, dim3(blocks), dim3(kBlockThreads), 0, s, a, st);
    return hipGetLastError();
}

hipError_t launch_pack_mask_many(const PackJob& first, const PackJob* jobs, int32_t n_jobs, int64_t blocks,
                                 hipStream_t s) {
    if (n_jobs <= 0 || blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_pack_mask<false>, dim3(grid_for(blocks, 1, kPackGrid)), dim3(kPackThreads), 0, s, first, jobs, n_jobs, blocks);
    return hipGetLastError();
}

hipError_t launch_check_sources_many(const MazeDev* mazes, const int32_t* src_rc, const int32_t* src_slot,
                                     int32_t n, int32_t* bad, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_check_sources_many, dim3(grid_for(n, 256)), dim3(256), 0, s, mazes, src_rc, src_slot, n,
                       bad);
    return hipGetLastError();
}

hipError_t launch_sweep(int T, int C, const RoundArgs& a, int32_t grid, hipStream_t s, hipEvent_t e0,
                        hipEvent_t e1) {
#define X(t, c) \
    if (T == t && C == c) return launch_sweep_T##t##_C##c(a, grid, s, e0, e1);
    OMAP_SWEEP_VARIANTS(X)
#undef X
    return hipErrorInvalidValue;
}

static int sweep_blocks_per_cu(int T, int C) {
#define X(t, c) \
    if (T == t && C == c) return sweep_blocks_per_cu_T##t##_C##c();
    OMAP_SWEEP_VARIANTS(X)
#undef X
    return 0;
}

int sweep_max_waves_per_cu(int T, int C) {
    const int b = sweep_blocks_per_cu(T, C);
    return (b > 1 ? b : 1) * kWavesPerBlock;
}

bool sweep_supported(int T, int C) {
#define X(t, c) if (T == t && C == c) return true;
    OMAP_SWEEP_VARIANTS(X)
#undef X
    return false;
}

hipError_t launch_reduce(const MazeDev* mazes, const int32_t* tile_maze, const uint8_t* touched,
                         int32_t tile_begin, int32_t tile_end, const int32_t* slot_select, int32_t tile_rows,
                         int32_t tile_cols, int32_t parity, int32_t* maze_min,
                         unsigned long long* maze_reached, hipStream_t s) {
    if (tile_end <= tile_begin) return hipSuccess;
    hipLaunchKernelGGL(k_reduce, dim3(tile_end - tile_begin), dim3(256), 0, s, mazes, tile_maze, touched,
                       tile_begin, slot_select, tile_rows, tile_cols, parity, maze_min,
                       maze_reached);
    return hipGetLastError();
}

hipError_t launch_front_report(const MazeDev* mazes, const unsigned long long* reached, const int32_t* layer,
                               const int32_t* last_round, const int64_t* visits, int32_t n_slots, int32_t* maze_min,
                               unsigned long long* maze_reached, int32_t* last_out, int64_t* visits_out,
                               hipStream_t s) {
    hipLaunchKernelGGL(k_front_report, dim3(grid_for(n_slots, 64)), dim3(64), 0, s, mazes, reached, layer, last_round,
                       visits, n_slots, maze_min, maze_reached, last_out, visits_out);
    return hipGetLastError();
}

size_t scan_work_bytes(int32_t n) {
    const size_t nb = ((size_t)n + kScanBlock - 1) / kScanBlock;
    return n <= kScanOneBlock ? 0 : 8 * nb + 4 * kBuckets * (nb + 1);
}

hipError_t launch_lengths_offsets(const MazeDev* mazes, const int32_t* tgt_slot, const int32_t* tgt_rc, int32_t n_tgt,
                                  int32_t parity, int32_t* len, int64_t* offsets, int32_t* order, void* work,
                                  uint64_t* posted, uint32_t tag, hipStream_t s) {
    if (n_tgt > kScanOneBlock && work != nullptr) {
        const int nb = (n_tgt + kScanBlock - 1) / kScanBlock;
        int64_t* const sums = static_cast<int64_t*>(work);
        int32_t* const counts = reinterpret_cast<int32_t*>(sums + nb);
        int32_t* const place = counts + (int64_t)nb * kBuckets;
        hipLaunchKernelGGL(k_block_sums, dim3(nb), dim3(kScanBlock), 0, s, mazes, tgt_slot, tgt_rc, parity, len, n_tgt,
                           sums, counts);
        hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(1024), 0, s, sums, counts, nb, place, posted, tag);
        hipLaunchKernelGGL(k_block_offsets, dim3(nb), dim3(kScanBlock), 0, s, len, n_tgt, sums, place, offsets, order);
        return hipGetLastError();
    }
    const bool within = n_tgt <= kScanLengths;
    if (mazes != nullptr && !within)
        hipLaunchKernelGGL(k_path_lengths, dim3(grid_for(n_tgt, 256)), dim3(256), 0, s, mazes, tgt_slot, tgt_rc, n_tgt,
                           parity, len);
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, s, within ? mazes : nullptr, tgt_slot, tgt_rc, parity, len,
                       n_tgt, offsets, order, posted, tag);
    return hipGetLastError();
}

hipError_t launch_walk(const MazeDev* mazes, const int32_t* tgt_slot, const int32_t* tgt_rc,
                       int32_t n_tgt, int32_t parity, const int32_t* len, const int64_t* offsets,
                       int32_t* cells, int64_t total, hipStream_t s, const int32_t* order, const WalkOut& out) {
    if (n_tgt <= 0) return hipSuccess;
    if ((n_tgt <= kWalkTileTargets && total >= (int64_t)n_tgt * kWalkTileMoves) ||
        (n_tgt <= kWalkTileTargetsLong && total >= (int64_t)n_tgt * kWalkTileMovesLong)) {
        hipLaunchKernelGGL(k_walk_tile, dim3(n_tgt), dim3(kTileWalkThreads), 0, s, mazes, tgt_slot, tgt_rc, n_tgt,
                           parity, len, offsets, cells, order, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_walk<false>, dim3((n_tgt + kWalkWaves - 1) / kWalkWaves), dim3(kLanes * kWalkWaves), 0, s,
                       mazes, tgt_slot, tgt_rc, n_tgt, parity, len, offsets, cells, order, nullptr, 0, out);
    return hipGetLastError();
}

hipError_t launch_walk_random(const MazeDev* mazes, const int32_t* tgt_slot, const int32_t* tgt_rc,
                              const int32_t* tgt_local, int32_t n_tgt, int32_t parity, uint64_t seed,
                              const int32_t* len, const int64_t* offsets, int32_t* cells, hipStream_t s,
                              const int32_t* order, const WalkOut& out) {
    if (n_tgt <= 0) return hipSuccess;
    if (n_tgt > kRandomLaneTargets) {
        hipLaunchKernelGGL(k_walk_random_lanes, dim3((n_tgt + kLanes - 1) / kLanes), dim3(kLanes), 0, s, mazes,
                           tgt_slot, tgt_rc, tgt_local, n_tgt, parity, seed, len, offsets, cells, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_walk<true>, dim3((n_tgt + kWalkWaves - 1) / kWalkWaves), dim3(kLanes * kWalkWaves), 0, s,
                       mazes, tgt_slot, tgt_rc, n_tgt, parity, len, offsets, cells, order, tgt_local, seed, out);
    return hipGetLastError();
}

hipError_t launch_walk_euclid(const MazeDev* mazes, const int32_t* tgt_slot, const int32_t* tgt_rc, int32_t n_tgt,
                              int32_t parity, int32_t* len, const int64_t* offsets, int32_t* cells, int64_t stride,
                              hipStream_t s, const WalkOut& out) {
    if (n_tgt <= 0) return hipSuccess;
    if (n_tgt > kEuclidLaneTargets) {
        const auto kernel = offsets != nullptr ? k_walk_euclid_lanes<true> : k_walk_euclid_lanes<false>;
        hipLaunchKernelGGL(kernel, dim3((n_tgt + kLanes - 1) / kLanes), dim3(kLanes), 0, s, mazes, tgt_slot, tgt_rc,
                           n_tgt, parity, len, offsets, cells, out);
        return hipGetLastError();
    }
    const dim3 grid((n_tgt + kWalkWaves - 1) / kWalkWaves), block(kLanes * kWalkWaves);
    const auto kernel = offsets != nullptr ? k_walk_euclid<true, false>
                        : cells != nullptr ? k_walk_euclid<true, true> : k_walk_euclid<false, true>;
    hipLaunchKernelGGL(kernel, grid, block, 0, s, mazes, tgt_slot, tgt_rc, n_tgt, parity, len, offsets, cells, stride,
                       out);
    return hipGetLastError();
}

hipError_t launch_gather_paths(const int32_t* points, int64_t stride, int32_t n_tgt, const int32_t* len,
                               const int64_t* offsets, int32_t* cells, hipStream_t s, const WalkOut& out) {
    if (n_tgt <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_paths, dim3((n_tgt + kWavesPerBlock - 1) / kWavesPerBlock), dim3(kBlockThreads), 0, s,
                       points, stride, n_tgt, len, offsets, cells, out);
    return hipGetLastError();
}

hipError_t launch_source_index(const MazeDev* mazes, const int32_t* tgt_slot, int32_t n_tgt,
                               const int32_t* len, const int64_t* offsets, const int32_t* cells,
                               const int32_t* src_sorted, const int32_t* src_base, const int32_t* src_n,
                               int32_t* out, hipStream_t s) {
    if (n_tgt <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_source_index, dim3(grid_for(n_tgt, 256)), dim3(256), 0, s, mazes, tgt_slot, n_tgt,
                       len, offsets, cells, src_sorted, src_base, src_n, out);
    return hipGetLastError();
}

hipError_t launch_activity(const MazeDev& md, int32_t parity, int32_t offset, int32_t* dst, int64_t dpitch,
                           hipStream_t s) {
    const int32_t col_blocks = (md.W + 4 * kLanes - 1) / (4 * kLanes);
    const int64_t row_blocks = ((int64_t)md.H + kWavesPerBlock * kCopyRows - 1) / (kWavesPerBlock * kCopyRows);
    hipLaunchKernelGGL(k_activity, dim3((uint32_t)(row_blocks * col_blocks)), dim3(kBlockThreads), 0, s, md, parity,
                       offset, dst, dpitch, col_blocks);
    return hipGetLastError();
}

__global__ void k_round_advance(int32_t* counter, int32_t add) { *counter += add; }

hipError_t launch_round_advance(int32_t* counter, int32_t add, hipStream_t s) {
    hipLaunchKernelGGL(k_round_advance, dim3(1), dim3(1), 0, s, counter, add);
    return hipGetLastError();
}

hipError_t launch_selftest(int32_t* out, hipStream_t s) {
    hipLaunchKernelGGL(k_selftest, dim3(1), dim3(64), 0, s, out);
    return hipGetLastError();
}


}  // namespace omap
