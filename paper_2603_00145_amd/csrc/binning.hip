// K2-K5: exclusive scan of tile counts, (tile, Gaussian) key emission, stable LSD radix sort
// of the keys, and per-tile list ranges.  Together they list, for every voxel tile of every
// grid, the Gaussians whose box overlaps it in ascending Gaussian id (the spatial query that
// stands in for the paper's block partition, Sec. 3.3.1).
#include "gm_internal.h"

namespace {

constexpr int SCAN_THREADS = 256;
constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_CHUNK = SCAN_THREADS * SCAN_ITEMS;
constexpr unsigned SCAN_PREFIX_BLOCKS = 2048;   // final-pass blocks that sum their own prefix

__global__ __launch_bounds__(256) void k_fill_u32(uint32_t* p, uint32_t v, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ __launch_bounds__(256) void k_copy_u32(const uint32_t* src, uint32_t* dst, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

// block-wide exclusive scan of one int64 per thread; returns the block total in *total
__device__ int64_t block_exclusive_scan(int64_t v, int64_t* total)
{
    __shared__ int64_t s_wave[SCAN_THREADS / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int64_t incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int64_t before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < SCAN_THREADS / 64; ++w) {
        const int64_t x = s_wave[w];
        if (w < wave) before += x;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return before + incl - v;
}

__global__ __launch_bounds__(SCAN_THREADS) void k_scan_reduce(const int32_t* in, int64_t n,
                                                               int64_t* part)
{
    const int64_t base = (int64_t)blockIdx.x * SCAN_CHUNK;
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        const int64_t i = base + (int64_t)k * SCAN_THREADS + threadIdx.x;
        if (i < n) s += in[i];
    }
    int64_t tot;
    block_exclusive_scan(s, &tot);
    if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// The chunk totals part[0..nb) replaced by their exclusive prefix sums, in place: one block
// walks them SCAN_CHUNK at a time with a running offset (used when the final pass has too many
// blocks to sum the totals before it one by one).
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_parts(int64_t* part, int64_t nb)
{
    int64_t running = 0;
    for (int64_t c0 = 0; c0 < nb; c0 += SCAN_CHUNK) {
        const int64_t base = c0 + (int64_t)threadIdx.x * SCAN_ITEMS;
        int64_t v[SCAN_ITEMS];
        int64_t sum = 0;
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; ++k) {
            v[k] = base + k < nb ? part[base + k] : 0;
            sum += v[k];
        }
        int64_t tot;
        int64_t run = block_exclusive_scan(sum, &tot) + running;
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; ++k) {
            if (base + k < nb) part[base + k] = run;
            run += v[k];
        }
        running += tot;
    }
}

// prefixed: part holds the exclusive prefix sums of the chunk totals (k_scan_parts ran);
// otherwise each block sums the totals before it.
__global__ __launch_bounds__(SCAN_THREADS) void k_scan_final(const int32_t* in, int64_t n,
                                                              const int64_t* part,
                                                              int64_t* out, int prefixed)
{
    // each thread owns SCAN_ITEMS consecutive elements of the block's chunk, moved with
    // 16-byte loads and stores where the chunk is whole and the buffers are aligned
    static_assert(SCAN_ITEMS == 8, "vector path moves 8 elements per thread");
    const int64_t base = (int64_t)blockIdx.x * SCAN_CHUNK + (int64_t)threadIdx.x * SCAN_ITEMS;
    const bool vec = base + SCAN_ITEMS <= n && ((uintptr_t)in & 31u) == 0 &&
                     ((uintptr_t)out & 15u) == 0;
    int32_t v[SCAN_ITEMS];
    if (vec) {
        const int4 a = *reinterpret_cast<const int4*>(in + base);
        const int4 b = *reinterpret_cast<const int4*>(in + base + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
        v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    } else {
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; ++k) {
            const int64_t i = base + k;
            v[k] = i < n ? in[i] : 0;
        }
    }
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) s += v[k];
    // this block's offset: the sum of the chunk totals before it (read from L2; integer,
    // so the order of the sum does not matter), or its prefix when the totals were scanned
    int64_t before;
    if (prefixed) {
        before = part[blockIdx.x];
    } else {
        int64_t pre = 0;
        for (int64_t b = threadIdx.x; b < (int64_t)blockIdx.x; b += SCAN_THREADS) pre += part[b];
        block_exclusive_scan(pre, &before);
    }
    int64_t tot;
    int64_t run = block_exclusive_scan(s, &tot) + before;
    int64_t r[SCAN_ITEMS];
#pragma unroll
    for (int k = 0; k < SCAN_ITEMS; ++k) {
        r[k] = run;
        run += v[k];
    }
    if (vec) {
        longlong2* o = reinterpret_cast<longlong2*>(out + base);
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS / 2; ++k) o[k] = make_longlong2(r[2 * k], r[2 * k + 1]);
    } else {
#pragma unroll
        for (int k = 0; k < SCAN_ITEMS; ++k)
            if (base + k < n) out[base + k] = r[k];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == SCAN_THREADS - 1) out[n] = run;
}

// The report of gm_bin, which the host reads after a stream synchronisation without a copy (host:
// pinned memory), written by threads 0 .. GM_MAX_GRIDS: every grid's first list entry (emission is
// grid-major and the sort keeps grids apart), the box volumes (to the caller's array as well) and
// the flags.
__device__ __forceinline__ void write_report(int n_grids, const unsigned long long* volume,
                                             const unsigned long long* tiles, uint32_t flags,
                                             int64_t* box_volume, BinReport* host)
{
    const int t = threadIdx.x;
    if (t <= GM_MAX_GRIDS) {
        unsigned long long start = 0ull;
        for (int g = 0; g < min(t, n_grids); ++g) start += tiles[g];
        host->grid_start[t] = t <= n_grids ? (int64_t)start : 0;
    }
    if (t < GM_MAX_GRIDS) host->box_volume[t] = t < n_grids ? volume[t] : 0ull;
    if (t < n_grids) box_volume[t] = (int64_t)volume[t];
    if (t < 4) host->flags[t] = t == 0 ? flags : 0u;
}

// One block: the chunks' tiles replaced by their exclusive prefix sums, and the report.
constexpr int BIN_SCAN_THREADS = 1024;
__global__ __launch_bounds__(BIN_SCAN_THREADS) void k_bin_scan(BinChunks c, int64_t per_grid, int n_grids,
                                                               int64_t* box_volume, BinReport* host)
{
    constexpr int WAVES = BIN_SCAN_THREADS / 64, ITEMS = 4;
    __shared__ int64_t s_wave[WAVES];
    __shared__ unsigned long long s_vol[GM_MAX_GRIDS], s_tiles[GM_MAX_GRIDS];
    __shared__ uint32_t s_flags;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x < GM_MAX_GRIDS) s_vol[threadIdx.x] = s_tiles[threadIdx.x] = 0ull;
    if (threadIdx.x == 0) s_flags = 0u;
    __syncthreads();
    int64_t running = 0;
    uint32_t flags = 0u;
    for (int g = 0; g < n_grids; ++g) {
        const int64_t first = running;
        unsigned long long vol = 0ull;
        for (int64_t c0 = 0; c0 < per_grid; c0 += BIN_SCAN_THREADS * ITEMS) {
            int64_t v[ITEMS], sum = 0;
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int64_t j = c0 + (int64_t)threadIdx.x * ITEMS + k;
                const bool in = j < per_grid;
                v[k] = in ? (int64_t)c.tiles[g * per_grid + j] : 0;
                vol += in ? c.volume[g * per_grid + j] : 0ull;
                flags |= in ? c.flags[g * per_grid + j] : 0u;
                sum += v[k];
            }
            int64_t incl = sum;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int64_t t = __shfl_up(incl, o, 64);
                if (lane >= o) incl += t;
            }
            if (lane == 63) s_wave[wave] = incl;
            __syncthreads();
            int64_t run = running + incl - sum;
            for (int w = 0; w < WAVES; ++w) {
                if (w < wave) run += s_wave[w];
                running += s_wave[w];
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < ITEMS; ++k) {
                const int64_t j = c0 + (int64_t)threadIdx.x * ITEMS + k;
                if (j < per_grid) c.tiles[g * per_grid + j] = (unsigned long long)run;
                run += v[k];
            }
        }
        for (int o = 32; o > 0; o >>= 1) vol += __shfl_down(vol, o, 64);
        if (lane == 0 && vol) atomicAdd(&s_vol[g], vol);
        if (threadIdx.x == 0) s_tiles[g] = (unsigned long long)(running - first);
    }
    if (flags) atomicOr(&s_flags, flags);
    __syncthreads();
    write_report(n_grids, s_vol, s_tiles, s_flags, box_volume, host);
}

// The overlapped tiles (z, y, x order) of (grid, Gaussian) idx into keys and vals from o on, unless
// they run past end.
__device__ __forceinline__ void emit_tiles(const EmitArgs& a, int64_t idx, uint32_t* keys,
                                           uint32_t* vals, int64_t o, int64_t end)
{
    const uint32_t* tb = a.tile_box + idx * 3;
    const uint32_t b0 = tb[0], b1 = tb[1], b2 = tb[2];
    const int lx = (int)(b0 & 0xffffu), ly = (int)(b0 >> 16), lz = (int)(b1 & 0xffffu);
    const int hx = (int)(b1 >> 16), hy = (int)(b2 & 0xffffu), hz = (int)(b2 >> 16);
    if (hx < lx || hy < ly || hz < lz) return;  // empty box: no tile
    const int k = (int)(idx / a.n);
    const uint32_t gid = (uint32_t)(idx - (int64_t)k * a.n);
    const GridConst& G = a.g[k];
    // the emission runs before the host has checked the total against the capacity
    if (o + (int64_t)(hx - lx + 1) * (hy - ly + 1) * (hz - lz + 1) > end) return;
    // the first tile emitted holds the box's lower corner: its entry carries GM_HOME_BIT
    uint32_t home = GM_HOME_BIT;
    for (int tz = lz; tz <= hz; ++tz)
        for (int ty = ly; ty <= hy; ++ty)
            for (int tx = lx; tx <= hx; ++tx) {
                keys[o] = (uint32_t)(G.tile_base + ((int64_t)tz * G.nty + ty) * G.ntx + tx);
                vals[o] = gid | home;
                home = 0u;
                ++o;
            }
}

// A chunk of BIN_CHUNK Gaussians of a grid per block, one per thread, their offsets formed here from
// a scan of their counts and the tiles of the chunks before them, a prefix sum (SCANNED) or summed
// here; without SCANNED the first block also writes the report.  1M Gaussians on three grids 44 us
// with k_bin_scan, 20k 5; with the offsets scanned over all the Gaussians in two launches, written
// and read again, and the report and its clearing in two more, 55 and 15.
constexpr int EMIT_LDS = 2048;     // entries, 16 KB
template <bool SCANNED>
__global__ __launch_bounds__(SCAN_THREADS) void k_emit(const EmitArgs a, int per_grid,
                                                       int64_t* box_volume, BinReport* host)
{
    static_assert(SCAN_THREADS == BIN_CHUNK, "a Gaussian per thread");
    const int c = blockIdx.x, k = c / per_grid;
    if (!SCANNED && c == 0) {
        __shared__ unsigned long long vol[GM_MAX_GRIDS], tiles[GM_MAX_GRIDS];
        __shared__ uint32_t flags;
        if (threadIdx.x < GM_MAX_GRIDS) vol[threadIdx.x] = tiles[threadIdx.x] = 0ull;
        if (threadIdx.x == 0) flags = 0u;
        __syncthreads();
        for (int j = threadIdx.x; j < a.n_grids * per_grid; j += SCAN_THREADS) {
            atomicAdd(&vol[j / per_grid], a.chunks.volume[j]);
            atomicAdd(&tiles[j / per_grid], a.chunks.tiles[j]);
            if (a.chunks.flags[j]) atomicOr(&flags, a.chunks.flags[j]);
        }
        __syncthreads();
        write_report(a.n_grids, vol, tiles, flags, box_volume, host);
    }
    int64_t before, tot;
    if (SCANNED) {
        before = (int64_t)a.chunks.tiles[c];
    } else {
        int64_t pre = 0;
        for (int j = threadIdx.x; j < c; j += SCAN_THREADS) pre += (int64_t)a.chunks.tiles[j];
        block_exclusive_scan(pre, &before);
    }
    const int64_t i = (int64_t)(c - k * per_grid) * BIN_CHUNK + threadIdx.x;
    const int64_t idx = (int64_t)k * a.n + i;
    const int64_t o = block_exclusive_scan(i < a.n ? a.tile_count[idx] : 0, &tot);
    // through LDS, so that consecutive threads write consecutive entries (a thread's own few, one
    // after the other, left 256 runs of stores a block: 2M Gaussians on one grid 43 us, 25 now);
    // what does not fit there or past the capacity goes out directly
    __shared__ uint32_t skey[EMIT_LDS], sval[EMIT_LDS];
    if (tot <= EMIT_LDS && before + tot <= a.capacity) {
        if (i < a.n) emit_tiles(a, idx, skey, sval, o, tot);
        __syncthreads();
        for (int e = threadIdx.x; e < (int)tot; e += SCAN_THREADS) {
            a.keys[before + e] = skey[e];
            a.vals[before + e] = sval[e];
        }
    } else if (i < a.n) {
        emit_tiles(a, idx, a.keys, a.vals, before + o, a.capacity);
    }
}

// ---- radix sort --------------------------------------------------------------------------
// The scatter's block holds 4096 keys (32 KB of LDS for keys and values): eight waves of
// eight 64-key rounds, so that a CU keeps 24 waves (three blocks) in flight through the load
// and store bursts.
//
// A short list (RS_FEW_BLOCKS) takes blocks of 2048 keys, whose digit counts are kept block by
// block and which sum the counts of all blocks for their offsets themselves: two launches a pass
// in place of four, and twice the blocks on an otherwise empty chip.  With one pass (at most 256
// tiles) the first block also knows every tile's start.  125k pairs in one pass 29 -> 12 us, 350k in
// two 47 -> 33.  The table each block reads grows with the blocks (1 KB each): at 1.35M pairs it
// would be 660 KB for each of 660 blocks.
constexpr int RS_THREADS = 512;
constexpr int RS_WAVES = RS_THREADS / 64;
template <bool FEW> constexpr int RS_ROUNDS = FEW ? 4 : 8;
template <bool FEW> constexpr int RS_BLOCK_KEYS = 64 * RS_ROUNDS<FEW> * RS_WAVES;
constexpr int64_t RS_FEW_BLOCKS = 192;
constexpr int RS_HIST_THREADS = 256;  // one per digit
static_assert(RS_BLOCK_KEYS<true> % (4 * RS_HIST_THREADS) == 0, "whole 16-byte loads per thread");
static_assert(RS_THREADS >= 256 && RS_THREADS % 256 == 0, "the digit phase uses the first 256 threads");

// Digit counts of one scatter block's keys.  Each wave counts into its own LDS histogram
// (fewer colliding atomics), full blocks read four keys per 16-byte load and add each run of
// equal digits among a load's four keys once (keys emitted for Gaussians close in space share
// tiles, so runs are common and fewer lanes collide), and the four histograms are summed per
// digit at the end.  ghist is digit-major ([digit][block]), or for FEW block-major.
template <bool FEW>
__global__ __launch_bounds__(RS_HIST_THREADS) void k_rs_hist(const uint32_t* keys, int64_t n,
                                                              int shift, uint32_t mask,
                                                              int32_t* ghist, int64_t nblocks)
{
    constexpr int HW = RS_HIST_THREADS / 64;
    constexpr int KEYS = RS_BLOCK_KEYS<FEW>;
    __shared__ uint32_t h[HW][256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int d = lane; d < 256; d += 64) h[wave][d] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * KEYS;
    const int64_t rem = n - base;
    const int nk = rem < KEYS ? (int)rem : KEYS;
    uint32_t* hw = h[wave];
    if (nk == KEYS && (reinterpret_cast<uintptr_t>(keys) & 15u) == 0) {
        const uint4* k4 = reinterpret_cast<const uint4*>(keys + base);
        uint4 v[KEYS / 4 / RS_HIST_THREADS];
#pragma unroll
        for (int j = 0; j < KEYS / 4 / RS_HIST_THREADS; ++j)
            v[j] = k4[threadIdx.x + j * RS_HIST_THREADS];
#pragma unroll
        for (int j = 0; j < KEYS / 4 / RS_HIST_THREADS; ++j) {
            const uint32_t d0 = (v[j].x >> shift) & mask, d1 = (v[j].y >> shift) & mask;
            const uint32_t d2 = (v[j].z >> shift) & mask, d3 = (v[j].w >> shift) & mask;
            // run lengths from each key to the end of its run of equal digits
            const uint32_t l3 = 1u;
            const uint32_t l2 = d3 == d2 ? l3 + 1u : 1u;
            const uint32_t l1 = d2 == d1 ? l2 + 1u : 1u;
            const uint32_t l0 = d1 == d0 ? l1 + 1u : 1u;
            // each run counted once, at its first key
            atomicAdd(&hw[d0], l0);
            if (d1 != d0) atomicAdd(&hw[d1], l1);
            if (d2 != d1) atomicAdd(&hw[d2], l2);
            if (d3 != d2) atomicAdd(&hw[d3], l3);
        }
    } else {
        for (int k = threadIdx.x; k < nk; k += RS_HIST_THREADS)
            atomicAdd(&hw[(keys[base + k] >> shift) & mask], 1u);
    }
    __syncthreads();
    const int d = threadIdx.x;
    if (d <= (int)mask) {  // the pass's digits only: rows of the digit-major histogram
        uint32_t t = 0;
#pragma unroll
        for (int w = 0; w < HW; ++w) t += h[w][d];
        ghist[FEW ? (int64_t)blockIdx.x * 256 + d : (int64_t)d * nblocks + blockIdx.x] = (int32_t)t;
    }
}

// Stable scatter.  Each wave of the block owns a run of keys and takes
// them in RS_ROUNDS rounds of 64 consecutive keys; lanes with equal digits are matched with ballots,
// so every key learns how many equal-digit keys precede it in the block.  The block's keys are
// first placed in LDS in digit order, then written out by consecutive threads, so that each
// digit's run leaves the block as one contiguous stretch of stores.  goff: the scanned digit-major
// counts; FEW reads the block-major counts, and with tile_start the first block writes where each
// digit (then the whole key) starts, for tiles 0 .. tiles.
template <bool FEW>
__global__ __launch_bounds__(RS_THREADS) void k_rs_scatter(const uint32_t* kin,
                                                            const uint32_t* vin, uint32_t* kout,
                                                            uint32_t* vout, int64_t n, int shift,
                                                            int dbits, const int64_t* goff,
                                                            const int32_t* ghist, int64_t nblocks,
                                                            int32_t* tile_start, int tiles)
{
    constexpr int ROUNDS = RS_ROUNDS<FEW>, KEYS = RS_BLOCK_KEYS<FEW>, WAVE_KEYS = 64 * ROUNDS;
    __shared__ uint32_t wcnt[RS_WAVES][256];
    __shared__ uint32_t wsum[RS_WAVES], wall[RS_WAVES];
    __shared__ uint32_t s_all[FEW ? RS_THREADS : 1], s_pre[FEW ? RS_THREADS : 1];
    __shared__ uint32_t dstart[256];
    __shared__ int64_t obase[256];
    __shared__ uint32_t skey[KEYS];
    __shared__ uint32_t sval[KEYS];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t mask = (1u << dbits) - 1u;
    for (int d = lane; d < 256; d += 64) wcnt[wave][d] = 0;
    __syncthreads();
    const uint64_t lt = (1ull << lane) - 1ull;
    const int64_t bbase = (int64_t)blockIdx.x * KEYS;
    const int64_t wbase = bbase + (int64_t)wave * WAVE_KEYS;
    uint32_t key[ROUNDS], val[ROUNDS], rank[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int64_t i = wbase + r * 64 + lane;
        const bool ok = i < n;
        key[r] = ok ? kin[i] : 0u;
        val[r] = ok ? vin[i] : 0u;
        const uint32_t dg = (key[r] >> shift) & mask;
        uint64_t peers = __ballot(ok);
        for (int b = 0; b < dbits; ++b) {
            const bool bit = (dg >> b) & 1u;
            const uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t before = (uint32_t)__popcll(peers & lt);
        uint32_t base = 0;
        if (ok) base = wcnt[wave][dg];
        rank[r] = base + before;
        if (ok && before == 0) wcnt[wave][dg] = base + (uint32_t)__popcll(peers);
    }
    if constexpr (FEW) {
        // the digit's count over all blocks and over those before this one, half of the blocks to
        // each half of the threads (digit threadIdx.x mod 256); rows past the mask are not written
        const int dd = threadIdx.x & 255;
        uint32_t all = 0, pre = 0;
        if (dd <= (int)mask) {
#pragma unroll 8
            for (int b = threadIdx.x >> 8; b < (int)nblocks; b += 2) {
                const uint32_t t = (uint32_t)ghist[b * 256 + dd];
                all += t;
                pre += b < (int)blockIdx.x ? t : 0u;
            }
        }
        s_all[threadIdx.x] = all;
        s_pre[threadIdx.x] = pre;
    }
    __syncthreads();
    // per digit: offsets of the waves' runs, the digit's block total, and its block-local
    // start (exclusive scan over the 256 digits: within each wave with shuffles, then across
    // the four waves)
    // (thread d < 256 takes digit d; waves 0-3 are whole, so the shuffles see full waves)
    const int d = threadIdx.x;
    const bool dig = d < 256;
    uint32_t run = 0, incl = 0, all = 0, all_incl = 0;
    if (dig) {
#pragma unroll
        for (int w = 0; w < RS_WAVES; ++w) {
            const uint32_t t = wcnt[w][d];
            wcnt[w][d] = run;
            run += t;
        }
        incl = run;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o);
            if (lane >= o) incl += y;
        }
        if (lane == 63) wsum[wave] = incl;
        if constexpr (FEW) {
            all = s_all[d] + s_all[d + 256];
            all_incl = all;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = __shfl_up(all_incl, o);
                if (lane >= o) all_incl += y;
            }
            if (lane == 63) wall[wave] = all_incl;
        }
    }
    __syncthreads();
    if (dig) {
        uint32_t before_w = 0;
        for (int w = 0; w < wave; ++w) before_w += wsum[w];
        const uint32_t ds = before_w + incl - run;
        dstart[d] = ds;
        if constexpr (FEW) {
            uint32_t first = all_incl - all;   // of the digit in the whole list
            for (int w = 0; w < wave; ++w) first += wall[w];
            obase[d] = (int64_t)first + s_pre[d] + s_pre[d + 256] - (int64_t)ds;
            if (tile_start && blockIdx.x == 0) {
                if (d <= tiles) tile_start[d] = (int32_t)first;
                if (d == 255 && tiles == 256) tile_start[256] = (int32_t)(first + all);
            }
        } else {
            obase[d] = d <= (int)mask ? goff[(int64_t)d * nblocks + blockIdx.x] - (int64_t)ds : 0;
        }
    }
    __syncthreads();
    // place the keys in digit order in LDS (positions < KEYS by construction)
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int64_t i = wbase + r * 64 + lane;
        if (i < n) {
            const uint32_t dg = (key[r] >> shift) & mask;
            const uint32_t lp = dstart[dg] + wcnt[wave][dg] + rank[r];
            skey[lp] = key[r];
            sval[lp] = val[r];
        }
    }
    __syncthreads();
    const int64_t rem = n - bbase;
    const int nkeys = rem < KEYS ? (int)rem : KEYS;
    for (int i = threadIdx.x; i < nkeys; i += RS_THREADS) {
        const uint32_t k = skey[i];
        const int64_t pos = obase[(k >> shift) & mask] + i;
        kout[pos] = k;
        vout[pos] = sval[i];
    }
}

__global__ __launch_bounds__(256) void k_tile_ranges(const uint32_t* keys, int64_t n,
                                                      int32_t* start, int64_t T)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t > T) return;
    int64_t lo = 0, hi = n;  // first index with keys[idx] >= t
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (keys[mid] < (uint32_t)t) lo = mid + 1;
        else hi = mid;
    }
    start[t] = (int32_t)lo;
}

inline unsigned grid_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

hipError_t launch_fill_u32(uint32_t* p, uint32_t value, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    unsigned nb = grid_for(n, 256);
    if (nb > 4096) nb = 4096;
    hipLaunchKernelGGL(k_fill_u32, dim3(nb), dim3(256), 0, s, p, value, n);
    return hipGetLastError();
}

hipError_t launch_bin_scan(const BinChunks& chunks, int64_t per_grid, int n_grids,
                           int64_t* box_volume, BinReport* host, hipStream_t s)
{
    hipLaunchKernelGGL(k_bin_scan, dim3(1), dim3(BIN_SCAN_THREADS), 0, s, chunks, per_grid, n_grids,
                       box_volume, host);
    return hipGetLastError();
}

hipError_t launch_copy_u32(const uint32_t* src, uint32_t* dst, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    unsigned nb = grid_for(n, 256);
    if (nb > 8192) nb = 8192;
    hipLaunchKernelGGL(k_copy_u32, dim3(nb), dim3(256), 0, s, src, dst, n);
    return hipGetLastError();
}

size_t scan_workspace_bytes(int64_t n)
{
    return (size_t)(grid_for(n > 0 ? n : 1, SCAN_CHUNK)) * sizeof(int64_t) + 256;
}

hipError_t launch_scan_i32_to_i64(const int32_t* in, int64_t* out, int64_t n, void* ws,
                                  hipStream_t s)
{
    if (n <= 0) {
        hipLaunchKernelGGL(k_fill_u32, dim3(1), dim3(256), 0, s, reinterpret_cast<uint32_t*>(out),
                           0u, (int64_t)2);
        return hipGetLastError();
    }
    const unsigned nb = grid_for(n, SCAN_CHUNK);
    int64_t* part = reinterpret_cast<int64_t*>(ws);
    hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(SCAN_THREADS), 0, s, in, n, part);
    // up to SCAN_PREFIX_BLOCKS blocks each sum the totals before them (a few L2 reads per
    // thread); beyond, one more pass scans the totals so that the final pass stays linear
    const int prefixed = nb > SCAN_PREFIX_BLOCKS ? 1 : 0;
    if (prefixed)
        hipLaunchKernelGGL(k_scan_parts, dim3(1), dim3(SCAN_THREADS), 0, s, part, (int64_t)nb);
    hipLaunchKernelGGL(k_scan_final, dim3(nb), dim3(SCAN_THREADS), 0, s, in, n, part, out,
                       prefixed);
    return hipGetLastError();
}

hipError_t launch_emit(const EmitArgs& a, bool scanned, int64_t* box_volume, BinReport* host,
                       hipStream_t s)
{
    if (a.n == 0) return hipSuccess;
    const unsigned per_grid = grid_for(a.n, BIN_CHUNK);
    const dim3 grid(per_grid * (unsigned)a.n_grids);
    if (scanned)
        hipLaunchKernelGGL(k_emit<true>, grid, dim3(SCAN_THREADS), 0, s, a, (int)per_grid, box_volume,
                           host);
    else
        hipLaunchKernelGGL(k_emit<false>, grid, dim3(SCAN_THREADS), 0, s, a, (int)per_grid, box_volume,
                           host);
    return hipGetLastError();
}

static void launch_tile_ranges(const uint32_t* sorted_keys, int64_t n_pairs, int32_t* tile_start,
                               int64_t total_tiles, hipStream_t s)
{
    hipLaunchKernelGGL(k_tile_ranges, dim3(grid_for(total_tiles + 1, 256)), dim3(256), 0, s,
                       sorted_keys, n_pairs, tile_start, total_tiles);
}

// (a short list's block-major counts, twice the blocks, fit where the long list's lie)
size_t radix_workspace_bytes(int64_t n)
{
    const int64_t nb = (n + RS_BLOCK_KEYS<false> - 1) / RS_BLOCK_KEYS<false>;
    const int64_t hn = 256 * (nb > 0 ? nb : 1);
    // ghist (int32), offsets (int64, hn + 1), scan partials
    return (size_t)hn * 4 + 256 + (size_t)(hn + 1) * 8 + 256 + scan_workspace_bytes(hn) + 256;
}

hipError_t launch_radix_sort(uint32_t* keys, uint32_t* vals, uint32_t* keys_alt,
                             uint32_t* vals_alt, int64_t n, int bits, void* ws,
                             int32_t* tile_start, int64_t tiles, hipStream_t s)
{
    if (bits <= 0) {   // one tile
        launch_tile_ranges(keys, n, tile_start, tiles, s);
        return hipGetLastError();
    }
    const int passes = (bits + 7) / 8;
    const int dbits = (bits + passes - 1) / passes;
    const int64_t few = (n + RS_BLOCK_KEYS<true> - 1) / RS_BLOCK_KEYS<true>;
    if (few <= RS_FEW_BLOCKS) {
        int32_t* counts = reinterpret_cast<int32_t*>(ws);
        for (int p = 0; p < passes; ++p) {
            const int shift = p * dbits;
            const int db = (bits - shift) < dbits ? (bits - shift) : dbits;
            hipLaunchKernelGGL(k_rs_hist<true>, dim3((unsigned)few), dim3(RS_HIST_THREADS), 0, s, keys,
                               n, shift, (1u << db) - 1u, counts, few);
            hipLaunchKernelGGL(k_rs_scatter<true>, dim3((unsigned)few), dim3(RS_THREADS), 0, s, keys,
                               vals, keys_alt, vals_alt, n, shift, db, nullptr, counts, few,
                               passes == 1 ? tile_start : nullptr, (int)tiles);
            uint32_t* t = keys; keys = keys_alt; keys_alt = t;
            t = vals; vals = vals_alt; vals_alt = t;
        }
        if (passes > 1) launch_tile_ranges(keys, n, tile_start, tiles, s);
        return hipGetLastError();
    }
    const int64_t nb = (n + RS_BLOCK_KEYS<false> - 1) / RS_BLOCK_KEYS<false>;
    const int64_t hn = 256 * nb;
    char* w = reinterpret_cast<char*>(ws);
    int32_t* ghist = reinterpret_cast<int32_t*>(w);
    w += ((size_t)hn * 4 + 255) / 256 * 256 + 256;
    int64_t* goff = reinterpret_cast<int64_t*>(w);
    w += ((size_t)(hn + 1) * 8 + 255) / 256 * 256 + 256;
    void* sws = w;
    uint32_t *ki = keys, *vi = vals, *ko = keys_alt, *vo = vals_alt;
    hipError_t err = hipSuccess;
    for (int p = 0; p < passes; ++p) {
        const int shift = p * dbits;
        const int db = (bits - shift) < dbits ? (bits - shift) : dbits;
        const uint32_t mask = (1u << db) - 1u;
        // the histogram holds the pass's 2^db digit rows of nb block counts each
        const int64_t hrows = (int64_t)nb << db;
        hipLaunchKernelGGL(k_rs_hist<false>, dim3((unsigned)nb), dim3(RS_HIST_THREADS), 0, s, ki, n, shift,
                           mask, ghist, nb);
        err = launch_scan_i32_to_i64(ghist, goff, hrows, sws, s);
        if (err != hipSuccess) return err;
        hipLaunchKernelGGL(k_rs_scatter<false>, dim3((unsigned)nb), dim3(RS_THREADS), 0, s, ki, vi, ko,
                           vo, n, shift, db, goff, nullptr, nb, nullptr, 0);
        uint32_t* t = ki; ki = ko; ko = t;
        t = vi; vi = vo; vo = t;
    }
    launch_tile_ranges(ki, n, tile_start, tiles, s);
    return hipGetLastError();
}
