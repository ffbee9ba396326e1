// K6: forward rendering of Magnetic Gaussians onto voxel tiles (Eq. 7; on stacks the
// Gaussian is pre-convolved with the slice profile, so the same formula applies with the
// record's amplitude and conic).
//
// A block owns one GM_TX x GM_TY x GM_TZ tile.  The tile's Gaussian list (ascending id) is cut
// into 2 to 16 parts (parts_of), one wavefront each, and every wavefront sums its part into its
// own LDS copy of the tile; the copies are added in a fixed order at the end.  (With one
// wavefront per tile the 192 tiles of three 64x64x16 stacks left most of the chip idle, each
// wavefront walking some 750 entries one dependent pass after the other: k_render 182 us, 33 us
// with 16 parts; at three 128x128x32 stacks 258 against 105 us.)
//
// A wavefront walks its part in batches of 32: a lane loads one record and prepares that
// Gaussian's piece (box intersect tile) in LDS.  Then the pieces are taken one pass after the
// other, in an order that fills the passes (place_piece).  A
// lane holds one (x, y) column of a piece's footprint and evaluates it on the tile's four
// planes, so the in-plane part of the exponent is formed once per column.  The tile keeps a
// column's four voxels side by side: a lane adds its column with one 16-byte read and one
// 16-byte write whatever planes the piece reaches (a plane outside the box gets exactly 0).
// What bounds it at the 256^3 workload is vector issue (92% busy; LDS 77%, of which 23 of bank
// conflicts): about 50 instructions per pass, four of them exponentials.  463 us there, 494 for a
// 320^3 volume of 2M Gaussians; with the pieces in list order and every piece added by itself 505
// and 545.  Evaluating only the planes a pass reaches (ten straight-line variants behind one
// branch, two halves of the tile, a path of its own for wide pieces) issued fewer but ran 4 to 13%
// slower, fetching the next pass's pieces one pass ahead 2-5% slower, and padding the tile's rows
// to 17, 20 or 21 columns changed no time.  A column is read and written whole, so pieces that
// reach few of the four planes pay for the others: 256x256x64 stacks of Gaussians 1.5 to 8 voxels
// wide are rendered 4 to 14% slower than with one add per voxel and reached plane.
// Short lists are taken by one wavefront a tile (k_render_one), with the same sums.
// Two consecutive pieces whose footprints sum to at most 64 columns share the wave (the first
// piece's columns on the low lanes).  Where no column is in both they are added at once, otherwise
// the first piece's lanes add into the tile before the second's, so every voxel's sum is formed in a fixed order and the result is the same on every
// run.
//
// With the paper's block query on a rotated grid (k_render_block, and k_render_field's MASK
// form) a Gaussian's voxels are not its box: each evaluated voxel of the box is also tested
// against the Gaussian's cell block (Eqs. 4-6) and gets zero when it fails (k_render_block
// forms the tile's voxel cells once per tile in LDS; the field kernel, short of LDS, forms
// them per voxel).
#include "nrf_core.h"

namespace {

__device__ __forceinline__ int sgpr(int v) { return __builtin_amdgcn_readfirstlane(v); }

// The tile in LDS: column (x, y) of the tile holds its GM_TZ voxels side by side, so that a
// lane adds a whole column with one 16-byte read and one 16-byte write; rows of the tile are
// ACC_P columns apart.
static_assert(GM_TX == 16 && GM_TY == 16 && GM_TZ == 4, "16 x 16 columns of one float4 each");
constexpr int ACC_P = 16;
constexpr int ACC_COLS = GM_TY * ACC_P;

// Per (Gaussian, tile) piece, prepared lane-parallel for a batch of list entries, in the
// frame of the piece's intersection origin (the box clipped to the tile): the centre's x offset
// plus 1/2 and its y offset, log2 of the amplitude, the base-2 conic (off-diagonals doubled),
// the footprint width (as a float and its reciprocal), the LDS column of the origin minus 1/2,
// and the z offset from the centre of each of the tile's planes (DZ_OUT on planes outside the
// box, where the value is then 2^-huge = 0).
struct alignas(16) Piece {
    float uxh, uy, lamp, kxx;
    float kyy, kzz, kxy, kxz;
    float kyz, inv_wx, wxf, basef;
    float dz0, dz1, dz2, dz3;
};
// kzz <= -KZZ_MIN (see accumulate_tile), so kzz dz^2 of a plane outside the box is at most
// -1e20 and the exponential exactly 0
constexpr float DZ_OUT = 1e25f, KZZ_MIN = 1e-30f;

// Keeps the compiler from moving or merging LDS accesses across this point.  The two groups of
// lanes of a wave that hold two different Gaussians may touch the same voxel; their
// read-add-writes must stay two separate, ordered sequences.
__device__ __forceinline__ void lds_order() { __asm__ __volatile__("" ::: "memory"); }

// Column f of piece p, passed as fh = f + 1/2: its values w = amp 2^Q on the tile's four planes,
// and its LDS column.  The column is (x, y) = (f mod wx, f div wx), found as
// y = floor(fh / wx) (the fraction (x + 1/2) / wx stays at least 1/(2 wx) from an integer, far
// beyond the reciprocal's error) and x + 1/2 = fh - y wx, all exact in float.
// Q = qxy + dz (bz + kzz dz) with qxy = dx (kxx dx + kxy dy) + kyy dy^2 + log2 amp and
// bz = kxz dx + kyz dy: centred in every axis, so no large terms cancel.
__device__ __forceinline__ void eval_column(const Piece& p, float fh, float4& w, int& col)
{
    const float yf = floorf(fh * p.inv_wx);
    const float xh = fmaf(-yf, p.wxf, fh);
    const float dx = xh - p.uxh;
    const float dy = yf - p.uy;
    col = (int)fmaf(yf, (float)ACC_P, xh + p.basef);     // an exact small integer
    const float qxy = fmaf(dx, fmaf(p.kxy, dy, p.kxx * dx), fmaf(p.kyy * dy, dy, p.lamp));
    const float bz = fmaf(p.kxz, dx, p.kyz * dy);
    w.x = __builtin_amdgcn_exp2f(fmaf(p.dz0, fmaf(p.kzz, p.dz0, bz), qxy));
    w.y = __builtin_amdgcn_exp2f(fmaf(p.dz1, fmaf(p.kzz, p.dz1, bz), qxy));
    w.z = __builtin_amdgcn_exp2f(fmaf(p.dz2, fmaf(p.kzz, p.dz2, bz), qxy));
    w.w = __builtin_amdgcn_exp2f(fmaf(p.dz3, fmaf(p.kzz, p.dz3, bz), qxy));
}

// The block query on a masked grid (Sec. 3.3.1, Eqs. 4-6): per piece of the batch, its first
// voxel in the plane, in grid coordinates, and its Gaussian's cell; per tile, the grid's
// index -> world affine and the query's resolution and radius.
struct PieceCell {
    int ix0, iy0, pad0, pad1;
    int4 cm;
};
struct MaskCtx {
    bool on;                // the tile's grid is masked
    const PieceCell* pcc;   // the wavefront's batch
    const double* m;
    double res;
    int radius;
    int t0z;                // the tile's first plane
    const int* vc;          // the tile's voxel cells [3][GM_TILE_VOX] (x, y, z planes), or NULL
};

// w = 0 on the planes of column fh of piece p (LDS column col, as eval_column maps it) whose
// voxel lies outside the block: from the tile's voxel cells when they are staged, else formed
// here
__device__ __forceinline__ void mask_column(const Piece& p, const PieceCell& q, const MaskCtx& mc,
                                            float fh, int col, float4& w)
{
    bool in[GM_TZ];
    if (mc.vc) {
        const long long r = mc.radius;
        // a lane past its piece reads some voxel's cells and stores nothing
        const int cc = min(max(col, 0), ACC_COLS - 1);
        const int v0 = min((cc / ACC_P) * GM_TX + cc % ACC_P, GM_TX * GM_TY - 1);
#pragma unroll
        for (int k = 0; k < GM_TZ; ++k) {
            const int vi = v0 + k * GM_TX * GM_TY;
            const long long dx = (long long)mc.vc[vi] - q.cm.x;
            const long long dy = (long long)mc.vc[GM_TILE_VOX + vi] - q.cm.y;
            const long long dz = (long long)mc.vc[2 * GM_TILE_VOX + vi] - q.cm.z;
            in[k] = dx >= -r && dx <= r && dy >= -r && dy <= r && dz >= -r && dz <= r;
        }
    } else {
        const float yf = floorf(fh * p.inv_wx);
        const float xh = fmaf(-yf, p.wxf, fh);        // x + 1/2 within the piece
        const int x = q.ix0 + (int)xh, y = q.iy0 + (int)yf;
#pragma unroll
        for (int k = 0; k < GM_TZ; ++k)
            in[k] = voxel_in_block(mc.m, mc.res, mc.radius, x, y, mc.t0z + k, q.cm);
    }
    if (!in[0]) w.x = 0.0f;
    if (!in[1]) w.y = 0.0f;
    if (!in[2]) w.z = 0.0f;
    if (!in[3]) w.w = 0.0f;
}

__device__ __forceinline__ void add_column(float4* acc, int col, const float4& w)
{
    float4 o = acc[col];
    o.x += w.x;
    o.y += w.y;
    o.z += w.z;
    o.w += w.w;
    acc[col] = o;
}

// List entries prepared per batch.
constexpr int RB = 32;

// LDS of NW wavefronts: their pieces, then their copies of the tile.  (In a pass of the last of
// RB pieces, the lanes past its footprint read the 64 bytes after it and store nothing; the
// copies follow so that those bytes are the block's own.)
template <int NW>
struct TileLds {
    Piece pcs[NW][RB];
    float4 accs[NW * ACC_COLS];
};

// Barrier before LDS written by some lanes of a wavefront is read by others of the same
// wavefront, which owns that LDS: a wavefront's LDS accesses execute in order, so only the
// compiler has to keep them in order.
__device__ __forceinline__ void wave_sync()
{
    lds_order();
    __builtin_amdgcn_wave_barrier();
}

// Origin and grid of flattened tile t of a launch (t < a.total_blocks).
struct TilePos {
    const RenderGrid* G;
    int lt;                 // tile within its grid
    int t0x, t0y, t0z;      // first voxel
};

__device__ __forceinline__ TilePos tile_pos(const RenderArgs& a, int t)
{
    int r = 0;
#pragma unroll 1
    while (r + 1 < a.n_render && t >= a.rg[r + 1].first_block) ++r;
    TilePos p;
    p.G = &a.rg[r];
    p.lt = t - p.G->first_block;
    const int tx = p.lt % p.G->ntx, ty = (p.lt / p.G->ntx) % p.G->nty;
    const int tz = p.lt / (p.G->ntx * p.G->nty);
    p.t0x = tx * GM_TX;
    p.t0y = ty * GM_TY;
    p.t0z = tz * GM_TZ;
    return p;
}

// Columns per thread in the epilogues of a tile finished by T threads (at least one).
template <int T>
constexpr int cols_per_thread() { return GM_TX * GM_TY / T > 0 ? GM_TX * GM_TY / T : 1; }

// loss mode: the tile's data values, loaded before the Gaussian list is walked so that their
// latency is hidden behind the accumulation (thread t of T: columns t, t + T, ...)
template <int T>
__device__ __forceinline__ void load_targets(const TilePos& P, int t,
                                             float (&tv)[cols_per_thread<T>()][GM_TZ])
{
    const RenderGrid& G = *P.G;
#pragma unroll
    for (int j = 0; j < cols_per_thread<T>(); ++j) {
        const int c = (j * T + t) % (GM_TX * GM_TY);
        const int gx = P.t0x + c % GM_TX, gy = P.t0y + c / GM_TX;
#pragma unroll
        for (int z = 0; z < GM_TZ; ++z) {
            const int gz = P.t0z + z;
            // outside the grid: a valid address (voxel 0) whose value goes unused
            const bool in = (gx < G.nx) & (gy < G.ny) & (gz < G.nz);
            const size_t v = in ? ((size_t)gz * G.ny + gy) * G.nx + gx : 0;
            tv[j][z] = __builtin_nontemporal_load(G.target + v);
        }
    }
}

// The lane's piece and column of one pass: lanes [0, Fa) take columns of piece j, the others
// of piece j + 1.
struct Pass {
    Piece p;
    float fh;
};
__device__ __forceinline__ Pass load_pass(const Piece* pc, int j, int Fa, int lane,
                                          float lane_fh)
{
    Pass q;
    const bool first = lane < Fa;
    q.p = *reinterpret_cast<const Piece*>(reinterpret_cast<const char*>(pc + j) +
                                          (first ? 0 : (int)sizeof(Piece)));
    q.fh = lane_fh - (first ? 0.0f : (float)Fa);
    return q;
}

// Place of a batch's piece with a footprint of F columns (called by the batch's lanes, below 32).
// Consecutive pieces share a pass where their columns fit 64: pieces of 33 to 48 columns go first,
// each before one of up to 16, then those of 17 to 32, which fit each other, then what is left.
// In list order a piece took 0.64 passes and 0.81 adds into the tile (two pieces of a pass that do
// not meet are added as one) at the 256^3 workload; in this order 0.58 and 0.71.  Sorted by size
// and matched from both ends it would be 0.55 passes; left and right pieces in turn, 0.68 adds
// (0.8% faster there, 0.3% slower with the field).
__device__ __forceinline__ int place_piece(int F)
{
    const bool a = F <= 16, b = !a && F <= 32, c = F > 32 && F <= 48;
    const uint32_t ma = (uint32_t)__ballot(a), mb = (uint32_t)__ballot(b), mc = (uint32_t)__ballot(c);
    const uint32_t md = (uint32_t)__ballot(F > 48);
    const int na = __popc(ma), nb = __popc(mb), nc = __popc(mc), m = min(na, nc);
    const int r = (int)__builtin_amdgcn_mbcnt_lo(a ? ma : b ? mb : c ? mc : md, 0u);
    if (a) return r < m ? 2 * r + 1 : nc + nb + r;
    if (b) return nc + m + r;
    if (c) return r < m ? 2 * r : m + r;
    return nc + nb + na + r;
}

// A tile's list [s, e) is cut into 2^a.parts_log2 parts (2 to 16), whole batches each: part k
// starts at entry part_start(k), and part_start(2^parts_log2) >= e.
struct TileList {
    int s, e, nbatch, log2p;
    __device__ __forceinline__ int part_start(int k) const
    {
        return s + ((nbatch * k) >> log2p) * RB;     // at most 2^31 / RB batches, 16 parts
    }
};
__device__ __forceinline__ TileList tile_list(const RenderArgs& a, const TilePos& P)
{
    const int64_t bt = P.G->bin_tile_base + P.lt;
    TileList l;
    l.s = sgpr(a.tile_start[bt]);
    l.e = sgpr(a.tile_start[bt + 1]);
    l.nbatch = (l.e - l.s + RB - 1) / RB;
    l.log2p = a.parts_log2;
    return l;
}

__device__ __forceinline__ float4 add4(const float4& a, const float4& b)
{
    return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
}

// acc (the tile's columns, LDS, owned by this wavefront) = the sum of parts [k0, k0 + np) of the
// tile's list, each part summed in list order and the parts one after the other (np > 1 only with
// PARTS).  Ends with a wave_sync.  MASK: on a masked grid every voxel is also tested against its
// Gaussian's cell block (pcc: the batch's PieceCells; vcell, when given: the tile's voxel cells).
template <bool MASK, bool PARTS>
__device__ __forceinline__ void accumulate_tile(const RenderArgs& a, const TilePos& P, float4* acc,
                                                Piece* pc, int lane, int k0, int np,
                                                PieceCell* pcc, const int* vcell)
{
    const TileList L = tile_list(a, P);
    const int s = L.part_start(k0), e = min(L.e, L.part_start(k0 + np));
    // PARTS: the sum of the finished parts, lane's columns lane + 64 j, and the next part's start
    float4 tot[4] = {};
    int k = k0 + 1, next = PARTS ? L.part_start(k0 + 1) : 0;
    // the part that ends before entry b is added; parts without entries would add zeros
    auto flush = [&](int b) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            tot[j] = add4(tot[j], acc[j * 64 + lane]);     // 0 + v = v: no value is negative
            acc[j * 64 + lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
        do {
            ++k;
            next = L.part_start(k);
        } while (k < k0 + np && b >= next);
    };
    const RenderGrid& G = *P.G;
    const int t0x = P.t0x, t0y = P.t0y, t0z = P.t0z;
    const float* __restrict__ recbase = a.records + (size_t)G.grid_index * a.n_gauss * 16;
    const int* __restrict__ pg = a.pair_gauss;
    const float lane_fh = (float)lane + 0.5f;

    for (int j = lane; j < ACC_COLS; j += 64) acc[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);

    // Software pipeline over batches: while a batch's pieces are evaluated, the next batch's
    // records and the list entries of the batch after it are in flight (lane i of a batch
    // holds entry b0 + i).  Out-of-range lanes load nothing and keep zeros.
    // (the id's home bit is cleared only when the record is loaded, so that no wait for the
    // entry is placed right after its load)
    auto load_id = [&](int b) -> int {
        return (lane < RB && b + lane < e) ? pg[b + lane] : -1;
    };
    float4 n0 = make_float4(0, 0, 0, 0), n1 = n0, n2 = n0, n3 = n0;   // next batch's records
    auto load_rec = [&](int entry) {
        if (entry != -1) {
            const uint32_t gid = (uint32_t)entry & GM_ID_MASK;
            const float4* src = reinterpret_cast<const float4*>(recbase + (size_t)gid * 16);
            n0 = src[0];
            n1 = src[1];
            n2 = src[2];
            n3 = src[3];
        }
    };
    int id_rec = load_id(s);     // the entry whose record is in n0..n3
    load_rec(id_rec);
    int id_next = load_id(s + RB);
    MaskCtx mc;
    mc.pcc = pcc;
    mc.m = G.index_to_world;
    mc.res = a.bq.res;
    mc.radius = a.bq.radius;
    mc.t0z = t0z;
    mc.vc = vcell;
    mc.on = MASK && G.masked;

#pragma unroll 1
    for (int b0 = s; b0 < e; b0 += RB) {
        const int nb = min(RB, e - b0);
        const float4 r0 = n0, r1 = n1, r2 = n2, r3 = n3;
        const int my_entry = id_rec;
        load_rec(id_next);
        id_rec = id_next;
        id_next = load_id(b0 + 2 * RB);
        wave_sync();
        if (PARTS)
            if (b0 >= next && k < k0 + np) flush(b0);
        // this lane's piece: footprint area with its first and last columns in x and y (4 bits
        // each, from bit 9 on), and its place in the batch
        int myF = 0, pos = lane;
        if (lane < nb) {
            const int lox = __float_as_int(r2.z), loy = __float_as_int(r2.w);
            const int loz = __float_as_int(r3.x), hix = __float_as_int(r3.y);
            const int hiy = __float_as_int(r3.z), hiz = __float_as_int(r3.w);
            const int ix0 = max(lox, t0x), iy0 = max(loy, t0y);
            const int wx = min(hix, t0x + GM_TX - 1) - ix0 + 1;
            const int wy = min(hiy, t0y + GM_TY - 1) - iy0 + 1;
            // a listed box overlaps the tile
            const bool ok = wx > 0 && wy > 0;
            const int wxe = ok ? wx : 1;
            Piece p;
            p.uxh = (r0.x - (float)(ix0 - lox)) + 0.5f;
            p.uy = r0.y - (float)(iy0 - loy);
            p.kxx = r1.x; p.kyy = r1.y; p.kxy = r1.w;
            p.kxz = r2.x; p.kyz = r2.y;
            // far below any visible curvature; keeps the planes outside the box at zero
            p.kzz = fminf(r1.z, -KZZ_MIN);
            // amp >= 0 (0 for an empty box, never listed): log2 0 = -inf gives zeros
            p.lamp = log2f(r0.w);
            p.wxf = (float)wxe;
            p.inv_wx = __builtin_amdgcn_rcpf(p.wxf);
            p.basef = (float)((iy0 - t0y) * ACC_P + (ix0 - t0x)) - 0.5f;
            const int zl = loz - t0z, zh = hiz - t0z;    // the box's planes in the tile's frame
            const float d0 = (float)(-zl);
            p.dz0 = zl <= 0 && zh >= 0 ? d0 - r0.z : DZ_OUT;
            p.dz1 = zl <= 1 && zh >= 1 ? (d0 + 1.0f) - r0.z : DZ_OUT;
            p.dz2 = zl <= 2 && zh >= 2 ? (d0 + 2.0f) - r0.z : DZ_OUT;
            p.dz3 = zl <= 3 && zh >= 3 ? (d0 + 3.0f) - r0.z : DZ_OUT;
            myF = ok ? wx * wy : 0;
            const int x0 = ix0 - t0x, y0 = iy0 - t0y;
            pos = place_piece(myF);
            pc[pos] = p;
            if (ok) myF |= x0 << 9 | (x0 + wx - 1) << 13 | y0 << 17 | (y0 + wy - 1) << 21;
            if (MASK && mc.on) {
                PieceCell q;
                q.ix0 = ix0;
                q.iy0 = iy0;
                q.pad0 = q.pad1 = 0;
                q.cm = a.bq.cells[(uint32_t)my_entry & GM_ID_MASK];
                pcc[pos] = q;
            }
        }
        myF = __builtin_amdgcn_ds_permute(pos << 2, myF);      // lane j: piece j of the new order
        // pieces j and j + 1 share a pass when their footprints sum to <= 64.  Lane j holds
        // that pass as one word: (columns of both << 16) | footprint of piece j, the upper half
        // equal to the lower where piece j goes alone, and bit 15 where no column is in both
        const int nextF = __shfl_down(myF, 1, 64);
        const int fa = myF & 0x1ff, fb = nextF & 0x1ff;
        const bool pair = lane + 1 < nb && fa + fb <= 64;
        const bool apart = (myF >> 13 & 15) < (nextF >> 9 & 15) || (nextF >> 13 & 15) < (myF >> 9 & 15) ||
                           (myF >> 21 & 15) < (nextF >> 17 & 15) || (nextF >> 21 & 15) < (myF >> 17 & 15);
        const int pk = fa | (pair && apart ? 0x8000 : 0) | ((pair ? fa + fb : fa) << 16);
        wave_sync();
        int j = 0;
        int k = __builtin_amdgcn_readlane(pk, 0);
        Pass q = load_pass(pc, 0, k & 0x1ff, lane, lane_fh);
#pragma unroll 1
        for (;;) {
            const int Fa = k & 0x1ff, Ft = k >> 16;
            const int F1 = k & 0x8000 ? Ft : Fa;       // columns added at once
            const int jn = j + (Ft > Fa ? 2 : 1);
            const bool more = jn < nb;
            k = __builtin_amdgcn_readlane(pk, more ? jn : j);
            float4 w;
            int col;
            eval_column(q.p, q.fh, w, col);
            if (MASK && mc.on)
                mask_column(q.p, mc.pcc[lane < Fa || Ft == Fa ? j : j + 1], mc, q.fh, col, w);
            // every lane evaluates (a lane past its piece's footprint computes values it
            // never stores), so no lane mask is needed around the evaluation
            lds_order();
            if (lane < F1) add_column(acc, col, w);
            lds_order();
            if (F1 < Ft) {
                if (lane >= Fa && lane < Ft) add_column(acc, col, w);
                lds_order();
            }
#pragma unroll 1
            for (int f = 64; f < Fa; f += 64) {
                eval_column(q.p, q.fh + (float)f, w, col);
                if (MASK && mc.on) mask_column(q.p, mc.pcc[j], mc, q.fh + (float)f, col, w);
                lds_order();
                if (lane + f < Fa) add_column(acc, col, w);
                lds_order();
            }
            if (!more) break;
            j = jn;
            q = load_pass(pc, j, k & 0x1ff, lane, lane_fh);
        }
    }
    wave_sync();
    if (PARTS && k > k0 + 1) {
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j * 64 + lane] = add4(tot[j], acc[j * 64 + lane]);
        wave_sync();
    }
}

// Every kernel sums a tile's parts in the same association, whichever wavefronts took them: with
// up to 8 parts one after the other, with 16 in consecutive pairs first.
constexpr int GROUPS = 8;

// Column col of the tile from the NP parts' copies of it
template <int NP>
__device__ __forceinline__ float4 sum_parts(const float4* accs, int col)
{
    constexpr int M = NP > GROUPS ? NP / GROUPS : 1;
    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int g = 0; g < NP / M; ++g) {
        float4 u = accs[g * M * ACC_COLS + col];
#pragma unroll
        for (int i = 1; i < M; ++i) u = add4(u, accs[(g * M + i) * ACC_COLS + col]);
        v = g == 0 ? u : add4(v, u);
    }
    return v;
}

// Writes the finished tile (plain mode), or (loss mode) the smooth-L1 data term on it (Eq. 11,
// beta = 1): dL/dI = clamp(I - y, -1, 1) / N, the rendering when G.out is set, and the tile's
// FP64 sum of smoothL1(I - y) to a.loss_part[part].  The tile is the sum of its NP parts' copies
// accs, finished by T threads (thread t: columns t, t + T, ...); red: LDS, one double per
// wavefront of them (unused for one wavefront).
template <int NP, int T>
__device__ __forceinline__ void finish_tile(const RenderArgs& a, const TilePos& P,
                                            const float4* accs,
                                            const float (&tv)[cols_per_thread<T>()][GM_TZ], int t,
                                            int part, double* red)
{
    const RenderGrid& G = *P.G;
    float* out = G.out;
    const float g_scale = (float)a.inv_n;
    double lsum = 0.0;
#pragma unroll
    for (int j = 0; j < cols_per_thread<T>(); ++j) {
        const int c = j * T + t;
        const int x = c % GM_TX, y = c / GM_TX;
        const int gx = P.t0x + x, gy = P.t0y + y;
        if (c >= GM_TX * GM_TY || gx >= G.nx || gy >= G.ny) continue;
        const float4 v = sum_parts<NP>(accs, y * ACC_P + x);
        const float val[GM_TZ] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int z = 0; z < GM_TZ; ++z) {
            const int gz = P.t0z + z;
            if (gz >= G.nz) continue;
            const size_t o = ((size_t)gz * G.ny + gy) * G.nx + gx;
            if (out) out[o] = val[z];
            if (!a.loss_part) continue;
            const float d = val[z] - tv[j][z];
            const float ad = fabsf(d);
            lsum += ad < 1.0f ? 0.5 * (double)d * (double)d : (double)ad - 0.5;
            G.dl[o] = fminf(fmaxf(d, -1.0f), 1.0f) * g_scale;
        }
    }
    if (!a.loss_part) return;
    for (int o = 32; o > 0; o >>= 1) lsum += __shfl_xor(lsum, o, 64);
    if (T == 64) {
        if ((t & 63) == 0) a.loss_part[part] = lsum;
        return;
    }
    if ((t & 63) == 0) red[t >> 6] = lsum;
    __syncthreads();
    if (t == 0) {
        double v = red[0];
#pragma unroll
        for (int w = 1; w < T / 64; ++w) v += red[w];
        a.loss_part[part] = v;
    }
}

template <int NW>
__global__ __launch_bounds__(64 * NW) void k_render(const RenderArgs a)
{
    __shared__ TileLds<NW> sh;
    __shared__ double red[NW];
    const int lane = threadIdx.x & 63, w = sgpr(threadIdx.x >> 6);
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const TilePos P = tile_pos(a, blk);
    float tv[cols_per_thread<64 * NW>()][GM_TZ];
    if (a.loss_part) load_targets<64 * NW>(P, threadIdx.x, tv);
    accumulate_tile<false, false>(a, P, sh.accs + w * ACC_COLS, sh.pcs[w], lane, w, 1, nullptr,
                                  nullptr);
    __syncthreads();
    finish_tile<NW, 64 * NW>(a, P, sh.accs, tv, threadIdx.x, a.part0 + blk, red);
}

// k_render with one wavefront for all of a tile's parts (up to 8), the same sums: for lists too short
// to share (one_wavefront), where what counts is how many tiles are in flight (six wavefronts per SIMD;
// with the targets of the loss held over the walk four, and 320^3 with lists of 83 took 185 us, not 160)
__global__ __launch_bounds__(64, 6) void k_render_one(const RenderArgs a)
{
    __shared__ TileLds<1> sh;
    const int lane = threadIdx.x;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const TilePos P = tile_pos(a, blk);
    accumulate_tile<false, true>(a, P, sh.accs, sh.pcs[0], lane, 0, 1 << a.parts_log2, nullptr, nullptr);
    float tv[cols_per_thread<64>()][GM_TZ];
    if (a.loss_part) load_targets<64>(P, lane, tv);
    finish_tile<1, 64>(a, P, sh.accs, tv, lane, a.part0 + blk, nullptr);
}

// k_render for launches that hold a masked grid (the block query on a rotated grid)
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_render_block(const RenderArgs a)
{
    __shared__ TileLds<NW> sh;
    __shared__ PieceCell pccs[NW][RB];
    __shared__ int vcell[3 * GM_TILE_VOX];
    __shared__ double red[NW];
    const int lane = threadIdx.x & 63, w = sgpr(threadIdx.x >> 6);
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const TilePos P = tile_pos(a, blk);
    float tv[cols_per_thread<64 * NW>()][GM_TZ];
    if (a.loss_part) load_targets<64 * NW>(P, threadIdx.x, tv);
    if (P.G->masked) {
        // the cells of the tile's voxels, clamped to [-2^30, 2^30] as the means' cells are
#pragma unroll 1
        for (int i = threadIdx.x; i < GM_TILE_VOX; i += 64 * NW) {
            double c[3];
            voxel_cells(P.G->index_to_world, a.bq.res, P.t0x + i % GM_TX,
                        P.t0y + (i / GM_TX) % GM_TY, P.t0z + i / (GM_TX * GM_TY), c);
#pragma unroll
            for (int u = 0; u < 3; ++u)
                vcell[u * GM_TILE_VOX + i] = (int)fmin(fmax(c[u], -1073741824.0), 1073741824.0);
        }
        __syncthreads();
    }
    accumulate_tile<true, false>(a, P, sh.accs + w * ACC_COLS, sh.pcs[w], lane, w, 1, pccs[w],
                                 vcell);
    __syncthreads();
    finish_tile<NW, 64 * NW>(a, P, sh.accs, tv, threadIdx.x, a.part0 + blk, red);
}

// Render + residual field (Sec. 3.4, Eq. 8: I_final = I + r) in one pass.  Blocks of FW
// wavefronts share the field's weights, staged once in LDS, and stay resident; the tiles of the
// launch are split into eight contiguous ranges, one per XCD, dealt to that XCD's blocks.  A
// tile is taken by one wavefront (TW = 1) or, on small grids whose tiles would leave wavefronts
// idle, by the whole block (TW = FW).  The tile's parts are rendered exactly as k_render does,
// then the field is evaluated on the tile's voxels in 64 groups of 16 (one x row each) and
// out_scale tanh(z_out) added to each voxel before the store or loss epilogue.  Each point's
// field value is the same arithmetic as the field's own forward kernel, so the result is bit
// for bit the render followed by gm_nrf_forward (and the loss the same terms).
constexpr int FW = 8;
static_assert(FW == GROUPS, "a block's wavefronts take one group of parts each");

// Two blocks fit a CU's LDS up to four layers of 64 inputs or three of 128: four wavefronts per
// SIMD, at most 128 registers each.
template <int KT, int DEPTH>
constexpr int field_waves(bool masked)
{
    const bool two = 2 * (sizeof(nrfcore::Lds<KT, DEPTH>) + sizeof(TileLds<FW>)) <= 160 * 1024;
    return two && !masked ? 4 : 2;
}

template <int KT, int DEPTH, bool MASK, int TW>
__global__ __launch_bounds__(64 * FW, (field_waves<KT, DEPTH>(MASK))) void k_render_field(const RenderArgs a, const NrfArgs f)
{
    __shared__ nrfcore::Lds<KT, DEPTH> sw;
    __shared__ TileLds<FW> sh;
    __shared__ PieceCell pccs[MASK ? FW : 1][RB];
    nrfcore::load_weights<KT, DEPTH>(f, sw);
    const int lane = threadIdx.x & 63, w = sgpr(threadIdx.x >> 6), g = lane >> 4, row = lane & 15;
    nrfcore::v4s wo[4];
    nrfcore::load_wout(f, wo);
    float4* own = sh.accs + w * ACC_COLS;           // this wavefront's copy
    float4* acc = TW == 1 ? own : sh.accs;          // the tile
    const int xcd = blockIdx.x & 7;
    const int nbx = (int)(gridDim.x >> 3);     // the launch has a multiple of 8 blocks
    const int T = a.total_blocks;
    const int lo = (int)((int64_t)T * xcd / 8), hi = (int)((int64_t)T * (xcd + 1) / 8);
    constexpr int TPB = FW / TW;               // tiles a block holds at a time
    const int np = (1 << a.parts_log2) / TW;            // parts per wavefront
    const int k0 = TW == 1 ? 0 : w * np;
#pragma unroll 1
    for (int t = lo + (int)(blockIdx.x >> 3) * TPB + w / TW; t < hi; t += nbx * TPB) {
        const TilePos P = tile_pos(a, t);
        const RenderGrid& G = *P.G;
        accumulate_tile<MASK, true>(a, P, own, sh.pcs[w], lane, k0, np, pccs[MASK ? w : 0], nullptr);
        if constexpr (TW > 1) {
            __syncthreads();
            for (int c = threadIdx.x; c < ACC_COLS; c += 64 * FW) {
                float4 v = sh.accs[c];
#pragma unroll
                for (int u = 1; u < FW; ++u) v = add4(v, sh.accs[u * ACC_COLS + c]);
                sh.accs[c] = v;
            }
            __syncthreads();
        }
        // the biases go where the wavefront's pieces were (read from global memory, under this
        // kernel's register pressure, each was waited for in the middle of a layer)
        nrfcore::v4f* bias = reinterpret_cast<nrfcore::v4f*>(sh.pcs[w]);
        static_assert(sizeof sh.pcs[0] >= 16 * DEPTH * sizeof(nrfcore::v4f), "room for the biases");
        wave_sync();
        nrfcore::load_biases<DEPTH>(f, bias, lane);
        wave_sync();
        const nrfcore::WeightsLds<KT, DEPTH> ws{sw, bias, lane};
        // Four rows at a time: lane group j keeps row j's output, so that one tanh (some 50
        // instructions, and all four groups used to form the same 16) serves all four.  With this
        // and the encoding's bands past n_freq left out, a 256^3 volume with the field went from
        // 1720 to 1671 us, three 256x256x64 stacks from 1497 to 1461.  What is left is vector
        // issue (76% busy): 7 issue slots per SiLU, 48 of them a row and lane.
#pragma unroll 1
        for (int q0 = w % TW; q0 < GM_TILE_VOX / 16; q0 += 4 * TW) {
            float zo = 0.0f;
#pragma unroll 1
            for (int j = 0; j < 4; ++j) {
                const int q = q0 + j * TW;
                const int vy = P.t0y + (q % GM_TY), vz = P.t0z + q / GM_TY, vx = P.t0x + row;
                if (vy >= G.ny || vz >= G.nz) continue;     // uniform over the wavefront
                const float x[3] = {nrfcore::world_coord(G.index_to_world, vx, vy, vz),
                                    nrfcore::world_coord(G.index_to_world + 4, vx, vy, vz),
                                    nrfcore::world_coord(G.index_to_world + 8, vx, vy, vz)};
                nrfcore::Tile<KT, DEPTH> Tl;
                nrfcore::tile_forward_w<KT, DEPTH>(f, ws, x, Tl);
                const float z = nrfcore::tile_output<KT, DEPTH>(f, Tl, wo);
                zo = g == j ? z : zo;
            }
            // (rows past the grid stay at tanh 0)
            const int q = q0 + g * TW;
            if (P.t0x + row < G.nx)
                reinterpret_cast<float*>(acc + (q % GM_TY) * ACC_P + row)[q / GM_TY] +=
                    f.out_scale * tanhf(zo);
        }
        if constexpr (TW == 1) {
            wave_sync();
            float tv[cols_per_thread<64>()][GM_TZ];
            if (a.loss_part) load_targets<64>(P, lane, tv);
            finish_tile<1, 64>(a, P, acc, tv, lane, a.part0 + t, nullptr);
            wave_sync();
        } else {
            // the loss sums go where the pieces were: no wavefront prepares pieces before the
            // next barrier
            __syncthreads();
            float tv[cols_per_thread<64 * FW>()][GM_TZ];
            if (a.loss_part) load_targets<64 * FW>(P, threadIdx.x, tv);
            finish_tile<1, 64 * FW>(a, P, acc, tv, threadIdx.x, a.part0 + t,
                                    reinterpret_cast<double*>(sh.pcs));
            __syncthreads();
        }
    }
}

// loss = inv_n * sum of the per-block sums, in a fixed order.  Each thread takes four
// partials per round (all four loads in flight), then a tree over the block.
constexpr int FIN_THREADS = 1024;

__global__ __launch_bounds__(FIN_THREADS) void k_render_loss_finish(const double* part, int nb,
                                                                    double inv_n, float* loss)
{
    __shared__ double sh[FIN_THREADS];
    const int t = threadIdx.x;
    double v = 0.0;
    for (int i = t; i < nb; i += 4 * FIN_THREADS) {
        double q[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int k = i + u * FIN_THREADS;
            q[u] = k < nb ? part[k] : 0.0;
        }
        v += (q[0] + q[1]) + (q[2] + q[3]);
    }
    sh[t] = v;
    __syncthreads();
    for (int o = FIN_THREADS / 2; o > 0; o >>= 1) {
        if (t < o) sh[t] += sh[t + o];
        __syncthreads();
    }
    if (t == 0) *loss = (float)(sh[0] * inv_n);
}

// Parts a tile's list is cut into, by the tiles of its grid (a property of the grid alone, so
// that every kernel and every listing of grids sums a tile the same way).  A small grid has too
// few tiles to fill the chip with a wavefront each.  Measured training iterations (us) at 2 / 4 /
// 8 / 16 wavefronts per tile: 64 tiles per grid 166 / 126 / 109 / 100; 216: 220 / 176 / 164 /
// 175; 512: 417 / 380 / 367 / 400; 1728: 553 / 524 / 527 / 674; 4096: 1150 / 1116 / 1142 / 1498;
// rendering one grid of 32000 tiles 675 / 686 / 773 / 1423.  (One wavefront per tile was slower by
// 3 to 40% than two at each.)
int parts_of(const RenderGrid& g)
{
    const int64_t tiles = (int64_t)g.ntx * g.nty * g.ntz;
    return tiles <= 128 ? 16 : tiles <= 1024 ? 8 : tiles <= 16384 ? 4 : 2;
}

// The grids of a that take np parts, as a launch of their own (no blocks: none)
RenderArgs with_parts(const RenderArgs& a, int np)
{
    RenderArgs r = a;
    r.parts_log2 = __builtin_ctz((unsigned)np);
    r.n_render = 0;
    r.total_blocks = 0;
    for (int k = 0; k < a.n_render; ++k) {
        if (parts_of(a.rg[k]) != np) continue;
        RenderGrid& g = r.rg[r.n_render++];
        g = a.rg[k];
        g.first_block = r.total_blocks;
        r.total_blocks += g.ntx * g.nty * g.ntz;
    }
    return r;
}

bool any_masked(const RenderArgs& a)
{
    bool masked = false;
    for (int k = 0; k < a.n_render; ++k) masked = masked || a.rg[k].masked;
    return masked;
}

// Whether the tiles of a launch are better taken by a wavefront each than by one per part: where the
// parts' wavefronts are more than the chip holds at a time (26 a CU) and the lists are short on average
// (a list of one batch is one part's whatever their number; the others' wavefronts only keep tiles
// waiting).  us with the parts' wavefronts and with one, by list length, 1- and 8-voxel Gaussians alike:
//     128^3 (2048 tiles, 4 parts)     15: 14, 11     32: 31, 27     79: 21, 27     159: 33, 45
//     three 128x128x32 (1536, 8)      12: 28, 19     48: 55, 50     68: 60, 68     199: 29, 53
//     200^3 (8450, 4)                 77: 56, 54     83: 107, 114   145: 89, 93    155: 92, 97
//     three 256x256x64 (12288, 4)     17: 109, 57    152: 214, 195  209: 165, 168  249: 196, 202
//     256^3 (16384, 4)                16: 64, 33     83: 103, 94    166: 176, 169  416: 374, 400
//     320^3 (32000, 2)                18: 122, 91    83: 167, 160   167: 295, 297
// The line through where the two meet: lists of 38 where the parts just fill the chip, 25 more for
// every time they fill it again, up to 200.
bool one_wavefront(const RenderArgs& a, int np)
{
    const double fill = (double)a.total_blocks * np / (26 * 256);
    return np <= GROUPS && fill > 1.0 && a.mean_list < fmin(200.0, 38.0 + 25.0 * (fill - 1.0));
}

template <int NW>
void launch_render_t(const RenderArgs& a, hipStream_t s)
{
    const dim3 grid((unsigned)a.total_blocks), block(64 * NW);
    if (any_masked(a))
        hipLaunchKernelGGL(k_render_block<NW>, grid, block, 0, s, a);
    else if (one_wavefront(a, NW))
        hipLaunchKernelGGL(k_render_one, grid, dim3(64), 0, s, a);
    else
        hipLaunchKernelGGL(k_render<NW>, grid, block, 0, s, a);
}

template <int KT, int DEPTH, bool MASK, int TW>
void launch_field_mt(const RenderArgs& a, const NrfArgs& f, hipStream_t s)
{
    // every block resident at once, a multiple of 8 (one share per XCD), capped by the tiles
    int dev = 0, cus = 0, per_cu = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(
        &per_cu, k_render_field<KT, DEPTH, MASK, TW>, 64 * FW, 0);
    int64_t full = (int64_t)(cus > 0 ? cus : 256) * (per_cu > 0 ? per_cu : 1);
    int64_t need = ((int64_t)a.total_blocks * TW + FW - 1) / FW;
    int64_t nb = need < full ? need : full;
    nb = (nb + 7) / 8 * 8;
    hipLaunchKernelGGL((k_render_field<KT, DEPTH, MASK, TW>), dim3((unsigned)nb), dim3(64 * FW), 0,
                       s, a, f);
}

template <int KT, int DEPTH>
void launch_field_t(const RenderArgs& a, const NrfArgs& f, hipStream_t s)
{
    if (any_masked(a)) {
        if ((1 << a.parts_log2) >= FW)
            launch_field_mt<KT, DEPTH, true, FW>(a, f, s);
        else
            launch_field_mt<KT, DEPTH, true, 1>(a, f, s);
    } else {
        if ((1 << a.parts_log2) >= FW)
            launch_field_mt<KT, DEPTH, false, FW>(a, f, s);
        else
            launch_field_mt<KT, DEPTH, false, 1>(a, f, s);
    }
}

hipError_t launch_field(const RenderArgs& a, const NrfArgs& f, hipStream_t s)
{
    switch ((f.in_pad >> 4) * 8 + f.depth) {
    case 4 * 8 + 1: launch_field_t<4, 1>(a, f, s); break;
    case 4 * 8 + 2: launch_field_t<4, 2>(a, f, s); break;
    case 4 * 8 + 3: launch_field_t<4, 3>(a, f, s); break;
    case 4 * 8 + 4: launch_field_t<4, 4>(a, f, s); break;
    case 8 * 8 + 1: launch_field_t<8, 1>(a, f, s); break;
    case 8 * 8 + 2: launch_field_t<8, 2>(a, f, s); break;
    case 8 * 8 + 3: launch_field_t<8, 3>(a, f, s); break;
    case 8 * 8 + 4: launch_field_t<8, 4>(a, f, s); break;
    default: return hipErrorInvalidValue;
    }
    return hipSuccess;
}

// f: with the residual field (NULL: without)
hipError_t launch_all(const RenderArgs& a, const NrfArgs* f, hipStream_t s)
{
    if (a.total_blocks == 0) return hipSuccess;
    int32_t part0 = 0;
    for (int np = 2; np <= 16; np *= 2) {
        RenderArgs r = with_parts(a, np);
        if (r.total_blocks == 0) continue;
        r.part0 = part0;
        part0 += r.total_blocks;
        if (f) {
            const hipError_t e = launch_field(r, *f, s);
            if (e != hipSuccess) return e;
        } else if (np == 2) {
            launch_render_t<2>(r, s);
        } else if (np == 4) {
            launch_render_t<4>(r, s);
        } else if (np == 8) {
            launch_render_t<8>(r, s);
        } else {
            launch_render_t<16>(r, s);
        }
    }
    if (a.loss_part)
        hipLaunchKernelGGL(k_render_loss_finish, dim3(1), dim3(FIN_THREADS), 0, s, a.loss_part,
                           a.total_blocks, a.inv_n, a.loss);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_render(const RenderArgs& a, hipStream_t s) { return launch_all(a, nullptr, s); }

hipError_t launch_render_field(const RenderArgs& a, const NrfArgs& f, hipStream_t s)
{
    return launch_all(a, &f, s);
}
