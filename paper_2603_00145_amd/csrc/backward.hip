// K7 + K8: gradients of L = sum_k sum_v dL/dI_k[v] I_k[v] (+ lambda_aniso * L_aniso,
// Eq. 12-13) with respect to every Gaussian parameter, boxes held fixed.
//
// K7 (grid-frame partials): a group of lanes per Gaussian gathers g = dL/dI over the voxels of
// the Gaussian's box on each listed grid, recomputing E = 2^Q (no per-voxel contributions are
// stored).  With delta = v - c, Q = delta^T K delta (K the record's base-2 conic as a
// symmetric matrix) and w = amp E, the ten grid-frame partials are
//     d amp = sum g E,   d c = -2 amp ln2 K m,   d K_ab = amp ln2 m_ab
// with the weighted moments m = sum g E delta and m_ab = sum g E delta_a delta_b.  A lane
// walks columns of the box along y, summing g E, g E dy and g E dy^2; the column's share of the
// ten moments follows from those three sums and its (dx, dz).  The moments are reduced across
// the group with DPP and turned into the partials once per (grid, Gaussian).  No global atomics
// are needed.  With the paper's block query on a rotated grid (k_partials<true>) every Gaussian of
// that grid takes the global-memory path and each voxel of its box is also tested against its
// cell block (Eqs. 4-6): the sums run over the voxels that pass.
//
// K8 (chain rule, FP64): thread per Gaussian.  The partials of every grid are pulled back
// through c = L mu + t, C = Sigma_g^-1, amp = alpha sqrt(det Sigma_idx / det Sigma_g),
// Sigma_idx = L Sigma L^T, Sigma = R diag(e^{2s}) R^T (Eq. 3), R(q/|q|) and
// alpha = sigmoid(logit), summed over grids, and added (+=) to the gradient buffers.
#include "gm_internal.h"
#include <type_traits>

namespace {

__device__ __forceinline__ int sgpr(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Sum of v over each aligned group of G lanes (every lane of the group ends with it): DPP adds
// across lane xor 1, xor 2, the half-row mirror and the row mirror, then the wavefront's rows.
template <int G>
__device__ __forceinline__ float group_sum(float v)
{
    static_assert(G == 4 || G == 8 || G == 64, "groups of 4, 8 or 64 lanes");
    int xi;
    xi = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xF, 0xF, false);  // xor 1
    v += __int_as_float(xi);
    xi = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xF, 0xF, false);  // xor 2
    v += __int_as_float(xi);
    if (G > 4) {
        xi = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x141, 0xF, 0xF, false); // half mirror
        v += __int_as_float(xi);
    }
    if (G == 64) {
        xi = __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x140, 0xF, 0xF, false); // mirror
        v += __int_as_float(xi);
        const int b = __float_as_int(v);
        v = (__int_as_float(__builtin_amdgcn_readlane(b, 0)) +
             __int_as_float(__builtin_amdgcn_readlane(b, 16))) +
            (__int_as_float(__builtin_amdgcn_readlane(b, 32)) +
             __int_as_float(__builtin_amdgcn_readlane(b, 48)));
    }
    return v;
}

// Largest / smallest value of v over the lanes 0, G, 2G, ... (one per group).
template <int G>
__device__ __forceinline__ int group_max(int v)
{
    int m = __builtin_amdgcn_readlane(v, 0);
#pragma unroll
    for (int r = 1; r < 64 / G; ++r) m = max(m, __builtin_amdgcn_readlane(v, r * G));
    return m;
}
template <int G>
__device__ __forceinline__ int group_min(int v)
{
    int m = __builtin_amdgcn_readlane(v, 0);
#pragma unroll
    for (int r = 1; r < 64 / G; ++r) m = min(m, __builtin_amdgcn_readlane(v, r * G));
    return m;
}

// dL/dI region a block stages in LDS: its tile plus a halo of 8 voxels on the upper side in x
// and y and 6 in z (a home Gaussian's box starts inside the tile; thick-slice boxes are short
// in z).  The z planes are RZS floats apart, RZS = 8 (mod 32), so the up-to-four z rows a lane
// row reads at one step sit in different LDS banks.
constexpr int RX = GM_TX + 8, RY = GM_TY + 8, RZ = GM_TZ + 6;
constexpr int RZS = RX * RY + 8;
// lanes per Gaussian in the rounds from LDS: setting a Gaussian up and reducing its moments costs
// about as much as walking its box, and is shared by as many Gaussians as a wavefront holds; with
// 2 lanes the rounds are too few and too uneven (256^3 workload: 399 us with 8 lanes, 378 with 4,
// 416 with 2)
constexpr int BWD_G = 4;
constexpr int PER_ROUND = 64 / BWD_G;
constexpr int WINB = 1024; // list entries a block sorts at a time
constexpr int EPT = WINB / 256;  // ... per thread
// longest column of lds_column: it reads that many rows whatever the box's length, so at most
// NK_MAX - 8 rows past the last plane's end (masked where they are used)
constexpr int NK_MAX = 12;
// and a box of fewer than 3 rows is walked from SHIFT rows above it (masked too), which lie PAD floats
// before the region at most
constexpr int SHIFT = 2, PAD = SHIFT * RX;
constexpr int REGION = PAD + RZ * RZS + (NK_MAX - 8) * RX;
// sort keys of home entries: boxes inside the staged region by (lane passes in x, z planes, y
// length), each capped; then one key for boxes reaching past the region
constexpr int KEY_X = 4, KEY_Z = 5, KEY_Y = 12;
constexpr int NKEY = KEY_X * KEY_Z * KEY_Y + 1;
constexpr uint32_t KEY_FEW = 1u << (KEY_X + KEY_Z + KEY_Y);   // a round's bit for short boxes
static_assert(RZS % 32 == 8, "z-plane stride must be 8 mod 32 banks");

// The row of a box that an LDS column's walk counts from.  Q_k and the moments are formed around
// it, so the closer it lies to the Gaussian's centre, the less cancels (a 3-sigma box of a 1-voxel
// Gaussian has 7 rows).  Counted from row 0 (1.7% fewer instructions, 353 against 355 us) the
// quaternions' gradients of 1M Gaussians on three 256x256x64 stacks were 3 times as far from
// binary64 (99 of 100 within 2.3e-7 of the largest; now 7.4e-8).  Row 3 gave 5.7e-8, but a larger
// error in boxes of few rows (the worst centre gradient 1.1e-6 against 3.9e-7).
// Boxes of one or two rows are walked from SHIFT = YC rows above them and so count from their first:
// their own row 2 lies outside them, where the exponent of a Gaussian a fraction of a voxel wide is
// large and cancels in the rows inside (at a width of 0.1 voxel sums were off by 1.8e-5 and second
// moments wholly lost; counted from their first row 4e-7).  From three rows on row 2 is no further
// from any row than row 0 is.
constexpr int YC = 2;
static_assert(SHIFT == YC, "a short box's first row is the one its walk counts from");

// Column sums s0 = sum ge, s1 = sum k ge, s2 = sum k^2 ge (ge = g 2^Q_k, k = row - YC) over the
// first NK rows of a column whose rows are RX floats apart in the staged region, all NK reads
// issued at immediate offsets before the first use; rows past the column (row >= ncol) are masked
// where they are used, and so are the first SHIFT of a short box's.  NK is the wavefront's longest
// column (up to NK_MAX), a compile-time constant, so the steps carry no branches.  (No contraction: a Gaussian's sums must not depend on
// the NK its wavefront takes.)
template <int NK, bool MASK>
__device__ __forceinline__ void lds_column(const float* __restrict__ region, uint32_t off,
                                           bool few, int ncol, float A, float B, float kyy,
                                           float& s0, float& s1, float& s2)
{
#pragma clang fp contract(off)
    float gv[NK];
#pragma unroll
    for (int r = 0; r < NK; ++r) gv[r] = region[off + r * RX];
#pragma unroll
    for (int r = 0; r < NK; ++r) {
        const int k = r - YC;
        const float Q = k == 0 ? A : fmaf((float)k, fmaf((float)k, kyy, B), A);
        // without MASK every active column of the wavefront is at least NK long and none is short
        const bool in = (r == 0 || r < ncol) && (r >= SHIFT || !few);
        const float gr = !MASK || in ? gv[r] : 0.0f;
        const float ge = gr * __builtin_amdgcn_exp2f(Q);
        if (r == 0) {
            s0 = ge;
            s1 = (float)k * ge;
            s2 = (float)(k * k) * ge;
            continue;
        }
        s0 += ge;
        if (k == 1 || k == -1) {
            s1 = k > 0 ? s1 + ge : s1 - ge;
            s2 += ge;
        } else if (k != 0) {
            s1 = fmaf((float)k, ge, s1);
            s2 = fmaf((float)(k * k), ge, s2);
        }
    }
}

// Sums over the planes of a lane's (y, z) sheet: sum gE, k (the row less YC) and dz moments.
struct Sheet {
    float s, k, kk, z, zz, kz;
};

// A lane's sheet of its Gaussian's box: planes 0 .. wz - 1 (none for an inactive lane), whose
// walk starts at region[off].  max_wz, max_wy: the wavefront's.  Q along a plane's column is
// A + k (B + k kyy) with A = Ab + dz (hz + kzz dz) and B = Bx + kyz dz.
template <int NK, bool MASK>
__device__ __forceinline__ void lds_sheet(const float* __restrict__ region, uint32_t off, int wz,
                                          int max_wz, bool few, int ncol, int max_wy, float cz,
                                          float Ab, float hz, float kzz, float Bx, float kyz,
                                          float kyy, Sheet& S)
{
#pragma clang fp contract(off)
    float zf = 0.0f;
#pragma unroll 1
    for (int z = 0; z < max_wz; ++z, zf += 1.0f, off += RZS) {
        const float dz = zf - cz;
        // a lane past its planes reads the region's first column and gets A = -inf, so its
        // every term is exactly zero
        const bool in = z < wz;
        const uint32_t o = in ? off : (uint32_t)PAD;
        const float A = in ? fmaf(dz, fmaf(kzz, dz, hz), Ab) : -__builtin_inff();
        const float B = fmaf(kyz, dz, Bx);
        float s0, s1, s2;
        lds_column<NK, MASK>(region, o, few, ncol, A, B, kyy, s0, s1, s2);
        if (NK == NK_MAX) {
#pragma unroll 1
            for (int r = NK_MAX; r < max_wy; ++r) {
                const float t = region[o + min(r, ncol - 1) * RX];
                const float gr = r < ncol ? t : 0.0f;
                const float fk = (float)(r - YC);
                const float ge = gr * __builtin_amdgcn_exp2f(fmaf(fk, fmaf(fk, kyy, B), A));
                s0 += ge;
                s1 = fmaf(fk, ge, s1);
                s2 = fmaf(fk * fk, ge, s2);
            }
        }
        const float az = s0 * dz;
        S.s += s0;
        S.k += s1;
        S.kk += s2;
        S.z += az;
        S.zz = fmaf(az, dz, S.zz);
        S.kz = fmaf(s1, dz, S.kz);
    }
}

// A Gaussian's 64-byte render record on one grid, as the group loads it (zeros when invalid).
struct Rec {
    float4 r0, r1, r2, r3;
};

// (an invalid lane group passes mine = 0 and gets Gaussian 0's record: finite values whose
// box is never walked)
__device__ __forceinline__ Rec load_record(const BackwardArgs& a, int gi, uint32_t mine)
{
    const int64_t gid = min((int64_t)(mine & GM_ID_MASK), a.n - 1);
    const float4* rp = reinterpret_cast<const float4*>(a.records + ((size_t)gi * a.n + gid) * 16);
    Rec r;
    r.r0 = rp[0];
    r.r1 = rp[1];
    r.r2 = rp[2];
    r.r3 = rp[3];
    return r;
}

// Lane sums of the weighted moments m = sum gE, m_a = sum gE delta_a, m_ab = sum gE delta_a
// delta_b over a lane's share of a box
struct Moments {
    float m, x, y, z, xx, yy, zz, xy, xz, yz;
};

// The moments added over each group of G lanes, turned into the ten grid-frame partials and
// stored by the group's first lane.
template <int G>
__device__ __forceinline__ void store_partials(const BackwardArgs& a, int gi, uint32_t mine,
                                               bool gvalid, const Rec& rec, Moments v)
{
    v.m = group_sum<G>(v.m);
    v.x = group_sum<G>(v.x);
    v.y = group_sum<G>(v.y);
    v.z = group_sum<G>(v.z);
    v.xx = group_sum<G>(v.xx);
    v.yy = group_sum<G>(v.yy);
    v.zz = group_sum<G>(v.zz);
    v.xy = group_sum<G>(v.xy);
    v.xz = group_sum<G>(v.xz);
    v.yz = group_sum<G>(v.yz);
    if ((threadIdx.x & (G - 1)) == 0 && gvalid) {
        const int64_t gid = min((int64_t)(mine & GM_ID_MASK), a.n - 1);
        // K as a full symmetric matrix has off-diagonal entries kxy/2, kxz/2, kyz/2
        const float Al = rec.r0.w * GM_LN2F;   // amp ln2
        const float hxy = 0.5f * rec.r1.w, hxz = 0.5f * rec.r2.x, hyz = 0.5f * rec.r2.y;
        const float tx = rec.r1.x * v.x + hxy * v.y + hxz * v.z;
        const float ty = hxy * v.x + rec.r1.y * v.y + hyz * v.z;
        const float tz = hxz * v.x + hyz * v.y + rec.r1.z * v.z;
        float2* o = reinterpret_cast<float2*>(a.grid_grads + ((size_t)gi * a.n + gid) * 10);
        o[0] = make_float2(v.m, -2.0f * Al * tx);
        o[1] = make_float2(-2.0f * Al * ty, -2.0f * Al * tz);
        o[2] = make_float2(Al * v.xx, Al * v.yy);
        o[3] = make_float2(Al * v.zz, Al * v.xy);
        o[4] = make_float2(Al * v.xz, Al * v.yz);
    }
}

// A round of Gaussians whose boxes lie inside the staged region, one per group of BWD_G lanes.
// A lane takes every BWD_G-th x of its box and walks the (y, z) sheet there, plane by plane, so
// everything that depends on x alone is formed once, a plane costs three FMAs to set up, and
// the x moments follow from the sheet's sums at the end.  rb: the round's keys, from bit 0 a bit
// per number of rows walked, then per plane count, then per number of x passes, then one for short
// boxes.
__device__ __forceinline__ void lds_round(const BackwardArgs& a, int gi, uint32_t mine, bool gvalid,
                                          const Rec& rec, const float* __restrict__ region,
                                          int t0x, int t0y, int t0z, uint32_t rb)
{
    const int ql = threadIdx.x & (BWD_G - 1);
    const float4 r0 = rec.r0, r1 = rec.r1, r2 = rec.r2, r3 = rec.r3;
    const int lox = __float_as_int(r2.z), loy = __float_as_int(r2.w), loz = __float_as_int(r3.x);
    const int wx = gvalid ? __float_as_int(r3.y) - lox + 1 : 0;
    int wy = __float_as_int(r3.z) - loy + 1;
    const int wz = __float_as_int(r3.w) - loz + 1;
    const bool few = wy <= SHIFT;
    const int shift = few ? SHIFT : 0;
    wy += shift;                                  // rows walked
    const float cx = r0.x, cz = r0.z;
    const float kxx = r1.x, kyy = r1.y, kzz = r1.z, kxy = r1.w;
    const float kxz = r2.x, kyz = r2.y;
    const int ncol = gvalid ? wy : 64;
    int max_wy = 32 - __clz(rb & ((1 << KEY_Y) - 1));
    const int min_wy = __ffs(rb & ((1 << KEY_Y) - 1));
    int max_wz = 32 - __clz((rb >> KEY_Y) & ((1 << KEY_Z) - 1));
    int max_wx = (32 - __clz((rb & ~KEY_FEW) >> (KEY_Y + KEY_Z))) * BWD_G;
    if (max_wy == KEY_Y) max_wy = group_max<BWD_G>(gvalid ? wy : 0);
    if (max_wz == KEY_Z) max_wz = group_max<BWD_G>(gvalid ? wz : 0);
    if (max_wx == KEY_X * BWD_G) max_wx = group_max<BWD_G>(wx);
    const float dy0 = (float)(YC - shift) - r0.y; // dy = dy0 + k at step k of a column
    const float g1 = dy0 * kxy, g2 = dy0 * kyz, A0 = kyy * dy0 * dy0, B0 = 2.0f * kyy * dy0;
    const uint32_t base =
        (uint32_t)(PAD + (loz - t0z) * RZS + (loy - t0y - shift) * RX + (lox - t0x));
    Moments v = {};
    float k1 = 0.0f, k2 = 0.0f, k1x = 0.0f, k1z = 0.0f;
    const int nk = min(max_wy, NK_MAX);
    const bool whole = min_wy >= nk && !(rb & KEY_FEW);
#pragma unroll 1
    for (int x = ql; x - ql < max_wx; x += BWD_G) {
        const float dx = (float)x - cx;
        const int nz = x < wx ? wz : 0;
        const uint32_t off = base + x;
        const float Ab = fmaf(dx, fmaf(kxx, dx, g1), A0);
        const float hz = fmaf(kxz, dx, g2);
        const float Bx = fmaf(kxy, dx, B0);
        Sheet S = {};
#define SHEET(K, M) \
        lds_sheet<K, M>(region, off, nz, max_wz, few, ncol, max_wy, cz, Ab, hz, kzz, Bx, kyz, kyy, S)
#define SHEETS(K) case K: if (whole) SHEET(K, false); else SHEET(K, true); break
        switch (nk) {
        SHEETS(3); SHEETS(4); SHEETS(5); SHEETS(6); SHEETS(7); SHEETS(8);
        SHEETS(9); SHEETS(10); SHEETS(11);
        default: SHEET(NK_MAX, true); break;
        }
#undef SHEETS
#undef SHEET
        const float ax = S.s * dx;
        v.m += S.s;
        v.x += ax;
        v.xx = fmaf(ax, dx, v.xx);
        v.z += S.z;
        v.zz += S.zz;
        v.xz = fmaf(S.z, dx, v.xz);
        k1 += S.k;
        k2 += S.kk;
        k1x = fmaf(S.k, dx, k1x);
        k1z += S.kz;
    }
    // from sums over the step k to moments in dy = dy0 + k (dy0 is the Gaussian's):
    // sum (dy0 + k) gE = k1 + dy0 m, sum (dy0 + k)^2 gE = k2 + dy0 (2 k1 + dy0 m), and the
    // products with dx and dz likewise
    v.y = fmaf(dy0, v.m, k1);
    v.yy = fmaf(dy0, fmaf(2.0f, k1, dy0 * v.m), k2);
    v.xy = fmaf(dy0, v.x, k1x);
    v.yz = fmaf(dy0, v.z, k1z);
    store_partials<BWD_G>(a, gi, mine, gvalid, rec, v);
}

// A round of Gaussians whose dL/dI is read from global memory: boxes reaching past the staged
// region, the block query's wide ones, and masked grids.  A group maps its lanes onto chunks of
// BWD_G (x, z) columns of its Gaussian's box and walks each column along y, eight rows' reads at
// a time.  The walk is centred in y: Q = qxz + dy (by + kyy dy) with dy = dy0 + k, and the column
// sums are in dy itself, so that a box much wider than its Gaussian (the block query) adds no
// large terms that cancel.
template <bool MASK, int G>
__device__ __forceinline__ void global_round(const BackwardArgs& a, int kk, uint32_t mine,
                                             bool gvalid, const Rec& rec, bool mk)
{
#pragma clang fp contract(off)
    const int ql = threadIdx.x & (G - 1);
    const int nx = a.nx[kk], ny = a.ny[kk];
    const float* __restrict__ g = a.dl_di[kk];
    const float4 r0 = rec.r0, r1 = rec.r1, r2 = rec.r2, r3 = rec.r3;
    // masked grid: the Gaussian's cell and the grid's index -> world affine
    const int4 cm = (MASK && mk) ? a.bq.cells[min((int64_t)(mine & GM_ID_MASK), a.n - 1)]
                                 : make_int4(0, 0, 0, 0);
    const double* mw = a.m[kk];
    const int lox = __float_as_int(r2.z), loy = __float_as_int(r2.w), loz = __float_as_int(r3.x);
    const int hix = __float_as_int(r3.y), hiy = __float_as_int(r3.z), hiz = __float_as_int(r3.w);
    // a listed Gaussian's box is never empty; an invalid lane group (past the round's end)
    // holds a finite record (Gaussian 0's) and takes no steps: its box counts as empty
    const bool nonempty = gvalid && lox <= hix && loy <= hiy && loz <= hiz;
    const int wx = nonempty ? hix - lox + 1 : 1;
    const int wy = nonempty ? hiy - loy + 1 : 0;
    const int wz = nonempty ? hiz - loz + 1 : 0;
    const float cx = r0.x, cz = r0.z;
    const float kxx = r1.x, kyy = r1.y, kzz = r1.z, kxy = r1.w;
    const float kxz = r2.x, kyz = r2.y;
    const int fp = wx * wz;                       // (x, z) footprint of the box
    const int max_chunks = group_max<G>((fp + G - 1) / G);
    const int max_wy = group_max<G>(wy);
    // y steps every active column of the wavefront takes (no mask needed below it)
    const int min_wy = group_min<G>(nonempty ? wy : 64);
    // column f -> (x, z) = (f mod wx, f div wx), with fh = f + 1/2: z = floor(fh / wx) (the
    // fraction stays at least 1/(2 wx) away from an integer, far beyond the hardware
    // reciprocal's error for any f < 2^20) and x + 1/2 = fh - z wx, exact in float
    const float wxf = (float)wx;
    const float inv_wx = __builtin_amdgcn_rcpf(wxf);
    const float dy0 = -r0.y;
    const float cxh = cx + 0.5f;
    const float qlh = (float)ql + 0.5f;
    Moments v = {};
#pragma unroll 1
    for (int c = 0; c < max_chunks; ++c) {
        const float fh = fmaf((float)c, (float)G, qlh);
        const bool act = fh < (float)fp;
        const float zf = floorf(fh * inv_wx);
        const float xh = fmaf(-zf, wxf, fh);
        const float dx = xh - cxh, dz = zf - cz;
        // a lane outside the footprint reads the grid's first column and gets Q = -inf, so
        // its every term is exactly zero
        const float by = fmaf(kxy, dx, kyz * dz);
        const float qxz = act ? fmaf(dx, fmaf(kxx, dx, kxz * dz), kzz * dz * dz)
                              : -__builtin_inff();
        const int vx = lox + (int)xh, vz = loz + (int)zf;
        const uint32_t off = act ? (uint32_t)((vz * ny + loy) * nx + vx) : 0u;
        const int ncol = act ? wy : 1;             // steps whose voxel lies in the box
        float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f;
#pragma unroll 1
        for (int kb = 0; kb < max_wy; kb += 8) {
            float gv[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int k = kb + j;
                if (k < max_wy) {
                    if (k < min_wy) {
                        gv[j] = (g + (size_t)k * nx)[off];
                    } else {
                        const int kc = min(k, ncol - 1);
                        const float t = (g + (size_t)kc * nx)[off];
                        gv[j] = k < ncol ? t : 0.0f;
                    }
                }
            }
            if (MASK && mk) {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (kb + j < max_wy &&
                        !voxel_in_block(mw, a.bq.res, a.bq.radius, vx, loy + kb + j, vz, cm))
                        gv[j] = 0.0f;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (kb + j < max_wy) {
                    const float dy = dy0 + (float)(kb + j);
                    const float Q = fmaf(dy, fmaf(kyy, dy, by), qxz);
                    const float ge = gv[j] * __builtin_amdgcn_exp2f(Q);
                    s0 += ge;
                    s1 = fmaf(dy, ge, s1);
                    s2 = fmaf(dy * dy, ge, s2);
                }
            }
        }
        const float ax = s0 * dx, az = s0 * dz;
        v.m += s0;
        v.x += ax;
        v.z += az;
        v.xx = fmaf(ax, dx, v.xx);
        v.zz = fmaf(az, dz, v.zz);
        v.xz = fmaf(ax, dz, v.xz);
        v.y += s1;
        v.yy += s2;
        v.xy = fmaf(s1, dx, v.xy);
        v.yz = fmaf(s1, dz, v.yz);
    }
    store_partials<G>(a, a.grid_index[kk], mine, gvalid, rec, v);
}

// Exclusive prefix sums of hist[0..NKEY) in place and the total in hist[NKEY], by one
// wavefront (a run of keys per lane).
__device__ __forceinline__ void scan_keys(int* hist, int lane)
{
    constexpr int PER = (NKEY + 63) / 64;
    int c[PER], sum = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int k = PER * lane + i;
        c[i] = k < NKEY ? hist[k] : 0;
        sum += c[i];
    }
    int incl = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(incl, d, 64);
        if (lane >= d) incl += t;
    }
    int off = incl - sum;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int k = PER * lane + i;
        if (k < NKEY) hist[k] = off;
        off += c[i];
    }
    if (lane == 63) hist[NKEY] = incl;
}

// One block (four wavefronts) per part of a tile's list (1 << parts_log2 parts per tile, by
// partial_parts below).  The block sorts the part's home Gaussians (home: the tile holds the box's
// lower corner, so every Gaussian of the grid is home exactly once), WINB list entries at a time,
// by the loop trips of their boxes: a counting sort over (x passes, planes, y length) with LDS
// atomics.  It stages the dL/dI region they need in LDS (coalesced rows).  The sorted Gaussians are
// taken PER_ROUND at a time, rounds dealt to the wavefronts in turn, so that the Gaussians of a
// round have similar loop trips and the wavefronts similar work.  Each Gaussian is read from LDS
// when its box lies inside the region (the common case) and from global memory otherwise.  A
// Gaussian's partials come from its own lanes only and do not depend on which others share its
// round, so the order the atomics give within a key does not change any result bit.  Gaussians
// with an empty box are in no list; gm_bin wrote their zeros.
//
// Bound by vector issue (173 M VALU instructions at the 256^3 workload, half of them walking
// boxes) and by latency: list, records, region and sort precede a block's first round, and five
// blocks a CU (29 KB of LDS, 96 VGPRs) have to cover that.  1M Gaussians on three 256x256x64
// stacks 378 us, 200k on 128x128x32 90, 20k on 64x64x16 38 (29 with the list in four parts); with
// eight lanes per Gaussian walking dense chunks of (x, z) columns, a column's place found anew for
// each, 425, 104 and 44.  Staging the records in LDS as well (four blocks a CU) took 460, the next
// round's records in flight while one is walked 443 (the registers cost a block, and the wait for
// them is also one for the stores in between).
template <bool MASK>
__global__ __launch_bounds__(256, MASK ? 4 : 5) void k_partials(const BackwardArgs a)
{
    __shared__ float region[REGION];        // from PAD on
    __shared__ uint32_t order[WINB];
    __shared__ int hist[NKEY + 1];
    __shared__ uint32_t round_box[WINB / PER_ROUND];
    __shared__ int zext;
    const int blk = xcd_remap(blockIdx.x, gridDim.x);
    const int lin = blk >> a.parts_log2;
    int kk = 0;                                            // listed grid of this block
#pragma unroll 1
    while (kk + 1 < a.n_ids && lin >= a.block_start[kk + 1]) ++kk;
    const int t = lin - a.block_start[kk];
    const int ntx = a.ntx[kk], nty = a.nty[kk];
    const int t0x = (t % ntx) * GM_TX, t0y = ((t / ntx) % nty) * GM_TY, t0z = (t / (ntx * nty)) * GM_TZ;
    const int64_t T = a.tile_base[kk] + t;
    int e0 = __builtin_amdgcn_readfirstlane(a.tile_start[T]);
    int e1 = __builtin_amdgcn_readfirstlane(a.tile_start[T + 1]);
    {   // this block's part of the tile's list
        const int per = (int)(((int64_t)(e1 - e0) + (1 << a.parts_log2) - 1) >> a.parts_log2);
        e0 = min(e0 + (blk & ((1 << a.parts_log2) - 1)) * per, e1);
        e1 = min(e0 + per, e1);
    }
    if (e0 == e1) return;  // block-uniform
    const int nx = a.nx[kk], ny = a.ny[kk], nz = a.nz[kk];
    const float* __restrict__ g = a.dl_di[kk];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int gi = a.grid_index[kk];
    const bool mk = MASK && a.masked[kk];   // block query on a rotated grid

    // list entry -> its sort key (-1: not a home entry) and the z planes its box reaches in
    // the region (0 when it reaches past the region; always on a masked grid, whose voxels
    // are tested in the global-memory path)
    auto classify = [&](int entry, uint32_t& v, int& zreach) -> int {
        zreach = 0;
        v = entry < e1 ? a.pair_gauss[entry] : 0u;
        if (entry >= e1 || !(v & GM_HOME_BIT)) return -1;
        if (mk) return NKEY - 1;
        const int4* rc = reinterpret_cast<const int4*>(
            a.records + ((size_t)gi * a.n + min((int64_t)(v & GM_ID_MASK), a.n - 1)) * 16);
        const int4 r2 = rc[2], r3 = rc[3];     // (kxz, kyz, lox, loy), (loz, hix, hiy, hiz)
        const int lx = r2.z, ly = r2.w, lz = r3.x, hx = r3.y, hy = r3.z, hz = r3.w;
        if (!(hx - t0x < RX && hy - t0y < RY && hz - t0z < RZ)) return NKEY - 1;
        if (a.block_query) {
            // a box much wider in y than its Gaussian (|kyy| wy^2 > 64; a 3-sigma box stays
            // below about 50) takes the global-memory path, whose walk is centred
            const float kyy = __int_as_float(rc[1].y);
            const float wyf = (float)(hy - ly + 1);
            if (fabsf(kyy) * wyf * wyf > 64.0f) return NKEY - 1;
        }
        zreach = hz - t0z + 1;
        return (min((hx - lx) / BWD_G, KEY_X - 1) * KEY_Z + min(hz - lz, KEY_Z - 1)) * KEY_Y +
               min(hy - ly, KEY_Y - 1);
    };
    uint32_t v[EPT];
    int key[EPT], rank[EPT];
    // counts the keys of entries [w0, w0 + WINB) into hist (zeroed before); a thread's rank
    // within its key is the count the atomic returns
    auto count_keys = [&](int w0, int& zmax) {
#pragma unroll
        for (int h = 0; h < EPT; ++h) {
            int zr;
            key[h] = classify(w0 + h * 256 + tid, v[h], zr);
            zmax = max(zmax, zr);
            rank[h] = key[h] >= 0 ? atomicAdd(&hist[key[h]], 1) : 0;
        }
    };
    auto scatter = [&]() {
#pragma unroll
        for (int h = 0; h < EPT; ++h)
            if (key[h] >= 0) {
                const int pos = hist[key[h]] + rank[h];
                order[pos] = v[h];
                if (key[h] < NKEY - 1) {
                    const int zx = key[h] / KEY_Y;
                    const int y = key[h] - zx * KEY_Y;
                    atomicOr(&round_box[pos / PER_ROUND],
                             (y < SHIFT ? KEY_FEW | (1u << (y + SHIFT)) : 1u << y) |
                             (1u << (KEY_Y + zx % KEY_Z)) | (1u << (KEY_Y + KEY_Z + zx / KEY_Z)));
                }
            }
    };
    // the rounds of one sorted window: n_lds Gaussians from LDS, then the rest from global
    // memory
    const int grp = lane / BWD_G;
    auto rounds = [&](int n_lds, int n_all) {
        const int nr = (n_lds + PER_ROUND - 1) / PER_ROUND;
#pragma unroll 1
        for (int q = 0; q < nr; q += 4) {
            // rounds grow with r: dealt out forwards and backwards in turn
            const int r = q + (q & 4 ? 3 - wv : wv);
            if (r >= nr) continue;
            const int ix = r * PER_ROUND + grp;
            const bool valid = ix < n_lds;
            const uint32_t m = valid ? order[ix] : 0u;
            const Rec rec = load_record(a, gi, m);
            lds_round(a, gi, m, valid, rec, region, t0x, t0y, t0z, (uint32_t)sgpr(round_box[r]));
        }
        // From global memory: a wavefront each, whose 64 lanes see a box in one or two reads'
        // latency, or eight lanes each with the block query, whose many small boxes past the region
        // are better taken eight at a time.  The width is the query's alone, so that a Gaussian's
        // sums do not depend on the others listed.  Partials of Gaussians 1, 2, 3 and 5 voxels wide
        // on three 256x256x64 stacks, us with 64 lanes and with 8: 367 and 398, 388 and 616, 390 and
        // 1048, 251 and 2003 (8 where a window holds more than 16 such boxes: 367, 447, 424, 363);
        // three 64x64x16 stacks, block query of radius 2, 3 and 4: 93 and 43, 115 and 73, 232 and 166.
        auto from_global = [&](auto g_lanes) {
            constexpr int GG = decltype(g_lanes)::value, PER = 64 / GG;
#pragma unroll 1
            for (int r = wv; r < (n_all - n_lds + PER - 1) / PER; r += 4) {
                const int ix = n_lds + r * PER + lane / GG;
                const bool valid = ix < n_all;
                const uint32_t m = valid ? order[ix] : 0u;
                const Rec gr = load_record(a, gi, m);
                global_round<MASK, GG>(a, kk, m, valid, gr, mk);
            }
        };
        if (a.block_query)
            from_global(std::integral_constant<int, 8>{});
        else
            from_global(std::integral_constant<int, 64>{});
    };

    // WINB entries of the list at a time.  With the first, the z planes the home boxes reach
    // (those that fit the region) are found over the whole list and only those planes staged.
    if (tid == 0) zext = 0;
#pragma unroll 1
    for (int w0 = e0; w0 < e1; w0 += WINB) {
        for (int i = tid; i < NKEY; i += 256) hist[i] = 0;
        if (tid < WINB / PER_ROUND) round_box[tid] = 0u;
        __syncthreads();
        int zmax = 0;
        count_keys(w0, zmax);
        if (w0 == e0) {
            for (int i = e0 + WINB + tid; i < e1; i += 256) {
                uint32_t vi;
                int zr;
                classify(i, vi, zr);
                zmax = max(zmax, zr);
            }
            if (zmax > 0) atomicMax(&zext, zmax);
        }
        __syncthreads();
        if (wv == 0) scan_keys(hist, lane);
        if (w0 == e0) {
            const int nzr = min(zext, nz - t0z);
            // rows of RX voxels along x: thread -> (x, y) of a plane, then the planes
            for (int i = tid; i < RX * RY; i += 256) {
                const int y = i / RX, x = i - y * RX;
                const int gx = t0x + x, gy = t0y + y;
                const bool in = gx < nx && gy < ny;
                const float* src = g + ((size_t)t0z * ny + gy) * nx + gx;
                float* dst = region + PAD + y * RX + x;
                for (int z = 0; z < nzr; ++z) {
                    dst[z * RZS] = in ? src[0] : 0.0f;
                    src += (size_t)nx * ny;
                }
            }
        }
        __syncthreads();
        scatter();
        __syncthreads();
        rounds(hist[NKEY - 1], hist[NKEY]);
        __syncthreads();                       // order, hist and round_box are free again
    }
}

// symmetric 3x3 stored full, row-major
__device__ __forceinline__ void mm3(const double* A, const double* B, double* C)
{
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            C[3 * i + j] = A[3 * i] * B[j] + A[3 * i + 1] * B[3 + j] + A[3 * i + 2] * B[6 + j];
}

__device__ __forceinline__ double inv3(const double* A, double* Ai)
{
    const double c00 = A[4] * A[8] - A[5] * A[7];
    const double c01 = A[5] * A[6] - A[3] * A[8];
    const double c02 = A[3] * A[7] - A[4] * A[6];
    const double det = A[0] * c00 + A[1] * c01 + A[2] * c02;
    const double id = 1.0 / det;
    Ai[0] = c00 * id;
    Ai[1] = (A[2] * A[7] - A[1] * A[8]) * id;
    Ai[2] = (A[1] * A[5] - A[2] * A[4]) * id;
    Ai[3] = c01 * id;
    Ai[4] = (A[0] * A[8] - A[2] * A[6]) * id;
    Ai[5] = (A[2] * A[3] - A[0] * A[5]) * id;
    Ai[6] = c02 * id;
    Ai[7] = (A[1] * A[6] - A[0] * A[7]) * id;
    Ai[8] = (A[0] * A[4] - A[1] * A[3]) * id;
    return det;
}

// One Gaussian on one grid: from its grid-frame partials pg (d amp, d c, d K) and its world
// covariance Sig, the derivative Gi = dL/dSigma_idx (C = Sigma_g^-1 gives dL/dSigma_g =
// -C G_C C; amp = alpha sqrt(det Sigma_idx / det Sigma_g) adds -1/2 d_amp amp C and
// +1/2 d_amp amp Sigma_idx^-1), the centre partial dc, and amp.
__device__ __forceinline__ double sigma_idx_grad(const GridConst& G, const double* Sig,
                                                 double alpha, const float* pg, double* dc,
                                                 double* Gi)
{
    const double damp = pg[0];
    dc[0] = pg[1];
    dc[1] = pg[2];
    dc[2] = pg[3];
    // full-matrix dL/dC from the base-2 conic partials: C-entry = K-entry * KAPPA
    const double GC[9] = {GM_KAPPA * pg[4], GM_KAPPA * pg[7], GM_KAPPA * pg[8],
                          GM_KAPPA * pg[7], GM_KAPPA * pg[5], GM_KAPPA * pg[9],
                          GM_KAPPA * pg[8], GM_KAPPA * pg[9], GM_KAPPA * pg[6]};
    const double* L = G.L;
    double T[9], SI[9];
    mm3(L, Sig, T);
    const double Lt[9] = {L[0], L[3], L[6], L[1], L[4], L[7], L[2], L[5], L[8]};
    mm3(T, Lt, SI);  // Sigma_idx
    double SG[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) SG[t] = SI[t];
    SG[8] += G.sig * G.sig;
    double C[9], SIi[9];
    const double detG = inv3(SG, C);
    const double detI = inv3(SI, SIi);
    const double amp = alpha * sqrt(detI / detG);
    double CG[9], CGC[9];
    mm3(C, GC, CG);
    mm3(CG, C, CGC);
    const double ha = 0.5 * damp * amp;
#pragma unroll
    for (int t = 0; t < 9; ++t) Gi[t] = -CGC[t] - ha * C[t] + ha * SIi[t];
    return amp;
}

// Normalised quaternion (w, x, y, z), its rotation R (Hamilton) and Sigma = R diag(S2) R^T.
__device__ __forceinline__ void world_covariance(const float* quat, const float* log_scale,
                                                 int64_t i, double* qh, double* qn, double* R,
                                                 double* S2, double* Sig)
{
    const double qw = quat[4 * i], qx = quat[4 * i + 1], qy = quat[4 * i + 2],
                 qz = quat[4 * i + 3];
    *qn = sqrt(qw * qw + qx * qx + qy * qy + qz * qz);
    const double w = qw / *qn, x = qx / *qn, y = qy / *qn, z = qz / *qn;
    qh[0] = w;
    qh[1] = x;
    qh[2] = y;
    qh[3] = z;
    R[0] = 1.0 - 2.0 * (y * y + z * z);
    R[1] = 2.0 * (x * y - w * z);
    R[2] = 2.0 * (x * z + w * y);
    R[3] = 2.0 * (x * y + w * z);
    R[4] = 1.0 - 2.0 * (x * x + z * z);
    R[5] = 2.0 * (y * z - w * x);
    R[6] = 2.0 * (x * z - w * y);
    R[7] = 2.0 * (y * z + w * x);
    R[8] = 1.0 - 2.0 * (x * x + y * y);
#pragma unroll
    for (int m = 0; m < 3; ++m) S2[m] = exp(2.0 * (double)log_scale[3 * i + m]);
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int q = 0; q < 3; ++q)
            Sig[3 * p + q] = R[3 * p] * S2[0] * R[3 * q] + R[3 * p + 1] * S2[1] * R[3 * q + 1] +
                             R[3 * p + 2] * S2[2] * R[3 * q + 2];
}

// three waves per SIMD (at most 168 VGPRs): a few registers more drop it to two, 25% slower
__global__ __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(3))) void k_chain(const ChainArgs a)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n) return;
    double qh[4], qn, R[9], S2[3], Sig[9];
    world_covariance(a.quat, a.log_scale, i, qh, &qn, R, S2, Sig);
    const double w = qh[0], x = qh[1], y = qh[2], z = qh[3];
    const double ls[3] = {a.log_scale[3 * i], a.log_scale[3 * i + 1], a.log_scale[3 * i + 2]};
    const double alpha = 1.0 / (1.0 + exp(-(double)a.logit[i]));

    double dmu[3] = {0, 0, 0}, GS[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0}, dalpha = 0.0;
#pragma unroll 1
    for (int k = 0; k < a.n_ids; ++k) {
        const GridConst& G = a.g[k];
        const int gi = a.grid_index[k];
        const float* pg = a.grid_grads + ((size_t)gi * a.n + i) * 10;
        if (a.tile_count[(size_t)gi * a.n + i] == 0) continue;  // empty box
        double dc[3], Gi[9];
        const double amp = sigma_idx_grad(G, Sig, alpha, pg, dc, Gi);
        const double* L = G.L;
        // mu
#pragma unroll
        for (int m = 0; m < 3; ++m) dmu[m] += L[m] * dc[0] + L[3 + m] * dc[1] + L[6 + m] * dc[2];
        // Sigma = L^T Gi L
        const double Lt[9] = {L[0], L[3], L[6], L[1], L[4], L[7], L[2], L[5], L[8]};
        double U[9], V9[9];
        mm3(Lt, Gi, U);
        mm3(U, L, V9);
#pragma unroll
        for (int t = 0; t < 9; ++t) GS[t] += V9[t];
        dalpha += (double)pg[0] * amp / alpha;
    }
    // Sigma = R diag(S2) R^T
    double GR[9], RtGR[9], GRR[9];
    mm3(GS, R, GR);  // G R
    double Rt[9] = {R[0], R[3], R[6], R[1], R[4], R[7], R[2], R[5], R[8]};
    mm3(Rt, GR, RtGR);
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int q = 0; q < 3; ++q) GRR[3 * p + q] = 2.0 * GR[3 * p + q] * S2[q];  // dL/dR
    double ds[3] = {2.0 * S2[0] * RtGR[0], 2.0 * S2[1] * RtGR[4], 2.0 * S2[2] * RtGR[8]};
    const double* g = GRR;
    double dq[4];
    dq[0] = 2.0 * (-z * g[1] + y * g[2] + z * g[3] - x * g[5] - y * g[6] + x * g[7]);
    dq[1] = 2.0 * (y * g[1] + z * g[2] + y * g[3] - 2.0 * x * g[4] - w * g[5] + z * g[6] +
                   w * g[7] - 2.0 * x * g[8]);
    dq[2] = 2.0 * (-2.0 * y * g[0] + x * g[1] + w * g[2] + x * g[3] + z * g[5] - w * g[6] +
                   z * g[7] - 2.0 * y * g[8]);
    dq[3] = 2.0 * (-2.0 * z * g[0] - w * g[1] + x * g[2] + w * g[3] - 2.0 * z * g[4] + y * g[5] +
                   x * g[6] + y * g[7]);
    const double dot = w * dq[0] + x * dq[1] + y * dq[2] + z * dq[3];
    // anisotropy regulariser (Eq. 13 on the actual scales)
    if (a.lambda_aniso != 0.0f) {
        int im = 0, in = 0;
#pragma unroll
        for (int m = 1; m < 3; ++m) {
            if (a.log_scale[3 * i + m] > a.log_scale[3 * i + im]) im = m;
            if (a.log_scale[3 * i + m] < a.log_scale[3 * i + in]) in = m;
        }
        const double ratio = exp(ls[im] - ls[in]);
        if (ratio > (double)a.lambda_r) {
            const double gr = (double)a.lambda_aniso * ratio / (double)a.n;
            ds[im] += gr;
            ds[in] -= gr;
        }
    }
    float gr[11];  // the gradient as float: mean (3), quat (4), log_scale (3), logit (1)
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        gr[m] = (float)dmu[m];
        gr[7 + m] = (float)ds[m];
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) gr[3 + m] = (float)((dq[m] - qh[m] * dot) / qn);
    gr[10] = (float)(dalpha * alpha * (1.0 - alpha));
    if (!a.adam) {
#pragma unroll
        for (int m = 0; m < 3; ++m) {
            a.g_mean[3 * i + m] += gr[m];
            a.g_log_scale[3 * i + m] += gr[7 + m];
        }
#pragma unroll
        for (int m = 0; m < 4; ++m) a.g_quat[4 * i + m] += gr[3 + m];
        a.g_logit[i] += gr[10];
        return;
    }
    // fused Adam: the value a zeroed gradient buffer would hold (0 + g), applied at once to
    // the parameter and its moments, group by group
    constexpr int width[4] = {3, 4, 3, 1}, first[4] = {0, 3, 7, 10};
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) {
#pragma unroll
        for (int m = 0; m < width[grp]; ++m) {
            const int64_t e = width[grp] * i + m;
            float pv = a.prm[grp][e], mv = a.m1[grp][e], vv = a.m2[grp][e];
            adam_elem(pv, mv, vv, 0.0f + gr[first[grp] + m], a.adam_s[grp]);
            a.m1[grp][e] = mv;
            a.m2[grp][e] = vv;
            a.prm[grp][e] = pv;
        }
    }
}

// Gradient with respect to each listed grid's world->index affine [L | t] (boxes fixed): per
// Gaussian, c = L mu + t contributes dc mu^T to dL/dL and dc to dL/dt, and Sigma_idx =
// L Sigma L^T contributes 2 Gi L Sigma.  One pass over the Gaussians per grid; FP64 block sums
// part[block][grid][12] (row-major 3x4), added in a fixed order by k_pose_sum.
constexpr int POSE_BLOCKS = 256, POSE_THREADS = 256;
static_assert(GM_POSE_WORKSPACE_BYTES(1) == (size_t)POSE_BLOCKS * 12 * sizeof(double),
              "the header's workspace size follows the block count");

__global__ __launch_bounds__(POSE_THREADS) void k_pose(const ChainArgs a, double* part)
{
    __shared__ double red[POSE_THREADS / 64][12];
    for (int k = 0; k < a.n_ids; ++k) {
        const GridConst& G = a.g[k];
        const int gi = a.grid_index[k];
        double acc[12];
#pragma unroll
        for (int j = 0; j < 12; ++j) acc[j] = 0.0;
        for (int64_t i = (int64_t)blockIdx.x * POSE_THREADS + threadIdx.x; i < a.n;
             i += (int64_t)gridDim.x * POSE_THREADS) {
            if (a.tile_count[(size_t)gi * a.n + i] == 0) continue;  // empty box
            double qh[4], qn, R[9], S2[3], Sig[9];
            world_covariance(a.quat, a.log_scale, i, qh, &qn, R, S2, Sig);
            const double alpha = 1.0 / (1.0 + exp(-(double)a.logit[i]));
            const float* pg = a.grid_grads + ((size_t)gi * a.n + i) * 10;
            double dc[3], Gi[9];
            sigma_idx_grad(G, Sig, alpha, pg, dc, Gi);
            double GL[9], GLS[9];
            mm3(Gi, G.L, GL);
            mm3(GL, Sig, GLS);
            const double mu[3] = {a.mean[3 * i], a.mean[3 * i + 1], a.mean[3 * i + 2]};
#pragma unroll
            for (int r = 0; r < 3; ++r) {
#pragma unroll
                for (int c = 0; c < 3; ++c) acc[4 * r + c] += dc[r] * mu[c] + 2.0 * GLS[3 * r + c];
                acc[4 * r + 3] += dc[r];
            }
        }
        // block sum: wavefront butterflies, then the four wavefronts in order
#pragma unroll
        for (int j = 0; j < 12; ++j)
            for (int o = 32; o > 0; o >>= 1) acc[j] += __shfl_xor(acc[j], o, 64);
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int j = 0; j < 12; ++j) red[threadIdx.x >> 6][j] = acc[j];
        __syncthreads();
        if (threadIdx.x < 12) {
            double v = 0.0;
            for (int w = 0; w < POSE_THREADS / 64; ++w) v += red[w][threadIdx.x];
            part[((size_t)blockIdx.x * a.n_ids + k) * 12 + threadIdx.x] = v;
        }
        __syncthreads();
    }
}

// one block per (grid, entry): the block partials added by a fixed tree in LDS
__global__ __launch_bounds__(POSE_BLOCKS) void k_pose_sum(const double* part, int nb, int n_ids,
                                                          double* out)
{
    __shared__ double sh[POSE_BLOCKS];
    const int e = blockIdx.x;   // (grid, entry)
    sh[threadIdx.x] = (int)threadIdx.x < nb ? part[(size_t)threadIdx.x * n_ids * 12 + e] : 0.0;
    __syncthreads();
    for (int o = POSE_BLOCKS / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[e] = sh[0];
}

}  // namespace

// Blocks per tile (log2): as many as leave the launch within what the chip holds at a time, since
// each part pays the sort and the staging again.  Three 64x64x16 stacks (192 tiles): a step of
// 128 us with four parts, 137 with one, 129 with eight; three 96x96x24 (648 tiles): 196 with two,
// 191 with one.  The block query's boxes are many times larger than the staging, and a part more
// even: 192 tiles at radius 3, 271 us with 16 parts, 286 with 8, 550 with one, 277 with 32.  Beyond what
// fills the chip once its parts only add launches' ends: the partials alone of three rotated stacks
// at radius 2 with 1, 2, 4 and 8 parts, us: 375 tiles 371, 296, 256, 198; 648: 411, 449, 345, 320; 1029:
// 486, 593, 527, 511; 1536: 655, 831, 777, 772; 3000: 1709, 2672, 2550, 1941 (axis-aligned 98 to 71, 89
// to 95, 119 to 176, 141 to 281, 419 to 721).
static int partial_parts_log2(int64_t tiles, bool block_query)
{
    const int64_t blocks = !block_query ? 1024 : tiles <= 768 ? 4096 : 0;
    int lg = 0;
    while (lg < 4 && tiles << (lg + 1) <= blocks) ++lg;
    return lg;
}

hipError_t launch_backward_partials(const BackwardArgs& args, hipStream_t s)
{
    if (args.n == 0 || args.n_ids == 0) return hipSuccess;
    const int32_t tiles = args.block_start[args.n_ids];   // of the listed grids
    if (tiles <= 0) return hipSuccess;
    BackwardArgs a = args;
    a.parts_log2 = partial_parts_log2(tiles, a.block_query != 0);
    bool masked = false;
    for (int k = 0; k < a.n_ids; ++k) masked = masked || a.masked[k];
    const dim3 grid((unsigned)tiles << a.parts_log2);
    if (masked)
        hipLaunchKernelGGL(k_partials<true>, grid, dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(k_partials<false>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_chain(const ChainArgs& a, hipStream_t s)
{
    if (a.n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_chain, dim3((unsigned)((a.n + 127) / 128)), dim3(128), 0, s, a);
    return hipGetLastError();
}

size_t pose_workspace_bytes(int n_ids) { return (size_t)POSE_BLOCKS * n_ids * 12 * sizeof(double); }

hipError_t launch_pose(const ChainArgs& a, double* out, void* ws, hipStream_t s)
{
    if (a.n_ids == 0) return hipSuccess;
    int64_t nb = (a.n + POSE_THREADS - 1) / POSE_THREADS;
    if (nb > POSE_BLOCKS) nb = POSE_BLOCKS;
    if (nb < 1) nb = 1;
    double* part = reinterpret_cast<double*>(ws);
    hipLaunchKernelGGL(k_pose, dim3((unsigned)nb), dim3(POSE_THREADS), 0, s, a, part);
    hipLaunchKernelGGL(k_pose_sum, dim3((unsigned)(a.n_ids * 12)), dim3(POSE_BLOCKS), 0, s, part,
                       (int)nb, a.n_ids, out);
    return hipGetLastError();
}
