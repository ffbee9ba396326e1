// SSIM term of the reconstruction loss (Sec. 3.5.2, Eq. 10) on whole stack slices, with its
// gradient, in one pass down strips of the slices (small stacks in tiles, ssim_tiles.hip).
//
// Every z-slice of a stack is a 2D image.  The SSIM map uses an 11 x 11 Gaussian window (the
// outer product of 11 taps g, sigma 1.5), zero padding outside the slice, C1 = 0.01^2 and
// C2 = 0.03^2.  L = 1 - mean of the map over every stack voxel, and with the window sums
// (mu_x, m_xx, m_xy) taken as the variables,
//     dL/dx_q = -(1/N) sum_p w(q - p) [S_mu + 2 x_q S_xx + y_q S_xy](p).
//
// The statistics and the map's partial derivatives are formed in FP64: the variances are
// differences of window sums (m - mu^2), whose cancellation would cost FP32 about four of its
// seven digits, and gfx950 issues FP64 FMAs at its FP32 (unpacked) rate.
//
// A wavefront takes a strip of OUT_X = 54 pixel columns (64 map columns, one per lane, R = 5 of
// them on either side for the adjoint) and a segment of rows, and walks it downwards one row at a
// time:
//   1. the row of x (prediction) and y (target) goes to LDS; each lane forms the horizontal
//      window sums of x, y, x^2 + y^2 (the variances enter only as their sum) and x y at its
//      column;
//   2. they are added into the 11 map rows the row belongs to, whose running vertical sums the
//      lane holds in registers; the map row that is now complete gives SSIM and its three
//      partials (zero outside the slice);
//   3. those are added into the 11 output rows they belong to (running sums again), and the
//      output row now complete takes its horizontal adjoint pass through LDS and
//      dl[q] += -(lambda / N) (A_mu + 2 x_q A_xx + y_q A_xy).
// So nothing between the input and the gradient is stored, each row's window sums are formed once
// per strip, and there is no barrier.  A segment reads 10 rows above and below its own.  The loop
// is unrolled over 11 rows, so that which running sum a row starts and completes is known at
// compile time.  Bound by vector issue: about 210 FP64 operations per row and lane, of which 54 of
// 64 lanes count.  Three 256x256x64 stacks: 0.252 ms; with 32 x 32 tiles of 1024 threads, every
// pass through LDS with a barrier after it, 0.444 ms (the tiles' halos cost 1.7 to 2.1 times the
// window sums).
// Each map position is summed by one wavefront and each pixel written by one; the wavefronts'
// FP64 sums are added in a fixed order, so loss and gradient are the same on every run.
#include <utility>

#include "ssim_core.h"

namespace {

using namespace ssimcore;

constexpr int OUT_X = 64 - 2 * R;                 // output columns of a strip
constexpr int ROW = 64 + 2 * R;                   // input columns of a strip
// two wavefronts per SIMD (up to 256 registers each) on 256 CUs: all blocks resident at once
constexpr int SIMDS = 1024, SLOTS = 2 * SIMDS;
static_assert(SLOTS <= MAX_PARTS, "a sum for every block");

struct Lds {
    float x[2][ROW], y[2][ROW];
    double u[3][ROW];          // an output row's vertical adjoint sums, lane l at l + R
};

// a wavefront has an Lds of its own: its LDS accesses execute in order, only the compiler has to keep them so
__device__ __forceinline__ void lds_order()
{
    __asm__ __volatile__("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

// Nothing is scheduled across this point: the phases of a row, interleaved, would hold more live
// values than the registers do.
#define PHASE() __builtin_amdgcn_sched_barrier(0)

struct Strip {
    const float* x;            // the slice
    const float* y;
    float* dl;
    int nx, ny, x0, y0, y1;    // first output column, output rows [y0, y1)
};

__device__ __forceinline__ Strip strip(const SsimArgs& a, int64_t t)
{
    int k = 0;
    while (t >= a.tile_begin[k + 1]) ++k;
    Strip s;
    s.nx = a.nx[k];
    s.ny = a.ny[k];
    const int64_t local = t - a.tile_begin[k];
    const int per_slice = a.tiles_x[k] * a.tiles_y[k];
    const int64_t z = local / per_slice;
    const int rem = (int)(local - z * per_slice);
    const int seg = rem / a.tiles_x[k];
    s.x0 = (rem - seg * a.tiles_x[k]) * OUT_X;
    s.y0 = seg * a.rows[k];
    s.y1 = min(s.y0 + a.rows[k], s.ny);
    const int64_t o = z * s.ny * s.nx;
    s.x = a.pred[k] + o;
    s.y = a.target[k] + o;
    s.dl = a.dl[k] + o;
    return s;
}

// row<0>, row<1>, ... row<10> for consecutive r
template <class F, int... P>
__device__ __forceinline__ void cycle(F& row, int& r, std::integer_sequence<int, P...>)
{
    ((row(std::integral_constant<int, P>{}), ++r), ...);
}

// Four strips to a block, one on each SIMD of its CU (blocks of one wavefront fall on the SIMDs as the
// launch before left them: 40 us or 56 for the same 920).  ALONE: a block takes so much LDS that a
// CU holds no second one while others are empty.
constexpr int WPB = 4;
template <bool ALONE>
__global__ __launch_bounds__(64 * WPB, ALONE ? 1 : 2) void k_ssim(const SsimArgs a, double* part, int nw)
{
    __shared__ struct { Lds w[WPB]; char room[ALONE ? 72 * 1024 : 1]; } all;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int first = (int)blockIdx.x * WPB + w;
    Lds& s = all.w[w];
    const int64_t total = a.tile_begin[a.n_stacks];
    double ssum = 0.0;
    if (lane < R) {            // the columns past the strip's lanes: read, never used
#pragma unroll
        for (int q = 0; q < 3; ++q) s.u[q][lane] = s.u[q][64 + R + lane] = 0.0;
    }
#pragma unroll 1
    for (int64_t t = first; t < total; t += gridDim.x * WPB) {
        const Strip S = strip(a, t);
        const int X = S.x0 - R + lane;                       // the lane's map column
        const bool in_x = X >= 0 && X < S.nx;
        const bool own = lane >= R && lane < R + OUT_X && in_x;
        // input columns of the lane's two LDS entries
        const int c0 = S.x0 - 2 * R + lane, c1 = c0 + 64;
        const bool i0 = c0 >= 0 && c0 < S.nx, i1 = lane < 2 * R && c1 < S.nx;
        // two input rows and one output row's pixel and gradient are in flight
        struct In {
            float x0, y0, x1, y1;
        };
        auto fetch = [&](int r) {
            const bool in = r >= 0 && r < S.ny;
            const float* xr = S.x + (int64_t)r * S.nx;
            const float* yr = S.y + (int64_t)r * S.nx;
            In n = {0.0f, 0.0f, 0.0f, 0.0f};
            if (in && i0) {
                n.x0 = xr[c0];
                n.y0 = yr[c0];
            }
            if (in && i1) {
                n.x1 = xr[c1];
                n.y1 = yr[c1];
            }
            return n;
        };
        struct Out {
            float x, y, d;
        };
        auto fetch_out = [&](int o) {
            Out n = {0.0f, 0.0f, 0.0f};
            if (o >= S.y0 && o < S.y1 && own) {
                n.x = (S.x + (int64_t)o * S.nx)[X];
                n.y = (S.y + (int64_t)o * S.nx)[X];
                n.d = (S.dl + (int64_t)o * S.nx)[X];
            }
            return n;
        };
        // running sums: of map rows (v) and of output rows (u); a row starts by assignment
        double v[WN][4], u[WN][3];
#pragma unroll
        for (int i = 0; i < WN; ++i) {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[i][q] = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) u[i][q] = 0.0;
        }
        const int r_end = S.y1 + 2 * R + 1;                  // an output row is finished a row late
        int r = S.y0 - 2 * R, buf = 0;                       // input row, its LDS buffer
        auto stage = [&](int b, const In& n) {
            lds_order();
            s.x[b][lane] = n.x0;
            s.y[b][lane] = n.y0;
            if (lane < 2 * R) {
                s.x[b][64 + lane] = n.x1;
                s.y[b][64 + lane] = n.y1;
            }
            lds_order();
        };
        stage(0, fetch(r));
        In nx = fetch(r + 1);
        Out no = fetch_out(r - 2 * R - 1);
        // One row of an unrolled cycle, p = (r - first row) mod 11.  The row's input is in LDS
        // already; the map row and output row that the previous input row completed are finished
        // here while it is read, and the output row's horizontal pass comes last, so that no LDS
        // access is waited for right after it is issued.
        auto row = [&](auto phase) {
            constexpr int p = decltype(phase)::value, pm = (p + WN - 1) % WN;
            // input row r into registers
            float xs[WN], ys[WN];
            lds_order();
#pragma unroll
            for (int i = 0; i < WN; ++i) xs[i] = s.x[buf][lane + i];
            PHASE();
            // 2. map row Y (its sums are complete) and its partials
            const int Y = r - 1 - R, o = Y - R;
            const double(&m)[4] = v[pm];
            const double mx = m[0], my = m[1];
            const double vxy = (m[2] - mx * mx) - my * my;          // var x + var y
            const double cxy = m[3] - mx * my;
            const double a1 = 2.0 * mx * my + GM_SSIM_C1, a2 = 2.0 * cxy + GM_SSIM_C2;
            const double b1 = mx * mx + my * my + GM_SSIM_C1, b2 = vxy + GM_SSIM_C2;
            const double rb = recip(b1 * b2), r1 = b2 * rb, r2 = b1 * rb;   // 1/b1, 1/b2
            const double sv = a1 * a2 * rb;
            const bool in = Y >= 0 && Y < S.ny && in_x;
            if (own && Y >= S.y0 && Y < S.y1) ssum += sv;
            const double pd[3] = {in ? 2.0 * my * (a2 - a1) * rb + 2.0 * mx * sv * (r2 - r1) : 0.0,
                                  in ? -sv * r2 : 0.0, in ? 2.0 * a1 * rb : 0.0};
            PHASE();
#pragma unroll
            for (int i = 0; i < WN; ++i) ys[i] = s.y[buf][lane + i];
            PHASE();
            // 3. into output rows Y - R .. Y + R: row Y - R + d in slot (pm + d) mod 11 with tap
            // 10 - d; d = 0 is complete, d = 10 starts.  (Rows above the segment's first: incomplete
            // sums, whose outputs are never emitted.)
#pragma unroll
            for (int d = 0; d < WN; ++d) {
                double(&w)[3] = u[(pm + d) % WN];
#pragma unroll
                for (int q = 0; q < 3; ++q)
                    w[q] = d == WN - 1 ? a.g[0] * pd[q] : fma(a.g[WN - 1 - d], pd[q], w[q]);
            }
            lds_order();
#pragma unroll
            for (int q = 0; q < 3; ++q) s.u[q][lane + R] = u[pm][q];
            PHASE();
            // 1. horizontal sums of row r, the taps of equal weight together
            double h[4];
            {
                const double xc = xs[R], yc = ys[R], gc = a.g[R];
                h[0] = gc * xc;
                h[1] = gc * yc;
                h[2] = gc * fma(xc, xc, yc * yc);
                h[3] = gc * (xc * yc);
            }
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const double xa = xs[i], xb = xs[2 * R - i], ya = ys[i], yb = ys[2 * R - i];
                const double gi = a.g[i];
                h[0] = fma(gi, xa + xb, h[0]);
                h[1] = fma(gi, ya + yb, h[1]);
                h[2] = fma(gi, fma(xa, xa, fma(ya, ya, fma(xb, xb, yb * yb))), h[2]);
                h[3] = fma(gi, fma(xa, ya, xb * yb), h[3]);
            }
            // the next input row to LDS, and the one after next on its way
            buf ^= 1;
            stage(buf, nx);
            nx = fetch(r + 2);
            PHASE();
            // 2. into map rows r - R .. r + R, slots from p
#pragma unroll
            for (int d = 0; d < WN; ++d) {
                double(&w)[4] = v[(p + d) % WN];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    w[q] = d == WN - 1 ? a.g[0] * h[q] : fma(a.g[WN - 1 - d], h[q], w[q]);
            }
            PHASE();
            // 3. output row o
            const Out cur = no;
            no = fetch_out(o + 1);
            if (o < S.y0 || o >= S.y1) return;
            lds_order();
            double g3[3];
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                g3[q] = a.g[R] * s.u[q][lane + R];
#pragma unroll
                for (int i = 0; i < R; ++i)
                    g3[q] = fma(a.g[i], s.u[q][lane + i] + s.u[q][lane + 2 * R - i], g3[q]);
            }
            if (own) {
                const double gq =
                    a.grad_scale * (g3[0] + 2.0 * (double)cur.x * g3[1] + (double)cur.y * g3[2]);
                (S.dl + (int64_t)o * S.nx)[X] = cur.d + (float)gq;
            }
        };
#pragma unroll 1
        while (r < r_end) cycle(row, r, std::make_integer_sequence<int, WN>{});
    }
    for (int o = 32; o > 0; o >>= 1) ssum += __shfl_xor(ssum, o, 64);
    if (lane == 0 && first < nw) part[first] = ssum;
}

__global__ __launch_bounds__(256) void k_ssim_finish(const double* part, int nb, double inv_n,
                                                     float* loss)
{
    __shared__ double sh[256];
    double v = 0.0;
    for (int i = threadIdx.x; i < nb; i += 256) v += part[i];
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *loss = inv_n > 0.0 ? (float)(1.0 - sh[0] * inv_n) : 0.0f;
}

// Which form a launch takes, and how its strips are cut, by what each is measured to take (us, the
// loss's sum included).  A wavefront of a strip walks its rows in whole cycles of 11 rows, 20 rows on
// top of the segment's own and one to finish.  Per cycle, with wavefronts for at most 1, 2, 3 or 4
// times the chip's SIMDs:
//     wavefronts     up to 1024   2048   3072   4096   6144
//     us a cycle     9 - 12       15     20     28     41
// A lone wavefront's rows are one dependent chain, so that a second on its SIMD adds half of its time
// and a short segment still costs three cycles.  The tiles of ssim_tiles.hip take 14, 24.5, 35, 53, 87,
// 163 and 330 us for up to 1, 2, 3, 5, 9, 18 and 38 times 256 tiles.  So the tiles are faster where
// they are few, or where the strips' 54 columns are badly filled.  Three stacks of square slices, us in
// tiles and in strips (the rule takes the smaller but for 72 of 128 x 128, 53.6):
//     slices      18        36        72       144       288       576
//     33 x 33               14 28     25 28    36 28     54 30     88 44
//     54 x 54     14 27     14 28     25 28    35 29     54 38     88 57
//     55 x 55     14 27     14 28     25 29    36 39     54 57     88 100
//     64 x 64     14 27     14 28     25 29    35 39     54 57     87 93
//     80 x 80     14 27     24 28     34 30    61 46     102 71    185 120
//     128 x 128   24 28     35 39     54 50    88 76     163 121
//     256 x 256   54 46     88 75     163 106
double strip_us(int64_t wavefronts, int64_t rows)
{
    const int64_t n = (wavefronts + SIMDS - 1) / SIMDS;
    const double cycle = n <= 1 ? 8.9 + 2.3 / SIMDS * (double)wavefronts
                                : 14.8 * (double)(n / 2) + 6.3 * (double)(n % 2);
    return cycle * (double)((rows + 4 * R + 1 + WN - 1) / WN);
}
double tiles_us(int64_t tiles)
{
    const double n = (double)((tiles + 255) / 256), few = 4.0 + 10.2 * n, many = 9.0 + 8.8 * n;
    return few < many ? few : many;
}

struct Plan {
    int rows;          // of a strip's segment; 0: tiles
    double us;
};

Plan plan(const SsimArgs& a, const int32_t* nz)
{
    int64_t tiles = 0;
    int most = 1;
    for (int k = 0; k < a.n_stacks; ++k) {
        most = a.ny[k] > most ? a.ny[k] : most;
        tiles += (int64_t)nz[k] * ((a.nx[k] + SSIM_TILE - 1) / SSIM_TILE) *
                 ((a.ny[k] + SSIM_TILE - 1) / SSIM_TILE);
    }
    Plan best = {0, tiles_us(tiles)};
    for (int segs = 1; segs <= 64; ++segs) {
        const int rows = (most + segs - 1) / segs;
        int64_t items = 0;
        for (int k = 0; k < a.n_stacks; ++k)
            items += (int64_t)nz[k] * ((a.nx[k] + OUT_X - 1) / OUT_X) * ((a.ny[k] + rows - 1) / rows);
        const double us = strip_us(items, rows);
        if (us < best.us) best = {rows, us};
        if (rows <= 4) break;
    }
    return best;
}

}  // namespace

hipError_t launch_ssim(SsimArgs& a, const int32_t* nz, int64_t n_voxels, float* loss, void* ws,
                       hipStream_t s)
{
    double* part = reinterpret_cast<double*>(ws);
    const int rows = plan(a, nz).rows;
    const int w = rows ? OUT_X : SSIM_TILE, h = rows ? rows : SSIM_TILE;
    int64_t total = 0;
    for (int k = 0; k < a.n_stacks; ++k) {
        a.rows[k] = h;
        a.tiles_x[k] = (a.nx[k] + w - 1) / w;
        a.tiles_y[k] = (a.ny[k] + h - 1) / h;
        a.tile_begin[k] = total;
        total += (int64_t)nz[k] * a.tiles_x[k] * a.tiles_y[k];
    }
    a.tile_begin[a.n_stacks] = total;
    int nb = (int)(total < SLOTS ? total : SLOTS);
    if (!rows)
        nb = launch_ssim_tiles(a, part, s);
    else if (nb > 0) {
        const dim3 grid((unsigned)((nb + WPB - 1) / WPB)), block(64 * WPB);
        if (nb <= SIMDS)
            hipLaunchKernelGGL(k_ssim<true>, grid, block, 0, s, a, part, nb);
        else
            hipLaunchKernelGGL(k_ssim<false>, grid, block, 0, s, a, part, nb);
    }
    hipLaunchKernelGGL(k_ssim_finish, dim3(1), dim3(256), 0, s, part, nb,
                       n_voxels > 0 ? 1.0 / (double)n_voxels : 0.0, loss);
    return hipGetLastError();
}
