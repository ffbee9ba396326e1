// K11: neural residual field (Sec. 3.4, Eq. 8) on MFMA: BF16 weights and activations,
// FP32 accumulation.
//
// r(x) = out_scale tanh(w_out . a_D + b_out),  a_l = SiLU(W_l a_{l-1} + b_l),
// a_0 = gamma(x) = (x, sin(2^k pi x), cos(2^k pi x), k < n_freq), zero-padded to in_pad.
//
// Layout trick: each layer is computed transposed, Z^T = W X^T, with gfx950's 16x16x32 BF16
// MFMA (A = 16 output features x 32 input features of W, B = 32 input features x 16 points).
// The result holds, per lane, 4 consecutive output features of one point; two such tiles are
// exactly the B operand of one 32-wide K step of the next layer (the weights are staged with
// the same K order), so activations never leave registers inside a layer stack.  The encoding
// is computed directly in that layout.
//
// Backward (for lists of sampled voxels): recompute, then per layer dZ_l = dA_l * SiLU'(Z_l),
// dW_l += dZ_l A_{l-1}^T over the points, dA_{l-1} = W_l^T dZ_l, all in one kernel.  The forward
// alone (k_nrf_forward) is in nrf_fwd.hip.
#include "nrf_core.h"

namespace {

using namespace nrfcore;

constexpr int FULL = 512;            // two blocks on each of 256 CUs, all resident at once
// A block's FP32 sums run over all its rounds, and their error grows with that: from 1M points on the
// launch takes FULL blocks more for every CUT rounds of one, up to MAX_BLOCKS (1.1 GB of partials).
// Every voxel of 256^3 in one call, against the sum of small calls: off by 2.8e-7 of the largest
// first-layer weight gradient, 1.4e-6 with 512 rounds a block, in the same 2.95 ms (3.21 ms with 16
// rounds a block, no closer).
constexpr int CUT = 32, MAX_BLOCKS = 32 * FULL;

// Floats of one block's partial gradients: dW of the first layer in the GPU's K order [W][16 KT],
// the hidden layers' [depth - 1][W][W], the biases [depth][W], w_out [W], b_out
__host__ __device__ constexpr int part_floats(int in_pad, int depth)
{
    return W * in_pad + (depth - 1) * W * W + depth * W + W + 1;
}

typedef __attribute__((address_space(3))) v4s* LdsQuad;

// gfx950's transposing LDS read: within each 16 lanes, source lane 4 j + c (its own address)
// gives element d to lane 4 c + d as that lane's element j
__device__ __forceinline__ v4s read_tr(const v4s* p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsQuad)(p));
}

template <int KT, int DEPTH>
struct GradLds {
    Lds<KT, DEPTH> w;
    v4f bias[DEPTH][16];           // [l][4 o + g]
    v4s w_out[16];                 // [4 o + g]
    // the round's four tiles [t][tile][quad], a lane's quad (point row, features 4 g ..) at
    // swizzle(lane)
    v4s enc[KT * 4 * 64];
    v4s act[DEPTH > 1 ? DEPTH - 1 : 1][4 * 4 * 64];
    v4s dz[4 * 4 * 64];            // of one layer at a time
    float out[4][W + 1];           // the output layer's sums, per wavefront
};

// Where the quad of lane 16 g + row is stored: rows of the upper two lane groups with row bit 2
// flipped, so that both the quads of one g (the writes) and the four g of four rows (the transposing
// reads) lie in 16 different bank pairs.
__device__ __forceinline__ int swizzle(int lane) { return lane ^ ((lane >> 3) & 4); }

// The lane whose quad lane 16 G + 4 j + c reads for read_tr to give it rows 4 G .. 4 G + 3 of feature
// 4 j + c: row 4 G + j of lane group c
__device__ __forceinline__ int source_lane(int lane)
{
    return (lane & 3) * 16 + (lane >> 4) * 4 + ((lane >> 2) & 3);
}

template <int KT, int DEPTH>
struct GradWeights {
    const GradLds<KT, DEPTH>& s;
    int lane;
    int wslot, wslot_tr;           // where the lane's piece of a hidden layer lies, and the one it
                                   // reads for read_tr
    __device__ v4f bias(const NrfArgs&, int l, int o) const { return s.bias[l][4 * o + (lane >> 4)]; }
    __device__ v8h in(int o, int u) const { return s.w.w_in[(o * (KT / 2) + u) * 64 + lane]; }
    __device__ v8h hid(int l, int o, int u) const
    {
        return s.w.w_hid[((l - 1) * 8 + o * 2 + u) * 64 + wslot];
    }
    // W_l^T as A operand (i-tile of inputs, o-tile of outputs): lane (g, row) gets
    // W_l[16 o + 4 g + j][16 i + row], from the quads of W_l's operand (o, i)
    __device__ v4s hid_t(int l, int i, int o) const
    {
        return read_tr(reinterpret_cast<const v4s*>(
                           &s.w.w_hid[((l - 1) * 8 + o * 2 + (i >> 1)) * 64 + wslot_tr]) + (i & 1));
    }
};

// A lane's point of a round: its grid (uniform), voxel and dL/dr there
struct Point {
    int k;
    bool valid;
    uint32_t v;
    float dl;
};

// A block takes rounds of 64 points, a tile of 16 to each wavefront, which runs the tile's forward
// and backward in registers.  For the weight gradients the K dimension is the points, so each
// layer's dZ and input go through LDS once: written as the quads (4 features of a point) that
// the lanes hold, read back transposed (4 points of a feature) as MFMA operands over all four
// tiles.  The output tiles of dW_l are dealt to the wavefronts as 2 x 2 (half the rows, half the
// columns), each wavefront's FP32 accumulators staying in registers over all its rounds; row
// sums (the bias gradients) are one more product, with ones.  W_l^T is read from the staged W_l,
// also transposed.  Every block leaves one partial of every gradient.
//
// Bound by vector issue: per tile some 1000 instructions, most of them the encoding, SiLU and
// SiLU'.  3 x 262144 points, 16 bands, depth 3: 162 us for all three grids in one launch and 10
// for the partials' sums (the biases read from global memory, each read a wait in the middle of
// a layer: 261).  With dZ and the activations written out in BF16 (700 MB, two bytes
// a lane at a time), a GEMM pass over them per layer and a chain launch per grid, the chain took
// 375, the GEMMs 220 and the partials' sums 80.
template <int KT, int DEPTH>
__global__ __launch_bounds__(256, DEPTH < 4 ? 2 : 1) void k_nrf_grad(const NrfArgs a, const NrfGrids gs,
                                                     float* __restrict__ part)
{
    __shared__ GradLds<KT, DEPTH> s;
    constexpr int CT = KT / 2;      // column tiles of dW_0 per wavefront
    const int lane = threadIdx.x & 63, g = lane >> 4, row = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wv >> 1, wc = wv & 1;
    if (threadIdx.x < 16) s.w_out[threadIdx.x] = reinterpret_cast<const v4s*>(a.w_out)[threadIdx.x];
    if (threadIdx.x < 16 * DEPTH) {
        const int l = threadIdx.x >> 4, q = threadIdx.x & 15;
        const float* b = (l == 0 ? a.b_in : a.b_hid + (l - 1) * W) + 4 * q;
        s.bias[l][q] = v4f{b[0], b[1], b[2], b[3]};
    }
    load_weights<KT, DEPTH, true>(a, s.w);
    const int lane_tr = source_lane(lane);
    const GradWeights<KT, DEPTH> ws{s, lane, lane ^ 4 * (lane >> 4), lane_tr ^ 4 * (lane_tr >> 4)};
    const int slot_tr = swizzle(lane_tr);
    // dW accumulators.  Row tile i of the wavefront is 2 wr + (i ^ wc), so that i = 0 is the one
    // whose row sums it takes.
    v4f acc0[2][CT], acch[DEPTH > 1 ? DEPTH - 1 : 1][2][2], accb[DEPTH];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int t = 0; t < CT; ++t) acc0[i][t] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int l = 0; l < DEPTH - 1; ++l)
            acch[l][i][0] = acch[l][i][1] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    }
#pragma unroll
    for (int l = 0; l < DEPTH; ++l) accb[l] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    // the output layer's gradient over this wavefront's points: gwo[4 o + j] for feature
    // 16 o + 4 g + j (sum of dzo a_D), gbo the sum of dzo (lanes of group 0; of terms of either sign,
    // it cancels the most)
    float gwo[16];
    double gbo = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) gwo[i] = 0.0f;

    const int64_t rounds = gs.round0[gs.n];
    auto point = [&](int64_t r, int k) {   // round r's voxel (grid k or a later one)
        Point p{k, false, 0u, 0.0f};
        if (r >= rounds) return p;
        while (r >= gs.round0[p.k + 1]) ++p.k;
        const int64_t i = (r - gs.round0[p.k]) * NRF_ROUND + 16 * wv + row;
        p.valid = i < gs.g[p.k].n_points;
        const int32_t* idx = gs.g[p.k].idx;
        if (p.valid) p.v = idx ? (uint32_t)idx[i] : (uint32_t)i;
        return p;
    };
    auto fetch_dl = [&](Point& p) { if (p.valid) p.dl = gs.g[p.k].dl_dr[p.v]; };
    Point cur, nxt = point(blockIdx.x, 0), far = point((int64_t)blockIdx.x + gridDim.x, nxt.k);
    fetch_dl(nxt);
#pragma unroll 1
    for (int64_t r = blockIdx.x; r < rounds; r += gridDim.x) {
        // voxels are read two rounds ahead and dL/dr one
        cur = nxt;
        nxt = far;
        fetch_dl(nxt);
        far = point(r + 2 * (int64_t)gridDim.x, far.k);
        const double* m = gs.g[cur.k].m;
        int vx = 0, vy = 0, vz = 0;
        if (cur.valid)
            voxel_xyz(cur.v, (uint32_t)gs.g[cur.k].nx, (uint32_t)gs.g[cur.k].ny, &vx, &vy, &vz);
        const float x[3] = {world_coord(m, vx, vy, vz), world_coord(m + 4, vx, vy, vz),
                            world_coord(m + 8, vx, vy, vz)};
        Tile<KT, DEPTH> T;
        tile_forward_w<KT, DEPTH>(a, ws, x, T);
        __syncthreads();            // the last round's products are done
        const int slot = wv * 64 + swizzle(lane);
#pragma unroll
        for (int t = 0; t < KT; ++t) s.enc[t * 256 + slot] = T.enc[t];
#pragma unroll
        for (int l = 0; l < DEPTH - 1; ++l)
#pragma unroll
            for (int t = 0; t < 4; ++t) s.act[l][t * 256 + slot] = T.act[l][t];
        v4s wo[4];                  // w_out as load_wout's operand
#pragma unroll
        for (int o = 0; o < 4; ++o) wo[o] = (row & 3) == 0 ? s.w_out[4 * o + g] : v4s{0, 0, 0, 0};
        const float zo = tile_output<KT, DEPTH>(a, T, wo);
        const float th = tanhf(zo);
        const float dzo = cur.valid ? cur.dl * gs.g[cur.k].scale * a.out_scale * (1.0f - th * th)
                                    : 0.0f;
        // dA_D = dzo w_out, then back through the layers
        v4f da[4];
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            const v4s h = T.act[DEPTH - 1][o], q = s.w_out[4 * o + g];
            gwo[4 * o + 0] += dzo * from_bf16((uint16_t)h.x);
            gwo[4 * o + 1] += dzo * from_bf16((uint16_t)h.y);
            gwo[4 * o + 2] += dzo * from_bf16((uint16_t)h.z);
            gwo[4 * o + 3] += dzo * from_bf16((uint16_t)h.w);
            da[o] = v4f{dzo * from_bf16((uint16_t)q.x), dzo * from_bf16((uint16_t)q.y),
                        dzo * from_bf16((uint16_t)q.z), dzo * from_bf16((uint16_t)q.w)};
        }
        if (g == 0) gbo += dzo;
#pragma unroll
        for (int l = DEPTH - 1; l >= 0; --l) {
            v4s dz[4];
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                const v4f d = T.d[l][o];
                dz[o] = pack4(da[o].x * d.x, da[o].y * d.y, da[o].z * d.z, da[o].w * d.w);
            }
            if (l < DEPTH - 1) __syncthreads();   // the products of the layer above are done
#pragma unroll
            for (int o = 0; o < 4; ++o) s.dz[o * 256 + slot] = dz[o];
            __syncthreads();
            if (l > 0) {
                // dA_{l-1} = W_l^T dZ_l
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int o = 0; o < 4; o += 2)
                        acc = mfma2(ws.hid_t(l, i, o), ws.hid_t(l, i, o + 1), dz[o], dz[o + 1], acc);
                    da[i] = acc;
                }
            }
            // dW_l += dZ_l A_{l-1}^T over the round's points, 32 at a time
            const v4s* in = l == 0 ? s.enc : s.act[l > 0 ? l - 1 : 0];
            const v4s ones = {0x3f80, 0x3f80, 0x3f80, 0x3f80};
#pragma unroll
            for (int st = 0; st < 4; st += 2) {
                v4s z[2][2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const v4s* q = &s.dz[((2 * wr + (i ^ wc)) * 4 + st) * 64 + slot_tr];
                    z[i][0] = read_tr(q);
                    z[i][1] = read_tr(q + 64);
                }
                accb[l] = mfma2(z[0][0], z[0][1], ones, ones, accb[l]);
#pragma unroll
                for (int t = 0; t < (l == 0 ? CT : 2); ++t) {
                    const v4s* q = &in[((wc * (l == 0 ? CT : 2) + t) * 4 + st) * 64 + slot_tr];
                    const v4s b0 = read_tr(q), b1 = read_tr(q + 64);
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        v4f& c = l == 0 ? acc0[i][t] : acch[l > 0 ? l - 1 : 0][i][t & 1];
                        c = mfma2(z[i][0], z[i][1], b0, b1, c);
                    }
                }
            }
        }
    }
    // acc holds rows 4 g + j of its row tile, column lane & 15 of its column tile
    constexpr int N = 16 * KT;
    float* out = part + (int64_t)blockIdx.x * part_floats(N, DEPTH);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m0 = 16 * (2 * wr + (i ^ wc)) + 4 * g;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
#pragma unroll
            for (int t = 0; t < CT; ++t) out[(m0 + j) * N + 16 * (wc * CT + t) + row] = acc0[i][t][j];
#pragma unroll
            for (int l = 0; l < DEPTH - 1; ++l)
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    out[W * N + (l * W + m0 + j) * W + 16 * (wc * 2 + t) + row] = acch[l][i][t][j];
        }
    }
    out += W * N + (DEPTH - 1) * W * W;
    if (row == 0) {
#pragma unroll
        for (int l = 0; l < DEPTH; ++l)
#pragma unroll
            for (int j = 0; j < 4; ++j) out[l * W + 16 * (2 * wr + wc) + 4 * g + j] = accb[l][j];
    }
    out += DEPTH * W;
    // the output layer: sum over the 16 points of each lane group, then over the wavefronts
#pragma unroll
    for (int i = 0; i < 16; ++i)
        for (int o = 1; o < 16; o <<= 1) gwo[i] += __shfl_xor(gwo[i], o, 64);
    for (int o = 1; o < 16; o <<= 1) gbo += __shfl_xor(gbo, o, 64);
    if (row == 0) {
#pragma unroll
        for (int o = 0; o < 4; ++o)
#pragma unroll
            for (int j = 0; j < 4; ++j) s.out[wv][16 * o + 4 * g + j] = gwo[4 * o + j];
        if (g == 0) s.out[wv][W] = (float)gbo;
    }
    __syncthreads();
    if (threadIdx.x <= W)
        out[threadIdx.x] = (s.out[0][threadIdx.x] + s.out[1][threadIdx.x]) +
                           (s.out[2][threadIdx.x] + s.out[3][threadIdx.x]);
}

// Every gradient += the sum of its nb partials, in a fixed order: 64 elements per block, whose
// SUM_WAVES wavefronts share the partials (partial c to wavefront c mod SUM_WAVES), each with
// four independent accumulators so that its loads are in flight together, then the wavefronts'
// sums are added in order.  In binary64, which takes no longer here: with the blocks' b_out sums,
// 262144 points' gradients are 2.0e-7 from the exact sums in place of 5.4e-7.  The first layer's weights go from the GPU's K order to the natural
// one (padding slots are dropped).
constexpr int SUM_WAVES = 16;
constexpr int SUM_THREADS = 64 * SUM_WAVES;

template <int KT, int DEPTH>
__global__ __launch_bounds__(SUM_THREADS) void k_nrf_sums(const NrfArgs a,
                                                          const float* __restrict__ part, int nb)
{
    constexpr int N = 16 * KT, n = part_floats(N, DEPTH);
    __shared__ double sh[SUM_WAVES][64];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    int e = blockIdx.x * 64 + l;
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    if (e < n) {
        const float* p = part + e;
        int c = w;
        for (; c + 3 * SUM_WAVES < nb; c += 4 * SUM_WAVES) {
            a0 += p[(int64_t)c * n];
            a1 += p[(int64_t)(c + SUM_WAVES) * n];
            a2 += p[(int64_t)(c + 2 * SUM_WAVES) * n];
            a3 += p[(int64_t)(c + 3 * SUM_WAVES) * n];
        }
        for (; c < nb; c += SUM_WAVES) a0 += p[(int64_t)c * n];
    }
    sh[w][l] = (a0 + a1) + (a2 + a3);
    __syncthreads();
    if (threadIdx.x >= 64 || e >= n) return;
    double all = 0.0;
#pragma unroll
    for (int i = 0; i < SUM_WAVES; ++i) all += sh[i][l];
    const float sum = (float)all;
    if (e < W * N) {
        const int nf = natural_feature<KT>(e % N, a.n_freq);
        if (nf >= 0) a.g_w_in[e / N * N + nf] += sum;
        return;
    }
    e -= W * N;
    if (e < (DEPTH - 1) * W * W) {
        a.g_w_hid[e] += sum;
        return;
    }
    e -= (DEPTH - 1) * W * W;
    if (e < W)
        a.g_b_in[e] += sum;
    else if (e < DEPTH * W)
        a.g_b_hid[e - W] += sum;
    else if (e < DEPTH * W + W)
        a.g_w_out[e - DEPTH * W] += sum;
    else
        a.g_b_out[0] += sum;
}

__global__ __launch_bounds__(256) void k_to_bf16(const float* __restrict__ in,
                                                 uint16_t* __restrict__ out, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        out[i] = to_bf16(in[i]);
}

int grad_blocks(int64_t rounds)
{
    if (rounds < FULL) return (int)rounds;
    const int64_t nb = (rounds + FULL * CUT - 1) / (FULL * CUT) * FULL;
    return (int)(nb < MAX_BLOCKS ? nb : MAX_BLOCKS);
}

template <int KT, int DEPTH>
void launch_grad_t(const NrfArgs& a, const NrfGrids& gs, float* part, hipStream_t s)
{
    const int nb = grad_blocks(gs.round0[gs.n]);
    hipLaunchKernelGGL((k_nrf_grad<KT, DEPTH>), dim3((unsigned)nb), dim3(256), 0, s, a, gs, part);
    hipLaunchKernelGGL((k_nrf_sums<KT, DEPTH>),
                       dim3((unsigned)((part_floats(16 * KT, DEPTH) + 63) / 64)), dim3(SUM_THREADS), 0,
                       s, a, part, nb);
}

}  // namespace

int nrf_max_bands(int in_pad) { return in_pad == 64 ? max_bands<4>() : max_bands<8>(); }

size_t nrf_part_floats(int64_t rounds, int in_pad, int depth)
{
    const int nb = grad_blocks(rounds);
    return (size_t)(nb > 0 ? nb : 1) * part_floats(in_pad, depth);
}

hipError_t launch_nrf_backward(const NrfArgs& a, const NrfGrids& gs, float* part, hipStream_t s)
{
    if (gs.round0[gs.n] <= 0) return hipSuccess;
    GM_NRF_DISPATCH(launch_grad_t, a, gs, part, s)
    return hipGetLastError();
}

hipError_t launch_to_bf16(const float* in, uint16_t* out, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    int64_t b = (n + 255) / 256;
    if (b > 4096) b = 4096;
    hipLaunchKernelGGL(k_to_bf16, dim3((unsigned)b), dim3(256), 0, s, in, out, n);
    return hipGetLastError();
}
