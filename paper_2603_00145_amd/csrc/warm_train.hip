// K12 training: the warm-start network's forward and the gradients of its weights (layers in
// warm.hip): two kernels over the samples for layers 1-2 and 3-4 with the loss head between the
// passes of the second, one for the backward of layers 1-2, and one that adds their blocks'
// partial sums.
//
// All products run on gfx950's 16x16x32 BF16 MFMA with FP32 accumulation.
//   - Every quantity that is rounded to BF16 (the activations and the gradients through the
//     pre-activations) is summed over K = (channel, tap) in that order, 32 at a time, however
//     the operands lie, so that the roundings do not depend on this file's layouts.  (Inference
//     sums tap by tap, see warm_fwd.hip: there a rounding that falls the other way is one of
//     thousands in an output; a weight gradient would show it in its fifth digit.)  The operand
//     of such a product is gathered element by element from LDS at precomputed offsets.
//   - A weight gradient, dW = dZ^T X, sums over positions, in FP32 to the end, so its order is
//     free: a lane's half operand is four output positions along x, which a stride-2 window reads
//     at every other x.  The inputs lie in LDS as groups of four such values, one group per
//     x tap, and dZ comes from its product as four positions of a channel per lane (positions on
//     the rows), the operand as it is.
// Each block keeps its weight-gradient sums in registers over all its samples and writes them
// once.  A batch of 1024 gives each of 256 blocks four samples; the kernels are bound by the
// latency of their phases (one wavefront per SIMD), not by throughput (20 GFLOP a step): 49, 50, 86
// and 17 us, the whole training step 205 us.  One kernel per layer and direction, each storing its
// activations and gathering operands from memory or per output channel tile, took 960 us of a
// 1118 us step; the same kernels as here with every K step one tap (one 16-byte read per operand)
// 206 us, but their gradients differ by 1.5e-4 through roundings that fall the other way.
#include "warm_core.h"

namespace {

using namespace warmcore;

constexpr int WT = WS_WT;                 // a 32x32x27 layer's weights or gradient, elements
constexpr int MAX_BLOCKS = 256;

// a block's sums of the last two layers and the head, in floats
constexpr int P34_W3 = 0, P34_W4 = WT, P34_WL = P34_W4 + CO * KP4, P34_B4 = P34_WL + 8 * CO,
              P34_B3 = P34_B4 + CO, P34_B2 = P34_B3 + CO, P34_BL = P34_B2 + CO,
              P34 = P34_BL + 8;
// ... and of the first two: dW2, dW1 as [channel tile 2][column tile 6][lane][4], db1
constexpr int N1 = 6;                     // column tiles of the first layer's 81 (c, tap), padded
constexpr int P12_W2 = 0, P12_W1 = WT, P12_B1 = P12_W1 + 2 * N1 * 64 * 4, P12 = P12_B1 + CO;
static_assert(P34 % 4 == 0 && P12 % 4 == 0, "partials move as float4");

// sum over the four lane groups of a wavefront (every lane ends with its column's)
__device__ __forceinline__ float group_sum4(float v)
{
    v += __shfl_xor(v, 16, 64);
    return v + __shfl_xor(v, 32, 64);
}
__device__ __forceinline__ float sum_bf16(v4s v)
{
    return (from_bf16((uint16_t)v.x) + from_bf16((uint16_t)v.y)) +
           (from_bf16((uint16_t)v.z) + from_bf16((uint16_t)v.w));
}

// First K step of parity class c (bits z, y, x) of the second layer's input positions: class c
// has 2^popcount(c) taps, 32 output channels each, taps fastest
__host__ __device__ constexpr int class_steps(int c)
{
    int n = 0;
    for (int d = 0; d < c; ++d) n += 1 << ((d & 1) + (d >> 1 & 1) + (d >> 2));
    return n;
}

// Element i of [K step][channel tile][lane][8] of the backward's weight operands (row or column =
// input channel): layer 2 in the classes' K order, then layer 3 in the order (output channel, tap)
constexpr int PACK_BLOCKS = 2 * WT / 8 / 256;
static_assert(PACK_BLOCKS * 256 * 8 == 2 * WT, "whole blocks of packed operands");

__device__ void pack_weights(const WsNet& net, uint16_t* wt, int e)
{
    const int layer = e / (WT / 8), r = e % (WT / 8);
    const int lane = r & 63, ct = r >> 6 & 1, st = r >> 7;
    const uint16_t* W = net.w[1 + layer] + (16 * ct + (lane & 15)) * 27;
    int c = 0;
    while (layer == 0 && c < 7 && class_steps(c + 1) <= st) ++c;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int k = 32 * (layer == 0 ? st - class_steps(c) : st) + 16 * (i >> 2) + 4 * (lane >> 4) +
                      (i & 3);
        int o, tap;
        if (layer == 1) {
            o = k / 27;
            tap = k % 27;
        } else {
            const int nc = 1 << ((c & 1) + (c >> 1 & 1) + (c >> 2));
            int bits = k % nc;
            o = k / nc;
            tap = 0;
            const int wt3[3] = {1, 3, 9};
            for (int ax = 0; ax < 3; ++ax) {
                int kk = 1;
                if (c >> ax & 1) {
                    kk = bits & 1 ? 2 : 0;
                    bits >>= 1;
                }
                tap += kk * wt3[ax];
            }
        }
        wt[e * 8 + i] = W[o * KP2 + tap];
    }
}

// ---- forward of layers 1 and 2: one sample at a time ----------------------------------------
// The second layer's input in LDS: position (z, y, x), each >= -1, at 40 elements per x with even
// and odd x apart (neighbouring outputs of the stride-2 window read neighbouring slots).
constexpr int A_POS = 40, A_ROW = 46 * 8, A_Z = 9 * A_ROW;
__device__ __forceinline__ constexpr int a_x(int x) { return (x & 1) ? 5 + (x >> 1) : x >> 1; }

struct LdsF12 {
    alignas(16) uint16_t in[PATCH];
    alignas(16) uint16_t a1[9 * A_Z];
    alignas(16) uint16_t off[27 * 4 * 8];   // [K step][lane group][element]: offset in a1
};

__global__ __launch_bounds__(256, 1) void k_ws_train12(const WsNet net, const uint16_t* __restrict__ X,
                                                       int64_t B, const WsWork w)
{
    __shared__ LdsF12 s;
    const int nb = (int)gridDim.x - PACK_BLOCKS;
    if ((int)blockIdx.x >= nb) {
        pack_weights(net, w.wt, ((int)blockIdx.x - nb) * 256 + (int)threadIdx.x);
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, wv = sgpr(tid >> 6), g = lane >> 4, col = lane & 15;
    Natural1 l1;
    l1.load(net.w[0], lane);
    v4s w2[27][2][2];                       // [K step][channel tile][half]
#pragma unroll
    for (int st = 0; st < 27; ++st)
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                w2[st][m][h] = *reinterpret_cast<const v4s*>(net.w[1] + (16 * m + col) * KP2 + 32 * st +
                                                             16 * h + 4 * g);
    for (int i = tid; i < PATCH; i += 256) s.in[i] = 0;
    for (int i = tid; i < 9 * A_Z; i += 256) s.a1[i] = 0;
    for (int i = tid; i < 27 * 32; i += 256) {
        const int k = natural_k(i), c = k / 27, t = k % 27;
        s.off[i] = (uint16_t)((t / 9) * A_Z + (t / 3 % 3) * A_ROW + a_x(t % 3) * A_POS + c);
    }
    __syncthreads();    // a patch's rows are staged by other wavefronts than the ones that clear them
    float bias1[2][4], bias2[2][4];
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            bias1[m][j] = net.b[0][16 * m + 4 * g + j];
            bias2[m][j] = net.b[1][16 * m + 4 * g + j];
        }
    const bool stager = tid < 192;
    uint4 nx = make_uint4(0u, 0u, 0u, 0u);
    if (stager && blockIdx.x < B) nx = reinterpret_cast<const uint4*>(X + (int64_t)blockIdx.x * 1536)[tid];
    const int x1 = col & 7, y1 = col >> 3;
    uint16_t* out1 = s.a1 + A_Z + (y1 + 1) * A_ROW + a_x(x1 + 1) * A_POS + 4 * g;
    // second layer: wavefront = output plane, the lane's (y, x) of it
    const uint16_t* in2 = s.a1 + 2 * wv * A_Z + 2 * (col >> 2) * A_ROW + (col & 3) * A_POS;
#pragma unroll 1
    for (int64_t b = blockIdx.x; b < B; b += nb) {
        if (stager) stage_patch(s.in, tid, nx);
        __syncthreads();
        if (stager && b + nb < B)
            nx = reinterpret_cast<const uint4*>(X + (b + nb) * 1536)[tid];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int z = 2 * wv + (i >> 2), y = 2 * (i & 3);
            v4f c[2] = {};
            v8s xv[3];
            l1.patch(s.in + (z * 10 + y + y1) * 12 + x1, xv);
#pragma unroll
            for (int st = 0; st < 3; ++st)
#pragma unroll
                for (int m = 0; m < 2; ++m) c[m] = mfma8(l1.w[m][st], xv[st], c[m]);
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const v4f zz = v4f{c[m].x + bias1[m][0], c[m].y + bias1[m][1], c[m].z + bias1[m][2],
                                   c[m].w + bias1[m][3]};
                *reinterpret_cast<v4s*>(out1 + z * A_Z + y * A_ROW + 16 * m) = silu4(zz);
            }
        }
        __syncthreads();
        v4f c[2] = {};
#pragma unroll
        for (int st = 0; st < 27; ++st) {
            const v8s xv = gather8(in2, s.off + (st * 4 + g) * 8);
#pragma unroll
            for (int m = 0; m < 2; ++m) c[m] = mfma8(join(w2[st][m][0], w2[st][m][1]), xv, c[m]);
        }
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int64_t o = ((b * 4 + wv) * 16 + col) * CO + 16 * m + 4 * g;
            const v4f zz = v4f{c[m].x + bias2[m][0], c[m].y + bias2[m][1], c[m].z + bias2[m][2],
                               c[m].w + bias2[m][3]};
            *reinterpret_cast<v4s*>(w.a2 + o) = silu4(zz);
            *reinterpret_cast<v4f*>(w.z2 + o) = zz;
        }
    }
}

// ---- layers 3 and 4 forward, the loss head, and their backward: four samples at a time ------
constexpr int P3 = 125 * CO;              // a sample's second-layer activations, positions >= -1
constexpr int D3 = 6 * 6 * 6;             // dZ3 of a channel with a zero between its outputs

struct Lds34 {
    alignas(16) uint16_t a2[4 * P3 + 4 * 16];  // [sample][z + 1][y + 1][x + 1][channel], 32 bytes apart
    alignas(16) uint16_t dil[4 * CO * D3];     // [sample][channel][t + 1]^3, output o at t = 2 o
    alignas(16) uint16_t off3[27 * 4 * 8];     // K order (channel, tap): offsets in a2
    alignas(16) int16_t offd[27 * 4 * 8];      // K order (output channel, tap): offsets in dil
    alignas(16) float z3[4][8][CO];
    alignas(16) float z4[4][CO];
    alignas(16) uint16_t a3[4 * CO * 8];       // [sample][channel][position]
    alignas(16) uint16_t dz3t[4 * CO * 8];     // [sample][channel][position]
    float dz4[4][CO], dout[4][8], out[4][8], a4[4][CO];
    float red[2][256];
};
constexpr int P3S = P3 + 16;

__global__ __launch_bounds__(256, 1) void k_ws_train34(const WsNet net, const WsHeadArgs h,
                                                       const WsWork w, int64_t B)
{
    __shared__ Lds34 s;
    const int tid = threadIdx.x, lane = tid & 63, wv = sgpr(tid >> 6), g = lane >> 4, col = lane & 15;
    for (int i = tid; i < 4 * P3S; i += 256) s.a2[i] = 0;
    for (int i = tid; i < 4 * CO * D3; i += 256) s.dil[i] = 0;
    for (int i = tid; i < 27 * 32; i += 256) {
        const int k = natural_k(i), c = k / 27, t = k % 27, kz = t / 9, ky = t / 3 % 3, kx = t % 3;
        s.off3[i] = (uint16_t)(((kz * 5 + ky) * 5 + kx) * CO + c);
        s.offd[i] = (int16_t)(c * D3 - ((kz * 6 + ky) * 6 + kx));
    }
    float acc4[CO], accl = 0.0f, b4 = 0.0f, bl = 0.0f, b3[4] = {}, b2[2][4] = {};
#pragma unroll
    for (int o = 0; o < CO; ++o) acc4[o] = 0.0f;
    double loss = 0.0;
    v4f acc3[7][2][2];                    // taps wv, wv + 4, ...; channel tiles of o and c
#pragma unroll
    for (int i = 0; i < 7; ++i)
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < 2; ++n) acc3[i][m][n] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    // the 4 x 8 (sample, position) columns of layers 3: wavefront = (channel tile, column tile)
    const int m3 = 16 * (wv & 1), s3 = 2 * (wv >> 1) + (col >> 3), p3 = col & 7;
    const int c4 = tid >> 3, t4 = tid & 7;     // thread = (c, tap) of the fourth layer's weights
#pragma unroll 1
    for (int64_t b = (int64_t)blockIdx.x * 4; b < B; b += (int64_t)gridDim.x * 4) {
        __syncthreads();
        for (int i = tid; i < 4 * 64 * CO / 8; i += 256) {
            const int q = i & 255, p = q >> 2;       // 8 channels of position p of sample i / 256
            const int e = (((p >> 4) + 1) * 5 + (p >> 2 & 3) + 1) * 5 + (p & 3) + 1;
            *reinterpret_cast<uint4*>(s.a2 + (i >> 8) * P3S + e * CO + (q & 3) * 8) =
                reinterpret_cast<const uint4*>(w.a2 + b * 64 * CO)[i];
        }
        __syncthreads();
        // layer 3
        {
            const uint16_t* src =
                s.a2 + s3 * P3S + ((2 * (p3 >> 2) * 5 + 2 * (p3 >> 1 & 1)) * 5 + 2 * (p3 & 1)) * CO;
            const uint16_t* wr = net.w[2] + (m3 + col) * KP2 + 4 * g;
            v4f c = {};
#pragma unroll 9
            for (int st = 0; st < 27; ++st) {
                const v8s wv8 = join(*reinterpret_cast<const v4s*>(wr + 32 * st),
                                     *reinterpret_cast<const v4s*>(wr + 32 * st + 16));
                c = mfma8(wv8, gather8(src, s.off3 + (st * 4 + g) * 8), c);
            }
            v4f z;
#pragma unroll
            for (int j = 0; j < 4; ++j) z[j] = c[j] + net.b[2][m3 + 4 * g + j];
            *reinterpret_cast<v4f*>(&s.z3[s3][p3][m3 + 4 * g]) = z;
            const v4s a = silu4(z);
#pragma unroll
            for (int j = 0; j < 4; ++j) s.a3[(s3 * CO + m3 + 4 * g + j) * 8 + p3] = (uint16_t)a[j];
        }
        __syncthreads();
        // layer 4: column = sample (the columns past the fourth repeat it), K = c 8 + tap
        if (wv < 2) {
            const int sm = min(col, 3);
            const uint16_t* wr = net.w[3] + (16 * wv + col) * KP4 + 4 * g;
            const uint16_t* src = s.a3 + sm * CO * 8 + 4 * g;
            v4f c = {};
#pragma unroll
            for (int st = 0; st < 8; ++st)
                c = mfma2(*reinterpret_cast<const v4s*>(wr + 32 * st),
                          *reinterpret_cast<const v4s*>(wr + 32 * st + 16),
                          *reinterpret_cast<const v4s*>(src + 32 * st),
                          *reinterpret_cast<const v4s*>(src + 32 * st + 16), c);
            if (col < 4)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    s.z4[col][16 * wv + 4 * g + j] = c[j] + net.b[3][16 * wv + 4 * g + j];
        }
        __syncthreads();
        // head
        if (tid < 4 * CO) s.a4[tid >> 5][tid & 31] = silu(s.z4[tid >> 5][tid & 31]);
        __syncthreads();
        if (tid < 32) s.out[tid >> 3][tid & 7] = ws_head_output(h, s.a4[tid >> 3], tid & 7);
        __syncthreads();
        if (tid < 4) loss += (double)ws_head_loss(h, b + tid, s.out[tid], s.dout[tid]);
        __syncthreads();
        if (tid < 4 * CO) {
            const int i = tid >> 5, c = tid & 31;
            s.dz4[i][c] = from_bf16(to_bf16(ws_head_back(h, s.dout[i], c) * nrfcore::dsilu(s.z4[i][c])));
        }
        __syncthreads();
        // thread = (j, c) of the head's 8 x 32 weights
#pragma unroll
        for (int i = 0; i < 4; ++i) accl += s.dout[i][tid >> 5] * s.a4[i][tid & 31];
        if (tid < 8)
            for (int i = 0; i < 4; ++i) bl += s.dout[i][tid];
        if (tid < CO)
            for (int i = 0; i < 4; ++i) b4 += s.dz4[i][tid];
        // dW4
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float a3 = from_bf16(s.a3[(i * CO + c4) * 8 + t4]);
#pragma unroll
            for (int o = 0; o < CO; ++o) acc4[o] = fmaf(s.dz4[i][o], a3, acc4[o]);
        }
        // dZ3: K = o 8 + tap, of which only tap = the position is not zero; a lane's half step
        // holds output channel 4 st + 2 h + g / 2 and taps 4 (g % 2) ..
        {
            v4f c = {};
#pragma unroll
            for (int st = 0; st < 8; ++st) {
                v4s av[2], bv[2];
#pragma unroll
                for (int hh = 0; hh < 2; ++hh) {
                    const int o = 4 * st + 2 * hh + (g >> 1);
                    av[hh] = *reinterpret_cast<const v4s*>(net.w[3] + o * KP4 + (m3 + col) * 8 + 4 * (g & 1));
                    const short d = (p3 >> 2) == (g & 1) ? (short)to_bf16(s.dz4[s3][o]) : (short)0;
                    const int j = p3 & 3;
                    bv[hh] = v4s{j == 0 ? d : (short)0, j == 1 ? d : (short)0, j == 2 ? d : (short)0,
                                 j == 3 ? d : (short)0};
                }
                c = mfma2(av[0], av[1], bv[0], bv[1], c);
            }
            const v4s dz = dsilu4(c, *reinterpret_cast<const v4f*>(&s.z3[s3][p3][m3 + 4 * g]));
            const int d0 = ((2 * (p3 >> 2) + 1) * 6 + 2 * (p3 >> 1 & 1) + 1) * 6 + 2 * (p3 & 1) + 1;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int ch = s3 * CO + m3 + 4 * g + j;
                b3[j] += from_bf16((uint16_t)dz[j]);
                s.dz3t[ch * 8 + p3] = (uint16_t)dz[j];
                s.dil[ch * D3 + d0] = (uint16_t)dz[j];
            }
        }
        __syncthreads();
        // dW3: K = (sample g, 8 positions)
        v8s da[2];
#pragma unroll
        for (int m = 0; m < 2; ++m)
            da[m] = *reinterpret_cast<const v8s*>(s.dz3t + (g * CO + 16 * m + col) * 8);
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            const int t = wv + 4 * i;
            if (t >= 27) break;
            const int t0 = ((t / 9 * 5) + t / 3 % 3) * 5 + t % 3;
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                v8s x;
#pragma unroll
                for (int p = 0; p < 8; ++p)
                    x[p] = (short)s.a2[g * P3S + (t0 + (2 * (p >> 2) * 5 + 2 * (p >> 1 & 1)) * 5 +
                                                  2 * (p & 1)) * CO + 16 * n + col];
                acc3[i][0][n] = mfma8(da[0], x, acc3[i][0][n]);
                acc3[i][1][n] = mfma8(da[1], x, acc3[i][1][n]);
            }
        }
        // dZ2: wavefront = sample, column tile = plane of its 64 positions, K = (o, tap)
        {
            v4f c[4][2] = {};
            const uint16_t* src = s.dil + wv * CO * D3 + (2 * 6 + (col >> 2) + 2) * 6 + (col & 3) + 2;
            const v8s* wt = reinterpret_cast<const v8s*>(w.wt + WT) + lane;
#pragma unroll 3
            for (int st = 0; st < 27; ++st) {
                const v8s w0 = wt[st * 128], w1 = wt[st * 128 + 64];
                const v8s of = *reinterpret_cast<const v8s*>(s.offd + (st * 4 + g) * 8);
#pragma unroll
                for (int n = 0; n < 4; ++n) {
                    v8s d;
#pragma unroll
                    for (int j = 0; j < 8; ++j) d[j] = (short)src[n * 36 + of[j]];
                    c[n][0] = mfma8(w0, d, c[n][0]);
                    c[n][1] = mfma8(w1, d, c[n][1]);
                }
            }
#pragma unroll
            for (int n = 0; n < 4; ++n)
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const int64_t q = (b + wv) * 64 * CO;
                    const int p = n * 16 + col, ch = 16 * m + 4 * g;
                    const v4s dz = dsilu4(c[n][m], *reinterpret_cast<const v4f*>(w.z2 + q + p * CO + ch));
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        b2[m][j] += from_bf16((uint16_t)dz[j]);
                        w.dz2[q + (ch + j) * 64 + p] = (uint16_t)dz[j];
                    }
                }
        }
    }
    float* part = w.part34 + (int64_t)blockIdx.x * P34;
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        const int t = wv + 4 * i;
        if (t >= 27) break;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < 2; ++n)
                *reinterpret_cast<v4f*>(part + P34_W3 + (((t * 2 + m) * 2 + n) * 64 + lane) * 4) =
                    acc3[i][m][n];
    }
#pragma unroll
    for (int o = 0; o < CO; ++o) part[P34_W4 + o * KP4 + tid] = acc4[o];
    part[P34_WL + tid] = accl;
    if (tid < CO) part[P34_B4 + tid] = b4;
    if (tid < 8) part[P34_BL + tid] = bl;
    loss += __shfl_xor(loss, 1, 64);      // threads 0..3 hold the samples' sums
    loss += __shfl_xor(loss, 2, 64);
    if (tid == 0) w.loss_part[blockIdx.x] = loss;
    // bias sums: over the 16 columns of a lane group, then the wavefronts that share a channel
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float u = b3[j], v[2] = {b2[0][j], b2[1][j]};
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) {
            u += __shfl_xor(u, o, 64);
            v[0] += __shfl_xor(v[0], o, 64);
            v[1] += __shfl_xor(v[1], o, 64);
        }
        if (col == 0) {
            s.red[0][(wv >> 1) * CO + m3 + 4 * g + j] = u;
            s.red[1][wv * CO + 4 * g + j] = v[0];
            s.red[1][wv * CO + 16 + 4 * g + j] = v[1];
        }
    }
    __syncthreads();
    if (tid < CO) {
        part[P34_B3 + tid] = s.red[0][tid] + s.red[0][CO + tid];
        part[P34_B2 + tid] = (s.red[1][tid] + s.red[1][CO + tid]) +
                             (s.red[1][2 * CO + tid] + s.red[1][3 * CO + tid]);
    }
}

// ---- backward of layers 2 and 1: one sample at a time --------------------------------------------------
// The first layer is formed again (its activations are not kept), transposed: rows = 16 positions
// of one (iz, y parity, x parity), columns = channels, so that a lane holds channel c at (iz,
// 2 g + py, 2 j + px), j < 4.
constexpr int G_C = 9 * 9 * 12 + 0;       // a channel's input groups: [z + 1][y + 1][kx][4]
constexpr int DZC = 125;                  // a channel of dZ2, [oz 5][oy 5][ox 5] (zeros past 3)
constexpr int XG_C = 10 * 10 * 16;        // a patch channel's groups: [z + 1][y + 1][s][4]

struct Lds12 {
    alignas(16) uint16_t in[PATCH];
    alignas(16) uint16_t xg[3 * XG_C];
    union {
        alignas(16) uint16_t a1[CO * G_C];
        float w1[4][2 * N1 * 64 * 4];     // the wavefronts' sums at the end
    };
    alignas(16) uint16_t wt[WT];
    alignas(16) uint16_t dzs[CO * DZC];
    alignas(16) uint16_t dzt[CO * 64];    // [channel][position]
    float red[4][CO];
};
static_assert(sizeof(Lds12) <= 160 * 1024, "one block per CU");

__global__ __launch_bounds__(256, 1) void k_ws_back12(const WsWork w, const uint16_t* __restrict__ W1,
                                                      const float* __restrict__ bias1,
                                                      const uint16_t* __restrict__ X, int64_t B)
{
    __shared__ Lds12 s;
    const int tid = threadIdx.x, lane = tid & 63, wv = sgpr(tid >> 6), g = lane >> 4, col = lane & 15;
    Natural1 l1;
    l1.load(W1, lane);
    const float bias[2] = {bias1[col], bias1[16 + col]};
    for (int i = tid; i < PATCH; i += 256) s.in[i] = 0;
    for (int i = tid; i < 3 * XG_C; i += 256) s.xg[i] = 0;
    for (int i = tid; i < CO * G_C; i += 256) s.a1[i] = 0;
    for (int i = tid; i < CO * DZC; i += 256) s.dzs[i] = 0;
    for (int i = tid; i < WT / 8; i += 256)
        reinterpret_cast<uint4*>(s.wt)[i] = reinterpret_cast<const uint4*>(w.wt)[i];
    v4f acc2[7][2][2], acc1[2][N1];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int i = 0; i < 7; ++i) acc2[i][m][n] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int n = 0; n < N1; ++n) acc1[m][n] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    }
    float b1[2] = {0.0f, 0.0f};
    // the lane's column (c, tap) of the first layer's weight gradient in the patch groups
    // (columns past 80 repeat the first; their sums are dropped)
    int xo[N1];
#pragma unroll
    for (int n = 0; n < N1; ++n) {
        const int k = 16 * n + col < 81 ? 16 * n + col : 0;
        xo[n] = (k / 27) * XG_C + (k / 9 % 3) * 160 + (k / 3 % 3) * 16 + (k % 3) * 4 + g * 32;
    }
    const bool stager = tid < 192;
    uint16_t* xrow = s.xg + (tid >> 6) * XG_C + ((tid >> 3 & 7) + 1) * 160 + ((tid & 7) + 1) * 16;
    // dZ2: thread = 8 positions (two rows of x) of a channel
    uint16_t* drow = s.dzs + (tid >> 3) * DZC + ((tid >> 1 & 3) * 5 + (tid & 1) * 2) * 5;
    uint4 nx = make_uint4(0u, 0u, 0u, 0u), nt = nx;
    auto fetch = [&](int64_t b) {
        if (stager) nx = reinterpret_cast<const uint4*>(X + b * 1536)[tid];
        nt = reinterpret_cast<const uint4*>(w.dz2 + b * 64 * CO)[tid];
    };
    if (blockIdx.x < B) fetch(blockIdx.x);
    const int ay = col >> 2, ax = col & 3;           // a tile row's place in its class
#pragma unroll 1
    for (int64_t b = blockIdx.x; b < B; b += gridDim.x) {
        __syncthreads();
        if (stager) {
            stage_patch(s.in, tid, nx);
            // groups s: x = 2 j + s - 1
            const uint32_t e0 = nx.x, e1 = nx.y, e2 = nx.z, e3 = nx.w;
            const uint32_t ev0 = (e0 & 0xffffu) | (e1 << 16), ev1 = (e2 & 0xffffu) | (e3 << 16);
            const uint32_t od0 = (e0 >> 16) | (e1 & 0xffff0000u), od1 = (e2 >> 16) | (e3 & 0xffff0000u);
            uint4* q = reinterpret_cast<uint4*>(xrow);
            q[0] = make_uint4(od0 << 16, (od0 >> 16) | (od1 << 16), ev0, ev1);
            q[1] = make_uint4(od0, od1, (ev0 >> 16) | (ev1 << 16), ev1 >> 16);
        }
        reinterpret_cast<uint4*>(s.dzt)[tid] = nt;
        {
            const uint32_t q[4] = {nt.x, nt.y, nt.z, nt.w};
#pragma unroll
            for (int i = 0; i < 8; ++i) drow[(i >> 2) * 5 + (i & 3)] = (uint16_t)(q[i >> 1] >> (16 * (i & 1)));
        }
        __syncthreads();
        if (b + gridDim.x < B) fetch(b + gridDim.x);
        // the first layer again: tile q of this wavefront = (plane 2 wv + q / 4, py, px)
        v4f z1[8][2];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int iz = 2 * wv + (q >> 2), py = q >> 1 & 1, px = q & 1;
            v8s xv[3];
            l1.patch(s.in + (iz * 10 + 2 * ay + py) * 12 + 2 * ax + px, xv);
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                v4f c = {};
#pragma unroll
                for (int st = 0; st < 3; ++st) c = mfma8(xv[st], l1.w[m][st], c);
                z1[q][m] = v4f{c.x + bias[m], c.y + bias[m], c.z + bias[m], c.w + bias[m]};
            }
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const uint64_t a = __builtin_bit_cast(uint64_t, silu4(z1[q][m]));
                uint64_t* dst = reinterpret_cast<uint64_t*>(
                    s.a1 + (16 * m + col) * G_C + ((iz + 1) * 9 + 2 * g + py + 1) * 12);
                // output ox reads x = 2 ox - 1 + kx: even x through kx = 1, odd through 2 and 0
                if (px == 0) {
                    dst[1] = a;
                } else {
                    dst[2] = a;
                    dst[0] = a << 16;
                }
            }
        }
        __syncthreads();
        // dW2: K = positions, oy = g, ox = j; a K step is two planes oz
        {
            v4s dz[2][4];
#pragma unroll
            for (int m = 0; m < 2; ++m)
#pragma unroll
                for (int oz = 0; oz < 4; ++oz)
                    dz[m][oz] = *reinterpret_cast<const v4s*>(s.dzt + (16 * m + col) * 64 + oz * 16 + 4 * g);
#pragma unroll
            for (int i = 0; i < 7; ++i) {
                const int t = wv + 4 * i;
                if (t >= 27) break;
                const int kz = t / 9, ky = t / 3 % 3, kx = t % 3;
#pragma unroll
                for (int n = 0; n < 2; ++n) {
                    const uint16_t* src =
                        s.a1 + (16 * n + col) * G_C + (kz * 9 + 2 * g + ky) * 12 + kx * 4;
                    v4s x[4];
#pragma unroll
                    for (int oz = 0; oz < 4; ++oz)
                        x[oz] = *reinterpret_cast<const v4s*>(src + 2 * oz * 9 * 12);
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        acc2[i][m][n] = mfma2(dz[m][0], dz[m][1], x[0], x[1], acc2[i][m][n]);
                        acc2[i][m][n] = mfma2(dz[m][2], dz[m][3], x[2], x[3], acc2[i][m][n]);
                    }
                }
            }
        }
        // dZ1 of the wavefront's tiles, and with it dW1: K = the positions of two tiles (px = 0, 1)
#pragma unroll
        for (int pz = 0; pz < 2; ++pz)
#pragma unroll
            for (int py = 0; py < 2; ++py) {
                v4s dz[2][2];             // [px][channel tile]
#pragma unroll
                for (int px = 0; px < 2; ++px) {
                    // K order of the class (output channel, then the taps of its odd axes, x's the
                    // lowest bit: bit 0 -> tap 0 and the output one further, bit 1 -> tap 2)
                    v4f d[2] = {};
                    const int nc = 1 << (pz + py + px), st0 = class_steps(pz * 4 + py * 2 + px);
                    const int og = nc == 8 ? g >> 1 : nc == 1 ? 4 * g : nc == 2 ? 2 * g : g;
                    const uint16_t* src = s.dzs + og * DZC + (wv * 5 + ay) * 5 + ax +
                                          (nc == 8 && !(g & 1) ? 25 : 0);
#pragma unroll
                    for (int st = 0; st < nc; ++st) {
                        v8s a;
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            // element i: half i / 4, k = 32 st + 16 (i / 4) + 4 g + i % 4
                            const int k = 32 * st + 16 * (i >> 2) + (i & 3);
                            const int o = k / nc, bits = k % nc;
                            int sh = 0, off = o * DZC;
                            if (px) off += (bits >> sh++ & 1) ? 0 : 1;
                            if (py) off += (bits >> sh++ & 1) ? 0 : 5;
                            if (pz && nc < 8) off += (bits >> sh & 1) ? 0 : 25;
                            a[i] = (short)src[off];
                        }
                        const v8s* wt = reinterpret_cast<const v8s*>(s.wt) + (st0 + st) * 128 + lane;
                        d[0] = mfma8(a, wt[0], d[0]);
                        d[1] = mfma8(a, wt[64], d[1]);
                    }
#pragma unroll
                    for (int m = 0; m < 2; ++m) {
                        dz[px][m] = dsilu4(d[m], z1[4 * pz + 2 * py + px][m]);
                        b1[m] += sum_bf16(dz[px][m]);
                    }
                }
                const uint16_t* src = s.xg + (2 * wv + pz) * 160 + py * 16;
#pragma unroll
                for (int n = 0; n < N1; ++n) {
                    const v4s x0 = *reinterpret_cast<const v4s*>(src + xo[n]);
                    const v4s x1 = *reinterpret_cast<const v4s*>(src + xo[n] + 4);
#pragma unroll
                    for (int m = 0; m < 2; ++m)
                        acc1[m][n] = mfma2(dz[0][m], dz[1][m], x0, x1, acc1[m][n]);
                }
            }
    }
    float* part = w.part12 + (int64_t)blockIdx.x * P12;
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        const int t = wv + 4 * i;
        if (t >= 27) break;
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int n = 0; n < 2; ++n)
                *reinterpret_cast<v4f*>(part + P12_W2 + (((t * 2 + m) * 2 + n) * 64 + lane) * 4) =
                    acc2[i][m][n];
    }
    __syncthreads();                      // every wavefront is done with a1
#pragma unroll
    for (int m = 0; m < 2; ++m) {
#pragma unroll
        for (int n = 0; n < N1; ++n)
            *reinterpret_cast<v4f*>(&s.w1[wv][((m * N1 + n) * 64 + lane) * 4]) = acc1[m][n];
        const float v = group_sum4(b1[m]);
        if (g == 0) s.red[wv][16 * m + col] = v;
    }
    __syncthreads();
    for (int i = tid; i < 2 * N1 * 64; i += 256) {
        v4f v = *reinterpret_cast<const v4f*>(&s.w1[0][4 * i]);
#pragma unroll
        for (int u = 1; u < 4; ++u) v += *reinterpret_cast<const v4f*>(&s.w1[u][4 * i]);
        *reinterpret_cast<v4f*>(part + P12_W1 + 4 * i) = v;
    }
    if (tid < CO) part[P12_B1 + tid] = (s.red[0][tid] + s.red[1][tid]) + (s.red[2][tid] + s.red[3][tid]);
}

// ---- sums over the blocks ------------------------------------------------------------------
// Block of 1024 threads = 64 float4 columns x 16 groups of partials, each group's sums in two
// chains, the groups added in order; then the column goes to its place in the gradients.  The
// columns are those of a part34 record followed by those of a part12 record.
constexpr int Q34 = P34 / 4, Q12 = P12 / 4;

__global__ __launch_bounds__(1024) void k_ws_sums(const WsWork w, const WsGrads g, int nb, int64_t B,
                                                  float* __restrict__ loss)
{
    __shared__ v4f sh[16][64];
    const int l = threadIdx.x & 63, u = threadIdx.x >> 6;
    const int q = blockIdx.x * 64 + l;
    const bool a34 = q < Q34;
    const float* src = a34 ? w.part34 + 4 * q : w.part12 + 4 * (q - Q34);
    const int64_t stride = a34 ? P34 : P12;
    v4f s0 = {}, s1 = {};
    if (q < Q34 + Q12) {
        int i = u;
        for (; i + 16 < nb; i += 32) {
            s0 += *reinterpret_cast<const v4f*>(src + i * stride);
            s1 += *reinterpret_cast<const v4f*>(src + (i + 16) * stride);
        }
        if (i < nb) s0 += *reinterpret_cast<const v4f*>(src + i * stride);
    }
    sh[u][l] = s0 + s1;
    if (blockIdx.x == 0 && u == 1) {
        double v = 0.0;
        for (int i = l; i < nb; i += 64) v += w.loss_part[i];
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        if (l == 0) loss[0] = (float)(v / (double)B);
    }
    __syncthreads();
    if (u != 0 || q >= Q34 + Q12) return;
    v4f v = sh[0][l];
#pragma unroll
    for (int i = 1; i < 16; ++i) v += sh[i][l];
    const int e = 4 * (a34 ? q : q - Q34);           // first element within its record
    // a 32x32x27 layer: [tap][o tile][c tile][lane][4], lane holding rows o of column c
    const bool w3 = a34 && e < P34_W4, w2 = !a34 && e < P12_W1;
    if (w3 || w2) {
        float* dst = w3 ? g.w[2] : g.w[1];
        const int ln = (e >> 2) & 63, n = (e >> 8) & 1, m = (e >> 9) & 1, t = e >> 10;
        const int o = 16 * m + 4 * (ln >> 4), c = 16 * n + (ln & 15);
#pragma unroll
        for (int j = 0; j < 4; ++j) dst[(o + j) * KP2 + c * 27 + t] += v[j];
        return;
    }
    if (!a34 && e < P12_B1) {
        const int f = (e - P12_W1) >> 2, ln = f & 63, n = (f >> 6) % N1, m = (f >> 6) / N1;
        const int o = 16 * m + 4 * (ln >> 4), k = 16 * n + (ln & 15);
        if (k < 81) {
#pragma unroll
            for (int j = 0; j < 4; ++j) g.w[0][(o + j) * KP1 + k] += v[j];
        }
        return;
    }
    float* dst;
    if (!a34) dst = g.b[0] + e - P12_B1;
    else if (e < P34_WL) dst = g.w[3] + e - P34_W4;
    else if (e < P34_B4) dst = g.wl + e - P34_WL;
    else if (e < P34_B3) dst = g.b[3] + e - P34_B4;
    else if (e < P34_B2) dst = g.b[2] + e - P34_B3;
    else if (e < P34_BL) dst = g.b[1] + e - P34_B2;
    else dst = g.bl + e - P34_BL;
#pragma unroll
    for (int j = 0; j < 4; ++j) dst[j] += v[j];
}

int blocks(int64_t B) { return (int)(B / 4 < MAX_BLOCKS ? B / 4 : MAX_BLOCKS); }

}  // namespace

size_t ws_part_floats(int64_t B) { return (size_t)blocks(B) * (P34 + P12); }
size_t ws_loss_parts(int64_t B) { return (size_t)blocks(B); }
size_t ws_wt_elems() { return 2 * (size_t)WT; }
float* ws_part12(float* part, int64_t B) { return part + (size_t)blocks(B) * P34; }

hipError_t launch_ws_train(const WsNet& net, const uint16_t* X0, int64_t B, const WsWork& w,
                           const WsHeadArgs& head, const WsGrads& g, float* loss, hipStream_t s)
{
    const int nb = blocks(B);
    hipLaunchKernelGGL(k_ws_train12, dim3((unsigned)nb + PACK_BLOCKS), dim3(256), 0, s, net, X0, B, w);
    hipLaunchKernelGGL(k_ws_train34, dim3((unsigned)nb), dim3(256), 0, s, net, head, w, B);
    hipLaunchKernelGGL(k_ws_back12, dim3((unsigned)nb), dim3(256), 0, s, w, net.w[0], net.b[0], X0, B);
    hipLaunchKernelGGL(k_ws_sums, dim3((Q34 + Q12 + 63) / 64), dim3(1024), 0, s, w, g, nb, B, loss);
    return hipGetLastError();
}
