// K12 inference: the warm-start network's convolutions in two kernels whose activations stay on chip
// (see warm.hip for the layers).  k_ws_conv12 takes a sample's patch through the first two
// convolutions, the 8^3 x 32 activations between them in LDS; k_ws_conv34 takes 16 samples
// through the last two.  Only the 4^3 x 32 activations (4 KB a sample) go through memory.
//
// Every convolution is a GEMM on gfx950's 16x16x32 BF16 MFMA, M = 16 output channels, N = 16
// output positions.  From the second layer on a K step of 32 is one tap with all 32 input
// channels and activations lie channel-last, so that a lane's B operand (8 channels of its
// position) is one 16-byte read at an address that is a per-lane base plus a constant per tap.
// In the first layer (3 channels) a lane's half operand is the four x neighbours of one
// (channel, kz, ky), the fourth against a zero weight: 8 contiguous bytes from one of two copies
// of the patch, the second shifted by one element, so that either parity of x reads whole words.
// The MFMA result holds four consecutive channels of a position per lane: 8 bytes of the next
// layer's input.
//
// Per sample k_ws_conv12 issues 472 MFMAs (1900 cycles on a CU's four SIMDs), the vector
// instructions of 288 SiLUs per lane (3200 cycles) and 380 KB of LDS reads (3000 cycles); it takes
// about 5700 (9.7 ms for a million samples), the matrix and vector work of a SIMD overlapping only
// between its two wavefronts.  (Forming a tile's activations while the next tile's products run:
// 3%; enforcing that interleaving instruction by instruction: slower.)  k_ws_conv34 takes 2.3 ms
// for them, bound by the latency of its input reads.  A kernel per layer with the operands
// gathered element by element took 80 ms.
#include "warm_core.h"

namespace {

using namespace warmcore;

// The first layer's activations: position (z, y, x), x, y, z >= -1, at 40 elements (80 bytes) per
// x with even and odd x apart (a stride-2 read then walks neighbouring slots); rows of 46 16-byte
// slots.  The 8 positions (4 x, 2 y) that share a read cycle fall in 8 different 16-byte slots of
// the 128-byte bank row.
constexpr int A_POS = 40, A_ROW = 46 * 8, A_Z = 9 * A_ROW;
// slot of padded x (0..8): even 0..4, odd 5..8
__device__ __forceinline__ constexpr int a_x(int x) { return (x & 1) ? 5 + (x >> 1) : x >> 1; }

struct Lds12 {
    uint32_t in[2 * IN_COPY];
    alignas(16) uint16_t a1[9 * A_Z];
};
static_assert(sizeof(Lds12) <= 80 * 1024, "two blocks per CU");
static_assert(CO * KP2 <= 9 * A_Z, "the second layer's weights pass through the activations' space");

__global__ __launch_bounds__(256, 2) void k_ws_conv12(const uint16_t* __restrict__ W1,
                                                      const float* __restrict__ b1,
                                                      const uint16_t* __restrict__ W2,
                                                      const float* __restrict__ b2,
                                                      const uint16_t* __restrict__ X, int64_t B,
                                                      uint16_t* __restrict__ A2)
{
    __shared__ Lds12 s;
    const int lane = threadIdx.x & 63, w = sgpr(threadIdx.x >> 6), g = lane >> 4, col = lane & 15;
    Layer1 l1;
    l1.load(W1, lane);
    // the second layer's weights of channel tile w & 1, tap by tap, through LDS
    const int m2 = 16 * (w & 1), n2 = (w >> 1) * 2;      // ... for output planes n2, n2 + 1
    for (int i = threadIdx.x; i < CO * KP2 / 4; i += 256)     // (weights are 8-byte aligned)
        reinterpret_cast<uint2*>(s.a1)[i] = reinterpret_cast<const uint2*>(W2)[i];
    __syncthreads();
    v8s w2[27];
#pragma unroll
    for (int t = 0; t < 27; ++t)
#pragma unroll
        for (int i = 0; i < 8; ++i) w2[t][i] = (short)s.a1[(m2 + col) * KP2 + (8 * g + i) * 27 + t];
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * IN_COPY; i += 256) s.in[i] = 0u;
    for (int i = threadIdx.x; i < 9 * A_Z / 8; i += 256)
        reinterpret_cast<uint4*>(s.a1)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();    // a patch's rows are staged by other wavefronts than the ones that clear them
    v4f bias1[2], bias2;
#pragma unroll
    for (int m = 0; m < 2; ++m)
        bias1[m] = v4f{b1[16 * m + 4 * g], b1[16 * m + 4 * g + 1], b1[16 * m + 4 * g + 2],
                       b1[16 * m + 4 * g + 3]};
    bias2 = v4f{b2[m2 + 4 * g], b2[m2 + 4 * g + 1], b2[m2 + 4 * g + 2], b2[m2 + 4 * g + 3]};

    // thread t < 192 stages row t of the patch (channel, z, y): 8 values
    const int sr = threadIdx.x;
    const bool stager = sr < 192;
    const int srow = patch_row(sr);
    uint4 nx = make_uint4(0u, 0u, 0u, 0u);
    if (stager && blockIdx.x < B) nx = reinterpret_cast<const uint4*>(X + (int64_t)blockIdx.x * 1536)[sr];
    // the lane's position within a column tile of the first layer (x, and y of two) and of the
    // second (x, y of 4 x 4)
    const int x1 = col & 7, y1 = col >> 3;
    const uint32_t* in0 = s.in + (x1 & 1) * IN_COPY + (x1 >> 1) + y1 * IN_ROW;
    uint16_t* out1 = s.a1 + A_Z + (y1 + 1) * A_ROW + a_x(x1 + 1) * A_POS + 4 * g;
    const uint16_t* in2 = s.a1 + 2 * n2 * A_Z + 2 * (col >> 2) * A_ROW + (col & 3) * A_POS + 8 * g;
#pragma unroll 1
    for (int64_t b = blockIdx.x; b < B; b += gridDim.x) {
        // every wavefront has read the last sample's patch (the barrier after the first layer)
        if (stager) stage_patch_row(s.in, srow, nx);
        __syncthreads();    // ... and every wavefront is done with the last sample's activations
        if (stager && b + gridDim.x < B)
            nx = reinterpret_cast<const uint4*>(X + (b + gridDim.x) * 1536)[sr];
        // first layer: wavefront w takes planes 2 w, 2 w + 1, four tiles (two rows of y) each; the
        // next tile's products run while a tile's activations are formed
        v4f c0, c1;
        auto conv1 = [&](int i, v4f& d0, v4f& d1) {
            const uint32_t* src = in0 + (2 * w + (i >> 2)) * IN_Z + 2 * (i & 3) * IN_ROW;
            d0 = bias1[0];
            d1 = bias1[1];
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                v4s bv[2];
                l1.patch(src, st, bv);
                d0 = mfma2(l1.w[0][st][0], l1.w[0][st][1], bv[0], bv[1], d0);
                d1 = mfma2(l1.w[1][st][0], l1.w[1][st][1], bv[0], bv[1], d1);
            }
        };
        conv1(0, c0, c1);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            v4f n0 = c0, n1 = c1;
            if (i < 7) conv1(i + 1, n0, n1);
            uint16_t* dst = out1 + (2 * w + (i >> 2)) * A_Z + 2 * (i & 3) * A_ROW;
            *reinterpret_cast<v4s*>(dst) = silu4(c0);
            *reinterpret_cast<v4s*>(dst + 16) = silu4(c1);
            c0 = n0;
            c1 = n1;
        }
        __syncthreads();
        // second layer: 27 taps, two output planes
        v4f c[2] = {bias2, bias2};
#pragma unroll
        for (int t = 0; t < 27; ++t) {
            const int kz = t / 9, ky = t / 3 % 3, kx = t % 3;
            const uint16_t* src = in2 + kz * A_Z + ky * A_ROW + a_x(kx) * A_POS;
#pragma unroll
            for (int p = 0; p < 2; ++p)
                c[p] = mfma8(w2[t], *reinterpret_cast<const v8s*>(src + 2 * p * A_Z), c[p]);
        }
#pragma unroll
        for (int p = 0; p < 2; ++p)
            *reinterpret_cast<v4s*>(A2 + ((b * 4 + n2 + p) * 16 + col) * CO + m2 + 4 * g) =
                silu4(c[p]);
    }
}

// Layers three and four of 16 samples at a time; wavefront w takes samples 4 w .. 4 w + 3 (two
// column tiles of 2 samples x 8 positions) through the third, both weights in LDS in operand
// order, the inputs straight from memory (a sample's 4 KB is read by its wavefront only).
constexpr int A3_S = 8 * CO + 8;     // a sample's third-layer activations, 16 bytes of padding

struct Lds34 {
    v8s w3[27 * 2 * 64];
    v8s w4[8 * 2 * 64];
    alignas(16) uint16_t a3[16 * A3_S];
};
static_assert(sizeof(Lds34) <= 80 * 1024, "two blocks per CU");

__global__ __launch_bounds__(256, 2) void k_ws_conv34(const uint16_t* __restrict__ W3,
                                                      const float* __restrict__ b3,
                                                      const uint16_t* __restrict__ W4,
                                                      const float* __restrict__ b4,
                                                      const uint16_t* __restrict__ A2, int64_t B,
                                                      float* __restrict__ Z4)
{
    __shared__ Lds34 s;
    const int lane = threadIdx.x & 63, w = sgpr(threadIdx.x >> 6), g = lane >> 4, col = lane & 15;
    for (int e = threadIdx.x; e < 27 * 2 * 64; e += 256) {
        const int l = e & 63, m = (e >> 6) & 1, t = e >> 7;
        const uint16_t* src = W3 + (16 * m + (l & 15)) * KP2 + 8 * (l >> 4) * 27 + t;
        v8s v;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (short)src[27 * i];
        s.w3[e] = v;
    }
    for (int e = threadIdx.x; e < 8 * 2 * 64; e += 256) {
        const int l = e & 63, m = (e >> 6) & 1, t = e >> 7;
        const uint16_t* src = W4 + (16 * m + (l & 15)) * KP4 + 8 * (l >> 4) * 8 + t;
        v8s v;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (short)src[8 * i];
        s.w4[e] = v;
    }
    v4f bias3[2], bias4;
#pragma unroll
    for (int m = 0; m < 2; ++m)
        bias3[m] = v4f{b3[16 * m + 4 * g], b3[16 * m + 4 * g + 1], b3[16 * m + 4 * g + 2],
                       b3[16 * m + 4 * g + 3]};
    const int m4 = 16 * (w & 1);
    bias4 = v4f{b4[m4 + 4 * g], b4[m4 + 4 * g + 1], b4[m4 + 4 * g + 2], b4[m4 + 4 * g + 3]};
    __syncthreads();
    const int o = col & 7, oz = o >> 2, oy = (o >> 1) & 1, ox = o & 1;
#pragma unroll 1
    for (int64_t b0 = (int64_t)blockIdx.x * 16; b0 < B; b0 += (int64_t)gridDim.x * 16) {
        const int sl = 4 * w + (col >> 3);            // the lane's sample of column tile 0
        const uint16_t* src = A2 + (b0 + sl) * (64 * CO) + 8 * g;
        v4f c[2][2] = {{bias3[0], bias3[1]}, {bias3[0], bias3[1]}};
#pragma unroll
        for (int t = 0; t < 27; ++t) {
            const int kz = t / 9, ky = t / 3 % 3, kx = t % 3;
            // input index 2 o - 1 + k: below 0 for k = 0 at o = 0 (padding), at most 3
            const bool in = (kz > 0 || oz > 0) && (ky > 0 || oy > 0) && (kx > 0 || ox > 0);
            const int iz = max(2 * oz - 1 + kz, 0), iy = max(2 * oy - 1 + ky, 0),
                      ix = max(2 * ox - 1 + kx, 0);
            const int p = (iz * 4 + iy) * 4 + ix;
            const v8s a0 = s.w3[(2 * t) * 64 + lane], a1 = s.w3[(2 * t + 1) * 64 + lane];
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                v8s v = *reinterpret_cast<const v8s*>(src + n * 2 * 64 * CO + p * CO);
                if (!in) v = v8s{0, 0, 0, 0, 0, 0, 0, 0};
                c[n][0] = mfma8(a0, v, c[n][0]);
                c[n][1] = mfma8(a1, v, c[n][1]);
            }
        }
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            uint16_t* dst = s.a3 + (sl + 2 * n) * A3_S + o * CO + 4 * g;
            *reinterpret_cast<v4s*>(dst) = silu4(c[n][0]);
            *reinterpret_cast<v4s*>(dst + 16) = silu4(c[n][1]);
        }
        __syncthreads();
        if (w < 2) {      // fourth layer: column = sample, one channel tile per wavefront
            v4f z = bias4;
#pragma unroll
            for (int t = 0; t < 8; ++t)
                z = mfma8(s.w4[(2 * t + w) * 64 + lane],
                          *reinterpret_cast<const v8s*>(s.a3 + col * A3_S + t * CO + 8 * g), z);
            *reinterpret_cast<v4f*>(Z4 + (b0 + col) * CO + m4 + 4 * g) = z;
        }
        __syncthreads();
    }
}

}  // namespace

hipError_t launch_ws_infer(const WsNet& net, const uint16_t* X0, int64_t B, const WsWork& w,
                           hipStream_t s)
{
    if (B <= 0) return hipSuccess;
    // two resident blocks per CU, each walking its share of the samples
    const int64_t n12 = B < 512 ? B : 512, n34 = B / 16 < 512 ? B / 16 : 512;
    hipLaunchKernelGGL(k_ws_conv12, dim3((unsigned)n12), dim3(256), 0, s, net.w[0], net.b[0],
                       net.w[1], net.b[1], X0, B, w.a2);
    hipLaunchKernelGGL(k_ws_conv34, dim3((unsigned)n34), dim3(256), 0, s, net.w[2], net.b[2],
                       net.w[3], net.b[3], w.a2, B, w.z4);
    return hipGetLastError();
}
