// Device code shared by the warm-start network's forward and backward kernels: the first layer's
// operands and their layout in LDS, and channel-last MFMA products.
#ifndef GM_WARM_CORE_H
#define GM_WARM_CORE_H
#include "nrf_core.h"

namespace warmcore {

using nrfcore::from_bf16;
using nrfcore::to_bf16;
using nrfcore::mfma2;
using nrfcore::pack4;
using nrfcore::silu;
using nrfcore::v4f;
using nrfcore::v4s;
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef short v8s __attribute__((ext_vector_type(8)));

__device__ __forceinline__ int sgpr(int v) { return __builtin_amdgcn_readfirstlane(v); }

// 32-wide K step: lane group g supplies slots 8 g + i in A and in B alike
__device__ __forceinline__ v4f mfma8(v8s a, v8s b, v4f c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a),
                                                   __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}
__device__ __forceinline__ v4s silu4(v4f z)
{
    return pack4(silu(z.x), silu(z.y), silu(z.z), silu(z.w));
}
// four gradients through SiLU: d SiLU'(z), rounded to BF16
__device__ __forceinline__ v4s dsilu4(v4f d, v4f z)
{
    return pack4(d.x * nrfcore::dsilu(z.x), d.y * nrfcore::dsilu(z.y), d.z * nrfcore::dsilu(z.z),
                 d.w * nrfcore::dsilu(z.w));
}

constexpr int CO = 32, KP1 = 96, KP2 = 864, KP4 = 256;   // channels, padded K of the weights

// The patch in LDS: two copies of [channel][z + 1][y + 1] rows of 12 BF16 (6 words), x from -1 in
// the first, from 0 in the second; the copies 12 (mod 32) words apart so that the rows two
// lane groups read sit in different banks.
constexpr int IN_ROW = 6, IN_Z = 10 * IN_ROW, IN_C = 10 * IN_Z, IN_COPY = 3 * IN_C + 4;

// thread t < 192 holds row t of a patch (channel, z, y): the word of its first value's row
__device__ __forceinline__ int patch_row(int t)
{
    return (t >> 6) * IN_C + ((t >> 3 & 7) + 1) * IN_Z + ((t & 7) + 1) * IN_ROW;
}
// its 8 values v into both copies
__device__ __forceinline__ void stage_patch_row(uint32_t* in, int row, uint4 v)
{
    uint32_t* r0 = in + row;
    uint32_t* r1 = r0 + IN_COPY;
    r0[0] = v.x << 16;
    r0[1] = (v.x >> 16) | (v.y << 16);
    r0[2] = (v.y >> 16) | (v.z << 16);
    r0[3] = (v.z >> 16) | (v.w << 16);
    r0[4] = v.w >> 16;
    r1[0] = v.x;
    r1[1] = v.y;
    r1[2] = v.z;
    r1[3] = v.w;
}

// The first layer's weights (both channel tiles) as an operand of 4 K steps: a lane's half
// operand is the four x neighbours of K group q = (channel, kz, ky) = 8 st + 4 h + g, the fourth
// weight zero (groups past 26 all zero); off: the group's word offset in the patch.
struct Layer1 {
    v4s w[2][4][2];
    int off[4][2];
    __device__ __forceinline__ void load(const uint16_t* W1, int lane)
    {
        const int g = lane >> 4, col = lane & 15;
#pragma unroll
        for (int st = 0; st < 4; ++st)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int q = 8 * st + 4 * h + g, qq = q < 27 ? q : 0;
                off[st][h] = (qq / 9) * IN_C + (qq / 3 % 3) * IN_Z + (qq % 3) * IN_ROW;
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    const uint16_t* src = W1 + (16 * m + col) * KP1 + 3 * qq;
                    w[m][st][h] = q < 27 ? v4s{(short)src[0], (short)src[1], (short)src[2], 0}
                                         : v4s{0, 0, 0, 0};
                }
            }
    }
    // the patch operand of K step st at the lane's position (src: its first word)
    __device__ __forceinline__ void patch(const uint32_t* src, int st, v4s (&bv)[2]) const
    {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t* r = src + off[st][h];
            bv[h] = __builtin_bit_cast(v4s, make_uint2(r[0], r[1]));
        }
    }
};

// ---- the training step's operands: K = (channel, tap) in that order --------------------------
// Element i of a lane of group g in K step st: half i / 4, k = 32 st + 16 (i / 4) + 4 g + i % 4.
// For e = (st 4 + g) 8 + i:
__device__ __forceinline__ int natural_k(int e)
{
    return 32 * (e >> 5) + 16 * (e >> 2 & 1) + 4 * (e >> 3 & 3) + (e & 3);
}
__device__ __forceinline__ v8s join(v4s a, v4s b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }

// eight elements at src + off[0..7] (off: 16-byte aligned, LDS)
__device__ __forceinline__ v8s gather8(const uint16_t* src, const uint16_t* off)
{
    const uint4 o = *reinterpret_cast<const uint4*>(off);
    const uint32_t q[4] = {o.x, o.y, o.z, o.w};
    v8s v;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = (short)src[(q[i >> 1] >> (16 * (i & 1))) & 0xffffu];
    return v;
}

// The patch in LDS as [channel][z + 1][y + 1] rows of 12 BF16, x from -1
constexpr int PATCH = 3 * 10 * 10 * 12;
// thread t < 192 stages row t of a patch (channel, z, y): 8 values
__device__ __forceinline__ void stage_patch(uint16_t* in, int t, uint4 v)
{
    uint32_t* r = reinterpret_cast<uint32_t*>(in + ((t >> 6) * 100 + ((t >> 3 & 7) + 1) * 10 + (t & 7) + 1) * 12);
    r[0] = v.x << 16;
    r[1] = (v.x >> 16) | (v.y << 16);
    r[2] = (v.y >> 16) | (v.z << 16);
    r[3] = (v.z >> 16) | (v.w << 16);
    r[4] = v.w >> 16;
}
// the first layer's weights (both channel tiles) and a position's patch operand, three K steps
struct Natural1 {
    v8s w[2][3];
    int off[24];
    __device__ __forceinline__ void load(const uint16_t* W1, int lane)
    {
        const int g = lane >> 4, col = lane & 15;
#pragma unroll
        for (int st = 0; st < 3; ++st) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const uint16_t* src = W1 + (16 * m + col) * KP1 + 32 * st + 4 * g;
                w[m][st] = join(*reinterpret_cast<const v4s*>(src), *reinterpret_cast<const v4s*>(src + 16));
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int k = 32 * st + 16 * (i >> 2) + 4 * g + (i & 3);
                off[8 * st + i] =
                    k < 81 ? (k / 27) * 1200 + (k / 9 % 3) * 120 + (k / 3 % 3) * 12 + k % 3 : -1;
            }
        }
    }
    __device__ __forceinline__ void patch(const uint16_t* src, v8s (&x)[3]) const
    {
#pragma unroll
        for (int st = 0; st < 3; ++st)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int o = off[8 * st + i];
                // only the last K step has padding
                const short v = (short)src[st == 2 ? max(o, 0) : o];
                x[st][i] = st == 2 && o < 0 ? (short)0 : v;
            }
    }
};

constexpr int WS_WT = 27 * 2 * 64 * 8;    // elements of a packed 32x32x27 layer

// ---- loss head: linear 32 -> 8, residual assembly, loss and its gradient ---------------------
// output j of a sample with last activations a4
__device__ __forceinline__ float ws_head_output(const WsHeadArgs& h, const float* a4, int j)
{
    float s = h.bl[j];
#pragma unroll
    for (int c = 0; c < CO; ++c) s += h.wl[j * CO + c] * a4[c];
    return s;
}
// the Gaussian parameters of sample b from its outputs: log-scale, quaternion, logit
__device__ __forceinline__ void ws_head_params(const WsHeadArgs& h, int64_t b, const float* out,
                                               double (&s_)[3], double (&q_)[4], double& lg)
{
#pragma unroll
    for (int m = 0; m < 3; ++m) s_[m] = (double)h.s0[3 * b + m] + out[m];
    q_[0] = 1.0 + out[3];
    q_[1] = (double)out[4];
    q_[2] = (double)out[5];
    q_[3] = (double)out[6];
    lg = (double)h.logit0[b] + out[7];
}
__device__ inline void rot_from_q(const double q[4], double R[9])
{
    const double w = q[0], x = q[1], y = q[2], z = q[3];
    R[0] = 1.0 - 2.0 * (y * y + z * z);
    R[1] = 2.0 * (x * y - w * z);
    R[2] = 2.0 * (x * z + w * y);
    R[3] = 2.0 * (x * y + w * z);
    R[4] = 1.0 - 2.0 * (x * x + z * z);
    R[5] = 2.0 * (y * z - w * x);
    R[6] = 2.0 * (x * z - w * y);
    R[7] = 2.0 * (y * z + w * x);
    R[8] = 1.0 - 2.0 * (x * x + y * y);
}

// sample b's loss, and the gradient of the batch's mean loss with respect to its outputs
__device__ inline float ws_head_loss(const WsHeadArgs& h, int64_t b, const float* out, float* dout)
{
    double s_[3], q_[4], lg;
    ws_head_params(h, b, out, s_, q_, lg);
    // loss: |Sigma - Sigma*|_F^2 / |Sigma*|_F^2 + (logit - logit*)^2, mean over samples
    const double qn = sqrt(q_[0] * q_[0] + q_[1] * q_[1] + q_[2] * q_[2] + q_[3] * q_[3]);
    const double qh[4] = {q_[0] / qn, q_[1] / qn, q_[2] / qn, q_[3] / qn};
    double R[9];
    rot_from_q(qh, R);
    const double S2[3] = {exp(2.0 * s_[0]), exp(2.0 * s_[1]), exp(2.0 * s_[2])};
    const float* st = h.sig_t + 6 * b;  // xx yy zz xy xz yz
    const double T[9] = {st[0], st[3], st[4], st[3], st[1], st[5], st[4], st[5], st[2]};
    double S[9], num = 0.0, den = 0.0;
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            S[3 * p + q] = R[3 * p] * S2[0] * R[3 * q] + R[3 * p + 1] * S2[1] * R[3 * q + 1] +
                           R[3 * p + 2] * S2[2] * R[3 * q + 2];
            num += (S[3 * p + q] - T[3 * p + q]) * (S[3 * p + q] - T[3 * p + q]);
            den += T[3 * p + q] * T[3 * p + q];
        }
    const double dlg_ = lg - (double)h.logit_t[b];
    const float loss = (float)(num / den + dlg_ * dlg_);
    const double inv = 1.0 / (double)h.n;
    double G[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) G[t] = 2.0 * (S[t] - T[t]) / den * inv;
    // Sigma = R diag(S2) R^T
    double GR[9], RtGR[9];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int q = 0; q < 3; ++q)
            GR[3 * p + q] = G[3 * p] * R[q] + G[3 * p + 1] * R[3 + q] + G[3 * p + 2] * R[6 + q];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int q = 0; q < 3; ++q)
            RtGR[3 * p + q] = R[p] * GR[q] + R[3 + p] * GR[3 + q] + R[6 + p] * GR[6 + q];
    double g[9];
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int q = 0; q < 3; ++q) g[3 * p + q] = 2.0 * GR[3 * p + q] * S2[q];
    double d8[8];
    d8[0] = 2.0 * S2[0] * RtGR[0];
    d8[1] = 2.0 * S2[1] * RtGR[4];
    d8[2] = 2.0 * S2[2] * RtGR[8];
    const double w = qh[0], x = qh[1], y = qh[2], z = qh[3];
    double dq[4];
    dq[0] = 2.0 * (-z * g[1] + y * g[2] + z * g[3] - x * g[5] - y * g[6] + x * g[7]);
    dq[1] = 2.0 * (y * g[1] + z * g[2] + y * g[3] - 2.0 * x * g[4] - w * g[5] + z * g[6] + w * g[7] -
                   2.0 * x * g[8]);
    dq[2] = 2.0 * (-2.0 * y * g[0] + x * g[1] + w * g[2] + x * g[3] + z * g[5] - w * g[6] + z * g[7] -
                   2.0 * y * g[8]);
    dq[3] = 2.0 * (-2.0 * z * g[0] - w * g[1] + x * g[2] + w * g[3] - 2.0 * z * g[4] + y * g[5] +
                   x * g[6] + y * g[7]);
    const double dot = w * dq[0] + x * dq[1] + y * dq[2] + z * dq[3];
#pragma unroll
    for (int m = 0; m < 4; ++m) d8[3 + m] = (dq[m] - qh[m] * dot) / qn;
    d8[7] = 2.0 * dlg_ * inv;
#pragma unroll
    for (int j = 0; j < 8; ++j) dout[j] = (float)d8[j];
    return loss;
}
// gradient with respect to last activation c
__device__ __forceinline__ float ws_head_back(const WsHeadArgs& h, const float* dout, int c)
{
    float da = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j) da += h.wl[j * CO + c] * dout[j];
    return da;
}

}  // namespace warmcore
#endif
