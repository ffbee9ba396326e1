// K12: warm-start network - per Gaussian a 3-channel 8^3 patch of the registered stacks
// through four 3D convolutions (width 32, BF16 weights and activations, FP32 accumulation on
// MFMA) and a linear head that predicts residuals (d log-scale 3, d quaternion 4, d logit 1)
// on top of the devoxelization initialisation.  Training backward (dX and dW) on MFMA.
//
// Inference's convolutions are in warm_fwd.hip, a training step's forward and backward in
// warm_train.hip, the loss head's arithmetic in warm_core.h; here are the patch gather, the
// training targets and inference's head.
#include "warm_core.h"

namespace {

using namespace warmcore;

// ---- patch gather -------------------------------------------------------------------------
// One block per Gaussian: a thread samples four patch points of a z column in every stack, so that
// the terms of x and y in the three index sums are formed once and 16 reads are in flight (a point
// outside the stack reads voxel 0).  NEAR, where every stack is wider than one voxel and small
// enough for 24-bit rows and 32-bit byte offsets: the two x neighbours of a corner pair are one
// 8-byte read, and the four pairs lie at one offset from four uniform bases (the clamp leaves
// y0 + 1 and z0 + 1 inside wherever the stack has two rows or planes).  Otherwise eight reads at
// 64-bit offsets.  A million patches (3.1 GB written) 3.2 ms at 57 vector
// instructions a sample; with two points a thread, a branch around each and the row offsets formed
// per corner, 93 instructions, 3.9 ms.
struct __attribute__((packed, aligned(4))) XPair {
    float a, b;
};

__device__ __forceinline__ float lerp(float a, float b, float f) { return fmaf(1.0f - f, a, f * b); }

constexpr int GATHER_THREADS = 128;

template <bool NEAR>
__global__ __launch_bounds__(GATHER_THREADS) void k_ws_gather(const WsGatherArgs a)
{
    constexpr int ZSTEP = GATHER_THREADS / 64, POINTS = 8 / ZSTEP;
    const int64_t b = blockIdx.x;
    const int v0 = threadIdx.x;
    const int x = v0 % 8, y = (v0 / 8) % 8, z = v0 / 64;
    const double wx = (double)fmaf(a.spacing, (float)x - 3.5f, a.means[3 * b]);
    const double wy = (double)fmaf(a.spacing, (float)y - 3.5f, a.means[3 * b + 1]);
    double wz[POINTS];
#pragma unroll
    for (int j = 0; j < POINTS; ++j)
        wz[j] = (double)fmaf(a.spacing, (float)(z + j * ZSTEP) - 3.5f, a.means[3 * b + 2]);
    uint16_t* out = a.patches + b * 3 * 512;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const GridConst& S = a.s[k];
        double xy[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) xy[r] = fma(S.L[3 * r], wx, S.L[3 * r + 1] * wy);
        const float ex = (float)(S.nx - 1), ey = (float)(S.ny - 1), ez = (float)(S.nz - 1);
        const int lx = max(S.nx - 2, 0), ly = max(S.ny - 2, 0), lz = max(S.nz - 2, 0);
        const int64_t dx = S.nx > 1 ? 1 : 0, dy = S.ny > 1 ? S.nx : 0;
        const int64_t dz = S.nz > 1 ? (int64_t)S.ny * S.nx : 0;
        const float* const d00 = a.data[k];
        const float* const d10 = d00 + dy;
        const float* const d01 = d00 + dz;
        const float* const d11 = d01 + dy;
        XPair p00[POINTS], p10[POINTS], p01[POINTS], p11[POINTS];   // p<y><z>: rows y0 + y, z0 + z
        float fx[POINTS], fy[POINTS], fz[POINTS];
        bool in[POINTS];
#pragma unroll
        for (int j = 0; j < POINTS; ++j) {
            float px = (float)(fma(S.L[2], wz[j], xy[0]) + S.t[0]);
            float py = (float)(fma(S.L[5], wz[j], xy[1]) + S.t[1]);
            float pz = (float)(fma(S.L[8], wz[j], xy[2]) + S.t[2]);
            in[j] = px >= 0.0f && py >= 0.0f && pz >= 0.0f && px <= ex && py <= ey && pz <= ez;
            px = in[j] ? px : 0.0f;
            py = in[j] ? py : 0.0f;
            pz = in[j] ? pz : 0.0f;
            const int x0 = min((int)px, lx), y0 = min((int)py, ly), z0 = min((int)pz, lz);
            fx[j] = px - (float)x0;
            fy[j] = py - (float)y0;
            fz[j] = pz - (float)z0;
            if (NEAR) {
                const uint32_t o = (__umul24(__umul24(z0, S.ny) + y0, S.nx) + x0) * 4u;
                auto pair = [o](const float* d) {
                    return *reinterpret_cast<const XPair*>(reinterpret_cast<const char*>(d) + o);
                };
                p00[j] = pair(d00);
                p10[j] = pair(d10);
                p01[j] = pair(d01);
                p11[j] = pair(d11);
            } else {
                const int64_t o = ((int64_t)z0 * S.ny + y0) * S.nx + x0;
                auto pair = [o, dx](const float* d) { return XPair{d[o], d[o + dx]}; };
                p00[j] = pair(d00);
                p10[j] = pair(d10);
                p01[j] = pair(d01);
                p11[j] = pair(d11);
            }
        }
#pragma unroll
        for (int j = 0; j < POINTS; ++j) {
            const float c00 = lerp(p00[j].a, p00[j].b, fx[j]), c10 = lerp(p10[j].a, p10[j].b, fx[j]);
            const float c01 = lerp(p01[j].a, p01[j].b, fx[j]), c11 = lerp(p11[j].a, p11[j].b, fx[j]);
            const float val = lerp(lerp(c00, c10, fy[j]), lerp(c01, c11, fy[j]), fz[j]);
            out[k * 512 + v0 + j * ZSTEP * 64] = to_bf16(in[j] ? val : 0.0f);
        }
    }
}

// ---- inference head: one thread per sample, one wavefront per block --------------------------
__global__ __launch_bounds__(64) void k_ws_head(const WsHeadArgs a)
{
    const int64_t b = (int64_t)blockIdx.x * 64 + threadIdx.x;
    if (b >= a.n) return;
    float a4[CO], out[8];
#pragma unroll
    for (int c = 0; c < CO; ++c) a4[c] = silu(a.z4[b * CO + c]);
#pragma unroll
    for (int j = 0; j < 8; ++j) out[j] = ws_head_output(a, a4, j);
    double s_[3], q_[4], lg;
    ws_head_params(a, b, out, s_, q_, lg);
#pragma unroll
    for (int m = 0; m < 3; ++m) a.s_out[3 * b + m] = (float)s_[m];
#pragma unroll
    for (int m = 0; m < 4; ++m) a.q_out[4 * b + m] = (float)q_[m];
    a.logit_out[b] = (float)lg;
}

// Training targets: Sigma = R(q/|q|) diag(e^{2 s}) R^T per Gaussian in FP64, stored as
// (xx, yy, zz, xy, xz, yz).
__global__ __launch_bounds__(256) void k_ws_targets(const float* __restrict__ ls,
                                                    const float* __restrict__ quat, int64_t n,
                                                    float* __restrict__ sig6)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double q[4] = {quat[4 * i], quat[4 * i + 1], quat[4 * i + 2], quat[4 * i + 3]};
    const double qn = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    const double qh[4] = {q[0] / qn, q[1] / qn, q[2] / qn, q[3] / qn};
    double R[9];
    rot_from_q(qh, R);
    const double S2[3] = {exp(2.0 * (double)ls[3 * i]), exp(2.0 * (double)ls[3 * i + 1]),
                          exp(2.0 * (double)ls[3 * i + 2])};
    auto sig = [&](int p, int r) {
        return R[3 * p] * S2[0] * R[3 * r] + R[3 * p + 1] * S2[1] * R[3 * r + 1] +
               R[3 * p + 2] * S2[2] * R[3 * r + 2];
    };
    float* o = sig6 + 6 * i;
    o[0] = (float)sig(0, 0);
    o[1] = (float)sig(1, 1);
    o[2] = (float)sig(2, 2);
    o[3] = (float)sig(0, 1);
    o[4] = (float)sig(0, 2);
    o[5] = (float)sig(1, 2);
}

}  // namespace

hipError_t launch_ws_gather(const WsGatherArgs& a, hipStream_t s)
{
    if (a.n <= 0) return hipSuccess;
    bool near = true;
    for (const GridConst& S : a.s)
        near = near && S.nx > 1 && (int64_t)S.ny * S.nz < (1 << 24) &&
               (int64_t)S.nx * S.ny * S.nz < (1 << 30);
    auto kernel = near ? k_ws_gather<true> : k_ws_gather<false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)a.n), dim3(GATHER_THREADS), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_ws_head(const WsHeadArgs& head, hipStream_t s)
{
    hipLaunchKernelGGL(k_ws_head, dim3((unsigned)((head.n + 63) / 64)), dim3(64), 0, s, head);
    return hipGetLastError();
}

hipError_t launch_ws_targets(const float* ls, const float* quat, int64_t n, float* sig6,
                             hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_ws_targets, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, ls,
                       quat, n, sig6);
    return hipGetLastError();
}
