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
// One block per Gaussian: thread t samples the patch points t and t + 256 in every stack, so that
// the 24 reads of a point are independent.  The two x neighbours of a corner pair are one 8-byte
// read (four reads per sample instead of eight) at 32-bit offsets.  Bound by the address rate of
// the scattered reads: 3.9 ms for a million patches (one thread per sample and 64-bit indices:
// 10.4 ms), which write 3.1 GB.
struct __attribute__((packed, aligned(4))) XPair {
    float a, b;
};

__device__ __forceinline__ float lerp(float a, float b, float f) { return fmaf(1.0f - f, a, f * b); }

__global__ __launch_bounds__(256) void k_ws_gather(const WsGatherArgs a)
{
    const int64_t b = blockIdx.x;
    const float m0 = a.means[3 * b], m1 = a.means[3 * b + 1], m2 = a.means[3 * b + 2];
#pragma unroll
    for (int v = threadIdx.x; v < 512; v += 256) {
        const int z = v / 64, y = (v / 8) % 8, x = v % 8;
        const float wx = fmaf(a.spacing, (float)x - 3.5f, m0);
        const float wy = fmaf(a.spacing, (float)y - 3.5f, m1);
        const float wz = fmaf(a.spacing, (float)z - 3.5f, m2);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const GridConst& S = a.s[k];
            auto index = [&](int r) {
                return (float)(fma(S.L[3 * r + 2], (double)wz,
                                   fma(S.L[3 * r], (double)wx, S.L[3 * r + 1] * (double)wy)) +
                               S.t[r]);
            };
            const float px = index(0), py = index(1), pz = index(2);
            float val = 0.0f;
            if (px >= 0.0f && py >= 0.0f && pz >= 0.0f && px <= (float)(S.nx - 1) &&
                py <= (float)(S.ny - 1) && pz <= (float)(S.nz - 1)) {
                const int x0 = min((int)px, max(S.nx - 2, 0)), y0 = min((int)py, max(S.ny - 2, 0)),
                          z0 = min((int)pz, max(S.nz - 2, 0));
                const int y1 = min(y0 + 1, S.ny - 1), z1 = min(z0 + 1, S.nz - 1);
                const float fx = px - (float)x0, fy = py - (float)y0, fz = pz - (float)z0;
                const float* d = a.data[k];
                XPair p00, p10, p01, p11;      // (y0, z0), (y1, z0), (y0, z1), (y1, z1)
                const int r00 = (z0 * S.ny + y0) * S.nx + x0, r10 = (z0 * S.ny + y1) * S.nx + x0;
                const int r01 = (z1 * S.ny + y0) * S.nx + x0, r11 = (z1 * S.ny + y1) * S.nx + x0;
                if (S.nx > 1) {                // x0 + 1 lies in the stack
                    p00 = *reinterpret_cast<const XPair*>(d + r00);
                    p10 = *reinterpret_cast<const XPair*>(d + r10);
                    p01 = *reinterpret_cast<const XPair*>(d + r01);
                    p11 = *reinterpret_cast<const XPair*>(d + r11);
                } else {
                    p00 = XPair{d[r00], d[r00]};
                    p10 = XPair{d[r10], d[r10]};
                    p01 = XPair{d[r01], d[r01]};
                    p11 = XPair{d[r11], d[r11]};
                }
                const float c00 = lerp(p00.a, p00.b, fx), c10 = lerp(p10.a, p10.b, fx);
                const float c01 = lerp(p01.a, p01.b, fx), c11 = lerp(p11.a, p11.b, fx);
                val = lerp(lerp(c00, c10, fy), lerp(c01, c11, fy), fz);
            }
            a.patches[(b * 3 + k) * 512 + v] = to_bf16(val);
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
    hipLaunchKernelGGL(k_ws_gather, dim3((unsigned)a.n), dim3(256), 0, s, a);
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
