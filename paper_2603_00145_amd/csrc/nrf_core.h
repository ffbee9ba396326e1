// Device code of the neural residual field (Sec. 3.4, Eq. 8) shared by the field's own kernels
// and by the renderer's fused epilogue: BF16 operands on gfx950's 16x16x32 MFMA with FP32
// accumulation, the sinusoidal encoding computed in the MFMA operand layout, weights staged in
// LDS in operand order, and the forward of one 16-point tile kept in registers.
#ifndef GM_NRF_CORE_H
#define GM_NRF_CORE_H
#include "gm_internal.h"

namespace nrfcore {

typedef short v4s __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int W = 64;          // hidden width (fixed); in_pad is 64 or 128, depth 1..4

// float -> bfloat16 bits, round to nearest even (gfx950's v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint16_t to_bf16(float f)
{
    return __builtin_bit_cast(uint16_t, (__bf16)f);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

// four floats -> BF16 bits, round to nearest even, two per v_cvt_pk_bf16_f32
__device__ __forceinline__ v4s pack4(float a, float b, float c, float d)
{
    const uint32_t lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{a, b}, v2bf));
    const uint32_t hi = __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{c, d}, v2bf));
    return __builtin_bit_cast(v4s, (uint64_t)lo | ((uint64_t)hi << 32));
}

typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// gfx950's 16x16x32 BF16 MFMA on two 16-wide K halves: lane group g supplies, in A and in B
// alike, slots 4 g + j of the first half (a0, b0) and of the second (a1, b1), so the sum runs
// over all 32 slots whatever order the hardware gives them.  A 16x16x16 operand tile of each
// half is used unchanged, and the result has the 16x16x16 layout (lane group g: rows 4 g + j).
__device__ __forceinline__ v4f mfma2(v4s a0, v4s a1, v4s b0, v4s b1, v4f c)
{
    const v8bf a = __builtin_bit_cast(v8bf, __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7));
    const v8bf b = __builtin_bit_cast(v8bf, __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7));
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

typedef short v8h __attribute__((ext_vector_type(8)));

// the same with both halves of A in one operand
__device__ __forceinline__ v4f mfma_a8(v8h a, v4s b0, v4s b1, v4f c)
{
    const v8bf b = __builtin_bit_cast(v8bf, __builtin_shufflevector(b0, b1, 0, 1, 2, 3, 4, 5, 6, 7));
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), b, c, 0, 0, 0);
}

// sigmoid with the hardware reciprocal (1 ulp; the field runs in BF16): exp(-z) overflows to
// +inf for very negative z, whose reciprocal is 0, the right limit
__device__ __forceinline__ float sigm(float z) { return __builtin_amdgcn_rcpf(1.0f + __expf(-z)); }
__device__ __forceinline__ float silu(float z) { return z * sigm(z); }
// SiLU'(z) from z and its sigmoid
__device__ __forceinline__ float dsilu(float z, float s) { return s * (1.0f + z * (1.0f - s)); }
__device__ __forceinline__ float dsilu(float z) { return dsilu(z, sigm(z)); }

// World coordinate of voxel (vx, vy, vz): binary64 without contraction (hipcc fuses a * b + c
// by default, the pragma stops it here), rounded once to binary32.
__device__ __forceinline__ float world_coord(const double* M, int vx, int vy, int vz)
{
#pragma clang fp contract(off)
    double s = M[0] * (double)vx;
    s = s + M[1] * (double)vy;
    s = s + M[2] * (double)vz;
    s = s + M[3];
    return (float)s;
}

// Order of the encoding along the first layer's K dimension on the GPU.  The MFMA B operand of
// K-tile t gives lane group g = lane / 16 the features 16 t + 4 g + j, j < 4; call c = 4 t + j
// the column of that slot.  The last column holds the raw coordinates (x[g] for g < 3, else
// padding); column c = 6 q + m holds frequency band 4 q + g of kind m (sin of axis m for m < 3,
// cos of axis m - 3).  Kind, axis and band offset are compile-time constants of the unrolled
// encoding loop and the lane group only shifts the band, so nothing per slot has to be looked
// up or kept in registers.  The first layer's weights are permuted into this order when they
// are staged and its weight gradient is permuted back.  Bands: up to 8 with 4 K-tiles, 20 with 8.
template <int KT>
__host__ __device__ constexpr int max_bands() { return 4 * ((4 * KT - 1) / 6); }

// natural feature index (x_a: a; sin(2^k pi x_a): 3 + 6 k + a; cos: 6 + 6 k + a) of GPU slot
// i = 16 t + 4 g + j, or -1 for padding
template <int KT>
__device__ __forceinline__ int natural_feature(int i, int n_freq)
{
    const int t = i >> 4, g = (i >> 2) & 3, j = i & 3, c = 4 * t + j;
    if (c == 4 * KT - 1) return g < 3 ? g : -1;
    const int q = c / 6, m = c - 6 * q, band = 4 * q + g;
    return band < n_freq ? 3 + 6 * band + m : -1;
}

// The encoding of the lane's point, in the B operand layout of the K-tiles.  Slots of bands past
// n_freq hold any finite value: their weights are staged as zeros and their weight gradients
// dropped (the lane groups of a band group that n_freq cuts are not masked, a band group past it
// is left out).
template <int KT>
__device__ __forceinline__ void encode(const float x[3], int n_freq, v4s b0[KT])
{
    const int g = (threadIdx.x >> 4) & 3;
    float v[4 * KT];
#pragma unroll
    for (int c = 0; c < 4 * KT - 1; ++c) v[c] = 0.0f;
    v[4 * KT - 1] = g == 0 ? x[0] : g == 1 ? x[1] : g == 2 ? x[2] : 0.0f;
#pragma unroll
    for (int q = 0; q < max_bands<KT>() / 4; ++q) {
        if (q > 0 && 4 * q >= n_freq) continue;   // uniform
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const float phi = ldexpf(x[a], 4 * q - 1 + g);        // exact power-of-two scaling
            const float frac = phi - rintf(phi);                  // exact
            // v_sin_f32 / v_cos_f32 take their argument in revolutions
            v[6 * q + a] = __builtin_amdgcn_sinf(frac);
            v[6 * q + 3 + a] = __builtin_amdgcn_cosf(frac);
        }
    }
#pragma unroll
    for (int t = 0; t < KT; ++t) b0[t] = pack4(v[4 * t], v[4 * t + 1], v[4 * t + 2], v[4 * t + 3]);
}

// Weights staged in LDS in MFMA A-operand order: operand (o, u) of a layer, K-tiles 2 u and 2 u + 1, is
// 64 lanes x 8 BF16, lane (g, row) holding W[16 o + row][32 u + 4 g + j] and [.. + 16], so that a
// wavefront reads an operand as 1 KB of consecutive 16-byte pieces.  (As two 8-byte pieces the reads
// came paired across operands, and 28 moves a tile put the halves together: with those gone and
// the biases in LDS, the field on a 256^3 volume went from 1600 to 1554 us, on three 256x256x64
// stacks from 1427 to 1390.)  Sized for KT K-tiles of the first layer and DEPTH - 1 hidden layers.
template <int KT, int DEPTH>
struct Lds {
    v8h w_in[2 * KT * 64];                                 // [o][u][lane], GPU encoding order
    v8h w_hid[(DEPTH > 1 ? DEPTH - 1 : 1) * 8 * 64];       // [l][o][u][lane]
};

// Stages the weights (every thread of the block takes part; ends with a block barrier).
// SWZ: within an operand of a hidden layer lane (g, row)'s piece is stored at row ^ 4 g, so that the
// transposing reads of the backward find 16 pieces of every lane group in different banks too.
template <int KT, int DEPTH, bool SWZ = false>
__device__ void load_weights(const NrfArgs& a, Lds<KT, DEPTH>& s)
{
    constexpr int U = KT / 2;
    for (int e = threadIdx.x; e < 4 * U * 64; e += blockDim.x) {
        const int lane = e & 63, u = (e >> 6) % U, o = (e >> 6) / U;
        const int g = lane >> 4, row = lane & 15;
        const uint16_t* src = a.w_in + (16 * o + row) * (16 * KT);
        v8h v;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int nf = natural_feature<KT>(32 * u + 16 * (j >> 2) + 4 * g + (j & 3), a.n_freq);
            v[j] = nf >= 0 ? (short)src[nf] : (short)0;
        }
        s.w_in[e] = v;
    }
    const int nh = (DEPTH - 1) * 8 * 64;
    for (int e = threadIdx.x; e < nh; e += blockDim.x) {
        const int lane = e & 63, u = (e >> 6) & 1, o = (e >> 7) & 3, l = e >> 9;
        const int g = lane >> 4, row = lane & 15;
        const uint16_t* src = a.w_hid + l * W * W + (16 * o + row) * W + 32 * u + 4 * g;
        v8h v;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = (short)src[16 * (j >> 2) + (j & 3)];
        s.w_hid[SWZ ? e ^ (4 * g) : e] = v;
    }
    __syncthreads();
}

// (x, y, z) of voxel v (grids hold < 2^31 voxels, so 32-bit division suffices)
__device__ __forceinline__ void voxel_xyz(uint32_t v, uint32_t nx, uint32_t ny, int* vx, int* vy,
                                          int* vz)
{
    const uint32_t q = v / nx;
    *vx = (int)(v - q * nx);
    const uint32_t r = q / ny;
    *vy = (int)(q - r * ny);
    *vz = (int)r;
}
__device__ __forceinline__ void point_xyz(const NrfArgs& a, int64_t p, int* vx, int* vy, int* vz)
{
    voxel_xyz(a.idx ? (uint32_t)a.idx[p] : (uint32_t)p, (uint32_t)a.nx, (uint32_t)a.ny, vx, vy, vz);
}

// Forward for the 16 points of a tile, in the register layout o-tile x 4 features of point
// lane & 15: the encoding (GPU order) and the BF16 activations, and for the backward SiLU' of
// every pre-activation (not formed where it is not used).
template <int KT, int DEPTH>
struct Tile {
    v4s enc[KT];
    v4s act[DEPTH][4];
    v4f d[DEPTH][4];
    __device__ __forceinline__ void layer(int l, int o, v4f z)
    {
        const v4f s = {sigm(z.x), sigm(z.y), sigm(z.z), sigm(z.w)};
        act[l][o] = pack4(z.x * s.x, z.y * s.y, z.z * s.z, z.w * s.w);
        d[l][o] = v4f{dsilu(z.x, s.x), dsilu(z.y, s.y), dsilu(z.z, s.z), dsilu(z.w, s.w)};
    }
};

// the lane's four biases of o-tile o of layer l
__device__ __forceinline__ v4f global_bias(const NrfArgs& a, int l, int o)
{
    const int f = 16 * o + 4 * ((threadIdx.x >> 4) & 3);
    const float* b = l == 0 ? a.b_in : a.b_hid + (l - 1) * W;
    return v4f{b[f], b[f + 1], b[f + 2], b[f + 3]};
}
// Where tile_forward_w takes the layers' MFMA A operands from: the LDS stage, read at each use,
// or the wavefront's registers (each lane its piece of every operand, 2 KT + 8 (DEPTH - 1)
// pieces, copied once from the stage; the per-tile LDS reads of the weights, 512 bytes per lane,
// then disappear).
template <int KT, int DEPTH>
struct WeightsLds {
    const Lds<KT, DEPTH>& s;
    const v4f* b;                  // biases, [l][4 o + g]
    int lane;
    __device__ v4f bias(const NrfArgs&, int l, int o) const { return b[16 * l + 4 * o + (lane >> 4)]; }
    __device__ v8h in(int o, int u) const { return s.w_in[(o * (KT / 2) + u) * 64 + lane]; }
    __device__ v8h hid(int l, int o, int u) const
    {
        return s.w_hid[((l - 1) * 8 + o * 2 + u) * 64 + lane];
    }
};
template <int KT, int DEPTH>
struct WeightsReg {
    v8h w_in[2 * KT];
    v8h w_hid[(DEPTH > 1 ? DEPTH - 1 : 1) * 8];
    __device__ void load(const Lds<KT, DEPTH>& s, int lane)
    {
#pragma unroll
        for (int i = 0; i < 2 * KT; ++i) w_in[i] = s.w_in[i * 64 + lane];
#pragma unroll
        for (int i = 0; i < (DEPTH - 1) * 8; ++i) w_hid[i] = s.w_hid[i * 64 + lane];
    }
    __device__ v4f bias(const NrfArgs& a, int l, int o) const { return global_bias(a, l, o); }
    __device__ v8h in(int o, int u) const { return w_in[o * (KT / 2) + u]; }
    __device__ v8h hid(int l, int o, int u) const { return w_hid[(l - 1) * 8 + o * 2 + u]; }
};

template <int KT, int DEPTH, typename WS>
__device__ __forceinline__ void tile_forward_w(const NrfArgs& a, const WS& ws, const float x[3],
                                               Tile<KT, DEPTH>& T)
{
    encode<KT>(x, a.n_freq, T.enc);
    // layer 1
#pragma unroll
    for (int o = 0; o < 4; ++o) {
        v4f acc = ws.bias(a, 0, o);   // bias as C
#pragma unroll
        for (int t = 0; t < KT; t += 2)
            acc = mfma_a8(ws.in(o, t / 2), T.enc[t], T.enc[t + 1], acc);
        T.layer(0, o, acc);
    }
    // hidden layers
#pragma unroll
    for (int l = 1; l < DEPTH; ++l) {
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            v4f acc = ws.bias(a, l, o);
#pragma unroll
            for (int t = 0; t < 4; t += 2)
                acc = mfma_a8(ws.hid(l, o, t / 2), T.act[l - 1][t], T.act[l - 1][t + 1], acc);
            T.layer(l, o, acc);
        }
    }
}

// Stages the biases for WeightsLds: quad e of 16 DEPTH by thread e (of at least that many)
template <int DEPTH>
__device__ __forceinline__ void load_biases(const NrfArgs& a, v4f* b, int e)
{
    if (e < 16 * DEPTH) {
        const float* q = e < 16 ? a.b_in + 4 * e : a.b_hid + 4 * (e - 16);
        b[e] = v4f{q[0], q[1], q[2], q[3]};
    }
}

// The output layer as a 16-row MFMA A operand whose rows 0, 4, 8 and 12 are w_out and the other
// rows zero: lane (g, row) of those rows holds w_out[16 t + 4 g + j] of K-tile t.  Loaded once
// per wavefront.
__device__ __forceinline__ void load_wout(const NrfArgs& a, v4s (&wo)[4])
{
    const int lane = threadIdx.x & 63, g = lane >> 4, row = lane & 15;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const v4s v = *reinterpret_cast<const v4s*>(a.w_out + 16 * t + 4 * g);
        wo[t] = (row & 3) == 0 ? v : v4s{0, 0, 0, 0};
    }
}

// output pre-activation z_o of the tile's point from the BF16 activations of the last layer,
// on the matrix cores (wo from load_wout): row 4 g of the product, held by lane group g, is
// w_out . a_D for the lane's point.
template <int KT, int DEPTH>
__device__ __forceinline__ float tile_output(const NrfArgs& a, const Tile<KT, DEPTH>& T,
                                             const v4s (&wo)[4])
{
    v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
    acc = mfma2(wo[0], wo[1], T.act[DEPTH - 1][0], T.act[DEPTH - 1][1], acc);
    acc = mfma2(wo[2], wo[3], T.act[DEPTH - 1][2], T.act[DEPTH - 1][3], acc);
    return acc.x + a.b_out[0];
}

// Grid of a tile loop: every block resident at once (the blocks then take equal shares of the
// tiles, with no partial last wave of blocks), capped by the work.
template <typename K>
inline unsigned blocks_for_tiles(K kernel, int64_t ntiles)
{
    int dev = 0, cus = 0, per_cu = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, 0);
    int64_t full = (int64_t)(cus > 0 ? cus : 256) * (per_cu > 0 ? per_cu : 1);
    int64_t b = (ntiles + 3) / 4;
    if (b > full) b = full;
    if (b < 1) b = 1;
    return (unsigned)b;
}

}  // namespace nrfcore

// supported shapes: in_pad 64 or 128 (4 or 8 K-tiles; at most max_bands<KT>() bands), depth 1..4
#define GM_NRF_DISPATCH(FN, ...)                                                           \
    switch ((a.in_pad >> 4) * 8 + a.depth) {                                               \
    case 4 * 8 + 1: FN<4, 1>(__VA_ARGS__); break;                                          \
    case 4 * 8 + 2: FN<4, 2>(__VA_ARGS__); break;                                          \
    case 4 * 8 + 3: FN<4, 3>(__VA_ARGS__); break;                                          \
    case 4 * 8 + 4: FN<4, 4>(__VA_ARGS__); break;                                          \
    case 8 * 8 + 1: FN<8, 1>(__VA_ARGS__); break;                                          \
    case 8 * 8 + 2: FN<8, 2>(__VA_ARGS__); break;                                          \
    case 8 * 8 + 3: FN<8, 3>(__VA_ARGS__); break;                                          \
    case 8 * 8 + 4: FN<8, 4>(__VA_ARGS__); break;                                          \
    default: return hipErrorInvalidValue;                                                  \
    }

#endif
