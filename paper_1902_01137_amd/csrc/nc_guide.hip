// nc_guide.hip -- the learned proposal: an MLP from a scattering vertex
// (normalised position, incoming direction, log extinction) to a mixture of
// von Mises-Fisher lobes over the outgoing direction, trained on the
// tracer's own vertices by weighted maximum likelihood.
//
// Network 15 -> 64 -> 64 -> 64 -> 40 (8 lobes x (logit, mean direction 3,
// log concentration)), ReLU on hidden layers; its inputs are a vertex's 7
// values and 8 Fourier features of its horizontal position (guide_feature).  Products run on the matrix
// cores (v_mfma_f32_16x16x16_bf16: bf16 operands, fp32 accumulation); master
// weights, Adam moments and gradients are fp32.  Padded layer shapes (in x
// out): 16x64, 64x64, 64x64, 64x48.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "nc_internal.hpp"

namespace nc {

// ---------------------------------------------------------------------------
// Shapes and parameter layout (flat fp32, per layer W [out][in] row-major
// then b [out]; the same order as the oracle's)
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int guide_in(int l) { return l == 0 ? kGuideIn : kGuideWidth; }
__host__ __device__ constexpr int guide_out(int l) { return l == kGuideLayers - 1 ? kGuideOut : kGuideWidth; }
__host__ __device__ constexpr int guide_in_pad(int l) { return l == 0 ? 16 : kGuideWidth; }
__host__ __device__ constexpr int guide_out_pad(int l) { return l == kGuideLayers - 1 ? 48 : kGuideWidth; }

// ---------------------------------------------------------------------------
// The network on a tile of 16 records, by one wave.  Every layer's product is
// taken as (weights) x (activations)^T, so that a lane (mrow = lane % 16, kq =
// lane / 16) ends with four consecutive units, 16 nt + 4 kq + i, of record mrow:
// one 8-byte store makes them the next layer's operand, a row of LDS per record.
// The weights stay in registers (96 of them) for all the tiles of a wave.
// ---------------------------------------------------------------------------
constexpr int kRow = kGuideWidth + 8;   // shorts per record's row of LDS (16-byte steps, rows in different banks)

struct GuideFrags {
    bf16x4 w0[4], w1[4][4], w2[4][4], w3[3][4];   // [output tile][k tile]
};

constexpr int kFragRows = 3 * kGuideWidth + 48;   // rows of W_0..W_3 in LDS, kRow shorts each

// The workgroup's (256 threads) copy of the weights through LDS: every wave
// needs all of them, and from L2 each would fetch them again.  Ends with the
// last read, before a barrier the caller has anyway.
__device__ __attribute__((always_inline)) inline void load_frags(const GuideWeights &W, short (*lds)[kRow], GuideFrags &F)
{
    const int tid = threadIdx.x, mrow = tid & 15, kq = (tid >> 4) & 3;
    constexpr int first[kGuideLayers] = {0, kGuideWidth, 2 * kGuideWidth, 3 * kGuideWidth};
#pragma unroll
    for (int layer = 0; layer < kGuideLayers; ++layer) {
        const int per = guide_in_pad(layer) / 8, count = guide_out_pad(layer) * per;   // 16-byte pieces
        for (int e = tid; e < count; e += 256)
            *reinterpret_cast<uint4 *>(&lds[first[layer] + e / per][8 * (e % per)]) =
                reinterpret_cast<const uint4 *>(W.w[layer])[e];
    }
    __syncthreads();
    auto frag = [&](int layer, int nt, int kt) __attribute__((always_inline)) {
        return *reinterpret_cast<const bf16x4 *>(&lds[first[layer] + nt * 16 + mrow][kt * 16 + 4 * kq]);
    };
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        F.w0[nt] = frag(0, nt, 0);
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
            F.w1[nt][kt] = frag(1, nt, kt);
            F.w2[nt][kt] = frag(2, nt, kt);
            if (nt < 3) F.w3[nt][kt] = frag(3, nt, kt);
        }
    }
}

// A lane's share of a record: the vertex's x and y, and the raw values that are its inputs 4 kq + i.
struct TileRecord {
    float x, y, raw[4];
};

__device__ __attribute__((always_inline)) inline TileRecord load_record(const float *q, int kq)
{
    TileRecord t;
    t.x = q[0];
    t.y = q[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) t.raw[i] = q[min(4 * kq + i, kGuideRaw - 1)];
    return t;
}

// the four network inputs 4 kq + i (as guide_feature; zero for a record that is none)
__device__ __attribute__((always_inline)) inline bf16x4 tile_inputs(const TileRecord &t, bool ok, int kq)
{
    bf16x4 b;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int k = 4 * kq + i, j = k - kGuideRaw;
        const float v = ((j >> 1) & 1 ? t.y : t.x) * (j < 4 ? 4.0f : 8.0f);
        const float f = (j & 1) ? __builtin_amdgcn_cosf(v) : __builtin_amdgcn_sinf(v);
        b[i] = to_bf16(!ok | (k >= kGuideIn) ? 0.0f : k < kGuideRaw ? t.raw[i] : f);
    }
    return b;
}

__device__ inline void lds_order()
{
    // (lanes of one wave: LDS operations complete in order; this keeps the compiler to it)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// bias: [layer][64] in LDS; act: the wave's 16 rows of kRow shorts; z: the raw outputs of tiles 0..2.
__device__ __attribute__((always_inline)) inline void tile_forward(const GuideFrags &F, const float (*bias)[kGuideWidth],
                                                                   short *act, bf16x4 x, int mrow, int kq, f32x4 z[3])
{
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    short *row = act + mrow * kRow + 4 * kq;
    bf16x4 b[4];
    auto finish = [&](int layer, int nt, const f32x4 &c) __attribute__((always_inline)) {
        const float4 bs = *reinterpret_cast<const float4 *>(&bias[layer][16 * nt + 4 * kq]);
        const bf16x4 h = {to_bf16(fmaxf(c[0] + bs.x, 0.0f)), to_bf16(fmaxf(c[1] + bs.y, 0.0f)),
                          to_bf16(fmaxf(c[2] + bs.z, 0.0f)), to_bf16(fmaxf(c[3] + bs.w, 0.0f))};
        *reinterpret_cast<bf16x4 *>(row + 16 * nt) = h;
    };
    auto next = [&]() __attribute__((always_inline)) {
        lds_order();
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) b[kt] = *reinterpret_cast<const bf16x4 *>(row + 16 * kt);
        lds_order();
    };
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) finish(0, nt, mfma16(F.w0[nt], x, zero));
    next();
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        f32x4 c = zero;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) c = mfma16(F.w1[nt][kt], b[kt], c);
        finish(1, nt, c);
    }
    next();
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        f32x4 c = zero;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) c = mfma16(F.w2[nt][kt], b[kt], c);
        finish(2, nt, c);
    }
    next();
#pragma unroll
    for (int nt = 0; nt < 3; ++nt) {
        f32x4 c = zero;
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) c = mfma16(F.w3[nt][kt], b[kt], c);
        const float4 bs = *reinterpret_cast<const float4 *>(&bias[3][16 * nt + 4 * kq]);
        z[nt] = f32x4{c[0] + bs.x, c[1] + bs.y, c[2] + bs.z, c[3] + bs.w};
    }
}

// four floats at any float's address
struct __attribute__((packed, aligned(4))) Float4Any {
    float v[4];
};

// X: records as rows of `rec_stride` floats, the vertex's 7 values first (the 15
// network inputs are formed from them); Z: n x 48 raw outputs, fp32.
// Bound by latency below some 10^4 records and by LDS and matrix core issue above;
// with a wave per workgroup that fetched its weights from L2 for every tile,
// 131072 records took 64 us and 10^6 352 us, now 18 and 72 (152 registers: three
// workgroups a CU).
__global__ __launch_bounds__(256) void guide_forward_kernel(GuideWeights W, const float *__restrict__ X, int n,
                                                            int rec_stride, float *__restrict__ Z)
{
    __shared__ __align__(16) float bias[kGuideLayers][kGuideWidth];
    __shared__ __align__(16) short lds[kFragRows][kRow];   // the weights, then each wave's 16 rows
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, mrow = lane & 15, kq = lane >> 4;
    if (lane < guide_out_pad(wv)) bias[wv][lane] = W.b[wv][lane];   // (a wave per layer)
    GuideFrags F;
    load_frags(W, lds, F);
    __syncthreads();
    for (long long r0 = ((long long)blockIdx.x * 4 + wv) * 16; r0 < n; r0 += (long long)gridDim.x * 64) {
        const long long r = r0 + mrow;
        const bool ok = r < n;
        f32x4 z[3];
        const TileRecord t = load_record(X + (size_t)(ok ? r : 0) * rec_stride, kq);
        tile_forward(F, bias, &lds[16 * wv][0], tile_inputs(t, ok, kq), mrow, kq, z);
        lds_order();
        if (ok) {
#pragma unroll
            for (int nt = 0; nt < 3; ++nt)
                *reinterpret_cast<Float4Any *>(Z + (size_t)r * 48 + 16 * nt + 4 * kq) =
                    Float4Any{{z[nt][0], z[nt][1], z[nt][2], z[nt][3]}};
        }
    }
}

// ---------------------------------------------------------------------------
// Mixture of vMF lobes from the raw outputs of one record.
// ---------------------------------------------------------------------------
__device__ inline float vmf_norm(float kappa)
{
    // kappa / (2 pi (1 - exp(-2 kappa)))
    return kappa / (2.0f * kPi * (-expm1f(-2.0f * kappa)));
}

__global__ void weight_sum_kernel(const float *__restrict__ rec, int n, int rec_stride, double *out)
{
    double s = 0.0;
    for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < n; r += gridDim.x * blockDim.x)
        s += (double)rec[(size_t)r * rec_stride + 10];
    __shared__ double red[256];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int s2 = blockDim.x / 2; s2 > 0; s2 >>= 1) {
        if ((int)threadIdx.x < s2) red[threadIdx.x] += red[threadIdx.x + s2];
        __syncthreads();
    }
    if (threadIdx.x == 0) unsafeAtomicAdd(out, red[0]);
}

// ---------------------------------------------------------------------------
// Forward, loss and backward over one chunk of records per workgroup (4 waves),
// 64 records at a time, with nothing in memory between them.  Forward: a wave
// computes its 16 outputs of every layer, for all 64 records.  Loss
//   L = -sum w ln q / sum w, q = sum_j pi_j vmf(mu_j, kappa_j; w_out)
// and d loss / d outputs: a wave its 16 records, two lobes a lane.  Backward, from
// the last layer to the first: the weight gradient dW_l += dZ_l^T Hin_l (the records
// are the product's k) and, for l > 0, dZ_{l-1} = (dZ_l W_l) masked by the ReLU of
// H_{l-1}, both on the matrix cores.  A wave keeps its share of the weight-gradient
// tiles in registers over the whole chunk: layer 3 tiles (o-tile 0..2, i-tile =
// wave), layers 2 and 1 (o-tile 0..3, i-tile = wave), layer 0 (o-tile = wave).  At
// the end every sum is written once to the workgroup's row of `part` (no atomics;
// the Adam kernel adds the rows).  Rounding is as if the layers were kernels of
// their own: activations, inputs and dZ to bf16 where a product takes them, outputs,
// loss, sums and gradients in fp32.
// Bound by the latency of each 64 records' chain through the layers (of 19 k cycles
// the loss takes 5 k, a layer 1 to 3 k) at the two workgroups a CU that 250 registers
// leave.  131072 records: 65 us, where the forward, loss and backward kernels with
// activations in memory took 66, 29 and 80 us.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int guide_param_off(int l)
{
    return l == 0 ? 0 : guide_param_off(l - 1) + guide_out(l - 1) * guide_in(l - 1) + guide_out(l - 1);
}
static_assert(guide_param_off(kGuideLayers) == kGuideParams, "parameter layout");

// A workgroup's row of partial sums: the weight-gradient tiles as the matrix
// cores leave them (lane, then its four outputs o = 16 ot + 4 kq + j of input 16 it +
// mrow: a tile is one store of 16 bytes a lane, where rows in the parameters' order
// took four of 4 bytes in 64-byte pieces), then the biases [layer][64].
constexpr int kPartTiles = 4 + 16 + 16 + 12;
constexpr int kPartRow = kPartTiles * 256 + kGuideLayers * kGuideWidth;
__host__ __device__ constexpr int part_tile(int L, int ot, int it)
{
    return L == 0 ? ot : 4 + 16 * (L - 1) + 4 * ot + it;
}
// the parameter at position e of a row (-1: padding)
__device__ inline int part_param(int e)
{
    if (e >= kPartTiles * 256) {
        const int L = (e - kPartTiles * 256) / kGuideWidth, o = (e - kPartTiles * 256) % kGuideWidth;
        return o < guide_out(L) ? guide_param_off(L) + guide_out(L) * guide_in(L) + o : -1;
    }
    const int tile = e >> 8, lane = (e >> 2) & 63, j = e & 3;
    const int L = tile < 4 ? 0 : 1 + (tile - 4) / 16, k = tile < 4 ? tile : (tile - 4) % 16;
    const int ot = L == 0 ? k : k >> 2, it = L == 0 ? 0 : k & 3;
    const int o = 16 * ot + 4 * (lane >> 4) + j, i = 16 * it + (lane & 15);
    return o < guide_out(L) && i < guide_in(L) ? guide_param_off(L) + o * guide_in(L) + i : -1;
}

// (rows by record; a product over the records reads them by column, col_frag)
struct TrainLds {
    short h[3][64][kRow];               // hidden activations H0..H2
    short dz[2][64][kRow];              // d loss / d raw outputs and down the layers (current, next)
    float z[64][52];                    // raw outputs
    short x[64][24];                    // network inputs
    float bias[kGuideLayers][kGuideWidth];
};
static_assert(sizeof(TrainLds) <= 80 * 1024, "two workgroups a CU");

// Records 4 kq + (0..3) of column c0 + mrow, from the 16 rows at `rows`: the
// transposing LDS read gives a lane, of the 16 eight-byte pieces that its group of
// 16 lanes addresses, element mrow % 4 of pieces mrow / 4 + (0, 4, 8, 12).
template <int kStride>
__device__ __attribute__((always_inline)) inline bf16x4 col_frag(const short (*rows)[kStride], int c0, int mrow, int kq)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (__attribute__((address_space(3))) bf16x4 *)&rows[4 * kq + (mrow >> 2)][c0 + 4 * (mrow & 3)]);
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void
guide_train_kernel(GuideWeights W, const float *__restrict__ rec, int rec_stride, int n, int chunk,
                   const double *__restrict__ wsum, float *__restrict__ part, double *__restrict__ loss)
{
    __shared__ __align__(16) TrainLds S;
    const int tid = threadIdx.x, wv = tid >> 6, lane = tid & 63;
    const int mrow = lane & 15, kq = lane >> 4;
    if (lane < guide_out_pad(wv)) S.bias[wv][lane] = W.b[wv][lane];   // (a wave per layer)
    // the wave's output tile of each layer (the last one has three)
    auto frag = [&](int layer, int kt) __attribute__((always_inline)) {
        return *reinterpret_cast<const bf16x4 *>(W.w[layer] + (16 * wv + mrow) * guide_in_pad(layer) + 16 * kt + 4 * kq);
    };
    bf16x4 f0 = frag(0, 0), f1[4], f2[4], f3[4];
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
        f1[kt] = frag(1, kt);
        f2[kt] = frag(2, kt);
        f3[kt] = bf16x4{0, 0, 0, 0};
        if (wv < 3) f3[kt] = frag(3, kt);
    }
    // the backward products' operand: W_l^T, input 16 wv + mrow, outputs 16 kt + 4 kq + (0..3)
    bf16x4 t3[3], t2[4], t1[4];
#pragma unroll
    for (int kt = 0; kt < 4; ++kt) {
        const int i = 16 * wv + mrow, o = 16 * kt + 4 * kq;
        if (kt < 3) t3[kt] = *reinterpret_cast<const bf16x4 *>(W.wt[3] + i * guide_out_pad(3) + o);
        t2[kt] = *reinterpret_cast<const bf16x4 *>(W.wt[2] + i * guide_out_pad(2) + o);
        t1[kt] = *reinterpret_cast<const bf16x4 *>(W.wt[1] + i * guide_out_pad(1) + o);
    }
    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 g3[3], g2[4], g1[4], g0 = zero;
    // bias sums: of the lane's outputs (two lobes) over its records, and of units 16 wv + 4 kq + j over records mrow
    float b3[10] = {}, b2[4] = {}, b1[4] = {}, b0[4] = {};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        if (t < 3) g3[t] = zero;
        g2[t] = zero, g1[t] = zero;
    }
    const float inv_w = (float)(1.0 / wsum[0]);
    const int rbeg = blockIdx.x * chunk, rend = min(n, rbeg + chunk);
    const int mine = 16 * wv + mrow;      // the lane's record of the 64
    double li = 0.0;
    // the record of the next 64 is on its way while these are worked on
    TileRecord next;
    float wo_next[4];
    auto fetch = [&](int first) __attribute__((always_inline)) {
        const float *q = rec + (size_t)(first + min(mine, n - 1 - first)) * rec_stride;
        next = load_record(q, kq);
#pragma unroll
        for (int a = 0; a < 4; ++a) wo_next[a] = q[7 + a];
    };
    fetch(rbeg);
    for (int r0 = rbeg; r0 < rend; r0 += 64) {
        __syncthreads();   // the records before are done with the LDS
        {
            const bool ok = r0 + mine < rend;
            const bf16x4 x = tile_inputs(next, ok, kq);
            const float wo[3] = {wo_next[0], wo_next[1], wo_next[2]};
            const float wr = wo_next[3];
            if (r0 < n - 64) fetch(r0 + 64);
            *reinterpret_cast<bf16x4 *>(&S.x[mine][4 * kq]) = x;
            // the forward layers, a wave its 16 outputs of all 64 records: as (weights) x
            // (activations)^T, so that a lane ends with four units of one record
            auto units = [&](int layer, int t, const f32x4 &c) __attribute__((always_inline)) {
                const float4 bs = *reinterpret_cast<const float4 *>(&S.bias[layer][16 * wv + 4 * kq]);
                *reinterpret_cast<bf16x4 *>(&S.h[layer][16 * t + mrow][16 * wv + 4 * kq]) =
                    bf16x4{to_bf16(fmaxf(c[0] + bs.x, 0.0f)), to_bf16(fmaxf(c[1] + bs.y, 0.0f)),
                           to_bf16(fmaxf(c[2] + bs.z, 0.0f)), to_bf16(fmaxf(c[3] + bs.w, 0.0f))};
            };
            auto product = [&](const bf16x4 f[4], int t, short (*in)[kRow]) __attribute__((always_inline)) {
                f32x4 c = zero;
#pragma unroll
                for (int kt = 0; kt < 4; ++kt)
                    c = mfma16(f[kt], *reinterpret_cast<const bf16x4 *>(&in[16 * t + mrow][16 * kt + 4 * kq]), c);
                return c;
            };
            __syncthreads();
#pragma unroll
            for (int t = 0; t < 4; ++t)
                units(0, t, mfma16(f0, *reinterpret_cast<const bf16x4 *>(&S.x[16 * t + mrow][4 * kq]), zero));
            __syncthreads();
#pragma unroll
            for (int t = 0; t < 4; ++t) units(1, t, product(f1, t, S.h[0]));
            __syncthreads();
#pragma unroll
            for (int t = 0; t < 4; ++t) units(2, t, product(f2, t, S.h[1]));
            __syncthreads();
            if (wv < 3) {
                const float4 bs = *reinterpret_cast<const float4 *>(&S.bias[3][16 * wv + 4 * kq]);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const f32x4 c = product(f3, t, S.h[2]);
                    *reinterpret_cast<f32x4 *>(&S.z[16 * t + mrow][16 * wv + 4 * kq]) =
                        f32x4{c[0] + bs.x, c[1] + bs.y, c[2] + bs.z, c[3] + bs.w};
                }
            }
            __syncthreads();
            // the lane's lobes 2 kq and 2 kq + 1: five outputs each
            float z[10];
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                const float2 v = *reinterpret_cast<const float2 *>(&S.z[mine][10 * kq + 2 * k]);
                z[2 * k] = v.x;
                z[2 * k + 1] = v.y;
            }
            float amax = fmaxf(z[0], z[5]);
            amax = fmaxf(amax, __shfl_xor(amax, 16));
            amax = fmaxf(amax, __shfl_xor(amax, 32));
            float pi[2], v[2], kap[2], cw[2], nm[2], mu[2][3];
#pragma unroll
            for (int j = 0; j < 2; ++j) pi[j] = expf(z[5 * j] - amax);
            // (sums over the eight lobes in their order, in all four lanes)
            float psum = 0.0f;
#pragma unroll
            for (int k = 0; k < 8; ++k) psum += __shfl(pi[k & 1], 16 * (k >> 1) + mrow);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                pi[j] /= psum;
                const float m0 = z[5 * j + 1], m1 = z[5 * j + 2], m2 = z[5 * j + 3];
                nm[j] = fmaxf(sqrtf(m0 * m0 + m1 * m1 + m2 * m2), 1e-12f);
                mu[j][0] = m0 / nm[j];
                mu[j][1] = m1 / nm[j];
                mu[j][2] = m2 / nm[j];
                kap[j] = expf(fminf(fmaxf(z[5 * j + 4], kLogKappaMin), kLogKappaMax));
                cw[j] = mu[j][0] * wo[0] + mu[j][1] * wo[1] + mu[j][2] * wo[2];
                v[j] = vmf_norm(kap[j]) * expf(kap[j] * (cw[j] - 1.0f));
            }
            float qv = 0.0f;
#pragma unroll
            for (int k = 0; k < 8; ++k)
                qv += __shfl(pi[k & 1], 16 * (k >> 1) + mrow) * __shfl(v[k & 1], 16 * (k >> 1) + mrow);
            qv = fmaxf(qv, 1e-30f);
            if (ok && kq == 0) li += -(double)wr * log((double)qv);
            const float s = -wr * inv_w;
            float g[10];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const float rj = pi[j] * v[j] / qv;
                g[5 * j] = s * (rj - pi[j]);
                const float e2 = expf(-2.0f * kap[j]);
                const float dlk = 1.0f / kap[j] - 2.0f * e2 / (-expm1f(-2.0f * kap[j])) + (cw[j] - 1.0f);
                const float zs = z[5 * j + 4];
                g[5 * j + 4] = (zs > kLogKappaMin && zs < kLogKappaMax) ? s * rj * dlk * kap[j] : 0.0f;
                const float f = s * rj * kap[j] / nm[j];
#pragma unroll
                for (int a = 0; a < 3; ++a) g[5 * j + 1 + a] = f * (wo[a] - cw[j] * mu[j][a]);
            }
            typedef short bf16x2 __attribute__((ext_vector_type(2)));
            short *dr = &S.dz[0][mine][0];
#pragma unroll
            for (int k = 0; k < 10; k += 2) {
                const float v0 = ok ? g[k] : 0.0f, v1 = ok ? g[k + 1] : 0.0f;
                b3[k] += v0;
                b3[k + 1] += v1;
                *reinterpret_cast<bf16x2 *>(dr + 10 * kq + k) = bf16x2{to_bf16(v0), to_bf16(v1)};
            }
            *reinterpret_cast<bf16x2 *>(dr + kGuideOut + 2 * kq) = bf16x2{0, 0};
        }
        __syncthreads();
        // dZ of the layer below, units 16 wv + (0..15) of all 64 records, into the other buffer
        auto backprop = [&](const bf16x4 *wt, int ktiles, int layer, int cur, float bsum[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                f32x4 c = zero;
#pragma unroll
                for (int kt = 0; kt < ktiles; ++kt)
                    c = mfma16(wt[kt], *reinterpret_cast<const bf16x4 *>(&S.dz[cur][16 * t + mrow][16 * kt + 4 * kq]), c);
                // lane holds dZ[record 16 t + mrow][16 wv + 4 kq + j]
                const bf16x4 h = *reinterpret_cast<const bf16x4 *>(&S.h[layer][16 * t + mrow][16 * wv + 4 * kq]);
                bf16x4 e;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float d = h[j] > 0 ? c[j] : 0.0f;   // (the bits of a bf16: positive or +0)
                    bsum[j] += d;
                    e[j] = to_bf16(d);
                }
                *reinterpret_cast<bf16x4 *>(&S.dz[cur ^ 1][16 * t + mrow][16 * wv + 4 * kq]) = e;
            }
        };
        auto weights = [&](int layer, int cur, f32x4 *g, int otiles) __attribute__((always_inline)) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bf16x4 b = col_frag<kRow>(&S.h[layer][16 * t], 16 * wv, mrow, kq);
#pragma unroll
                for (int ot = 0; ot < otiles; ++ot)
                    g[ot] = mfma16(col_frag<kRow>(&S.dz[cur][16 * t], 16 * ot, mrow, kq), b, g[ot]);
            }
        };
        // layer 3: in H2, out 48 (3 o-tiles)
        weights(2, 0, g3, 3);
        backprop(t3, 3, 2, 0, b2);
        __syncthreads();
        // layer 2: in H1
        weights(1, 1, g2, 4);
        backprop(t2, 4, 1, 1, b1);
        __syncthreads();
        // layer 1: in H0
        weights(0, 0, g1, 4);
        backprop(t1, 4, 0, 0, b0);
        __syncthreads();
        // layer 0: in the 15 network inputs (one i-tile), o-tile = wave
#pragma unroll
        for (int t = 0; t < 4; ++t)
            g0 = mfma16(col_frag<kRow>(&S.dz[1][16 * t], 16 * wv, mrow, kq), col_frag<24>(&S.x[16 * t], 0, mrow, kq), g0);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) li += __shfl_xor(li, off);
    if (lane == 0) unsafeAtomicAdd(loss, li);
    // the workgroup's sums, as they lie in the lanes (PartRow)
    float *P = part + (size_t)blockIdx.x * kPartRow;
    auto put_w = [&](int tile, const f32x4 &acc) { *reinterpret_cast<f32x4 *>(P + tile * 256 + lane * 4) = acc; };
    // a sum over the 16 lanes that share kq
    auto sum16 = [&](float v) __attribute__((always_inline)) {
#pragma unroll
        for (int off = 8; off >= 1; off >>= 1) v += __shfl_xor(v, off);
        return v;
    };
    float *PB = P + kPartTiles * 256;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float s0 = sum16(b0[j]), s1 = sum16(b1[j]), s2 = sum16(b2[j]);
        if (mrow == 0) {
            PB[16 * wv + 4 * kq + j] = s0;
            PB[kGuideWidth + 16 * wv + 4 * kq + j] = s1;
            PB[2 * kGuideWidth + 16 * wv + 4 * kq + j] = s2;
        }
    }
    // the last layer's: each wave has those of its records
    float(*b4)[kGuideWidth] = S.bias;   // (done with)
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 10; ++k) {
        const float s = sum16(b3[k]);
        if (mrow == 0) b4[wv][10 * kq + k] = s;
    }
    __syncthreads();
    if (tid < kGuideOut) PB[3 * kGuideWidth + tid] = (b4[0][tid] + b4[1][tid]) + (b4[2][tid] + b4[3][tid]);
#pragma unroll
    for (int ot = 0; ot < 4; ++ot) {
        if (ot < 3) put_w(part_tile(3, ot, wv), g3[ot]);
        put_w(part_tile(2, ot, wv), g2[ot]);
        put_w(part_tile(1, ot, wv), g1[ot]);
    }
    put_w(part_tile(0, wv, 0), g0);
}

// ---------------------------------------------------------------------------
// The gradient as the sum of the workgroups' rows, then (apply) Adam on the
// fp32 master parameter and its bf16 copies in the padded weight matrices
// (padding entries are never written: they stay zero).
// ---------------------------------------------------------------------------
struct GuidePacked {
    short *w[4];
    short *wt[4];
    float *b[4];
};

// Block of 256 threads per 32 parameters: eight groups of 32 threads add
// every eighth row (consecutive parameters: coalesced rows), then LDS.
constexpr int kAdamParams = 32;
static_assert(kPartRow % kAdamParams == 0, "whole blocks");

__global__ __launch_bounds__(256) void guide_adam_kernel(float *p, float *m, float *v, float *g,
                                                         const float *__restrict__ part, int nparts, int apply,
                                                         float lr, float b1, float b2, float eps, float c1, float c2,
                                                         GuidePacked out, const double *acc, double *d_loss)
{
    __shared__ float red[8][kAdamParams];
    if (d_loss && blockIdx.x == 0 && threadIdx.x < 2) d_loss[threadIdx.x] = acc[threadIdx.x];
    const int t = threadIdx.x & (kAdamParams - 1), grp = threadIdx.x / kAdamParams;
    const int e = blockIdx.x * kAdamParams + t;   // position in a row of partial sums
    float s = 0.0f;
    {
        // (the loads of eight rows in flight, added in their order)
#pragma unroll 8
        for (int k = grp; k < nparts; k += 8) s += part[(size_t)k * kPartRow + e];
    }
    red[grp][t] = s;
    __syncthreads();
    const int q = part_param(e);
    if (grp != 0 || q < 0) return;
    float gi = 0.0f;
#pragma unroll
    for (int k = 0; k < 8; ++k) gi += red[k][t];
    g[q] = gi;
    if (!apply) return;
    const float mi = b1 * m[q] + (1.0f - b1) * gi;
    const float vi = b2 * v[q] + (1.0f - b2) * gi * gi;
    m[q] = mi;
    v[q] = vi;
    const float pq = p[q] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    p[q] = pq;
    int L = 0;
    while (L + 1 < kGuideLayers && q >= guide_param_off(L + 1)) ++L;
    const int w = q - guide_param_off(L), on = guide_out(L), in_n = guide_in(L);
    if (w < on * in_n) {
        const int o = w / in_n, i = w - o * in_n;
        const short h = to_bf16(pq);
        out.w[L][o * guide_in_pad(L) + i] = h;
        out.wt[L][i * guide_out_pad(L) + o] = h;
    } else {
        out.b[L][w - on * in_n] = pq;
    }
}

__global__ void pack_weights_kernel(const float *params, short *w, short *wt, float *bias, int param_off, int out_n,
                                    int in_n, int out_pad, int in_pad)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= out_pad * in_pad) return;
    const int o = e / in_pad, i = e % in_pad;
    const float val = (o < out_n && i < in_n) ? params[param_off + o * in_n + i] : 0.0f;
    const short h = to_bf16(val);
    w[(size_t)o * in_pad + i] = h;
    wt[(size_t)i * out_pad + o] = h;
    if (i == 0) bias[o] = o < out_n ? params[param_off + out_n * in_n + o] : 0.0f;
}

__global__ void fill_f64_kernel(double *p, size_t n, double v)
{
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
GuideWeights guide_weights(const nc_guide *gd)
{
    GuideWeights W;
    for (int l = 0; l < kGuideLayers; ++l) {
        W.w[l] = gd->d_w[l];
        W.wt[l] = gd->d_wt[l];
        W.b[l] = gd->d_bias[l];
    }
    return W;
}

hipError_t guide_pack(const nc_ctx *ctx, nc_guide *gd)
{
    for (int l = 0; l < kGuideLayers; ++l) {
        const int op = guide_out_pad(l), ip = guide_in_pad(l);
        hipLaunchKernelGGL(pack_weights_kernel, dim3((op * ip + 255) / 256), dim3(256), 0, ctx->stream, gd->d_params,
                           gd->d_w[l], gd->d_wt[l], gd->d_bias[l], guide_param_off(l), guide_out(l), guide_in(l), op,
                           ip);
    }
    return hipGetLastError();
}

hipError_t guide_forward(const nc_ctx *ctx, const nc_guide *gd, const float *X, int n, int rec_stride, float *Z)
{
    // (a wave's weights are loaded once: no more workgroups than are resident together)
    const int blocks = std::max(1, std::min((n + 63) / 64, 3 * ctx->num_cus));
    hipLaunchKernelGGL(guide_forward_kernel, dim3(blocks), dim3(256), 0, ctx->stream, guide_weights(gd), X, n,
                       rec_stride, Z);
    return hipGetLastError();
}

// Workgroups of the training pass: chunks of at least 128 records, at most
// kBwdParts of them (their partial gradients are rows of the scratch buffer).
constexpr int kBwdParts = 512;

static void backward_split(int n, int &parts, int &chunk)
{
    parts = std::max(1, std::min(kBwdParts, (n + 127) / 128));
    chunk = (((n + parts - 1) / parts) + 15) & ~15;
    parts = std::max(1, (n + chunk - 1) / chunk);
}

hipError_t guide_ensure_scratch(nc_guide *gd)
{
    if (gd->d_scratch) return hipSuccess;
    // the workgroups' partial gradients (kBwdParts rows)
    return hipMalloc(&gd->d_scratch, sizeof(float) * (size_t)kBwdParts * kPartRow);
}

hipError_t guide_train_step(const nc_ctx *ctx, nc_guide *gd, const float *rec, int n, int rec_stride, float lr,
                            double *d_loss, bool apply)
{
    hipError_t e = guide_ensure_scratch(gd);
    if (e != hipSuccess) return e;
    float *part = gd->d_scratch;
    // the loss / weight-sum accumulators start at zero
    hipLaunchKernelGGL(fill_f64_kernel, dim3(1), dim3(64), 0, ctx->stream, gd->d_acc, (size_t)2, 0.0);
    hipLaunchKernelGGL(weight_sum_kernel, dim3(std::max(1, std::min(1024, (n + 255) / 256))), dim3(256), 0,
                       ctx->stream, rec, n, rec_stride, gd->d_acc + 1);
    int parts = 1, chunk = 16;
    backward_split(n, parts, chunk);
    hipLaunchKernelGGL(guide_train_kernel, dim3(parts), dim3(256), 0, ctx->stream, guide_weights(gd), rec, rec_stride, n,
                       chunk, (const double *)(gd->d_acc + 1), part, gd->d_acc);
    float c1 = 1.0f, c2 = 1.0f;
    const float b1 = 0.9f, b2 = 0.999f;
    if (apply) {
        gd->step += 1;
        c1 = 1.0f - std::pow(b1, (float)gd->step);
        c2 = 1.0f - std::pow(b2, (float)gd->step);
    }
    GuidePacked out;
    for (int l = 0; l < kGuideLayers; ++l) {
        out.w[l] = gd->d_w[l];
        out.wt[l] = gd->d_wt[l];
        out.b[l] = gd->d_bias[l];
    }
    hipLaunchKernelGGL(guide_adam_kernel, dim3(kPartRow / kAdamParams), dim3(256), 0, ctx->stream, gd->d_params,
                       gd->d_m, gd->d_v, gd->d_grad, (const float *)part, parts, apply ? 1 : 0, lr, b1, b2, 1e-8f,
                       c1, c2, out, (const double *)gd->d_acc, d_loss);
    return hipGetLastError();
}

}  // namespace nc
