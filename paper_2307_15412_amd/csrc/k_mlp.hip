// k_mlp.hip -- the learned ray proposal: scene probe, training histogram,
// a 4-layer MLP (18 -> 64 -> 64 -> 64 -> 1, ReLU) with forward, backward and
// Adam kernels, and the sampling table (softmax mixed with the uniform density,
// then its CDF) that the tracer's importance sampler reads.
//
// Weights and activations are stored in FP16; every product is formed and
// accumulated in FP32 (an FP16 x FP16 product is exact in FP32).  Every layer
// runs on the matrix cores: the forward pass in FP16 MFMA, the backward pass
// and the weight gradients in FP32 MFMA (the gradients fall below FP16's
// normal range), 32 rows per wavefront; the weight gradients are reduced in
// a fixed order.
#include <algorithm>

#include <hip/hip_fp16.h>

#include "rr_internal.h"

namespace {

#define NAZ 128
#define NEL 64
#define NBINS (NAZ * NEL)
#define NIN 18
#define NH 64
#define OFF_W1 0
#define OFF_B1 (OFF_W1 + NH * NIN)
#define OFF_W2 (OFF_B1 + NH)
#define OFF_B2 (OFF_W2 + NH * NH)
#define OFF_W3 (OFF_B2 + NH)
#define OFF_B3 (OFF_W3 + NH * NH)
#define OFF_W4 (OFF_B3 + NH)
#define OFF_B4 (OFF_W4 + NH)
#define NPARAMS (OFF_B4 + 1)

static_assert(NPARAMS == RR_MLP_PARAMS, "parameter count");

__device__ __forceinline__ float h16(float x) { return __half2float(__float2half(x)); }

// input k of row r: k = 0, 1 the bin's azimuth and elevation centre mapped
// to [-1, 1], k = 2 .. 17 the scene code (all rounded to FP16)
__device__ __forceinline__ float row_input_k(const float *codes, int64_t r, int k)
{
    const int64_t s = r / NBINS;
    const int b = (int)(r - s * NBINS);
    if (k == 0) return h16(2.0f * ((float)(b % NAZ) + 0.5f) / (float)NAZ - 1.0f);
    if (k == 1) return h16(2.0f * ((float)(b / NAZ) + 0.5f) / (float)NEL - 1.0f);
    return h16(codes[s * 16 + k - 2]);
}

// forward on the matrix cores (v_mfma_f32_32x32x16_f16: FP16 operands, FP32
// accumulation; an FP16 x FP16 product is exact in FP32).  A wavefront takes
// 32 rows at a time, as the columns of the product: the weights (out x in, 16
// inputs a step; layer 1's 18 inputs padded to 32 with zeros) are the A
// operand, kept in registers for all of the wavefront's rows, the activations
// (in x rows) the B operand.  A lane's results are then outputs of its own
// row: after bias, ReLU and the FP16 rounding in FP32, exchanging four
// outputs with the other half of the wavefront (v_permlane32_swap) makes them
// the next layer's B operand, without LDS.  Logit: each lane's 32 products
// with W4, then the two halves.  Bound by those vector operations (1 048 576
// rows: 31 us; with activations as the A operand and through LDS 61 us).
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
#define MF_FRAGS (2 * 2 + 2 * 4 * 2)  // A fragments: layer 1 (2 output blocks x 2 input steps), layers 2, 3 (2 x 4 each)
#define MF_WAVES 3                    // wavefronts a SIMD: 162 registers
#define MF_WGS (256 * MF_WAVES)       // workgroups of a full launch

// fragment (output block cb, input step kc) of a layer with weights
// w[out][in] (in-width nin): lane l holds output 32 cb + l % 32, inputs
// 16 kc + 8 (l / 32) .. + 7, rounded to FP16 (zero beyond nin)
__device__ __forceinline__ u32x4 wfrag(const float *w, int nin, int cb, int kc, int l)
{
    const int j = 32 * cb + (l & 31), i0 = 16 * kc + 8 * (l >> 5);
    f16x8 v;
#pragma unroll
    for (int e = 0; e < 8; e++) v[e] = (_Float16)(i0 + e < nin ? w[j * nin + i0 + e] : 0.0f);
    return __builtin_bit_cast(u32x4, v);
}

__global__ __launch_bounds__(256, MF_WAVES) void k_mlp_fwd(const float *P, const float *codes, int64_t n,
                                                    __half *acts, float *z)
{
    __shared__ u32x4 Wf[MF_FRAGS][64];
    __shared__ float4 Bs[4][NH / 4];   // biases of layers 1-3, W4
    for (int q = threadIdx.x; q < MF_FRAGS * 64; q += blockDim.x) {
        const int f = q >> 6, l = q & 63;
        u32x4 v;
        if (f < 4) v = wfrag(P + OFF_W1, NIN, f >> 1, f & 1, l);
        else if (f < 12) v = wfrag(P + OFF_W2, NH, (f - 4) >> 2, (f - 4) & 3, l);
        else v = wfrag(P + OFF_W3, NH, (f - 12) >> 2, (f - 12) & 3, l);
        Wf[f][l] = v;
    }
    if (threadIdx.x < 4 * NH) {
        const int L = threadIdx.x / NH, q = threadIdx.x % NH;
        const int off[4] = {OFF_B1, OFF_B2, OFF_B3, OFF_W4};
        reinterpret_cast<float *>(Bs[L])[q] = h16(P[off[L] + q]);
    }
    const float b4 = h16(P[OFF_B4]);
    __syncthreads();
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 31, half = lane >> 5;
    u32x4 W[MF_FRAGS];
#pragma unroll
    for (int f = 0; f < MF_FRAGS; f++) W[f] = Wf[f][lane];

    const int64_t step = (int64_t)gridDim.x * 128;
    for (int64_t r0 = ((int64_t)blockIdx.x * 4 + w) * 32; r0 < n; r0 += step) {
        const int64_t r = r0 + row;
        asm volatile("" ::: "memory");   // the biases stay in LDS: 128 registers
        // layer 1: inputs 8 half .. + 7 (step 0) and 16 + 8 half .. (step 1);
        // the 32 rows share their scene
        u32x4 A[4];
        {
            const float *code = codes + r0 / NBINS * 16;
            f16x8 a0, a1;
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const float lo = e < 2 ? row_input_k(codes, r, e) : code[max(e - 2, 0)];
                a0[e] = (_Float16)(half ? code[e + 6] : lo);
                a1[e] = (_Float16)(!half && e < NIN - 16 ? code[min(14 + e, 15)] : 0.0f);
            }
            A[0] = __builtin_bit_cast(u32x4, a0);
            A[1] = __builtin_bit_cast(u32x4, a1);
        }
        float logit = half ? 0.0f : b4;
#pragma unroll
        for (int L = 0; L < 3; L++) {
            const int nk = L == 0 ? 2 : 4;                   // input steps of the layer
            const int fb = L == 0 ? 0 : (L == 1 ? 4 : 12);   // its first fragment
            u32x4 N[4];
#pragma unroll
            for (int cb = 0; cb < 2; cb++) {
                f32x16 acc;
#pragma unroll
                for (int e = 0; e < 16; e++) acc[e] = 0.0f;
#pragma unroll
                for (int kc = 0; kc < 4; kc++)
                    if (kc < nk)
                        acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                            __builtin_bit_cast(f16x8, W[fb + cb * nk + kc]),
                            __builtin_bit_cast(f16x8, A[kc]), acc, 0, 0, 0);
                // D layout: register e of lane l is output 8 (e / 4) +
                // 4 (l / 32) + e % 4 of the block, row l % 32
                unsigned g[4][2];
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const float4 b = Bs[L][8 * cb + 2 * q + half];
                    const f16x2 zero = {(_Float16)0.0f, (_Float16)0.0f};
                    f16x2 lo = {(_Float16)(acc[4 * q] + b.x), (_Float16)(acc[4 * q + 1] + b.y)};
                    f16x2 hi = {(_Float16)(acc[4 * q + 2] + b.z), (_Float16)(acc[4 * q + 3] + b.w)};
                    lo = __builtin_elementwise_max(lo, zero);
                    hi = __builtin_elementwise_max(hi, zero);
                    if (L == 2) {
                        const float4 v = Bs[3][8 * cb + 2 * q + half];
                        logit = fmaf(v.x, (float)lo[0], logit);
                        logit = fmaf(v.y, (float)lo[1], logit);
                        logit = fmaf(v.z, (float)hi[0], logit);
                        logit = fmaf(v.w, (float)hi[1], logit);
                    }
                    g[q][0] = __builtin_bit_cast(unsigned, lo);
                    g[q][1] = __builtin_bit_cast(unsigned, hi);
                }
                // outputs 0-3 and 8-11 of a step (lower half), 4-7 and 12-15
                // (upper) into 0-7 and 8-15
#pragma unroll
                for (int q = 0; q < 4; q += 2) {
                    const auto x = __builtin_amdgcn_permlane32_swap(g[q][0], g[q + 1][0], false, false);
                    const auto y = __builtin_amdgcn_permlane32_swap(g[q][1], g[q + 1][1], false, false);
                    N[2 * cb + (q >> 1)] = u32x4{x[0], y[0], x[1], y[1]};
                }
            }
#pragma unroll
            for (int kc = 0; kc < 4; kc++) A[kc] = N[kc];
            if (acts) {
#pragma unroll
                for (int kc = 0; kc < 4; kc++)
                    *reinterpret_cast<u32x4 *>(acts + ((int64_t)L * n + r) * NH + 16 * kc + 8 * half) = A[kc];
            }
        }
        logit += __shfl_xor(logit, 32);
        if (half == 0) z[r] = logit;
    }
}

// per scene: softmax of the logits; loss -sum H log q / sum H and its
// gradient dz = (q - H / sum H) / n_scenes (zero for a scene with no target);
// a thread keeps its eight bins in registers, wavefronts reduce by shuffles
template <class Op>
__device__ __forceinline__ float block_reduce(float v, float *red, Op op)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = op(v, __shfl_xor(v, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = red[threadIdx.x & 15];
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) v = op(v, __shfl_xor(v, o));
    return v;
}

__global__ __launch_bounds__(1024) void k_softmax_grad(const float *z, const float *H, int n_scenes,
                                                       float *dz, float *loss)
{
    __shared__ float red[4][16];
    const int s = blockIdx.x;
    float zv[8], hv[8];
    auto add = [](float a, float b) { return a + b; };
    float mx = -3.0e38f, hsum = 0.0f;
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const int64_t b = (int64_t)s * NBINS + k * 1024 + threadIdx.x;
        zv[k] = z[b];
        hv[k] = H[b];
        mx = fmaxf(mx, zv[k]);
        hsum += hv[k];
    }
    mx = block_reduce(mx, red[0], [](float a, float b) { return fmaxf(a, b); });
    float es = 0.0f;
#pragma unroll
    for (int k = 0; k < 8; k++) es += __expf(zv[k] - mx);
    const float Hs = block_reduce(hsum, red[1], add);
    const float lse = logf(block_reduce(es, red[2], add));
    float l = 0.0f;
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const float logq = zv[k] - mx - lse;
        float d = 0.0f;
        if (Hs > 0.0f) {
            l -= hv[k] * logq;
            d = (__expf(logq) - hv[k] / Hs) / (float)n_scenes;
        }
        dz[(int64_t)s * NBINS + k * 1024 + threadIdx.x] = d;
    }
    l = block_reduce(l, red[3], add);
    if (threadIdx.x == 0) loss[s] = Hs > 0.0f ? l / Hs / (float)n_scenes : 0.0f;
}

// Backward pass and weight gradients on the matrix cores in FP32
// (v_mfma_f32_32x32x2f32): the gradients fall below FP16's normal range, so
// they stay FP32 throughout.  A wavefront takes 32 rows at a time:
//   d3 = [h3 > 0] dz W4               (vector units),  gW4 += dz h3
//   gW3 += d3^T h2,  d2 = [h2 > 0] (d3 W3)
//   gW2 += d2^T h1,  d1 = [h1 > 0] (d2 W2)
// with d in its own LDS tile (row-major floats), the FP16 activations beside
// it, and the sums over its rows in registers throughout.  32 rows share
// their elevation and scene, so gW1 needs only d1's column sums and its sums
// with the azimuth.  The four wavefronts of a workgroup are added in order,
// the workgroups' rows of the partial table by two more passes: the gradient
// is the same bits on every run.
// One wavefront a SIMD (its sums alone take 128 registers); bound by the 256
// MFMAs of 64 cycles a tile, which take 27 us for 131 072 rows, and by the LDS
// turns between them that one wavefront cannot hide: 65 us.  A backward kernel
// that wrote d1-d3 (98 us) and one kernel a layer that read them again (4 x 34)
// were bound by those 200 MB and short of wavefronts.
#define GR_RS (NH + 1)            // row stride of a gradient tile (floats)
#define GR_HS (NH + 8)            // of an activation tile (halves)
#define GR_WGS 256                // most workgroups, one a compute unit
#define GR_VEC (4 * NH + NH * NIN + 4)
#define GR_D (32 * GR_RS * 4)
#define GR_WAVE (GR_D + 3 * 32 * GR_HS * 2)
#define GR_MAIN (2 * NH * NH * 2 + 4 * GR_WAVE)
#define GR_RED (4 * (2 * NH * NH + GR_VEC) * 4)
#define WG_RUN 32                 // rows of the partial table added per first-pass run

// LDS of a wavefront alone: its operations run in order, the compiler must
// not move them
__device__ __forceinline__ void lds_turn()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_wave_barrier();
}

__global__ __launch_bounds__(256, 1) void k_mlp_grad(const float *P, const float *dz, int64_t n,
                                                     const __half *acts, const float *codes,
                                                     int per_wg, float *part)
{
    __shared__ uint4 lds[(GR_RED > GR_MAIN ? GR_RED : GR_MAIN) / 16];
    char *base = reinterpret_cast<char *>(lds);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 31, kk = lane >> 5;
    _Float16 *Ws = reinterpret_cast<_Float16 *>(base);   // W3, W2 as [out j][in i] (FP16 values: exact)
    char *own = base + 2 * NH * NH * 2 + w * GR_WAVE;
    float *D = reinterpret_cast<float *>(own);
    _Float16 *Hl = reinterpret_cast<_Float16 *>(own + GR_D);
    for (int q = threadIdx.x; q < NH * NH; q += 256) {
        Ws[q] = (_Float16)P[OFF_W3 + q];
        Ws[NH * NH + q] = (_Float16)P[OFF_W2 + q];
    }
    const float w4 = h16(P[OFF_W4 + lane]);
    __syncthreads();

    f32x16 g3[2][2], g2[2][2];
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int e = 0; e < 16; e++) g3[i][j][e] = g2[i][j][e] = 0.0f;
    float g1[NIN];
#pragma unroll
    for (int c = 0; c < NIN; c++) g1[c] = 0.0f;
    float gw4 = 0.0f, gb4 = 0.0f, b3 = 0.0f, b2[2] = {0.0f, 0.0f}, b1 = 0.0f;

    // tiles of 32 rows: the workgroup's 4 per_wg, one in four for a wavefront;
    // the next tile's activations are loaded while this one is worked on
    const int64_t tiles = n / 32, t1 = min(tiles, ((int64_t)blockIdx.x + 1) * per_wg * 4);
    int64_t t = (int64_t)blockIdx.x * per_wg * 4 + w;
    u32x4 pre[3][4];
    float predz = 0.0f;
    auto load = [&](int64_t tile) {
#pragma unroll
        for (int L = 0; L < 3; L++)
#pragma unroll
            for (int q = 0; q < 4; q++)
                pre[L][q] = reinterpret_cast<const u32x4 *>(acts + ((int64_t)L * n + tile * 32) * NH)[q * 64 + lane];
        predz = dz[tile * 32 + col];
    };
    if (t < t1) load(t);
    for (; t < t1; t += 4) {
        lds_turn();
#pragma unroll
        for (int L = 0; L < 3; L++)
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int x = q * 64 + lane;
                *reinterpret_cast<u32x4 *>(Hl + (L * 32 + (x >> 3)) * GR_HS + 8 * (x & 7)) = pre[L][q];
            }
        const float dzv = predz;
        if (t + 4 < t1) load(t + 4);
        lds_turn();
        // d3: lane j over the tile's rows
#pragma unroll
        for (int rr = 0; rr < 32; rr++) {
            const float zr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(dzv), rr));
            const float h = (float)Hl[(2 * 32 + rr) * GR_HS + lane];
            const float v = h > 0.0f ? zr * w4 : 0.0f;
            D[rr * GR_RS + lane] = v;
            gw4 = fmaf(zr, h, gw4);
            b3 += v;
        }
        gb4 += dzv;
        lds_turn();
#pragma unroll
        for (int L = 0; L < 2; L++) {
            const _Float16 *h = Hl + (1 - L) * 32 * GR_HS;
            // gW[a][c] += sum_r D[r][a] h[r][c]: lane l takes D[r + l / 32][a]
            // and h[r + l / 32][c], a, c = l % 32 (+ 32), two rows a step
#pragma unroll 4
            for (int ks = 0; ks < 16; ks++) {
                const int r = 2 * ks + kk;
                float a[2], c[2];
#pragma unroll
                for (int i = 0; i < 2; i++) {
                    a[i] = D[r * GR_RS + 32 * i + col];
                    c[i] = (float)h[r * GR_HS + 32 * i + col];
                    if (L == 1) b2[i] += a[i];
                }
#pragma unroll
                for (int i = 0; i < 2; i++)
#pragma unroll
                    for (int j = 0; j < 2; j++) {
                        f32x16 &g = L == 0 ? g3[i][j] : g2[i][j];
                        g = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], c[j], g, 0, 0, 0);
                    }
            }
            // out[r][i] = sum_j D[r][j] W[j][i]: A[r][k = j] = D, B[k = j][i] = W
            f32x16 acc[2];
#pragma unroll
            for (int cb = 0; cb < 2; cb++)
#pragma unroll
                for (int e = 0; e < 16; e++) acc[cb][e] = 0.0f;
#pragma unroll 8
            for (int ks = 0; ks < NH / 2; ks++) {
                const int k = 2 * ks + kk;
                const float av = D[col * GR_RS + k];
#pragma unroll
                for (int cb = 0; cb < 2; cb++)
                    acc[cb] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                        av, (float)Ws[(L * NH + k) * NH + 32 * cb + col], acc[cb], 0, 0, 0);
            }
            lds_turn();
            // D layout: register e of lane l is row 8 (e / 4) + 4 (l / 32) +
            // e % 4, column l % 32 of the block
            float sum[2] = {0.0f, 0.0f}, saz[2] = {0.0f, 0.0f};
#pragma unroll
            for (int cb = 0; cb < 2; cb++)
#pragma unroll
                for (int e = 0; e < 16; e++) {
                    const int rr = 8 * (e >> 2) + 4 * kk + (e & 3), i = 32 * cb + col;
                    const float v = (float)h[rr * GR_HS + i] > 0.0f ? acc[cb][e] : 0.0f;
                    if (L == 0) {
                        D[rr * GR_RS + i] = v;
                    } else {
                        // (azimuth centres are odd multiples of 1 / 128: exact in FP16)
                        const int ia = (int)((t * 32) & (NAZ - 1)) + rr;
                        sum[cb] += v;
                        saz[cb] = fmaf(v, (float)(2 * ia + 1 - NAZ) / (float)NAZ, saz[cb]);
                    }
                }
            if (L == 1) {
                // lane a = 32 kk + col of layer 1
#pragma unroll
                for (int cb = 0; cb < 2; cb++) {
                    sum[cb] += __shfl_xor(sum[cb], 32);
                    saz[cb] += __shfl_xor(saz[cb], 32);
                }
                const float sa = kk ? sum[1] : sum[0];
                b1 += sa;
                g1[0] += kk ? saz[1] : saz[0];
#pragma unroll
                for (int c = 1; c < NIN; c++) g1[c] = fmaf(sa, row_input_k(codes, t * 32, c), g1[c]);
            }
            lds_turn();
        }
    }
    __syncthreads();
    // the wavefronts' sums at the parameters' places, added in order
    float *red = reinterpret_cast<float *>(base);
    float *M = red + w * 2 * NH * NH, *V = red + 4 * 2 * NH * NH + w * GR_VEC;
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
            for (int e = 0; e < 16; e++) {
                const int q = (32 * i + 8 * (e >> 2) + 4 * kk + (e & 3)) * NH + 32 * j + col;
                M[q] = g3[i][j][e];
                M[NH * NH + q] = g2[i][j][e];
            }
    V[lane] = gw4;
    V[NH + lane] = b3;
    {
        // the even rows' sum (lanes 0..31) plus the odd rows'
        const float x0 = b2[0] + __shfl_xor(b2[0], 32), x1 = b2[1] + __shfl_xor(b2[1], 32);
        V[2 * NH + lane] = kk ? x1 : x0;
    }
    V[3 * NH + lane] = b1;
#pragma unroll
    for (int c = 0; c < NIN; c++) V[4 * NH + lane * NIN + c] = g1[c];
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) gb4 += __shfl_xor(gb4, o);
    if (lane == 0) V[4 * NH + NH * NIN] = gb4;
    __syncthreads();
    float *G = part + (int64_t)blockIdx.x * NPARAMS;
    const float *V0 = red + 4 * 2 * NH * NH;
    for (int q = threadIdx.x; q < 2 * NH * NH; q += 256) {
        const float x = ((red[q] + red[2 * NH * NH + q]) + red[4 * NH * NH + q]) + red[6 * NH * NH + q];
        G[(q < NH * NH ? OFF_W3 : OFF_W2 - NH * NH) + q] = x;
    }
    for (int q = threadIdx.x; q < 4 * NH + NH * NIN + 1; q += 256) {
        const float x = ((V0[q] + V0[GR_VEC + q]) + V0[2 * GR_VEC + q]) + V0[3 * GR_VEC + q];
        const int L = q / NH;
        const int to = q < 4 * NH ? (L == 0 ? OFF_W4 : L == 1 ? OFF_B3 : L == 2 ? OFF_B2 : OFF_B1) + q % NH
                     : q < 4 * NH + NH * NIN ? OFF_W1 + q - 4 * NH : OFF_B4;
        G[to] = x;
    }
}

// first pass: run y of the partial table (rows y WG_RUN .. + WG_RUN - 1, in
// order) into row nb + y
__global__ __launch_bounds__(256) void k_wgrad_sum(float *part, int nb)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NPARAMS) return;
    const int y = blockIdx.y;
    const int b0 = y * WG_RUN, b1 = min(nb, b0 + WG_RUN);
    float s = 0.0f;
#pragma unroll 8
    for (int b = b0; b < b1; b++) s += part[(int64_t)b * NPARAMS + i];
    part[(int64_t)(nb + y) * NPARAMS + i] = s;
}

// second pass: those runs in order into G; lr > 0: then a step of Adam
// (Kingma & Ba), FP32 master parameters and moments
__global__ __launch_bounds__(256) void k_wgrad_sum2(const float *part, int nb, int runs, float *G,
                                                    AdamArgs a)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= NPARAMS) return;
    float g = 0.0f;
    for (int y = 0; y < runs; y++) g += part[(int64_t)(nb + y) * NPARAMS + i];
    G[i] = g;
    if (!(a.lr > 0.0f)) return;
    const float mi = a.b1 * a.m[i] + (1.0f - a.b1) * g;
    const float vi = a.b2 * a.v[i] + (1.0f - a.b2) * g * g;
    a.m[i] = mi;
    a.v[i] = vi;
    a.P[i] -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
}

// sampling table for one scene: q_mix = (1 - beta) d / sum d + beta / NBINS
// with d = exp(power z) (kappa = 0: the softmax of power z), or, with kappa >
// 0, d = sqrt(x / (kappa + x)) where x = NBINS softmax(z) is a bin's fitted
// return density relative to the mean (the density of least variance x cost
// when a ray costs kappa mean returns); cdf[0] = 0, cdf[b + 1] = cdf[b] +
// q_mix[b] (FP64, block scan), normalised
__global__ __launch_bounds__(1024) void k_build_cdf(const float *z, float beta, float power,
                                                    float kappa, double *cdf)
{
    __shared__ double red[1024];
    __shared__ float fred[1024];
    const int t = threadIdx.x;
    float mx = -3.0e38f;
    for (int b = t; b < NBINS; b += 1024) mx = fmaxf(mx, z[b]);
    fred[t] = mx;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if (t < o) fred[t] = fmaxf(fred[t], fred[t + o]);
        __syncthreads();
    }
    mx = fred[0];
    __syncthreads();
    // each thread owns 8 consecutive bins
    const double pw = kappa > 0.0f ? 1.0 : (double)power;
    double e[8];
    double s = 0.0;
    for (int k = 0; k < 8; k++) {
        e[k] = exp(pw * ((double)z[t * 8 + k] - (double)mx));
        s += e[k];
    }
    red[t] = s;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if (t < o) red[t] += red[t + o];
        __syncthreads();
    }
    double tot = red[0];
    __syncthreads();
    if (kappa > 0.0f) {
        // x = NBINS e / tot; d = sqrt(x / (kappa + x)); then normalise d
        double s2 = 0.0;
        for (int k = 0; k < 8; k++) {
            const double x = (double)NBINS * e[k] / tot;
            e[k] = sqrt(x / ((double)kappa + x));
            s2 += e[k];
        }
        red[t] = s2;
        __syncthreads();
        for (int o = 512; o > 0; o >>= 1) {
            if (t < o) red[t] += red[t + o];
            __syncthreads();
        }
        tot = red[0];
        __syncthreads();
    }
    double loc = 0.0;
    double q[8];
    for (int k = 0; k < 8; k++) {
        q[k] = (1.0 - (double)beta) * e[k] / tot + (double)beta / (double)NBINS;
        loc += q[k];
    }
    // inclusive scan of per-thread sums (Hillis-Steele)
    red[t] = loc;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        double y = t >= o ? red[t - o] : 0.0;
        __syncthreads();
        red[t] += y;
        __syncthreads();
    }
    const double total = red[1023];
    double run = red[t] - loc;
    for (int k = 0; k < 8; k++) {
        run += q[k];
        cdf[t * 8 + k + 1] = run / total;
    }
    if (t == 0) cdf[0] = 0.0;
    __syncthreads();
    if (t == 1023) cdf[NBINS] = 1.0;
}

}  // namespace

hipError_t launch_mlp_forward(const float *P, const float *codes, int64_t n, __half *acts, float *z,
                              hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (n % NBINS) return hipErrorInvalidValue;   // whole scenes
    const int64_t wgs = std::min<int64_t>((n + 127) / 128, MF_WGS);
    hipLaunchKernelGGL(k_mlp_fwd, dim3((unsigned)wgs), dim3(256), 0, s, P, codes, n, acts, z);
    return hipGetLastError();
}

hipError_t launch_softmax_grad(const float *z, const float *H, int n_scenes, float *dz, float *loss,
                               hipStream_t s)
{
    if (n_scenes <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_softmax_grad, dim3(n_scenes), dim3(1024), 0, s, z, H, n_scenes, dz, loss);
    return hipGetLastError();
}

// workgroups of the gradient kernel: equal numbers of 128-row steps
static int grad_wgs(int64_t n, int &per_wg)
{
    const int64_t steps = (n + 127) / 128;
    per_wg = (int)((steps + GR_WGS - 1) / GR_WGS);
    return (int)((steps + per_wg - 1) / per_wg);
}

int64_t mlp_part_rows(int64_t n)
{
    int per;
    const int nb = grad_wgs(std::max<int64_t>(n, 1), per);
    return nb + (nb + WG_RUN - 1) / WG_RUN;
}

AdamArgs adam_args(float *P, float *m, float *v, float lr, int step)
{
    AdamArgs a;
    a.P = P;
    a.m = m;
    a.v = v;
    a.lr = lr;
    a.b1 = 0.9f;
    a.b2 = 0.999f;
    a.c1 = 1.0f - powf(a.b1, (float)step);
    a.c2 = 1.0f - powf(a.b2, (float)step);
    a.eps = 1e-8f;
    return a;
}

hipError_t launch_mlp_backward(const float *P, const float *dz, int64_t n, const __half *acts,
                               const float *codes, float *part, float *grad, const AdamArgs &adam,
                               hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (n % NBINS) return hipErrorInvalidValue;   // whole scenes: 32 rows share scene and elevation
    int per;
    const int nb = grad_wgs(n, per);
    hipLaunchKernelGGL(k_mlp_grad, dim3(nb), dim3(256), 0, s, P, dz, n, acts, codes, per, part);
    const int runs = (nb + WG_RUN - 1) / WG_RUN;
    hipLaunchKernelGGL(k_wgrad_sum, dim3((NPARAMS + 255) / 256, runs), dim3(256), 0, s, part, nb);
    hipLaunchKernelGGL(k_wgrad_sum2, dim3((NPARAMS + 255) / 256), dim3(256), 0, s, part, nb, runs, grad,
                       adam);
    return hipGetLastError();
}

hipError_t launch_build_cdf(const float *z, float beta, float power, float kappa, double *cdf,
                            hipStream_t s)
{
    hipLaunchKernelGGL(k_build_cdf, dim3(1), dim3(1024), 0, s, z, beta, power, kappa, cdf);
    return hipGetLastError();
}
