// k_bpmfma.hip -- delay-and-sum back-projection on the matrix cores.
//
// image(x) = sum_n sum_t a_t(n) sum_r S_n[t, r] b_r(n),
//     a_t(n) = exp(+j 2 pi f_n |x - tx_t| / c),  b_r(n) = exp(+j 2 pi f_n |x - rx_r| / c),
// because the two legs of the delay add: the inner sum over receivers is, for
// every frequency, the complex product of the cube slice S_n (Tx x Rx) with
// the matrix of receive phasors of a block of voxels (Rx x voxels), the same
// multiply-adds as the brute-force sum.  A workgroup of eight wavefronts (two
// per SIMD) owns 128 voxels, 16 per wavefront; per frequency each wavefront
// computes U = S_n B (for 96 Tx and Rx six 16 x 16 blocks, three 32-receiver
// steps, split bf16 hi + lo, 216 v_mfma_f32_16x16x32_bf16) and adds
// sum_t a_t U[t, voxel] on the vector units; the two wavefronts of a SIMD
// overlap one's phasor work with the other's products.  S_n, prepared once in
// the A-operand fragment layout, is double-buffered in LDS and loaded by LDS
// DMA one frequency ahead.  Smaller arrays run on fewer blocks and steps (a
// 30 x 37 array on 2 x 2 instead of 6 x 3).  Needs at most 96 transmitters
// and receivers.
//
// Few frequencies do for a block of near voxels: over a block whose delays
// stay within H of its centre's, the factor exp(j 2 pi k df (d - dc) / c) is
// band-limited in k, so it is interpolated from n of the K samples (the nodes
// r_j and coefficients L of rr_bands.cpp, error below 2e-7):
//     image(x) = sum_j sum_tr exp(j 2 pi f_{r_j} d / c) S'_j[t, r],
//     S'_j[t, r] = exp(-j 2 pi r_j df dc / c) sum_k L[k, j] exp(j 2 pi k df dc / c) S_k[t, r]:
// the same product with n = 12 slices per block instead of K = 128 (the hand's
// 81 x 201 x 201 voxels of 1 mm in 324 blocks of 23 mm).  The block's slices
// are formed in FP32 on the vector units (k_bp_block).  The host picks n and
// the block edge by modelled time; a coarse grid or a short sweep keeps every
// sample.  Measured: the hand's image 67 -> 7.9 ms (12 nodes; slices 0.4 ms),
// the products at 1.19 PFLOP/s, where a large bf16 matrix product reaches
// 1.2-1.4 (the FP64 legs of a voxel and the first slice's load are a fifth of
// a workgroup's time); a 30 x 37
// array on 17 x 41 x 39 voxels at 33 samples 0.169 -> 0.061 ms by its smaller
// tile alone.
//
// Leg lengths are formed in FP64 once per voxel and rounded to FP32, from where
// every phase starts (below 256 turns in an imaging volume of a few tens of
// centimetres: the rounding is worth up to 7.6e-6 turn).  At every sample the
// phase is the FP32 product of the rounded leg with f_n / c, good to ~1e-5
// turn; at nodes, whose few roundings of that product would not average out,
// it is the rounded leg's phase at the middle frequency, reduced in FP64, plus
// the few turns from there.  The hardware sin/cos take turns.
#include <algorithm>
#include <cmath>

#include "rr_internal.h"

namespace {

#define BG_W 8                 // wavefronts per workgroup
#define BG_VW 16               // voxels per wavefront
// an array takes TB = 2, 4 or 6 blocks of 16 Tx rows and RS = 1, 2 or 3 steps
// of 32 receivers; 4 TB RS fragments of 1 KiB per frequency (4 planes)

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned pack_bf16(float x, float y)
{
    f32x2 v = {x, y};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ void split_bf16(float x, float y, unsigned &hi, unsigned &lo)
{
    hi = pack_bf16(x, y);
    lo = pack_bf16(x - __uint_as_float(hi << 16), y - __uint_as_float(hi & 0xffff0000u));
}

__device__ __forceinline__ bf16x8 as_bf(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ uint4 neg(uint4 v)
{
    return make_uint4(v.x ^ 0x80008000u, v.y ^ 0x80008000u, v.z ^ 0x80008000u, v.w ^ 0x80008000u);
}

#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(a), as_bf(b), c, 0, 0, 0)

// Cube slices in the A-operand layout of the 16 x 16 x 32 product: fragment
// (n, tb, rs, plane) lane l holds S_n[16 tb + l % 16][32 rs + 8 (l / 16) + e],
// e = 0..7, as bf16; planes: real hi, real lo, imaginary hi, imaginary lo;
// zero outside T x R.
__device__ __forceinline__ void store_frag(const float2 *v, uint4 *Sf, int64_t frag, int lane)
{
    uint4 p[4];
    unsigned *rh = &p[0].x, *rl = &p[1].x, *ih = &p[2].x, *il = &p[3].x;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        split_bf16(v[2 * q].x, v[2 * q + 1].x, rh[q], rl[q]);
        split_bf16(v[2 * q].y, v[2 * q + 1].y, ih[q], il[q]);
    }
#pragma unroll
    for (int q = 0; q < 4; q++) Sf[(frag * 4 + q) * 64 + lane] = p[q];
}

__global__ void k_bp_prep(const float2 *cube, int64_t stride, int T, int R, int K, int TB, int RS,
                          uint4 *Sf)
{
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (int64_t)K * TB * RS * 64) return;
    const int lane = (int)(g & 63);
    int64_t f = g >> 6;
    const int rs = (int)(f % RS);
    f /= RS;
    const int tb = (int)(f % TB);
    const int n = (int)(f / TB);
    const int t = tb * 16 + (lane & 15);
    const int r0 = rs * 32 + (lane >> 4) * 8;
    float2 v[8];
    for (int e = 0; e < 8; e++)
        v[e] = t < T && r0 + e < R ? cube[((int64_t)t * R + r0 + e) * stride + n] : make_float2(0.0f, 0.0f);
    store_frag(v, Sf, g >> 6, lane);
}

__device__ __forceinline__ double dist3(double x, double y, double z, const double *p)
{
    const double dx = x - p[0], dy = y - p[1], dz = z - p[2];
    return sqrt(dx * dx + dy * dy + dz * dz);
}

__device__ __forceinline__ double frac(double x) { return x - floor(x); }

// sqrt(v) by the FP32 root and two Newton steps in FP64: the first leaves up to
// 4e-14, the second, with the residual formed exactly, what its own rounding
// leaves (2e8 values against the correctly rounded root, with the FP32 root
// and reciprocal each up to a unit off: 862 differ, by one FP64 unit, and no
// leg after its rounding to FP32; after one step 10 legs).  188 legs a voxel are a
// tenth of the kernel at 12 nodes: the hand's image takes 8.17 ms with the
// full root, 7.91 with this one.  0 at 0.
__device__ __forceinline__ double leg_sqrt(double v)
{
    const float s = __builtin_amdgcn_sqrtf((float)v);
    const double h = (double)(s > 0.0f ? 0.5f * __builtin_amdgcn_rcpf(s) : 0.0f);
    double d = (double)s;
    d = fma(fma(-d, d, v), h, d);
    return fma(fma(-d, d, v), h, d);
}

// the voxels of an axis in block b of nb: [at, end), sizes differing by one
__device__ __forceinline__ void block_span(int b, int nb, int n, int &at, int &end)
{
    at = (int)((int64_t)b * n / nb);
    end = (int)((int64_t)(b + 1) * n / nb);
}

struct BpMfmaArgs {
    const uint4 *Sf;          // [block][node] fragments
    const double *tx, *rx;
    int T, R, K;
    double f0, df, inv_c;
    double x0, y0, z0, step;
    int nx, ny, nz;
    int nbx, nby, nbz;        // blocks per axis (1 x 1 x 1: every sample, the whole volume)
    int wgs;                  // workgroups per block
    int n;                    // nodes (K: every sample)
    const int32_t *nodes;     // [n] samples, or NULL: 0 .. K - 1
    float2 *image;
};

// Cube samples [channel][k] to [k][channel], so that the blocks' wavefronts
// read consecutive channels.
__global__ __launch_bounds__(256) void k_bp_turn(const float2 *cube, int64_t stride, int C, int K,
                                                 float2 *out)
{
    __shared__ float2 sh[32][33];
    const int cb = (C + 31) / 32;
    const int c0 = (int)(blockIdx.x % cb) * 32, k0 = (int)(blockIdx.x / cb) * 32;
    const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
    for (int q = 0; q < 4; q++) {
        const int c = c0 + y + 8 * q, k = k0 + x;
        if (c < C && k < K) sh[y + 8 * q][x] = cube[(int64_t)c * stride + k];
    }
    __syncthreads();
    for (int q = 0; q < 4; q++) {
        const int k = k0 + y + 8 * q, c = c0 + x;
        if (c < C && k < K) out[(int64_t)k * C + c] = sh[x][y + 8 * q];
    }
}

// The slices S'_j of one block of voxels: a workgroup per (block, Tx block,
// receiver step), one of its 16 x 32 channels a lane.  Per sample one exact
// integer phase, its hardware sin/cos and n real-by-complex multiply-adds with
// uniform coefficients; then through LDS into the fragment layout.
template <int N>
__global__ __launch_bounds__(512) void k_bp_block(BpMfmaArgs A, const float2 *turned, const float *L,
                                                  int TB, int RS, uint4 *Sf)
{
    __shared__ float2 sh[N][512];
    const int tid = threadIdx.x;
    int id = blockIdx.x;
    const int rs = id % RS;
    id /= RS;
    const int tb = id % TB;
    const int blk = id / TB;
    const int bz = blk % A.nbz, by = blk / A.nbz % A.nby, bx = blk / A.nbz / A.nby;
    int i0, i1, j0, j1, k0, k1;
    block_span(bx, A.nbx, A.nx, i0, i1);
    block_span(by, A.nby, A.ny, j0, j1);
    block_span(bz, A.nbz, A.nz, k0, k1);
    const double x = A.x0 + 0.5 * (i0 + i1 - 1) * A.step, y = A.y0 + 0.5 * (j0 + j1 - 1) * A.step,
                 z = A.z0 + 0.5 * (k0 + k1 - 1) * A.step;
    const int t = tb * 16 + (tid >> 5), r = rs * 32 + (tid & 31);
    float2 acc[N];
#pragma unroll
    for (int j = 0; j < N; j++) acc[j] = make_float2(0.0f, 0.0f);
    if (t < A.T && r < A.R) {
        const double dc = dist3(x, y, z, A.tx + 3 * t) + dist3(x, y, z, A.rx + 3 * r);
        const unsigned gamma =
            (unsigned)(unsigned long long)llrint(frac(dc * A.df * A.inv_c) * 4294967296.0);
        const int64_t C = (int64_t)A.T * A.R;
        const float2 *s = turned + (int64_t)t * A.R + r;
        unsigned u = 0u;
#pragma unroll 2
        for (int k = 0; k < A.K; k++, u += gamma) {
            const float2 v = s[k * C];
            const float f = (float)(int)u * 2.3283064365386963e-10f;
            const float c = __builtin_amdgcn_cosf(f), w = __builtin_amdgcn_sinf(f);
            const float re = v.x * c - v.y * w, im = v.x * w + v.y * c;
#pragma unroll
            for (int j = 0; j < N; j++) {
                const float l = L[(int64_t)j * A.K + k];
                acc[j].x = fmaf(l, re, acc[j].x);
                acc[j].y = fmaf(l, im, acc[j].y);
            }
        }
#pragma unroll
        for (int j = 0; j < N; j++) {
            const float f = (float)(int)(gamma * (unsigned)A.nodes[j]) * 2.3283064365386963e-10f;
            const float c = __builtin_amdgcn_cosf(f), w = -__builtin_amdgcn_sinf(f);
            acc[j] = make_float2(acc[j].x * c - acc[j].y * w, acc[j].x * w + acc[j].y * c);
        }
    }
#pragma unroll
    for (int j = 0; j < N; j++) sh[j][tid] = acc[j];
    __syncthreads();
    // fragment lane l of node j: row l % 16, receivers 8 (l / 16) + e
    for (int e = tid; e < N * 64; e += 512) {
        const int j = e >> 6, lane = e & 63;
        float2 v[8];
        for (int q = 0; q < 8; q++) v[q] = sh[j][(lane & 15) * 32 + (lane >> 4) * 8 + q];
        store_frag(v, Sf, (((int64_t)blk * N + j) * TB + tb) * RS + rs, lane);
    }
}

template <int TB, int RS>
__global__ __launch_bounds__(BG_W * 64, TB * RS == 2 ? 4 : 2) void k_bp_mfma(BpMfmaArgs A)
{
    constexpr int NF = 4 * TB * RS;
    __shared__ uint4 Ss[2][NF * 64];
    __shared__ double elem[3 * (TB * 16 + RS * 32)];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q4 = lane >> 4;
    const int blk = blockIdx.x / A.wgs;
    const int bz = blk % A.nbz, by = blk / A.nbz % A.nby, bx = blk / A.nbz / A.nby;
    int i0, i1, j0, j1, k0, k1;
    block_span(bx, A.nbx, A.nx, i0, i1);
    block_span(by, A.nby, A.ny, j0, j1);
    block_span(bz, A.nbz, A.nz, k0, k1);
    const int64_t row = k1 - k0, plane = row * (j1 - j0), n_vox = plane * (i1 - i0);
    const int64_t first = (int64_t)(blockIdx.x - blk * A.wgs) * (BG_W * BG_VW);
    if (first >= n_vox) return;
    // LDS DMA of one frequency's fragments, shared by the wavefronts
    const uint4 *Sb = A.Sf + (int64_t)blk * A.n * (NF * 64);
    auto fetch = [&](int n, int buf) {
        const uint4 *src = Sb + (int64_t)n * (NF * 64) + lane;
#pragma unroll
        for (int q = 0; q < NF / BG_W; q++) {
            const int c = w * (NF / BG_W) + q;
            __builtin_amdgcn_global_load_lds(
                (const __attribute__((address_space(1))) void *)(src + c * 64),
                (__attribute__((address_space(3))) void *)(&Ss[buf][c * 64]), 16, 0, 0);
        }
    };
    fetch(0, 0);                          // in flight while the legs are formed
    for (int e = threadIdx.x; e < 3 * (A.T + A.R); e += BG_W * 64)
        elem[e] = e < 3 * A.T ? A.tx[e] : A.rx[e - 3 * A.T];
    const int64_t v = first + w * BG_VW + (lane & 15);
    const bool valid = v < n_vox;
    const int64_t vv = valid ? v : 0;
    const int i = i0 + (int)(vv / plane);
    const int64_t rem = vv % plane;
    const int j = j0 + (int)(rem / row), k = k0 + (int)(rem % row);
    const double x = A.x0 + (double)i * A.step, y = A.y0 + (double)j * A.step,
                 z = A.z0 + (double)k * A.step;
    // this lane's legs, metres and (nodes) turns at the middle sample's
    // frequency: the Tx rows of its accumulator elements (16 tb + 4 q4 + e)
    // and the Rx rows of its B-operand slots (32 rs + 8 q4 + e)
    const double fmid = A.nodes ? (A.f0 + 0.5 * (A.K - 1) * A.df) * A.inv_c : 0.0;
    float dt[TB * 4], pt[TB * 4], dr[RS * 8], pr[RS * 8];
    __syncthreads();
    auto leg = [&](const double *e, float &d, float &turns) {
        const double ax = x - e[0], ay = y - e[1], az = z - e[2];
        d = (float)leg_sqrt(ax * ax + ay * ay + az * az);
        const double u = (double)d * fmid;
        turns = (float)(u - rint(u));
    };
#pragma unroll
    for (int tb = 0; tb < TB; tb++)
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const int t = tb * 16 + 4 * q4 + e;
            leg(elem + 3 * min(t, A.T - 1), dt[tb * 4 + e], pt[tb * 4 + e]);
        }
#pragma unroll
    for (int rs = 0; rs < RS; rs++)
#pragma unroll
        for (int e = 0; e < 8; e++) {
            const int r = rs * 32 + 8 * q4 + e;
            leg(elem + 3 * (A.T + min(r, A.R - 1)), dr[rs * 8 + e], pr[rs * 8 + e]);
        }
    float img_re = 0.0f, img_im = 0.0f;
    // the B operands of one frequency: receive phasors of this lane's voxel
    // for its receiver slots, split into six bf16 planes per step
    struct BOps {
        uint4 rh[RS], rl[RS], ih[RS], il[RS], nih[RS], nil[RS];
    };
    auto gen_b = [&](float fc, BOps &b) {
#pragma unroll
        for (int rs = 0; rs < RS; rs++) {
            float br[8], bi[8];
#pragma unroll
            for (int e = 0; e < 8; e++) {
                const float ph = fmaf(dr[rs * 8 + e], fc, pr[rs * 8 + e]);
                br[e] = __builtin_amdgcn_cosf(ph);
                bi[e] = __builtin_amdgcn_sinf(ph);
            }
            unsigned *prh = &b.rh[rs].x, *prl = &b.rl[rs].x, *pih = &b.ih[rs].x, *pil = &b.il[rs].x;
#pragma unroll
            for (int q = 0; q < 4; q++) {
                split_bf16(br[2 * q], br[2 * q + 1], prh[q], prl[q]);
                split_bf16(bi[2 * q], bi[2 * q + 1], pih[q], pil[q]);
            }
            b.nih[rs] = neg(b.ih[rs]);
            b.nil[rs] = neg(b.il[rs]);
        }
    };
    // turns per metre of sample n, of node n beyond the middle frequency
    auto freq = [&](int n) {
        return A.nodes ? (float)(((double)A.nodes[n] - 0.5 * (A.K - 1)) * A.df * A.inv_c)
                       : (float)((A.f0 + (double)n * A.df) * A.inv_c);
    };
    f32x4 ur[TB], ui[TB];
    // transmit phasors of this lane's Tx rows times U (D layout: element e of
    // lane l is row 4 (l / 16) + e, column l % 16 of each block)
    auto tx_sum = [&](float fc) {
#pragma unroll
        for (int tb = 0; tb < TB; tb++)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const float ph = fmaf(dt[tb * 4 + e], fc, pt[tb * 4 + e]);
                const float ar = __builtin_amdgcn_cosf(ph), ai = __builtin_amdgcn_sinf(ph);
                img_re = fmaf(ar, ur[tb][e], fmaf(-ai, ui[tb][e], img_re));
                img_im = fmaf(ar, ui[tb][e], fmaf(ai, ur[tb][e], img_im));
            }
    };
    // The two wavefronts of a SIMD take turns: the leading half (w >= 4)
    // starts a frequency with its matrix products while the other half adds
    // the last frequency's Tx sum and generates this one's phasors, and the
    // other way round after that, so that neither waits for the other's
    // vector work.  With two Tx blocks' sums in turn and priority for products
    // the hand's image takes 7.4 instead of 8.1 ms (Tx sums of both halves
    // before the barrier, one block at a time): 1.19 PFLOP/s of split products.
    const bool lead = w >= BG_W / 2;
    BOps b;
    if (lead) gen_b(freq(0), b);
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    const f32x4 zero = {};
    for (int n = 0; n < A.n; n++) {
        if (!lead) {
            if (n) tx_sum(freq(n - 1));
            gen_b(freq(n), b);
        }
        const uint4 *S = Ss[n & 1];
        __builtin_amdgcn_s_setprio(1);    // products first, vector work in between
#pragma unroll
        for (int rs = 0; rs < RS; rs++) {
            // two Tx blocks at a time: four independent sums in turn (a chain's
            // next product waits for the last one's result)
#pragma unroll
            for (int tb = 0; tb < TB; tb += 2) {
                // U_re += Sr Br - Si Bi, U_im += Sr Bi + Si Br (hi*hi + hi*lo + lo*hi)
                auto both = [&](int pl, const uint4 &re, const uint4 &im, bool set) {
#pragma unroll
                    for (int h = 0; h < 2; h++) {
                        const uint4 f = S[(((tb + h) * RS + rs) * 4 + pl) * 64 + lane];
                        ur[tb + h] = MFMA(f, re, set ? zero : ur[tb + h]);
                        ui[tb + h] = MFMA(f, im, set ? zero : ui[tb + h]);
                    }
                };
                both(0, b.rh[rs], b.ih[rs], rs == 0);
                both(0, b.rl[rs], b.il[rs], false);
                both(1, b.rh[rs], b.ih[rs], false);
                both(2, b.nih[rs], b.rh[rs], false);
                both(2, b.nil[rs], b.rl[rs], false);
                both(3, b.nih[rs], b.rh[rs], false);
            }
        }
        __builtin_amdgcn_s_setprio(0);
        // every wavefront has read this frequency's slice: the next one may
        // be requested into the other buffer
        if (n + 1 < A.n) fetch(n + 1, (n + 1) & 1);
        if (lead) {
            tx_sum(freq(n));
            if (n + 1 < A.n) gen_b(freq(n + 1), b);
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    }
    if (!lead) tx_sum(freq(A.n - 1));
    // the four lanes l % 16 + 16 q hold the four quarters of one voxel's Tx rows
    img_re += __shfl_xor(img_re, 16);
    img_im += __shfl_xor(img_im, 16);
    img_re += __shfl_xor(img_re, 32);
    img_im += __shfl_xor(img_im, 32);
    if (valid && q4 == 0)
        A.image[((int64_t)i * A.ny + j) * A.nz + k] = make_float2(img_re, img_im);
}

int tx_blocks(int T) { return T <= 32 ? 2 : T <= 64 ? 4 : 6; }
int rx_steps(int R) { return (R + 31) / 32; }

// Longest change of a leg over a block of half-extents h about its centre: by
// the mean value theorem it is g . h' for a unit vector g from an element to a
// point of the volume and |h'_i| <= h_i; g_i is at most the axis's greatest
// element-to-volume offset over that and the other axes' least.
double leg_reach(const BpGrid &G, const double *elem_box, const double *h)
{
    double least[3], most[3], g[3];
    for (int a = 0; a < 3; a++) {
        const double v0 = G.lo[a], v1 = G.hi[a], e0 = elem_box[a], e1 = elem_box[3 + a];
        least[a] = std::max(0.0, std::max(v0 - e1, e0 - v1));
        most[a] = std::max(std::fabs(v1 - e0), std::fabs(e1 - v0));
    }
    for (int a = 0; a < 3; a++) {
        const int b = (a + 1) % 3, c = (a + 2) % 3;
        const double n = std::sqrt(most[a] * most[a] + least[b] * least[b] + least[c] * least[c]);
        g[a] = n > 0.0 ? most[a] / n : 1.0;
    }
    // max of g . h over |g_i| <= g[i], |g| <= 1: along h, axes at their bound
    // fixed and the rest of the unit length given to the others
    bool at[3] = {false, false, false};
    double sum = 0.0, left = 1.0;
    for (int it = 0; it < 3; it++) {
        double hh = 0.0;
        for (int a = 0; a < 3; a++)
            if (!at[a]) hh += h[a] * h[a];
        const double s = hh > 0.0 ? std::sqrt(std::max(left, 0.0) / hh) : 0.0;
        int hit = -1;
        for (int a = 0; a < 3; a++)
            if (!at[a] && s * h[a] > g[a]) hit = a;
        if (hit < 0) return sum + s * hh;
        at[hit] = true;
        sum += g[hit] * h[hit];
        left -= g[hit] * g[hit];
    }
    return sum;
}

}  // namespace

// The plan of least modelled time: every sample over the whole volume, or the
// nodes of a class over blocks as large as its reach z allows.  Per voxel,
// frequency and full 96 x 96 tile 1.6e-4 us (66 ms for 3.27e6 voxels at 128
// samples), 100 us of start-up shared with what runs anyway; a block's slices
// 2 n + 16 vector instructions per channel and sample, and 8 bytes of bf16
// planes per channel and node written and read by its workgroups.
BpPlan bp_plan(const BpGrid &G, const BandClasses &cls)
{
    BpPlan best{};
    const int TB = tx_blocks(G.T), RS = rx_steps(G.R);
    const double tile = TB * RS / 18.0, C = (double)G.T * G.R;
    const double vox = (double)G.n[0] * G.n[1] * G.n[2];
    const double rate = 1.6e-4 * (0.2 + 0.8 * tile);
    best.n = G.K;
    best.cls = -1;
    for (int a = 0; a < 3; a++) best.nb[a] = 1;
    best.wgs = (int)std::min<double>((vox + BG_W * BG_VW - 1) / (BG_W * BG_VW), 2147483647.0);
    double cost = vox * G.K * rate;
    // device full from 256 workgroups on: fewer take as long as one each
    auto rounds = [&](double wgs) { return std::max(1.0, 256.0 / std::max(wgs, 1.0)); };
    cost *= rounds(best.wgs);
    for (int q = 0; q < cls.count; q++) {
        const double reach = cls.z[q] / (M_PI * std::fabs(G.df) * (G.K - 1)) / G.inv_c;
        int edge = 1, over = 513;        // the longest edge within reach
        while (over - edge > 1) {
            const int e = (edge + over) / 2;
            double h[3];
            for (int a = 0; a < 3; a++) h[a] = 0.5 * (std::min(e, G.n[a]) - 1) * G.step;
            if (leg_reach(G, G.box, h) + leg_reach(G, G.box + 6, h) <= reach) edge = e; else over = e;
        }
        if (edge < 2) continue;
        BpPlan p{};
        p.cls = q;
        p.n = cls.n[q];
        double blocks = 1.0, big = 1.0;
        for (int a = 0; a < 3; a++) {
            p.nb[a] = (G.n[a] + edge - 1) / edge;
            blocks *= p.nb[a];
            big *= (G.n[a] + p.nb[a] - 1) / p.nb[a];
        }
        p.wgs = (int)((big + BG_W * BG_VW - 1) / (BG_W * BG_VW));
        // fewer than 2^32 threads a launch, at most 4 GiB of slices
        if (blocks * p.wgs * (BG_W * 64) >= 4294967296.0 || blocks * p.n * TB * RS * 4096.0 > 4.0 * (1u << 30))
            continue;
        const double t = blocks * p.wgs * BG_W * BG_VW * p.n * rate * rounds(blocks * p.wgs) +
                         blocks * C * G.K * (2.0 * p.n + 16.0) * 2.6e-8 + blocks * C * p.n * 2e-6 + 15.0;
        if (t < cost) {
            cost = t;
            best = p;
        }
    }
    best.frag_bytes = (int64_t)best.nb[0] * best.nb[1] * best.nb[2] * best.n * TB * RS * 4096;
    best.turn_bytes = best.cls >= 0 ? (int64_t)(C * G.K * 8) : 0;
    return best;
}

hipError_t launch_bp_mfma(const BpGrid &G, const BpPlan &P, const float2 *cube, int64_t stride,
                          const double *tx, const double *rx, const int32_t *nodes, const float *coef,
                          float2 *turned, uint4 *Sf, float2 *image, hipStream_t s)
{
    if (G.K <= 0) return hipSuccess;
    if (G.T < 1 || G.R < 1 || G.T > 96 || G.R > 96) return hipErrorInvalidValue;
    const int TB = tx_blocks(G.T), RS = rx_steps(G.R), C = G.T * G.R;
    const int64_t blocks = (int64_t)P.nb[0] * P.nb[1] * P.nb[2];
    BpMfmaArgs A;
    A.Sf = Sf;
    A.tx = tx;
    A.rx = rx;
    A.T = G.T;
    A.R = G.R;
    A.K = G.K;
    A.f0 = G.f0;
    A.df = G.df;
    A.inv_c = G.inv_c;
    A.x0 = G.lo[0];
    A.y0 = G.lo[1];
    A.z0 = G.lo[2];
    A.step = G.step;
    A.nx = G.n[0];
    A.ny = G.n[1];
    A.nz = G.n[2];
    A.nbx = P.nb[0];
    A.nby = P.nb[1];
    A.nbz = P.nb[2];
    A.wgs = P.wgs;
    A.n = P.n;
    A.nodes = P.cls >= 0 ? nodes : nullptr;
    A.image = image;
    if (P.cls < 0) {
        const int64_t nf = (int64_t)G.K * TB * RS * 64;
        hipLaunchKernelGGL(k_bp_prep, dim3((unsigned)((nf + 255) / 256)), dim3(256), 0, s, cube, stride,
                           G.T, G.R, G.K, TB, RS, Sf);
    } else {
        const int tb = ((C + 31) / 32) * ((G.K + 31) / 32);
        hipLaunchKernelGGL(k_bp_turn, dim3((unsigned)tb), dim3(256), 0, s, cube, stride, C, G.K, turned);
        const dim3 g((unsigned)(blocks * TB * RS)), t(512);
#define BP_BLOCK(N) case N: hipLaunchKernelGGL(k_bp_block<N>, g, t, 0, s, A, turned, coef, TB, RS, Sf); break
        switch (P.n) {
        BP_BLOCK(8);
        BP_BLOCK(12);
        BP_BLOCK(16);
        BP_BLOCK(20);
        BP_BLOCK(24);
        BP_BLOCK(28);
        BP_BLOCK(32);
        default: return hipErrorInvalidValue;
        }
#undef BP_BLOCK
    }
    const dim3 g((unsigned)(blocks * P.wgs)), t(BG_W * 64);
#define BP_MAIN(TBV, RSV) \
    if (TB == TBV && RS == RSV) hipLaunchKernelGGL((k_bp_mfma<TBV, RSV>), g, t, 0, s, A)
    BP_MAIN(2, 1);
    BP_MAIN(2, 2);
    BP_MAIN(2, 3);
    BP_MAIN(4, 1);
    BP_MAIN(4, 2);
    BP_MAIN(4, 3);
    BP_MAIN(6, 1);
    BP_MAIN(6, 2);
    BP_MAIN(6, 3);
#undef BP_MAIN
    return hipGetLastError();
}
