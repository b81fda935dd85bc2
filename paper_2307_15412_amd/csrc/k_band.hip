// k_band.hip -- bands of path lengths: the one-chirp sum of a shared launch
// from a few samples per band instead of every sample.
//
// Path p adds exp(-j 2 pi k gamma_p) to sample k (gamma = B d / (K c) turns).
// Paths whose lengths, over every channel, lie in one narrow band make a sum
// that is band-limited about the band's centre gamma_b, so its values at n of
// the K samples (the nodes) give all of them:
//     s[k] = exp(-j 2 pi k gamma_b) sum_j L[k, j] exp(+j 2 pi r_j gamma_b) s[r_j],
// with L the coefficients of rr_bands.cpp (error below 2e-7 of a path's
// amplitude).  The returns of a street or a hand crowd into a few range bins
// (99 % of the large-MIMO street's 1e5 paths within 4 m, 512 samples cover
// 154 m), so the Tx x Rx products of the product engine run over 12-24 nodes
// instead of 128-512 samples.  What is left is the expansion, 2 n + 4 FP32
// multiply-adds per channel, sample and band, and the cube itself.  Measured:
// the hand's cube (94 x 94 channels, 128 samples, 5.0e5 paths) 13.9 -> 2.1 ms,
// of it the products 2.0 (14.4 at every sample), leg tables 0.25; the resting
// paths of the large-MIMO cube 5.4 -> 0.4 ms.  The products' vector work (two
// hardware sin/cos per phasor) still bounds them, as at every sample.
//
// On the device, so that a batched launch can capture it: every path gets a
// band (BK_BINS range bins wide, by the middle of its lengths), counts and extents
// per band come from block histograms, one workgroup then plans (which bands
// run on which class of nodes; thin ones, bands too wide for every class and
// what lies beyond RR_BANDS bands go together into a last list computed at
// every sample) and the paths are placed in band order, stably, so that the
// sums repeat bit for bit.
#include <algorithm>

#include "rr_internal.h"

namespace {

#define BK_T 1024
#define BK_P 4096          // paths per block of the histograms
#define BK_NONE 511        // key of no path (all bits set)
// width of a band in range bins: the separable model's bands, which have the
// array's offsets taken out, then reach z = 1.34 and run on 8 nodes (products
// of the large-MIMO street 0.17 ms, at two bins a band 0.25); the hand's run
// on 12 to 20 nodes (mean 15.6, at two bins 16.8; 0.4 bins 15.3)
#define BK_BINS 0.85

__device__ __forceinline__ double frac(double x) { return x - floor(x); }

__device__ __forceinline__ double dist3(const double *a, const double *b)
{
    const double dx = a[0] - b[0], dy = a[1] - b[1], dz = a[2] - b[2];
    return sqrt(dx * dx + dy * dy + dz * dz);
}

// least and greatest distance of q from the points of a box (a bound for the
// array's elements within it)
__device__ __forceinline__ void box_dist(const double *q, const double *lo, const double *hi,
                                         double &dmin, double &dmax)
{
    double n2 = 0.0, f2 = 0.0;
    for (int a = 0; a < 3; a++) {
        const double u = lo[a] - q[a], v = q[a] - hi[a];
        const double n = fmax(fmax(u, v), 0.0), f = fmax(fabs(u), fabs(v));
        n2 += n * n;
        f2 += f * f;
    }
    dmin = sqrt(n2);
    dmax = sqrt(f2);
}

__device__ __forceinline__ int64_t path_count(const int64_t *lo, const int64_t *hi, int64_t Ppad)
{
    return min(max(*hi - *lo, (int64_t)0), Ppad);
}

// Per path the band, per block the count and the extent of every band.  The
// extents are lengths >= 0 as FP32 bits, which order as integers.
__global__ __launch_bounds__(BK_T) void k_band_key(BandArgs A)
{
    __shared__ unsigned cnt[RR_BANDS + 1], lo_s[RR_BANDS + 1], hi_s[RR_BANDS + 1];
    for (int64_t p = (int64_t)blockIdx.x * BK_T + threadIdx.x; p < A.perm_cap; p += (int64_t)gridDim.x * BK_T)
        A.perm[p] = -1;
    const int64_t n = path_count(A.L.rng_lo, A.L.rng_hi, A.Ppad);
    const int64_t base = (int64_t)blockIdx.x * BK_P;
    if (base >= n) return;
    for (int b = threadIdx.x; b <= RR_BANDS; b += BK_T) {
        cnt[b] = 0u;
        lo_s[b] = 0x7f800000u;
        hi_s[b] = 0u;
    }
    __syncthreads();
    const SynPath *paths = A.L.paths + *A.L.rng_lo;
    for (int j = 0; j < BK_P / BK_T; j++) {
        const int64_t p = base + j * BK_T + threadIdx.x;
        if (p >= n) break;
        const SynPath &P = paths[p];
        const int K = P.K;
        double inner = 0.0;
        for (int q = 1; q < K; q++) inner += dist3(P.P[q], P.P[q - 1]);
        double lo, hi;
        if (A.L.sep) {
            const double *os = P.src >= 0 ? A.L.tx + 3 * P.src : A.L.oT;
            lo = hi = dist3(P.P[0], os) + inner + dist3(A.L.oR, P.P[K - 1]);
        } else {
            double a, b, c, d;
            box_dist(P.P[0], A.tx_lo, A.tx_hi, a, b);
            box_dist(P.P[K - 1], A.rx_lo, A.rx_hi, c, d);
            lo = a + inner + c;
            hi = b + inner + d;
        }
        const double bins = 0.5 * (lo + hi) * A.bins_per_m;
        const double at = bins / BK_BINS;
        const int band = at < (double)RR_BANDS ? (int)at : RR_BANDS;
        A.keys[p] = (uint16_t)band;
        atomicAdd(&cnt[band], 1u);
        atomicMin(&lo_s[band], __float_as_uint((float)lo));
        atomicMax(&hi_s[band], __float_as_uint((float)hi));
    }
    __syncthreads();
    for (int b = threadIdx.x; b <= RR_BANDS; b += BK_T) {
        const int64_t o = (int64_t)blockIdx.x * (RR_BANDS + 1) + b;
        A.hist[o] = cnt[b];
        A.extent[o] = make_uint2(lo_s[b], hi_s[b]);
    }
}

// inclusive scan over a 512-thread block
__device__ __forceinline__ int scan512(int v, int *sh, int &total)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int off = 1; off < 64; off <<= 1) {
        const int u = __shfl_up(v, off);
        if (lane >= off) v += u;
    }
    __syncthreads();
    if (lane == 63) sh[w] = v;
    __syncthreads();
    total = 0;
    int before = 0;
    for (int j = 0; j < 8; j++) {
        if (j < w) before += sh[j];
        total += sh[j];
    }
    return v + before;
}

// One workgroup: classes of the bands, the order of the paths and the list of
// segments (at most `len` paths of one band each), their products' work items
// (four samples of one segment) and the slots of their partial sums.
__global__ __launch_bounds__(512) void k_band_plan(BandArgs A)
{
    __shared__ int sh[8];
    __shared__ unsigned long long work;
    __shared__ int s_first[RR_BANDS + 2], s_item[RR_BANDS + 2], s_slot[RR_BANDS + 2];
    __shared__ int s_base[RR_BANDS + 1], s_cnt[RR_BANDS + 1], s_grp[RR_BANDS + 1];
    const int b = threadIdx.x;                 // list b < RR_BANDS: a band; RR_BANDS: the rest
    const int64_t n = path_count(A.L.rng_lo, A.L.rng_hi, A.Ppad);
    const int nblk = (int)((n + BK_P - 1) / BK_P);
    if (b == 0) work = 0ull;
    int cnt = 0;
    unsigned lo = 0x7f800000u, hi = 0u;
    if (b <= RR_BANDS)
#pragma unroll 8
        for (int i = 0; i < nblk; i++) {
            const int64_t o = (int64_t)i * (RR_BANDS + 1) + b;
            const uint2 e = A.extent[o];
            cnt += (int)A.hist[o];
            lo = min(lo, e.x);
            hi = max(hi, e.y);
        }
    int cls = -1;
    unsigned gamma = 0u;
    if (b < RR_BANDS && cnt >= BAND_THIN) {
        const double l = __uint_as_float(lo), h = __uint_as_float(hi);
        const double z = M_PI * (A.K - 1) / A.K * 0.5 * (h - l) * A.bins_per_m;
        for (int q = A.cls.count - 1; q >= 0; q--)
            if (z <= (double)A.cls.z[q]) cls = q;
        gamma = (unsigned)(unsigned long long)llrint(frac(0.5 * (l + h) * A.L.dfc) * 4294967296.0);
    }
    // the paths of a list: a band's own, or those of every band without a class
    int total;
    const int nodes = cls >= 0 ? A.cls.n[cls] : A.K;
    scan512(cls >= 0 || b > RR_BANDS ? 0 : cnt, sh, total);
    const int mine = cls >= 0 ? cnt : b == RR_BANDS ? total : 0;
    const int pad = (mine + 31) & ~31;
    int all;
    const int base = scan512(pad, sh, all) - pad;
    const int groups = (nodes + 3) / 4;
    if (pad) atomicAdd(&work, (unsigned long long)pad * groups);
    // chunks as long as fill the target exactly when every list ends in a
    // short one
    int ends;
    scan512(pad ? groups : 0, sh, ends);
    const unsigned long long fit = (unsigned long long)max(A.target - ends, A.target / 2);
    const int len = max(256, (int)(((work + fit - 1) / fit + 31) & ~31ull));
    const int chunks = (pad + len - 1) / len;
    int n_segs, n_items, n_slots, n_out;
    const int seg0 = scan512(chunks, sh, n_segs) - chunks;
    const int item0 = scan512(chunks * groups, sh, n_items) - chunks * groups;
    const int slot0 = scan512(chunks * groups * 4, sh, n_slots) - chunks * groups * 4;
    const int out0 = scan512(chunks ? 1 : 0, sh, n_out) - (chunks ? 1 : 0);
    int n_rows;
    const int rows = chunks > 1 ? (cls >= 0 ? nodes : groups * 4) : 0;
    const int row0 = scan512(rows, sh, n_rows) - rows;
    if (b <= RR_BANDS) {
        s_first[b] = seg0;
        s_item[b] = item0;
        s_slot[b] = slot0;
        s_base[b] = base;
        s_cnt[b] = pad;
        s_grp[b] = cls >= 0 ? groups : -groups;
        // where this band's paths go: its own list, or after those of the
        // classless bands before it
        A.plan->base[b] = base;
        if (chunks) {
            BandOut &o = A.plan->out[out0];
            o.cls = cls;
            o.n = cls >= 0 ? nodes : groups * 4;
            o.chunks = chunks;
            o.slot0 = slot0;
            o.row0 = row0;
            o.gamma = gamma;
        }
    }
    if (b == 0) {
        A.plan->used = all;
        A.plan->n_segs = n_segs;
        A.plan->n_items = n_items;
        A.plan->n_out = n_out;
        A.plan->n_rows = n_rows;
        A.plan->next = 0;
    }
    __syncthreads();
    // classless bands: consecutive places in the last list
    int dummy;
    const int left = b <= RR_BANDS && cls < 0 ? cnt : 0;
    const int before = scan512(left, sh, dummy) - left;
    if (b <= RR_BANDS && cls < 0) A.plan->base[b] = s_base[RR_BANDS] + before;
    for (int s = b; s < n_segs; s += 512) {
        int l = 0, h = RR_BANDS;
        while (l < h) {
            const int m = (l + h + 1) / 2;
            if (s_first[m] <= s) l = m; else h = m - 1;
        }
        // empty lists share their first segment with the next one: the last
        // list that starts at or before s is the one that holds it
        const int c = s - s_first[l], g = abs(s_grp[l]);
        BandSeg q;
        q.p0 = s_base[l] + c * len;
        q.np = min(len, s_cnt[l] - c * len);
        q.groups = g;
        q.item0 = s_item[l] + c * g;
        q.slot0 = s_slot[l] + c * g * 4;
        q.cls = -1;
        if (s_grp[l] > 0)
            for (int k = 0; k < A.cls.count; k++)
                if (A.cls.n[k] == 4 * g) q.cls = k;
        A.segs[s] = q;
    }
}

// Stable placement: within a block, paths of one band in path order (rank in
// the wavefront by ballots over the key's bits, wavefronts in turn), blocks
// after one another.
__global__ __launch_bounds__(BK_T) void k_band_place(BandArgs A)
{
    __shared__ int at[RR_BANDS + 1];
    __shared__ int wcnt[BK_T / 64][RR_BANDS + 1];
    const int64_t n = path_count(A.L.rng_lo, A.L.rng_hi, A.Ppad);
    const int64_t base = (int64_t)blockIdx.x * BK_P;
    if (base >= n) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int b = threadIdx.x; b <= RR_BANDS; b += BK_T) {
        int v = A.plan->base[b];
#pragma unroll 8
        for (int i = 0; i < (int)blockIdx.x; i++) v += (int)A.hist[(int64_t)i * (RR_BANDS + 1) + b];
        at[b] = v;
    }
    for (int j = 0; j < BK_P / BK_T; j++) {
        __syncthreads();
        for (int e = threadIdx.x; e < BK_T / 64 * (RR_BANDS + 1); e += BK_T) (&wcnt[0][0])[e] = 0;
        __syncthreads();
        const int64_t p = base + j * BK_T + threadIdx.x;
        const int key = p < n ? (int)A.keys[p] : BK_NONE;
        unsigned long long same = ~0ull;
        for (int bit = 0; bit < 9; bit++) {
            const bool set = (key >> bit) & 1;
            const unsigned long long m = __ballot(set);
            same &= set ? m : ~m;
        }
        const int rank = __popcll(same & ((1ull << lane) - 1));
        if (rank == 0 && key <= RR_BANDS) wcnt[w][key] = __popcll(same);
        __syncthreads();
        for (int b = threadIdx.x; b <= RR_BANDS; b += BK_T) {
            int run = at[b];
            for (int v = 0; v < BK_T / 64; v++) {
                const int c = wcnt[v][b];
                wcnt[v][b] = run;
                run += c;
            }
            at[b] = run;
        }
        __syncthreads();
        if (key <= RR_BANDS) A.perm[wcnt[w][key] + rank] = (int32_t)p;
    }
}

__device__ __forceinline__ float2 cis(unsigned u, float sign)
{
    float s, c;
    sincospif((float)(int)u * 4.6566128730773926e-10f, &s, &c);   // 2 u / 2^32
    return make_float2(c, sign * s);
}

// The chunks' partial sums of every list of several added in order, into its
// first chunk's: one thread per (partial sum, channel) of the first chunk, so
// that the loads of many chunks are in flight at once (summed as the
// expansion read them, the hand's 280 MB took 0.26 ms).
__global__ __launch_bounds__(256) void k_band_sum(const BandPlan *plan, float2 *part, int C)
{
    const int c = blockIdx.x * 256 + threadIdx.x;
    const int n_rows = plan->n_rows;
    for (int row = blockIdx.y; row < n_rows; row += gridDim.y) {
        // lists of one chunk have no rows and start where the next one does
        int lo = 0, hi = plan->n_out - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) / 2;
            if (plan->out[mid].row0 <= row) lo = mid; else hi = mid - 1;
        }
        while (plan->out[lo].chunks < 2) lo--;
        const BandOut B = plan->out[lo];
        if (c >= C) continue;
        float2 *p = part + ((int64_t)B.slot0 + row - B.row0) * C + c;
        const int64_t step = (int64_t)B.n * C;
        float2 v = p[0];
#pragma unroll 8
        for (int i = 1; i < B.chunks; i++) {
            const float2 u = p[i * step];
            v.x += u.x;
            v.y += u.y;
        }
        p[0] = v;
    }
}

// Samples of BE_C channels (one a lane, over the block) from the lists' sums:
// a band's node sums, the centre's rotation taken out, go to LDS; each lane
// forms its sample for every channel with its own coefficients, L[.][k], and
// turns it back.  The last list's sums are samples already.
#define BE_C 8
__global__ __launch_bounds__(512) void k_band_expand(BandArgs A, const float2 *part, int C, float2 *out)
{
    __shared__ float2 z[2][RR_BAND_NMAX][BE_C];
    const int c0 = blockIdx.x * BE_C;
    const int k = blockIdx.y * blockDim.x + threadIdx.x;
    const bool kv = k < A.K;
    const int kc = kv ? k : A.K - 1;
    float2 acc[BE_C];
#pragma unroll
    for (int c = 0; c < BE_C; c++) acc[c] = make_float2(0.0f, 0.0f);
    const int n_out = A.plan->n_out;
    for (int o = 0; o < n_out; o++) {
        const BandOut B = A.plan->out[o];
        if (B.cls < 0) {
            const float2 *p = part + ((int64_t)B.slot0 + kc) * C;
#pragma unroll
            for (int c = 0; c < BE_C; c++) {
                const float2 v = p[min(c0 + c, C - 1)];
                acc[c].x += v.x;
                acc[c].y += v.y;
            }
            continue;
        }
        const int32_t *nodes = A.nodes + B.cls * RR_BAND_NMAX;
        for (int e = threadIdx.x; e < B.n * BE_C; e += blockDim.x) {
            const int j = e / BE_C, c = min(c0 + e % BE_C, C - 1);
            const float2 v = part[((int64_t)B.slot0 + j) * C + c];
            const float2 r = cis(B.gamma * (unsigned)nodes[j], 1.0f);
            z[o & 1][j][e % BE_C] = make_float2(v.x * r.x - v.y * r.y, v.x * r.y + v.y * r.x);
        }
        // one barrier per band: the other buffer's readers passed the last one
        __syncthreads();
        float2 y[BE_C];
#pragma unroll
        for (int c = 0; c < BE_C; c++) y[c] = make_float2(0.0f, 0.0f);
        const float *L = A.coef + A.cls.coef[B.cls] + kc;
#pragma unroll 4
        for (int j = 0; j < B.n; j++) {
            const float l = L[(int64_t)j * A.K];
#pragma unroll
            for (int c = 0; c < BE_C; c++) {
                const float2 v = z[o & 1][j][c];
                y[c].x = fmaf(l, v.x, y[c].x);
                y[c].y = fmaf(l, v.y, y[c].y);
            }
        }
        const float2 r = cis(B.gamma * (unsigned)kc, -1.0f);
#pragma unroll
        for (int c = 0; c < BE_C; c++) {
            acc[c].x += y[c].x * r.x - y[c].y * r.y;
            acc[c].y += y[c].x * r.y + y[c].y * r.x;
        }
    }
    if (!kv) return;
#pragma unroll
    for (int c = 0; c < BE_C; c++)
        if (c0 + c < C) out[(int64_t)(c0 + c) * A.K + k] = acc[c];
}

}  // namespace

int64_t band_blocks(int64_t Ppad) { return (Ppad + BK_P - 1) / BK_P; }

hipError_t launch_band_plan(const BandArgs &A, hipStream_t s)
{
    if (A.Ppad <= 0 || A.cls.count <= 0 || A.target <= 0) return hipErrorInvalidValue;
    const dim3 g((unsigned)band_blocks(A.Ppad));
    hipLaunchKernelGGL(k_band_key, g, dim3(BK_T), 0, s, A);
    hipLaunchKernelGGL(k_band_plan, dim3(1), dim3(512), 0, s, A);
    hipLaunchKernelGGL(k_band_place, g, dim3(BK_T), 0, s, A);
    return hipGetLastError();
}

hipError_t launch_band_expand(const BandArgs &A, float2 *part, int C, float2 *out, hipStream_t s)
{
    const int cb = (C + 255) / 256;
    hipLaunchKernelGGL(k_band_sum, dim3((unsigned)cb, (unsigned)std::max(1, std::min(512, 4096 / cb))),
                       dim3(256), 0, s, A.plan, part, C);
    const int t = std::min(512, (A.K + 63) / 64 * 64);
    const dim3 g((unsigned)((C + BE_C - 1) / BE_C), (unsigned)((A.K + t - 1) / t));
    hipLaunchKernelGGL(k_band_expand, g, dim3(t), 0, s, A, part, C, out);
    return hipGetLastError();
}
