// k_synth.hip -- direct coherent summation of received paths into the FMCW
// beat-signal cube (Section III-B, Eq. 4, with the stepped frequency replaced
// by the chirp's instantaneous frequency f_k = f0 + B k / K).
//
// Each lane owns one (channel, chirp) row and a run of KR consecutive fast-time
// samples.  Paths are staged through LDS in chunks.  For every (path, row) of
// the chunk the workgroup forms the path length once, in FP64, and reduces
// the carrier phase f0 d / c and the per-sample step B d / (K c) modulo one
// cycle in FP64 (the phase at 77 GHz is ~1e4 cycles, beyond FP32), keeping
// both as 32-bit fixed-point turns in an LDS table.  A lane then forms the
// start phase of its run exactly in integer arithmetic (beta + k0 gamma modulo
// 2^32), takes the hardware sin/cos of it and of the step (input in turns),
// and walks the run by complex rotation, accumulating in FP32 registers.
//
// A path whose every hit rests adds the same to every chirp, so the records
// come in two parts (paths at rest, moving paths): the first part is summed
// once, into chirp 0 of the cube (k_synth_rest), and the sum over the moving
// paths is added to it chirp by chirp (k_synth_direct).  On the street, where
// 99.8 % of the paths lie on the static ground, that is 1/128 of the work.
// A further kernel evaluates individual cube entries fully in FP64 for checks
// at sizes where the whole cube is not needed.
#include <algorithm>

#include "rr_internal.h"

namespace {

#define SYN_T 256
#define SYN_CHUNK 32
#define SYN_TAB 4096      // (path, row) phase entries per chunk: 32 KiB of LDS

__device__ __forceinline__ double dist3(double ax, double ay, double az, double bx, double by,
                                        double bz)
{
    double dx = ax - bx, dy = ay - by, dz = az - bz;
    return sqrt(dx * dx + dy * dy + dz * dz);
}

// Per (path, channel, chirp): lengths such that the phase of sample k is
//   phi_k = d_base * f0 / c + k * d_step * B / (K c)   (cycles).
// Exact model: d_base = d_step = |p_1(m) - tx_t| + inner(m) + |rx_r - p_K(m)|.
// Separable model: d_step = D(m) = |p_1(m) - o_s| + inner(m) + |o_R - p_K(m)|
// and d_base = D(m) + dT + dR with the channel offsets dT, dR taken at chirp 0.
__device__ __forceinline__ void path_lengths(const SynthArgs &A, const SynPath &P, double tau,
                                             const double *tx, const double *rx, double &d_base,
                                             double &d_step)
{
    const int K = P.K;
    double x1 = P.P[0][0] + P.V[0][0] * tau, y1 = P.P[0][1] + P.V[0][1] * tau,
           z1 = P.P[0][2] + P.V[0][2] * tau;
    double xk = x1, yk = y1, zk = z1;
    double inner = 0.0;
    for (int j = 1; j < K; j++) {
        double x = P.P[j][0] + P.V[j][0] * tau, y = P.P[j][1] + P.V[j][1] * tau,
               z = P.P[j][2] + P.V[j][2] * tau;
        inner += dist3(x, y, z, xk, yk, zk);
        xk = x; yk = y; zk = z;
    }
    if (A.model == RR_EXACT) {
        double d = dist3(x1, y1, z1, tx[0], tx[1], tx[2]) + inner +
                   dist3(rx[0], rx[1], rx[2], xk, yk, zk);
        d_base = d;
        d_step = d;
    } else {
        double os[3];
        if (P.src >= 0) {
            os[0] = A.tx[3 * P.src]; os[1] = A.tx[3 * P.src + 1]; os[2] = A.tx[3 * P.src + 2];
        } else {
            os[0] = A.oT[0]; os[1] = A.oT[1]; os[2] = A.oT[2];
        }
        const double *p1 = P.P[0], *pk = P.P[K - 1];
        double dT = dist3(p1[0], p1[1], p1[2], tx[0], tx[1], tx[2]) -
                    dist3(p1[0], p1[1], p1[2], os[0], os[1], os[2]);
        double dR = dist3(rx[0], rx[1], rx[2], pk[0], pk[1], pk[2]) -
                    dist3(A.oR[0], A.oR[1], A.oR[2], pk[0], pk[1], pk[2]);
        double D = dist3(x1, y1, z1, os[0], os[1], os[2]) + inner +
                   dist3(A.oR[0], A.oR[1], A.oR[2], xk, yk, zk);
        d_base = D + (dT + dR);
        d_step = D;
    }
}

__device__ __forceinline__ double frac(double x) { return x - floor(x); }

// x modulo one cycle as 32-bit fixed-point turns
__device__ __forceinline__ unsigned turns_u32(double x)
{
    return (unsigned)(unsigned long long)llrint(frac(x) * 4294967296.0);
}

// fixed-point turns -> FP32 turns in [-1/2, 1/2)
__device__ __forceinline__ float turns_f32(unsigned u)
{
    return (float)(int)u * 2.3283064365386963e-10f;
}

// One workgroup tile of the moving paths: rows rb * RPB .. of group g (a Tx in
// the per-element mode, everything in the shared mode), every sample of those
// rows, row = (m - m0) RC + channel of the group; chirp 0 of the cube, the sum
// over the paths at rest, is added.  Chirp 0 itself is a launch of its own
// (m0 = 0, one row per channel) after every other chirp has read it.
template <int KR>
__device__ void synth_block(const SynthArgs &A, int g, int rb, int rows_per_group, int RC, int m0,
                            SynPath *sp, uint2 *tab)
{
    const int TPR = A.K / KR;
    const int RPB = SYN_T / TPR;
    const int lrow = threadIdx.x / TPR;
    const int row = rb * RPB + lrow;
    const int k0 = (threadIdx.x % TPR) * KR;
    const bool valid = lrow < RPB && row < rows_per_group;
    const double f0c = A.f0 * A.inv_c;
    const double bkc = A.bw / (double)A.K * A.inv_c;
    float are[KR], aim[KR];
#pragma unroll
    for (int k = 0; k < KR; k++) { are[k] = 0.0f; aim[k] = 0.0f; }
    const int64_t p0 = A.mranges[g];
    const int64_t p1 = A.mov_limit > 0 ? min(A.mranges[g + 1], p0 + A.mov_limit) : A.mranges[g + 1];
    const int chunk = min(SYN_CHUNK, SYN_TAB / RPB);
    for (int64_t base = p0; base < p1; base += chunk) {
        const int cnt = (int)min((int64_t)chunk, p1 - base);
        __syncthreads();
        {
            const float4 *srcv = reinterpret_cast<const float4 *>(A.paths + base);
            float4 *dstv = reinterpret_cast<float4 *>(sp);
            const int nv = cnt * (int)(sizeof(SynPath) / sizeof(float4));
            for (int i = threadIdx.x; i < nv; i += SYN_T) dstv[i] = srcv[i];
        }
        __syncthreads();
        // phase table, entry q * RPB + l: (beta, gamma) of path q in row l
        for (int e = threadIdx.x; e < cnt * RPB; e += SYN_T) {
            const int q = e / RPB, l = e - q * RPB;
            const int rw = rb * RPB + l;
            uint2 v = make_uint2(0u, 0u);
            if (rw < rows_per_group) {
                const int m = m0 + rw / RC, cc = rw - (rw / RC) * RC;
                const int c = A.shared ? cc : g * A.nrx + cc;
                const int t = c / A.nrx, r = c - (c / A.nrx) * A.nrx;
                const double tx[3] = {A.tx[3 * t], A.tx[3 * t + 1], A.tx[3 * t + 2]};
                const double rx[3] = {A.rx[3 * r], A.rx[3 * r + 1], A.rx[3 * r + 2]};
                double db, ds;
                path_lengths(A, sp[q], (double)m * A.t_rep, tx, rx, db, ds);
                v = make_uint2(turns_u32(db * f0c), turns_u32(ds * bkc));
            }
            tab[e] = v;
        }
        __syncthreads();
        if (!valid) continue;
        for (int q = 0; q < cnt; q++) {
            const uint2 ph = tab[q * RPB + lrow];
            const float a = (float)sp[q].amp;
            // exp(-j 2 pi phi) = cos - j sin, phi in turns
            const float u0 = turns_f32(ph.x + (unsigned)k0 * ph.y);
            const float u1 = turns_f32(ph.y);
            float pr = a * __builtin_amdgcn_cosf(u0), pi = -a * __builtin_amdgcn_sinf(u0);
            const float rr = __builtin_amdgcn_cosf(u1), ri = -__builtin_amdgcn_sinf(u1);
#pragma unroll
            for (int k = 0; k < KR; k++) {
                are[k] += pr;
                aim[k] += pi;
                float nr = pr * rr - pi * ri;
                float ni = pr * ri + pi * rr;
                pr = nr;
                pi = ni;
            }
        }
    }
    if (!valid) return;
    const int m = m0 + row / RC, cc = row - (row / RC) * RC;
    const int c = A.shared ? cc : g * A.nrx + cc;
    const float2 *rest = A.cube + (int64_t)c * A.M * A.K + k0;
    float2 *out = A.cube + ((int64_t)c * A.M + m) * A.K + k0;
#pragma unroll
    for (int k = 0; k < KR; k++) {
        const float2 b = rest[k];
        out[k] = make_float2(b.x + are[k], b.y + aim[k]);
    }
}

// Chirp 0 of channel c: the sum over the paths at rest of its group, a part of
// its samples by one workgroup (rest_shape).  TPR lanes (a power of two) cover
// the part's samples, KR each; the other lanes take the same samples of every (REST_T / TPR)-th path, so that a few
// channels of many paths still fill a compute unit's lanes (the tiny scene's
// 4 channels of 2 400 paths and 16 chirps: 20 us here and 2 x 9 us for the
// moving part, against 1.47 ms for the sum of all paths chirp by chirp), and
// the lanes' sums are added in a fixed order: across the wavefront, then over
// the wavefronts through LDS.
struct RestLds {
    uint2 tab[REST_T];        // (beta, gamma) of the chunk's paths
    float amp[REST_T];
    float2 red[REST_T * 8];   // partial sums, eight samples a lane at a time
};
template <int KR>
__device__ void rest_block(const SynthArgs &A, int c, int part, int TPR, RestLds &L)
{
    const int tid = threadIdx.x;
    const int t = c / A.nrx, r = c - t * A.nrx;
    const int g = A.shared ? 0 : t;
    const int pos = tid & (TPR - 1), sub = tid / TPR, G = REST_T / TPR;
    const int kp = part * TPR * KR;       // the part's first sample
    const unsigned k0 = (unsigned)(kp + pos * KR);
    const double f0c = A.f0 * A.inv_c;
    const double bkc = A.bw / (double)A.K * A.inv_c;
    const double tx[3] = {A.tx[3 * t], A.tx[3 * t + 1], A.tx[3 * t + 2]};
    const double rx[3] = {A.rx[3 * r], A.rx[3 * r + 1], A.rx[3 * r + 2]};
    const int64_t p0 = A.ranges[g];
    const int64_t p1 = A.rest_limit > 0 ? min(A.ranges[g + 1], p0 + A.rest_limit) : A.ranges[g + 1];
    float are[KR], aim[KR];
#pragma unroll
    for (int k = 0; k < KR; k++) { are[k] = 0.0f; aim[k] = 0.0f; }
    for (int64_t base = p0; base < p1; base += REST_T) {
        const int cnt = (int)min((int64_t)REST_T, p1 - base);
        __syncthreads();
        if (tid < cnt) {
            const SynPath &P = A.paths[base + tid];
            double db, ds;
            path_lengths(A, P, 0.0, tx, rx, db, ds);
            L.tab[tid] = make_uint2(turns_u32(db * f0c), turns_u32(ds * bkc));
            L.amp[tid] = (float)P.amp;
        }
        __syncthreads();
        for (int q = sub; q < cnt; q += G) {
            const uint2 ph = L.tab[q];
            const float a = L.amp[q];
            const float u0 = turns_f32(ph.x + k0 * ph.y);
            const float u1 = turns_f32(ph.y);
            float pr = a * __builtin_amdgcn_cosf(u0), pi = -a * __builtin_amdgcn_sinf(u0);
            const float rr = __builtin_amdgcn_cosf(u1), ri = -__builtin_amdgcn_sinf(u1);
#pragma unroll
            for (int k = 0; k < KR; k++) {
                are[k] += pr;
                aim[k] += pi;
                const float nr = pr * rr - pi * ri;
                const float ni = pr * ri + pi * rr;
                pr = nr;
                pi = ni;
            }
        }
    }
    for (int off = TPR; off < 64; off <<= 1)
#pragma unroll
        for (int k = 0; k < KR; k++) {
            are[k] += __shfl_xor(are[k], off);
            aim[k] += __shfl_xor(aim[k], off);
        }
    // wavefront w now holds samples of positions (w % wps) 64 + lane
    const int wps = TPR > 64 ? TPR / 64 : 1, np = REST_T / 64 / wps;
    const int lane = tid & 63, w = tid >> 6;
    float2 *out = A.cube + (int64_t)c * A.M * A.K;
    for (int h = 0; h < KR; h += 8) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KR; k++)
            if (lane < TPR && k >= h && k < h + 8) L.red[(w * 64 + lane) * 8 + k - h] = make_float2(are[k], aim[k]);
        __syncthreads();
        for (int o = tid; o < TPR * 8; o += REST_T) {
            const int ps = o >> 3, kk = h + (o & 7), k = kp + ps * KR + kk;
            if (kk >= KR || k >= A.K) continue;
            float2 v = make_float2(0.0f, 0.0f);
            for (int j = 0; j < np; j++) {
                const float2 x = L.red[((j * wps + (ps >> 6)) * 64 + (ps & 63)) * 8 + (o & 7)];
                v.x += x.x;
                v.y += x.y;
            }
            out[k] = v;
        }
    }
}

// item: the parts of channel 0, of channel 1, ...
__device__ __forceinline__ void rest_tile(const SynthArgs &A, int item, RestLds &L)
{
    const RestShape s = rest_shape(A.K, A.ntx * A.nrx);
    const int c = item / s.parts, part = item - c * s.parts;
    switch (s.kr) {
    case 1: rest_block<1>(A, c, part, s.lanes, L); break;
    case 2: rest_block<2>(A, c, part, s.lanes, L); break;
    case 4: rest_block<4>(A, c, part, s.lanes, L); break;
    case 8: rest_block<8>(A, c, part, s.lanes, L); break;
    case 12: rest_block<12>(A, c, part, s.lanes, L); break;
    default: rest_block<16>(A, c, part, s.lanes, L); break;
    }
}

__global__ __launch_bounds__(REST_T) void k_synth_rest(SynthArgs A, int item0)
{
    __shared__ RestLds L;
    rest_tile(A, item0 + blockIdx.x, L);
}

template <int KR>
__global__ __launch_bounds__(SYN_T) void k_synth_direct(SynthArgs A, int rows_per_group, int RC,
                                                        unsigned blocks_per_group, int m0, unsigned block0)
{
    __shared__ SynPath sp[SYN_CHUNK];
    __shared__ uint2 tab[SYN_TAB];
    const unsigned b = block0 + blockIdx.x, g = b / blocks_per_group;
    synth_block<KR>(A, (int)g, (int)(b - g * blocks_per_group), rows_per_group, RC, m0, sp, tab);
}

// the next item of a persistent kernel: the same in every lane, kept in
// scalar registers with the scene it belongs to
__device__ __forceinline__ bool next_item(long long *slot, unsigned long long *work,
                                          const int64_t *item_start, int S, int &scene, int &local)
{
    __syncthreads();
    if (threadIdx.x == 0) *slot = (long long)atomicAdd(work, 1ull);
    __syncthreads();
    const long long iv = *slot;
    const int64_t it = (int64_t)(((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane(
                                      (int)(iv >> 32)) << 32) |
                                 (unsigned)__builtin_amdgcn_readfirstlane((int)iv));
    if (it >= item_start[S]) return false;
    int lo = 0, hi = S - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (item_start[mid] <= it) lo = mid; else hi = mid - 1;
    }
    scene = __builtin_amdgcn_readfirstlane(lo);
    local = (int)(it - item_start[scene]);
    return true;
}

// Batched, persistent: workgroups pull (scene, channel) items of the paths at
// rest, then (scene, tile) items of the moving ones, from a device counter;
// each scene carries its own tile shape (samples per lane KR, chosen by the
// autotuner) and its path ranges come from the batched scan.
__global__ __launch_bounds__(REST_T) void k_batch_rest(const SynthArgs *scenes,
                                                       const int64_t *item_start, int S,
                                                       unsigned long long *work)
{
    __shared__ RestLds L;
    __shared__ long long s_item;
    int scene, local;
    while (next_item(&s_item, work, item_start, S, scene, local)) {
        const SynthArgs A = scenes[scene];
        rest_tile(A, local, L);
    }
}

// first: chirp 0 alone (its rest sum is then replaced by the whole), else
// every other chirp
__global__ __launch_bounds__(SYN_T) void k_batch_synth(const SynthArgs *scenes,
                                                       const BatchSynthInfo *info,
                                                       const int64_t *item_start, int S, int first,
                                                       unsigned long long *work)
{
    __shared__ SynPath sp[SYN_CHUNK];
    __shared__ uint2 tab[SYN_TAB];
    __shared__ long long s_item;
    int scene, local;
    while (next_item(&s_item, work, item_start, S, scene, local)) {
        const SynthArgs A = scenes[scene];
        const BatchSynthInfo I = info[scene];
        const int bpg = first ? I.bpg0 : I.bpg;
        const int g = local / bpg;
        const int rb = local - g * bpg;
        const int rows = first ? I.rc : I.rows_per_group, m0 = first ? 0 : 1;
        switch (I.kr) {
#if RR_BATCH_MAX_KR >= 32
        case 32: synth_block<32>(A, g, rb, rows, I.rc, m0, sp, tab); break;
#endif
        case 16: synth_block<16>(A, g, rb, rows, I.rc, m0, sp, tab); break;
        case 8: synth_block<8>(A, g, rb, rows, I.rc, m0, sp, tab); break;
        case 4: synth_block<4>(A, g, rb, rows, I.rc, m0, sp, tab); break;
        case 2: synth_block<2>(A, g, rb, rows, I.rc, m0, sp, tab); break;
        default: synth_block<1>(A, g, rb, rows, I.rc, m0, sp, tab); break;
        }
    }
}

// one block per requested entry; FP64 phase, FP64 sin/cos, FP64 accumulation
__global__ __launch_bounds__(256) void k_synth_sampled(SynthArgs A, const int64_t *idx)
{
    __shared__ double sre[256], sim[256];
    const int64_t f = idx[blockIdx.x];
    const int64_t MK = (int64_t)A.M * A.K;
    if (f < 0 || f >= (int64_t)(A.ntx * A.nrx) * MK) {
        if (threadIdx.x == 0) A.cube[blockIdx.x] = make_float2(__builtin_nanf(""), __builtin_nanf(""));
        return;
    }
    const int c = (int)(f / MK);
    const int m = (int)((f / A.K) % A.M);
    const int k = (int)(f % A.K);
    const int t = c / A.nrx, r = c % A.nrx;
    const double tx[3] = {A.tx[3 * t], A.tx[3 * t + 1], A.tx[3 * t + 2]};
    const double rx[3] = {A.rx[3 * r], A.rx[3 * r + 1], A.rx[3 * r + 2]};
    const double tau = (double)m * A.t_rep;
    const double fk = A.f0 + A.bw * (double)k / (double)A.K;
    const int g = A.shared ? 0 : t;
    const int64_t p0 = A.ranges[g], n0 = A.ranges[g + 1] - p0;
    const int64_t p1 = A.mranges[g], n = n0 + A.mranges[g + 1] - p1;
    double re = 0.0, im = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += 256) {
        const int64_t p = i < n0 ? p0 + i : p1 + (i - n0);
        const SynPath &P = A.paths[p];
        double db, ds;
        path_lengths(A, P, tau, tx, rx, db, ds);
        double phase = (A.f0 * db + (fk - A.f0) * ds) * A.inv_c;
        double fr = frac(phase);
        double s, cs;
        sincospi(2.0 * fr, &s, &cs);
        re += P.amp * cs;
        im -= P.amp * s;
    }
    sre[threadIdx.x] = re;
    sim[threadIdx.x] = im;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) {
            sre[threadIdx.x] += sre[threadIdx.x + off];
            sim[threadIdx.x] += sim[threadIdx.x + off];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) A.cube[blockIdx.x] = make_float2((float)sre[0], (float)sim[0]);
}

// velocity of path i's hit q (NULL: none)
__device__ __forceinline__ const double *hit_velocity(const PathSoA &P, int q, int64_t i,
                                                      const BatchVel &bv)
{
    const int vid = P.vid[q * P.cap + i];
    if (vid >= 0 && vid < bv.nobj) return bv.obj_vel + 3 * vid;
    if (vid >= bv.nobj && vid < bv.nobj + bv.npts) return bv.pt_vel + 3 * (vid - bv.nobj);
    return nullptr;
}

__device__ __forceinline__ bool at_rest(const PathSoA &P, int64_t i, const BatchVel &bv)
{
    if (bv.M <= 1) return true;
    const int K = P.K[i];
    bool rest = true;
#pragma unroll
    for (int q = 0; q < RR_KMAX; q++)
        if (q < K) {
            const double *v = hit_velocity(P, q, i, bv);
            if (v && (v[0] != 0.0 || v[1] != 0.0 || v[2] != 0.0)) rest = false;
        }
    return rest;
}

__device__ __forceinline__ SynPath syn_record(const PathSoA &P, int64_t i, const BatchVel &bv)
{
    SynPath s;
#pragma unroll
    for (int q = 0; q < RR_KMAX; q++) {
        const double *v = hit_velocity(P, q, i, bv);
#pragma unroll
        for (int a = 0; a < 3; a++) {
            s.P[q][a] = P.p[(3 * q + a) * P.cap + i];
            s.V[q][a] = v ? v[a] : 0.0;
        }
    }
    s.amp = P.amp[i];
    s.K = P.K[i];
    s.src = P.src[i];
    return s;
}

// The records in two parts, each in path order: a count of the paths at rest
// per block of PREP_T, then every block adds the counts before it (one pass
// over a list that is 1/1024 of the paths) and places its own records.
#define PREP_T 1024
__global__ __launch_bounds__(PREP_T) void k_rest_count(PathSoA P, int64_t n, BatchVel bv,
                                                       uint32_t *bsums, int32_t *info)
{
    const int64_t i = (int64_t)blockIdx.x * PREP_T + threadIdx.x;
    const int c = __syncthreads_count(i < n && at_rest(P, i, bv));
    if (threadIdx.x == 0) {
        bsums[blockIdx.x] = (uint32_t)c;
        info[2 + blockIdx.x] = c;
        if (blockIdx.x == 0) info[0] = P.src[0];
        if (blockIdx.x == gridDim.x - 1) info[1] = P.src[n - 1];
    }
}

// paths at rest before this thread's path, and of all n (nb blocks)
__device__ __forceinline__ void rest_rank(bool rest, const uint32_t *bsums, int64_t nb,
                                          uint32_t &before, uint32_t &total)
{
    __shared__ uint32_t sh_w[PREP_T / 64], sh_b[PREP_T / 64], sh_t[PREP_T / 64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const unsigned long long m = __ballot(rest);
    uint32_t b = 0, t = 0;
    for (int64_t j = threadIdx.x; j < nb; j += PREP_T) {
        const uint32_t x = bsums[j];
        t += x;
        if (j < (int64_t)blockIdx.x) b += x;
    }
    for (int off = 32; off > 0; off >>= 1) {
        b += __shfl_xor(b, off);
        t += __shfl_xor(t, off);
    }
    if (lane == 0) {
        sh_w[w] = (uint32_t)__popcll(m);
        sh_b[w] = b;
        sh_t[w] = t;
    }
    __syncthreads();
    before = (uint32_t)__popcll(m & ((1ull << lane) - 1));
    total = 0;
    for (int j = 0; j < PREP_T / 64; j++) {
        before += sh_b[j] + (j < w ? sh_w[j] : 0u);
        total += sh_t[j];
    }
}

// Record i into its place.  The whole record is loaded before the ranks are
// known, and whether it rests is read from it: loaded after them, behind two
// more rounds of loads, the hand's 4.96e5 records took 59 instead of 48 us.
__device__ __forceinline__ void place_record(const PathSoA &P, int64_t i, int64_t n, const BatchVel &bv,
                                             const uint32_t *bsums, int64_t nb, uint32_t *pre,
                                             SynPath *out)
{
    const SynPath s = syn_record(P, min(i, n - 1), bv);
    bool rest = i < n;
    if (bv.M > 1) {
#pragma unroll
        for (int q = 0; q < RR_KMAX; q++)
            if (q < s.K && (s.V[q][0] != 0.0 || s.V[q][1] != 0.0 || s.V[q][2] != 0.0)) rest = false;
    }
    uint32_t before, total;
    rest_rank(rest, bsums, nb, before, total);
    if (i >= n) return;
    pre[i] = before;
    if (i == n - 1) pre[n] = total;
    out[rest ? (int64_t)before : (int64_t)total + (i - (int64_t)before)] = s;
}

__global__ __launch_bounds__(PREP_T) void k_syn_prep(PathSoA P, int64_t n, BatchVel bv,
                                                     const uint32_t *bsums, uint32_t *pre,
                                                     SynPath *out)
{
    place_record(P, (int64_t)blockIdx.x * PREP_T + threadIdx.x, n, bv, bsums, gridDim.x, pre, out);
}

// ranges of group g's paths in the two parts (src sorted; first path whose
// source is >= g0 + g, g = 0 .. n_groups): per-Tx groups with g0 = 0, the
// single group of a shared launch (every src = -1) with g0 = -1
__global__ void k_rest_ranges(const int32_t *src, int64_t n, int n_groups, int g0,
                              const uint32_t *pre, int64_t *rest, int64_t *mov)
{
    int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g > n_groups) return;
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        int64_t mid = (lo + hi) / 2;
        if (src[mid] < g0 + g) lo = mid + 1; else hi = mid;
    }
    const int64_t r = n > 0 ? pre[lo] : 0, all = n > 0 ? pre[n] : 0;
    rest[g] = r;
    mov[g] = all + lo - r;
}

// the velocity tables of the scene whose virtual rays hold ray v (the paths
// of the batched pool are in virtual ray order)
__device__ __forceinline__ const BatchVel &batch_scene(int64_t v, const int64_t *vr_start, int S,
                                                       const BatchVel *vel)
{
    int lo = 0, hi = S - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (vr_start[mid] <= v) lo = mid; else hi = mid - 1;
    }
    return vel[lo];
}

// Paths of the batched pool that the synthesis stages read: all of them, or
// none once rays returned more than the pool holds.  The scatter then leaves
// places of the pool unwritten (whatever path a dropped record belonged to),
// so every range is empty and the cubes are zero until the host, which sees
// the same counter, has grown the pool and run the launch again.
__device__ __forceinline__ int64_t pool_paths(const unsigned long long *total, int64_t cap)
{
    return (int64_t)*total <= cap ? (int64_t)*total : 0;
}

__global__ __launch_bounds__(PREP_T) void k_batch_rest_count(PathSoA P,
                                                             const unsigned long long *total,
                                                             int64_t cap, const int64_t *vr_start,
                                                             int S, const BatchVel *vel,
                                                             uint32_t *bsums)
{
    const int64_t i = (int64_t)blockIdx.x * PREP_T + threadIdx.x;
    const int64_t n = pool_paths(total, cap);
    bool rest = false;
    if (i < n) rest = at_rest(P, i, batch_scene(P.ray[i], vr_start, S, vel));
    const int c = __syncthreads_count(rest);
    if (threadIdx.x == 0) bsums[blockIdx.x] = (uint32_t)c;
}

// synthesis records of the batched path pool: the scene of a path follows
// from its virtual ray id
__global__ __launch_bounds__(PREP_T) void k_batch_prep(PathSoA P, const unsigned long long *total,
                                                       int64_t cap, const int64_t *vr_start, int S,
                                                       const BatchVel *vel, const uint32_t *bsums,
                                                       uint32_t *pre, SynPath *out)
{
    const int64_t i = (int64_t)blockIdx.x * PREP_T + threadIdx.x;
    const int64_t n = pool_paths(total, cap);
    if ((int64_t)blockIdx.x * PREP_T >= n) {
        if (n == 0 && i == 0) pre[0] = 0;
        return;
    }
    const BatchVel &bv = batch_scene(P.ray[min(i, n - 1)], vr_start, S, vel);
    place_record(P, i, n, bv, bsums, (n + PREP_T - 1) / PREP_T, pre, out);
}

// per-scene path ranges from the batched exclusive scan: paths of virtual
// rays [vr0 + t n_vps, ...) start at the prefix of vr0 + t n_vps; then those of
// the two parts of the records.  host (pinned): records appended, paths, and
// the groups' starts in the path list.
__global__ void k_batch_ranges(const uint8_t *counts, const uint32_t *bsums, int64_t V,
                               const unsigned long long *total, const unsigned long long *counter,
                               int64_t cap, const BatchRangeInfo *ri, int S, const uint32_t *pre,
                               int64_t *rest, int64_t *mov, int64_t *host)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s == 0) {
        host[0] = (int64_t)*counter;
        host[1] = (int64_t)*total;
    }
    if (s >= S) return;
    const BatchRangeInfo &R = ri[s];
    const int64_t tot = pool_paths(total, cap);
    auto put = [&](int g, int64_t v) {
        const int64_t o = min(v < V ? (int64_t)count_prefix(counts, bsums, v) : tot, tot);
        const int64_t r = pre[o];
        rest[R.base + g] = r;
        mov[R.base + g] = (int64_t)pre[tot] + o - r;
        host[2 + R.base + g] = o;
    };
    if (R.shared) {
        put(0, R.vr0);
        put(1, R.vr0 + R.n_vps);
    } else {
        for (int g = 0; g <= R.n_groups; g++) put(g, R.vr0 + (int64_t)g * R.n_vps);
    }
}

__global__ void k_fill_u64(unsigned long long *p, int64_t n, unsigned long long v)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

}  // namespace

hipError_t launch_batch_synth(int stage, const SynthArgs *scenes, const BatchSynthInfo *info,
                              const int64_t *item_start, int S, int64_t n_items,
                              unsigned long long *work, hipStream_t s)
{
    int dev = 0, cus = 256;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const int64_t grid = std::min<int64_t>(n_items, (int64_t)cus * 8);
    if (grid <= 0) return hipSuccess;
    if (stage == 0)
        hipLaunchKernelGGL(k_batch_rest, dim3((unsigned)grid), dim3(REST_T), 0, s, scenes,
                           item_start, S, work);
    else
        hipLaunchKernelGGL(k_batch_synth, dim3((unsigned)grid), dim3(SYN_T), 0, s, scenes, info,
                           item_start, S, stage == 2 ? 1 : 0, work);
    return hipGetLastError();
}

int64_t rest_blocks(int64_t n) { return (n + PREP_T - 1) / PREP_T; }

hipError_t launch_batch_prep(const PathSoA &paths, const unsigned long long *total, int64_t cap,
                             const int64_t *vr_start, int S, const BatchVel *vel, uint32_t *bsums,
                             uint32_t *pre, SynPath *out, hipStream_t s)
{
    if (cap <= 0) return hipSuccess;
    const dim3 g((unsigned)rest_blocks(cap));
    hipLaunchKernelGGL(k_batch_rest_count, g, dim3(PREP_T), 0, s, paths, total, cap, vr_start, S,
                       vel, bsums);
    hipLaunchKernelGGL(k_batch_prep, g, dim3(PREP_T), 0, s, paths, total, cap, vr_start, S, vel,
                       bsums, pre, out);
    return hipGetLastError();
}

hipError_t launch_batch_ranges(const uint8_t *counts, const uint32_t *bsums, int64_t V,
                               const unsigned long long *total, const unsigned long long *counter,
                               int64_t cap, const BatchRangeInfo *ri, int S, const uint32_t *pre,
                               int64_t *rest, int64_t *mov, int64_t *host, hipStream_t s)
{
    hipLaunchKernelGGL(k_batch_ranges, dim3((unsigned)((S + 63) / 64)), dim3(64), 0, s, counts, bsums, V,
                       total, counter, cap, ri, S, pre, rest, mov, host);
    return hipGetLastError();
}

hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

static BatchVel one_scene(const double *obj_vel, int nobj, const double *pt_vel, int npts, int split)
{
    BatchVel bv;
    bv.obj_vel = obj_vel;
    bv.pt_vel = pt_vel;
    bv.nobj = nobj;
    bv.npts = npts;
    bv.M = split ? 2 : 1;
    return bv;
}

hipError_t launch_rest_count(const PathSoA &paths, int64_t n, const double *obj_vel, int nobj,
                             const double *pt_vel, int npts, int split, uint32_t *bsums,
                             int32_t *info, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_rest_count, dim3((unsigned)rest_blocks(n)), dim3(PREP_T), 0, s, paths, n,
                       one_scene(obj_vel, nobj, pt_vel, npts, split), bsums, info);
    return hipGetLastError();
}

hipError_t launch_syn_prep(const PathSoA &paths, int64_t n, const double *obj_vel, int nobj,
                           const double *pt_vel, int npts, int split, const uint32_t *bsums,
                           uint32_t *pre, SynPath *out, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_syn_prep, dim3((unsigned)rest_blocks(n)), dim3(PREP_T), 0, s, paths, n,
                       one_scene(obj_vel, nobj, pt_vel, npts, split), bsums, pre, out);
    return hipGetLastError();
}

hipError_t launch_rest_ranges(const int32_t *src, int64_t n, int n_groups, int g0,
                              const uint32_t *pre, int64_t *rest, int64_t *mov, hipStream_t s)
{
    hipLaunchKernelGGL(k_rest_ranges, dim3((unsigned)((n_groups + 1 + 255) / 256)), dim3(256), 0,
                       s, src, n, n_groups, g0, pre, rest, mov);
    return hipGetLastError();
}

// rows of one launch: RC channels of every group for chirps m0 ..
template <int KR>
static hipError_t launch_kr(const SynthArgs &a, int n_groups, int rows_per_group, int RC, int m0,
                            hipStream_t s)
{
    const int TPR = a.K / KR;
    const int RPB = SYN_T / TPR;
    const int bpg = (rows_per_group + RPB - 1) / RPB;
    // a launch holds fewer than 2^32 threads
    const int64_t blocks = (int64_t)bpg * n_groups, step = (int64_t)1 << 23;
    if (blocks >= (int64_t)1 << 32) return hipErrorInvalidValue;
    for (int64_t b = 0; b < blocks; b += step)
        hipLaunchKernelGGL(k_synth_direct<KR>, dim3((unsigned)std::min(step, blocks - b)), dim3(SYN_T), 0, s, a,
                           rows_per_group, RC, (unsigned)bpg, m0, (unsigned)b);
    return hipGetLastError();
}

hipError_t launch_synth_direct(const SynthArgs &a, int n_groups, int rows_per_group,
                               hipStream_t s)
{
    const int RC = a.shared ? a.ntx * a.nrx : a.nrx;
    int kr = 32;
    while (kr > 1 && a.K % kr != 0) kr >>= 1;
    if (a.K / kr > SYN_T) return hipErrorInvalidValue;
    // a launch holds fewer than 2^32 threads: 2^22 channels at a time
    const int64_t items = rest_items(a.K, a.ntx * a.nrx), step = (int64_t)1 << 22;
    for (int64_t i = 0; i < items; i += step)
        hipLaunchKernelGGL(k_synth_rest, dim3((unsigned)std::min(step, items - i)), dim3(REST_T), 0, s, a, (int)i);
    if (a.M <= 1) return hipGetLastError();
    for (int m0 = 1; m0 >= 0; m0--) {
        const int rows = m0 ? rows_per_group - RC : RC;
        hipError_t e;
        switch (kr) {
        case 32: e = launch_kr<32>(a, n_groups, rows, RC, m0, s); break;
        case 16: e = launch_kr<16>(a, n_groups, rows, RC, m0, s); break;
        case 8: e = launch_kr<8>(a, n_groups, rows, RC, m0, s); break;
        case 4: e = launch_kr<4>(a, n_groups, rows, RC, m0, s); break;
        case 2: e = launch_kr<2>(a, n_groups, rows, RC, m0, s); break;
        default: e = launch_kr<1>(a, n_groups, rows, RC, m0, s); break;
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_synth_sampled(const SynthArgs &a, const int64_t *idx, int64_t n_idx,
                                hipStream_t s)
{
    if (n_idx <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_synth_sampled, dim3((unsigned)n_idx), dim3(256), 0, s, a, idx);
    return hipGetLastError();
}
