// Internal declarations shared by the host code and the kernel launchers of
// libradray.  Not part of the public ABI (see include/radray.h).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/radray.h"

#define RR_TRACE_BLOCK 128
#define RR_STACK 32          // BVH depth bound (the builder guarantees depth <= 31)
#define RR_LEAF_MAX 8        // triangles per leaf (3-bit count in the child reference)

// ---------------------------------------------------------------------------
// device-side structure-of-arrays path list (planes of `cap` elements)
// ---------------------------------------------------------------------------
struct PathSoA {
    int32_t *src = nullptr;
    int32_t *K = nullptr;
    int64_t *ray = nullptr;
    int32_t *loc = nullptr;   // index of the path among its ray's paths (temp list only)
    int32_t *tri = nullptr;   // [RR_KMAX][cap]
    int32_t *vid = nullptr;   // [RR_KMAX][cap]
    double *p = nullptr;      // [RR_KMAX*3][cap]
    double *L = nullptr;
    double *amp = nullptr;
    int64_t cap = 0;
};

// ---------------------------------------------------------------------------
// BVH on the device.  Node (64 B): child boxes and child references
//   n[0] = (lo0.x, lo0.y, lo0.z, hi0.x)   n[1] = (hi0.y, hi0.z, lo1.x, lo1.y)
//   n[2] = (lo1.z, hi1.x, hi1.y, hi1.z)   n[3] = (ref0, ref1, 0, 0) as int bits
// Reference r >= 0: internal node r.  r < 0: leaf, x = ~r, first triangle
// x >> 3 of the leaf-ordered triangle array, count (x & 7) + 1.
// Leaf triangle (48 B): (v0.xyz, v1.x) (v1.yz, v2.xy) (v2.z, id, obj, 0)
// with id/obj stored as int bits.
// ---------------------------------------------------------------------------
struct HostBvh {
    std::vector<float> nodes;    // 16 floats per node
    std::vector<float> tris;     // 12 floats per triangle
    int depth = 0;
};

// Field of view of a per-triangle launch as seen from its sources (the Tx
// phase centre, or every Tx element): cosines and sines of the azimuth
// bounds, sines of the elevation bounds.
struct RrFov {
    const double *src;
    int32_t n_src;
    double c0, s0, c1, s1, slo, shi;
};
int rr_build_pieces(const float *verts, const int32_t *tris, int64_t n_tris, const double *o,
                    double omega_max, int depth_max, const RrFov *fov, int64_t limit,
                    std::vector<double> &pverts, std::vector<int32_t> &parent);
int rr_build_bvh(const float *verts, int64_t nv, const int32_t *tris, const int32_t *tri_obj,
                 const float *obj_alpha, int64_t nt, HostBvh &out, std::string &err);

// ---------------------------------------------------------------------------
// prefix of the rays' path counts: sums before every tile, and the tile's own
// counts up to the ray
// ---------------------------------------------------------------------------
#define RR_SCAN_TILE 256

#ifdef __HIP__
__device__ __forceinline__ uint32_t sum_counts(uint4 v)
{
    return __builtin_amdgcn_sad_u8(
        v.x, 0u, __builtin_amdgcn_sad_u8(
                     v.y, 0u, __builtin_amdgcn_sad_u8(v.z, 0u, __builtin_amdgcn_sad_u8(v.w, 0u, 0u))));
}

// paths of the rays before ray v
__device__ __forceinline__ uint32_t count_prefix(const uint8_t *counts, const uint32_t *bsums, int64_t v)
{
    const int64_t b = v / RR_SCAN_TILE;
    const uint4 *c = reinterpret_cast<const uint4 *>(counts + b * RR_SCAN_TILE);
    const int in = (int)(v - b * RR_SCAN_TILE), full = in >> 4, part = in & 15;
    uint32_t s = bsums[b];
#pragma unroll 8
    for (int k = 0; k < full; k++) s += sum_counts(c[k]);
    const uint8_t *t = reinterpret_cast<const uint8_t *>(c + full);
    for (int k = 0; k < part; k++) s += t[k];
    return s;
}
#endif

// ---------------------------------------------------------------------------
// trace kernel arguments (by value)
// ---------------------------------------------------------------------------
struct TraceArgs {
    const float4 *nodes;
    const float4 *ltris;
    int has_bvh;
    const double *tx;         // [ntx][3]
    const double *pt_pos;     // [npts][3]
    const double *pt_ap;      // [npts]
    double oT[3], oR[3];
    double r2;
    int shared;
    int nobj, npts;
    int64_t n_src, n_per_src, n_virt_per_src;
    double inv_per_src;       // 1 / n_per_src
    double at, bt, slo, shi, omega;
    int bmax;
    uint64_t seed;
    int sampler;
    const double *cdf;
    int n_az, n_el;
    const double *pieces;     // [n_pieces][9] vertices of the per-triangle launch's pieces
    const int32_t *piece_parent;   // [n_pieces] triangle a piece's rays must hit first
    int tri_g;                // g: g^2 rays per piece and source
    double fov_c0, fov_s0, fov_c1, fov_s1;   // cos, sin of the azimuth bounds
    int64_t vbase;            // first virtual ray of this scene in the (batched) ray space
    const int32_t *order;     // [n_traced] ray of each lane (coherent order) or null
    // outputs
    int32_t *hits;            // [n_src*n_per_src][bmax+1] or null
    uint8_t *counts;          // indexed by vbase + virtual ray; zero before the launch
    PathSoA tmp;
    unsigned long long *counter;   // records appended
    int *err_flag;
    int stack;                // entries of a lane's traversal stack, at most RR_STACK
};

// caller-supplied rays (device arrays)
struct UserRays {
    const double *orig;       // [n][3]
    const double *dir;        // [n][3]
    const double *amp;        // [n]
    const int32_t *src;       // [n]
    int64_t n;
};

// ---------------------------------------------------------------------------
// synthesis path record (AoS, prepared from the path list)
// ---------------------------------------------------------------------------
struct SynPath {
    double P[RR_KMAX][3];     // hit points at t = 0
    double V[RR_KMAX][3];     // their velocities
    double amp;
    int32_t K;
    int32_t src;
};

// The records of a synthesis are split in two, each part in path order: the
// paths at rest (every hit on an object of zero velocity), whose sum is the
// same for every chirp and is formed once, then the moving ones.
struct SynthArgs {
    const SynPath *paths;
    const int64_t *ranges;    // [n_groups + 1] paths at rest of each group
    const int64_t *mranges;   // [n_groups + 1] moving paths of each group
    int64_t n_paths;
    const double *tx, *rx;    // device [n][3]
    int ntx, nrx;
    double oT[3], oR[3];
    int shared;
    int model;
    double f0, bw, t_rep, inv_c;
    int M, K;
    float2 *cube;
// > 0: at most this many paths of each group, at rest and moving (the
    // autotuner's timings of large scenes)
    int64_t rest_limit, mov_limit;
};

// back-projection (imaging): one single-sweep cube onto a voxel grid
#define RR_BP_KMAX 4096          // longest sweep: one channel fills the staging buffer
struct BackProjArgs {
    const float2 *cube;       // channel c's sweep at cube + c * stride
    int64_t stride;
    const double *tx, *rx;    // device [n][3]
    int ntx, nrx, C, K;
    double f0, df, inv_c;
    double x0, y0, z0, step;  // voxel (i, j, k) at (x0 + i step, y0 + j step, z0 + k step)
    int nx, ny, nz;
    int64_t n_vox;
    float2 *image;            // [nx][ny][nz]
};

// largest samples-per-lane tile of the batched synthesis kernel (its
// register use, hence its occupancy, follows the largest tile it contains)
#ifndef RR_BATCH_MAX_KR
#define RR_BATCH_MAX_KR 32
#endif

// The direct engine's sum over the paths at rest: `parts` workgroups of
// `lanes` x `kr` samples a channel (the last may be short).  A lane's run is
// never longer than the moving paths' (the largest power of two that divides
// K, here at most 16): every rotation of a run adds its rounding, and 195
// samples in runs of 13 were 4.3e-7 off the FP64 sum of 64 paths, in runs of
// one 1.3e-7.  The short runs of such counts take many lanes a channel; few
// channels then give their samples to several workgroups, up to one a compute
// unit (56 channels x 51 samples, 2.6e5 paths: 3.18 -> 1.87 ms; 4 x 87 and a
// trace of 2.9e5 rays 272 -> 185 us).  Each part forms the paths' lengths
// again, so it keeps 16 lanes of work beside them: with one lane of 16 samples
// a part, 64 x 4 took as long as undivided, and the rest stage of a batch of
// eight streets, whose channels fill the chip, 137 instead of 68 us.
#define REST_T 512
struct RestShape {
    int kr, lanes, parts;
};
static __host__ __device__ inline RestShape rest_shape(int K, int C)
{
    RestShape s;
    const int run = (K & -K) < 16 ? K & -K : 16;
    s.lanes = 1;
    while (s.lanes * run < K && s.lanes < REST_T) s.lanes <<= 1;
    const int kr = (K + s.lanes - 1) / s.lanes;
    s.kr = kr <= 2 ? kr : kr <= 4 ? 4 : (kr + 3) / 4 * 4;
    auto parts = [&] { return (K + s.lanes * s.kr - 1) / (s.lanes * s.kr); };
    while (s.lanes > 16 && (int64_t)C * parts() < 256) s.lanes >>= 1;
    s.parts = parts();
    return s;
}
inline int64_t rest_items(int K, int C) { return (int64_t)C * rest_shape(K, C).parts; }

// batched launch: per-scene tables read by the persistent kernels
struct BatchSynthInfo {
    int kr;                   // samples per lane (tile shape)
    int rows_per_group;
    int rc;                   // channels per group
    int bpg;                  // workgroups per group for the chirps after the first
    int bpg0;                 // workgroups per group for the first chirp
};
struct BatchVel {
    const double *obj_vel;
    const double *pt_vel;
    int nobj, npts;
    int M;                    // chirps: with one, every path counts as at rest
};
struct BatchRangeInfo {
    int64_t vr0;              // first virtual ray of the scene
    int64_t n_vps;            // virtual rays per source
    int64_t base;             // first entry of the scene in the ranges table
    int n_groups;
    int shared;
};

// launchers (defined in the .hip files)
hipError_t launch_trace(const TraceArgs &a, int64_t n_traced, hipStream_t s);
// Coherent ray order of a uniform or proposal launch: rays sorted by source
// and the 2^bits x 2^bits cell of their first direction, in chunks of 2^shift
// rays of one source, per of them a source.
struct OrderTab {
    int bits, shift;
    unsigned per;
    int64_t chunk0, src0;     // batch: the scene's first chunk and source
    unsigned *cells;          // n_src 4^bits counters, zero before
    unsigned *ray_cells;      // n_traced cells and ranks
    unsigned *first;          // n_src per 4^bits places
    int32_t *order;           // n_traced ray indices
};
OrderTab trace_order_tab(int64_t n_per_src);
hipError_t launch_trace_order(const TraceArgs &a, int64_t n_traced, const OrderTab &O, hipStream_t s);
// every scene's at once: chunks and sources in total, bits of the largest
hipError_t launch_batch_order(const TraceArgs *scenes, const OrderTab *tabs, int S, int64_t chunks,
                              int64_t sources, int bits, hipStream_t s);
hipError_t launch_points(const TraceArgs &a, hipStream_t s);
// k_trace plus exact work counters: stats[0] BVH nodes fetched, stats[1] leaf
// triangle records fetched, stats[2] closest-hit queries (summed, not cleared)
hipError_t launch_trace_count(const TraceArgs &a, int64_t n_traced, unsigned long long *stats,
                              hipStream_t s);
hipError_t launch_trace_user(const TraceArgs &a, const UserRays &u, hipStream_t s);
hipError_t launch_set_alpha(float4 *ltris, int64_t n_tris, const float *tri_alpha,
                            const float *obj_alpha, hipStream_t s);
int freq_k_step();
int freq_k_group();   // samples per exact-GEMM workgroup
// leg tables of the records *rng_lo .. *rng_hi of `paths` (read on the device,
// at most Ppad of them); own_tx: one X row per chirp, each path's own
// transmitter (see freq_own_tx); sep: the separable model's legs, from the
// phase centres oT, oR
struct FreqLegs {
    const SynPath *paths;
    const int64_t *rng_lo, *rng_hi;
    const double *tx, *rx;
    int T, R, M;
    double t_rep, f0c, dfc;
    int sep;
    double oT[3], oR[3];
    // bands: the tables hold *used entries, entry p of record perm[p] (-1: none)
    const int32_t *perm, *used;
};
hipError_t launch_freq_prep(const FreqLegs &L, int64_t Ppad, bool own_tx, uint2 *xt, uint2 *yt,
                            float *amp, int32_t *src, hipStream_t s);
// the X table keeps one row per chirp (each path's own transmitter) for a
// per-element launch on the sample split with transmitter groups, else one
// per (chirp, transmitter); entries (8 bytes each) of both tables
bool freq_own_tx(int tile, bool per_element, bool has_groups);
int64_t freq_table_entries(int T, int R, int M, int64_t Ppad, bool own_tx);
// exact product engine layouts: Tx x Rx tile 16, 32, 48, 64 or 96, or 1 (one
// channel per wavefront, samples split); the layout of least modelled time,
// the modelled time (relative) of one, and the path splits of a launch
int freq_tile(int T, int R, int K, bool per_element);
double freq_tile_cost(int T, int R, int K, int tile, bool per_element);
int freq_splits(int tile, int T, int R, int M, int K);
int freq_chirps(int tile, int T, int R, int M, int K);
int64_t freq_partial(int tile, int T, int R, int M, int K);
// the exact model's AUTO rule: the best product layout is modelled at least
// 1.5x the direct engine's throughput
bool freq_pays(int T, int R, int K, bool per_element);
// The layout of the moving paths of a launch on layout `tile`: up to
// FREQ_MOV_KS of them run as the sample split, whose wavefronts write whole
// runs of samples (the tiles store 8 bytes per channel and sample).
#define FREQ_MOV_KS 1024
int freq_mov_tile(int tile, int T, int R, int K, bool per_element);
// cube[c][m][k] = rest[c][k] (if given) + the sum over the paths of the
// tables, whose count is read on the device (*rng_hi - *rng_lo, at most Ppad)
// and divided evenly over the splits.  groups (may be NULL; per-element
// launch, tile 1): [T + 1] path range of each transmitter, offset by
// groups[0].  The launch does its work only if gate_lo < count <= gate_hi.
struct FreqSum {
    const uint2 *xt, *yt;
    const float *amp;
    const int32_t *src;
    int T, R, M, K;
    int64_t Ppad;
    int per_element, tile;
    const int64_t *rng_lo, *rng_hi, *groups;
    int64_t gate_lo, gate_hi;
    const float2 *rest;
    float2 *partial, *cube;
};
hipError_t launch_freq_gemm(const FreqSum &q, hipStream_t s);
struct BandArgs;
// the products of a band plan (tile layouts), partial sums [slot][channel];
// at most max_items work items
int freq_band_fit(int tile);   // workgroups the chip holds at a time
hipError_t launch_freq_bands(const FreqSum &q, const BandArgs &B, int64_t max_items, hipStream_t s);
// Bands of path lengths (k_band.hip): classes of node counts for K samples,
// by rising reach z (half the phase that the band's edge gathers over the
// chirp); nodes [class][RR_BAND_NMAX] sample indices, coef from coef[class]:
// [node][sample]
#define RR_BAND_NMAX 32
#define RR_BAND_CLASSES 7
struct BandClasses {
    int32_t count;
    int32_t n[RR_BAND_CLASSES];
    float z[RR_BAND_CLASSES];
    int32_t coef[RR_BAND_CLASSES];
};
BandClasses rr_band_classes(int K, std::vector<int32_t> &nodes, std::vector<float> &coef);
int rr_band_nodes(int K);     // nodes of the largest class of K samples (0: none)
#define RR_BANDS 256          // bands (k_band.hip); longer paths go to the last list
// A band costs its sums' expansion, about 1 700 path x four-node products of
// 3 072 channels (0.5 us): fewer paths than this are cheaper at every sample.
#define BAND_THIN 48
// back-projection on the matrix cores: the volume, array and sweep; a plan
// (blocks of voxels per axis, workgroups per block, n nodes of class cls, or
// cls = -1: every sample over the whole volume) with the bytes of its slices
// and of the transposed cube
struct BpGrid {
    double lo[3], hi[3], step;
    int n[3];
    int T, R, K;
    double f0, df, inv_c;
    const double *box;        // bounds of the Tx, then of the Rx elements
};
struct BpPlan {
    int cls, n;
    int nb[3], wgs;
    int64_t frag_bytes, turn_bytes;
};
BpPlan bp_plan(const BpGrid &G, const BandClasses &cls);
hipError_t launch_bp_mfma(const BpGrid &G, const BpPlan &P, const float2 *cube, int64_t stride,
                          const double *tx, const double *rx, const int32_t *nodes, const float *coef,
                          float2 *turned, uint4 *Sf, float2 *image, hipStream_t s);
struct BandSeg {              // at most one chunk of a list's paths
    int32_t p0, np;           // places in the sorted tables (multiples of 32)
    int32_t cls;              // class of nodes, -1: every sample
    int32_t groups;           // work items: four nodes (samples) each
    int32_t item0, slot0;     // first work item, first partial sum ([slot][channel])
};
struct BandOut {              // one list as the expansion reads it
    int32_t cls, n;           // n partial sums per chunk
    int32_t chunks, slot0;
    int32_t row0;             // first of its n rows among the lists of several chunks
    uint32_t gamma;           // centre, turns per sample
};
struct BandPlan {
    int32_t used, n_segs, n_items, n_out;
    int32_t n_rows;           // partial sums to add over chunks
    int32_t next;             // work item counter of the products
    int32_t base[RR_BANDS + 1];
    BandOut out[RR_BANDS + 1];
};
// the paths at rest of a shared launch in bands; at most `target` + B n / 4
// + K / 4 + 1 work items (B bands, n nodes of the largest class; as many
// segments), four partial sums each
struct BandArgs {
    FreqLegs L;               // one chirp
    int64_t Ppad, perm_cap;   // capacity in paths, in table entries
    int K;
    double bins_per_m;        // B / c
    double tx_lo[3], tx_hi[3], rx_lo[3], rx_hi[3];
    BandClasses cls;
    const int32_t *nodes;
    const float *coef;
    int target;
    uint16_t *keys;           // [Ppad]
    uint32_t *hist;           // [blocks][RR_BANDS + 1]
    uint2 *extent;            // [blocks][RR_BANDS + 1]
    int32_t *perm;            // [perm_cap]
    BandPlan *plan;
    BandSeg *segs;
};
int64_t band_blocks(int64_t Ppad);
hipError_t launch_band_plan(const BandArgs &A, hipStream_t s);
hipError_t launch_band_expand(const BandArgs &A, float2 *part, int C, float2 *out, hipStream_t s);
hipError_t launch_refit(float4 *nodes, float *ubox, const int32_t *order,
                        const int64_t *level_start, int n_levels, float4 *ltris, int64_t n_tris,
                        const int32_t *tris, const float *verts, double pad, hipStream_t s);
hipError_t launch_backproject(const BackProjArgs &a, hipStream_t s);
hipError_t launch_max_projection(const float2 *img, int64_t nx, int64_t nyz, float *out,
                                 float *peak, float floor_db, hipStream_t s);
hipError_t launch_check_user(const UserRays &u, int shared, int ntx, int *flag, hipStream_t s);
// What every trace starts from: counts (a multiple of 16 bytes allocated),
// *counter, *err_flag (or null) and nk cell counts zero.
hipError_t launch_trace_clear(uint8_t *counts, int64_t V, unsigned long long *counter, int *err_flag,
                              unsigned *cells, int64_t nk, hipStream_t s);
// bsums[b] = paths of the rays before tile b; *total = their number; host
// (pinned, or null) = {*counter, *err_flag}
hipError_t launch_scan_u8(const uint8_t *counts, int64_t n, uint32_t *bsums, int64_t nb_cap,
                          unsigned long long *total, const unsigned long long *counter,
                          const int *err_flag, unsigned long long *host, hipStream_t s);
int64_t scan_u8_blocks(int64_t n);
hipError_t launch_scatter(const PathSoA &tmp, const unsigned long long *counter, int64_t tmp_cap,
                          const uint8_t *counts, const uint32_t *bsums, const PathSoA &dst,
                          int64_t keep, hipStream_t s);
// the first n paths into dst's planes; a null plane is left out
hipError_t launch_copy_paths(const PathSoA &src, int64_t n, const PathSoA &dst, hipStream_t s);

// Synthesis records in two parts (see SynthArgs): rest_blocks(n) block counts
// and n + 1 prefix entries of scratch.  split = 0 keeps every path in the
// first part.  launch_rest_ranges then gives the ranges of every group in
// both parts from the ranges `all` in the path list (may be the `rest` table
// itself), or from the sorted sources of one scene when all is NULL.
int64_t rest_blocks(int64_t n);
hipError_t launch_rest_count(const PathSoA &paths, int64_t n, const double *obj_vel, int nobj,
                             const double *pt_vel, int npts, int split, uint32_t *bsums,
                             int32_t *info, hipStream_t s);
hipError_t launch_syn_prep(const PathSoA &paths, int64_t n, const double *obj_vel, int nobj,
                           const double *pt_vel, int npts, int split, const uint32_t *bsums,
                           uint32_t *pre, SynPath *out, hipStream_t s);
hipError_t launch_rest_ranges(const int32_t *src, int64_t n, int n_groups, int g0,
                              const uint32_t *pre, int64_t *rest, int64_t *mov, hipStream_t s);
// direct engine: the paths at rest into chirp 0 of every channel, then that
// row plus the moving paths into every other chirp, then the moving paths
// into chirp 0
hipError_t launch_synth_direct(const SynthArgs &a, int n_groups, int rows_per_group,
                               hipStream_t s);
hipError_t launch_synth_sampled(const SynthArgs &a, const int64_t *idx, int64_t n_idx,
                                hipStream_t s);

// split-bf16 complex GEMM engine (k_gemm.hip)
int gemm_row_pad();
int gemm_a_bytes();
int gemm_col_tile();
int gemm_k_step();
hipError_t launch_gemm_prep_tr(const SynthArgs &a, int Ppad, float2 *T, float2 *R, hipStream_t s);
hipError_t launch_gemm_prep_a(const float2 *T, const float2 *R, int nrx, int C, int Cpad, int Ppad,
                              uint4 *Af, hipStream_t s);
hipError_t launch_gemm_prep_b(const SynthArgs &a, int Ppad, uint4 *Bp, hipStream_t s);
hipError_t launch_gemm_main(const uint4 *Af, const uint4 *Bp, int Cpad, int Ppad, int C, int M,
                            int K, const float2 *rest, float2 *cube, hipStream_t s);

// learned proposal (k_trace.hip: probe and histogram; k_mlp.hip: network)
hipError_t launch_probe(const TraceArgs &a, float *code, hipStream_t s);
hipError_t launch_hist(const TraceArgs &a, int64_t n_traced, const int32_t *hits,
                       const int32_t *tri_obj, int n_az, int n_el, float *H, hipStream_t s);
#include <hip/hip_fp16.h>
hipError_t launch_mlp_forward(const float *P, const float *codes, int64_t n, __half *acts, float *z,
                              hipStream_t s);
hipError_t launch_softmax_grad(const float *z, const float *H, int n_scenes, float *dz, float *loss,
                               hipStream_t s);
// lr > 0: a step of Adam after the gradient
struct AdamArgs {
    float *P, *m, *v;
    float lr, b1, b2, c1, c2, eps;
};
AdamArgs adam_args(float *P, float *m, float *v, float lr, int step);
// Backward pass, weight gradients and Adam.  The rows (whole scenes) are
// split over at most 256 workgroups, each writing its partial sums into part;
// two passes then add them in a fixed order (runs of consecutive workgroups,
// then the runs) into grad (every entry written).  part holds
// mlp_part_rows(n) rows of RR_MLP_PARAMS floats.
int64_t mlp_part_rows(int64_t n);
hipError_t launch_mlp_backward(const float *P, const float *dz, int64_t n, const __half *acts,
                               const float *codes, float *part, float *grad, const AdamArgs &adam,
                               hipStream_t s);
hipError_t launch_build_cdf(const float *z, float beta, float power, float kappa, double *cdf,
                            hipStream_t s);
hipError_t launch_batch_trace(const TraceArgs *scenes, const int64_t *chunk_start, int S, int stack,
                              int64_t n_chunks, hipStream_t s);
// stage 0: paths at rest into chirp 0 (items: channels), 1: the other chirps,
// 2: moving paths into chirp 0
hipError_t launch_batch_synth(int stage, const SynthArgs *scenes, const BatchSynthInfo *info,
                              const int64_t *item_start, int S, int64_t n_items,
                              unsigned long long *work, hipStream_t s);
hipError_t launch_batch_prep(const PathSoA &paths, const unsigned long long *total, int64_t cap,
                             const int64_t *vr_start, int S, const BatchVel *vel, uint32_t *bsums,
                             uint32_t *pre, SynPath *out, hipStream_t s);
// rest / mov: ranges of every scene's groups in the two parts of the records;
// host (pinned): records appended, paths, the groups' starts in the path list
hipError_t launch_batch_ranges(const uint8_t *counts, const uint32_t *bsums, int64_t V,
                               const unsigned long long *total, const unsigned long long *counter,
                               int64_t cap, const BatchRangeInfo *ri, int S, const uint32_t *pre,
                               int64_t *rest, int64_t *mov, int64_t *host, hipStream_t s);
hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v, hipStream_t s);
