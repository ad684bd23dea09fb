// Internal definitions shared by the HIP kernels and the host runtime of the
// MPPI library.  Nothing here is part of the public C ABI (include/mppi.h).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace mppi_impl {

constexpr int kBlock = 256;          // threads per workgroup (4 wave64)
constexpr int kMaxEgo = 4;
constexpr int kMaxT = 2048;
constexpr int kMaxWaypoints = 2048;
constexpr int kMaxCircles = 1024;
constexpr int kMaxK = 1 << 24;

// Per-instance state that stays resident on the device between iterations.
struct DevState {
    unsigned long long n_iter;  // Philox counter words 2-3: iteration number
    unsigned int reserved;
    int status;                 // 0 or MPPI_E_NONFINITE of the last iteration
    double s_min;               // min_k S_k
    double z;                   // sum_k exp(-(S_k - s_min)/lambda)
    double log_z;
    double ess;                 // z^2 / sum_k exp(-2 (S_k - s_min)/lambda)
};

// Partial results of one tile of samples: a row of the shifted weighted
// perturbation sums N_b of every (t, control) at [2t + d], and a head
//   [0] m_b (tile minimum)  [1] Z_b  [2] Q_b (sum of squares)  [3] unused
// kept in a compact array of its own (heads of consecutive tiles are
// consecutive), so that the combine reads all heads in a few lines.
constexpr int kHeadDoubles = 4;

// With per-step weights a partial row holds, for every step t, the tile
// minimum of the cost-to-go, the shifted exponential sums and the two
// weighted perturbation sums ([5t .. 5t+4]); there is no head array.
inline __host__ __device__ int partial_stride(int T, int per_step)
{
    return per_step ? 5 * T : 2 * T;
}

// Layout of the partials buffer of an instance: the tile rows, then 2T
// doubles where the iteration kernel keeps the controls it sampled around
// (read by the combine kernel when it smooths), then (total-cost weights)
// the tile heads.
inline __host__ __device__ size_t partial_heads_offset(int T, int per_step, size_t tiles)
{
    return tiles * (size_t)partial_stride(T, per_step) + 2 * (size_t)T;
}
inline __host__ __device__ size_t partial_doubles(int T, int per_step, size_t tiles)
{
    return partial_heads_offset(T, per_step, tiles) + (per_step ? 0 : kHeadDoubles * tiles);
}

// Tile partials are merged by the combine kernel, which takes up to kDirect
// rows in one pass.  Larger instances first merge their tiles by a tree of
// fixed shape (k_merge, a launch per level): a node of level l + 1 merges up
// to kFanIn consecutive nodes of level l, until at most kDirect nodes remain.
// The shape depends on the tile count only.
constexpr int kDirect = 2048;
// The combine kernel comes in two widths: up to kDirectSmall nodes (two heads
// per thread) and up to kDirect (eight per thread); a launch takes the
// narrowest that holds its largest instance.
constexpr int kDirectSmall = 512;
constexpr int kFanIn = 16;
// Nodes left for the combine kernel and the tiles each one spans.
inline __host__ __device__ int combine_nodes(int n_tiles, size_t* span)
{
    int n = n_tiles;
    size_t sp = 1;
    while (n > kDirect) {
        n = (n + kFanIn - 1) / kFanIn;
        sp *= kFanIn;
    }
    if (span) *span = sp;
    return n;
}

// Steps of U each combine workgroup updates.
constexpr int kCombineSteps = 4;
inline __host__ __device__ int combine_groups(int T) { return (T + kCombineSteps - 1) / kCombineSteps; }
// Step group of combine workgroup b of a grid `groups` wide.  A group's
// columns are 64 bytes of each tile row, the other half of their 128-byte
// line belongs to the neighbouring group; workgroups reach the 8 XCDs round
// robin (b and b + 8 share one), so within every whole run of 16 groups,
// groups 2p and 2p + 1 are given to two such blocks and the second finds
// the lines in their XCD's L2 instead of fetching them again.  A last run
// shorter than 16 keeps block b on group b.  A single instance's grid is
// padded to whole runs (blocks past the horizon return at once); a batch's,
// one row per instance, is not, to spare it the empty blocks.
inline __host__ __device__ int combine_group_of_block(int b, int grid)
{
    if ((b | 15) >= grid) return b;
    return (b & ~15) + 2 * (b & 7) + ((b >> 3) & 1);
}
inline __host__ __device__ int combine_grid(int groups, int n_inst)
{
    return n_inst == 1 ? (groups + 15) / 16 * 16 : groups;
}

// Everything one launch needs to run one MPPI iteration of one instance.
// Scene arrays are in the ego frame (x0's position subtracted) and float32.
struct InstDesc {
    int K, T, n_wp, n_c;
    int lanes;            // lanes per sample (G)
    int n_tiles;          // ceil(K / (kBlock / lanes))
    float dt, inv_dt, inv_L;
    float sig_a, sig_d;
    float a_min, a_max, d_min, d_max, v_max;
    float w_track, w_speed, w_effort, alpha, w_coll;
    float d_safe_c, d_safe_0;
    float ego_off[kMaxEgo];
    int n_ego;
    float px0, py0;       // initial position relative to the scene origin
    float th0, v0;        // initial yaw and speed
    double lambda;
    uint32_t key0, key1;  // Philox key = seed
    int shift;            // shift U by one step before the iteration (warm start)
    int cull;             // wave-level culling of waypoint chunks and circles
    int smooth;           // end with the Savitzky-Golay filter of eq. (sg)
    float w_target, w_yaw;// weights of c_target and c_yaw (0: term skipped)
    int coll_only;        // c_safe_dist only when d_obj <= 0
    int per_step;         // 1: weights from the cost-to-go per step
    int eps_stage;        // 1: tiles keep their perturbations in LDS (lds_layout)
    int wave_prio;        // 1: wave priority falls with the block index (see iteration_tile)
    int occ;              // iteration kernel it is launched with, kOcc... (host-side)
    int model;            // 1: 5-state model of eq. (5), steering-rate control
    float steer0;         // its initial steering angle
    float ego_ext;        // max |ego_off|
    int out_slot;         // slot in the gathered results of a batch (-1: none)
    unsigned mail_seq;    // number of the results that a batch leaves at mail
    double* mail;         // pinned host buffer (its device address) that receives
                          // U, the state and mail_seq after a batch; or nullptr
    // device pointers
    const float2* wp_xy;  // [n_wp]
    const float* wp_vref; // [n_wp]
    const float* wp_yaw;  // [n_wp]
    const float4* wp_box; // [chunks] (x_lo, x_hi, y_lo, y_hi) of each chunk
    const int* scene_flags; // [0]: every waypoint has the same reference speed
    const float4* c_pv;   // [n_c] (x, y, vx, vy)
    const float* c_rr;    // [n_c] r_c + r_ego
    const float* c_reach; // [n_c] circle_reach of each
    const float4* c_grp;  // circle_groups(n_c) groups of kCircleGroup consecutive
                          // circles, three float4s each: positions (x_lo, x_hi,
                          // y_lo, y_hi), velocities alike, largest c_reach
    double* U;            // [T][2]
    float* S;             // [K]
    float2* eps;          // [T][K]
    double* partials;     // partial_doubles(T, per_step, n_tiles)
    float* q;             // [T][K] stage costs (per-step weights)
    double* Stk;          // [T][K] cost-to-go (per-step weights; row 0 always, the
                          // other rows only when a tile works in global memory)
    DevState* st;
};

// Iteration kernels (the "occupancy" launch choice): the default compilation
// of k_batch, the one for kHiOccWaves waves per SIMD (8 and 16 lanes per
// sample only), and the split kernel (4, 8 and 16 lanes per sample, culling on).
constexpr int kOccDefault = 0;
constexpr int kOccHigh = 1;
constexpr int kOccSplit = 2;
constexpr int kOccModes = 3;
constexpr int kHiOccWaves = 5;

// Header of a batch arena in device memory: followed by the tile prefix
// (n_inst + 1 ints) at off_prefix and the descriptors at off_descs.
// Instances are grouped by kernel variant: class c = 50 * occ + 25 * model +
// 5 * lane_index + ne (occ the iteration kernel; model 0 or 1 (5-state);
// lane_index 0..4 for 1, 2, 4, 8, 16 lanes per sample, of the split kernel 0
// for 16 with per-step weights; ne = ego circles that meet
// obstacle circles, 0..4) owns instances [cls_begin[c], cls_begin[c+1]).
constexpr int kLaneClasses = 50 * kOccModes;
struct BatchHdr {
    int n_inst;
    int total_tiles;
    int off_prefix;
    int off_descs;
    int cls_begin[kLaneClasses + 1];
    int pad[2];
};

// Dynamic LDS layout of the iteration kernel for a given scene size.
struct LdsLayout {
    size_t c_pv, wp_box, wp_xy, red, wp_vref, wp_yaw, c_rr, omega, eps, qs, ss, total;
    int eps_staged;  // the tile's applied perturbations are kept at eps, and
                     // with per-step weights its stage costs at qs and its
                     // cost-to-go at ss
};

// Largest LDS copy of a tile's applied perturbations ([2T][spb + 1] floats)
// and, with per-step weights, stage costs ([T][spb + 1] floats) and
// cost-to-go ([T][spb + 1] doubles, rows padded by one).
constexpr size_t kEpsStageMax = 48 << 10;
// The copy is made when the workgroup's LDS stays within kLdsShared (five
// workgroups per compute unit), or within kLdsAlone for an instance launched
// alone with at most two tiles per compute unit (256 units).
constexpr size_t kLdsShared = 32 << 10;
constexpr size_t kLdsAlone = 64 << 10;

// Waypoints are grouped in chunks of this many consecutive points; each chunk
// has an axis-aligned bounding box in LDS for the wave-level culling.  A
// chunk is kChunkQ 16-byte (two-point) reads; the culled scan fetches
// kChunkTrip chunks per memory round trip.  (At the sine-lane workload
// chunks of 16 are 2% faster and chunks of 4 are 4% slower; at the paper's
// small scenes chunks of 16 are 5-8% slower.)
constexpr int kChunk = 8;
static_assert(kChunk == 4 || kChunk == 8 || kChunk == 16, "chunks of 4, 8 or 16 waypoints");
constexpr int kChunkQ = kChunk / 2;
constexpr int kChunkTrip = kChunk < 16 ? 16 / kChunk : 1;
// The per-lane culling bound takes the waypoints kSeedAhead, 2 kSeedAhead and
// 3 kSeedAhead after the start of the lane's previous closest chunk.
constexpr int kSeedAhead = 4;

// Scenes of more than kListedCircles circles are staged with their circles in
// order along the scene's longer axis, the moving ones after the others, and
// described in groups for the scan by rows: a wave tests a group per lane and
// then the circles of the near groups, instead of all of them, and those near
// one row lie together in its list (512 circles, a third of the groups near;
// stress instance 2.22 -> 1.65 ms, K = 4096 there 67 -> 53 us).
constexpr int kListedCircles = 64;
constexpr int kCircleGroup = 16;
inline __host__ __device__ int circle_groups(int n_c)
{
    return n_c > kListedCircles ? (n_c + kCircleGroup - 1) / kCircleGroup : 0;
}
// Radius around a circle's centre at the middle of a span of 16 steps that holds
// the circle throughout it, above float32 rounding: of the radius, and of the
// two times, whose difference of 7.5 steps carries up to 2^-23 of the horizon's
// 2048 (3e-5 of it, whatever the velocity).
template <typename F>  // (floats or vectors of them)
inline F circle_margin(F rr, F above_zero)  // (above_zero: max(rr, 0))
{
    return rr + 0.01f + 1e-6f * above_zero;
}
template <typename F>
inline F circle_travel(F speed, float dt)
{
    return 7.5f * dt * (1.0f + 1e-4f) * speed;
}
inline float circle_reach(float rr, float vx, float vy, float dt)
{
    return circle_margin(rr, fmaxf(rr, 0.0f)) + circle_travel(sqrtf(vx * vx + vy * vy), dt);
}

inline __host__ __device__ size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// scene_lds: the tile keeps a copy of the scene in LDS (the full scans of an
// instance without culling read it there; the culled scans read the scene
// from global memory, through the scalar cache for wave-uniform candidates).
inline __host__ __device__ LdsLayout lds_layout(int n_wp, int n_c, int T, int spb, int eps_stage,
                                                int per_step, int scene_lds)
{
    LdsLayout L;
    size_t o = 0;
    const size_t sc = scene_lds ? 1 : 0;
    L.c_pv = o;    o += sc * (size_t)n_c * 16;
    L.wp_box = o;  o += sc * (size_t)((n_wp + kChunk - 1) / kChunk) * 16;
    L.wp_xy = o;   o += sc * (size_t)((n_wp + kChunk - 1) / kChunk) * kChunk * 8;  // padded
    L.red = o;     o += 64 * 8;           // block reduction scratch (doubles)
    L.wp_vref = o; o += sc * (size_t)n_wp * 4;
    L.wp_yaw = o;  o += sc * (size_t)n_wp * 4;
    L.c_rr = o;    o += sc * (size_t)n_c * 4;
    o = align_up(o, 8);
    L.omega = o;   o += (size_t)spb * 8;   // float64 weights
    const size_t eb = (size_t)2 * T * (spb + 1) * 4;
    const size_t qb = per_step ? align_up((size_t)T * (spb + 1) * 4, 8) : 0;
    const size_t sb = per_step ? (size_t)T * (spb + 1) * 8 : 0;
    L.eps_staged = eps_stage && eb + qb + sb <= kEpsStageMax;
    L.eps = o;     o += L.eps_staged ? eb : 0;
    o = align_up(o, 8);
    L.qs = o;      o += L.eps_staged ? qb : 0;
    L.ss = o;      o += L.eps_staged ? sb : 0;
    L.total = align_up(o, 16);
    return L;
}

// The split iteration kernel (mppi_split.hpp): of each of a tile's four walker
// waves, one wave scans the waypoints and, with ego circles and obstacles, one
// the circles; the walker's states pass through a ring of split_ring(G) spans
// of 16 steps (28 KB of states and costs; at two lanes per sample one span
// takes 57).
inline __host__ __device__ constexpr int split_ring(int lanes) { return lanes >= 4 ? lanes / 4 : 1; }
inline __host__ __device__ constexpr int split_threads(int ne) { return kBlock * (ne > 0 ? 3 : 2); }
// Waves per SIMD that the kernel is compiled for.  A workgroup is three, so at 8
// and 4 lanes per sample, where some variants would take 81 to 85 registers, only
// one workgroup of these fitted a compute unit (131072 x 64, 512 circles, 4 ego
// circles 720 us against 439 with six; a batch of four of 65536 x 100, 12 circles,
// 3 ego circles 660 against 460).  (At 16 it takes at most 73 by itself.)
inline constexpr int split_waves(int lanes, int ne) { return lanes < 16 ? 6 : split_threads(ne) / 256; }
// Two workgroups of the split kernel share a compute unit's 160 KB of LDS.
// With more it is one, and k_batch's four are the faster again once every
// unit has a tile.
constexpr size_t kSplitLds = 80 << 10;
constexpr size_t kSplitLdsAlone = 160 << 10;
struct SplitLayout {
    size_t state, circ, wxy, cost, safe, extra, eps, qs, ss, carry, red, sk, counts, total;
    int staged;  // the tile keeps its perturbations at eps
};
inline __host__ __device__ SplitLayout split_layout(int T, int n_wp, int lanes, int per_step)
{
    SplitLayout L;
    size_t o = 0;
    const int spb = kBlock / lanes;                       // samples per tile
    const size_t n = (size_t)split_ring(lanes) * 16 * spb;  // steps in the ring
    L.state = o;  o += n * 16;
    L.circ = o;   o += (size_t)(kBlock / 64) * 65 * 32;
    L.wxy = o;    o += (size_t)((n_wp + kChunk - 1) / kChunk) * kChunk * 8;
    L.cost = o;   o += n * 4;
    L.safe = o;   o += n * 4;
    L.extra = o;  o += n * 4;
    // the cost-to-go is formed once the ring is free, and takes its place
    // where it fits
    const size_t ss = per_step ? (size_t)T * (spb + 1) * 8 : 0;
    L.ss = ss <= o ? 0 : o;
    o += ss <= o ? 0 : ss;
    L.carry = o;  o += lanes < 16 ? (size_t)spb * 16 : 0;
    L.red = o;    o += lanes < 16 ? (size_t)(64 + spb) * 8 : 0;
    L.qs = o;     o += per_step ? align_up((size_t)T * (spb + 1) * 4, 8) : 0;
    L.sk = o;     o += (size_t)spb * 4;
    L.counts = o; o += 4 * (kBlock / 64) * 4;
    // below 16 lanes per sample the perturbations are read back from L2 where
    // their copy would keep a second workgroup off the compute unit
    const size_t eps = (size_t)2 * T * (spb + 1) * 4;
    L.staged = lanes == 16 || o + eps <= kSplitLds;
    L.eps = o;    o += L.staged ? eps : 0;
    L.total = align_up(o, 16);
    return L;
}

// Dynamic LDS of the iteration kernel of an instance.
inline size_t iteration_lds(const InstDesc& d)
{
    return d.occ == kOccSplit ? split_layout(d.T, d.n_wp, d.lanes, d.per_step).total
                              : lds_layout(d.n_wp, d.n_c, d.T, kBlock / d.lanes, d.eps_stage, d.per_step,
                                           !d.cull).total;
}

// Launchers (mppi_kernels.hip).  All enqueue on `stream` and return the
// launch error, if any.
// Iteration kernel, one workgroup per tile: one instance (d0, hdr_dev ==
// nullptr) or lanes class `cls` of the batch described by the arena at
// hdr_dev (lanes is the launch shape of every instance it processes).
hipError_t launch_batch(int lanes, int ne, int model, int occ, int per_step, const InstDesc* d0,
                        const BatchHdr* hdr_dev, int cls, int grid, size_t smem,
                        hipStream_t stream);


// The split kernel, as launch_batch launches it (mppi_split.hip; at 4 and 8
// lanes per sample mppi_split_wide.hip, total-cost weights only).
hipError_t launch_split(int lanes, int ne, int model, int per_step, const InstDesc* d0, const BatchHdr* hdr_dev,
                        int cls, int grid, size_t smem, hipStream_t stream);
hipError_t launch_split_wide(int lanes, int ne, int model, const InstDesc* d0, const BatchHdr* hdr_dev, int cls,
                             int grid, size_t smem, hipStream_t stream);

// Merge of the tiles of one instance, or of every instance of a batch, down to
// at most kDirect nodes each (nothing to launch up to kDirect tiles);
// max_tiles: the most tiles among the instances whose weights are by total
// cost.
hipError_t launch_merge(const InstDesc* d0, const BatchHdr* hdr_dev, int max_tiles, int n_inst,
                        hipStream_t stream);

// Combine of the tile rows of one instance (d0, hdr_dev == nullptr) or of
// every instance of a batch (n_inst rows of the grid, groups = largest
// combine_groups(T) among them).
// max_nodes: the largest combine_nodes() among the instances.
hipError_t launch_combine(const InstDesc* d0, const BatchHdr* hdr_dev, int groups, int n_inst,
                          int max_nodes, hipStream_t stream);

// Ego circles that take part in the obstacle term of an instance.
inline int active_ego(int n_ego, int n_c) { return n_c > 0 ? n_ego : 0; }
hipError_t launch_shift_batch(const BatchHdr* hdr_dev, int n_inst, hipStream_t stream);
// Copies, for every instance with out_slot >= 0, U [2T], the status and the
// iteration counter to out + out_slot * slot_doubles.
hipError_t launch_gather(const BatchHdr* hdr_dev, int n_inst, double* out, int slot_doubles,
                         hipStream_t stream);
hipError_t launch_weights(const InstDesc& d, double* w_out, hipStream_t stream);

// Optimal rollout of Alg. 1 (float64, world frame) from x0 under the nominal
// controls U [T][2]: states [T+1][4] and applied controls [T][2].
struct TrajArgs {
    double x0[4];
    double steer0;  // initial steering angle (model 1)
    int T;
    int model;      // 1: 5-state model, states written with 5 columns
    double dt, wheelbase, a_min, a_max, d_min, d_max, v_max;
};
// A handle's pinned result buffer: U [T][2], the device state, then (64-byte
// aligned) the word that holds the number of the last results written.
inline __host__ __device__ size_t done_offset(int T)
{
    return align_up(sizeof(double) * 2 * (size_t)T + sizeof(DevState), 64);
}
// Leaves the results of every instance of a batch that has a mail buffer there.
hipError_t launch_mail(const BatchHdr* hdr_dev, int n_inst, hipStream_t stream);
// U [n] and the device state into host memory the device can write (pinned),
// then seq into *flag there.
hipError_t launch_export_controls(const double* U, int n, const DevState* st, double* out_u,
                                  DevState* out_st, unsigned* flag, unsigned seq, hipStream_t stream);
hipError_t launch_trajectory(const TrajArgs& a, const double* U, double* states, double* applied,
                             unsigned* flag, unsigned seq, hipStream_t stream);
// `bytes` (a multiple of 16) from pinned host memory (its device address) to
// device memory, then seq into *flag (unless flag is nullptr).
hipError_t launch_stage(const void* src, void* dst, size_t bytes, unsigned* flag, unsigned seq,
                        hipStream_t stream);
hipError_t launch_shift(double* U, int T, int steps, hipStream_t stream);
hipError_t launch_copy(const float4* src, float4* dst, size_t n16, hipStream_t stream);
hipError_t launch_debug_philox(uint32_t key0, uint32_t key1, unsigned long long n_iter,
                               uint32_t k0, uint32_t nk, uint32_t j0, uint32_t nj,
                               uint32_t* out, hipStream_t stream);

}  // namespace mppi_impl
