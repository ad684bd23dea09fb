// HIP kernel (gfx950 / CDNA4): the iteration kernel with the parts of a
// sample's rollout given to different waves (the split iteration kernel).
//
// k_batch (mppi_kernels.hip) gives every part of a sample's rollout to the
// sample's own 16 lanes.  A block of 16 steps is then one long chain --
// noise, noise check, five prefix sums, the waypoint scan, the circle scan --
// and an instance that does not fill the chip (K = 8192 at 16 lanes is two
// waves per SIMD) runs at the latency of that chain, block after block.
// Only the prefix sums of the walk carry state from block to block.  Here a
// workgroup of a tile (16 samples at 16 lanes per sample, 32 at 8, 64 at 4) has,
// for each quarter of its samples,
//
//   walker  noise, noise check and dynamics of every block; it leaves each
//           step's state in LDS, and later collects the steps' costs;
//   path    closest waypoint, tracking and speed cost of the walker's states;
//   circles clearance to the obstacle circles (only with ego circles and
//           obstacles);
//
// one wave each, which run concurrently: the scans of block b overlap the
// walk of the blocks after it.  States pass through a ring in LDS, in spans of
// 16 steps whatever the block; each wave counts the spans it has finished in
// LDS, and waits on the others' counts.  A walker waits only for spans that it
// wrote before, a scanning wave only for the walker, so every wait ends.
//
// What bounds it: VALU issue, at K = 4096 (three waves per SIMD) as at the
// largest instances; before, the chain's latency.  Iteration by HIP events,
// k_batch before and this kernel now: K = 1024, T = 50 18.4 -> 12.3 us; Table I
// shape 12.5 -> 9.8; K = 4096, T = 100 31.8 -> 17.9; sine lane (K = 8192,
// T = 100) 37.1 -> 24.8; K = 32768 95.8 -> 75.7; stress instance 3.09 -> 1.65
// ms; 256 uneven instances 3.03 -> 2.72 ms.  Candidates by rows instead of by
// wave (mppi_device.hpp) took the sine lane from 30.4 to 27 and K = 4096 in
// the stress scene from 152 to 68 us (with its circles in groups 53).
//
// The arithmetic of a step is the same code in both kernels and sums are
// formed in the same order, so their results are the same bit for bit, and
// which of them runs is only a matter of speed (occ in InstDesc).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "mppi_device.hpp"
#include "mppi_internal.hpp"

namespace mppi_impl {

namespace {

constexpr int kGroups = kBlock / 64;   // a walker, a path and a circles wave each
constexpr int kCircList = 2 * 65;      // float4s of a list of circles in LDS

// Waits until the count at p has reached n.  Every lane reads the same
// address, so the loop is uniform.
__device__ __forceinline__ void wait_count(const int* p, int n)
{
    while (__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < n)
        __builtin_amdgcn_s_sleep(1);
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}
__device__ __forceinline__ void post_count(int* p, int n)
{
    __hip_atomic_store(p, n, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// A span is 16 steps of every sample of the tile: 16 / G blocks of the walk,
// and for the scanning waves 16 / G row blocks of four samples by 16 steps a
// wave.  The ring holds split_ring(G) of them.
struct SplitLds {
    float4* state;  // [ring][kGroups][64 * 16 / G] (x, y, heading, v) after a step (place)
    float* cost;    // input cost (walker), then the cost but for the obstacle
                    // term and the extra terms (path), at the same places
    float* safe;    // obstacle cost before its weight (circles)
    float* extra;   // extra terms (path)
    float* eps;     // [2T][spb + 1] applied perturbations, columns as in k_batch
    float* sk;      // [spb] total costs
    float* qs;      // [T][spb + 1] stage costs (per-step weights)
    double* ss;     // [T][spb + 1] cost-to-go (per-step weights)
    float4* circ;   // [kGroups][65] circles of each circles wave (put_circle)
    float4* carry;  // [spb] where each sample's last span ended (path, G < 16)
    double* red;    // [64] reductions and
    double* omega;  // [spb] weights of the tile (G < 16)
    int* walked;    // [kGroups] spans finished by each walker
    int* tracked;   // [kGroups] by each path wave
    int* cleared;   // [kGroups] by each circles wave
    int* copied;    // [kGroups] waypoints copied by each path wave
    float4* wxy;    // [chunks][kChunkQ] the waypoints
};

__device__ __forceinline__ SplitLds split_bind(unsigned char* base, const SplitLayout& L)
{
    SplitLds s;
    s.state = reinterpret_cast<float4*>(base + L.state);
    s.cost = reinterpret_cast<float*>(base + L.cost);
    s.safe = reinterpret_cast<float*>(base + L.safe);
    s.extra = reinterpret_cast<float*>(base + L.extra);
    s.eps = reinterpret_cast<float*>(base + L.eps);
    s.sk = reinterpret_cast<float*>(base + L.sk);
    s.qs = reinterpret_cast<float*>(base + L.qs);
    s.ss = reinterpret_cast<double*>(base + L.ss);
    s.circ = reinterpret_cast<float4*>(base + L.circ);
    s.carry = reinterpret_cast<float4*>(base + L.carry);
    s.red = reinterpret_cast<double*>(base + L.red);
    s.omega = s.red + 64;
    s.walked = reinterpret_cast<int*>(base + L.counts);
    s.tracked = s.walked + kGroups;
    s.cleared = s.tracked + kGroups;
    s.copied = s.cleared + kGroups;
    s.wxy = reinterpret_cast<float4*>(base + L.wxy);
    return s;
}

// Place of step i of sample q of a wave's span: 16 steps a sample, each sample's
// turned by one more so that a walker's lanes, which hold the same steps of
// many samples below 16 lanes per sample, write to different banks.  A row
// block's lanes read 16 consecutive places in some order either way.
template <int G>
__device__ __forceinline__ int place(int q, int i)
{
    return G == 16 ? q * 16 + i : q * 16 + ((i + q) & 15);
}
// First step of the walk, at most 0: a horizon that is not a whole number of
// blocks starts with the partial one where that keeps step pairs together.
template <int G>
__device__ __forceinline__ int first_step(int T)
{
    const int rem = T % G;
    return (rem != 0 && (rem & 1) == 0) ? rem - G : 0;
}
__device__ __forceinline__ int span_count(int T, int t_first) { return (T - t_first + 15) / 16; }

// Minimum over the 16 lanes of each DPP row (in every lane).
__device__ __forceinline__ double row_min(double v)
{
    v = fmin(v, dpp_d<0xB1>(v));
    v = fmin(v, dpp_d<0x4E>(v));
    v = fmin(v, dpp_d<0x141>(v));
    return fmin(v, dpp_d<0x140>(v));
}

// Returns the total cost of the lane's sample as the weights take it (+inf
// where it is not finite or past the last sample).
template <int G, int NE, bool M5, bool PS>
__device__ __forceinline__ float walker(const InstDesc& d, const SplitLds& s, int tile, int g, bool staged)
{
    constexpr int kSpb = kBlock / G, kBlocks = 16 / G, kRing = split_ring(G);
    const int lane = threadIdx.x & 63;
    const int T = d.T, K = d.K;
    const int r = lane % G;
    const int smp = lane / G;                // sample of the wave
    const int grp = g * (64 / G) + smp;      // and of the tile
    const int k = tile * kSpb + grp;
    const bool valid = k < K;
    const int kk = valid ? k : K - 1;  // idle groups replay the last sample
    const unsigned long long n_iter = ld_g(&d.st->n_iter, 0);
    const int t_first = first_step<G>(T);
    const int n_blk = (T - t_first + G - 1) / G;
    const int n_span = span_count(T, t_first);
    double ua_next = ld_g(d.U, 2 * min(max(t_first + r, 0), T - 1));
    double ud_next = ld_g(d.U, 2 * min(max(t_first + r, 0), T - 1) + 1);
    WalkState w = {d.px0, d.py0, d.th0, d.v0, d.steer0};
    uint4 held = make_uint4(0u, 0u, 0u, 0u);
    float S = 0.0f, comp = 0.0f;  // Kahan pair of this lane's steps
    const bool full = d.w_target != 0.0f || d.w_yaw != 0.0f;
    auto slot = [&](int span) { return ((span % kRing) * kGroups + g) * (64 * kBlocks); };

    // the costs of this lane's steps of a span, once both scans have them
    auto collect = [&](int span) {
        wait_count(&s.tracked[g], span + 1);
        if (NE > 0) wait_count(&s.cleared[g], span + 1);
        const int at = slot(span);
#pragma unroll
        for (int j = 0; j < kBlocks; ++j) {
            const int i = at + place<G>(smp, j * G + r);
            float q = s.cost[i];
            if (NE > 0) q = fmaf(d.w_coll, s.safe[i], q);
            q = q + (full ? s.extra[i] : 0.0f);
            const int tm = t_first + span * 16 + j * G + r;
            if (tm >= 0 && tm < T) {
                if (PS) {
                    if (valid) st_g(d.q, (size_t)tm * K + k, q);
                    s.qs[tm * (kSpb + 1) + grp] = q;
                }
                const float yk = q - comp;
                const float tk = S + yk;
                comp = (tk - S) - yk;
                S = tk;
            }
        }
    };

    for (int blk = 0; blk < n_blk; ++blk) {
        const int span = blk / kBlocks, j = blk % kBlocks;
        const int t0 = t_first + blk * G;
        const int tm = t0 + r;
        const float2 Um = make_float2((float)ua_next, (float)ud_next);
        if (t0 + G < T) {
            const int tn = min(max(t0 + G + r, 0), T - 1);
            ua_next = ld_g(d.U, 2 * tn);
            ud_next = ld_g(d.U, 2 * tn + 1);
        }
        const StepControl ctl = block_controls<G, M5>(d, kk, t0, r, blk, n_iter, Um, held);
        StepState o;
        walk_block<G, M5>(d, ctl, t0, r, w, o);
        const float ea = o.a - Um.x, ed = ctl.dl - Um.y;
        const float q = input_cost(d, Um.x, Um.y, ea, ed);
        if (j == 0 && span >= kRing) collect(span - kRing);
        const int i = slot(span) + place<G>(smp, j * G + r);
        s.state[i] = make_float4(o.x, o.y, o.th, o.v);
        s.cost[i] = q;
        if (j == kBlocks - 1 || blk == n_blk - 1) post_count(&s.walked[g], span + 1);
        if (tm >= 0 && tm < T) {
            if (valid) st_wt(d.eps, (size_t)tm * K + k, make_float2(ea, ed));
            if (G == 16 || staged) {
                s.eps[(2 * tm) * (kSpb + 1) + grp] = ea;
                s.eps[(2 * tm + 1) * (kSpb + 1) + grp] = ed;
            }
        }
    }
    for (int span = max(n_span - kRing, 0); span < n_span; ++span) collect(span);

    // per-sample total over the G lanes (float64)
    double Sd = (double)S - (double)comp;
    if (G >= 2) Sd += dpp_d<0xB1>(Sd);
    if (G >= 4) Sd += dpp_d<0x4E>(Sd);
    if (G >= 8) Sd += dpp_d<0x141>(Sd);
    if (G >= 16) Sd += dpp_d<0x140>(Sd);
    float Sk = (float)Sd;
    if (!valid || !isfinite(Sk)) Sk = INFINITY;
    if (r == 0) {
        if (valid) st_g(d.S, k, (float)Sd);
        s.sk[grp] = Sk;
    }
    return Sk;
}

template <int G>
__device__ __forceinline__ void path_wave(const InstDesc& d, const SplitLds& s, int g)
{
    constexpr int kBlocks = 16 / G, kRing = split_ring(G);
    const int lane = threadIdx.x & 63;
    const int T = d.T;
    const int r = lane & 15;
    const int t_first = first_step<G>(T);
    const int n_span = span_count(T, t_first);
    const bool full = d.w_target != 0.0f || d.w_yaw != 0.0f;
    // the waypoints in LDS, copied by the path waves of the tile together
    const int n_ch = (d.n_wp + kChunk - 1) / kChunk;
    for (int i = threadIdx.x - kBlock; i < n_ch * kChunkQ; i += kBlock)
        s.wxy[i] = ld_g(reinterpret_cast<const float4*>(d.wp_xy), i);
    post_count(&s.copied[g], 1);
    float4 box[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        box[i] = r + 16 * i < n_ch ? ld_g(d.wp_box, r + 16 * i)
                                   : make_float4(INFINITY, -INFINITY, INFINITY, -INFINITY);
    const bool vref_uniform = ld_g(d.scene_flags, 0) != 0;
    const float vref0 = as_const(d.wp_vref)[0];
    // The position and the closest waypoint that a bound starts from: the lane's
    // previous step's, at 16 lanes per sample, or else where the sample's last
    // span ended; before the first the scene's origin and the waypoint that the
    // scene names for it.
    float xg = 0.0f, yg = 0.0f;
    int base = ld_g(d.scene_flags, 1);
    const float inv_sp = __builtin_bit_cast(float, ld_g(d.scene_flags, 2));
    float4* carry = s.carry + g * (64 / G);
    if (G < 16 && lane < 64 / G) carry[lane] = make_float4(0.0f, 0.0f, __builtin_bit_cast(float, base), 0.0f);
    float x_end = d.px0, y_end = d.py0;  // the position that the span started from
    for (int i = 0; i < kGroups; ++i) wait_count(&s.copied[i], 1);
    for (int span = 0; span < n_span; ++span) {
        wait_count(&s.walked[g], span + 1);
        const int at = ((span % kRing) * kGroups + g) * (64 * kBlocks);
        const int tm = t_first + span * 16 + r;
#pragma unroll 1
        for (int b = 0; b < kBlocks; ++b) {
            const int smp = 4 * b + (lane >> 4);
            const int i = at + place<G>(smp, r);
            const float4 st = s.state[i];
            const float q = s.cost[i];
            if (G < 16) {
                const float4 c = carry[smp];
                xg = c.x;
                yg = c.y;
                base = __builtin_bit_cast(int, c.z);
                x_end = span ? c.x : d.px0;
                y_end = span ? c.y : d.py0;
            }
            // position before the lane's step: the previous lane's after its
            // step, the end of the previous span for the first lane
            float xp = 0.0f, yp = 0.0f;
            if (d.w_target != 0.0f) {
                xp = __builtin_bit_cast(float, dpp_i<0x111>(__builtin_bit_cast(int, x_end),
                                                            __builtin_bit_cast(int, st.x)));
                yp = __builtin_bit_cast(float, dpp_i<0x111>(__builtin_bit_cast(int, y_end),
                                                            __builtin_bit_cast(int, st.y)));
                if (G == 16) {
                    x_end = dpp_f<0x15F>(st.x);
                    y_end = dpp_f<0x15F>(st.y);
                }
            }
            float ext;
            const float c = path_cost_rows(d, s.wxy, box, inv_sp, tm >= 0 && tm < T, vref0, vref_uniform,
                                           xg, yg, base, st.x, st.y, st.w, q, st.z, xp, yp, ext);
            s.cost[i] = c;
            if (full) s.extra[i] = ext;
            if (G < 16 && r == 15) carry[smp] = make_float4(st.x, st.y, __builtin_bit_cast(float, base), 0.0f);
        }
        post_count(&s.tracked[g], span + 1);
    }
}

template <int G, int NE>
__device__ __forceinline__ void circles_wave(const InstDesc& d, const SplitLds& s, int g)
{
    constexpr int kBlocks = 16 / G, kRing = split_ring(G);
    const int lane = threadIdx.x & 63;
    const int T = d.T;
    const int t_first = first_step<G>(T);
    const int n_span = span_count(T, t_first);
    float4* list = s.circ + g * kCircList;
    RowCircles rc;
    row_circles_init(d, list, rc);
    for (int span = 0; span < n_span; ++span) {
        wait_count(&s.walked[g], span + 1);
        const int at = ((span % kRing) * kGroups + g) * (64 * kBlocks);
        const int t0 = t_first + span * 16;
        const int tm = t0 + (lane & 15);
#pragma unroll 1
        for (int b = 0; b < kBlocks; ++b) {
            const int i = at + place<G>(4 * b + (lane >> 4), lane & 15);
            const float4 st = s.state[i];
            s.safe[i] = obstacle_cost_rows<NE>(d, list, rc, tm >= 0 && tm < T, st.x, st.y, st.z, st.w, t0);
        }
        post_count(&s.cleared[g], span + 1);
    }
}

template <int G, int NE, bool M5, bool PS>
__device__ __forceinline__ void split_tile(const InstDesc& d, int tile, unsigned char* smem)
{
    constexpr int kThreads = split_threads(NE), kSpb = kBlock / G;
    const int tid = threadIdx.x;
    const int T = d.T, K = d.K;
    const SplitLayout L = split_layout(T, d.n_wp, G, PS);
    const SplitLds s = split_bind(smem, L);
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int role = wv / kGroups, g = wv % kGroups;

    if (tid < 4 * kGroups) s.walked[tid] = 0;
    // the controls sampled around, kept for the smoothing combine
    if (d.smooth && tile == 0 && role == 1) {
        double* keep = d.partials + (size_t)d.n_tiles * partial_stride(T, d.per_step);
        for (int i = tid - kBlock; i < 2 * T; i += kBlock) st_g(keep, i, ld_g(d.U, i));
    }
    __syncthreads();  // the counts are cleared
    float Sk = INFINITY;
    if (role == 0) {
        Sk = walker<G, NE, M5, PS>(d, s, tile, g, L.staged);
    } else if (role == 1) {
        path_wave<G>(d, s, g);
    } else if (NE > 0) {
        circles_wave<G, NE>(d, s, g);
    }
    if (G < 16) {
        tile_partials<G, kThreads>(d, tile, Sk, s.red, s.omega, s.eps, L.staged);
        return;
    }
    if (PS) {
        per_step_partials<kThreads, kSpb>(d, tile, s.eps, s.qs, s.ss, true);
        return;
    }
    __syncthreads();

    // Tile partial, as in k_batch: the tile minimum, the float64 weights
    // (lane j < 16 of every wave holds sample j's, so that no second barrier
    // is needed) and one column (step, control) per thread, by as many waves
    // as there are columns for (all of them: 8% of the kernel's instructions
    // at T = 100).
    if (64 * wv >= 2 * T) return;
    const int n_valid = min(kSpb, K - tile * kSpb);
    Sk = s.sk[tid & (kSpb - 1)];
    const double m_b = row_min((double)Sk);
    double om = 0.0;
    if (isfinite(m_b) && Sk < INFINITY) om = exp(-((double)Sk - m_b) / d.lambda);
    double wj[kSpb];
#pragma unroll
    for (int j = 0; j < kSpb; ++j) wj[j] = lane_d(om, j);
    double* part = d.partials + (size_t)tile * partial_stride(T, 0);
    for (int col = tid; col < 2 * T; col += kThreads) {
        const float* e = s.eps + col * (kSpb + 1);
        double acc = 0.0;
        if (n_valid == kSpb) {
            float ev[kSpb];
#pragma unroll
            for (int j = 0; j < kSpb; ++j) ev[j] = e[j];
#pragma unroll
            for (int j = 0; j < kSpb; ++j) acc = fma(wj[j], (double)ev[j], acc);
        } else {
#pragma unroll
            for (int j = 0; j < kSpb; ++j)
                if (j < n_valid) acc = fma(wj[j], (double)e[j], acc);
        }
        st_g(part, col, acc);
    }
    if (wv == 0) {
        // Z_b and the sum of squares in k_batch's order: the four samples of
        // a group by pairs, then the groups (the squares come through lane
        // reads, so that none is fused into its sum)
        const double sq = om * om;
        double z = 0.0, q = 0.0;
#pragma unroll
        for (int i = 0; i < kGroups; ++i) {
            const double zi = (wj[4 * i] + wj[4 * i + 1]) + (wj[4 * i + 2] + wj[4 * i + 3]);
            const double qi = (lane_d(sq, 4 * i) + lane_d(sq, 4 * i + 1)) +
                              (lane_d(sq, 4 * i + 2) + lane_d(sq, 4 * i + 3));
            z = i == 0 ? zi : z + zi;
            q = i == 0 ? qi : q + qi;
        }
        if (tid == 0) {
            double* hd = d.partials + partial_heads_offset(T, 0, d.n_tiles) + kHeadDoubles * tile;
            st_g(hd, 0, m_b);
            st_g(hd, 1, z);
            st_g(hd, 2, q);
            st_g(hd, 3, 0.0);
        }
    }
}

// One instance: a workgroup per tile.
template <int G, int NE, bool M5, bool PS>
__global__ __launch_bounds__(split_threads(NE)) __attribute__((amdgpu_waves_per_eu(split_waves(G, NE))))
void k_split(InstDesc d0)
{
    extern __shared__ __align__(16) unsigned char smem[];
    split_tile<G, NE, M5, PS>(d0, blockIdx.x, smem);
}

// The instances of class cls of a batch.
template <int G, int NE, bool M5, bool PS>
__global__ __launch_bounds__(split_threads(NE)) __attribute__((amdgpu_waves_per_eu(split_waves(G, NE))))
void k_split_batch(const BatchHdr* __restrict__ hdr, int cls)
{
    extern __shared__ __align__(16) unsigned char smem[];
    with_batch_tile(hdr, cls, blockIdx.x, [&](const InstDesc& d, int tile) {
        split_tile<G, NE, M5, PS>(load_desc(d), tile, smem);
    });
}

template <int G, int NE, bool M5, bool PS>
hipError_t launch_split_v(const InstDesc* d0, const BatchHdr* hdr_dev, int cls, int grid, size_t smem,
                          hipStream_t stream)
{
    const dim3 g(grid), b(split_threads(NE));
    if (d0) hipLaunchKernelGGL((k_split<G, NE, M5, PS>), g, b, smem, stream, *d0);
    else hipLaunchKernelGGL((k_split_batch<G, NE, M5, PS>), g, b, smem, stream, hdr_dev, cls);
    return hipGetLastError();
}

template <int G, bool PS>
hipError_t launch_split_g(int ne, int model, const InstDesc* d0, const BatchHdr* hdr_dev, int cls, int grid,
                          size_t smem, hipStream_t stream)
{
#define MPPI_LAUNCH_NE(N)                                                                          \
    case N:                                                                                         \
        return model ? launch_split_v<G, N, true, PS>(d0, hdr_dev, cls, grid, smem, stream)         \
                     : launch_split_v<G, N, false, PS>(d0, hdr_dev, cls, grid, smem, stream);
    switch (ne) {
    MPPI_LAUNCH_NE(0)
    MPPI_LAUNCH_NE(1)
    MPPI_LAUNCH_NE(2)
    MPPI_LAUNCH_NE(3)
    MPPI_LAUNCH_NE(4)
    default: return hipErrorInvalidValue;
    }
#undef MPPI_LAUNCH_NE
}

}  // namespace

}  // namespace mppi_impl
