// HIP kernels (gfx950 / CDNA4) for one MPPI iteration of the planner of
// arXiv 2308.01654 (Algorithm 1, noise generation through the input update,
// with the costs of Sec. III and Sec. IV-C).
//
// An iteration is two launches.  The iteration kernel (k_batch) gives each
// workgroup a tile of samples; G lanes ("lanes per sample", 1..16)
// cooperate on one sample:
//
//   phase 1  rollout.  The horizon is walked in blocks of G steps.  Lane r of
//            a group draws the Philox/Box-Muller perturbation of step t0+r
//            and applies the control bounds; the speed before each step
//            (the noise check's speed cap) and the heading and position of
//            eq. (5) come from prefix sums over the G lanes, so each lane
//            holds the state reached at its own step.  Each lane then
//            evaluates the (expensive) stage cost of its own step: the
//            waypoint scan and the ego-circle x obstacle-circle distances,
//            culled per wave.  Costs are Kahan-summed per lane and combined
//            per sample in float64.  Applied perturbations are stored
//            time-major [T][K] as float2 (and kept in LDS for phase 2).
//   phase 2  tile partials.  Tile minimum m_b, then (float64)
//            omega_i = exp(-(S_i - m_b)/lambda), Z_b = sum omega_i and, for
//            every (t, control) column, the float64 sum of the products
//            omega_i * eps_eff[t][i] over the tile.
//
// Above kDirect tiles a fixed-shape tree (k_merge) merges them until kDirect
// nodes remain.  mppi_split.hpp has another iteration kernel, for 16, 8 and
// 4 lanes per sample, with the same results.
//
// The combine kernel (k_combine) merges the node rows in node order with the
// rescale exp(-(m_b - m)/lambda) and updates U in float64: U_t += N_t / Z
// (eq. (update-input)); it bumps the iteration counter and records S_min,
// log Z and the effective sample size.  Every order of summation is fixed,
// so results do not depend on which workgroup finishes first.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include "mppi_device.hpp"
#include "mppi_internal.hpp"

namespace mppi_impl {

// M5: the 5-state model of eq. (5) -- the steering angle is part of the state
// and the second control is the steering rate.
template <int G, int NE, bool M5>
__device__ __forceinline__ void iteration_tile(const InstDesc& d, int tile, unsigned char* smem)
{
    const int tid = threadIdx.x;
    constexpr int SPB = kBlock / G;  // samples per tile
    const int T = d.T;
    const int K = d.K;
    const LdsLayout L = lds_layout(d.n_wp, d.n_c, T, SPB, d.eps_stage, d.per_step, !d.cull);
    const Lds s = lds_bind(smem, L);

    // The culled scans read the scene from global memory, so the rollout
    // starts at once; the full scans (no culling) read a copy in LDS.
    if (!d.cull) {
        for (int i = tid; i < d.n_c; i += kBlock) {
            s.c_pv[i] = ld_g(d.c_pv, i);
            s.c_rr[i] = ld_g(d.c_rr, i);
        }
        const int n_wp_pad = (d.n_wp + kChunk - 1) / kChunk * kChunk;
        for (int i = tid; i < n_wp_pad; i += kBlock) {
            // padding points at infinity are never the closest
            s.wp_xy[i] = ld_g(d.wp_xy, i);
            if (i < d.n_wp) {
                s.wp_vref[i] = ld_g(d.wp_vref, i);
                s.wp_yaw[i] = ld_g(d.wp_yaw, i);
            }
        }
        // (x_lo, x_hi, y_lo, y_hi) of every chunk, formed with the scene
        for (int c = tid; c * kChunk < d.n_wp; c += kBlock) s.wp_box[c] = ld_g(d.wp_box, c);
    }
    // the controls sampled around, kept for the smoothing combine
    if (d.smooth && tile == 0) {
        double* keep = d.partials + (size_t)d.n_tiles * partial_stride(T, d.per_step);
        for (int i = tid; i < 2 * T; i += kBlock) st_g(keep, i, ld_g(d.U, i));
    }
    const unsigned long long n_iter = ld_g(&d.st->n_iter, 0);
    // one reference speed for every waypoint: the closest index is not needed
    const bool vref_uniform = ld_g(d.scene_flags, 0) != 0;
    const float vref0 = as_const(d.wp_vref)[0];
    if (!d.cull) __syncthreads();

    // ---------------------------------------------------------------- phase 1
    const int grp = tid / G;
    const int r = tid % G;
    const int k_base = tile * SPB;
    const int k = k_base + grp;
    const bool valid = k < K;
    const int kk = valid ? k : K - 1;  // idle groups replay the last sample

    LaneCull lc;
    lc.box = lane_chunk_box(d, tid & 63);
    lane_circle(d, tid & 63, lc.cpv, lc.crr);
    WalkState w = {d.px0, d.py0, d.th0, d.v0, d.steer0};
    float S = 0.0f, comp = 0.0f;  // Kahan pair of this lane's steps
    int seed = -1;                // closest chunk at this lane's previous step
    uint4 held = make_uint4(0u, 0u, 0u, 0u);  // Philox words kept for the next block
    // A horizon that is not a whole number of blocks starts with the partial
    // block (its leading lanes own no step), where the samples are still
    // close together and the culled scans are short, rather than ending with
    // it, where they have spread the most.  Kept even so that Philox step
    // pairs stay within a lane pair.
    const int rem = T % G;
    const int t_first = (rem != 0 && (rem & 1) == 0) ? rem - G : 0;
    // the nominal control of the lane's step (float64 in global memory),
    // fetched one block ahead
    double ua_next = ld_g(d.U, 2 * min(max(t_first + r, 0), T - 1));
    double ud_next = ld_g(d.U, 2 * min(max(t_first + r, 0), T - 1) + 1);
    int blk = 0;
    for (int t0 = t_first; t0 < T; t0 += G, ++blk) {
        // Where two waves share a SIMD, the one in the earlier block issues
        // first (wave priority 3 in blocks 0-1, 2 in 2-3, 1 in 4-5, then 0),
        // so that the pair tends to finish together instead of leaving the
        // later one to run alone at the end.
        if (d.wave_prio) {
            switch (min(blk >> 1, 3)) {
            case 0: __builtin_amdgcn_s_setprio(3); break;
            case 1: __builtin_amdgcn_s_setprio(2); break;
            case 2: __builtin_amdgcn_s_setprio(1); break;
            default: __builtin_amdgcn_s_setprio(0); break;
            }
        }
        const int tm = t0 + r;
        const float2 Um = make_float2((float)ua_next, (float)ud_next);
        if (t0 + G < T) {
            const int tn = min(max(t0 + G + r, 0), T - 1);
            ua_next = ld_g(d.U, 2 * tn);
            ud_next = ld_g(d.U, 2 * tn + 1);
        }
        // the lane's waypoints ahead of its previous closest chunk (the
        // culling's own bound), fetched before they are needed
        float2 sw[3];
        if (d.cull) {
            const int sb = max(seed, 0) * kChunk;
#pragma unroll
            for (int u = 0; u < 3; ++u) sw[u] = ld_g32(d.wp_xy, (unsigned)min(sb + (u + 1) * kSeedAhead, d.n_wp - 1));
        }
        const StepControl ctl = block_controls<G, M5>(d, kk, t0, r, blk, n_iter, Um, held);
        StepState o;
        walk_block<G, M5>(d, ctl, t0, r, w, o);
        const float mx = o.x, my = o.y, mth = o.th, mv = o.v;
        const float mc = __cosf(mth), ms = __sinf(mth);
        const float mUa = Um.x, mUd = Um.y;
        const float mea = o.a - Um.x, med = ctl.dl - Um.y;
        const bool act = tm >= 0 && tm < T;
        // the culling's own bound (consumes the waypoint loads of the block
        // start before the store below enters the vector-memory counter)
        float own_d2 = INFINITY;
        if (d.cull && seed >= 0) {
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                const float dx = mx - sw[u].x;
                const float dy = my - sw[u].y;
                own_d2 = fminf(own_d2, fmaf(dy, dy, dx * dx));
            }
        }
        // The applied perturbation is stored now, before the stage cost: the
        // store then retires during the scans instead of holding up the next
        // block's first wait on the vector-memory counter (loads and stores
        // share it and complete in order).
        if (act) {
            if (valid) st_wt(d.eps, (size_t)tm * K + k, make_float2(mea, med));
            if (L.eps_staged) {
                s.eps[(2 * tm) * (SPB + 1) + grp] = mea;
                s.eps[(2 * tm + 1) * (SPB + 1) + grp] = med;
            }
        }
        float q = 0.0f;
        if (d.cull)
            q = stage_cost_culled<NE>(d, own_d2, vref0, lc, vref_uniform, act, seed, mx, my, mc, ms, mv, mUa, mUd, mea, med, tm,
                                      max(t0, 0), min(t0 + G, T) - 1, mth, o.xp, o.yp);
        else if (act)
            q = stage_cost<NE>(d, s, mx, my, mc, ms, mv, mUa, mUd, mea, med, tm, mth, o.xp, o.yp);
        if (act && d.per_step) {
            if (valid) st_g(d.q, (size_t)tm * K + k, q);
            if (L.eps_staged) s.qs[tm * (SPB + 1) + grp] = q;
        }
        if (act) {
            const float yk = q - comp;
            const float tk = S + yk;
            comp = (tk - S) - yk;
            S = tk;
        }
    }

    // per-sample total over the G lanes (float64)
    double Sd = (double)S - (double)comp;
    if (G >= 2) Sd += dpp_d<0xB1>(Sd);
    if (G >= 4) Sd += dpp_d<0x4E>(Sd);
    if (G >= 8) Sd += dpp_d<0x141>(Sd);
    if (G >= 16) Sd += dpp_d<0x140>(Sd);
    float Sk = (float)Sd;
    if (!valid || !isfinite(Sk)) Sk = INFINITY;
    if (valid && r == 0) st_g(d.S, k, (float)Sd);

    // ---------------------------------------------------------------- phase 2
    // the tile's last steps go first
    if (d.wave_prio) __builtin_amdgcn_s_setprio(3);
    if (d.per_step) {
        per_step_partials<kBlock, SPB>(d, tile, s.eps, s.qs, s.ss, L.eps_staged);
    } else {
        tile_partials<G, kBlock>(d, tile, Sk, s.red, s.omega, s.eps, L.eps_staged);
    }
}

// One level of the merge of an instance with more than kDirect tiles, before
// its combine: node g of the next level merges up to kFanIn consecutive nodes
// of this one (tiles at level 0) in order, with the log-sum-exp shift to
// their common minimum; its row and head replace those of its first tile.
// One workgroup per node.  (A launch of its own: as the end of the iteration
// kernel, with a ticket per group and a device-wide release by every tile,
// the merge kept the tiles' workgroups resident through the releases.)
__device__ void merge_node(const InstDesc& d, int level, int g)
{
    __shared__ double sc_lds[kFanIn];
    int n_l = d.n_tiles;  // nodes at this level
    size_t span = 1;      // tiles per node
    for (int l = 0; l < level && n_l > kDirect; ++l) {
        n_l = (n_l + kFanIn - 1) / kFanIn;
        span *= kFanIn;
    }
    const int first = g * kFanIn;
    if (d.per_step || n_l <= kDirect || first >= n_l) return;
    const int nc = min(kFanIn, n_l - first);
    const int tid = threadIdx.x;
    const int T = d.T;
    const int stride = partial_stride(T, 0);
    double* rows = d.partials + (size_t)first * span * stride;
    const size_t cstride = span * stride;  // between consecutive children
    double* head = d.partials + partial_heads_offset(T, 0, d.n_tiles) + kHeadDoubles * (size_t)first * span;
    if (tid < 64) {
        const double* h = head + kHeadDoubles * (size_t)min(tid, nc - 1) * span;
        const double mi = tid < nc ? ld_g(h, 0) : INFINITY;
        const double zi = tid < nc ? ld_g(h, 1) : 0.0;
        const double qi = tid < nc ? ld_g(h, 2) : 0.0;
        const double mm = wave_min(mi);
        // a child whose samples are all non-finite has m = +inf and weight 0
        const double sc = (tid < nc && isfinite(mi)) ? exp(-(mi - mm) / d.lambda) : 0.0;
        const double zz = wave_sum(zi * sc);
        const double qq = wave_sum(qi * sc * sc);
        if (tid < kFanIn) sc_lds[tid] = sc;
        if (tid == 0) {
            st_g(head, 0, mm);
            st_g(head, 1, zz);
            st_g(head, 2, qq);
        }
    }
    __syncthreads();
    for (int col = tid; col < 2 * T; col += kBlock) {
        const double* src = rows + col;
        // every child in flight at once, merged in child order
        double pv[kFanIn];
#pragma unroll
        for (int u = 0; u < kFanIn; ++u) pv[u] = u < nc ? ld_g(src, (size_t)u * cstride) : 0.0;
        double acc = 0.0;
#pragma unroll
        for (int u = 0; u < kFanIn; ++u)
            if (u < nc) acc += pv[u] * sc_lds[u];
        st_g(rows, col, acc);
    }
}

__global__ __launch_bounds__(kBlock) void k_merge(InstDesc d0, const BatchHdr* __restrict__ hdr, int level)
{
    if (!hdr) {
        merge_node(d0, level, blockIdx.x);
        return;
    }
    if ((int)blockIdx.y >= hdr->n_inst) return;
    merge_node(reinterpret_cast<const InstDesc*>(
                   reinterpret_cast<const unsigned char*>(hdr) + hdr->off_descs)[blockIdx.y],
               level, blockIdx.x);
}

hipError_t launch_merge(const InstDesc* d0, const BatchHdr* hdr_dev, int max_tiles, int n_inst,
                        hipStream_t stream)
{
    InstDesc zero;
    memset(&zero, 0, sizeof zero);
    int level = 0;
    for (int n = max_tiles; n > kDirect; ++level) {
        n = (n + kFanIn - 1) / kFanIn;
        hipLaunchKernelGGL(k_merge, dim3(n, n_inst), dim3(kBlock), 0, stream, d0 ? *d0 : zero, hdr_dev, level);
    }
    return hipGetLastError();
}

// Combine (Alg. 1, the normaliser and the input update of eq.
// (update-input)): merges the KH * kBlock (<= kDirect) or fewer remaining node rows of one
// instance.  Every workgroup forms the global minimum m and the node scales
// exp(-(m_b - m)/lambda), Z and Q itself (node order, fixed trees), then
// updates kCombineSteps steps of U: U_t += N_t / Z with N_t summed over the
// nodes in a fixed order (each thread a chunk of consecutive nodes in order,
// the chunks of a wave by a fixed butterfly, then the four waves in order).
// With smoothing it also updates the two steps on either side
// (from the controls the iteration kernel kept) and writes its own steps
// after eq. (sg).  Workgroup 0 records the statistics and bumps the
// iteration counter.  Nothing is written if no sample cost is finite.
// With MULTI the workgroup takes step groups cg to cg_end - 1, forming the
// scales once; otherwise group cg.
template <int KH, bool MULTI>
__device__ void combine(const InstDesc& d, int cg, int cg_end)
{
    extern __shared__ __align__(16) unsigned char csm[];
    double* sc = reinterpret_cast<double*>(csm);   // [KH * kBlock + 16] node scales
    double* red = sc + KH * kBlock + 16;           // [64] reductions
    double* part = red + 64;                       // [4 waves][16 slots] column partials
    double* un = part + kBlock;                    // [16] updated worked columns
    const int tid = threadIdx.x;
    const int T = d.T;
    int s0 = cg * kCombineSteps;
    if (s0 >= T) return;
    int s1 = min(s0 + kCombineSteps, T);
    int w0 = d.smooth ? max(s0 - 2, 0) : s0;
    int w1 = d.smooth ? min(s1 + 2, T) : s1;
    int ncol = 2 * (w1 - w0);          // worked columns, 2 * w0 first
    int slots = ncol <= 8 ? 8 : 16;    // threads per chunk
    int chunks = kBlock / slots;
    const int stride = partial_stride(T, 0);
    size_t span = 1;
    const int n = combine_nodes(d.n_tiles, &span);
    const size_t nstride = span * stride;    // between nodes
    const double* rows = d.partials;
    const double* heads = d.partials + partial_heads_offset(T, 0, d.n_tiles);

    // One round trip: the node heads (KH per thread, from the
    // compact head array), the controls sampled around and the first sixteen
    // nodes of this thread's chunk of its worked column.  Every load is
    // issued unconditionally at an index clamped into its array and the
    // value is replaced by the neutral element afterwards, so the heads can
    // be used while the row loads are still in flight and the sums below run
    // without branches (an added +0.0 leaves a sum that started at +0.0
    // unchanged, so the results are those of skipping the term).
    constexpr int kH = KH;
    double mh[kH], zh[kH], qh[kH];
#pragma unroll
    for (int r = 0; r < kH; ++r) {
        const int i = tid + r * kBlock;
        const double* h = heads + kHeadDoubles * (size_t)min(i, n - 1) * span;
        mh[r] = ld_g(h, 0);
        zh[r] = ld_g(h, 1);
        qh[r] = ld_g(h, 2);
    }
    int slot = tid % slots, chunk = tid / slots;
    int per = (n + chunks - 1) / chunks;
    int i0 = min(chunk * per, n), i1 = min(i0 + per, n);
    bool worked = slot < ncol;
    const double* src = rows + min(2 * w0 + slot, 2 * T - 1);
    // the controls the iteration sampled around (kept after the tile rows when
    // smoothing, since other workgroups rewrite U), loaded with the rest
    const double* u_old = d.smooth ? d.partials + (size_t)d.n_tiles * stride : d.U;
    double u_ld = ld_g(u_old, min(2 * w0 + tid, 2 * T - 1));
    double pv[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) pv[u] = ld_g(src, (size_t)min(i0 + u, n - 1) * nstride);
    // (z and q masked by a product, which keeps their loads ahead of the
    // rows': a select lets the compiler sink them into the branch below)
#pragma unroll
    for (int r = 0; r < kH; ++r) {
        const bool in = tid + r * kBlock < n;
        const double keep = in ? 1.0 : 0.0;
        mh[r] = in ? mh[r] : INFINITY;
        zh[r] *= keep;
        qh[r] *= keep;
    }

    // global minimum
    double mloc = mh[0];
#pragma unroll
    for (int r = 1; r < kH; ++r) mloc = fmin(mloc, mh[r]);
    const double wm = wave_min(mloc);
    const int wv = tid >> 6;
    if ((tid & 63) == 0) red[wv] = wm;
    __syncthreads();
    double m = red[0];
#pragma unroll
    for (int i = 1; i < kBlock / 64; ++i) m = fmin(m, red[i]);
    if (!isfinite(m)) {
        if (cg == 0 && tid == 0) d.st->status = -4;  // MPPI_E_NONFINITE: U and n unchanged
        return;
    }
    // node scales (every slot of the scale array written, 0 beyond the
    // nodes and in the 16 slots of padding), Z and Q (thread, wave, then
    // waves in order)
    if (tid < 16) sc[kH * kBlock + tid] = 0.0;
    double zl = 0.0, ql = 0.0;
#pragma unroll
    for (int r = 0; r < kH; ++r) {
        const double si = isfinite(mh[r]) ? exp(-(mh[r] - m) / d.lambda) : 0.0;
        sc[tid + r * kBlock] = si;
        zl += zh[r] * si;
        ql += qh[r] * si * si;
    }
    const double wz = wave_sum(zl), wq = wave_sum(ql);
    if ((tid & 63) == 0) {
        red[4 + wv] = wz;
        red[8 + wv] = wq;
    }
    __syncthreads();  // also publishes the scales
    double z = red[4], q = red[8];
#pragma unroll
    for (int i = 1; i < kBlock / 64; ++i) {
        z += red[4 + i];
        q += red[8 + i];
    }

    const bool first = cg == 0;
    for (;;) {
        // weighted perturbation sums of the worked columns, nodes in order
        // (i0 + u and b + u stay below n + 16: the padding covers them)
        double acc = 0.0;
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const double pu = (worked && i0 + u < i1) ? pv[u] : 0.0;
            acc += pu * sc[i0 + u];
        }
        for (int b = i0 + 16; b < i1; b += 16) {
#pragma unroll
            for (int u = 0; u < 16; ++u) pv[u] = ld_g(src, (size_t)min(b + u, n - 1) * nstride);
#pragma unroll
            for (int u = 0; u < 16; ++u) {
                const double pu = (worked && b + u < i1) ? pv[u] : 0.0;
                acc += pu * sc[b + u];
            }
        }
        // the column's sum over the chunks: the chunks of a wave (lanes slots
        // apart) by a fixed butterfly, then the four waves in order
        if (slots == 8) acc += dpp_d<0x128>(acc);  // row_ror:8, lanes 8 apart in a row
        acc = add_lanes_16_apart(acc);
        acc = add_lanes_32_apart(acc);
        if ((tid & 63) < slots) part[wv * 16 + (tid & 63)] = acc;
        __syncthreads();
        if (tid < ncol) {
            const double nsum = ((part[tid] + part[16 + tid]) + part[32 + tid]) + part[48 + tid];
            const int col = 2 * w0 + tid;
            const double u = u_ld + nsum / z;
            if (d.smooth) un[tid] = u;
            else d.U[col] = u;
        }
        if (d.smooth) {
            __syncthreads();
            // eq. (sg) on the own steps: u*_t = (-3 u_{t-2} + 12 u_{t-1} + 17 u_t +
            // 12 u_{t+1} - 3 u_{t+2}) / 35, the end values repeated beyond the horizon
            const int own = 2 * (s1 - s0);
            if (tid < own) {
                const int t = s0 + (tid >> 1), c2 = tid & 1;
                auto at = [&](int i) { return un[2 * (min(max(i, 0), T - 1) - w0) + c2]; };
                const double sm = -3.0 * at(t - 2) + 12.0 * at(t - 1) + 17.0 * at(t) +
                                  12.0 * at(t + 1) - 3.0 * at(t + 2);
                d.U[2 * s0 + tid] = sm / 35.0;
            }
        }
        if (!MULTI || ++cg >= cg_end || cg * kCombineSteps >= T) break;
        // the next group's rows
        s0 = cg * kCombineSteps;
        s1 = min(s0 + kCombineSteps, T);
        w0 = d.smooth ? max(s0 - 2, 0) : s0;
        w1 = d.smooth ? min(s1 + 2, T) : s1;
        ncol = 2 * (w1 - w0);
        slots = ncol <= 8 ? 8 : 16;
        chunks = kBlock / slots;
        slot = tid % slots;
        chunk = tid / slots;
        per = (n + chunks - 1) / chunks;
        i0 = min(chunk * per, n);
        i1 = min(i0 + per, n);
        worked = slot < ncol;
        src = rows + min(2 * w0 + slot, 2 * T - 1);
        u_ld = ld_g(u_old, min(2 * w0 + tid, 2 * T - 1));
#pragma unroll
        for (int u = 0; u < 16; ++u) pv[u] = ld_g(src, (size_t)min(i0 + u, n - 1) * nstride);
        __syncthreads();  // part and un are read
    }
    if (first && tid == 0) {
        d.st->s_min = m;
        d.st->z = z;
        d.st->log_z = log(z);
        d.st->ess = z * z / q;
        d.st->status = 0;
        d.st->n_iter = d.st->n_iter + 1ull;
    }
}

// Combine with per-step weights: the tile rows hold, per step t, the tile
// minimum m_b,t of the cost-to-go and the shifted sums Z, Q, N_a, N_d.  A
// workgroup updates kCombineSteps steps (and, with smoothing, the two on
// either side): per step the minimum over the tiles, each tile's sums
// shifted to it by exp(-(m_b,t - m_t)/lambda), U_t += N_t / Z_t.  Thread
// (chunk, slot) takes step slot over a chunk of consecutive tiles, in tile
// order; the chunks of a wave are merged by a fixed butterfly, then the four
// waves in order.  The step-0 heads and the first kPsBatch rows of the
// thread's chunk are loaded in one round trip and kept in registers for both
// passes.  A sample whose total cost is finite has a finite cost-to-go at
// every step, so every step is finite exactly when step 0 is; without a
// finite step 0 nothing is written.  Workgroup 0 records the statistics of
// step 0.
constexpr int kPsBatch = 16;

__device__ void combine_per_step(const InstDesc& d, int cg)
{
    extern __shared__ __align__(16) unsigned char csm[];
    double* red = reinterpret_cast<double*>(csm);  // [64]
    double* part = red + 64;                       // [4 waves][8 slots][4] wave partials
    double* mt = part + 4 * kBlock;                // [8] step minima
    double* un = mt + 8;                           // [16] updated worked columns
    const int tid = threadIdx.x;
    const int T = d.T;
    const int s0 = cg * kCombineSteps;
    if (s0 >= T) return;
    const int s1 = min(s0 + kCombineSteps, T);
    const int w0 = d.smooth ? max(s0 - 2, 0) : s0;
    const int w1 = d.smooth ? min(s1 + 2, T) : s1;
    const int nst = w1 - w0;                 // worked steps (at most 8)
    constexpr int kSlots = 8;                // threads per chunk
    constexpr int kChunks = kBlock / kSlots;
    const size_t stride = partial_stride(T, 1);
    const int n = d.n_tiles;
    const double* rows = d.partials;
    const int wv = tid >> 6;

    const int slot = tid % kSlots, chunk = tid / kSlots;
    const bool worked = slot < nst;
    const int t = w0 + min(slot, nst - 1);
    const int per = (n + kChunks - 1) / kChunks;
    const int b0 = min(chunk * per, n), b1 = min(b0 + per, n);
    const double* col = rows + 5 * (size_t)t;
    const double* u_old = d.smooth ? d.partials + (size_t)n * stride : d.U;
    // One round trip: the step-0 heads, the controls sampled around and the
    // chunk's first rows.  Loads are issued unconditionally at indices
    // clamped into the arrays and the neutral values selected afterwards
    // (+inf for a minimum; the sums below then add exact zeros), so that no
    // load waits behind a branch.
    const int uc = 2 * (w0 + min(tid, nst - 1));
    const double ua_ld = ld_g(u_old, uc), ud_ld = ld_g(u_old, uc + 1);
    double m0v[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) m0v[r] = ld_g(rows, (size_t)min(tid + r * kBlock, n - 1) * stride);
    double hv[kPsBatch][5];
#pragma unroll
    for (int u = 0; u < kPsBatch; ++u) {
        const double* h = col + (size_t)min(b0 + u, n - 1) * stride;
#pragma unroll
        for (int c = 0; c < 5; ++c) hv[u][c] = ld_g(h, c);
    }
    double m0 = INFINITY;
#pragma unroll
    for (int r = 0; r < 2; ++r) m0 = fmin(m0, tid + r * kBlock < n ? m0v[r] : INFINITY);
    for (int b = tid + 2 * kBlock; b < n; b += kBlock) m0 = fmin(m0, rows[(size_t)b * stride]);
#pragma unroll
    for (int u = 0; u < kPsBatch; ++u) {
        const bool on = worked && b0 + u < b1;
        const double keep = on ? 1.0 : 0.0;
        hv[u][0] = on ? hv[u][0] : INFINITY;
#pragma unroll
        for (int c = 1; c < 5; ++c) hv[u][c] *= keep;
    }

    // step 0: minimum over the tiles (every workgroup)
    const double w0m = wave_min(m0);
    if ((tid & 63) == 0) red[wv] = w0m;
    __syncthreads();
    m0 = red[0];
#pragma unroll
    for (int i = 1; i < kBlock / 64; ++i) m0 = fmin(m0, red[i]);
    if (!isfinite(m0)) {
        if (cg == 0 && tid == 0) d.st->status = -4;  // MPPI_E_NONFINITE: U and n unchanged
        return;
    }

    // per-step minimum: the chunk (rows past the first batch loaded again),
    // the chunks of the wave, then the waves
    double ml = INFINITY;
#pragma unroll
    for (int u = 0; u < kPsBatch; ++u) ml = fmin(ml, hv[u][0]);
    if (worked)
        for (int b = b0 + kPsBatch; b < b1; ++b) ml = fmin(ml, col[(size_t)b * stride]);
#pragma unroll
    for (int o = kSlots; o < 64; o <<= 1) ml = fmin(ml, __shfl_xor(ml, o, 64));
    if ((tid & 63) < kSlots) part[4 * (wv * kSlots + slot)] = ml;
    __syncthreads();
    if (tid < kSlots) {
        double m = part[4 * tid];
#pragma unroll
        for (int w = 1; w < kBlock / 64; ++w) m = fmin(m, part[4 * (w * kSlots + tid)]);
        mt[tid] = m;
    }
    __syncthreads();

    // shifted sums of the chunk's tiles in tile order
    // (m is finite for a worked step, so a tile with m_b,t = +inf -- or a
    // slot of the batch past the chunk -- gets exp(-inf) = +0 exactly and
    // adds zeros: no branch per tile)
    double z = 0.0, qq = 0.0, na = 0.0, nd = 0.0;
    if (worked) {
        const double m = mt[slot];
        const double lam = d.lambda;
        auto add = [&](const double (&h)[5]) {
            const double sc = exp(-(h[0] - m) / lam);
            z += h[1] * sc;
            qq += h[2] * sc * sc;
            na += h[3] * sc;
            nd += h[4] * sc;
        };
#pragma unroll
        for (int u = 0; u < kPsBatch; ++u) add(hv[u]);
        for (int b = b0 + kPsBatch; b < b1; ++b) {
            const double* hp = col + (size_t)b * stride;
            const double h[5] = {hp[0], hp[1], hp[2], hp[3], hp[4]};
            add(h);
        }
    }
#pragma unroll
    for (int o = kSlots; o < 64; o <<= 1) {
        z += __shfl_xor(z, o, 64);
        qq += __shfl_xor(qq, o, 64);
        na += __shfl_xor(na, o, 64);
        nd += __shfl_xor(nd, o, 64);
    }
    __syncthreads();  // the minima in part are read
    if ((tid & 63) < kSlots) {
        double* pw = part + 4 * (wv * kSlots + slot);
        pw[0] = z;
        pw[1] = qq;
        pw[2] = na;
        pw[3] = nd;
    }
    __syncthreads();
    if (tid < nst) {
        double zt = 0.0, qt = 0.0, sa = 0.0, sd = 0.0;
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) {
            const double* pc = part + 4 * (w * kSlots + tid);
            zt += pc[0];
            qt += pc[1];
            sa += pc[2];
            sd += pc[3];
        }
        const int tt = w0 + tid;
        const double ua = ua_ld + sa / zt;
        const double ud = ud_ld + sd / zt;
        if (d.smooth) {
            un[2 * tid] = ua;
            un[2 * tid + 1] = ud;
        } else {
            d.U[2 * tt] = ua;
            d.U[2 * tt + 1] = ud;
        }
        if (cg == 0 && tt == 0) {
            d.st->s_min = mt[0];
            d.st->z = zt;
            d.st->log_z = log(zt);
            d.st->ess = zt * zt / qt;
            d.st->status = 0;
            d.st->n_iter = d.st->n_iter + 1ull;
        }
    }
    if (d.smooth) {
        __syncthreads();
        const int own = 2 * (s1 - s0);
        if (tid < own) {
            const int ts = s0 + (tid >> 1), c2 = tid & 1;
            auto at = [&](int i) { return un[2 * (min(max(i, 0), T - 1) - w0) + c2]; };
            const double sm = -3.0 * at(ts - 2) + 12.0 * at(ts - 1) + 17.0 * at(ts) +
                              12.0 * at(ts + 1) - 3.0 * at(ts + 2);
            d.U[2 * s0 + tid] = sm / 35.0;
        }
    }
}

// One instance (d0, hdr == nullptr) or instance blockIdx.y of a batch, whose
// workgroups take gpw consecutive step groups each; KH node heads per thread.
template <int KH, bool MULTI>
__global__ __launch_bounds__(kBlock) void k_combine(InstDesc d0, const BatchHdr* __restrict__ hdr, int gpw)
{
    if (!MULTI && !hdr) {
        const int cg = combine_group_of_block(blockIdx.x, gridDim.x);
        if (d0.per_step) combine_per_step(d0, cg);
        else combine<KH, false>(d0, cg, cg + 1);
        return;
    }
    if ((int)blockIdx.y >= hdr->n_inst) return;
    const InstDesc& d = reinterpret_cast<const InstDesc*>(
        reinterpret_cast<const unsigned char*>(hdr) + hdr->off_descs)[blockIdx.y];
    const int cg = MULTI ? (int)blockIdx.x * gpw : combine_group_of_block(blockIdx.x, gridDim.x);
    if (!d.per_step) {
        combine<KH, MULTI>(d, cg, cg + gpw);
        return;
    }
    for (int i = 0; i < (MULTI ? gpw : 1); ++i) {
        if (i) __syncthreads();  // the group before is done with the LDS
        combine_per_step(d, cg + i);
    }
}

template <int KH>
static void launch_combine_k(const InstDesc& a, const BatchHdr* hdr_dev, int groups, int n_inst, int gpw,
                             hipStream_t stream)
{
    const size_t smem = sizeof(double) * (KH * kBlock + 64 + 4 * kBlock + 8 + 16);
    if (gpw > 1)
        hipLaunchKernelGGL((k_combine<KH, true>), dim3((groups + gpw - 1) / gpw, n_inst), dim3(kBlock), smem,
                           stream, a, hdr_dev, gpw);
    else
        hipLaunchKernelGGL((k_combine<KH, false>), dim3(combine_grid(groups, n_inst), n_inst), dim3(kBlock),
                           smem, stream, a, hdr_dev, gpw);
}

hipError_t launch_combine(const InstDesc* d0, const BatchHdr* hdr_dev, int groups, int n_inst,
                          int max_nodes, hipStream_t stream)
{
    InstDesc zero;
    memset(&zero, 0, sizeof zero);
    // Every workgroup forms the scales of all nodes, so in a large batch it
    // takes up to four groups, as long as 1024 workgroups are left (256 uneven
    // instances of up to 1024 nodes: combine 150 -> 108 us, iteration 2.69 ->
    // 2.66 ms; with eight groups the same).
    constexpr int kMaxGroups = 4;
    int gpw = 1;
    while (gpw < kMaxGroups && (long)groups * n_inst / (2 * gpw) >= 1024) gpw *= 2;
    const InstDesc& a = d0 ? *d0 : zero;
    if (max_nodes <= kDirectSmall) launch_combine_k<kDirectSmall / kBlock>(a, hdr_dev, groups, n_inst, gpw, stream);
    else launch_combine_k<kDirect / kBlock>(a, hdr_dev, groups, n_inst, gpw, stream);
    return hipGetLastError();
}

// Inclusive prefix sum (MAX = false) or maximum (MAX = true) over the lanes of
// a wave (float64): inside each row of 16 by row shifts, then lane 15 of rows
// 0 and 2 into the row after each, then lane 31 into rows 2 and 3.
template <int CTRL, int ROW_MASK, bool MAX>
__device__ __forceinline__ double scan_stage(double v)
{
    const long long id = __builtin_bit_cast(long long, MAX ? -INFINITY : 0.0);
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp((int)id, (int)b, CTRL, ROW_MASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(id >> 32), (int)(b >> 32), CTRL, ROW_MASK, 0xf, false);
    const double u = __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
    return MAX ? fmax(v, u) : v + u;
}
template <bool MAX>
__device__ __forceinline__ double wave_scan(double v)
{
    v = scan_stage<0x111, 0xf, MAX>(v);  // row_shr:1
    v = scan_stage<0x112, 0xf, MAX>(v);
    v = scan_stage<0x114, 0xf, MAX>(v);
    v = scan_stage<0x118, 0xf, MAX>(v);
    v = scan_stage<0x142, 0xa, MAX>(v);  // row_bcast:15
    return scan_stage<0x143, 0xc, MAX>(v);  // row_bcast:31
}

// Exclusive prefix sums (MAX = false) or maxima (MAX = true) of N values over
// the threads of a workgroup in thread order (float64), the scans side by
// side: inside a wave by lane moves, the totals of the earlier waves through
// LDS (red: N * kBlock / 64 doubles).  Thread 0 gets 0 (sum) or -inf
// (maximum).
template <bool MAX, int N>
__device__ __forceinline__ void block_excl(double (&v)[N], double* red)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const double id = MAX ? -INFINITY : 0.0;
    double incl[N];
#pragma unroll
    for (int i = 0; i < N; ++i) incl[i] = wave_scan<MAX>(v[i]);
    if (blockDim.x > 64) {
        __syncthreads();  // red is free
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (lane == 63) red[i * (kBlock / 64) + wv] = incl[i];
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        double excl = __shfl_up(incl[i], 1, 64);
        if (lane == 0) excl = id;
        double before = id;
        for (int w = 0; w < wv; ++w)
            before = MAX ? fmax(before, red[i * (kBlock / 64) + w]) : before + red[i * (kBlock / 64) + w];
        v[i] = MAX ? fmax(before, excl) : before + excl;
    }
}
template <bool MAX>
__device__ __forceinline__ double block_excl(double v, double* red)
{
    double a[1] = {v};
    block_excl<MAX, 1>(a, red);
    return a[0];
}

// A store to the host's memory, past every cache of the device (relaxed, system
// scope).
__device__ __forceinline__ void st_host(double* p, size_t i, double v)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p) + i, __builtin_bit_cast(unsigned long long, v),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// Tells the host that a workgroup's results are in its memory: once every
// thread's stores there (st_host) are acknowledged, the flag.  (A system-scope
// fence would also write back what the device's L2 holds for others.)
__device__ __forceinline__ void post_host(unsigned* flag, unsigned seq)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(flag, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Optimal rollout of Alg. 1 in float64 and world coordinates: from x0,
// x*_{t+1} = F(x*_t, u*_t) (eq. (5), explicit Euler from the old state), each
// nominal control put through the noise check with zero noise (bounds, speed
// cap, braking bound last).  One workgroup, each thread a run of consecutive
// steps.  While the start is within v_max and a_min <= 0 the braking bound
// cannot bind and the capped speeds have the closed form of the iteration
// kernel's walk (v_t = min(v_0 + S_t, v_max + S_t - max_{1<=k<=t} S_k), S_t
// the sum of the first t commanded changes); heading, steering angle
// (5-state model) and position are prefix sums of their increments.  A start
// above v_max, or a positive a_min (the braking bound then lifts the speed
// above v_max whenever the cap falls below it), is walked step by step by one
// thread.  kP: steps per thread at most (the launch has a step per thread
// wherever T allows: the tangents, sines and cosines of the unused ones had
// been most of the kernel, 6.6 us at T = 16 and 100).
template <int kP>
__global__ __launch_bounds__(kBlock) void k_trajectory(TrajArgs a, const double* __restrict__ U,
                                                       double* __restrict__ xs,
                                                       double* __restrict__ us, unsigned* flag, unsigned seq)
{
    __shared__ double red[2 * (kBlock / 64)];
    // Up to 256 steps the results are gathered here and leave in one run of
    // consecutive stores (the states' columns are strided: each value was a bus
    // write of its own).
    __shared__ double out[kP == 1 ? 7 * (kBlock + 1) : 1];
    const int cols = a.model ? 5 : 4;  // the 5-state model also writes delta
    const int T = a.T;
    const int ns = cols * (T + 1);
    auto put1 = [&](double* p, int at, int i, double v) {
        if (kP == 1) out[at + i] = v;
        else p[i] = v;
    };
    auto leave = [&]() {
        __syncthreads();
        if (kP == 1) {
            for (int i = threadIdx.x; i < ns; i += blockDim.x) st_host(xs, i, out[i]);
            for (int i = threadIdx.x; i < 2 * T; i += blockDim.x) st_host(us, i, out[ns + i]);
        } else {
            __threadfence_system();
        }
        post_host(flag, seq);
    };
    auto put = [&](int t, double x, double y, double th, double v, double delta) {
        const int o = cols * t;
        put1(xs, 0, o, x);
        put1(xs, 0, o + 1, y);
        put1(xs, 0, o + 2, th);
        put1(xs, 0, o + 3, v);
        if (a.model) put1(xs, 0, o + 4, delta);
    };
    if (!(a.x0[3] <= a.v_max) || a.a_min > 0.0) {
        if (threadIdx.x == 0) {
            double x = a.x0[0], y = a.x0[1], th = a.x0[2], v = a.x0[3], delta = a.steer0;
            put(0, x, y, th, v, delta);
            for (int t = 0; t < T; ++t) {
                double acc = fmin(fmax(U[2 * t], a.a_min), a.a_max);
                acc = fmax(fmin(acc, (a.v_max - v) / a.dt), a.a_min);
                const double u2 = fmin(fmax(U[2 * t + 1], a.d_min), a.d_max);
                const double vdt = a.dt * v;
                const double xn = x + vdt * cos(th);
                const double yn = y + vdt * sin(th);
                // the steering angle is the control, or (5-state model) the state
                const double thn = th + vdt * tan(a.model ? delta : u2) / a.wheelbase;
                if (a.model) delta += a.dt * u2;
                v += a.dt * acc;
                x = xn;
                y = yn;
                th = thn;
                put1(us, ns, 2 * t, acc);
                put1(us, ns, 2 * t + 1, u2);
                put(t + 1, x, y, th, v, delta);
            }
        }
        leave();
        return;
    }
    const int P = kP == 1 ? 1 : (T + kBlock - 1) / kBlock;
    const int t0 = threadIdx.x * P;
    double acmd[kP], u2[kP], ds[kP];
    // commanded speed changes and their sums before each own step
    double run = 0.0;
#pragma unroll
    for (int j = 0; j < kP; ++j) {
        const int t = t0 + j;
        acmd[j] = u2[j] = 0.0;
        if (j < P && t < T) {
            acmd[j] = fmin(fmax(U[2 * t], a.a_min), a.a_max);
            u2[j] = fmin(fmax(U[2 * t + 1], a.d_min), a.d_max);
        }
        ds[j] = run;
        run += a.dt * acmd[j];
    }
    const double s_before = block_excl<false>(run, red);  // S at this thread's first step
    // S_t of every own step, and the maximum of S_k over 1 <= k <= t: the
    // earlier threads' maximum, then this thread's running one
    double sv[kP], qv[kP];
    double qrun = -INFINITY;
#pragma unroll
    for (int j = 0; j < kP; ++j) {
        sv[j] = s_before + ds[j];
        if (j < P && t0 + j >= 1 && t0 + j < T) qrun = fmax(qrun, sv[j]);
        qv[j] = qrun;
    }
    const double qp = block_excl<true>(qrun, red);
    double v[kP], acc[kP], dth[kP], dd[kP];
    double drun = 0.0;
#pragma unroll
    for (int j = 0; j < kP; ++j) {
        const double q = fmax(qp, qv[j]);
        v[j] = t0 + j == 0 ? a.x0[3] : fmin(a.x0[3] + sv[j], a.v_max + sv[j] - q);
        acc[j] = fmax(fmin(acmd[j], (a.v_max - v[j]) / a.dt), a.a_min);
        dd[j] = drun;  // steering change before the own step, within the thread
        drun += a.model ? a.dt * u2[j] : 0.0;
    }
    const double d_before = a.model ? block_excl<false>(drun, red) : 0.0;
    double run_th = 0.0;
#pragma unroll
    for (int j = 0; j < kP; ++j) {
        const double delta = a.steer0 + d_before + dd[j];
        const double tn = tan(a.model ? delta : u2[j]);
        dth[j] = run_th;
        run_th += (j < P && t0 + j < T) ? a.dt * v[j] * tn / a.wheelbase : 0.0;
    }
    const double th_before = block_excl<false>(run_th, red);
    double run_x = 0.0, run_y = 0.0, dx[kP], dy[kP];
#pragma unroll
    for (int j = 0; j < kP; ++j) {
        const double th = a.x0[2] + th_before + dth[j];
        dx[j] = run_x;
        dy[j] = run_y;
        if (j < P && t0 + j < T) {
            run_x += a.dt * v[j] * cos(th);
            run_y += a.dt * v[j] * sin(th);
        }
    }
    double xy_before[2] = {run_x, run_y};
    block_excl<false, 2>(xy_before, red);
    const double x_before = xy_before[0], y_before = xy_before[1];
#pragma unroll
    for (int j = 0; j < kP; ++j) {
        const int t = t0 + j;
        if (j >= P || t >= T) break;
        put1(us, ns, 2 * t, acc[j]);
        put1(us, ns, 2 * t + 1, u2[j]);
        put(t, a.x0[0] + x_before + dx[j], a.x0[1] + y_before + dy[j], a.x0[2] + th_before + dth[j],
            v[j], a.steer0 + d_before + dd[j]);
        if (t == T - 1) {
            // the state after the last step
            const double vdt = a.dt * v[j];
            const double th = a.x0[2] + th_before + dth[j];
            const double delta = a.steer0 + d_before + dd[j];
            put(T, a.x0[0] + x_before + dx[j] + vdt * cos(th), a.x0[1] + y_before + dy[j] + vdt * sin(th),
                th + vdt * tan(a.model ? delta : u2[j]) / a.wheelbase, v[j] + a.dt * acc[j],
                delta + (a.model ? a.dt * u2[j] : 0.0));
        }
    }
    leave();
}

// Iteration kernel for one or many instances of one launch shape (G lanes
// per sample): one workgroup per tile.  The lanes-per-sample shape is a
// property of the instance, so an instance computes the same bits alone or in
// any batch.
template <int G, int NE, bool M5>
__device__ __forceinline__ void any_tile(const InstDesc& d0, const BatchHdr* __restrict__ hdr, int cls,
                                         unsigned char* smem)
{
    if (!hdr) {
        if ((int)blockIdx.x < d0.n_tiles) iteration_tile<G, NE, M5>(d0, blockIdx.x, smem);
        return;
    }
    with_batch_tile(hdr, cls, blockIdx.x, [&](const InstDesc& d, int tile) {
        iteration_tile<G, NE, M5>(d, tile, smem);
    });
}

template <int G, int NE, bool M5>
__global__ __launch_bounds__(kBlock) void k_batch(InstDesc d0, const BatchHdr* __restrict__ hdr,
                                                  int cls)
{
    extern __shared__ __align__(16) unsigned char smem[];
    any_tile<G, NE, M5>(d0, hdr, cls, smem);
}

// The same kernel compiled for five waves per SIMD (at most 96 VGPRs, a few
// spilled in some variants): the shape for instances with many more waves
// than the GPU holds at once, where the extra wave hides more latency than
// the spills cost.
template <int G, int NE, bool M5>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kHiOccWaves)))
void k_batch_hi(InstDesc d0, const BatchHdr* __restrict__ hdr, int cls)
{
    extern __shared__ __align__(16) unsigned char smem[];
    any_tile<G, NE, M5>(d0, hdr, cls, smem);
}

// occ: kOccDefault or kOccHigh (the latter for 8 and 16 lanes per sample
// only; other shapes take the default compilation).
template <int G, bool M5, int OCC>
static hipError_t launch_gm(int ne, const InstDesc& a, const BatchHdr* hdr_dev, int cls, int grid,
                            size_t smem, hipStream_t stream)
{
    const dim3 g(grid), b(kBlock);
#define MPPI_LAUNCH_NE(N)                                                                        \
    case N:                                                                                       \
        if constexpr (OCC == kOccHigh)                                                            \
            hipLaunchKernelGGL((k_batch_hi<G, N, M5>), g, b, smem, stream, a, hdr_dev, cls);     \
        else                                                                                      \
            hipLaunchKernelGGL((k_batch<G, N, M5>), g, b, smem, stream, a, hdr_dev, cls);        \
        break;
    switch (ne) {
    MPPI_LAUNCH_NE(0)
    MPPI_LAUNCH_NE(1)
    MPPI_LAUNCH_NE(2)
    MPPI_LAUNCH_NE(3)
    MPPI_LAUNCH_NE(4)
    default: return hipErrorInvalidValue;
    }
#undef MPPI_LAUNCH_NE
    return hipGetLastError();
}

template <int G, int OCC>
static hipError_t launch_go(int ne, int model, const InstDesc& a, const BatchHdr* hdr_dev,
                            int cls, int grid, size_t smem, hipStream_t stream)
{
    return model ? launch_gm<G, true, OCC>(ne, a, hdr_dev, cls, grid, smem, stream)
                 : launch_gm<G, false, OCC>(ne, a, hdr_dev, cls, grid, smem, stream);
}

template <int G>
static hipError_t launch_g(int ne, int model, int occ, const InstDesc& a, const BatchHdr* hdr_dev,
                           int cls, int grid, size_t smem, hipStream_t stream)
{
    if constexpr (G >= 8) {
        if (occ == kOccHigh) return launch_go<G, kOccHigh>(ne, model, a, hdr_dev, cls, grid, smem, stream);
    }
    return launch_go<G, kOccDefault>(ne, model, a, hdr_dev, cls, grid, smem, stream);
}

hipError_t launch_batch(int lanes, int ne, int model, int occ, int per_step, const InstDesc* d0,
                        const BatchHdr* hdr_dev, int cls, int grid, size_t smem,
                        hipStream_t stream)
{
    if (occ == kOccSplit) return launch_split(lanes, ne, model, per_step, d0, hdr_dev, cls, grid, smem, stream);
    InstDesc zero;
    memset(&zero, 0, sizeof zero);
    const InstDesc& a = d0 ? *d0 : zero;
    switch (lanes) {
    case 1: return launch_g<1>(ne, model, occ, a, hdr_dev, cls, grid, smem, stream);
    case 2: return launch_g<2>(ne, model, occ, a, hdr_dev, cls, grid, smem, stream);
    case 4: return launch_g<4>(ne, model, occ, a, hdr_dev, cls, grid, smem, stream);
    case 8: return launch_g<8>(ne, model, occ, a, hdr_dev, cls, grid, smem, stream);
    case 16: return launch_g<16>(ne, model, occ, a, hdr_dev, cls, grid, smem, stream);
    default: return hipErrorInvalidValue;
    }
}

// Receding-horizon shift of every instance that asks for it (one workgroup
// per instance): U_t <- U_{min(t + 1, T-1)}.
__global__ void k_shift_batch(const BatchHdr* __restrict__ hdr)
{
    __shared__ double buf[2 * kMaxT];
    const InstDesc* descs = reinterpret_cast<const InstDesc*>(
        reinterpret_cast<const unsigned char*>(hdr) + hdr->off_descs);
    const int inst = blockIdx.x;
    if (inst >= hdr->n_inst) return;
    const InstDesc& d = descs[inst];
    if (!d.shift) return;
    const int T = d.T;
    for (int i = threadIdx.x; i < 2 * T; i += blockDim.x) buf[i] = d.U[i];
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * T; i += blockDim.x) {
        const int t = min((i >> 1) + 1, T - 1);
        d.U[i] = buf[2 * t + (i & 1)];
    }
}

hipError_t launch_shift_batch(const BatchHdr* hdr_dev, int n_inst, hipStream_t stream)
{
    hipLaunchKernelGGL(k_shift_batch, dim3(n_inst), dim3(256), 0, stream, hdr_dev);
    return hipGetLastError();
}

__global__ void k_gather(const BatchHdr* __restrict__ hdr, double* __restrict__ out,
                         int slot_doubles)
{
    const InstDesc* descs = reinterpret_cast<const InstDesc*>(
        reinterpret_cast<const unsigned char*>(hdr) + hdr->off_descs);
    const int inst = blockIdx.x;
    if (inst >= hdr->n_inst) return;
    const InstDesc& d = descs[inst];
    if (d.out_slot < 0) return;
    double* o = out + (size_t)d.out_slot * slot_doubles;
    for (int i = threadIdx.x; i < 2 * d.T; i += blockDim.x) o[i] = d.U[i];
    if (threadIdx.x == 0) {
        o[2 * d.T] = (double)d.st->status;
        o[2 * d.T + 1] = (double)d.st->n_iter;
    }
}

hipError_t launch_gather(const BatchHdr* hdr_dev, int n_inst, double* out, int slot_doubles,
                         hipStream_t stream)
{
    hipLaunchKernelGGL(k_gather, dim3(n_inst), dim3(256), 0, stream, hdr_dev, out, slot_doubles);
    return hipGetLastError();
}

// Normalised weights of the last iteration: w_k = exp(-(S_k - S_min)/lambda)/Z,
// from the float32 totals S or, with per-step weights, from the float64
// cost-to-go of step 0 (S0, the totals those weights were formed from).
__global__ void k_weights(const float* __restrict__ S, const double* __restrict__ S0, int K,
                          double lambda, const DevState* __restrict__ st, double* __restrict__ w)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K) return;
    const double sk = S0 ? S0[k] : (double)S[k];
    w[k] = isfinite(sk) ? exp(-(sk - st->s_min) / lambda) / st->z : 0.0;
}

// The nominal controls and the device state copied into the caller's pinned
// host memory.
__device__ __forceinline__ void export_results(const double* U, int n, const DevState* st, double* out_u,
                                               DevState* out_st, unsigned* flag, unsigned seq)
{
    constexpr int kWords = sizeof(DevState) / sizeof(double);
    static_assert(kWords * sizeof(double) == sizeof(DevState), "whole words");
    if (threadIdx.x < kWords)
        st_host(reinterpret_cast<double*>(out_st), threadIdx.x, reinterpret_cast<const double*>(st)[threadIdx.x]);
    for (int i = threadIdx.x; i < n; i += kBlock) st_host(out_u, i, U[i]);
    post_host(flag, seq);
}

// (one launch instead of two copies back)
__global__ __launch_bounds__(kBlock) void k_export_controls(const double* __restrict__ U, int n,
                                                            const DevState* __restrict__ st,
                                                            double* __restrict__ out_u,
                                                            DevState* __restrict__ out_st,
                                                            unsigned* flag, unsigned seq)
{
    export_results(U, n, st, out_u, out_st, flag, seq);
}

// The same for every instance of a batch, one workgroup each: the batch's
// results are in the host's memory when it ends, and a read of an instance
// afterwards launches nothing (256 reads after a batch: 2.7 -> 0.7 ms).
__global__ __launch_bounds__(kBlock) void k_mail(const BatchHdr* __restrict__ hdr)
{
    if ((int)blockIdx.x >= hdr->n_inst) return;
    const InstDesc& d = reinterpret_cast<const InstDesc*>(
        reinterpret_cast<const unsigned char*>(hdr) + hdr->off_descs)[blockIdx.x];
    if (!d.mail) return;
    unsigned* flag = reinterpret_cast<unsigned*>(reinterpret_cast<unsigned char*>(d.mail) + done_offset(d.T));
    export_results(d.U, 2 * d.T, d.st, d.mail, reinterpret_cast<DevState*>(d.mail + 2 * d.T), flag, d.mail_seq);
}

hipError_t launch_mail(const BatchHdr* hdr_dev, int n_inst, hipStream_t stream)
{
    hipLaunchKernelGGL(k_mail, dim3(n_inst), dim3(kBlock), 0, stream, hdr_dev);
    return hipGetLastError();
}

hipError_t launch_export_controls(const double* U, int n, const DevState* st, double* out_u,
                                  DevState* out_st, unsigned* flag, unsigned seq, hipStream_t stream)
{
    hipLaunchKernelGGL(k_export_controls, dim3(1), dim3(kBlock), 0, stream, U, n, st, out_u,
                       out_st, flag, seq);
    return hipGetLastError();
}

hipError_t launch_trajectory(const TrajArgs& a, const double* U, double* states, double* applied,
                             unsigned* flag, unsigned seq, hipStream_t stream)
{
    // a step per thread up to 256 steps, of one wave up to 64
    const dim3 g(1), b(a.T <= 64 ? 64 : kBlock);
    if (a.T <= kBlock)
        hipLaunchKernelGGL(k_trajectory<1>, g, b, 0, stream, a, U, states, applied, flag, seq);
    else
        hipLaunchKernelGGL(k_trajectory<kMaxT / kBlock>, g, b, 0, stream, a, U, states, applied, flag, seq);
    return hipGetLastError();
}

// A staged scene from the pinned host buffer to the device, read over the bus
// by one workgroup with every load of a thread in flight; the flag tells the
// host that the buffer may be filled again.  (Against a copy command and an
// event: 8.7 -> 4.6 us a scene of 4 KB with the kernel after it, where the
// event's packet alone held up the queue for 4 us.)
constexpr int kStageThreads = 1024;
__global__ __launch_bounds__(kStageThreads) void k_stage(const f4v* __restrict__ src, f4v* __restrict__ dst,
                                                         int n, unsigned* flag, unsigned seq)
{
    for (int i0 = 0; i0 < n; i0 += 4 * kStageThreads) {
        f4v v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * kStageThreads + (int)threadIdx.x;
            if (i < n) v[u] = as_global(src)[i];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * kStageThreads + (int)threadIdx.x;
            if (i < n) as_global(dst)[i] = v[u];
        }
    }
    // (a thread's stores were issued once its loads had returned)
    __syncthreads();
    if (flag && threadIdx.x == 0) __hip_atomic_store(flag, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

hipError_t launch_stage(const void* src, void* dst, size_t bytes, unsigned* flag, unsigned seq,
                        hipStream_t stream)
{
    hipLaunchKernelGGL(k_stage, dim3(1), dim3(kStageThreads), 0, stream, static_cast<const f4v*>(src),
                       static_cast<f4v*>(dst), (int)(bytes / 16), flag, seq);
    return hipGetLastError();
}

hipError_t launch_weights(const InstDesc& d, double* w_out, hipStream_t stream)
{
    hipLaunchKernelGGL(k_weights, dim3((d.K + 255) / 256), dim3(256), 0, stream, d.S,
                       d.per_step ? d.Stk : nullptr, d.K, d.lambda, d.st, w_out);
    return hipGetLastError();
}

// Receding-horizon shift: U_t <- U_{min(t + steps, T-1)}.
__global__ void k_shift(double* U, int T, int steps)
{
    extern __shared__ double buf[];
    for (int i = threadIdx.x; i < 2 * T; i += blockDim.x) buf[i] = U[i];
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * T; i += blockDim.x) {
        const int t = min((i >> 1) + steps, T - 1);
        U[i] = buf[2 * t + (i & 1)];
    }
}

hipError_t launch_shift(double* U, int T, int steps, hipStream_t stream)
{
    hipLaunchKernelGGL(k_shift, dim3(1), dim3(256), (size_t)T * 2 * sizeof(double), stream, U,
                       T, steps);
    return hipGetLastError();
}

// Streaming copy used to calibrate traffic counters.
__global__ void k_copy(const float4* __restrict__ src, float4* __restrict__ dst, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        dst[i] = src[i];
}

hipError_t launch_copy(const float4* src, float4* dst, size_t n16, hipStream_t stream)
{
    hipLaunchKernelGGL(k_copy, dim3(4096), dim3(256), 0, stream, src, dst, n16);
    return hipGetLastError();
}

__global__ void k_debug_philox(uint32_t key0, uint32_t key1, unsigned long long n_iter,
                               uint32_t k0, uint32_t nk, uint32_t j0, uint32_t nj, uint32_t* out)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (uint64_t)nk * nj) return;
    const uint32_t k = k0 + (uint32_t)(i / nj);
    const uint32_t j = j0 + (uint32_t)(i % nj);
    const uint4 r = philox4x32_10(make_uint4(k, j, (uint32_t)n_iter, (uint32_t)(n_iter >> 32)),
                                  key0, key1);
    reinterpret_cast<uint4*>(out)[i] = r;
}

hipError_t launch_debug_philox(uint32_t key0, uint32_t key1, unsigned long long n_iter,
                               uint32_t k0, uint32_t nk, uint32_t j0, uint32_t nj,
                               uint32_t* out, hipStream_t stream)
{
    const uint64_t n = (uint64_t)nk * nj;
    hipLaunchKernelGGL(k_debug_philox, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream,
                       key0, key1, n_iter, k0, nk, j0, nj, out);
    return hipGetLastError();
}

}  // namespace mppi_impl
