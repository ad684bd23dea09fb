// Host runtime behind the C ABI of include/mppi.h: handle life cycle,
// validation, ego-frame staging of the scene, single and batched launches
// (batches replayed as HIP graphs), result export, checkpointing, the
// launch-shape tuning table and profiling.
#include <hip/hip_runtime.h>
#include <dlfcn.h>
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "mppi_host.hpp"

using namespace mppi_impl;

namespace mppi_impl {

thread_local std::string g_last_error;

mppi_status fail(mppi_status s, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return s;
}

size_t pow2_at_least(size_t v, size_t lo)
{
    size_t p = lo;
    while (p < v) p <<= 1;
    return p;
}

static size_t scene_bytes(int n_wp, int n_c) { return scene_layout(n_wp, n_c).bytes; }

// ---- validation ---------------------------------------------------------------

mppi_status validate_scene(const mppi_config& c, const double x0[4], const mppi_scene* sc)
{
    if (!x0 || !sc) return fail(MPPI_E_INVALID, "x0 and scene must not be NULL");
    for (int i = 0; i < 4; ++i)
        if (!isfinite(x0[i])) return fail(MPPI_E_INVALID, "x0[%d] is not finite", i);
    const int n_wp = sc->n_waypoints, n_c = sc->n_circles;
    if (n_wp < 1 || n_wp > c.max_waypoints || !sc->waypoints)
        return fail(MPPI_E_INVALID, "n_waypoints=%d outside [1, %d] or waypoints NULL", n_wp,
                    c.max_waypoints);
    if (n_c < 0 || n_c > c.max_circles || (n_c > 0 && !sc->circles))
        return fail(MPPI_E_INVALID, "n_circles=%d outside [0, %d] or circles NULL", n_c,
                    c.max_circles);
    for (int i = 0; i < 4 * n_wp; ++i)
        if (!isfinite(sc->waypoints[i])) return fail(MPPI_E_INVALID, "waypoint value not finite");
    for (int i = 0; i < 5 * n_c; ++i)
        if (!isfinite(sc->circles[i])) return fail(MPPI_E_INVALID, "circle value not finite");
    return MPPI_OK;
}

mppi_status validate_config(const mppi_config* c)
{
    if (!c) return fail(MPPI_E_INVALID, "config is NULL");
    if (c->K < 1 || c->K > kMaxK) return fail(MPPI_E_INVALID, "K=%d outside [1, %d]", c->K, kMaxK);
    if (c->T < 1 || c->T > kMaxT) return fail(MPPI_E_INVALID, "T=%d outside [1, %d]", c->T, kMaxT);
    if (!(c->dt > 0) || !isfinite(c->dt)) return fail(MPPI_E_INVALID, "dt must be finite and > 0");
    if (!(c->wheelbase > 0) || !isfinite(c->wheelbase))
        return fail(MPPI_E_INVALID, "wheelbase must be finite and > 0");
    if (!(c->lambda > 0) || !isfinite(c->lambda))
        return fail(MPPI_E_INVALID, "lambda must be finite and > 0");
    if (!(c->gamma > 0) || !isfinite(c->gamma)) return fail(MPPI_E_INVALID, "gamma must be > 0");
    for (int i = 0; i < 2; ++i) {
        if (!(c->sigma[i] >= 0) || !isfinite(c->sigma[i]))
            return fail(MPPI_E_INVALID, "sigma[%d] must be finite and >= 0", i);
        if (isnan(c->u_min[i]) || isnan(c->u_max[i]) || !(c->u_min[i] <= c->u_max[i]))
            return fail(MPPI_E_INVALID, "u_min[%d] <= u_max[%d] required", i, i);
        if (c->u_min[i] == INFINITY || c->u_max[i] == -INFINITY)
            return fail(MPPI_E_INVALID, "bounds %d exclude every control", i);
    }
    if (isnan(c->v_max)) return fail(MPPI_E_INVALID, "v_max is NaN");
    const double ws[6] = {c->w_track, c->w_speed, c->w_effort, c->w_coll, c->d_safe_c, c->d_safe_0};
    for (double w : ws)
        if (!isfinite(w)) return fail(MPPI_E_INVALID, "cost weights must be finite");
    if (c->n_ego < 0 || c->n_ego > kMaxEgo)
        return fail(MPPI_E_INVALID, "n_ego=%d outside [0, %d]", c->n_ego, kMaxEgo);
    if (!isfinite(c->ego_r)) return fail(MPPI_E_INVALID, "ego_r must be finite");
    for (int e = 0; e < c->n_ego; ++e)
        if (!isfinite(c->ego_off[e])) return fail(MPPI_E_INVALID, "ego_off must be finite");
    if (c->max_waypoints < 1 || c->max_waypoints > kMaxWaypoints)
        return fail(MPPI_E_INVALID, "max_waypoints=%d outside [1, %d]", c->max_waypoints,
                    kMaxWaypoints);
    if (c->max_circles < 0 || c->max_circles > kMaxCircles)
        return fail(MPPI_E_INVALID, "max_circles=%d outside [0, %d]", c->max_circles,
                    kMaxCircles);
    if (c->smoothing != 0 && c->smoothing != 1)
        return fail(MPPI_E_INVALID, "smoothing must be 0 or 1");
    if (!isfinite(c->w_target) || !isfinite(c->w_yaw))
        return fail(MPPI_E_INVALID, "w_target and w_yaw must be finite");
    if (c->collision_only != 0 && c->collision_only != 1)
        return fail(MPPI_E_INVALID, "collision_only must be 0 or 1");
    if (c->model != 0 && c->model != 1) return fail(MPPI_E_INVALID, "model must be 0 or 1");
    if (c->per_step_weights != 0 && c->per_step_weights != 1)
        return fail(MPPI_E_INVALID, "per_step_weights must be 0 or 1");
    return MPPI_OK;
}

mppi_status usable(mppi_t* h)
{
    if (!h) return fail(MPPI_E_INVALID, "handle is NULL");
    if (h->sticky != MPPI_OK)
        return fail(h->sticky, "handle is unusable after an earlier device failure");
    return MPPI_OK;
}

// ---- scene staging ------------------------------------------------------------

SceneLayout scene_layout(int n_wp, int n_c)
{
    SceneLayout L;
    L.o_pv = 0;
    L.o_xy = L.o_pv + align_up((size_t)n_c * 16, 16);
    // waypoints padded to whole chunks (points at infinity)
    L.o_vr = L.o_xy + align_up((size_t)(n_wp + kChunk - 1) / kChunk * kChunk * 8, 16);
    L.o_yw = L.o_vr + align_up((size_t)n_wp * 4, 16);
    L.o_rr = L.o_yw + align_up((size_t)n_wp * 4, 16);
    L.o_reach = L.o_rr + align_up((size_t)n_c * 4, 16);
    L.o_grp = L.o_reach + align_up((size_t)n_c * 4, 16);
    // bounding box of every chunk, then the scene's flags
    L.o_box = L.o_grp + (size_t)circle_groups(n_c) * 48;
    L.o_flags = L.o_box + (size_t)(n_wp + kChunk - 1) / kChunk * 16;
    L.bytes = L.o_flags + 16;
    return L;
}

// Vectors of the host's, compared and selected lane by lane.
typedef float hf4 __attribute__((vector_size(16)));
typedef int hi4 __attribute__((vector_size(16)));
typedef double hd2 __attribute__((vector_size(16)));
static inline hf4 vmin(hf4 a, hf4 b) { return b < a ? b : a; }
static inline hf4 vmax(hf4 a, hf4 b) { return a < b ? b : a; }
static inline hf4 to_floats(const double* p, hd2 less)
{
    typedef float f2 __attribute__((vector_size(8)));
    hd2 a, b;
    memcpy(&a, p, sizeof a);
    memcpy(&b, p + 2, sizeof b);
    return __builtin_shufflevector(__builtin_convertvector(a - less, f2), __builtin_convertvector(b, f2), 0, 1, 2, 3);
}

// Ego-frame float32 copy of the scene (float64 subtraction of the origin).
// Host time bounds the staging of small instances, so vectors of the host's are
// used: 221 waypoints and 60 circles take 0.6 us (in scalars 1.3), 221 and 200 1.7
// (3.1), 301 and 512 4.2 (6.6), 2048 without circles 4.4 (10.9).
void write_scene(unsigned char* dst, const SceneLayout& L, const mppi_config& c,
                 const double origin[2], const mppi_scene* sc)
{
    float2* xy = reinterpret_cast<float2*>(dst + L.o_xy);
    float* vr = reinterpret_cast<float*>(dst + L.o_vr);
    float* yw = reinterpret_cast<float*>(dst + L.o_yw);
    float* rr = reinterpret_cast<float*>(dst + L.o_rr);
    const hd2 org = {origin[0], origin[1]};
    const hf4 top = {INFINITY, INFINITY, INFINITY, INFINITY};
    // By chunks: (x_lo, x_hi, y_lo, y_hi) of each chunk's float32 positions, for
    // the culling; whether one reference speed is that of every waypoint; and the
    // waypoint nearest to the origin.
    float4* box = reinterpret_cast<float4*>(dst + L.o_box);
    const int n_wp = sc->n_waypoints;
    const float vr0 = (float)sc->waypoints[3];
    bool uniform = true;
    int j0 = 0;
    float near2 = INFINITY;
    for (int c0 = 0; c0 < n_wp; c0 += kChunk) {
        hf4 lo = top, hi = -top;  // of (x, y, yaw, reference speed)
        float d2[kChunk], least = INFINITY;
        const int n = std::min(kChunk, n_wp - c0);
        for (int u = 0; u < n; ++u) {
            const int j = c0 + u;
            const hf4 w = to_floats(sc->waypoints + 4 * j, org);
            xy[j] = make_float2(w[0], w[1]);
            yw[j] = w[2];
            vr[j] = w[3];
            lo = vmin(lo, w);
            hi = vmax(hi, w);
            d2[u] = w[0] * w[0] + w[1] * w[1];
            least = std::min(least, d2[u]);
        }
        for (int j = c0 + n; j % kChunk; ++j) xy[j] = make_float2(INFINITY, INFINITY);
        box[c0 / kChunk] = make_float4(lo[0], hi[0], lo[1], hi[1]);
        uniform = uniform && lo[3] == vr0 && hi[3] == vr0;
        if (least < near2) {
            near2 = least;
            for (int u = n - 1; u >= 0; --u)
                if (d2[u] == least) j0 = c0 + u;
        }
    }
    // flag 0: one reference speed; then the waypoint nearest to the origin and the
    // inverse of the mean spacing of those that follow it: where the scan by rows
    // starts looking
    int* flags = reinterpret_cast<int*>(dst + L.o_flags);
    const int ja = std::max(std::min(j0, n_wp - 1 - kChunk), 0);
    const int jb = std::min(ja + kChunk, n_wp - 1);
    const float len = hypotf(xy[jb].x - xy[ja].x, xy[jb].y - xy[ja].y);
    const float inv_sp = len > 1e-6f ? (float)(jb - ja) / len : 0.0f;
    flags[0] = uniform;
    flags[1] = j0;
    memcpy(&flags[2], &inv_sp, sizeof inv_sp);
    flags[3] = 0;
    // The circles as given, or -- the order is free, a clearance is a minimum --
    // along the longer axis of their positions, the moving ones last, by a
    // counting sort.
    const int n_c = sc->n_circles;
    hf4* pv = reinterpret_cast<hf4*>(dst + L.o_pv);
    float* reach = reinterpret_cast<float*>(dst + L.o_reach);
    const int n_grp = circle_groups(n_c);
    auto circle = [&](int i) {  // (x, y, vx, vy) of the i-th given
        const double* o = sc->circles + 5 * i;
        const double q[4] = {o[0], o[1], o[3], o[4]};
        return to_floats(q, org);
    };
    auto radius = [&](int i) { return (float)(sc->circles[5 * i + 2] + c.ego_r); };
    const float dt = (float)c.dt;
    if (!n_grp) {
        for (int i = 0; i < n_c; ++i) {
            pv[i] = circle(i);
            rr[i] = radius(i);
            reach[i] = circle_reach(rr[i], pv[i][2], pv[i][3], dt);
        }
        return;
    }
    constexpr int kBuckets = 128;
    hf4 given[kMaxCircles];
    hf4 lo = top, hi = -top;
    for (int i = 0; i < n_c; ++i) {
        given[i] = circle(i);
        lo = vmin(lo, given[i]);
        hi = vmax(hi, given[i]);
    }
    const int axis = hi[0] - lo[0] >= hi[1] - lo[1] ? 0 : 1;
    const float first = lo[axis], scale = (kBuckets - 1.0f) / std::max(hi[axis] - lo[axis], 1e-9f);
    // four at a time: reach and bucket (beyond float32 the product is no number:
    // the first bucket)
    int at[2 * kBuckets + 1] = {};
    hf4 r4[kMaxCircles / 4], reach4[kMaxCircles / 4];
    hi4 bucket4[kMaxCircles / 4];
    const int* bucket = reinterpret_cast<const int*>(bucket4);
    for (int i = 0; i < n_c; i += 4) {
        hf4 q[4], r;
        for (int u = 0; u < 4; ++u) {
            q[u] = given[std::min(i + u, n_c - 1)];
            r[u] = radius(std::min(i + u, n_c - 1));
        }
        const hf4 xa = __builtin_shufflevector(q[0], q[1], 0, 4, 1, 5), xb = __builtin_shufflevector(q[2], q[3], 0, 4, 1, 5);
        const hf4 va = __builtin_shufflevector(q[0], q[1], 2, 6, 3, 7), vb = __builtin_shufflevector(q[2], q[3], 2, 6, 3, 7);
        const hf4 x = axis ? __builtin_shufflevector(xa, xb, 2, 3, 6, 7) : __builtin_shufflevector(xa, xb, 0, 1, 4, 5);
        const hf4 vx = __builtin_shufflevector(va, vb, 0, 1, 4, 5), vy = __builtin_shufflevector(va, vb, 2, 3, 6, 7);
        const hf4 zero = {}, k = vmin((x - first) * scale, zero + (kBuckets - 1.0f));
        r4[i / 4] = r;
        reach4[i / 4] = circle_margin(r, vmax(r, zero)) + circle_travel(__builtin_elementwise_sqrt(vx * vx + vy * vy), dt);
        bucket4[i / 4] = __builtin_convertvector(k > zero ? k : zero, hi4) +
                         (((vx != zero) | (vy != zero)) & kBuckets);
        for (int u = 0; u < 4 && i + u < n_c; ++u) ++at[bucket[i + u] + 1];
    }
    for (int b = 0; b < 2 * kBuckets; ++b) at[b + 1] += at[b];
    for (int i = 0; i < n_c; ++i) {
        const int to = at[bucket[i]]++;
        pv[to] = given[i];
        rr[to] = reinterpret_cast<const float*>(r4)[i];
        reach[to] = reinterpret_cast<const float*>(reach4)[i];
    }
    float4* grp = reinterpret_cast<float4*>(dst + L.o_grp);
    for (int g = 0; g < n_grp; ++g) {
        const int i0 = g * kCircleGroup, i1 = std::min(i0 + kCircleGroup, n_c);
        hf4 glo = top, ghi = -top;
        float most = -INFINITY;
        for (int i = i0; i < i1; i += 4) {
            const int e = i1 - 1;
            const hf4 q[4] = {pv[i], pv[std::min(i + 1, e)], pv[std::min(i + 2, e)], pv[std::min(i + 3, e)]};
            glo = vmin(glo, vmin(vmin(q[0], q[1]), vmin(q[2], q[3])));
            ghi = vmax(ghi, vmax(vmax(q[0], q[1]), vmax(q[2], q[3])));
        }
        for (int i = i0; i < i1; ++i) most = std::max(most, reach[i]);
        float4 p = make_float4(glo[0], ghi[0], glo[1], ghi[1]), v = make_float4(glo[2], ghi[2], glo[3], ghi[3]);
        bool finite = true;
        for (int a = 0; a < 4; ++a) finite = finite && isfinite(glo[a]) && isfinite(ghi[a]);
        if (!finite) {  // beyond float32: a group that is near everything
            p = make_float4(-1e30f, 1e30f, -1e30f, 1e30f);
            v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            most = INFINITY;
        }
        grp[3 * g] = p;
        grp[3 * g + 1] = v;
        grp[3 * g + 2] = make_float4(most, 0.0f, 0.0f, 0.0f);
    }
}

// ---- launch-shape tuning table ------------------------------------------------
// Lines "k_log2 t_bucket c_bucket lanes" written by the autotuner
// (paper_2308_01654_amd/autotune.py) into tuning.txt next to the library, or
// the file named by MPPI_TUNING_FILE.  A shape's lanes per sample depends only
// on its own (K, T, circle count).

struct TuneEntry {
    int k, t, c, lanes;
    int stage;  // 1: the tiles may keep their perturbations in LDS; 0: read back from L2
    int occ;    // 1: the high-occupancy compilation of the iteration kernel
};
static std::vector<TuneEntry> g_tune;
static std::once_flag g_tune_once;

static int k_bucket(int K)
{
    int b = 0;
    while ((1 << b) < K && b < 30) ++b;
    return b;
}
static int t_bucket(int T)
{
    return T <= 16 ? 0 : T <= 32 ? 1 : T <= 64 ? 2 : T <= 128 ? 3 : T <= 256 ? 4 : 5;
}
static int c_bucket(int n) { return n == 0 ? 0 : n <= 16 ? 1 : n <= 64 ? 2 : n <= 256 ? 3 : 4; }

static void load_tuning()
{
    std::string path;
    if (const char* e = getenv("MPPI_TUNING_FILE")) {
        path = e;
    } else {
        Dl_info info;
        if (dladdr((void*)&load_tuning, &info) && info.dli_fname) {
            path = info.dli_fname;
            const size_t slash = path.rfind('/');
            path = (slash == std::string::npos ? std::string(".") : path.substr(0, slash)) +
                   "/tuning.txt";
        }
    }
    FILE* f = path.empty() ? nullptr : fopen(path.c_str(), "r");
    if (!f) return;
    char line[256];
    while (fgets(line, sizeof line, f)) {
        if (line[0] == '#') continue;
        TuneEntry t;
        t.stage = 1;  // the optional fifth and sixth columns
        t.occ = 0;
        const int n = sscanf(line, "%d %d %d %d %d %d", &t.k, &t.t, &t.c, &t.lanes, &t.stage,
                             &t.occ);
        if (n >= 4 && (t.stage == 0 || t.stage == 1) && t.occ >= 0 && t.occ <= kOccHigh &&
            (t.lanes == 1 || t.lanes == 2 || t.lanes == 4 || t.lanes == 8 || t.lanes == 16))
            g_tune.push_back(t);
    }
    fclose(f);
}

static int heuristic_lanes(const mppi_config& c)
{
    // Enough lanes to give every SIMD of the 256 CUs two waves.
    const long target = 2L * 256 * 4 * 64;
    int g = 1;
    while (g < 16 && (long)g * c.K < target) g <<= 1;
    return g;
}

int auto_lanes(const mppi_config& c, int n_c)
{
    std::call_once(g_tune_once, load_tuning);
    const int kb = k_bucket(c.K), tb = t_bucket(c.T), cb = c_bucket(n_c);
    const TuneEntry* best = nullptr;
    for (const TuneEntry& e : g_tune)
        if (e.t == tb && e.c == cb && (!best || abs(e.k - kb) < abs(best->k - kb))) best = &e;
    int g = best ? best->lanes : heuristic_lanes(c);
    while (g > 1 && g > c.T) g >>= 1;
    return g;
}

static const TuneEntry* tune_entry(const mppi_config& c, int n_c)
{
    std::call_once(g_tune_once, load_tuning);
    const int kb = k_bucket(c.K), tb = t_bucket(c.T), cb = c_bucket(n_c);
    const TuneEntry* best = nullptr;
    for (const TuneEntry& e : g_tune)
        if (e.t == tb && e.c == cb && (!best || abs(e.k - kb) < abs(best->k - kb))) best = &e;
    return best;
}

// The tuning table's staging choice for the bucket auto_lanes uses (1 when
// the table has no such column or no bucket).
int auto_stage(const mppi_config& c, int n_c)
{
    const TuneEntry* e = tune_entry(c, n_c);
    return e ? e->stage : 1;
}

int auto_occ(const mppi_config& c, int n_c)
{
    const TuneEntry* e = tune_entry(c, n_c);
    return e ? e->occ : 0;
}

// Where the split kernel beats k_batch.  It hides the latency of a chain behind
// other waves, and it culls by rows, which pays once the samples have drifted
// apart; it needs more waves for a sample, and its waves wait for one another.  So
// it wins wherever the launch has at most two tiles for each of the 256 compute
// units (us, k_batch -> split: 16 lanes, 1024 x 50, 3 circles 18.1 -> 12.3; 8192 x
// 100, 60 circles 34.8 -> 23.2; 8 lanes, 16384 x 24, 12 circles 17.0 -> 15.3; 4
// lanes, 32768 x 64, 60 circles 46 -> 35; a batch of 4 of 2048 x 16, 16 lanes: 1.06
// times), and in larger launches from a horizon on:
//  * 16 lanes, alone: always (16384 x 33: 1.1 to 1.2 times, 32768 x 150 1.2 to 1.6).
//    In a batch (the descriptors come from memory) from 48 steps (2048 tiles: 32
//    steps 0.96 to 0.99 times, 48 steps 1.03 to 1.08, 100 steps 1.06 to 1.16), with
//    per-step weights from 64 (24 steps 0.90, 48 steps 0.97 to 0.99, 100 steps 1.17
//    to 1.3); without circles always;
//  * 8 lanes, alone: from 32 steps with circles that are all listed (1024 tiles: 24
//    steps 0.93, 32 steps 1.05 to 1.07, 64 steps 1.15 to 1.18), else from 80 (200 and
//    512 circles: 50 steps 0.85 to 0.9, 64 steps 0.94 to 1.04, 80 steps 1.0 to 1.13;
//    none: 50 steps 0.9 to 1.06, 80 steps 1.04 to 1.1).  In a batch from 128 steps
//    (2048 tiles: 80 steps 0.94 to 1.09, 128 steps 1.1 to 1.35), with listed circles
//    from 100 (1.02 to 1.14);
//  * 4 lanes, alone: with listed circles while its tiles keep their perturbations
//    (131072 x 64: 1.05 to 1.07; x 80 0.92 to 0.94), else from 128 steps (1.03 to 1.3).
//    In a batch from 150 (2048 tiles: 128 steps 0.96 to 1.17, 150 steps 1.04 to 1.3).
// Paths of more than 64 chunks, whose boxes a wave then reads 16 at a time for
// every row, take what the circles' groups do not win back.  In launches of few
// tiles it pays up to 1536 waypoints at 16 lanes (8192 x 50: 1000 waypoints 1.01 to
// 1.17 times, 2048 0.9 to 1.04; x 100: 1500 1.3), below them up to 640 (16384 x 50 at
// 8: 520 waypoints 0.98 to 1.13, 1000 0.86 to 1.03), from 100 steps 1024 (1000: 0.96 to
// 1.3), with grouped circles always (1.05 to 1.3).  In larger ones with grouped
// circles up to 1024 (8 lanes, 65536 x 100: 1000 waypoints 1.01 to 1.13, 2048 0.9), from
// 100 steps 1536 (with 512 circles 1500: 1.25), from 150 always (x 200, 2048: 1.3 to
// 1.5); with listed ones from 200 steps up to 640 (1.06 to 1.3; 100 steps 0.8 to 1.1).
// Below 64 steps at 4 lanes, without circles there, with per-step weights below 16
// lanes and at 2 lanes it is not used (131072 x 32 at 2: 86 -> 112).
static bool split_pays(const mppi_config& c, int n_wp, int n_c, int lanes, bool staged, int tiles, bool alone)
{
    if (lanes < 4 || (lanes < 16 && c.per_step_weights)) return false;
    if (lanes == 4 && (c.T < 64 || n_c == 0)) return false;
    const bool few = tiles <= 2 * 256, listed = n_c <= kListedCircles;
    if (n_wp > 64 * kChunk) {
        const int most =
            few ? (!listed ? kMaxWaypoints : lanes == 16 ? 1536 : c.T >= 100 ? 1024 : 640)
                : (!listed ? (c.T >= 150 ? kMaxWaypoints : c.T >= 100 ? 1536 : 1024)
                           : (n_c > 0 && c.T >= 200 ? 640 : 0));
        if (n_wp > most) return false;
    }
    if (few) return true;
    switch (lanes) {
    case 16: return alone || n_c == 0 || c.T >= (c.per_step_weights ? 64 : 48);
    case 8: return c.T >= (alone ? (listed && n_c > 0 ? 32 : 80) : (listed && n_c > 0 ? 100 : 128));
    default: return c.T >= (alone ? 128 : 150) || (alone && listed && staged);
    }
}

// The compilation of k_batch; the second exists for 8 and 16 lanes per sample.
static int k_batch_occ(const mppi_t* h, int n_c, int lanes)
{
    if (lanes < 8) return kOccDefault;
    return h->occ_req >= 0 ? h->occ_req : auto_occ(h->cfg, n_c);
}

int occ_choice(const mppi_t* h, int n_wp, int n_c, int lanes, int batch_tiles)
{
    const mppi_config& c = h->cfg;
    const bool alone = batch_tiles == 0;
    const int tiles = alone ? (int)(((long)c.K * lanes + kBlock - 1) / kBlock) : batch_tiles;
    if (!h->no_cull && h->occ_req < 0 && lanes >= 4) {
        const SplitLayout L = split_layout(c.T, n_wp, lanes, c.per_step_weights);
        const bool one_each = alone && tiles <= 256;  // at most a tile per compute unit
        if ((L.total <= kSplitLds || (one_each && L.total <= kSplitLdsAlone)) &&
            split_pays(c, n_wp, n_c, lanes, L.staged, tiles, alone))
            return kOccSplit;
    }
    return k_batch_occ(h, n_c, lanes);
}

// Whether the split kernel could run an instance of a batch at 16 lanes per
// sample, where it exists for every configuration.
static bool split_could(const mppi_t* h, int n_wp, int lanes)
{
    return lanes == 16 && !h->no_cull && h->occ_req < 0 &&
           split_layout(h->cfg.T, n_wp, 16, h->cfg.per_step_weights).total <= kSplitLds;
}

// ---- profiling --------------------------------------------------------------------

// Events come from the handle's pool (created on first use) so that
// profiling adds little host time between launches.
static hipError_t pool_event(mppi_t* h, hipEvent_t* e)
{
    if (!h->event_pool.empty()) {
        *e = h->event_pool.back();
        h->event_pool.pop_back();
        return hipSuccess;
    }
    return hipEventCreate(e);
}

mppi_status record_launch(mppi_t* h, int kind, hipEvent_t* a)
{
    (void)kind;
    if (!h || !h->prof) return MPPI_OK;
    HIP_TRY(pool_event(h, a));
    HIP_TRY(hipEventRecord(*a, h->stream));
    return MPPI_OK;
}

mppi_status record_end(mppi_t* h, int kind, hipEvent_t a)
{
    if (!h || !h->prof) return MPPI_OK;
    hipEvent_t b;
    HIP_TRY(pool_event(h, &b));
    HIP_TRY(hipEventRecord(b, h->stream));
    h->events.push_back(ProfEvent{a, b, kind});
    return MPPI_OK;
}

static mppi_status drain_profile(mppi_t* h)
{
    if (h->events.empty()) return MPPI_OK;
    HIP_TRY(hipStreamSynchronize(h->stream));
    for (const ProfEvent& e : h->events) {
        float ms = 0.f;
        HIP_TRY(hipEventElapsedTime(&ms, e.a, e.b));
        h->prof_ms[e.kind] += ms;
        h->prof_n[e.kind] += 1;
        h->event_pool.push_back(e.a);
        h->event_pool.push_back(e.b);
    }
    h->events.clear();
    return MPPI_OK;
}

// Work is about to be enqueued for one handle.
static void mail_behind(mppi_t* h)
{
    if (h->mail_behind) h->mail_behind->store(true, std::memory_order_relaxed);
}

template <typename F>
static mppi_status launch_aux(mppi_t* h, F&& f)
{
    mail_behind(h);
    hipEvent_t a = nullptr;
    mppi_status s = record_launch(h, 1, &a);
    if (s != MPPI_OK) return s;
    HIP_TRY(f());
    return record_end(h, 1, a);
}

// The pinned, coherent host buffers the device writes results into (U and
// the state; the optimal trajectory), made by the first read or the first batch
// that leaves results there: handles that are never read and step alone or in
// small batches, and a server's vehicles, hold no pinned pages.
static mppi_status host_buffers(mppi_t* h)
{
    if (h->ctl_host) return MPPI_OK;
    const size_t T = (size_t)h->cfg.T;
    hipError_t e;
    if ((e = hipHostMalloc((void**)&h->traj, sizeof(double) * (5 * (T + 1) + 2 * T),
                           hipHostMallocCoherent)) != hipSuccess ||
        (e = hipHostGetDevicePointer((void**)&h->traj_dev, h->traj, 0)) != hipSuccess ||
        (e = hipHostMalloc((void**)&h->ctl_host, done_offset(T) + 64, hipHostMallocCoherent)) !=
            hipSuccess ||
        (e = hipHostGetDevicePointer((void**)&h->ctl_dev, h->ctl_host, 0)) != hipSuccess) {
        if (h->traj) (void)hipHostFree(h->traj);
        if (h->ctl_host) (void)hipHostFree(h->ctl_host);
        h->traj = h->traj_dev = h->ctl_host = h->ctl_dev = nullptr;
        return fail(MPPI_E_NOMEM, "hipHostMalloc: %s", hipGetErrorString(e));
    }
    h->done = reinterpret_cast<volatile uint32_t*>(reinterpret_cast<unsigned char*>(h->ctl_host) + done_offset(T));
    h->done_dev = reinterpret_cast<unsigned*>(reinterpret_cast<unsigned char*>(h->ctl_dev) + done_offset(T));
    *h->done = h->seq;
    return MPPI_OK;
}

// Whether the device has set *flag, a word of pinned host memory, to seq or a
// later number, looking at it for at most kSpinUs.
constexpr int kSpinUs = 300;
static bool word_set(const volatile uint32_t* flag, uint32_t seq)
{
    return (int32_t)(__atomic_load_n(flag, __ATOMIC_ACQUIRE) - seq) >= 0;
}
static bool spin_word(const volatile uint32_t* flag, uint32_t seq)
{
    const auto t0 = std::chrono::steady_clock::now();
    for (unsigned i = 1; !word_set(flag, seq); ++i) {
        __builtin_ia32_pause();
        if (i % 64 == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::microseconds(kSpinUs))
            return word_set(flag, seq);
    }
    return true;
}

// Waits until the device has set *flag to seq at the end of a kernel of h's
// stream, by which time everything enqueued before it is done as well.  The
// word is there 4 us before a synchronisation of the stream would return (11.7
// -> 7.7 us for an export from an idle stream); after kSpinUs, or where the word
// never comes -- a device failure, a stream under capture -- the stream is
// synchronised, which reports it.
static mppi_status wait_done(mppi_t* h, const volatile uint32_t* flag, uint32_t seq)
{
    if (!spin_word(flag, seq)) HIP_TRY(hipStreamSynchronize(h->stream));
    return MPPI_OK;
}

// The word behind a staging buffer that holds the number of its last upload
// whose data the device has read.
static volatile uint32_t* staged_word(mppi_t* h, int i)
{
    return reinterpret_cast<volatile uint32_t*>(h->staging[i] + align_up(h->scene_cap, 64));
}

// The capture that h's stream is in (its number and one), or 0.
static unsigned long long capture_of(mppi_t* h)
{
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    if (hipStreamGetCaptureInfo(h->stream, &c, &id) != hipSuccess) (void)hipGetLastError();
    return c == hipStreamCaptureStatusActive ? id + 1 : 0;
}

// Waits until the device has read the last upload from staging buffer b.  Only
// that upload is waited for, not what other handles or the caller have put on
// the stream behind it.  (Replans of 131072 x 100, 60 circles, enqueued without a
// read between them take the same time as with the stream synchronised after the
// spin, 324 and 325 us a step.)  The stream is asked now and then whether it has
// failed, but not while it is being captured, which the question would end.
static mppi_status wait_staged(mppi_t* h, int b, bool capturing)
{
    const volatile uint32_t* word = staged_word(h, b);
    const uint32_t seq = h->staged_seq[b];
    if (spin_word(word, seq)) return MPPI_OK;
    constexpr int kAsk = 1000;  // sleeps, of 75 us with the timer's slack
    for (int i = 1; !word_set(word, seq); ++i) {
        std::this_thread::sleep_for(std::chrono::microseconds(20));
        if (capturing || i % kAsk) continue;
        const hipError_t e = hipStreamQuery(h->stream);
        if (e == hipSuccess) break;  // everything enqueued is done, the upload too
        if (e != hipErrorNotReady) HIP_TRY(e);
        (void)hipGetLastError();
    }
    return MPPI_OK;
}

// Work that changes U is about to be enqueued.  Under capture it runs when the
// caller launches the graph, which the handle does not see: from then on no
// batch leaves the handle's results in the host's memory.
static void changes_results(mppi_t* h)
{
    h->mail = 0;
    mail_behind(h);
    if (h->captured) return;
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(h->stream, &c) != hipSuccess) (void)hipGetLastError();
    else if (c == hipStreamCaptureStatusNone) return;
    h->captured = true;
}

// Whether the batch that set U and the device state leaves them in the handle's
// pinned buffer, with no work of its handles enqueued since.
static bool mailed(const mppi_t* h)
{
    return h->mail && !h->mail_behind->load(std::memory_order_relaxed);
}

// U's first nu values and the device state into that buffer, by one small kernel
// that then sets the handle's word to h->seq.
static mppi_status enqueue_export(mppi_t* h, int nu)
{
    const mppi_status s = host_buffers(h);
    if (s != MPPI_OK) return s;
    mail_behind(h);
    ++h->seq;
    HIP_TRY(launch_export_controls(h->U, nu, h->st, h->ctl_dev,
                                   reinterpret_cast<DevState*>(h->ctl_dev + 2 * h->cfg.T), h->done_dev,
                                   h->seq, h->stream));
    return MPPI_OK;
}

// U's first nu values and the device state in the handle's pinned buffer, after
// everything enqueued so far.
static mppi_status export_results(mppi_t* h, int nu)
{
    // What the caller has enqueued on the stream since the batch is waited for as
    // well.  Asking the stream costs 0.1 us while it is idle and 20 us while a
    // kernel retires, so behind other work of the batch's handles, which they
    // know of, an export is the faster way (64 handles, controls and trajectory
    // of each in turn: 38.4 us a handle with the question, 25.9 this way).
    if (mailed(h)) {
        const mppi_status s = wait_done(h, h->done, h->mail);
        if (s != MPPI_OK) return s;
        if (hipStreamQuery(h->stream) != hipSuccess) {
            (void)hipGetLastError();
            HIP_TRY(hipStreamSynchronize(h->stream));
        }
        return MPPI_OK;
    }
    const mppi_status s = enqueue_export(h, nu);
    return s == MPPI_OK ? wait_done(h, h->done, h->seq) : s;
}

// The device state after everything enqueued so far: written by one small
// kernel into the pinned host buffer.
static mppi_status read_state(mppi_t* h, DevState* out)
{
    const mppi_status s = export_results(h, 0);
    if (s != MPPI_OK) return s;
    *out = *reinterpret_cast<const DevState*>(h->ctl_host + 2 * h->cfg.T);
    return MPPI_OK;
}

static mppi_status sync_status(mppi_t* h)
{
    if (!h->stepped) {
        HIP_TRY(hipStreamSynchronize(h->stream));
        return MPPI_OK;
    }
    // The stream is synchronised at once: waiting for the word first and for the
    // stream after it takes 14.8 us where this takes 11.6.
    const mppi_status s = mailed(h) ? MPPI_OK : enqueue_export(h, 0);
    if (s != MPPI_OK) return s;
    HIP_TRY(hipStreamSynchronize(h->stream));
    if (reinterpret_cast<const DevState*>(h->ctl_host + 2 * h->cfg.T)->status != 0)
        return fail(MPPI_E_NONFINITE, "every sample cost of the last step was non-finite");
    return MPPI_OK;
}

// ---- handles ----------------------------------------------------------------------

void handle_release(mppi_t* h)
{
    if (h->stream) (void)hipStreamSynchronize(h->stream);
    for (const ProfEvent& e : h->events) {
        (void)hipEventDestroy(e.a);
        (void)hipEventDestroy(e.b);
    }
    for (hipEvent_t e : h->event_pool) (void)hipEventDestroy(e);
    (void)hipFree(h->U);
    (void)hipFree(h->S);
    (void)hipFree(h->eps);
    (void)hipFree(h->partials);
    (void)hipFree(h->q);
    (void)hipFree(h->Stk);
    (void)hipFree(h->wbuf);
    if (h->traj) (void)hipHostFree(h->traj);
    if (h->ctl_host) (void)hipHostFree(h->ctl_host);
    (void)hipFree(h->st);
    (void)hipFree(h->scene);
    if (h->batch) {
        ws_destroy(h->batch);
        h->batch = nullptr;
    }
    for (int i = 0; i < 2; ++i) {
        if (h->staging[i]) (void)hipHostFree(h->staging[i]);
    }
    if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
}

mppi_status handle_create(const mppi_config* cfg, void* hip_stream, bool with_scratch,
                          mppi_t** out)
{
    if (!out) return fail(MPPI_E_INVALID, "out is NULL");
    *out = nullptr;
    mppi_status s = validate_config(cfg);
    if (s != MPPI_OK) return s;
    mppi_t* h = new (std::nothrow) mppi();
    if (!h) return fail(MPPI_E_NOMEM, "host allocation failed");
    h->cfg = *cfg;
    const int K = cfg->K, T = cfg->T;
    h->max_tiles = (K + (kBlock / 16) - 1) / (kBlock / 16);
    h->scene_cap = scene_bytes(cfg->max_waypoints, cfg->max_circles);
    auto bail = [&](mppi_status st, const char* what, hipError_t e) {
        handle_release(h);
        delete h;
        return fail(st, "%s: %s", what, hipGetErrorString(e));
    };
    hipError_t e;
    if (hip_stream) {
        h->stream = (hipStream_t)hip_stream;
    } else {
        if ((e = hipStreamCreateWithFlags(&h->stream, hipStreamNonBlocking)) != hipSuccess)
            return bail(MPPI_E_DEVICE, "hipStreamCreate", e);
        h->own_stream = true;
    }
    if ((e = hipMalloc((void**)&h->U, sizeof(double) * 2 * T)) != hipSuccess ||
        (e = hipMalloc((void**)&h->st, sizeof(DevState))) != hipSuccess)
        return bail(MPPI_E_NOMEM, "hipMalloc", e);
    if (with_scratch) {
        struct { void** p; size_t n; } allocs[] = {
            {(void**)&h->S, sizeof(float) * K},
            {(void**)&h->eps, sizeof(float2) * (size_t)T * K},
            {(void**)&h->partials,
             sizeof(double) * partial_doubles(T, cfg->per_step_weights, (size_t)h->max_tiles)},
            {(void**)&h->wbuf, sizeof(double) * (size_t)K},
            {(void**)&h->scene, h->scene_cap},
        };
        for (auto& a : allocs)
            if ((e = hipMalloc(a.p, a.n)) != hipSuccess) return bail(MPPI_E_NOMEM, "hipMalloc", e);
        if (cfg->per_step_weights &&
            ((e = hipMalloc((void**)&h->q, sizeof(float) * (size_t)T * K)) != hipSuccess ||
             (e = hipMalloc((void**)&h->Stk, sizeof(double) * (size_t)T * K)) != hipSuccess))
            return bail(MPPI_E_NOMEM, "hipMalloc", e);
        for (int i = 0; i < 2; ++i) {
            // the scene, then the word that the device sets once it has read it
            if ((e = hipHostMalloc((void**)&h->staging[i], align_up(h->scene_cap, 64) + 64,
                                   hipHostMallocCoherent)) != hipSuccess ||
                (e = hipHostGetDevicePointer((void**)&h->staging_dev[i], h->staging[i], 0)) != hipSuccess)
                return bail(MPPI_E_NOMEM, "hipHostMalloc", e);
            *staged_word(h, i) = 0;
        }
        if ((e = hipMemsetAsync(h->S, 0, sizeof(float) * K, h->stream)) != hipSuccess)
            return bail(MPPI_E_DEVICE, "initialise device state", e);
    }
    if ((e = hipMemsetAsync(h->U, 0, sizeof(double) * 2 * T, h->stream)) != hipSuccess ||
        (e = hipMemsetAsync(h->st, 0, sizeof(DevState), h->stream)) != hipSuccess ||
        (e = hipStreamSynchronize(h->stream)) != hipSuccess)
        return bail(MPPI_E_DEVICE, "initialise device state", e);
    if (const char* env = getenv("MPPI_LANES_PER_SAMPLE")) {
        const int g = atoi(env);
        if (g == 1 || g == 2 || g == 4 || g == 8 || g == 16) h->lanes_req = g;
    }
    *out = h;
    return MPPI_OK;
}

// Whether the tiles of d keep their perturbations in LDS (see kLdsShared).
int stage_allowed(const mppi_t* h, int n_c)
{
    return h->stage_req >= 0 ? h->stage_req : auto_stage(h->cfg, n_c);
}

void choose_eps_stage(InstDesc& d, bool alone, int allowed)
{
    const LdsLayout L = lds_layout(d.n_wp, d.n_c, d.T, kBlock / d.lanes, 1, d.per_step, !d.cull);
    d.eps_stage = allowed && L.eps_staged &&
                  (L.total <= kLdsShared || (alone && d.n_tiles <= 512 && L.total <= kLdsAlone));
}

// Descriptor of one iteration of handle h from state x0 on the scene at
// `scene` (device), staged relative to `origin`, launched alone (occ < 0) or in a
// batch with iteration kernel occ.
void fill_desc(InstDesc& d, const mppi_t* h, const double x0[4], const double origin[2],
               const unsigned char* scene, const SceneLayout& L, int n_wp, int n_c, int shift,
               int occ)
{
    const mppi_config& c = h->cfg;
    const bool alone = occ < 0;
    memset(&d, 0, sizeof d);
    d.K = c.K;
    d.T = c.T;
    d.n_wp = n_wp;
    d.n_c = n_c;
    d.lanes = h->lanes_req ? h->lanes_req : auto_lanes(c, n_c);
    d.n_tiles = (c.K + (kBlock / d.lanes) - 1) / (kBlock / d.lanes);
    // two or more waves per SIMD (256 compute units x 4): the block-ordered
    // wave priority pays; with fewer it only costs its instructions
    d.wave_prio = (long)c.K * d.lanes >= 2L * 1024 * 64 ? 1 : 0;
    d.occ = alone ? occ_choice(h, n_wp, n_c, d.lanes, 0) : occ;
    d.dt = (float)c.dt;
    d.inv_dt = (float)(1.0 / c.dt);
    d.inv_L = (float)(1.0 / c.wheelbase);
    d.sig_a = (float)c.sigma[0];
    d.sig_d = (float)c.sigma[1];
    d.a_min = (float)c.u_min[0];
    d.a_max = (float)c.u_max[0];
    d.d_min = (float)c.u_min[1];
    d.d_max = (float)c.u_max[1];
    d.v_max = (float)c.v_max;
    d.w_track = (float)c.w_track;
    d.w_speed = (float)c.w_speed;
    d.w_effort = (float)c.w_effort;
    d.alpha = (float)((c.gamma - 1.0) / (2.0 * c.gamma));
    // (no obstacle term without ego circles or obstacles: a batch may give the
    // instance to a kernel that adds it, and beyond float32 times 0 is no number)
    d.w_coll = active_ego(c.n_ego, n_c) ? (float)c.w_coll : 0.0f;
    d.d_safe_c = (float)c.d_safe_c;
    d.d_safe_0 = (float)c.d_safe_0;
    d.n_ego = c.n_ego;
    for (int e = 0; e < kMaxEgo; ++e) d.ego_off[e] = e < c.n_ego ? (float)c.ego_off[e] : 0.f;
    d.px0 = (float)(x0[0] - origin[0]);
    d.py0 = (float)(x0[1] - origin[1]);
    d.th0 = (float)x0[2];
    d.v0 = (float)x0[3];
    d.lambda = c.lambda;
    d.key0 = (uint32_t)c.seed;
    d.key1 = (uint32_t)(c.seed >> 32);
    d.shift = shift;
    d.cull = h->no_cull ? 0 : 1;
    d.smooth = c.smoothing;
    d.w_target = (float)c.w_target;
    d.w_yaw = (float)c.w_yaw;
    d.coll_only = c.collision_only;
    d.model = c.model;
    d.per_step = c.per_step_weights;
    d.steer0 = (float)h->steer0;
    d.ego_ext = 0.f;
    for (int e = 0; e < c.n_ego; ++e) d.ego_ext = fmaxf(d.ego_ext, (float)fabs(c.ego_off[e]));
    d.out_slot = -1;
    d.c_pv = reinterpret_cast<const float4*>(scene + L.o_pv);
    d.wp_xy = reinterpret_cast<const float2*>(scene + L.o_xy);
    d.wp_vref = reinterpret_cast<const float*>(scene + L.o_vr);
    d.wp_yaw = reinterpret_cast<const float*>(scene + L.o_yw);
    d.wp_box = reinterpret_cast<const float4*>(scene + L.o_box);
    d.scene_flags = reinterpret_cast<const int*>(scene + L.o_flags);
    d.c_rr = reinterpret_cast<const float*>(scene + L.o_rr);
    d.c_reach = reinterpret_cast<const float*>(scene + L.o_reach);
    d.c_grp = reinterpret_cast<const float4*>(scene + L.o_grp);
    d.U = h->U;
    d.S = h->S;
    d.eps = h->eps;
    d.partials = h->partials;
    d.q = h->q;
    d.Stk = h->Stk;
    d.st = h->st;
    choose_eps_stage(d, alone, stage_allowed(h, n_c));
}

// ---- batched launches ---------------------------------------------------------------

static bool graphs_enabled()
{
    static int on = -1;
    if (on < 0) {
        const char* e = getenv("MPPI_BATCH_GRAPH");
        on = (e && e[0] == '0') ? 0 : 1;
    }
    return on == 1;
}

mppi_status ws_create(BatchWs** out)
{
    BatchWs* b = new (std::nothrow) BatchWs();
    if (!b) return fail(MPPI_E_NOMEM, "host allocation failed");
    hipError_t e = hipSuccess;
    for (int i = 0; i < 2 && e == hipSuccess; ++i)
        e = hipEventCreateWithFlags(&b->done[i], hipEventDisableTiming);
    if (e != hipSuccess) {
        delete b;
        return fail(MPPI_E_DEVICE, "batch workspace: %s", hipGetErrorString(e));
    }
    *out = b;
    return MPPI_OK;
}

static void ws_drop_graphs(BatchWs* b)
{
    for (GraphEntry& g : b->graphs) {
        (void)hipGraphExecDestroy(g.exec);
        (void)hipGraphDestroy(g.graph);
    }
    b->graphs.clear();
}

void ws_destroy(BatchWs* b)
{
    if (!b) return;
    for (int i = 0; i < 2; ++i)
        if (b->pending[i]) (void)hipEventSynchronize(b->done[i]);
    ws_drop_graphs(b);
    (void)hipFree(b->arena);
    for (int i = 0; i < 2; ++i) {
        if (b->stage[i]) (void)hipHostFree(b->stage[i]);
        if (b->done[i]) (void)hipEventDestroy(b->done[i]);
    }
    delete b;
}

static hipError_t ws_reserve(BatchWs* b, size_t cap, hipStream_t stream)
{
    if (b->cap >= cap) return hipSuccess;
    hipError_t e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return e;
    ws_drop_graphs(b);
    (void)hipFree(b->arena);
    b->arena = nullptr;
    for (int i = 0; i < 2; ++i) {
        if (b->stage[i]) (void)hipHostFree(b->stage[i]);
        b->stage[i] = nullptr;
        b->pending[i] = false;
    }
    b->cap = 0;
    if ((e = hipMalloc((void**)&b->arena, cap)) != hipSuccess) return e;
    for (int i = 0; i < 2; ++i)
        if ((e = hipHostMalloc((void**)&b->stage[i], cap, hipHostMallocDefault)) != hipSuccess)
            return e;
    b->cap = cap;
    return hipSuccess;
}

mppi_status batch_enqueue(BatchWs* ws, hipStream_t stream, mppi_t* const* hs, const double* x0s,
                          const mppi_scene* scenes, const InstExtra* extra, int n, mppi_t* prof,
                          double* gather_dev, int slot_doubles, bool use_graph)
{
    mppi_t* h = prof;  // HIP_TRY marks it unusable on a device failure
    const size_t off_prefix = align_up(sizeof(BatchHdr), 16);
    const size_t off_descs = align_up(off_prefix + sizeof(int) * (size_t)(n + 1), 16);
    size_t bytes = align_up(off_descs + sizeof(InstDesc) * (size_t)n, 16);
    std::vector<SceneLayout> lay(n);
    std::vector<size_t> soff(n, 0);
    if (scenes) {
        for (int i = 0; i < n; ++i) {
            lay[i] = scene_layout(scenes[i].n_waypoints, scenes[i].n_circles);
            soff[i] = bytes;
            bytes += align_up(lay[i].bytes, 16);
        }
    }
    const size_t bucket = pow2_at_least(bytes, 64 << 10);
    HIP_TRY(ws_reserve(ws, bucket, stream));
    const BatchHdr* hdr_dev = reinterpret_cast<const BatchHdr*>(ws->arena);
    const int b = ws->cur;
    if (ws->pending[b]) {
        HIP_TRY(hipEventSynchronize(ws->done[b]));
        ws->pending[b] = false;
    }
    unsigned char* host = ws->stage[b];

    // group by kernel variant, longest tiles first inside a group
    std::vector<int> order(n), cls(n), occ(n);
    std::vector<double> work(n);
    long total = 0;  // tiles of the batch
    for (int i = 0; i < n; ++i) {
        const int nc = scenes ? scenes[i].n_circles : hs[i]->n_c;
        cls[i] = hs[i]->lanes_req ? hs[i]->lanes_req : auto_lanes(hs[i]->cfg, nc);
        total += ((long)hs[i]->cfg.K * cls[i] + kBlock - 1) / kBlock;
    }
    if (total > (1L << 30)) return fail(MPPI_E_INVALID, "batch too large");
    // Instances at 16 lanes that either kernel can run all take the one that more
    // of their tiles would, where the others are few: a launch of its own for a
    // few tiles leaves most of the chip idle (8 instances, one of them of 4096 x
    // 40: 151 us with it in k_batch and the others in the split kernel, 139 so).
    constexpr long kFewTiles = 1024;
    const int batch_tiles = (int)total;
    long in_split = 0, in_k_batch = 0;
    for (int i = 0; i < n; ++i) {
        const int nw = scenes ? scenes[i].n_waypoints : hs[i]->n_wp;
        const int nc = scenes ? scenes[i].n_circles : hs[i]->n_c;
        occ[i] = occ_choice(hs[i], nw, nc, cls[i], batch_tiles);
        if (split_could(hs[i], nw, cls[i])) (occ[i] == kOccSplit ? in_split : in_k_batch) += (hs[i]->cfg.K + 15) / 16;
    }
    const bool together = in_split && in_k_batch && std::min(in_split, in_k_batch) < kFewTiles;
    for (int i = 0; i < n; ++i) {
        const mppi_config& c = hs[i]->cfg;
        const int nw = scenes ? scenes[i].n_waypoints : hs[i]->n_wp;
        const int nc = scenes ? scenes[i].n_circles : hs[i]->n_c;
        const int g = cls[i];
        const int gi = g == 1 ? 0 : g == 2 ? 1 : g == 4 ? 2 : g == 8 ? 3 : 4;
        order[i] = i;
        if (together && split_could(hs[i], nw, g))
            occ[i] = in_split >= in_k_batch ? kOccSplit : k_batch_occ(hs[i], nc, g);
        cls[i] = 50 * occ[i] + 25 * (c.model ? 1 : 0) +
                 5 * (occ[i] == kOccSplit && c.per_step_weights ? 0 : gi) + active_ego(c.n_ego, nc);
        work[i] = (double)c.T * (73.0 + 6.0 * nw + 7.0 * c.n_ego * nc);
    }
    // The split kernel without the circles waves is launched for instances that
    // have no circles only if no other class can take them: a launch of a few
    // tiles of its own leaves most of the chip idle (of 256 uneven instances,
    // four without circles: 56 us).
    bool has[kLaneClasses] = {};
    for (int i = 0; i < n; ++i) has[cls[i]] = true;
    for (int i = 0; i < n; ++i) {
        const int with = cls[i] + hs[i]->cfg.n_ego;
        if (cls[i] >= 50 * kOccSplit && cls[i] % 5 == 0 && has[with]) cls[i] = with;
    }
    std::stable_sort(order.begin(), order.end(), [&](int a, int c) {
        return cls[a] != cls[c] ? cls[a] < cls[c] : work[a] > work[c];
    });
    // A batch of kMailBatch or more handles leaves their results in the host's
    // memory at its end (launch_mail): 3 us there (one of 16 instances of 8192 x 24
    // takes 107 us, one of 16 uneven ones 200), whether they are read or not, against a
    // launch of its own, 8 us with the wait, for every handle read.
    constexpr int kMailBatch = 16;
    const bool mail = !extra && n >= kMailBatch;
    for (int i = 0; i < n; ++i) hs[i]->mail = 0;
    BatchHdr* hdr = reinterpret_cast<BatchHdr*>(host);
    int* prefix = reinterpret_cast<int*>(host + off_prefix);
    InstDesc* descs = reinterpret_cast<InstDesc*>(host + off_descs);
    total = 0;
    size_t smem = 0, smem_split = 0;
    int any_shift = 0, any_out = 0, combine_g = 0, max_nodes = 0, most_tiles = 0;
    for (int j = 0; j < n; ++j) {
        const int i = order[j];
        mppi_t* hi = hs[i];
        const double* x0 = x0s + 4 * i;
        const InstExtra* ex = extra ? &extra[i] : nullptr;
        const int sh = ex && ex->shift ? 1 : 0;
        if (scenes) {
            const double origin[2] = {x0[0], x0[1]};
            write_scene(host + soff[i], lay[i], hi->cfg, origin, &scenes[i]);
            fill_desc(descs[j], hi, x0, origin, ws->arena + soff[i], lay[i], scenes[i].n_waypoints,
                      scenes[i].n_circles, sh, occ[i]);
        } else {
            fill_desc(descs[j], hi, x0, hi->origin, hi->scene, hi->lay, hi->n_wp, hi->n_c, sh,
                      occ[i]);
        }
        if (ex) {
            descs[j].S = ex->S;
            descs[j].eps = ex->eps;
            descs[j].partials = ex->partials;
            descs[j].q = ex->q;
            descs[j].Stk = ex->Stk;
            descs[j].out_slot = ex->out_slot;
            any_out |= ex->out_slot >= 0;
        }
        if (mail && !hi->captured && host_buffers(hi) == MPPI_OK) {
            descs[j].mail = hi->ctl_dev;
            descs[j].mail_seq = ++hi->seq;
        }
        prefix[j] = (int)total;
        total += descs[j].n_tiles;
        size_t& lds = descs[j].occ == kOccSplit ? smem_split : smem;
        lds = std::max(lds, iteration_lds(descs[j]));
        any_shift |= sh;
        combine_g = std::max(combine_g, combine_groups(descs[j].T));
        max_nodes = std::max(max_nodes, combine_nodes(descs[j].n_tiles, nullptr));
        if (!descs[j].per_step) most_tiles = std::max(most_tiles, descs[j].n_tiles);
    }
    prefix[n] = (int)total;
    hdr->n_inst = n;
    hdr->total_tiles = (int)total;
    hdr->off_prefix = (int)off_prefix;
    hdr->off_descs = (int)off_descs;
    int grids[kLaneClasses];
    {
        int j = 0;
        for (int c = 0; c < kLaneClasses; ++c) {
            hdr->cls_begin[c] = j;
            while (j < n && cls[order[j]] == c) ++j;
            const int tiles = prefix[j] - prefix[hdr->cls_begin[c]];
            grids[c] = tiles > 0 ? (int)pow2_at_least((size_t)tiles, 1) : 0;
        }
        hdr->cls_begin[kLaneClasses] = n;
    }
    const size_t smem_b = align_up(smem, 4096), smem_s = align_up(smem_split, 4096);
    const int node_limit = max_nodes <= kDirectSmall ? kDirectSmall : kDirect;
    // the merge's grid, rounded up like the others (0: nothing to merge)
    const int merge_tiles = most_tiles > kDirect ? (int)pow2_at_least((size_t)most_tiles, 1) : 0;
    const int n_blocks = (int)pow2_at_least((size_t)n, 1);
    const int shift_blocks = any_shift ? n_blocks : 0;
    const int gather_blocks = (gather_dev && any_out) ? n_blocks : 0;
    static const int kClassLanes[5] = {1, 2, 4, 8, 16};
    auto launch_class = [&](int c, int grid) {
        const int occ = c / 50, li = (c % 25) / 5;
        const bool ps = occ == kOccSplit && li == 0;  // (the split kernel's class for per-step weights)
        return launch_batch(ps ? 16 : kClassLanes[li], c % 5, (c % 50) / 25, occ, ps, nullptr, hdr_dev, c, grid,
                            occ == kOccSplit ? smem_s : smem_b, stream);
    };
    auto enqueue_device_work = [&](size_t copy_bytes) -> hipError_t {
        hipError_t e = hipMemcpyAsync(ws->arena, host, copy_bytes, hipMemcpyHostToDevice, stream);
        if (e == hipSuccess && shift_blocks) e = launch_shift_batch(hdr_dev, shift_blocks, stream);
        for (int c = 0; c < kLaneClasses && e == hipSuccess; ++c)
            if (grids[c] > 0)
                e = launch_class(c, grids[c]);
        if (e == hipSuccess) e = launch_merge(nullptr, hdr_dev, merge_tiles, n_blocks, stream);
        if (e == hipSuccess && combine_g)
            e = launch_combine(nullptr, hdr_dev, combine_g, n_blocks, max_nodes, stream);
        if (e == hipSuccess && gather_blocks)
            e = launch_gather(hdr_dev, gather_blocks, gather_dev, slot_doubles, stream);
        return e;
    };

    hipEvent_t a = nullptr;
    mppi_status s = record_launch(prof, 0, &a);
    if (s != MPPI_OK) return s;
    if (use_graph && graphs_enabled()) {
        GraphEntry* ge = nullptr;
        for (GraphEntry& g : ws->graphs)
            if (g.bytes == bucket && g.smem == smem_b && g.smem_split == smem_s && g.buf == b &&
                g.shift_blocks == shift_blocks && g.gather_blocks == gather_blocks &&
                g.combine_g == combine_g && g.combine_y == (combine_g ? n_blocks : 0) &&
                g.combine_nodes == node_limit && g.merge_tiles == merge_tiles && memcmp(g.grids, grids, sizeof grids) == 0)
                ge = &g;
        if (!ge) {
            if (ws->graphs.size() >= 64) {
                // a cached graph may still be running on the stream
                HIP_TRY(hipStreamSynchronize(stream));
                ws_drop_graphs(ws);
            }
            GraphEntry g;
            g.bytes = bucket;
            g.smem = smem_b;
            g.smem_split = smem_s;
            memcpy(g.grids, grids, sizeof grids);
            g.buf = b;
            g.shift_blocks = shift_blocks;
            g.gather_blocks = gather_blocks;
            g.combine_g = combine_g;
            g.combine_y = combine_g ? n_blocks : 0;
            g.combine_nodes = node_limit;
            g.merge_tiles = merge_tiles;
            g.graph = nullptr;
            g.exec = nullptr;
            HIP_TRY(hipStreamBeginCapture(stream, hipStreamCaptureModeThreadLocal));
            const hipError_t e = enqueue_device_work(bucket);
            const hipError_t e2 = hipStreamEndCapture(stream, &g.graph);
            HIP_TRY(e);
            HIP_TRY(e2);
            HIP_TRY(hipGraphInstantiate(&g.exec, g.graph, nullptr, nullptr, 0));
            ws->graphs.push_back(g);
            ge = &ws->graphs.back();
        }
        HIP_TRY(hipGraphLaunch(ge->exec, stream));
    } else {
        HIP_TRY(enqueue_device_work(bytes));
    }
    if ((s = record_end(prof, 0, a)) != MPPI_OK) return s;
    if (mail) {
        if (!ws->behind) ws->behind = std::make_shared<std::atomic<bool>>();
        HIP_TRY(launch_mail(hdr_dev, n, stream));
        ws->behind->store(false, std::memory_order_relaxed);
    }
    HIP_TRY(hipEventRecord(ws->done[b], stream));
    ws->pending[b] = true;
    ws->cur ^= 1;
    for (int j = 0; j < n; ++j) {
        hs[order[j]]->stepped = true;
        if (descs[j].mail) {
            hs[order[j]]->mail = descs[j].mail_seq;
            hs[order[j]]->mail_behind = ws->behind;
        }
        hs[order[j]]->last_lanes = descs[j].lanes;
        hs[order[j]]->last_occ = descs[j].occ;
        memcpy(hs[order[j]]->last_x0, x0s + 4 * order[j], sizeof(double) * 4);
        hs[order[j]]->last_steer0 = hs[order[j]]->steer0;
    }
    return MPPI_OK;
}

}  // namespace mppi_impl

// =====================================================================================
// C ABI
// =====================================================================================

extern "C" {

const char* mppi_version(void) { return "mppi-mi355x 0.2 (gfx950)"; }

const char* mppi_status_str(mppi_status s)
{
    switch (s) {
    case MPPI_OK: return "ok";
    case MPPI_E_INVALID: return "invalid argument";
    case MPPI_E_NOMEM: return "out of memory";
    case MPPI_E_DEVICE: return "device failure";
    case MPPI_E_NONFINITE: return "all sample costs non-finite";
    case MPPI_E_BUSY: return "busy";
    case MPPI_E_NOT_READY: return "not ready";
    default: return "unknown status";
    }
}

const char* mppi_last_error(void) { return g_last_error.c_str(); }

mppi_status mppi_create(const mppi_config* cfg, void* hip_stream, mppi_t** out)
{
    return handle_create(cfg, hip_stream, true, out);
}

mppi_status mppi_destroy(mppi_t* h)
{
    if (!h) return MPPI_OK;
    handle_release(h);
    delete h;
    return MPPI_OK;
}

mppi_status mppi_set_scene(mppi_t* h, const double x0[4], const mppi_scene* sc)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if ((s = validate_scene(h->cfg, x0, sc)) != MPPI_OK) return s;
    const int b = h->cur;
    // A captured upload reads its buffer when the graph is launched: a third one
    // in one capture would overwrite the first.  It says nothing when it has read
    // the buffer, which a launch long after would say of a later upload.
    const unsigned long long capture = capture_of(h);
    if (capture && h->staged_capture[b] == capture)
        return fail(MPPI_E_INVALID, "a capture holds at most two scenes of a handle");
    if ((s = wait_staged(h, b, capture != 0)) != MPPI_OK) return s;
    const SceneLayout L = scene_layout(sc->n_waypoints, sc->n_circles);
    const double origin[2] = {x0[0], x0[1]};
    write_scene(h->staging[b], L, h->cfg, origin, sc);
    mail_behind(h);
    unsigned* word = reinterpret_cast<unsigned*>(h->staging_dev[b] + align_up(h->scene_cap, 64));
    if (capture) h->staged_capture[b] = capture;
    else ++h->staged_seq[b];
    HIP_TRY(launch_stage(h->staging_dev[b], h->scene, L.bytes, capture ? nullptr : word, h->staged_seq[b],
                         h->stream));
    h->cur ^= 1;
    h->has_scene = true;
    h->origin[0] = origin[0];
    h->origin[1] = origin[1];
    h->n_wp = sc->n_waypoints;
    h->n_c = sc->n_circles;
    h->lay = L;
    return MPPI_OK;
}

mppi_status mppi_step_resident(mppi_t* h, const double x0[4])
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (!h->has_scene) return fail(MPPI_E_INVALID, "no scene has been set");
    if (!x0) return fail(MPPI_E_INVALID, "x0 must not be NULL");
    for (int i = 0; i < 4; ++i)
        if (!isfinite(x0[i])) return fail(MPPI_E_INVALID, "x0[%d] is not finite", i);
    changes_results(h);
    InstDesc d;
    fill_desc(d, h, x0, h->origin, h->scene, h->lay, h->n_wp, h->n_c, 0, -1);
    hipEvent_t a = nullptr;
    if ((s = record_launch(h, 0, &a)) != MPPI_OK) return s;
    hipEvent_t a2 = nullptr;
    if ((s = record_launch(h, 2, &a2)) != MPPI_OK) return s;
    HIP_TRY(launch_batch(d.lanes, active_ego(d.n_ego, d.n_c), d.model, d.occ, d.per_step, &d, nullptr, 0,
                         d.n_tiles, iteration_lds(d), h->stream));
    if ((s = record_end(h, 2, a2)) != MPPI_OK) return s;
    if (!d.per_step) HIP_TRY(launch_merge(&d, nullptr, d.n_tiles, 1, h->stream));
    HIP_TRY(launch_combine(&d, nullptr, combine_groups(d.T), 1, combine_nodes(d.n_tiles, nullptr),
                           h->stream));
    if ((s = record_end(h, 0, a)) != MPPI_OK) return s;
    h->last_lanes = d.lanes;
    h->last_occ = d.occ;
    h->stepped = true;
    memcpy(h->last_x0, x0, sizeof(double) * 4);
    h->last_steer0 = h->steer0;
    return MPPI_OK;
}

mppi_status mppi_step(mppi_t* h, const double x0[4], const mppi_scene* sc)
{
    mppi_status s = mppi_set_scene(h, x0, sc);
    if (s != MPPI_OK) return s;
    return mppi_step_resident(h, x0);
}

mppi_status mppi_step_batch(mppi_t* const* hs, const double* x0s, const mppi_scene* scenes,
                            int32_t n)
{
    if (!hs || !x0s || n < 1) return fail(MPPI_E_INVALID, "handles, states and n >= 1 required");
    mppi_t* lead = hs[0];
    mppi_status s;
    for (int i = 0; i < n; ++i) {
        if ((s = usable(hs[i])) != MPPI_OK) return s;
        if (!hs[i]->S) return fail(MPPI_E_INVALID, "handle %d has no iteration buffers", i);
        if (hs[i]->stream != lead->stream)
            return fail(MPPI_E_INVALID, "every handle of a batch must use the same stream");
        for (int j = 0; j < i; ++j)
            if (hs[j] == hs[i]) return fail(MPPI_E_INVALID, "handle %d appears twice", i);
        if (scenes) {
            if ((s = validate_scene(hs[i]->cfg, x0s + 4 * i, &scenes[i])) != MPPI_OK) return s;
        } else {
            if (!hs[i]->has_scene) return fail(MPPI_E_INVALID, "handle %d has no scene", i);
            for (int k = 0; k < 4; ++k)
                if (!isfinite(x0s[4 * i + k])) return fail(MPPI_E_INVALID, "x0 not finite");
        }
    }
    if (!lead->batch && (s = ws_create(&lead->batch)) != MPPI_OK) return s;
    return batch_enqueue(lead->batch, lead->stream, hs, x0s, scenes, nullptr, n, lead, nullptr, 0,
                         true);
}

mppi_status mppi_sync(mppi_t* h)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    return sync_status(h);
}

mppi_status mppi_get_controls(mppi_t* h, double* out, size_t n)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (!out || n < (size_t)2 * h->cfg.T)
        return fail(MPPI_E_INVALID, "output buffer needs %d doubles", 2 * h->cfg.T);
    // U and the state written by one small kernel straight into pinned host
    // memory (no copies back to wait for)
    const int nu = 2 * h->cfg.T;
    if ((s = export_results(h, nu)) != MPPI_OK) return s;
    memcpy(out, h->ctl_host, sizeof(double) * nu);
    if (h->stepped && reinterpret_cast<const DevState*>(h->ctl_host + nu)->status != 0)
        return fail(MPPI_E_NONFINITE, "every sample cost of the last step was non-finite");
    return MPPI_OK;
}

mppi_status mppi_set_controls(mppi_t* h, const double* U, size_t n)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (!U || n < (size_t)2 * h->cfg.T)
        return fail(MPPI_E_INVALID, "controls need %d doubles", 2 * h->cfg.T);
    for (int i = 0; i < 2 * h->cfg.T; ++i)
        if (!isfinite(U[i])) return fail(MPPI_E_INVALID, "controls must be finite");
    h->mail = 0;
    HIP_TRY(hipStreamSynchronize(h->stream));
    HIP_TRY(hipMemcpy(h->U, U, sizeof(double) * 2 * h->cfg.T, hipMemcpyHostToDevice));
    return MPPI_OK;
}

mppi_status mppi_shift(mppi_t* h, int32_t steps)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (steps < 0) return fail(MPPI_E_INVALID, "steps must be >= 0");
    if (steps == 0) return MPPI_OK;
    changes_results(h);
    return launch_aux(h, [&] { return launch_shift(h->U, h->cfg.T, steps, h->stream); });
}

mppi_status mppi_get_state(mppi_t* h, double* U, size_t n, uint64_t* n_iter, uint64_t* seed)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (!U || n < (size_t)2 * h->cfg.T)
        return fail(MPPI_E_INVALID, "state buffer needs %d doubles", 2 * h->cfg.T);
    // U and the state through the pinned export buffer (one small kernel)
    const int nu = 2 * h->cfg.T;
    if ((s = export_results(h, nu)) != MPPI_OK) return s;
    memcpy(U, h->ctl_host, sizeof(double) * nu);
    if (n_iter) *n_iter = reinterpret_cast<const DevState*>(h->ctl_host + nu)->n_iter;
    if (seed) *seed = h->cfg.seed;
    return MPPI_OK;
}

mppi_status mppi_set_state(mppi_t* h, const double* U, size_t n, uint64_t n_iter)
{
    mppi_status s = mppi_set_controls(h, U, n);
    if (s != MPPI_OK) return s;
    DevState st;
    HIP_TRY(hipMemcpy(&st, h->st, sizeof st, hipMemcpyDeviceToHost));
    st.n_iter = n_iter;
    st.reserved = 0;
    st.status = 0;
    HIP_TRY(hipMemcpy(h->st, &st, sizeof st, hipMemcpyHostToDevice));
    h->stepped = false;
    return MPPI_OK;
}

mppi_status mppi_get_costs(mppi_t* h, float* out, size_t n)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (!out || n < (size_t)h->cfg.K) return fail(MPPI_E_INVALID, "buffer needs K floats");
    HIP_TRY(hipStreamSynchronize(h->stream));
    HIP_TRY(hipMemcpy(out, h->S, sizeof(float) * h->cfg.K, hipMemcpyDeviceToHost));
    return MPPI_OK;
}

mppi_status mppi_get_weights(mppi_t* h, double* out, size_t n)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (!out || n < (size_t)h->cfg.K) return fail(MPPI_E_INVALID, "buffer needs K doubles");
    if ((s = sync_status(h)) != MPPI_OK) return s;
    if (!h->stepped) return fail(MPPI_E_NOT_READY, "no step has completed");
    InstDesc d;
    memset(&d, 0, sizeof d);
    d.K = h->cfg.K;
    d.S = h->S;
    d.per_step = h->cfg.per_step_weights;
    d.Stk = h->Stk;
    d.lambda = h->cfg.lambda;
    d.st = h->st;
    s = launch_aux(h, [&] { return launch_weights(d, h->wbuf, h->stream); });
    if (s != MPPI_OK) return s;
    HIP_TRY(hipStreamSynchronize(h->stream));
    HIP_TRY(hipMemcpy(out, h->wbuf, sizeof(double) * h->cfg.K, hipMemcpyDeviceToHost));
    return MPPI_OK;
}

mppi_status mppi_get_noise(mppi_t* h, float* out, size_t n)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    const size_t need = (size_t)2 * h->cfg.T * h->cfg.K;
    if (!out || n < need) return fail(MPPI_E_INVALID, "buffer needs 2*T*K floats");
    HIP_TRY(hipStreamSynchronize(h->stream));
    HIP_TRY(hipMemcpy(out, h->eps, sizeof(float) * need, hipMemcpyDeviceToHost));
    return MPPI_OK;
}

mppi_status mppi_get_trajectory(mppi_t* h, double* states, size_t n_states, double* controls,
                                size_t n_controls)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    const int T = h->cfg.T;
    const size_t cols = h->cfg.model ? 5 : 4;
    if (!h->stepped) return fail(MPPI_E_INVALID, "no step has been taken");
    if (states && n_states < cols * (T + 1))
        return fail(MPPI_E_INVALID, "states needs %zu*(T+1) doubles", cols);
    if (controls && n_controls < (size_t)2 * T)
        return fail(MPPI_E_INVALID, "controls needs 2*T doubles");
    TrajArgs a;
    const mppi_config& c = h->cfg;
    for (int i = 0; i < 4; ++i) a.x0[i] = h->last_x0[i];
    a.steer0 = h->last_steer0;
    a.T = T;
    a.model = c.model;
    a.dt = c.dt;
    a.wheelbase = c.wheelbase;
    a.a_min = c.u_min[0];
    a.a_max = c.u_max[0];
    a.d_min = c.u_min[1];
    a.d_max = c.u_max[1];
    a.v_max = c.v_max;
    // states then controls, written by the kernel straight into the pinned
    // host buffer: no copy back to wait for
    const size_t ns = cols * (T + 1), nu = (size_t)2 * T;
    if ((s = host_buffers(h)) != MPPI_OK) return s;
    const uint32_t seq = ++h->seq;
    mail_behind(h);
    HIP_TRY(launch_trajectory(a, h->U, h->traj_dev, h->traj_dev + ns, h->done_dev, seq, h->stream));
    if ((s = wait_done(h, h->done, seq)) != MPPI_OK) return s;
    if (states) memcpy(states, h->traj, sizeof(double) * ns);
    if (controls) memcpy(controls, h->traj + ns, sizeof(double) * nu);
    return MPPI_OK;
}

mppi_status mppi_get_stage_costs(mppi_t* h, float* out, size_t n)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (!h->cfg.per_step_weights || !h->q)
        return fail(MPPI_E_INVALID, "stage costs are kept only with per-step weights");
    const size_t need = (size_t)h->cfg.T * h->cfg.K;
    if (!out || n < need) return fail(MPPI_E_INVALID, "buffer needs T*K floats");
    HIP_TRY(hipStreamSynchronize(h->stream));
    HIP_TRY(hipMemcpy(out, h->q, sizeof(float) * need, hipMemcpyDeviceToHost));
    return MPPI_OK;
}

mppi_status mppi_set_steering(mppi_t* h, double delta0)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (!isfinite(delta0)) return fail(MPPI_E_INVALID, "steering angle must be finite");
    h->steer0 = delta0;
    return MPPI_OK;
}

mppi_status mppi_get_iter_stats(mppi_t* h, mppi_iter_stats* out)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (!out) return fail(MPPI_E_INVALID, "out is NULL");
    DevState st;
    s = read_state(h, &st);
    if (s != MPPI_OK) return s;
    out->s_min = st.s_min;
    out->log_z = st.log_z;
    out->ess = st.ess;
    out->n_iter = st.n_iter;
    out->status = st.status;
    out->lanes_per_sample = h->last_lanes;
    return MPPI_OK;
}

mppi_status mppi_set_lanes_per_sample(mppi_t* h, int32_t lanes)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (!(lanes == 0 || lanes == 1 || lanes == 2 || lanes == 4 || lanes == 8 || lanes == 16))
        return fail(MPPI_E_INVALID, "lanes per sample must be 0, 1, 2, 4, 8 or 16");
    h->lanes_req = lanes;
    return MPPI_OK;
}

mppi_status mppi_set_occupancy(mppi_t* h, int32_t mode)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (mode < -1 || mode > kOccHigh)
        return fail(MPPI_E_INVALID, "occupancy mode must be -1, 0 or 1");
    h->occ_req = mode;
    return MPPI_OK;
}

mppi_status mppi_get_kernel(mppi_t* h, int32_t* kernel)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (!kernel) return fail(MPPI_E_INVALID, "kernel is NULL");
    if (h->last_occ < 0) return fail(MPPI_E_NOT_READY, "no step has been taken");
    *kernel = h->last_occ;
    return MPPI_OK;
}

mppi_status mppi_set_staging(mppi_t* h, int32_t mode)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (mode < -1 || mode > 1) return fail(MPPI_E_INVALID, "staging mode must be -1, 0 or 1");
    h->stage_req = mode;
    return MPPI_OK;
}

mppi_status mppi_set_culling(mppi_t* h, int32_t on)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    h->no_cull = on ? 0 : 1;
    return MPPI_OK;
}

mppi_status mppi_get_stream(mppi_t* h, void** stream)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (!stream) return fail(MPPI_E_INVALID, "stream is NULL");
    *stream = (void*)h->stream;
    return MPPI_OK;
}

mppi_status mppi_set_profiling(mppi_t* h, int32_t on)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if ((s = drain_profile(h)) != MPPI_OK) return s;
    h->prof = on != 0;
    if (on) {
        h->prof_ms[0] = h->prof_ms[1] = h->prof_ms[2] = 0.0;
        h->prof_n[0] = h->prof_n[1] = h->prof_n[2] = 0;
        // events for a few hundred profiled steps, created now rather than
        // between launches
        while (h->event_pool.size() < 1024) {
            hipEvent_t e;
            HIP_TRY(hipEventCreate(&e));
            h->event_pool.push_back(e);
        }
    }
    return MPPI_OK;
}

mppi_status mppi_get_profile(mppi_t* h, mppi_profile* out)
{
    mppi_status s = usable(h);
    if (s != MPPI_OK) return s;
    if (!out) return fail(MPPI_E_INVALID, "out is NULL");
    if ((s = drain_profile(h)) != MPPI_OK) return s;
    out->iter_ms = h->prof_ms[0];
    out->iter_launches = h->prof_n[0];
    out->aux_ms = h->prof_ms[1];
    out->aux_launches = h->prof_n[1];
    out->rollout_ms = h->prof_ms[2];
    out->rollout_launches = h->prof_n[2];
    return MPPI_OK;
}

mppi_status mppi_debug_philox(uint64_t seed, uint64_t n_iter, uint32_t k0, uint32_t nk,
                              uint32_t j0, uint32_t nj, uint32_t* out, size_t n)
{
    const uint64_t cnt = (uint64_t)nk * nj;
    if (!out || n < 4 * cnt) return fail(MPPI_E_INVALID, "buffer needs 4*nk*nj words");
    if (cnt == 0) return MPPI_OK;
    if (cnt > (1ull << 28)) return fail(MPPI_E_INVALID, "nk*nj too large");
    uint32_t* dev = nullptr;
    hipError_t e = hipMalloc((void**)&dev, sizeof(uint32_t) * 4 * cnt);
    if (e != hipSuccess) return fail(MPPI_E_NOMEM, "hipMalloc: %s", hipGetErrorString(e));
    e = launch_debug_philox((uint32_t)seed, (uint32_t)(seed >> 32), n_iter, k0, nk, j0, nj, dev,
                            nullptr);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e == hipSuccess)
        e = hipMemcpy(out, dev, sizeof(uint32_t) * 4 * cnt, hipMemcpyDeviceToHost);
    (void)hipFree(dev);
    if (e != hipSuccess) return fail(MPPI_E_DEVICE, "debug philox: %s", hipGetErrorString(e));
    return MPPI_OK;
}

mppi_status mppi_bench_copy(size_t bytes, int32_t reps)
{
    const size_t n16 = bytes / 16;
    if (n16 == 0 || reps < 1) return fail(MPPI_E_INVALID, "bytes >= 16 and reps >= 1 required");
    float4 *a = nullptr, *b = nullptr;
    hipError_t e = hipMalloc((void**)&a, n16 * 16);
    if (e == hipSuccess) e = hipMalloc((void**)&b, n16 * 16);
    if (e == hipSuccess) e = hipMemset(a, 0, n16 * 16);
    for (int r = 0; r < reps && e == hipSuccess; ++r) e = launch_copy(a, b, n16, nullptr);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    (void)hipFree(a);
    (void)hipFree(b);
    if (e != hipSuccess) return fail(MPPI_E_DEVICE, "copy: %s", hipGetErrorString(e));
    return MPPI_OK;
}

}  // extern "C"
