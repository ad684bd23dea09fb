// Device code shared by the two iteration kernels (mppi_kernels.hip, where a
// wave does every part of its samples' rollouts, and mppi_split.hpp, where
// the parts are given to different waves): memory accesses, the noise, the
// stage cost and its culling, and wave reductions.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "mppi_internal.hpp"

namespace mppi_impl {

// Accesses to the instance's global arrays through pointers typed as global
// memory: the descriptor's pointers are generic, and generic (flat)
// accesses also count against the counter that scalar and LDS loads wait
// on, so every wait for a scalar candidate load would also wait for the
// rollout's in-flight global loads and stores.
typedef float f2v __attribute__((ext_vector_type(2)));
typedef float f4v __attribute__((ext_vector_type(4)));
template <typename T>
using gptr = __attribute__((address_space(1))) T*;
template <typename T>
__device__ __forceinline__ gptr<T> as_global(T* p)
{
    return (gptr<T>)p;
}
template <typename T>
__device__ __forceinline__ T ld_g(const T* p, size_t i)
{
    return as_global(p)[i];
}
__device__ __forceinline__ float2 ld_g(const float2* p, size_t i)
{
    const f2v v = as_global(reinterpret_cast<const f2v*>(p))[i];
    return make_float2(v.x, v.y);
}
__device__ __forceinline__ float4 ld_g(const float4* p, size_t i)
{
    const f4v v = as_global(reinterpret_cast<const f4v*>(p))[i];
    return make_float4(v.x, v.y, v.z, v.w);
}
// Element i (below 2^32 bytes from p) of a small array: a 32-bit offset from
// a uniform base, without 64-bit address arithmetic per lane.
__device__ __forceinline__ float2 ld_g32(const float2* p, unsigned i)
{
    const f2v v = *(gptr<const f2v>)((gptr<const char>)(const char*)p + i * 8u);
    return make_float2(v.x, v.y);
}
template <typename T>
__device__ __forceinline__ void st_g(T* p, size_t i, T v)
{
    as_global(p)[i] = v;
}
__device__ __forceinline__ void st_g(float2* p, size_t i, float2 v)
{
    f2v w;
    w.x = v.x;
    w.y = v.y;
    as_global(reinterpret_cast<f2v*>(p))[i] = w;
}
// A store written through the XCD's L2 to the device's coherence point (a
// relaxed agent-scope atomic store; its bits are those of the plain store).
// Each XCD has its own write-back L2, so the release at the end of a kernel
// writes back every line still dirty there before a dependent kernel can
// start; data written through is already out, and that release has less to
// do.  Used for the applied perturbations, written once and read by the
// host (and the next launch only through another kernel).
__device__ __forceinline__ void st_wt(float2* p, size_t i, float2 v)
{
    const unsigned long long bits = (unsigned long long)__float_as_uint(v.x) |
                                    ((unsigned long long)__float_as_uint(v.y) << 32);
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p) + i, bits, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// ----------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of the
// 4x32 S-box (two 32x32->64 multiplies, xor with the other half and the key)
// with a Weyl-sequence key schedule.
// ----------------------------------------------------------------------------
// (v_bitop3 with truth table 0x96 is the three-input exclusive or of gfx950)
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
        c = make_uint4(__builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c.y, k0, 0x96),
                       (uint32_t)p1,
                       __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c.w, k1, 0x96),
                       (uint32_t)p0);
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// Gaussian perturbation (before the noise check) of step t of sample k at
// iteration n: counter (k, t/2, n_lo, n_hi); words (r0, r1) for even t and
// (r2, r3) for odd t; u = ((r >> 9) + 1/2) 2^-23 is exact in float32;
// Box-Muller with the angle taken in revolutions by the hardware sin/cos.
__device__ __forceinline__ uint4 noise_words(const InstDesc& d, int k, int pair,
                                             unsigned long long n)
{
    return philox4x32_10(make_uint4((uint32_t)k, (uint32_t)pair, (uint32_t)n, (uint32_t)(n >> 32)),
                         d.key0, d.key1);
}

__device__ __forceinline__ float2 noise_from_words(const InstDesc& d, uint32_t ra, uint32_t rb)
{
    const float u1 = ((float)(ra >> 9) + 0.5f) * 0x1p-23f;
    const float u2 = ((float)(rb >> 9) + 0.5f) * 0x1p-23f;
    // -2 ln u1 = -2 ln(2) log2(u1)
    const float rho = __builtin_amdgcn_sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u1));
    return make_float2(d.sig_a * rho * __builtin_amdgcn_cosf(u2),
                       d.sig_d * rho * __builtin_amdgcn_sinf(u2));
}

__device__ __forceinline__ float2 draw_noise(const InstDesc& d, int k, int t,
                                             unsigned long long n)
{
    const uint4 r = noise_words(d, k, t >> 1, n);
    return noise_from_words(d, (t & 1) ? r.z : r.x, (t & 1) ? r.w : r.y);
}

struct Lds {
    float4* c_pv;
    float4* wp_box;
    float2* wp_xy;
    double* red;
    float* wp_vref;
    float* wp_yaw;
    float* c_rr;
    double* omega; // [spb] the tile's float64 exponential weights
    float* eps;  // [2T][spb + 1]: column 2t + c, sample j at (2t + c)(spb + 1) + j
    float* qs;   // [T][spb + 1] stage costs (per-step weights)
    double* ss;  // [T][spb + 1] cost-to-go (per-step weights), rows padded by one
};

__device__ __forceinline__ Lds lds_bind(unsigned char* base, const LdsLayout& L)
{
    Lds s;
    s.c_pv = reinterpret_cast<float4*>(base + L.c_pv);
    s.wp_box = reinterpret_cast<float4*>(base + L.wp_box);
    s.wp_xy = reinterpret_cast<float2*>(base + L.wp_xy);
    s.red = reinterpret_cast<double*>(base + L.red);
    s.wp_vref = reinterpret_cast<float*>(base + L.wp_vref);
    s.wp_yaw = reinterpret_cast<float*>(base + L.wp_yaw);
    s.c_rr = reinterpret_cast<float*>(base + L.c_rr);
    s.omega = reinterpret_cast<double*>(base + L.omega);
    s.eps = reinterpret_cast<float*>(base + L.eps);
    s.qs = reinterpret_cast<float*>(base + L.qs);
    s.ss = reinterpret_cast<double*>(base + L.ss);
    return s;
}

// Closest-waypoint update over chunk ch (kChunk consecutive waypoints, padded
// with points at infinity): the chunk is read with 16-byte LDS reads (two
// points each) and its distances are compared in index order, so ties keep
// the lowest index.
__device__ __forceinline__ void scan_chunk(const Lds& s, int ch, float x, float y, float& best,
                                           int& bj)
{
    const float4* p = reinterpret_cast<const float4*>(s.wp_xy) + ch * kChunkQ;
#pragma unroll
    for (int u = 0; u < kChunkQ; ++u) {
        const float4 q = p[u];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float dx = x - (h ? q.z : q.x);
            const float dy = y - (h ? q.w : q.y);
            const float dd = fmaf(dy, dy, dx * dx);
            if (dd < best) {
                best = dd;
                bj = ch * kChunk + 2 * u + h;
            }
        }
    }
}

// Clearance between the ego circles (centres ex, ey) and obstacle circle p
// at time tau: min_e ||P_e - O|| - (r_c + r_ego), with the square root taken
// once, of the smallest squared distance (the root is monotone).
template <int NE>
__device__ __forceinline__ float circle_gap(const float (&ex)[NE > 0 ? NE : 1],
                                            const float (&ey)[NE > 0 ? NE : 1], const float4& p,
                                            float rr, float tau)
{
    const float ox = fmaf(tau, p.z, p.x);
    const float oy = fmaf(tau, p.w, p.y);
    float m2 = 0.0f;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        const float dx = ex[e] - ox;
        const float dy = ey[e] - oy;
        const float d2 = fmaf(dy, dy, dx * dx);
        m2 = e == 0 ? d2 : fminf(m2, d2);
    }
    return __builtin_amdgcn_sqrtf(m2) - rr;
}

// The Sec. IV-C terms beyond tracking, speed and obstacles, each skipped at
// zero weight: c_target = 1 when the step from (xp, yp) to (x, y) ends
// farther from the target point (the last waypoint) -- the sign of
// |P - T|^2 - |P_prev - T|^2 = (P - P_prev).(P + P_prev - 2 T) -- and c_yaw,
// the heading th minus the yaw of closest waypoint bj, wrapped into
// [-pi, pi), squared.
// The waypoint arrays are read from wxy / wyaw: the tile's LDS copy, or
// (GLOBAL) the scene in global memory -- the same values either way.
template <bool GLOBAL>
__device__ __forceinline__ float extra_terms(const InstDesc& d, const float2* wxy,
                                             const float* wyaw, int bj, float x, float y,
                                             float th, float xp, float yp)
{
    float e = 0.0f;
    if (d.w_target != 0.0f) {
        const float2 tp = GLOBAL ? ld_g(wxy, d.n_wp - 1) : wxy[d.n_wp - 1];
        const float dx = x - xp, dy = y - yp;
        const float sx = (x - tp.x) + (xp - tp.x), sy = (y - tp.y) + (yp - tp.y);
        e = fmaf(d.w_target, fmaf(dx, sx, dy * sy) > 0.0f ? 1.0f : 0.0f, e);
    }
    if (d.w_yaw != 0.0f) {
        float dyaw = th - (GLOBAL ? ld_g(wyaw, bj) : wyaw[bj]);
        dyaw -= 6.28318530717958647692f *
                floorf((dyaw + 3.14159265358979323846f) * 0.15915494309189533577f);
        e = fmaf(d.w_yaw, dyaw * dyaw, e);
    }
    return e;
}

// Obstacle cost from the clearance d_obj and the safety distance ds; in the
// collision-only mode it counts only when an object is hit (d_obj <= 0).
__device__ __forceinline__ float safe_cost(const InstDesc& d, float ds, float d_obj)
{
    const float g = ds - d_obj;
    return (g > 0.0f && (!d.coll_only || d_obj <= 0.0f)) ? g * g : 0.0f;
}

// Stage cost on the state reached at step t (Sec. III input cost, Sec. IV-C
// tracking, speed and obstacle costs).  Every lane of the wave runs the same
// waypoint and circle loops, so the LDS reads are broadcasts.
template <int NE>
__device__ __forceinline__ float stage_cost(const InstDesc& d, const Lds& s, float x, float y,
                                            float c, float sn, float v, float Ua, float Ud,
                                            float ea, float ed, int t, float th, float xp,
                                            float yp)
{
    // c_dist = min_j ||P - W_j||^2; reference speed of the closest waypoint
    float best = INFINITY;
    int bj = 0;
    for (int ch = 0; ch * kChunk < d.n_wp; ++ch) scan_chunk(s, ch, x, y, best, bj);
    const float ext = extra_terms<false>(d, s.wp_xy, s.wp_yaw, bj, x, y, th, xp, yp);
    const float dv = v - s.wp_vref[bj];
    // q_u = w_effort (alpha eps.eps + U.eps + U.U / 2)
    const float q = d.w_effort * (d.alpha * fmaf(ea, ea, ed * ed) + fmaf(Ua, ea, Ud * ed) +
                                  0.5f * fmaf(Ua, Ua, Ud * Ud));
    float cost = fmaf(d.w_track, best, fmaf(d.w_speed, dv * dv, q));
    if (NE > 0) {
        float ex[NE > 0 ? NE : 1], ey[NE > 0 ? NE : 1];
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            ex[e] = fmaf(d.ego_off[e], c, x);
            ey[e] = fmaf(d.ego_off[e], sn, y);
        }
        const float tau = (float)(t + 1) * d.dt;
        float d_obj = INFINITY;
        for (int i = 0; i < d.n_c; ++i) {
            const float4 p = s.c_pv[i];
            const float rr = s.c_rr[i];
            d_obj = fminf(d_obj, circle_gap<NE>(ex, ey, p, rr, tau));
        }
        cost = fmaf(d.w_coll, safe_cost(d, fmaf(d.d_safe_c, v, d.d_safe_0), d_obj), cost);
    }
    return cost + ext;
}

// ----------------------------------------------------------------------------
// Wave-level culling helpers.
// ----------------------------------------------------------------------------

// Order-preserving map of float32 onto int32 (its own inverse): for non-NaN
// values the integer order of the keys is the float order, so wave minima and
// maxima run on integer DPP operations without NaN canonicalisation.
__device__ __forceinline__ int fkey(float f)
{
    const int b = __builtin_bit_cast(int, f);
    return b ^ ((b >> 31) & 0x7fffffff);
}
__device__ __forceinline__ float fkey_inv(int k)
{
    return __builtin_bit_cast(float, k ^ ((k >> 31) & 0x7fffffff));
}
constexpr float kNowhere = 1e30f;               // where nothing is: positions, distances below zero
constexpr int kKeyPosInf = 0x7f800000;          // fkey(+inf)
constexpr int kKeyNegInf = (int)0x807fffffu;    // fkey(-inf)

// Cross-lane move by a DPP control; lanes outside row_mask receive `idv`,
// the identity of the reduction that consumes the value.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ int dpp_i(int idv, int x)
{
    return __builtin_amdgcn_update_dpp(idv, x, CTRL, ROW_MASK, 0xf, false);
}
constexpr int kIntMax = 0x7fffffff;
constexpr int kIntMin = (int)0x80000000u;

// Prefix sums inside aligned groups of G lanes (G <= 16, so a group lies in
// one DPP row): the inclusive sum (or maximum) up to lane r of the group,
// the value of lane r - 1 (0 for the first lane), and the group's last
// lane's value.  With G = 16 a group is a whole row, and a row shift by N
// already gives lanes r < N nothing from another group (bound_ctrl reads 0;
// without it the lane keeps the identity passed as the old value), so no
// lane mask is needed.
template <int N>
__device__ __forceinline__ float dpp_shr(float v)
{
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x110 + N, 0xf, 0xf, true));
}
template <int G>
__device__ __forceinline__ float seg_scan(float v, int r)
{
    if (G == 16) {
        v += dpp_shr<1>(v);
        v += dpp_shr<2>(v);
        v += dpp_shr<4>(v);
        v += dpp_shr<8>(v);
        return v;
    }
    if (G >= 2) { const float u = dpp_shr<1>(v); v += r >= 1 ? u : 0.0f; }
    if (G >= 4) { const float u = dpp_shr<2>(v); v += r >= 2 ? u : 0.0f; }
    if (G >= 8) { const float u = dpp_shr<4>(v); v += r >= 4 ? u : 0.0f; }
    return v;
}
template <int G>
__device__ __forceinline__ float seg_scan_max(float v, int r)
{
    if (G == 16) {
        // on order-preserving integer keys (non-NaN floats): one DPP max per
        // stage; lanes r < N keep the identity
        int k = fkey(v);
        k = max(k, dpp_i<0x111>(kIntMin, k));
        k = max(k, dpp_i<0x112>(kIntMin, k));
        k = max(k, dpp_i<0x114>(kIntMin, k));
        k = max(k, dpp_i<0x118>(kIntMin, k));
        return fkey_inv(k);
    }
    if (G >= 2) { const float u = dpp_shr<1>(v); v = r >= 1 ? fmaxf(v, u) : v; }
    if (G >= 4) { const float u = dpp_shr<2>(v); v = r >= 2 ? fmaxf(v, u) : v; }
    if (G >= 8) { const float u = dpp_shr<4>(v); v = r >= 4 ? fmaxf(v, u) : v; }
    return v;
}
template <int G>
__device__ __forceinline__ float seg_prev(float incl, int r)
{
    if (G == 1) return 0.0f;
    const float u = dpp_shr<1>(incl);
    if (G == 16) return u;
    return r >= 1 ? u : 0.0f;
}
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v)
{
    return __builtin_bit_cast(
        float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
// The group's last lane's value in every lane of the group, by DPP: quad
// permutes for groups of 2 and 4, row broadcasts (row_newbcast) of lanes 7
// and 15 for groups of 8 and 16.
template <int G>
__device__ __forceinline__ float group_last(float v, int gbase)
{
    (void)gbase;
    if (G == 1) return v;
    if (G == 2) return dpp_f<0xF5>(v);   // quad_perm [1, 1, 3, 3]
    if (G == 4) return dpp_f<0xFF>(v);   // quad_perm [3, 3, 3, 3]
    const float hi = dpp_f<0x15F>(v);    // row_newbcast:15
    if (G == 16) return hi;
    const float lo = dpp_f<0x157>(v);    // row_newbcast:7
    return (threadIdx.x & 8) ? hi : lo;
}

// Wave-wide reduction stages: swap neighbours and quad halves, mirror inside
// half rows and rows (every lane then holds its row's result), broadcast lane
// 15 into rows 1 and 3 and lane 31 into rows 2 and 3; lane 63 ends with the
// result over all 64 lanes.  Five independent reductions (two minima, three
// maxima) advance stage by stage so that their DPP latencies overlap.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ void red5_stage(int& a, int& b, int& c, int& e, int& f)
{
    a = min(a, dpp_i<CTRL, ROW_MASK>(kIntMax, a));
    b = min(b, dpp_i<CTRL, ROW_MASK>(kIntMax, b));
    c = max(c, dpp_i<CTRL, ROW_MASK>(kIntMin, c));
    e = max(e, dpp_i<CTRL, ROW_MASK>(kIntMin, e));
    f = max(f, dpp_i<CTRL, ROW_MASK>(kIntMin, f));
}

__device__ __forceinline__ int lane63(int x) { return __builtin_amdgcn_readlane(x, 63); }

// Bounding box of the positions of the lanes with inc set, and the largest
// safety distance among them (keys of +-inf for an empty set).
struct WaveBox {
    float xlo, xhi, ylo, yhi, dsmax;
};

// The box of each row of 16 lanes (of a sample's 16 steps, at 16 lanes per
// sample), in every lane of the row, as keys.
struct BoxKeys {
    int a, b, c, e, f;
};
__device__ __forceinline__ WaveBox box_of_keys(const BoxKeys& k)
{
    WaveBox w;
    w.xlo = fkey_inv(k.a);
    w.ylo = fkey_inv(k.b);
    w.xhi = fkey_inv(k.c);
    w.yhi = fkey_inv(k.e);
    w.dsmax = fkey_inv(k.f);
    return w;
}
__device__ __forceinline__ BoxKeys row_box(bool inc, float x, float y, float ds)
{
    BoxKeys k;
    k.a = inc ? fkey(x) : kKeyPosInf;
    k.b = inc ? fkey(y) : kKeyPosInf;
    k.c = inc ? fkey(x) : kKeyNegInf;
    k.e = inc ? fkey(y) : kKeyNegInf;
    k.f = inc ? fkey(ds) : kKeyNegInf;
    red5_stage<0xB1>(k.a, k.b, k.c, k.e, k.f);   // quad_perm [1,0,3,2]
    red5_stage<0x4E>(k.a, k.b, k.c, k.e, k.f);   // quad_perm [2,3,0,1]
    red5_stage<0x141>(k.a, k.b, k.c, k.e, k.f);  // row_half_mirror
    red5_stage<0x140>(k.a, k.b, k.c, k.e, k.f);  // row_mirror
    return k;
}
// The wave's box from the rows'.
__device__ __forceinline__ WaveBox wave_box_of_rows(BoxKeys k)
{
    red5_stage<0x142, 0xa>(k.a, k.b, k.c, k.e, k.f);  // row_bcast:15
    red5_stage<0x143, 0xc>(k.a, k.b, k.c, k.e, k.f);  // row_bcast:31
    k.a = lane63(k.a);
    k.b = lane63(k.b);
    k.c = lane63(k.c);
    k.e = lane63(k.e);
    k.f = lane63(k.f);
    return box_of_keys(k);
}
__device__ __forceinline__ WaveBox wave_box(bool inc, float x, float y, float ds)
{
    return wave_box_of_rows(row_box(inc, x, y, ds));
}

// Wave minimum and maximum of non-negative floats (their bit patterns are
// ordered), advanced stage by stage together.
__device__ __forceinline__ void wave_minmax_nonneg(float vmin, float vmax, float& omin,
                                                   float& omax)
{
    int a = __builtin_bit_cast(int, vmin);
    int b = __builtin_bit_cast(int, vmax);
    a = min(a, dpp_i<0xB1>(kIntMax, a));
    b = max(b, dpp_i<0xB1>(kIntMin, b));
    a = min(a, dpp_i<0x4E>(kIntMax, a));
    b = max(b, dpp_i<0x4E>(kIntMin, b));
    a = min(a, dpp_i<0x141>(kIntMax, a));
    b = max(b, dpp_i<0x141>(kIntMin, b));
    a = min(a, dpp_i<0x140>(kIntMax, a));
    b = max(b, dpp_i<0x140>(kIntMin, b));
    a = min(a, dpp_i<0x142, 0xa>(kIntMax, a));
    b = max(b, dpp_i<0x142, 0xa>(kIntMin, b));
    a = min(a, dpp_i<0x143, 0xc>(kIntMax, a));
    b = max(b, dpp_i<0x143, 0xc>(kIntMin, b));
    omin = __builtin_bit_cast(float, lane63(a));
    omax = __builtin_bit_cast(float, lane63(b));
}

// Wave minimum of non-negative floats.
__device__ __forceinline__ float wave_min_nonneg(float v)
{
    int a = __builtin_bit_cast(int, v);
    a = min(a, dpp_i<0xB1>(kIntMax, a));
    a = min(a, dpp_i<0x4E>(kIntMax, a));
    a = min(a, dpp_i<0x141>(kIntMax, a));
    a = min(a, dpp_i<0x140>(kIntMax, a));
    a = min(a, dpp_i<0x142, 0xa>(kIntMax, a));
    a = min(a, dpp_i<0x143, 0xc>(kIntMax, a));
    return __builtin_bit_cast(float, lane63(a));
}

// Read-only scene data fetched with wave-uniform addresses: the constant
// address space makes these scalar loads.
template <typename T>
using const_ptr = const __attribute__((address_space(4))) T*;

template <typename T>
__device__ __forceinline__ const_ptr<float> as_const(const T* p)
{
    return (const_ptr<float>)(reinterpret_cast<const float*>(p));
}

// Element i of a float4 array seen as floats.
__device__ __forceinline__ float4 ld4(const_ptr<float> p, int i)
{
    return make_float4(p[4 * i], p[4 * i + 1], p[4 * i + 2], p[4 * i + 3]);
}

// Smallest squared distance from (x, y) to the 8 points of a waypoint chunk
// (padded at the end with points at infinity).
__device__ __forceinline__ float chunk_min(const float4 (&q)[kChunkQ], float x, float y)
{
    float m = INFINITY;
#pragma unroll
    for (int u = 0; u < kChunkQ; ++u) {
        const float dx0 = x - q[u].x, dy0 = y - q[u].y;
        const float dx1 = x - q[u].z, dy1 = y - q[u].w;
        m = fminf(m, fmaf(dy0, dy0, dx0 * dx0));
        m = fminf(m, fmaf(dy1, dy1, dx1 * dx1));
    }
    return m;
}

// Scans the chunks whose bits are set in m (ascending, kChunkTrip per memory
// round trip, read from global memory with scalar loads): best = smallest
// squared distance, bch = first chunk that attains it.  A short last group
// repeats its first chunk: the repeat cannot be strictly smaller, so nothing
// changes, and the group's loads are issued together without a branch
// between them.
__device__ __forceinline__ void scan_chunks(const_ptr<float> wp4, int base, unsigned long long m,
                                            float x, float y, float& best, int& bch)
{
    while (m) {
        int c[kChunkTrip];
        c[0] = base + __builtin_ctzll(m);
        m &= m - 1;
#pragma unroll
        for (int i = 1; i < kChunkTrip; ++i) {
            c[i] = m ? base + __builtin_ctzll(m) : c[0];
            m &= m - 1;
        }
        float4 q[kChunkTrip][kChunkQ];
#pragma unroll
        for (int i = 0; i < kChunkTrip; ++i)
#pragma unroll
            for (int u = 0; u < kChunkQ; ++u) q[i][u] = ld4(wp4, c[i] * kChunkQ + u);
#pragma unroll
        for (int i = 0; i < kChunkTrip; ++i) {
            const float mi = chunk_min(q[i], x, y);
            if (mi < best) {
                best = mi;
                bch = c[i];
            }
        }
    }
}

// Index of the first point of chunk bch at squared distance best from
// (x, y): together with scan_chunks this is the lowest index attaining the
// minimum, as in the sequential scan (index 0 when no distance is finite).
__device__ __forceinline__ int chunk_argmin(const float2* wxy, int bch, float best, float x,
                                            float y)
{
    if (!(best < INFINITY)) return 0;
    const float4* p = reinterpret_cast<const float4*>(wxy) + bch * kChunkQ;
    int bj = bch * kChunk;
#pragma unroll
    for (int u = kChunkQ - 1; u >= 0; --u) {
        const float4 q = ld_g(p, u);
#pragma unroll
        for (int h = 1; h >= 0; --h) {
            const float dx = x - (h ? q.z : q.x);
            const float dy = y - (h ? q.w : q.y);
            if (fmaf(dy, dy, dx * dx) == best) bj = bch * kChunk + 2 * u + h;
        }
    }
    return bj;
}

// Per-lane culling data that stays in registers through the rollout: the
// bounding box of chunk `lane` and obstacle circle `lane` (the first 64 of
// each; larger scenes read the rest from global memory).
struct LaneCull {
    float4 box;   // (x_lo, x_hi, y_lo, y_hi) of chunk lane; empty past the end
    float4 cpv;   // circle lane (x, y, vx, vy); at infinity past the end
    float crr;    // its radius plus the ego radius
};

__device__ __forceinline__ float4 lane_chunk_box(const InstDesc& d, int lane)
{
    const int n_ch = (d.n_wp + kChunk - 1) / kChunk;
    return lane < n_ch ? ld_g(d.wp_box, lane) : make_float4(INFINITY, -INFINITY, INFINITY, -INFINITY);
}
__device__ __forceinline__ void lane_circle(const InstDesc& d, int lane, float4& cpv, float& crr)
{
    cpv = lane < d.n_c ? ld_g(d.c_pv, lane) : make_float4(INFINITY, INFINITY, 0.0f, 0.0f);
    crr = lane < d.n_c ? ld_g(d.c_rr, lane) : 0.0f;
}

// Sec. III input cost of one step: q_u = w_effort (alpha eps.eps + U.eps + U.U / 2).
__device__ __forceinline__ float input_cost(const InstDesc& d, float Ua, float Ud, float ea, float ed)
{
    return d.w_effort * (d.alpha * fmaf(ea, ea, ed * ed) + fmaf(Ua, ea, Ud * ed) +
                         0.5f * fmaf(Ua, Ua, Ud * Ud));
}

// The stage cost of stage_cost, with the two scans restricted to what can
// matter for this wave (all 64 lanes call it; `act` lanes are evaluated).
// The result is bit-identical to the full scans:
//  * waypoints: two bounds on every lane's nearest distance^2 -- the
//    smallest over chunks of the largest distance^2 between the wave's
//    position box and the chunk box, and the largest over lanes of the
//    lane's own distance^2 (same arithmetic as the scan) to three waypoints
//    ahead of its previous closest chunk; UB is the smaller.  A chunk whose
//    smallest distance^2 to the wave box exceeds UB (with a relative margin
//    far above float32 rounding) holds no candidate, and the remaining
//    chunks are scanned in index order, so ties resolve exactly as in the
//    full scan;
//  * circles: a circle whose centre, swept over the wave's time range, stays
//    farther than max(d_safe) + r_c + r_ego from the box of the wave's ego
//    circles cannot make c_safe positive for any lane, so it is skipped.
// Lanes whose position or speed is not finite are left out of the wave box:
// their own cost is not finite under either scan.  A safety distance beyond
// float32 counts as +inf, near which every circle is; one that is not a number
// costs nothing under either scan.  The scene is read from global memory
// (wave-uniform candidates through the scalar cache); own_d2 is the lane's
// squared distance to the nearest of three waypoints ahead of its previous
// closest chunk (+inf without one), formed by the caller, and vref0 the
// reference speed of waypoint 0.  One function: as two, one for each scan, more
// of what both keep in scalar registers was spilled (lane reads in the 16-lane
// kernel 774 against 459; 8192 x 100, 60 circles 37.0 -> 34.8 us, 16384 x 600, 12
// circles 369 -> 337).
template <int NE>
__device__ __forceinline__ float stage_cost_culled(const InstDesc& d, float own_d2,
                                                   float vref0, const LaneCull& lc,
                                                   bool vref_uniform, bool act,
                                                   int& seed, float x, float y,
                                                   float c, float sn, float v, float Ua, float Ud,
                                                   float ea, float ed, int t, int t_lo, int t_hi,
                                                   float th, float xp, float yp)
{
    const int lane = threadIdx.x & 63;
    const float ds = fmaf(d.d_safe_c, v, d.d_safe_0);
    const bool inc = act && isfinite(x) && isfinite(y) && isfinite(v);
    const WaveBox wb = wave_box(inc, x, y, fmaxf(ds, -kNowhere));

    // ---- waypoints
    const int n_ch = (d.n_wp + kChunk - 1) / kChunk;
    const const_ptr<float> wp4 = as_const(d.wp_xy);
    float best = INFINITY;
    int bch = 0;
    auto far2 = [&](const float4& b) {  // largest distance^2, wave box to chunk box
        const float dx = fmaxf(wb.xhi - b.x, b.y - wb.xlo);
        const float dy = fmaxf(wb.yhi - b.z, b.w - wb.ylo);
        return fmaf(dy, dy, dx * dx);
    };
    auto near2 = [&](const float4& b) {  // smallest distance^2, wave box to chunk box
        const float gx = fmaxf(fmaxf(b.x - wb.xhi, wb.xlo - b.y), 0.0f);
        const float gy = fmaxf(fmaxf(b.z - wb.yhi, wb.ylo - b.w), 0.0f);
        return fmaf(gy, gy, gx * gx);
    };
    // A second bound from the lane itself: its distance^2 to three waypoints
    // ahead of the chunk it was closest to at its previous step (seed), the
    // largest over the lanes of the wave; lanes without a seed give +inf.  (A
    // chunk must lie below the threshold: one at +inf, like the empty boxes past
    // the last chunk, is never a candidate, even where the threshold is +inf.)
    const float own = inc ? own_d2 : 0.0f;
    if (n_ch <= 64) {
        float ub_box, ub_own;
        wave_minmax_nonneg(far2(lc.box), own, ub_box, ub_own);
        const float thr = fmaf(fminf(ub_box, ub_own), 1.0f + 1e-5f, 1e-6f);
        scan_chunks(wp4, 0, __ballot(near2(lc.box) < thr), x, y, best, bch);
    } else {
        const float4 empty = make_float4(INFINITY, -INFINITY, INFINITY, -INFINITY);
        float ub, ub_own;
        wave_minmax_nonneg(far2(lc.box), own, ub, ub_own);
        ub = fminf(ub, ub_own);
        for (int base = 64; base < n_ch; base += 64)
            ub = fminf(ub, wave_min_nonneg(far2(base + lane < n_ch ? ld_g(d.wp_box, base + lane) : empty)));
        const float thr = fmaf(ub, 1.0f + 1e-5f, 1e-6f);
        scan_chunks(wp4, 0, __ballot(near2(lc.box) < thr), x, y, best, bch);
        for (int base = 64; base < n_ch; base += 64) {
            const float4 b = base + lane < n_ch ? ld_g(d.wp_box, base + lane) : empty;
            scan_chunks(wp4, base, __ballot(near2(b) < thr), x, y, best, bch);
        }
    }
    if (best < INFINITY) seed = bch;
    // the closest index, needed for its reference speed (unless every
    // waypoint has the same one) and for its yaw
    const bool need_idx = !vref_uniform || d.w_yaw != 0.0f;
    const int bj = need_idx ? chunk_argmin(d.wp_xy, bch, best, x, y) : 0;
    const float vref = vref_uniform ? vref0 : ld_g(d.wp_vref, bj);
    const float ext = extra_terms<true>(d, d.wp_xy, d.wp_yaw, bj, x, y, th, xp, yp);
    const float dv = v - vref;
    float cost = fmaf(d.w_track, best, fmaf(d.w_speed, dv * dv, input_cost(d, Ua, Ud, ea, ed)));

    // ---- obstacle circles
    if (NE > 0) {
        float ex[NE > 0 ? NE : 1], ey[NE > 0 ? NE : 1];
#pragma unroll
        for (int e = 0; e < NE; ++e) {
            ex[e] = fmaf(d.ego_off[e], c, x);
            ey[e] = fmaf(d.ego_off[e], sn, y);
        }
        const float exlo = wb.xlo - d.ego_ext, exhi = wb.xhi + d.ego_ext;
        const float eylo = wb.ylo - d.ego_ext, eyhi = wb.yhi + d.ego_ext;
        const float tau_lo = (float)(t_lo + 1) * d.dt;
        const float tau_hi = (float)(t_hi + 1) * d.dt;
        const float tau = (float)(t + 1) * d.dt;
        auto close = [&](const float4& p, float rr) {
            const float xa = fmaf(tau_lo, p.z, p.x), xb = fmaf(tau_hi, p.z, p.x);
            const float ya = fmaf(tau_lo, p.w, p.y), yb = fmaf(tau_hi, p.w, p.y);
            const float gx = fmaxf(fmaxf(fminf(xa, xb) - exhi, exlo - fmaxf(xa, xb)), 0.0f);
            const float gy = fmaxf(fmaxf(fminf(ya, yb) - eyhi, eylo - fmaxf(ya, yb)), 0.0f);
            // collision-only: only circles that can reach an ego circle matter
            const float lim = (d.coll_only ? 0.0f : wb.dsmax) + rr + 0.01f;
            return lim > 0.0f && fmaf(gy, gy, gx * gx) < lim * lim;
        };
        const const_ptr<float> cpv = as_const(d.c_pv);
        const const_ptr<float> crr = as_const(d.c_rr);
        float d_obj = INFINITY;
        for (int base = 0; base < d.n_c; base += 64) {
            bool need;
            if (base == 0) {
                need = close(lc.cpv, lc.crr);
            } else {
                need = base + lane < d.n_c && close(ld_g(d.c_pv, base + lane), ld_g(d.c_rr, base + lane));
            }
            unsigned long long m = __ballot(need);
            while (m) {
                // four candidates per round trip, loads issued together; a
                // short last group repeats its first candidate (the minimum
                // is unchanged)
                int idx[4];
                idx[0] = base + __builtin_ctzll(m);
                m &= m - 1;
#pragma unroll
                for (int u = 1; u < 4; ++u) {
                    idx[u] = m ? base + __builtin_ctzll(m) : idx[0];
                    m &= m - 1;
                }
                float4 p[4];
                float rr[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    p[u] = ld4(cpv, idx[u]);
                    rr[u] = crr[idx[u]];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) d_obj = fminf(d_obj, circle_gap<NE>(ex, ey, p[u], rr[u], tau));
            }
        }
        cost = fmaf(d.w_coll, safe_cost(d, ds, d_obj), cost);
    }
    return cost + ext;
}

// ----------------------------------------------------------------------------
// The same scans restricted row by row: at 16 lanes per sample a DPP row is
// one sample's block of 16 steps, and its box is far smaller than that of the
// wave's four samples, which drift apart along the horizon (stress scene:
// 2.7 circles and 4.2 chunks a row against 47 and 13 a wave; sine lane 2.4
// and 3.1 against 8.6 and 5.6).  Every row walks its own candidates, read
// from LDS, so a wave takes as many steps as its longest row.  Exactness is
// as above, with the row in place of the wave.
// ----------------------------------------------------------------------------

// Bits of the lane's own row in the ballot b.
__device__ __forceinline__ unsigned row_bits(unsigned long long b)
{
    const unsigned w = (threadIdx.x & 32) ? (unsigned)(b >> 32) : (unsigned)b;
    return (w >> (threadIdx.x & 16)) & 0xffffu;
}

// Row reductions of five values, two to their minima and three to their
// maxima, in every lane of the row.  Written out with the float minimum and
// maximum, which pass over a value that is not a number (a safety distance, the
// ego centres of a heading beyond float32): the compiler would quiet every moved
// value first, and the integer keys of the reductions above cost their way there
// and back (with the waves without columns leaving early: 6093 -> 5640 vector
// instructions per four samples of the sine lane, 26.5 -> 24.8 us an iteration).
// Four instructions lie between an instruction and the next that moves its
// result, as a lane move needs two.
__device__ __forceinline__ void row_reduce5(float& a, float& b, float& c, float& e, float& f)
{
#define MPPI_STAGE(CTRL)                                              \
    "v_min_f32_dpp %0, %0, %0 " CTRL " row_mask:0xf bank_mask:0xf\n" \
    "v_min_f32_dpp %1, %1, %1 " CTRL " row_mask:0xf bank_mask:0xf\n" \
    "v_max_f32_dpp %2, %2, %2 " CTRL " row_mask:0xf bank_mask:0xf\n" \
    "v_max_f32_dpp %3, %3, %3 " CTRL " row_mask:0xf bank_mask:0xf\n" \
    "v_max_f32_dpp %4, %4, %4 " CTRL " row_mask:0xf bank_mask:0xf\n"
    asm volatile("s_nop 1\n"
                 MPPI_STAGE("quad_perm:[1,0,3,2]")
                 MPPI_STAGE("quad_perm:[2,3,0,1]")
                 MPPI_STAGE("row_half_mirror")
                 MPPI_STAGE("row_mirror")
                 : "+v"(a), "+v"(b), "+v"(c), "+v"(e), "+v"(f));
#undef MPPI_STAGE
}

// Tracking and speed cost added to the input cost q, as stage_cost_culled.
// wxy: the waypoints in LDS, padded to whole chunks with points at infinity;
// box[i]: chunk (lane mod 16) + 16 i (instances of at most 64 chunks);
// (xg, yg) and base: the position at the lane's previous step and the
// waypoint it was closest to there, from which the lane's own bound takes the
// waypoint that the distance travelled since leads to (with it the rows scan
// what the true minima would leave them to).
__device__ __forceinline__ float path_cost_rows(const InstDesc& d, const float4* wxy, const float4 (&box)[4],
                                                float inv_sp, bool act, float vref0, bool vref_uniform,
                                                float& xg, float& yg, int& base, float x, float y,
                                                float v, float q, float th, float xp, float yp, float& ext)
{
    const int r = threadIdx.x & 15;
    const int n_ch = (d.n_wp + kChunk - 1) / kChunk;
    const bool inc = act && isfinite(x) && isfinite(y);
    float own;
    {
        const float gx = x - xg, gy = y - yg;
        const float step = __builtin_amdgcn_sqrtf(fmaf(gy, gy, gx * gx)) * inv_sp;
        const int j = (int)fminf(fmaxf((float)base + step, 0.0f), (float)(d.n_wp - 1));
        const float2 w = reinterpret_cast<const float2*>(wxy)[j];
        const float dx = x - w.x, dy = y - w.y;
        own = inc ? fmaf(dy, dy, dx * dx) : 0.0f;
    }
    float xlo = inc ? x : INFINITY, ylo = inc ? y : INFINITY;
    float xhi = inc ? x : -INFINITY, yhi = inc ? y : -INFINITY;
    row_reduce5(xlo, ylo, xhi, yhi, own);
    const float thr = fmaf(own, 1.0f + 1e-5f, 1e-6f);
    // smallest distance^2, row box to chunk box, below the threshold (never the
    // empty boxes past the last chunk, at +inf)
    auto near = [&](const float4& bx) {
        const float gx = fmaxf(fmaxf(bx.x - xhi, xlo - bx.y), 0.0f);
        const float gy = fmaxf(fmaxf(bx.z - yhi, ylo - bx.w), 0.0f);
        return fmaf(gy, gy, gx * gx) < thr;
    };
    // first and last candidate chunk of the row (those between are scanned too)
    int lo = 0x7fffffff, hi = -1;
    auto take = [&](int i, bool n) {
        const unsigned m = row_bits(__ballot(n));
        lo = m ? min(lo, 16 * i + __builtin_ctz(m)) : lo;
        hi = m ? 16 * i + 31 - __builtin_clz(m) : hi;
    };
    if (n_ch <= 64) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (16 * i < n_ch) take(i, near(box[i]));
    } else {
        for (int i = 0; 16 * i < n_ch; ++i) {
            const int ch = 16 * i + r;
            take(i, ch < n_ch && near(ld_g(d.wp_box, min(ch, n_ch - 1))));
        }
    }
    lo = max(min(lo, hi), 0);
    float best = INFINITY;
    int bch = 0;
    float4 p[kChunkQ];
    const float4* at = wxy + lo * kChunkQ;
#pragma unroll
    for (int u = 0; u < kChunkQ; ++u) p[u] = at[u];
    bool more;
    int ch = lo;
    do {
        // the next chunk is read while this one is scanned; a row that is
        // done repeats its last
        more = ch < hi;
        const int cn = more ? ch + 1 : ch;
        at = wxy + cn * kChunkQ;
        float4 n[kChunkQ];
#pragma unroll
        for (int u = 0; u < kChunkQ; ++u) n[u] = at[u];
        const float mi = chunk_min(p, x, y);
        if (mi < best) {
            best = mi;
            bch = ch;
        }
        ch = cn;
#pragma unroll
        for (int u = 0; u < kChunkQ; ++u) p[u] = n[u];
    } while (__ballot(more) != 0ull);
    xg = x;
    yg = y;
    base = bch * kChunk + kChunk / 2;
    // the closest index, needed for its reference speed (unless every
    // waypoint has the same one) and for its yaw
    int bj = 0;
    if (!vref_uniform || d.w_yaw != 0.0f) {
        if (best < INFINITY) {
            bj = bch * kChunk;
            at = wxy + bch * kChunkQ;
#pragma unroll
            for (int u = kChunkQ - 1; u >= 0; --u) {
                const float4 w = at[u];
#pragma unroll
                for (int h = 1; h >= 0; --h) {
                    const float dx = x - (h ? w.z : w.x);
                    const float dy = y - (h ? w.w : w.y);
                    if (fmaf(dy, dy, dx * dx) == best) bj = bch * kChunk + 2 * u + h;
                }
            }
        }
    }
    const float vref = vref_uniform ? vref0 : ld_g(d.wp_vref, bj);
    ext = extra_terms<true>(d, d.wp_xy, d.wp_yaw, bj, x, y, th, xp, yp);
    const float dv = v - vref;
    return fmaf(d.w_track, best, fmaf(d.w_speed, dv * dv, q));
}

// Circles in LDS for the scan by rows: entry e at 2e is (x, y, vx, vy); the
// radius follows, then circle_reach.  Entry 0 is a circle at infinity.
__device__ __forceinline__ void put_circle(float4* list, int e, const float4& p, float rr, float reach)
{
    list[2 * e] = p;
    list[2 * e + 1] = make_float4(rr, reach, 0.0f, 0.0f);
}
// A box of ego circle centres as centre and half extent (widened by the
// rounding of forming them), and the largest distance from a centre at which an
// obstacle circle counts.  A box without centres runs from kNowhere to -kNowhere:
// its half extent is so far below zero that nothing is near it.
struct EgoBox {
    float xc, yc, xh, yh, ds;
};
__device__ __forceinline__ EgoBox ego_box(const InstDesc& d, const WaveBox& b)
{
    EgoBox o;
    o.xc = 0.5f * (b.xlo + b.xhi);
    o.yc = 0.5f * (b.ylo + b.yhi);
    o.xh = fmaf(1e-6f, fabsf(b.xlo) + fabsf(b.xhi), 0.5f * (b.xhi - b.xlo));
    o.yh = fmaf(1e-6f, fabsf(b.ylo) + fabsf(b.yhi), 0.5f * (b.yhi - b.ylo));
    o.ds = d.coll_only ? 0.0f : b.dsmax;
    return o;
}
// Whether a circle (at (ox, oy) at the middle of the block) can come within
// the largest safety distance of a centre in the box (an empty box: no; a box
// whose centres are not numbers or a limit below zero: perhaps yes, which costs
// a look at the circle and no more).
__device__ __forceinline__ bool circle_near(const EgoBox& b, float ox, float oy, float reach)
{
    const float gx = fmaxf(fabsf(ox - b.xc) - b.xh, 0.0f);
    const float gy = fmaxf(fabsf(oy - b.yc) - b.yh, 0.0f);
    const float lim = b.ds + reach;
    return fmaf(gy, gy, gx * gx) < lim * lim;
}

// d_obj lowered by the circles of the list that bit i of m (entry e0 + i)
// names, every row its own; the next entry is read while one is evaluated.
template <int NE>
__device__ __forceinline__ float row_circle_scan(const float4* list, int e0, unsigned m,
                                                 const float (&ex)[NE > 0 ? NE : 1],
                                                 const float (&ey)[NE > 0 ? NE : 1], float tau,
                                                 float d_obj)
{
    auto at = [&](unsigned bits) { return list + 2 * (bits ? e0 + __builtin_ctz(bits) : 0); };
    if (__ballot(m != 0u) == 0ull) return d_obj;
    const float4* q = at(m);
    float4 p = q[0];
    float rr = q[1].x;
    do {
        m &= m - 1u;
        q = at(m);
        const float4 pn = q[0];
        const float rn = q[1].x;
        d_obj = fminf(d_obj, circle_gap<NE>(ex, ey, p, rr, tau));
        p = pn;
        rr = rn;
    } while (__ballot(m != 0u) != 0ull);
    return d_obj;
}

// What a wave keeps for the scan by rows: of at most kListedCircles circles all
// are in the list, and lane i of a row tests circles i, i + 16, i + 32 and
// i + 48 (p, reach); of more, lane i keeps group i (p[0] its positions, p[1] its
// velocities, reach[0]), and every span lists the circles of the near groups
// that are near the wave's box.
struct RowCircles {
    float4 p[4];
    float reach[4];
};
static_assert(kMaxCircles <= 64 * kCircleGroup && kListedCircles == 64, "a lane for every group");
__device__ __forceinline__ void row_circles_init(const InstDesc& d, float4* list, RowCircles& rc)
{
    const int lane = threadIdx.x & 63, r = lane & 15;
    const float4 far = make_float4(INFINITY, INFINITY, 0.0f, 0.0f);
    if (lane == 0) put_circle(list, 0, far, 0.0f, 0.0f);
    if (d.n_c > kListedCircles) {
        const int g = min(lane, circle_groups(d.n_c) - 1);
        rc.p[0] = ld_g(d.c_grp, 3 * g);
        rc.p[1] = ld_g(d.c_grp, 3 * g + 1);
        rc.reach[0] = ld_g(reinterpret_cast<const float*>(d.c_grp + 3 * g + 2), 0);
        return;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int c = r + 16 * i;
        rc.p[i] = c < d.n_c ? ld_g(d.c_pv, c) : far;
        const float rr = c < d.n_c ? ld_g(d.c_rr, c) : 0.0f;
        rc.reach[i] = c < d.n_c ? ld_g(d.c_reach, c) : 0.0f;
        if (lane < 16) put_circle(list, 1 + c, rc.p[i], rr, rc.reach[i]);
    }
}

// Obstacle cost before its weight of the lane's state at the end of step
// t0 + r of the block that starts at step t0.
template <int NE>
__device__ __forceinline__ float obstacle_cost_rows(const InstDesc& d, float4* list, const RowCircles& rc,
                                                    bool act, float x, float y, float th, float v, int t0)
{
    const int lane = threadIdx.x & 63, r = lane & 15;
    const float ds = fmaf(d.d_safe_c, v, d.d_safe_0);
    const bool inc = act && isfinite(x) && isfinite(y);
    const float c = __cosf(th), sn = __sinf(th);
    float ex[NE > 0 ? NE : 1], ey[NE > 0 ? NE : 1];
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        ex[e] = fmaf(d.ego_off[e], c, x);
        ey[e] = fmaf(d.ego_off[e], sn, y);
    }
    float xl = ex[0], xh = ex[0], yl = ey[0], yh = ey[0];
#pragma unroll
    for (int e = 1; e < NE; ++e) {
        xl = fminf(xl, ex[e]);
        xh = fmaxf(xh, ex[e]);
        yl = fminf(yl, ey[e]);
        yh = fmaxf(yh, ey[e]);
    }
    WaveBox row;
    row.xlo = inc ? xl : kNowhere;
    row.ylo = inc ? yl : kNowhere;
    row.xhi = inc ? xh : -kNowhere;
    row.yhi = inc ? yh : -kNowhere;
    row.dsmax = inc ? ds : -kNowhere;
    row_reduce5(row.xlo, row.ylo, row.xhi, row.yhi, row.dsmax);
    const EgoBox rb = ego_box(d, row);
    // the middle of the span's times (of a span that starts before the horizon
    // at the earliest its start: within 7.5 steps of every step it has)
    const float tau_m = fmaxf(((float)t0 + 8.5f) * d.dt, 0.0f);
    const float tau = (float)(t0 + r + 1) * d.dt;
    float d_obj = INFINITY;
    if (d.n_c <= kListedCircles) {
        unsigned m[2] = {0u, 0u};
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (16 * u < d.n_c) {
                const bool n = circle_near(rb, fmaf(tau_m, rc.p[u].z, rc.p[u].x),
                                           fmaf(tau_m, rc.p[u].w, rc.p[u].y), rc.reach[u]);
                m[u / 2] |= row_bits(__ballot(n)) << (16 * (u & 1));
            }
        d_obj = row_circle_scan<NE>(list, 1, m[0], ex, ey, tau, d_obj);
        if (d.n_c > 32) d_obj = row_circle_scan<NE>(list, 33, m[1], ex, ey, tau, d_obj);
        return safe_cost(d, ds, d_obj);
    }
    const WaveBox wbox = wave_box_of_rows({fkey(row.xlo), fkey(row.ylo), fkey(row.xhi), fkey(row.yhi),
                                           fkey(fmaxf(row.dsmax, -kNowhere))});  // (a number)
    const EgoBox wb = ego_box(d, wbox);
    int cnt = 0;
    auto flush = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int j = 0; j < cnt; j += 32) {
            unsigned m = 0u;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int e = j + 16 * u + r;
                const float4* q = list + 2 * (1 + e);  // (past the last entry: within the list)
                const float4 p = q[0];
                const bool n = circle_near(rb, fmaf(tau_m, p.z, p.x), fmaf(tau_m, p.w, p.y), q[1].y) && e < cnt;
                m |= row_bits(__ballot(n)) << (16 * u);
            }
            d_obj = row_circle_scan<NE>(list, 1 + j, m, ex, ey, tau, d_obj);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        cnt = 0;
    };
    // groups near the wave's box, by lanes (tau_m >= 0: a group's positions lie
    // between its least with the least velocity and its greatest with the
    // greatest; the margin is the box's)
    const float gx = fmaxf(fmaxf(fmaf(tau_m, rc.p[1].x, rc.p[0].x) - (wb.xc + wb.xh),
                                 (wb.xc - wb.xh) - fmaf(tau_m, rc.p[1].y, rc.p[0].y)), 0.0f);
    const float gy = fmaxf(fmaxf(fmaf(tau_m, rc.p[1].z, rc.p[0].z) - (wb.yc + wb.yh),
                                 (wb.yc - wb.yh) - fmaf(tau_m, rc.p[1].w, rc.p[0].w)), 0.0f);
    const float glim = wb.ds + rc.reach[0];
    unsigned long long groups =
        __ballot(lane < circle_groups(d.n_c) && fmaf(gy, gy, gx * gx) < glim * glim);
    // their circles, four groups at a time
    while (groups) {
        int mine = -1;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int g = groups ? (int)__builtin_ctzll(groups) : -1;
            groups &= groups - 1;
            mine = (lane >> 4) == u ? g : mine;
        }
        const int c = mine * kCircleGroup + r;
        const bool in = mine >= 0 && c < d.n_c;
        const int i = in ? c : 0;
        const float4 p = ld_g(d.c_pv, i);
        const float rr = ld_g(d.c_rr, i);
        const float reach = ld_g(d.c_reach, i);
        const bool n = in && circle_near(wb, fmaf(tau_m, p.z, p.x), fmaf(tau_m, p.w, p.y), reach);
        const unsigned long long b = __ballot(n);
        const int add = __builtin_popcountll(b);
        if (cnt + add > 64) flush();
        if (n)
            put_circle(list, 1 + cnt + __builtin_amdgcn_mbcnt_hi((unsigned)(b >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)b, 0u)),
                       p, rr, reach);
        cnt += add;
    }
    flush();
    return safe_cost(d, ds, d_obj);
}

// A float64 value of another lane by DPP (two 32-bit moves).
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned int)lo);
}

// A float64 value of one lane, wave-uniform (two lane reads into scalar
// registers).
__device__ __forceinline__ double lane_d(double v, int lane)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)b, lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned int)lo);
}

// Butterfly reductions over the 64 lanes of a wave (every lane active; every
// lane ends with the same value): lane pairs and quad halves by quad
// permutes; then, each quad holding one value, the half-row mirror pairs
// each quad with the other quad of its half-row, and the row mirror each
// half-row with the other half; the four row values, read into scalar
// registers, are combined as (row 0 with row 1) with (row 2 with row 3) --
// the value the cross-row butterfly gives in every lane.
__device__ __forceinline__ double wave_sum(double v)
{
    v += dpp_d<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v += dpp_d<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    v += dpp_d<0x141>(v);  // row_half_mirror
    v += dpp_d<0x140>(v);  // row_mirror
    return (lane_d(v, 0) + lane_d(v, 16)) + (lane_d(v, 32) + lane_d(v, 48));
}

__device__ __forceinline__ double wave_min(double v)
{
    v = fmin(v, dpp_d<0xB1>(v));
    v = fmin(v, dpp_d<0x4E>(v));
    v = fmin(v, dpp_d<0x141>(v));
    v = fmin(v, dpp_d<0x140>(v));
    return fmin(fmin(lane_d(v, 0), lane_d(v, 16)), fmin(lane_d(v, 32), lane_d(v, 48)));
}

// v plus the value of the lane 16 (32) apart, the same in both lanes of the
// pair.  With both operands equal, the gfx950 permlane swap leaves each lane
// its own value in one result and its partner's in the other (which is
// which depends on the lane), so their sum is the pair's sum either way.
__device__ __forceinline__ double add_lanes_16_apart(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    const double x = __builtin_bit_cast(double, ((long long)hi[0] << 32) | (long long)lo[0]);
    const double y = __builtin_bit_cast(double, ((long long)hi[1] << 32) | (long long)lo[1]);
    return x + y;
}
__device__ __forceinline__ double add_lanes_32_apart(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)b, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(b >> 32), (unsigned)(b >> 32), false, false);
    const double x = __builtin_bit_cast(double, ((long long)hi[0] << 32) | (long long)lo[0]);
    const double y = __builtin_bit_cast(double, ((long long)hi[1] << 32) | (long long)lo[1]);
    return x + y;
}


// State of a sample at the start of a block of G steps (the same in the G
// lanes of its group).
struct WalkState {
    float x, y, th, v;
    float delta;  // steering angle (5-state model only)
};
// Control of one step of one sample after the state-independent part of the
// noise check.
struct StepControl {
    float a, dl;  // acceleration; steering angle (5-state model: steering rate)
    float tn;     // the angle's tangent (5-state model: the rate)
};
// What one step of one sample reaches.
struct StepState {
    float x, y, th, v;  // the state after the step
    float a;            // the applied acceleration
    float xp, yp;       // the position before it (set for c_target only)
};

// Control of step t0 + r of sample k, drawn by lane r of the sample's group
// of G; U: the step's nominal control; held: the Philox words kept from the
// first block of a pair for the second.
template <int G, bool M5>
__device__ __forceinline__ StepControl block_controls(const InstDesc& d, int k, int t0, int r,
                                                      int blk, unsigned long long n_iter, float2 Um,
                                                      uint4& held)
{
    StepControl c;
    // This lane's step: perturbation, the state-independent part of the
    // noise check (control bounds) and -- for the steering-angle control --
    // its tangent.  With the 5-state model the second control is the
    // steering rate.
    // One Philox call gives the words of two consecutive steps.  With
    // G >= 2 lanes per sample the calls of two blocks are made together
    // in the first of them: lane 2i holds step pair i of that block and
    // lane 2i + 1 pair i of the next, and each lane takes its step's two
    // words from itself or its neighbour (quad-permute DPP).  Lanes
    // outside the horizon draw the words of their own (unused) steps.
    float2 em;
    if (G == 1) {
        em = draw_noise(d, k, min(max(t0 + r, 0), d.T - 1), n_iter);
    } else {
        const bool second = (blk & 1) != 0;
        if (!second) held = noise_words(d, k, t0 / 2 + ((r & 1) ? G / 2 : 0) + (r >> 1), n_iter);
        uint32_t ra, rw;
        if (!second) {  // odd lanes take the odd-step words of the even lane below
            const uint32_t nz = (uint32_t)dpp_i<0xA0>(0, (int)held.z);
            const uint32_t nw = (uint32_t)dpp_i<0xA0>(0, (int)held.w);
            ra = (r & 1) ? nz : held.x;
            rw = (r & 1) ? nw : held.y;
        } else {        // even lanes take the even-step words of the odd lane above
            const uint32_t nx = (uint32_t)dpp_i<0xF5>(0, (int)held.x);
            const uint32_t ny = (uint32_t)dpp_i<0xF5>(0, (int)held.y);
            ra = (r & 1) ? held.z : nx;
            rw = (r & 1) ? held.w : ny;
        }
        em = noise_from_words(d, ra, rw);
    }
    c.a = fminf(fmaxf(Um.x + em.x, d.a_min), d.a_max);
    c.dl = fminf(fmaxf(Um.y + em.y, d.d_min), d.d_max);
    c.tn = M5 ? c.dl : __tanf(c.dl);
    return c;
}

// One block of G steps, lane r of a sample's group taking step t0 + r with
// control c: its state after the step in o, the sample's state at the end of
// the block in w.
template <int G, bool M5>
__device__ __forceinline__ void walk_block(const InstDesc& d, const StepControl& c, int t0, int r,
                                           WalkState& w, StepState& o)
{
    const int gbase = threadIdx.x & ~(G - 1);  // first lane of this sample's group
    const bool lead = t0 + r < 0;  // before the horizon: no step, no increment
    // The lane's step within the block, opaque to the compiler so that the
    // per-step "own step" tests stay in the loop as vector compares
    // instead of G hoisted scalar masks (which exhaust the SGPRs).
    int rb = r;
    asm volatile("" : "+v"(rb));
    // Speed before the own step.  The noise check caps the acceleration
    // so that v <= v_max and applies the braking bound last.  With
    // a_min <= 0 and the speed at the block start within v_max the
    // braking bound cannot bind (the cap (v_max - v)/dt is >= 0 >= a_min),
    // and the capped recursion v_{i+1} = min(v_i + dt a_i, v_max) has the
    // closed form
    //   v_r = min(v_0 + S_r, v_max + S_r - max_{1<=k<=r} S_k),
    // S_k = sum_{j<k} dt a_j: a prefix sum and a prefix maximum over the G
    // lanes.  Otherwise (a_min > 0, where the braking bound lifts the speed
    // above v_max whenever the cap falls below a_min, or a wave with a
    // sample above v_max) the G lanes run the recursion step by step
    // (accelerations exchanged PF at a time), each keeping the speed
    // before its own step.  Steps past the horizon (last block) are run
    // too; the lanes that own them are inactive.  Lanes before it (first
    // block) add zero increments, which leave the closed form unchanged
    // (their prefix sums equal v_0 <= v_max's).
    float vr = w.v;
    if (!(d.a_min > 0.0f) && __ballot(w.v > d.v_max) == 0ull) {
        const float sincl = seg_scan<G>(lead ? 0.0f : d.dt * c.a, r);
        const float sr = seg_prev<G>(sincl, r);
        const float qr = seg_scan_max<G>(r >= 1 ? sr : -INFINITY, r);
        vr = fminf(w.v + sr, d.v_max + (sr - qr));
    } else {
        constexpr int PF = G < 4 ? G : 4;
        float apf[PF];
#pragma unroll
        for (int i = 0; i < G; ++i) {
            if (i % PF == 0) {
#pragma unroll
                for (int u = 0; u < PF; ++u)
                    apf[u] = G > 1 ? __shfl(c.a, gbase + i + u, 64) : c.a;
            }
            vr = i == rb ? w.v : vr;
            if (t0 + i >= 0) {
                float a = fminf(apf[i % PF], (d.v_max - w.v) * d.inv_dt);
                a = fmaxf(a, d.a_min);
                w.v = fmaf(d.dt, a, w.v);
            }
        }
    }
    // the own step's applied acceleration (noise check: speed cap,
    // braking bound last) and the speed after it; the block ends at the
    // last lane's
    float ma = fminf(c.a, (d.v_max - vr) * d.inv_dt);
    ma = fmaxf(ma, d.a_min);
    const float mv = fmaf(d.dt, ma, vr);
    o.v = mv;
    o.a = ma;
    w.v = group_last<G>(mv, gbase);
    // Eq. (5), explicit Euler: given the speeds, heading and position are
    // sums of per-step increments, formed by prefix sums over the G lanes
    // of the group (each lane adds its own step's increment).  With the
    // 5-state model the heading turns with the steering angle before the
    // step, itself the sum of the applied rates.
    const float vdt = lead ? 0.0f : vr * d.dt;
    float tn = c.tn;
    float ddel_blk = 0.0f;
    if (M5) {
        const float dincl = seg_scan<G>(lead ? 0.0f : d.dt * c.tn, r);
        tn = __tanf(w.delta + seg_prev<G>(dincl, r));
        ddel_blk = group_last<G>(dincl, gbase);
    }
    const float thincl = seg_scan<G>(vdt * d.inv_L * tn, r);
    const float thb = w.th + seg_prev<G>(thincl, r);  // heading before the own step
    o.th = w.th + thincl;                             // and after it
    const float xincl = seg_scan<G>(vdt * __cosf(thb), r);
    const float yincl = seg_scan<G>(vdt * __sinf(thb), r);
    o.x = w.x + xincl;
    o.y = w.y + yincl;
    // position before this lane's step (for c_target): the previous
    // lane's position after its step, the block start for the first
    o.xp = o.yp = 0.0f;
    if (d.w_target != 0.0f) {
        o.xp = w.x + seg_prev<G>(xincl, r);
        o.yp = w.y + seg_prev<G>(yincl, r);
    }
    // the state at the end of the block (the last lane's), for the next
    w.x += group_last<G>(xincl, gbase);
    w.y += group_last<G>(yincl, gbase);
    w.th += group_last<G>(thincl, gbase);
    if (M5) w.delta += ddel_blk;
}

// Tile partial (total-cost weights): the tile minimum of the samples' costs,
// the float64 exponential weights and their sums, and every column's weighted
// sum of the applied perturbations.  All NT threads call it; Sk is the cost of
// the sample of the lane's group of G, in the first kBlock threads.  red: 64
// doubles, omega: [spb], eps: the tile's LDS copy of its perturbations
// ([2T][spb + 1]) where it has one (staged).
template <int G, int NT>
__device__ __forceinline__ void tile_partials(const InstDesc& d, int tile, float Sk, double* red, double* omega,
                                              const float* eps, bool staged)
{
    constexpr int SPB = kBlock / G;
    const int tid = threadIdx.x;
    const int T = d.T, K = d.K;
    const int r = tid % G, grp = tid / G;
    const int k_base = tile * SPB;
    const int n_valid = min(SPB, K - k_base);
    double* part = d.partials + (size_t)tile * partial_stride(T, 0);
    // wave results through LDS, combined in wave order (two barriers)
    const int wv = tid >> 6;
    const bool mine = NT == kBlock || tid < kBlock;  // (uniform in a wave)
    const bool lane0 = (tid & 63) == 0;
    if (mine) {
        const double wmin = wave_min((double)Sk);
        if (lane0) red[wv] = wmin;
    }
    __syncthreads();
    double m_b = red[0];
#pragma unroll
    for (int i = 1; i < kBlock / 64; ++i) m_b = fmin(m_b, red[i]);
    if (mine) {
        double om = 0.0;
        if (r == 0 && isfinite(m_b) && Sk < INFINITY) om = exp(-((double)Sk - m_b) / d.lambda);
        if (r == 0) omega[grp] = om;
        const double wz = wave_sum(om);
        const double wq = wave_sum(om * om);
        if (lane0) {
            red[4 + wv] = wz;
            red[8 + wv] = wq;
        }
    }
    __syncthreads();  // also orders the omega stores
    double z_b = red[4], q_b = red[8];
#pragma unroll
    for (int i = 1; i < kBlock / 64; ++i) {
        z_b += red[4 + i];
        q_b += red[8 + i];
    }
    // Weighted perturbation sums, one column (step, control) per thread,
    // the float64 weights (the ones Z_b sums) times the float32
    // perturbations, summed in float64 in sample order: from
    // the tile's LDS copy of its perturbations (rows padded by one so
    // that the lanes of a wave read distinct banks) or, when that copy
    // does not fit, from global memory, sixteen loads in flight.
    constexpr int NB = SPB < 16 ? SPB : 16;
    for (int col = tid; col < 2 * T; col += NT) {
        if (staged) {
            const float* e = eps + col * (SPB + 1);
            double acc = 0.0;
            // whole tiles: every LDS read issued before the chain of FMAs
            if (n_valid == SPB) {
                for (int j0 = 0; j0 < SPB; j0 += NB) {
                    double om[NB];
                    float ev[NB];
#pragma unroll
                    for (int u = 0; u < NB; ++u) {
                        om[u] = omega[j0 + u];
                        ev[u] = e[j0 + u];
                    }
#pragma unroll
                    for (int u = 0; u < NB; ++u) acc = fma(om[u], (double)ev[u], acc);
                }
            } else {
                for (int j = 0; j < n_valid; ++j)
                    acc = fma(omega[j], (double)e[j], acc);
            }
            st_g(part, col, acc);
            continue;
        }
        const int t = col >> 1;
        const float* e =
            reinterpret_cast<const float*>(d.eps + (size_t)t * K + k_base) + (col & 1);
        double acc = 0.0;
        for (int i0 = 0; i0 < n_valid; i0 += NB) {
            float ev[NB];
#pragma unroll
            for (int u = 0; u < NB; ++u) ev[u] = (i0 + u < n_valid) ? ld_g(e, 2 * (i0 + u)) : 0.0f;
#pragma unroll
            for (int u = 0; u < NB; ++u)
                if (i0 + u < n_valid) acc = fma(omega[i0 + u], (double)ev[u], acc);
        }
        st_g(part, col, acc);
    }
    if (tid == 0) {
        double* hd = d.partials + partial_heads_offset(T, 0, d.n_tiles) + kHeadDoubles * tile;
        st_g(hd, 0, m_b);
        st_g(hd, 1, z_b);
        st_g(hd, 2, q_b);
        st_g(hd, 3, 0.0);
    }
}

// Per-step weights: the cost-to-go of every sample of the tile in
// float64, then per step the tile minimum, the shifted exponential
// sums and the weighted perturbations (one thread per step, samples
// in index order).  The cost-to-go is summed by segments of steps, G
// threads per sample: each sums its segment from its end back, then
// adds the totals of the later segments, last first.  The cost-to-go
// of step 0 (the total the weights of step 0 are formed from) is also
// written out.  From the tile's LDS copies when they fit, else
// through global memory.
// NT: the workgroup's threads; lds: eps, qs and ss are the tile's copies.
template <int NT, int SPB>
__device__ __forceinline__ void per_step_partials(const InstDesc& d, int tile, const float* eps, float* qs,
                                                  double* ss, bool lds)
{
    constexpr int kSeg = kBlock / SPB;  // segments of a sample's steps
    const int tid = threadIdx.x;
    const int T = d.T, K = d.K;
    const int k_base = tile * SPB;
    const int n_valid = min(SPB, K - k_base);
    double* part = d.partials + (size_t)tile * partial_stride(T, 1);
    __syncthreads();  // the tile's stage costs are stored
    {
        const int j = tid % SPB, p = tid / SPB;
        const int len = (T + kSeg - 1) / kSeg;
        const int ta = min(p * len, T), tb = min(ta + len, T);
        const bool on = j < n_valid && tid < kBlock;
        auto st_ld = [&](int t) {
            return lds ? ss[t * (SPB + 1) + j] : ld_g(d.Stk, (size_t)t * K + k_base + j);
        };
        auto st_st = [&](int t, double v) {
            if (lds) ss[t * (SPB + 1) + j] = v;
            else st_g(d.Stk, (size_t)t * K + k_base + j, v);
        };
        if (on) {
            double acc = 0.0;
            for (int t = tb - 1; t >= ta; --t) {
                acc += lds ? (double)qs[t * (SPB + 1) + j] : (double)ld_g(d.q, (size_t)t * K + k_base + j);
                st_st(t, acc);
            }
        }
        __syncthreads();
        double off = 0.0;
        if (on)
            for (int pp = kSeg - 1; pp > p; --pp)
                if (pp * len < T) off += st_ld(pp * len);
        __syncthreads();  // segment totals are read before they change
        if (on && p < kSeg - 1 && ta < T) {
            for (int t = ta; t < tb; ++t) st_st(t, st_ld(t) + off);
            if (lds && p == 0) st_g(d.Stk, k_base + j, st_ld(0));
        } else if (on && lds && p == 0) {
            st_g(d.Stk, k_base + j, st_ld(0));
        }
    }
    __syncthreads();
    if (lds) {
        // In LDS the three passes spread over the whole workgroup: the
        // per-step minima (one thread per step, kept where the stage
        // costs were), every sample's shifted exponential of every step
        // (written over its cost-to-go), then the sums per step in
        // sample order.
        double* mt = reinterpret_cast<double*>(qs);
        for (int t = tid; t < T; t += NT) {
            double m = INFINITY;
#pragma unroll 4
            for (int j = 0; j < n_valid; ++j) {
                const double v = ss[t * (SPB + 1) + j];
                if (isfinite(v) && v < m) m = v;
            }
            mt[t] = m;
        }
        __syncthreads();
        for (int i = tid; i < T * SPB; i += NT) {
            const int t = i / SPB, j = i % SPB;
            if (j >= n_valid) continue;
            double& sv = ss[t * (SPB + 1) + j];
            const double m = mt[t], v = sv;
            sv = isfinite(m) && isfinite(v) ? exp(-(v - m) / d.lambda) : 0.0;
        }
        __syncthreads();
        for (int t = tid; t < T; t += NT) {
            double z = 0.0, qq = 0.0, na = 0.0, nd = 0.0;
#pragma unroll 4
            for (int j = 0; j < n_valid; ++j) {
                const double om = ss[t * (SPB + 1) + j];
                z += om;
                qq += om * om;
                na += om * (double)eps[(2 * t) * (SPB + 1) + j];
                nd += om * (double)eps[(2 * t + 1) * (SPB + 1) + j];
            }
            double* o = part + 5 * t;
            st_g(o, 0, mt[t]);
            st_g(o, 1, z);
            st_g(o, 2, qq);
            st_g(o, 3, na);
            st_g(o, 4, nd);
        }
    }
    for (int t = tid; t < T && !lds; t += NT) {
        auto st_at = [&](int j) { return ld_g(d.Stk, (size_t)t * K + k_base + j); };
        double m = INFINITY;
        for (int j = 0; j < n_valid; ++j) {
            const double v = st_at(j);
            if (isfinite(v) && v < m) m = v;
        }
        double z = 0.0, qq = 0.0, na = 0.0, nd = 0.0;
        if (isfinite(m)) {
#pragma unroll 4
            for (int j = 0; j < n_valid; ++j) {
                const double v = st_at(j);
                const double om = isfinite(v) ? exp(-(v - m) / d.lambda) : 0.0;
                const float2 ev = ld_g(d.eps, (size_t)t * K + k_base + j);
                z += om;
                qq += om * om;
                na += om * (double)ev.x;
                nd += om * (double)ev.y;
            }
        }
        double* o = part + 5 * t;
        st_g(o, 0, m);
        st_g(o, 1, z);
        st_g(o, 2, qq);
        st_g(o, 3, na);
        st_g(o, 4, nd);
    }
}

// Calls f(instance, tile) for workgroup w of class cls of a batch; nothing past
// the last tile of the class (the grid is rounded up so that captured graphs
// can be replayed for other batches).  Tile w belongs to the instance whose
// tile range [prefix[i], prefix[i+1]) contains it; instances are ordered
// longest tile first, and the hardware dispatcher hands tiles to compute units
// as they free up.
template <typename F>
__device__ __forceinline__ void with_batch_tile(const BatchHdr* __restrict__ hdr, int cls, int w, F&& f)
{
    const unsigned char* base = reinterpret_cast<const unsigned char*>(hdr);
    const int i0 = hdr->cls_begin[cls];
    const int i1 = hdr->cls_begin[cls + 1];
    const int* prefix = reinterpret_cast<const int*>(base + hdr->off_prefix);
    const InstDesc* descs = reinterpret_cast<const InstDesc*>(base + hdr->off_descs);
    const int gw = w + prefix[i0];
    if (gw >= prefix[i1]) return;
    int lo = i0, hi = i1 - 1;  // largest i with prefix[i] <= gw
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (prefix[mid] <= gw) lo = mid; else hi = mid - 1;
    }
    f(descs[lo], gw - prefix[lo]);
}

// A batch instance's descriptor by value, read through the constant address
// space: scalar loads that no store or fence makes the compiler repeat.  (By
// reference the split kernel read its fields with vector loads, again after
// every wait: 256 uneven instances took 3.7 ms an iteration against 3.0.)
__device__ __forceinline__ InstDesc load_desc(const InstDesc& d)
{
    static_assert(sizeof(InstDesc) % 8 == 0, "whole words");
    struct Words {
        unsigned long long w[sizeof(InstDesc) / 8];
    } v;
    const const_ptr<unsigned long long> q = (const_ptr<unsigned long long>)(&d);
#pragma unroll
    for (unsigned i = 0; i < sizeof(InstDesc) / 8; ++i) v.w[i] = q[i];
    return __builtin_bit_cast(InstDesc, v);
}

}  // namespace mppi_impl
