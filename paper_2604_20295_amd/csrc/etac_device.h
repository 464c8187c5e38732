// Device building blocks of the ETac step on gfx950: the pinned FP64 contact
// predicate and the split-FP16 arithmetic of the residual network.
#pragma once

#include <cstddef>

#include "etac_internal.h"

namespace etac {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// Offsets of the packed network parameters (layout documented in etac.h).
constexpr int kW1 = 0, kB1 = 576, kW2 = 640, kB2 = 4736, kW3 = 4800, kB3 = 8896;
constexpr int kW4 = 8960, kB4 = 17152, kW5 = 17216, kB5 = 17408, kPhiN = 17411;

// ---------------------------------------------------------------------------
// contact (Sec. III-A: SDF contact of nodes with rigid objects)
// ---------------------------------------------------------------------------

struct Pen {
    bool inside;
    double depth, u0, u1, u2;
};

// Penetration of a node into one primitive.  FP64, every operation in the
// order written and rounded to nearest-even, no contraction into FMA:
//   d = p - t;  q_c = (R[0][c] d_0 + R[1][c] d_1) + R[2][c] d_2
//   sphere  : s = (d_0^2 + d_1^2) + d_2^2 < r^2,  depth = r - sqrt(s),
//             u = (depth / sqrt(s)) d
//   box     : |q_c| < h_c for all c; face = first argmin (h_c - |q_c|);
//             u = (sign(q_face) depth) R[:, face]  (sign(0) = +1)
//   capsule : z = clamp(q_2, -L, L), v = (q_0, q_1, q_2 - z), s = v.v < r^2,
//             u = (depth / sqrt(s)) R v
// A node on the centre point / axis segment gets depth r and u = -r n.
// Inside tests are sqrt-free; depth uses the correctly rounded FP64 sqrt, so
// the inside set and the deepest-object choice are reproducible bit for bit.
__device__ __forceinline__ Pen penetrate(int type, const float *sh, const float *R, const float *t,
                                         float px, float py, float pz, float nx, float ny, float nz) {
#pragma clang fp contract(off)
    Pen h;
    h.inside = false;
    h.depth = 0.0;
    h.u0 = h.u1 = h.u2 = 0.0;
    const double d0 = (double)px - (double)t[0];
    const double d1 = (double)py - (double)t[1];
    const double d2 = (double)pz - (double)t[2];
    if (type == ETAC_SPHERE) {
        const double r = (double)sh[0];
        const double s = (d0 * d0 + d1 * d1) + d2 * d2;
        if (!(s < r * r)) return h;
        h.inside = true;
        if (s == 0.0) {
            h.depth = r;
            h.u0 = -r * (double)nx; h.u1 = -r * (double)ny; h.u2 = -r * (double)nz;
            return h;
        }
        const double l = sqrt(s);
        h.depth = r - l;
        const double sc = h.depth / l;
        h.u0 = sc * d0; h.u1 = sc * d1; h.u2 = sc * d2;
        return h;
    }
    const double r00 = R[0], r01 = R[1], r02 = R[2];
    const double r10 = R[3], r11 = R[4], r12 = R[5];
    const double r20 = R[6], r21 = R[7], r22 = R[8];
    const double q0 = (r00 * d0 + r10 * d1) + r20 * d2;
    const double q1 = (r01 * d0 + r11 * d1) + r21 * d2;
    const double q2 = (r02 * d0 + r12 * d1) + r22 * d2;
    if (type == ETAC_BOX) {
        const double h0 = sh[0], h1 = sh[1], h2 = sh[2];
        if (!(fabs(q0) < h0)) return h;
        if (!(fabs(q1) < h1)) return h;
        if (!(fabs(q2) < h2)) return h;
        h.inside = true;
        double best = h0 - fabs(q0);
        int cs = 0;
        double qs = q0;
        const double s1 = h1 - fabs(q1);
        if (s1 < best) { best = s1; cs = 1; qs = q1; }
        const double s2 = h2 - fabs(q2);
        if (s2 < best) { best = s2; cs = 2; qs = q2; }
        h.depth = best;
        const double a = (qs >= 0.0) ? best : -best;
        const double c0 = cs == 0 ? r00 : (cs == 1 ? r01 : r02);
        const double c1 = cs == 0 ? r10 : (cs == 1 ? r11 : r12);
        const double c2 = cs == 0 ? r20 : (cs == 1 ? r21 : r22);
        h.u0 = a * c0; h.u1 = a * c1; h.u2 = a * c2;
        return h;
    }
    const double r = sh[0], L = sh[1];
    double z = q2;
    if (z < -L) z = -L;
    else if (z > L) z = L;
    const double v0 = q0, v1 = q1, v2 = q2 - z;
    const double s = (v0 * v0 + v1 * v1) + v2 * v2;
    if (!(s < r * r)) return h;
    h.inside = true;
    if (s == 0.0) {
        h.depth = r;
        h.u0 = -r * (double)nx; h.u1 = -r * (double)ny; h.u2 = -r * (double)nz;
        return h;
    }
    const double l = sqrt(s);
    h.depth = r - l;
    const double sc = h.depth / l;
    h.u0 = sc * ((r00 * v0 + r01 * v1) + r02 * v2);
    h.u1 = sc * ((r10 * v0 + r11 * v1) + r12 * v2);
    h.u2 = sc * ((r20 * v0 + r21 * v1) + r22 * v2);
    return h;
}

// Radius of a ball around the object's origin that contains the primitive.
__device__ __forceinline__ float bounding_radius(int type, const float *sh) {
    if (type == ETAC_SPHERE) return sh[0];
    if (type == ETAC_BOX) return sqrtf(sh[0] * sh[0] + sh[1] * sh[1] + sh[2] * sh[2]);
    return sh[0] + sh[1];
}

// One object of a scene row as the contact test reads it.
struct ObjRow {
    int type;
    float shape[4], rot[9], trans[3];
    float reach2;      // square of the ball test's radius
};

// The ball that rules a node out in FP32, with a relative margin of 1e-3 (far
// above FP32 rounding).
__device__ __forceinline__ float ball_reach2(int type, const float *shape) {
    const float rb = bounding_radius(type, shape) * 1.001f + 1e-3f;
    return rb * rb;
}

struct NodeContact {
    int best = -1;
    double bd = 0.0, b0 = 0.0, b1 = 0.0, b2 = 0.0;

    __device__ __forceinline__ void test(int o, int ty, const float *sh, const float *R, const float *t, float reach2,
                                         float px, float py, float pz, float nx, float ny, float nz) {
        const float dx = px - t[0], dy = py - t[1], dz = pz - t[2];
        if (dx * dx + dy * dy + dz * dz > reach2) return;
        const Pen h = penetrate(ty, sh, R, t, px, py, pz, nx, ny, nz);
        if (h.inside && (best < 0 || h.depth > bd)) {
            best = o;
            bd = h.depth;
            b0 = h.u0; b1 = h.u1; b2 = h.u2;
        }
    }
};

// Contact of one node with the candidate objects of scene row `row` (bit o
// of `cand`).  The ball test skips objects that cannot contain the node;
// survivors take the exact FP64 test.  Deepest penetration wins, lowest index
// on ties.  Returns the winning slot or -1; u is the winner's u_hat rounded to
// FP32.
__device__ __forceinline__ int contact_node(const SceneDev &S, size_t row, unsigned cand, float px, float py,
                                            float pz, float nx, float ny, float nz, float &u0, float &u1,
                                            float &u2) {
    NodeContact c;
    const int no = min(S.n_obj[row], S.O);   // device contents are not validated on the host
    for (int o = 0; o < no; ++o) {
        if (!((cand >> o) & 1u)) continue;
        const size_t eo = row * S.O + o;
        const int ty = S.type[eo];
        const float *sh = S.shape + 4 * eo;
        c.test(o, ty, sh, S.rot + 9 * eo, S.trans + 3 * eo, ball_reach2(ty, sh), px, py, pz, nx, ny, nz);
    }
    u0 = (float)c.b0; u1 = (float)c.b1; u2 = (float)c.b2;
    return c.best;
}

// The same from objects in LDS (an env's row).
__device__ __forceinline__ int contact_node(const ObjRow *obj, unsigned cand, float px, float py, float pz, float nx,
                                            float ny, float nz, float &u0, float &u1, float &u2) {
    NodeContact c;
    for (; cand; cand &= cand - 1) {     // ascending
        const int o = __ffs(cand) - 1;
        const ObjRow &r = obj[o];
        c.test(o, r.type, r.shape, r.rot, r.trans, r.reach2, px, py, pz, nx, ny, nz);
    }
    u0 = (float)c.b0; u1 = (float)c.b1; u2 = (float)c.b2;
    return c.best;
}

// dL/d(R, t) contribution of one active node from dL/du_hat = g (FP64),
// added to acc[0..8] (R, row-major) and acc[9..11] (t).
// The face / clamp choice repeats the forward's operation order.
__device__ inline void contact_adjoint_node(int type, const float *sh, const float *Rf, const float *tf, float px, float py,
                                     float pz, const double g[3], double acc[12]) {
#pragma clang fp contract(off)
    const double d[3] = {(double)px - (double)tf[0], (double)py - (double)tf[1], (double)pz - (double)tf[2]};
    double R[9];
    for (int c = 0; c < 9; ++c) R[c] = Rf[c];
    if (type == ETAC_SPHERE) {
        const double r = sh[0];
        const double s = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2];
        if (s == 0.0) return;
        const double l = sqrt(s);
        const double phi = r / l - 1.0, tphip = -r / (l * s);
        const double gd = g[0] * d[0] + g[1] * d[1] + g[2] * d[2];
        #pragma unroll
        for (int a = 0; a < 3; ++a) acc[9 + a] -= phi * g[a] + tphip * gd * d[a];
        return;
    }
    double q[3];
    for (int c = 0; c < 3; ++c) q[c] = (R[0 * 3 + c] * d[0] + R[1 * 3 + c] * d[1]) + R[2 * 3 + c] * d[2];
    if (type == ETAC_BOX) {
        double best = (double)sh[0] - fabs(q[0]);
        int cs = 0;
        for (int c = 1; c < 3; ++c) {
            const double sl = (double)sh[c] - fabs(q[c]);
            if (sl < best) { best = sl; cs = c; }
        }
        const double sg = q[cs] >= 0.0 ? 1.0 : -1.0;
        const double rc[3] = {R[cs], R[3 + cs], R[6 + cs]};
        const double grc = g[0] * rc[0] + g[1] * rc[1] + g[2] * rc[2];
        const double coef = sg * (double)sh[cs] - q[cs];
        #pragma unroll
        for (int a = 0; a < 3; ++a) {
            acc[9 + a] += grc * rc[a];
            acc[a * 3 + cs] += coef * g[a] - grc * d[a];
        }
        return;
    }
    const double r = sh[0], L = sh[1];
    double z = q[2];
    bool clamped = false;
    if (z < -L) { z = -L; clamped = true; }
    else if (z > L) { z = L; clamped = true; }
    const double v[3] = {q[0], q[1], q[2] - z};
    const double s = (v[0] * v[0] + v[1] * v[1]) + v[2] * v[2];
    if (s == 0.0) return;
    const double l = sqrt(s);
    const double phi = r / l - 1.0, tphip = -r / (l * s);
    double Rv[3], RTg[3];
    #pragma unroll
    for (int a = 0; a < 3; ++a) Rv[a] = R[a * 3] * v[0] + R[a * 3 + 1] * v[1] + R[a * 3 + 2] * v[2];
    for (int c = 0; c < 3; ++c) RTg[c] = R[c] * g[0] + R[3 + c] * g[1] + R[6 + c] * g[2];
    const double gRv = g[0] * Rv[0] + g[1] * Rv[1] + g[2] * Rv[2];
    double av[3];
    for (int c = 0; c < 3; ++c) av[c] = tphip * gRv * v[c] + phi * RTg[c];
    if (!clamped) av[2] = tphip * gRv * v[2];
    #pragma unroll
    for (int a = 0; a < 3; ++a) {
        for (int c = 0; c < 3; ++c) acc[a * 3 + c] += d[a] * av[c] + phi * g[a] * v[c];
        acc[9 + a] -= R[a * 3] * av[0] + R[a * 3 + 1] * av[1] + R[a * 3 + 2] * av[2];
    }
}

// Conservative test that a primitive's bounding ball (centre t) may reach the
// ball b = (centre, radius): relative margins of 1e-3 and 1e-5, far above
// FP32 rounding.
__device__ __forceinline__ bool ball_reaches(const float4 &b, int type, const float *shape, const float *t) {
    const float dx = b.x - t[0], dy = b.y - t[1], dz = b.z - t[2];
    const float reach = (b.w + bounding_radius(type, shape)) * 1.001f + 1e-3f;
    const float d2 = dx * dx + dy * dy + dz * dz;
    return d2 * (1.0f - 1e-5f) <= reach * reach;
}

// ---------------------------------------------------------------------------
// wave helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return threadIdx.x & 63; }

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Values that are equal across the workgroup but come from LDS must be made
// visibly uniform before they steer control flow that contains barriers:
// otherwise the compiler treats the branch as divergent and may split a wave
// around a barrier (e.g. one lane leaving to finish a store while the others
// re-enter the barrier and read stale LDS).
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ unsigned uniform(unsigned v) { return (unsigned)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ float uniform(float v) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

__device__ __forceinline__ unsigned lanes_below(unsigned long long mask) {
    return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// Maximum over the wave, returned in every lane.
__device__ __forceinline__ int wave_max_int(int v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = max(v, __shfl_xor(v, off));
    return v;
}
// Values of other lanes of the row of 16 by DPP, without the latency of LDS:
// lane ^ 1, ^ 2, ^ 7 (mirrored half row), ^ 8 (rotated by 8), ^ 15 (mirrored row).
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppXor7 = 0x141, kDppXor8 = 0x128, kDppXor15 = 0x140;
template <int CTRL>
__device__ __forceinline__ int dpp(int v) { return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true); }
template <int CTRL>
__device__ __forceinline__ float dpp(float v) { return __int_as_float(dpp<CTRL>(__float_as_int(v))); }

__device__ __forceinline__ unsigned wave_or(unsigned v) {
    v |= (unsigned)dpp<kDppXor1>((int)v);
    v |= (unsigned)dpp<kDppXor2>((int)v);
    v |= (unsigned)dpp<kDppXor7>((int)v);
    v |= (unsigned)dpp<kDppXor15>((int)v);
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    v = a[0] | a[1];
    const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return b[0] | b[1];
}

__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp<kDppXor1>(v));
    v = fmaxf(v, dpp<kDppXor2>(v));
    v = fmaxf(v, dpp<kDppXor7>(v));
    v = fmaxf(v, dpp<kDppXor15>(v));
    // rows 0 and 1, 2 and 3, then the halves
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Certified cutoff of the pair sums of Eq. 1 on far patches.  A run of 32 nodes
// is passed over when its box lies further than D from the box of the wave's
// own nodes, where exp(-alpha D) = 2^-50: every weight left out is below 2^-50,
// so a sum changes by less than 2^-50 times the sum of the |u_hat| that it left
// out (of |dL/dU| in the adjoint).  Where every term lies beyond D the sum
// becomes 0.
constexpr double kCutLog2 = 50.0;
// D^2 for the item's alpha, rounded up (no cutoff when alpha <= 0).
__device__ __forceinline__ float cutoff_d2(float alpha) {
    if (!(alpha > 0.0f)) return __builtin_inff();
    const double d = kCutLog2 / ((double)alpha * 1.4426950408889634);
    return (float)(d * d * (1.0 + 1e-6));
}

// ---------------------------------------------------------------------------
// residual network Phi on MFMA with split-FP16 operands
//
// Every FP32 operand x is split as x = hi + lo with hi = fp16(x) and
// lo = fp16(x - hi) (22 significant bits together), and a product is taken as
// hi*hi + hi*lo + lo*hi on v_mfma_f32_16x16x32_f16 with FP32 accumulation.
// The dropped lo*lo term is ~2^-22 relative, so a layer keeps FP32-level
// accuracy at the FP16 matrix rate (about 5x the FP32 matrix rate).
//
// Range.  The pair keeps 22 bits only while |x| lies in [2^-3, 2^15]: above
// 65504 hi overflows, below 2^-3 lo is subnormal (absolute floor 2^-25).  So
// every split operand carries a power-of-two scale that keeps it below 2^15
// (T) with its bound within a factor two of T; a block's small elements then
// lose relative precision only below 2^-40 of that bound.  The node inputs
// are scaled per item (2^ax from X, the largest |component| of the item's
// inputs, at least 1).  The weights are scaled per launch by constants
// chosen from their infinity norms (largest row sum of |w|, or column sum
// for a transposed use) so that the products land below T without a
// rescale: |h1| <= (||W1|| + 2 max|b1|) T 2^s1 < T for inputs below T, and so
// on through the layers.  The biases follow the item's scales.  Powers of
// two are exact: the scaling changes no value beyond the rounding of the
// splits.  (A weight block whose scaled maximum falls below 2^-3 keeps
// 2^-25 absolute accuracy, about 2^-19 of its largest element at worst.)
//
// A 16-node tile is processed by one wave in transposed form, Y^T = W X^T:
// the MFMA's M dimension is the layer's output features, N the 16 nodes, K the
// input features.  Lane l holds node (l & 15).  After a layer it holds output
// features 16 ot + 4 (l >> 4) + r (r = 0..3) of out-tile ot in register r of
// accumulator ot.  The next layer's K dimension is ordered so that these same
// registers are its B operand: in K step s, lane group q = l >> 4 supplies
// inputs 16 (2 s + (e >> 2)) + 4 q + (e & 3) for e = 0..7.  Weight fragments
// are pre-arranged in LDS in that order (hi and lo halves), so every A
// operand is one 16-byte LDS read.
// ---------------------------------------------------------------------------
typedef _Float16 half8 __attribute__((ext_vector_type(8)));

constexpr int kTopExp = 15;   // scaled operand bounds lie in [2^14, 2^15): T = 2^15
constexpr float kTop = 32768.0f;

// Exponent s of the scale 2^s that puts `bound` in [2^(kTopExp-1), 2^kTopExp);
// 0 for a zero or non-finite bound; clamped to [-100, 100].
__device__ __forceinline__ int range_exp(float bound) {
    if (!(bound > 0.0f) || !(bound <= 3.0e38f)) return 0;
    int e;
    (void)frexpf(bound, &e);   // bound = m 2^e, m in [0.5, 1)
    return max(-100, min(100, kTopExp - e));
}

// 2^s, exact for -149 <= s <= 127 (subnormal below -126).
__device__ __forceinline__ float pow2(int s) { return ldexpf(1.0f, s); }

// Scales of one item's activations (uniform; every thread computes the same
// values).  X bounds every component of the item's node inputs.
// x at 2^ax, h1 at 2^a1 = 2^(s1 + ax), f at 2^af = 2^(s2 + a1).
struct ItemScale {
    int ax, a1, af;
    float xmul;          // 2^ax
};

// LDS members that are read four floats at a time start at 16-byte boundaries.
#define ETAC_LDS_ALIGNED(type, member) \
    static_assert(alignof(type) % 16 == 0 && offsetof(type, member) % 16 == 0, #type "::" #member " is read 16 bytes at a time")

struct NetLds {
    half8 w1h[4 * 64], w1l[4 * 64];          // [ot][lane]    W1 2^s1, inputs padded 9 -> 32 (one K step)
    half8 w2h[4 * 2 * 64], w2l[4 * 2 * 64];  // [ot2][s][lane] W2 2^s2
    float b1[64], b2[64];
    float b1s[64], b2s[64];                  // per item: b1 2^a1, b2 2^af
    float part[kWaves][64];                  // per-wave partials
    // per launch: scale exponents of the staged weights (W1 2^s1, W2 2^s2) and of
    // the adjoint's transposed uses (W4[:, :64]^T 2^s4t, W2^T 2^s2t)
    int s1, s2, s4t, s2t;
};
ETAC_LDS_ALIGNED(NetLds, b1s);
ETAC_LDS_ALIGNED(NetLds, b2s);

typedef _Float16 half2t __attribute__((ext_vector_type(2)));
typedef unsigned uint2t __attribute__((ext_vector_type(2)));
typedef unsigned uint4t __attribute__((ext_vector_type(4)));

// x - (float)h exactly, for h the FP16 value in the low (HI_HALF false) or
// high half of a packed register: one v_fma_mix_f32 (-h * 1.0 + x with the
// FP16 operand converted inside the instruction).
template <bool HI_HALF>
__device__ __forceinline__ float sub_f16(float x, unsigned h2) {
    float r;
    if (HI_HALF) asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r) : "v"(h2), "v"(x));
    else asm("v_fma_mix_f32 %0, -%1, 1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r) : "v"(h2), "v"(x));
    return r;
}

// Split two floats: hi = fp16(a), fp16(b) packed; lo = fp16 of the exact
// remainders.  Four instructions per pair.
__device__ __forceinline__ void split2(float a, float b, unsigned &hi, unsigned &lo) {
    const half2t h = {(_Float16)a, (_Float16)b};
    hi = __builtin_bit_cast(unsigned, h);
    const half2t l = {(_Float16)sub_f16<false>(a, hi), (_Float16)sub_f16<true>(b, hi)};
    lo = __builtin_bit_cast(unsigned, l);
}

__device__ __forceinline__ void split8(const float v[8], half8 &hi, half8 &lo) {
    uint4t h, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        unsigned a, b;
        split2(v[2 * e], v[2 * e + 1], a, b);
        h[e] = a;
        l[e] = b;
    }
    hi = __builtin_bit_cast(half8, h);
    lo = __builtin_bit_cast(half8, l);
}

// Input feature of K step s, lane group q, element e of a 64 -> 64 layer.
__device__ __forceinline__ int chain_k(int s, int q, int e) { return 16 * (2 * s + (e >> 2)) + 4 * q + (e & 3); }

// Per-launch quantities of the range scaling (whole workgroup; the caller
// brackets it with barriers).  Wave w takes rows (or columns) 16 w + (l & 15);
// lane group q = l >> 4 sums a quarter of each, the quarters are added with
// two shuffles and the wave's largest sum goes to part.
// (row norms of W1 and W2, column norms of W2 and W4[:, :64], max |W4[:, :64]|, |b1|, |b2|)
constexpr int kNorms = 7;

__device__ void net_norms(float (&part)[kWaves][64], const float *phi) {
    const int lane = lane_id(), wave = threadIdx.x >> 6, q = lane >> 4;
    const int r = 16 * wave + (lane & 15);
    float s1 = 0.0f, s2 = 0.0f, t2 = 0.0f, t4 = 0.0f;
    float m4 = 0.0f, mb1 = 0.0f, mb2 = 0.0f;
#pragma unroll
    for (int d = 0; d < 16; ++d) {      // unrolled: every load in flight at once
        const int c = 16 * q + d;
        const float a = fabsf(phi[kW2 + r * 64 + c]), b = fabsf(phi[kW4 + r * 128 + c]);
        s2 += a;
        m4 = fmaxf(m4, b);
        t2 += fabsf(phi[kW2 + c * 64 + r]);
        t4 += fabsf(phi[kW4 + c * 128 + r]);
    }
    if (q == 0) {
        for (int c = 0; c < 9; ++c) s1 += fabsf(phi[kW1 + r * 9 + c]);
        mb1 = fabsf(phi[kB1 + r]);
        mb2 = fabsf(phi[kB2 + r]);
    }
    float v[kNorms] = {s1, s2, t2, t4, m4, mb1, mb2};
#pragma unroll
    for (int j = 0; j < 4; ++j) {   // sums over the four quarters
        v[j] += __shfl_xor(v[j], 16);
        v[j] += __shfl_xor(v[j], 32);
    }
#pragma unroll
    for (int j = 0; j < kNorms; ++j) {
        v[j] = wave_max(v[j]);
        part[wave][j] = v[j];      // identical in every lane
    }
}

// Scale exponents of W1, W2 and W4[:, :64] from the largest norms (see
// stage_net).
__device__ __forceinline__ void net_scales(const float (&v)[kNorms], int &s1, int &s2, int &s4) {
    s1 = range_exp((v[0] + 2.0f * v[5]) * kTop);
    s2 = range_exp((v[1] * kTop + 2.0f * v[6] * kTop * pow2(s1)));
    s4 = range_exp(v[4]);
}

// Stage the network into LDS in fragment order (whole workgroup), each
// weight matrix scaled by its per-launch power of two, and set the scale
// exponents.  With inputs x 2^ax below T (X at least 1, so 2^ax <= 2T):
//   h1 = W1 2^s1 x + b1 2^a1:  |h1| <= (||W1|| + 2 max|b1|) T 2^s1 < T,
//   f  = W2 2^s2 h1 + b2 2^af: |f| <= (||W2|| T + 2 max|b2| T 2^s1) 2^s2 < T,
//   W4 2^s4 with s4 from max |W4[:, :64]| (the tables' product; it is never split).
// Adjoint, with dL/dpre4 2^d4 below T: W4[:, :64]^T 2^s4t and W2^T 2^s2t by
// their column norms keep dL/dpre2 and dL/dpre1 below T.
// Ends with a barrier.
__device__ void stage_net(NetLds &L, const float *phi) {
    const int tid = threadIdx.x;
    net_norms(L.part, phi);
    __syncthreads();
    float v[kNorms];
#pragma unroll
    for (int j = 0; j < kNorms; ++j) {
        v[j] = L.part[0][j];
        for (int w = 1; w < kWaves; ++w) v[j] = fmaxf(v[j], L.part[w][j]);
    }
    const float n4t = v[3], n2t = v[2];
    int s1, s2, s4;
    net_scales(v, s1, s2, s4);
    const float e1 = pow2(s1), e2 = pow2(s2);
    for (int idx = tid; idx < 4 * 64; idx += kWG) {
        const int lane = idx & 63, ot = idx >> 6, q = lane >> 4;
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int in = 8 * q + e;
            x[e] = in < 9 ? phi[kW1 + (ot * 16 + (lane & 15)) * 9 + in] * e1 : 0.0f;
        }
        split8(x, L.w1h[idx], L.w1l[idx]);
    }
    for (int idx = tid; idx < 4 * 2 * 64; idx += kWG) {
        const int lane = idx & 63, s = (idx >> 6) & 1, ot2 = idx >> 7, q = lane >> 4;
        const int out = ot2 * 16 + (lane & 15);
        float a[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) a[e] = phi[kW2 + out * 64 + chain_k(s, q, e)] * e2;
        split8(a, L.w2h[idx], L.w2l[idx]);
    }
    for (int i = tid; i < 64; i += kWG) {
        L.b1[i] = phi[kB1 + i];
        L.b2[i] = phi[kB2 + i];
    }
    if (tid < 64) {   // wave 0, identical values
        L.s1 = s1; L.s2 = s2;
        L.s4t = range_exp(n4t * kTop);
        L.s2t = range_exp(n2t * kTop);
    }
    __syncthreads();
}

// Scales of the activations of an item whose inputs are bounded by X
// (uniform; every thread computes the same values, kept in scalar registers).
__device__ __forceinline__ ItemScale item_scale(const NetLds &L, float X) {
    ItemScale s;
    s.ax = uniform(range_exp(fmaxf(X, 1.0f)));
    s.a1 = uniform(L.s1) + s.ax;
    s.af = uniform(L.s2) + s.a1;
    s.xmul = uniform(pow2(s.ax));
    return s;
}

// Scaled biases of the encoder layers (threads < 64; the caller's next barrier
// publishes them).
__device__ __forceinline__ void item_biases(NetLds &L, const ItemScale &s) {
    if (threadIdx.x < 64) {
        const int i = threadIdx.x;
        L.b1s[i] = L.b1[i] * pow2(s.a1);
        L.b2s[i] = L.b2[i] * pow2(s.af);
    }
}

// Input bound of item (patch k) given the largest |u_hat| component of its nodes.
__device__ __forceinline__ float item_xbound(const MeshDev &M, int k, float umax) {
    return fmaxf(M.xbound[k], umax);
}

// Keeps the compiler from hoisting the (loop-invariant) LDS weight-fragment
// loads of a tile out of the node loops: hoisted, they would need ~280 extra
// registers per lane and spill.  Emits no instruction.
__device__ __forceinline__ void reload_fence() { asm volatile("" ::: "memory"); }

__device__ __forceinline__ floatx4 mfma16(const half8 &a, const half8 &b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// acc += A B with split operands (hi*hi + hi*lo + lo*hi)
__device__ __forceinline__ floatx4 mfma_split(const half8 &ah, const half8 &al, const half8 &bh, const half8 &bl,
                                              floatx4 acc) {
    acc = mfma16(ah, bh, acc);
    acc = mfma16(ah, bl, acc);
    return mfma16(al, bh, acc);
}

// max(x, 0) as a signed-integer max of the bits: negative floats (and -0)
// have negative bit patterns; one instruction, no NaN canonicalisation.
__device__ __forceinline__ float relu1(float x) { return __int_as_float(max(__float_as_int(x), 0)); }

__device__ __forceinline__ floatx4 relu4(floatx4 v) {
    floatx4 o;
#pragma unroll
    for (int r = 0; r < 4; ++r) o[r] = relu1(v[r]);
    return o;
}

// Split a D-layout 64-feature tile into the B operands of the two K steps of
// the next 64 -> 64 layer.
__device__ __forceinline__ void split_chain(const floatx4 x[4], half8 bh[2], half8 bl[2]) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = x[2 * s + (e >> 2)][e & 3];
        split8(v, bh[s], bl[s]);
    }
}

}  // namespace etac
