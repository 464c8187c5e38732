// Real-sensor regressor on gfx950: the displacement field of every (env,
// patch) item mapped to the eight taxel outputs of a real sensor by a
// PointNet-style network with a residual layer and attention pooling (the
// regressor of the paper's appendix, "Modeling Real Sensors").
//
//   k_live         : the envs in contact on each patch.
//   k_regress      : persistent, one workgroup of eight waves per CU with the
//                    per-node layers' weights resident in LDS; a unit is 256
//                    nodes of an item (more in a plan whose rows would take
//                    over 256 MB), taken by a wave (largest patches first,
//                    one each and then from a device work queue): 16-node
//                    tiles, two at a time, through the per-node layers on MFMA
//                    with an online softmax over the tiles.  The unit's
//                    maximum, sum of weights and weighted sum of features are
//                    a row of scratch.
//   k_regress_head : the rows of an item combined, and the head, in FP32.
//   k_regress_fill : items without contact have U = 0 on the whole patch, so
//                    their output is the patch's rest output, computed once
//                    per patch (an item behind the patch's last env in
//                    contact) and copied here.
//
// Per node:  x = [p - o_k, U] (6) -> h1 = relu(E1 x + e1) (64)
//            -> h2 = relu(E2 h1 + e2) + h1 (64) -> f = relu(E3 h2 + e3) (256)
//            -> s = a2 . tanh(A1 f + a1) + a0.
// Per item:  w = softmax(s), g = sum w f, y = D2 relu(D1 g + d1) + d2 (8).
//
// Precision: E1, the layer that sees positions and displacements, uses
// split-FP16 operands (hi + lo, FP32-level), so that displacements well
// below the position scale keep their bits; E2, E3 and A1 take FP16
// operands with FP32 accumulation; the pooled features are the FP16
// operands of A1 (f is held once, in 32 registers per tile); softmax
// weights, pooling sums and the head are FP32.  FP16 rounding is relative
// 2^-11 at most.
#include "etac_step.h"

namespace etac {

constexpr int kRegWG = 512;                  // eight waves, two per SIMD
constexpr int kRegWaves = kRegWG / 64;
constexpr int kRegNT = 2;                    // 16-node tiles per wave and pass (one weight read, kRegNT MFMAs)
// packed parameter offsets (FP32 values)
constexpr int kRE1 = 0, kRe1 = 384, kRE2 = 448, kRe2 = 4544, kRE3 = 4608, kRe3 = 20992;
constexpr int kRA1 = 21248, kRa1 = 54016, kRa2 = 54144, kRa0 = 54272, kRD1 = 54276, kRd1 = 87044;
constexpr int kRD2 = 87172, kRd2 = 88196, kRegN = 88204;
static_assert(kRegN == ETAC_REG_SIZE, "regressor parameter layout");
// 2 log2(e): A1 and a1 are stored times this, so that exp2 of the
// pre-activation is e^(2 z) and tanh z = 1 - 2 / (1 + e^(2 z)).
constexpr float kTwoLog2e = 2.8853900817779268f;

struct RegLds {
    half8 e1[4 * 64];                            // [E1 | e1] (x_6 = 1 carries e1): the three products of its split
                                                 // parts share one K step: lane group 0 hi hi, 2 hi lo, 3 lo hi
    half8 e2[4 * 2 * 64];                        // E2 FP16, [ot][s][lane], chain order
    half8 e3[16 * 2 * 64];                       // E3 FP16, [ot][s][lane], 256 outputs
    half8 a1[8 * 8 * 64];                        // 2 log2(e) A1 in FP16, [ot][s][lane], 128 outputs over 256 inputs
    float be2[64], be3[256], ba1[128], wa2[128]; // e2, e3, 2 log2(e) a1, -2 a2
};
ETAC_LDS_ALIGNED(RegLds, be2);
ETAC_LDS_ALIGNED(RegLds, be3);
ETAC_LDS_ALIGNED(RegLds, ba1);
ETAC_LDS_ALIGNED(RegLds, wa2);

struct RegParams {
    MeshDev mesh;
    const float *reg;         // [ETAC_REG_SIZE]
    const float *u;           // [3][E][N]
    const int *live, *live_cnt;      // [K][E], [K] envs in contact
    float *pooled;            // [units][256] weighted sum of a unit's features
    float2 *ml;               // [units] its largest score and its sum of weights
    unsigned *counter;        // [2] work queue, retired workgroups
    int E, unit;              // nodes of a unit
};

__device__ __forceinline__ int reg_parts(const RegParams &p, int k) {
    return (p.mesh.offset[k + 1] - p.mesh.offset[k] + p.unit - 1) / p.unit;
}

__device__ void stage_regressor(RegLds &L, const float *R) {
    const int tid = threadIdx.x;
    for (int idx = tid; idx < 4 * 64; idx += kRegWG) {
        const int lane = idx & 63, ot = idx >> 6, q = lane >> 4, o = ot * 16 + (lane & 15);
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = q == 1 ? 0.0f : e < 6 ? R[kRE1 + o * 6 + e] : e == 6 ? R[kRe1 + o] : 0.0f;
        half8 h, l;
        split8(x, h, l);
        L.e1[idx] = q == 3 ? l : h;
    }
    for (int idx = tid; idx < 4 * 2 * 64; idx += kRegWG) {
        const int lane = idx & 63, s = (idx >> 6) & 1, ot = idx >> 7, q = lane >> 4;
        half8 h;
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = (_Float16)R[kRE2 + (ot * 16 + (lane & 15)) * 64 + chain_k(s, q, e)];
        L.e2[idx] = h;
    }
    for (int idx = tid; idx < 16 * 2 * 64; idx += kRegWG) {
        const int lane = idx & 63, s = (idx >> 6) & 1, ot = idx >> 7, q = lane >> 4;
        half8 h;
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = (_Float16)R[kRE3 + (ot * 16 + (lane & 15)) * 64 + chain_k(s, q, e)];
        L.e3[idx] = h;
    }
    for (int idx = tid; idx < 8 * 8 * 64; idx += kRegWG) {
        const int lane = idx & 63, s = (idx >> 6) & 7, ot = idx >> 9, q = lane >> 4;
        half8 h;
#pragma unroll
        for (int e = 0; e < 8; ++e)
            h[e] = (_Float16)(kTwoLog2e * R[kRA1 + (ot * 16 + (lane & 15)) * 256 + chain_k(s, q, e)]);
        L.a1[idx] = h;
    }
    for (int i = tid; i < 64; i += kRegWG) L.be2[i] = R[kRe2 + i];
    for (int i = tid; i < 256; i += kRegWG) L.be3[i] = R[kRe3 + i];
    for (int i = tid; i < 128; i += kRegWG) {
        L.ba1[i] = kTwoLog2e * R[kRa1 + i];
        L.wa2[i] = -2.0f * R[kRa2 + i];
    }
}

// FP16 B operands of K step s from a D-layout feature tile (no lo part).
__device__ __forceinline__ half8 chain_f16(const floatx4 *x, int s) {
    half8 h;
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = (_Float16)x[2 * s + (e >> 2)][e & 3];
    return h;
}

// relu of two values, rounded to FP16 and packed (rounding commutes with relu).
__device__ __forceinline__ unsigned pack_relu(float a, float b) {
    half2t h = {(_Float16)a, (_Float16)b};
    h = __builtin_elementwise_max(h, half2t{(_Float16)0.0f, (_Float16)0.0f});
    return __builtin_bit_cast(unsigned, h);
}

// acc + w * (low or high FP16 half of h), in one mixed-precision FMA.
template <bool HI>
__device__ __forceinline__ float fma_half(float w, unsigned h, float acc) {
    float d;
    if (HI) asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[0,1,0] op_sel_hi:[0,1,0]" : "=v"(d) : "v"(w), "v"(h), "v"(acc));
    else asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[0,1,0]" : "=v"(d) : "v"(w), "v"(h), "v"(acc));
    return d;
}

// kRegNT 16-node tiles through the per-node layers.  Out: fb[i][s], the
// tile's features f (256) as FP16 B operands of A1 (element e is feature
// chain_k(s, l >> 4, e) of node l & 15), and sc[i], the attention score of
// the lane's node up to a constant (the same in the four lanes of a node).
// Each weight fragment is read from LDS once per pass and used by every
// tile; A1 runs output block by output block so that the tanh of one block
// overlaps the MFMAs of the next.
__device__ __forceinline__ void regress_tiles(const RegLds &L, const half8 (&x)[kRegNT], half8 (&fb)[kRegNT][8],
                                              float (&sc)[kRegNT]) {
    constexpr int NT = kRegNT;
    reload_fence();
    const int lane = lane_id(), gq = lane >> 4;
    floatx4 h1[NT][4];
    half8 v[8];
    floatx4 b2[4];
    {
        const floatx4 z = {0.0f, 0.0f, 0.0f, 0.0f};
        half8 w[4];
#pragma unroll
        for (int ot = 0; ot < 4; ++ot) w[ot] = L.e1[ot * 64 + lane];
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = L.e2[t * 64 + lane];
#pragma unroll
        for (int ot = 0; ot < 4; ++ot) b2[ot] = *reinterpret_cast<const floatx4 *>(&L.be2[ot * 16 + 4 * gq]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ot = 0; ot < 4; ++ot)
#pragma unroll
            for (int i = 0; i < NT; ++i) h1[i][ot] = relu4(mfma16(w[ot], x[i], z));
    }
    half8 b0[NT], b1[NT];   // h2 as FP16 B operands of E3
    {
        half8 c0[NT], c1[NT];   // h1 as FP16 B operands of E2
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            c0[i] = chain_f16(h1[i], 0);
            c1[i] = chain_f16(h1[i], 1);
        }
        floatx4 h2[NT][4];
#pragma unroll
        for (int ot = 0; ot < 4; ++ot)
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                h2[i][ot] = relu4(mfma16(v[2 * ot + 1], c1[i], mfma16(v[2 * ot], c0[i], b2[ot])));
#pragma unroll
                for (int r = 0; r < 4; ++r) h2[i][ot][r] += h1[i][ot][r];
            }
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            b0[i] = chain_f16(h2[i], 0);
            b1[i] = chain_f16(h2[i], 1);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // E3: the weights of the next two output tiles are requested, and the last
    // two packed, while the MFMAs of these run
    {
        half8 w[2][4];
        floatx4 bias[2][2], f[2][NT][2];
        auto request = [&](int s, int b) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                bias[b][j] = *reinterpret_cast<const floatx4 *>(&L.be3[(2 * s + j) * 16 + 4 * gq]);
                w[b][2 * j] = L.e3[((2 * s + j) * 2 + 0) * 64 + lane];
                w[b][2 * j + 1] = L.e3[((2 * s + j) * 2 + 1) * 64 + lane];
            }
        };
        auto pack = [&](int s, int b) {
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                uint4t v;
                v[0] = pack_relu(f[b][i][0][0], f[b][i][0][1]);
                v[1] = pack_relu(f[b][i][0][2], f[b][i][0][3]);
                v[2] = pack_relu(f[b][i][1][0], f[b][i][1][1]);
                v[3] = pack_relu(f[b][i][1][2], f[b][i][1][3]);
                fb[i][s] = __builtin_bit_cast(half8, v);
            }
        };
        request(0, 0);
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int b = s & 1;
            if (s < 7) request(s + 1, b ^ 1);
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int i = 0; i < NT; ++i) f[b][i][j] = mfma16(w[b][2 * j], b0[i], bias[b][j]);
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int i = 0; i < NT; ++i) f[b][i][j] = mfma16(w[b][2 * j + 1], b1[i], f[b][i][j]);
            if (s) pack(s - 1, b ^ 1);
            if (s < 7) __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
            for (int i = 0; i < 4 * NT; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (s) __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        pack(7, 1);
    }
    // A1, output tile by output tile: the tanh of one tile between the MFMAs of
    // the next, its weights requested a tile ahead.  a2 . tanh(z) = sum(a2) -
    // 2 a2 . 1 / (1 + e^(2 z)); the constant sum(a2) (like a0) cancels in the
    // softmax.
#pragma unroll
    for (int i = 0; i < NT; ++i) sc[i] = 0.0f;
    {
        half8 w[8];
        floatx4 t[2][NT], c, bias;
#pragma unroll
        for (int s = 0; s < 8; ++s) w[s] = L.a1[s * 64 + lane];
        bias = *reinterpret_cast<const floatx4 *>(&L.ba1[4 * gq]);
        c = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        auto tanhs = [&](const floatx4 (&x)[NT]) {
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    sc[i] += c[r] * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(x[i][r]));
        };
#pragma unroll
        for (int ot = 0; ot < 8; ++ot) {
            const int b = ot & 1;
#pragma unroll
            for (int i = 0; i < NT; ++i) t[b][i] = bias;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
#pragma unroll
                for (int i = 0; i < NT; ++i) t[b][i] = mfma16(w[s], fb[i][s], t[b][i]);
                if (ot < 7) w[s] = L.a1[((ot + 1) * 8 + s) * 64 + lane];
            }
            if (ot < 7) bias = *reinterpret_cast<const floatx4 *>(&L.ba1[(ot + 1) * 16 + 4 * gq]);
            if (ot) tanhs(t[b ^ 1]);
            c = *reinterpret_cast<const floatx4 *>(&L.wa2[ot * 16 + 4 * gq]);
#pragma unroll
            for (int s = 0; s < 8; ++s) {
#pragma unroll
                for (int i = 0; i < NT; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    if (ot) {
                        __builtin_amdgcn_sched_group_barrier(0x400, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);
                    }
                }
                if (ot < 7) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        tanhs(t[1]);
    }
    // over the four lanes of a node
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(sc[i]), __float_as_uint(sc[i]), false, false);
        sc[i] = __uint_as_float(a[0]) + __uint_as_float(a[1]);
        const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(sc[i]), __float_as_uint(sc[i]), false, false);
        sc[i] = __uint_as_float(b[0]) + __uint_as_float(b[1]);
    }
}

// v from the lane n places along in the same row of 16 lanes (DPP row_ror).
template <int n>
__device__ __forceinline__ float row_ror(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x120 + n, 0xf, 0xf, true));
}

// Sum over the 16 nodes of a lane group (one row of 16 lanes); every lane
// gets it, each in its own fixed order (the same in every row).
__device__ __forceinline__ float node_sum(float v) {
    v += row_ror<8>(v);
    v += row_ror<4>(v);
    v += row_ror<2>(v);
    v += row_ror<1>(v);
    return v;
}

__device__ __forceinline__ float node_max(float v) {
    v = fmaxf(v, row_ror<8>(v));
    v = fmaxf(v, row_ror<4>(v));
    v = fmaxf(v, row_ror<2>(v));
    v = fmaxf(v, row_ror<1>(v));
    return v;
}

// One unit on one wave: the 16-node tiles of part `part` of patch k through the
// per-node layers, an online softmax over the tiles (running maximum m,
// per-lane running sums of e^(s - m) and e^(s - m) f), to row `row`.
__device__ void regress_unit(const RegParams &p, const RegLds &L, int e, int k, int part, bool rest, int row) {
    const MeshDev &M = p.mesh;
    const int N = M.N, lane = lane_id(), q = lane >> 4;
    const int base = M.offset[k], n = M.offset[k + 1] - base;
    const size_t EN = (size_t)p.E * N;
    const float o0 = M.origin[3 * k], o1 = M.origin[3 * k + 1], o2 = M.origin[3 * k + 2];
    float m_run = -INFINITY, l_run = 0.0f;   // m_run uniform; l_run per lane (its node's weights)
    floatx4 acc[16];
#pragma unroll
    for (int ot = 0; ot < 16; ++ot) acc[ot] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    const int passes = p.unit / (16 * kRegNT), groups = min((n + 16 * kRegNT - 1) / (16 * kRegNT), (part + 1) * passes);
    // the next tiles' inputs are requested while these run; nodes beyond the
    // patch repeat its last and get no weight
    const float *pos = M.pos + base, *u = p.u + (size_t)e * N + base;
    float raw[kRegNT][6];
    auto fetch = [&](int tg) {
#pragma unroll
        for (int i = 0; i < kRegNT; ++i) {
            const int j = min(16 * (kRegNT * tg + i) + (lane & 15), n - 1);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                raw[i][c] = pos[(size_t)c * N + j];
                raw[i][3 + c] = u[(size_t)c * EN + j];
            }
        }
    };
    fetch(part * passes);
    for (int tg = part * passes; tg < groups; ++tg) {
        half8 x[kRegNT];
        bool valid[kRegNT];
#pragma unroll
        for (int i = 0; i < kRegNT; ++i) {
            valid[i] = 16 * (kRegNT * tg + i) + (lane & 15) < n;
            const float v[8] = {raw[i][0] - o0, raw[i][1] - o1, raw[i][2] - o2, rest ? 0.0f : raw[i][3],
                                rest ? 0.0f : raw[i][4], rest ? 0.0f : raw[i][5], 1.0f, 0.0f};      // 1 carries the bias e1
            half8 h, l;
            split8(v, h, l);
            x[i] = q == 2 ? l : h;
        }
        fetch(tg + 1);
        half8 fb[kRegNT][8];
        float s[kRegNT];
        regress_tiles(L, x, fb, s);
        float mt = -INFINITY;
#pragma unroll
        for (int i = 0; i < kRegNT; ++i) {
            s[i] = valid[i] ? s[i] : -INFINITY;
            mt = fmaxf(mt, s[i]);
        }
        mt = uniform(node_max(mt));   // the same in every lane; finite (node 0 of the first tile is valid)
        if (mt > m_run) {             // rescale the running sums to the new maximum
            const float c = __expf(m_run - mt);   // 0 on the first pass
#pragma unroll
            for (int ot = 0; ot < 16; ++ot)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[ot][r] *= c;
            l_run *= c;
            m_run = mt;
        }
#pragma unroll
        for (int i = 0; i < kRegNT; ++i) {
            const float w = valid[i] ? __expf(s[i] - m_run) : 0.0f;
            l_run += w;
#pragma unroll
            for (int s8 = 0; s8 < 8; ++s8) {
                const uint4t h = __builtin_bit_cast(uint4t, fb[i][s8]);
#pragma unroll
                for (int e2 = 0; e2 < 4; ++e2) {
                    const int ot = 2 * s8 + (e2 >> 1), r = 2 * (e2 & 1);
                    acc[ot][r] = fma_half<false>(w, h[e2], acc[ot][r]);
                    acc[ot][r + 1] = fma_half<true>(w, h[e2], acc[ot][r + 1]);
                }
            }
        }
    }
    // sums over the 16 node lanes: features 16 ot + 4 q + r in every lane of group q
    const float l = node_sum(l_run);
#pragma unroll
    for (int ot = 0; ot < 16; ++ot)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[ot][r] = node_sum(acc[ot][r]);
    if ((lane & 15) == 0) {
        float *g = p.pooled + (size_t)row * 256 + 4 * q;
#pragma unroll
        for (int ot = 0; ot < 16; ++ot) *reinterpret_cast<floatx4 *>(g + ot * 16) = acc[ot];
    }
    if (lane == 0) p.ml[row] = make_float2(m_run, l);
}

// Persistent; every wave takes units on its own (no barrier per unit).  Bound
// by the per-node layers (116 MFMAs and about 500 VALU cycles' worth of
// instructions per 16 nodes on either side of them).  Units of 256 nodes of the
// items in contact alone: with whole items claimed from a queue of every (env,
// patch), five of six of them without contact, 1024 hands spent 45 % of the
// wave time in claims and had 1.1 items a wave (395 us; 280 us now; units of
// 128 nodes 298 us).
__global__ __launch_bounds__(kRegWG) void k_regress(RegParams p) {
    __shared__ RegLds L;
    __shared__ int first[kMaxPatches + 1];
    const MeshDev &M = p.mesh;
    const int wave = uniform(threadIdx.x >> 6);
    stage_regressor(L, p.reg);
    const int total = unit_prefix<kRegWaves>(M.K, first, [&](int kk) {
        const int k = M.order[kk];
        return (p.live_cnt[k] + 1) * reg_parts(p, k);
    });
    int pos = wave * gridDim.x + blockIdx.x;
    while (pos < total) {
        const int kk = unit_rank(first, M.K, pos), k = uniform(M.order[kk]);
        const int parts = uniform(reg_parts(p, k)), local = pos - uniform(first[kk]);
        const int it = local / parts;
        const bool rest = it == uniform(p.live_cnt[k]);
        regress_unit(p, L, rest ? 0 : uniform(p.live[(size_t)k * p.E + it]), k, local - it * parts, rest, pos);
        // one atomic for the wave (lane 0 adds 1), executed by every lane so
        // that no lane-dependent branch enters the loop; lane 0's old value
        // is the claimed position
        const unsigned old = atomicAdd(&p.counter[0], lane_id() == 0 ? 1u : 0u);
        pos = (int)(gridDim.x * kRegWaves) + __builtin_amdgcn_readlane((int)old, 0);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        const unsigned done = atomicAdd(&p.counter[1], 1u);
        if (done == gridDim.x - 1) {   // last workgroup: reset the queue
            atomicExch(&p.counter[0], 0u);
            atomicExch(&p.counter[1], 0u);
        }
    }
}

// Pooled feature g = sum w f / sum w of every item from its units' rows, and
// the head y = D2 relu(D1 g + d1) + d2, in FP32, kHeadRows items per block
// pass; D1 streamed through LDS transposed in 32-column chunks, the next chunk
// requested while one is used.  Latency-bound: 16 items a pass give 1024 hands
// 145 blocks (32 items a pass and chunks loaded in turn: 34 us; 31 us).
constexpr int kHeadRows = 16;

__global__ __launch_bounds__(256) void k_regress_head(RegParams p, float *taxels, float *rest) {
    __shared__ alignas(16) float G[kHeadRows][256];
    __shared__ float DT[32][129];
    __shared__ float H[kHeadRows][128];
    __shared__ int items[kMaxPatches + 1], units[kMaxPatches + 1];
    __shared__ int row0[kHeadRows], rows[kHeadRows], out[kHeadRows];
    const MeshDev &M = p.mesh;
    const float *reg = p.reg;
    const int tid = threadIdx.x, o = tid & 127, rh = tid >> 7;
    constexpr int kHalf = kHeadRows / 2;
    const int total = unit_prefix<kWaves>(M.K, items, [&](int kk) { return p.live_cnt[M.order[kk]] + 1; });
    unit_prefix<kWaves>(M.K, units, [&](int kk) {
        const int k = M.order[kk];
        return (p.live_cnt[k] + 1) * reg_parts(p, k);
    });
    for (int b0 = blockIdx.x * kHeadRows; b0 < total; b0 += gridDim.x * kHeadRows) {
        __syncthreads();   // the previous pass is done with LDS
        if (tid < kHeadRows) {
            const int q = min(b0 + tid, total - 1);
            int lo = 0, hi = M.K - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (items[mid] <= q) lo = mid;
                else hi = mid - 1;
            }
            const int k = M.order[lo], local = q - items[lo], parts = reg_parts(p, k);
            row0[tid] = units[lo] + local * parts;
            rows[tid] = parts;
            out[tid] = local == p.live_cnt[k] ? -1 - k : p.live[(size_t)k * p.E + local] * M.K + k;
        }
        __syncthreads();
        for (int idx = tid; idx < kHeadRows * 64; idx += 256) {
            const int r = idx >> 6, c4 = idx & 63, f = row0[r], n = rows[r];
            float m = p.ml[f].x;
            for (int t = 1; t < n; ++t) m = fmaxf(m, p.ml[f + t].x);
            float l = 0.0f;
            floatx4 v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
            for (int t = 0; t < n; ++t) {
                const float2 ml = p.ml[f + t];
                const floatx4 a = *reinterpret_cast<const floatx4 *>(p.pooled + (size_t)(f + t) * 256 + 4 * c4);
                const float w = __expf(ml.x - m);
                l += w * ml.y;
                v += w * a;
            }
            *reinterpret_cast<floatx4 *>(&G[r][4 * c4]) = v * (1.0f / l);
        }
        float a[kHalf];
        const float bias = reg[kRd1 + o];
#pragma unroll
        for (int r = 0; r < kHalf; ++r) a[r] = bias;
        float next[16];
        auto request = [&](int c0) {
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const int idx = tid + 256 * t;
                next[t] = reg[kRD1 + (idx >> 5) * 256 + c0 + (idx & 31)];
            }
        };
        request(0);
#pragma unroll 1
        for (int c0 = 0; c0 < 256; c0 += 32) {
            __syncthreads();   // G written; DT free
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const int idx = tid + 256 * t;
                DT[idx & 31][idx >> 5] = next[t];
            }
            __syncthreads();
            request(min(c0 + 32, 224));
#pragma unroll 2
            for (int cc = 0; cc < 32; cc += 4) {
                const float w0 = DT[cc][o], w1 = DT[cc + 1][o], w2 = DT[cc + 2][o], w3 = DT[cc + 3][o];
#pragma unroll
                for (int r = 0; r < kHalf; ++r) {
                    const floatx4 g = *reinterpret_cast<const floatx4 *>(&G[rh * kHalf + r][c0 + cc]);
                    a[r] += w0 * g[0];
                    a[r] += w1 * g[1];
                    a[r] += w2 * g[2];
                    a[r] += w3 * g[3];
                }
            }
        }
#pragma unroll
        for (int r = 0; r < kHalf; ++r) H[rh * kHalf + r][o] = relu1(a[r]);
        __syncthreads();
        if (tid < kHeadRows * 8) {
            const int r = tid >> 3, j = tid & 7;
            if (b0 + r < total) {
                float y = reg[kRd2 + j];
                const float *d2 = reg + kRD2 + j * 128;
#pragma unroll 8
                for (int c = 0; c < 128; ++c) y += d2[c] * H[r][c];
                if (out[r] >= 0) taxels[(size_t)out[r] * 8 + j] = y;
                else rest[(size_t)(-1 - out[r]) * 8 + j] = y;
            }
        }
    }
}

__global__ __launch_bounds__(256) void k_regress_fill(const int32_t *n_active, const float *rest, int E, int K,
                                                      float *taxels) {
    const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (t >= (size_t)E * K * 8) return;
    const size_t item = t >> 3;
    if (n_active[item] == 0) taxels[t] = rest[(item % (size_t)K) * 8 + (t & 7)];
}

hipError_t launch_regress(const Plan &pl, const float *reg, int n_envs, const float *u, const int32_t *n_active,
                          float *taxels, hipStream_t st) {
    if (n_envs == 0) return hipSuccess;
    const RegParams p{pl.mesh, reg, u, pl.reg_live, pl.reg_cnt, pl.reg_pooled, pl.reg_ml, pl.counter, n_envs, pl.reg_unit};
    const int items = pl.K + n_envs * pl.K;
    const int slot = timer_begin(pl, ETAC_TIMER_REGRESS, st);
    launch_live(n_active, n_envs, pl.K, pl.reg_live, pl.reg_cnt, st);
    hipLaunchKernelGGL(k_regress, dim3(pl.cu_count), dim3(kRegWG), 0, st, p);
    hipError_t e = hipGetLastError();
    timer_end(pl, ETAC_TIMER_REGRESS, slot, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_regress_head, dim3(min(2 * pl.cu_count, (items + kHeadRows - 1) / kHeadRows)), dim3(256), 0, st, p, taxels,
                       pl.reg_rest);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t nt = (size_t)n_envs * pl.K * 8;
    hipLaunchKernelGGL(k_regress_fill, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, st, n_active, pl.reg_rest,
                       n_envs, pl.K, taxels);
    return hipGetLastError();
}

}  // namespace etac
