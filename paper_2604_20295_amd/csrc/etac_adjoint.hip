// Adjoint of the ETac step on gfx950: everything but the node pass.  For
// L = sum_i g_i . U_i, contact, tables and lists are made as in the forward,
// the pooled features read from its record or pooled again, and then
//   1. k_adj_wide / k_adj_narrow / k_adj_far : Eq. 1, transposed.  An active
//      node j gets g_j + sum over passive i of w_ij g_i, and
//      dL/dalpha_k = -sum_j u_hat_j . sum_i d_ij w_ij g_i.  W and d W are
//      symmetric, so these are products of the forward's matrices with the
//      passive nodes' g (far patches pair by pair).
//   2. k_adj_passive : the decoder's adjoint at passive nodes.  With
//      h4 = relu(W4 f + c4) and dL/dpre4 = (W5^T g) [h4 > 0] per env and node,
//      f is the same in every env: only sum over envs of dL/dpre4 is kept per
//      node, and per item its sum over nodes (s4 = db4).  dW5 and db5 here.
//   3. k_adj_item : per item the global MLP's adjoint from s4, and the
//      max-pool's routes: channel c's gradient goes to its arg-max node,
//      whatever it is, and to u_hat where that node is active.
//   4. k_adj_nodes (etac_backward.hip) : the encoder's adjoint at passive nodes,
//      once per node for all envs, from the sums of 2.
//   5. k_adj_contact : dL/d(R, t) of every winning object from dL/du_hat of its
//      active nodes, in FP64.
//   6. sums over items, nodes and workgroups in a fixed order.
// Every sum has an order fixed by the sizes of the call: results do not depend
// on which workgroup ran when.
#include <algorithm>

#include "etac_adjoint.h"

namespace etac {

// ---------------------------------------------------------------------------
// Eq. 1
// ---------------------------------------------------------------------------

// Pair-by-pair form of one active node, where a matrix would overflow: the
// sums with w and with d w.
__device__ void pair_adjoint(const AdjParams &p, int k, int e, int j, double (&a)[3], double (&b)[3]) {
    const MeshDev &M = p.s.mesh;
    const int N = M.N, base = M.offset[k], n = M.offset[k + 1] - base;
    const size_t EN = (size_t)p.s.E * N, row = (size_t)e * N + base;
    const unsigned long long *mask = p.s.itm.mask + (size_t)e * p.s.tile.NW + p.s.tile.word_off[k];
    float hi, lo;
    decay_rate(p.s.model.alpha[k], hi, lo);
#pragma unroll
    for (int c = 0; c < 3; ++c) a[c] = b[c] = 0.0;
    for (int i = 0; i < n; ++i) {
        if ((mask[i >> 6] >> (i & 63)) & 1ull) continue;
        float d;
        const double w = decay_weight_wide(M.pos[base + i] - M.pos[base + j], M.pos[N + base + i] - M.pos[N + base + j],
                                     M.pos[2 * N + base + i] - M.pos[2 * N + base + j], hi, lo, d);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const double wg = w * (double)p.grad_u[c * EN + row + i];      // beyond FP32's range here
            a[c] += wg;
            b[c] += (double)d * wg;
        }
    }
}

// The active rows of an env's four summed pair by pair (no register indexed at
// run time).
__device__ void pair_rows(const AdjParams &p, int k, int e, int i0, unsigned todo, doublex4 (&q)[3], doublex4 (&qd)[3]) {
    for (; todo; todo &= todo - 1) {
        const int row = __ffs(todo) - 1;
        double a[3], b[3];
        pair_adjoint(p, k, e, i0 + row, a, b);
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                q[c][x] = x == row ? a[c] : q[c][x];
                qd[c][x] = x == row ? b[c] : qd[c][x];
            }
    }
}

// Four consecutive values, the last ones 0 where fewer than four are left.
__device__ __forceinline__ floatx4 load4(const float *x, int left) {
    floatx4 v = {0.0f, 0.0f, 0.0f, 0.0f};
    if (left >= 4) __builtin_memcpy(&v, x, 16);
    else
#pragma unroll
        for (int i = 0; i < 3; ++i)
            if (i < left) v[i] = x[i];
    return v;
}

// dL/du_hat of the four consecutive nodes from local node i0 of one env: own
// gradient plus the decay part; active nodes only.  Returns their part of
// dL/dalpha (qd: the sums with d w).
__device__ __forceinline__ double finish_rows(const AdjParams &p, int k, int e, int base, int i0, int left,
                                              doublex4 (&q)[3], doublex4 (&qd)[3], bool dec, bool slow) {
    const int N = p.s.mesh.N, w0 = p.s.tile.word_off[k];
    const size_t EN = (size_t)p.s.E * N, at = (size_t)e * N + base + i0;
    // bits beyond the patch are clear
    const unsigned act = (unsigned)(p.s.itm.mask[(size_t)e * p.s.tile.NW + w0 + (i0 >> 6)] >> (i0 & 63)) & 0xfu;
    if (dec && (slow || not_finite(q) || not_finite(qd))) pair_rows(p, k, e, i0, act, q, qd);
    const float *u = uhat_source(p.s) + at;
    double da = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const floatx4 g = load4(p.grad_u + c * EN + at, left), uh = load4(u + c * EN, left);
#pragma unroll
        for (int x = 0; x < 4; ++x)
            if (((act >> x) & 1u) && dec) da -= (double)uh[x] * qd[c][x];
        const floatx4 o = dec ? __builtin_convertvector(widen(g) + q[c], floatx4) : g;
        float *out = p.gh + c * EN + at;
        if (act == 0xfu) {
            __builtin_memcpy(out, &o, 16);
        } else {
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if ((act >> x) & 1u) out[x] = o[x];
        }
    }
    return da;
}

// Wide tiles: 64 rows (a wave takes a row tile) times 32 envs, as the forward's,
// each B fragment against W and d W.  Bound by the matrix cores (4096 hands:
// 35.6 M MFMAs, 232 us at full rate) and the VALU beside them (the FP64 sums, and
// the reading and splitting of the envs' values): 672 us, 562 us with FP32 sums.
struct AdjWideLds {
    int first[kMaxPatches + 1];
    int env[32];
    ProductB b;
};

__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(2))) void k_adj_wide(AdjParams p) {
    __shared__ AdjWideLds L;
    const StepParams &S = p.s;
    const MeshDev &M = S.mesh;
    const TileDev &T = S.tile;
    const int K = M.K, N = M.N, lane = lane_id(), wave = uniform(threadIdx.x >> 6), gq = lane >> 4, col = lane & 15;
    const size_t EN = (size_t)S.E * N;
    const bool dec = step_decay(S);
    const int32_t *na = S.itm.n_act;
    const int total = product_units(S, L.first, 64, 32);
    for (int q = blockIdx.x; q < total; q += gridDim.x) {
        const ProductRef ref = product_ref(S, L.first, q, 64);
        const int k = ref.k, g0 = ref.group * 32;
        const int base = uniform(M.offset[k]), n = uniform(M.offset[k + 1]) - base, KS = (n + 31) >> 5;
        const int cnt = uniform(live_count(S, k));
        const int w0 = uniform(T.word_off[k]);
        __syncthreads();      // the previous unit is done with L
        if (threadIdx.x < 32) {
            const int e = g0 + threadIdx.x < cnt ? live_env(S, k, g0 + threadIdx.x) : -1;
            L.env[threadIdx.x] = (e >= 0 && S.dense && na[(size_t)e * K + k] == 0) ? -1 : e;
        }
        __syncthreads();
        int env[2];
        env[0] = L.env[col];
        env[1] = L.env[16 + col];
        const int rt = 4 * ref.row_block + wave, rts = (n + 15) >> 4;
        doublex4 acc[2][2][3];     // [W or d W][column tile][component]
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int c = 0; c < 3; ++c) acc[m][t][c] = doublex4{0.0, 0.0, 0.0, 0.0};
        const bool slow = matrix_overflows(M, S.model.alpha[k], k);
        if (dec && !slow) {
            const int mine = 16 * (wave & 1) + col, myenv = L.env[mine], safe = max(myenv, 0);
            const unsigned long long *mask = S.itm.mask + (size_t)safe * T.NW + w0;
            // rows beyond the patch repeat its last tile
            const size_t w_at = T.w_off[k] + (size_t)min(rt, rts - 1) * KS * 3 * 64 + lane;
            const uint4 *wa[2] = {S.tab.w + w_at, S.tab.wd + w_at};
            product_loop<2, true, 2>(L.b, wa, p.grad_u, (size_t)safe * N + base, EN, mask, myenv >= 0, n, KS, acc);
        }
        if (rt >= rts) continue;      // no barrier before the next unit's first
        const int i0 = 16 * rt + 4 * gq;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int e = env[t];
            double da = 0.0;
            if (e >= 0 && i0 < n) da = finish_rows(p, k, e, base, i0, n - i0, acc[0][t], acc[1][t], dec, slow);
            da += __shfl_xor(da, 16);
            da += __shfl_xor(da, 32);
            if (e >= 0) p.b.alpha_part[(size_t)e * T.NP + T.part_off[k] + rt] = da;      // the same in the 4 lane groups
        }
    }
}

// Narrow tiles: 16 rows times 16 envs, the K steps split over four waves.
struct AdjNarrowLds {
    int first[kMaxPatches + 1];
    doublex4 part[kWaves][6][64];
};

__global__ __launch_bounds__(kWG) void k_adj_narrow(AdjParams p) {
    __shared__ AdjNarrowLds L;
    const StepParams &S = p.s;
    const MeshDev &M = S.mesh;
    const TileDev &T = S.tile;
    const int K = M.K, N = M.N, lane = lane_id(), wave = uniform(threadIdx.x >> 6), gq = lane >> 4, col = lane & 15;
    const size_t EN = (size_t)S.E * N;
    const bool dec = step_decay(S);
    const int32_t *na = S.itm.n_act;
    const int total = unit_prefix<kWaves>(K, L.first, [&](int kk) {
        const int k = M.order[kk], n = M.offset[k + 1] - M.offset[k];
        return T.w_off[k] < 0 ? 0 : ((live_count(S, k) + 15) >> 4) * ((n + 15) >> 4);
    });
    for (int q = blockIdx.x; q < total; q += gridDim.x) {
        const int kk = unit_rank(L.first, K, q), k = uniform(M.order[kk]);
        const int base = uniform(M.offset[k]), n = uniform(M.offset[k + 1]) - base, KS = (n + 31) >> 5;
        const int cnt = uniform(live_count(S, k)), groups = (cnt + 15) >> 4;
        const int local = q - uniform(L.first[kk]), rt = local / groups, g0 = (local - rt * groups) * 16;
        const int w0 = uniform(T.word_off[k]);
        int e = g0 + col < cnt ? live_env(S, k, g0 + col) : -1;
        if (e >= 0 && S.dense && na[(size_t)e * K + k] == 0) e = -1;
        if (!__ballot(e >= 0)) continue;      // the same in every wave
        doublex4 acc[2][3];
#pragma unroll
        for (int m = 0; m < 2; ++m)
#pragma unroll
            for (int c = 0; c < 3; ++c) acc[m][c] = doublex4{0.0, 0.0, 0.0, 0.0};
        const bool slow = matrix_overflows(M, S.model.alpha[k], k);
        if (dec && !slow) {
            const size_t at = T.w_off[k] + (size_t)rt * KS * 3 * 64 + lane;
            const uint4 *wa[2] = {S.tab.w + at, S.tab.wd + at};
            const int safe = max(e, 0);
            const float *me = p.grad_u + (size_t)safe * N + base;
            const unsigned long long *mymask = S.itm.mask + (size_t)safe * T.NW + w0;
            uint4 a[2][3];
            float raw[3][8];
            unsigned bits = 0;
            auto fetch = [&](int s) {      // the next step's operands are requested before this one's are used
                const int j0 = 32 * s + 8 * gq;
                const bool in = e >= 0 && j0 < n;
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int c = 0; c < 3; ++c) a[m][c] = wa[m][(size_t)(s * 3 + c) * 64];
                bits = in ? ~(unsigned)(mymask[j0 >> 6] >> (j0 & 63)) & 0xffu : 0u;
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (in) load8(me + c * EN, j0, n, raw[c]);
            };
            if (wave < KS) fetch(wave);
            for (int s = wave; s < KS; s += kWaves) {
                bf16x8 b[3][3], y[2][3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    y[0][c] = __builtin_bit_cast(bf16x8, a[0][c]);
                    y[1][c] = __builtin_bit_cast(bf16x8, a[1][c]);
#pragma unroll
                    for (int x = 0; x < 8; ++x) raw[c][x] = (bits >> x) & 1u ? raw[c][x] : 0.0f;
                    split_bf16x3(raw[c], b[c]);
                }
                if (s + kWaves < KS) fetch(s + kWaves);
#pragma unroll
                for (int m = 0; m < 2; ++m)
#pragma unroll
                    for (int c = 0; c < 3; ++c) acc[m][c] += widen(mfma_bf16x3(y[m], b[c], floatx4{0.0f, 0.0f, 0.0f, 0.0f}));
            }
        }
        __syncthreads();          // the previous unit is done with L.part
#pragma unroll
        for (int f = 0; f < 6; ++f) L.part[wave][f][lane] = acc[f / 3][f % 3];
        __syncthreads();
        if (wave == 0) {          // a whole wave: lanes without an env take part in the shuffles
            const int i0 = 16 * rt + 4 * gq;
#pragma unroll
            for (int f = 0; f < 6; ++f) {
                doublex4 v = L.part[0][f][lane];
                for (int w = 1; w < kWaves; ++w) v += L.part[w][f][lane];
                acc[f / 3][f % 3] = v;
            }
            double da = 0.0;
            if (e >= 0 && i0 < n) da = finish_rows(p, k, e, base, i0, n - i0, acc[0], acc[1], dec, slow);
            da += __shfl_xor(da, 16);
            da += __shfl_xor(da, 32);
            if (e >= 0) p.b.alpha_part[(size_t)e * T.NP + T.part_off[k] + rt] = da;
        }
    }
}

// Far patches: a workgroup takes 256 active nodes of an item in the spatial
// order, a wave 64 of them, a lane one; the passive nodes' runs of 32 as in
// the forward.  An item has work in the tiles of its active nodes alone (6 of 64
// on 16384-node patches): taken item by item, a workgroup's stride over the units
// met the same tile every time, and one workgroup in ten had all of the work
// (384 scenes of four such patches: 15000 us, tile by tile 1740 us).
struct AdjFarLds {
    int first[kMaxPatches + 1];
    float4 a[kWaves][64];
    float2 b[kWaves][64];
};

__global__ __launch_bounds__(kWG) void k_adj_far(AdjParams p) {
    __shared__ AdjFarLds L;
    const StepParams &S = p.s;
    const MeshDev &M = S.mesh;
    const TileDev &T = S.tile;
    const int K = M.K, N = M.N, lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const size_t EN = (size_t)S.E * N;
    const bool dec = step_decay(S);
    const float *src = uhat_source(S);
    const int32_t *na = S.itm.n_act;
    const int total = unit_prefix<kWaves>(K, L.first, [&](int kk) {
        const int k = M.order[kk];
        return T.w_off[k] < 0 ? live_count(S, k) * ((M.offset[k + 1] - M.offset[k] + kWG - 1) / kWG) : 0;
    });
    for (int q = blockIdx.x; q < total; q += gridDim.x) {
        const int kk = unit_rank(L.first, K, q), k = uniform(M.order[kk]);
        const int base = uniform(M.offset[k]), n = uniform(M.offset[k + 1]) - base;
        // tile by tile, so that the tiles beyond an item's active nodes fall on every workgroup
        const int cnt = uniform(live_count(S, k)), local = q - uniform(L.first[kk]), tile = local / cnt;
        const int e = uniform(live_env(S, k, local - tile * cnt));
        const size_t item = (size_t)e * K + k, row = (size_t)e * N + base;
        const int m = uniform(na[item]);
        if (m == 0) continue;
        const int chunk = tile * kWaves + wave, s = chunk * 64 + lane;
        if (chunk * 64 >= n) continue;
        double *ap = p.b.alpha_part + (size_t)e * T.NP + T.part_off[k] + chunk;
        if (chunk * 64 >= m) {
            *ap = 0.0;            // every lane stores the same value
            continue;
        }
        const bool on = s < m;
        const int node = S.itm.alist[row + (on ? s : m - 1)], g = base + node;
        const float px = M.pos[g], py = M.pos[N + g], pz = M.pos[2 * N + g];
        const float ux = src[row + node], uy = src[EN + row + node], uz = src[2 * EN + row + node];
        double a0 = 0.0, a1 = 0.0, a2 = 0.0, da = 0.0;
        if (dec) {
            const float alpha = S.model.alpha[k], cut2 = cutoff_d2(alpha);
            float hi, lo;
            decay_rate(alpha, hi, lo);
            const int np = n - m;
            NearRuns runs(S.itm.pbox + 2 * ((size_t)e * S.itm.NB + S.itm.box_off[k]), (np + 31) >> 5, true, px, py, pz, cut2);
            const int *list = S.itm.plist + row;
            RunPair next;
            next.fetch(runs, M, list, np, base, p.grad_u + row, EN);
            while (next.r[0] >= 0) {
                const int c[2] = {next.c[0], next.c[1]};
                wave_sync();
                L.a[wave][lane] = make_float4(next.x[0], next.x[1], next.x[2], next.x[3]);
                L.b[wave][lane] = make_float2(next.x[4], next.x[5]);
                wave_sync();
                next.fetch(runs, M, list, np, base, p.grad_u + row, EN);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, t0 = 0.0f, t1 = 0.0f, t2 = 0.0f;
#pragma unroll 4
                    for (int i = 32 * h; i < 32 * h + c[h]; ++i) {
                        const float4 pa = L.a[wave][i];
                        const float2 pb = L.b[wave][i];
                        const float dx = pa.x - px, dy = pa.y - py, dz = pa.z - pz;
                        const float d = __builtin_amdgcn_sqrtf(dx * dx + dy * dy + dz * dz);
                        const float w = __builtin_amdgcn_exp2f(hi * d), dw = d * w;
                        s0 += w * pa.w; s1 += w * pb.x; s2 += w * pb.y;
                        t0 += dw * pa.w; t1 += dw * pb.x; t2 += dw * pb.y;
                    }
                    a0 += s0; a1 += s1; a2 += s2;
                    da -= t0 * ux + t1 * uy + t2 * uz;
                }
            }
        }
        if (on) {
            p.gh[row + node] = (float)((double)p.grad_u[row + node] + a0);
            p.gh[EN + row + node] = (float)((double)p.grad_u[EN + row + node] + a1);
            p.gh[2 * EN + row + node] = (float)((double)p.grad_u[2 * EN + row + node] + a2);
        }
        da = on ? da : 0.0;
        for (int off = 32; off >= 1; off >>= 1) da += __shfl_xor(da, off);
        *ap = da;
    }
}

// ---------------------------------------------------------------------------
// decoder's adjoint at passive nodes
// ---------------------------------------------------------------------------

// A wave takes 32 consecutive nodes (a half word) and the envs of one chunk in
// contact on their patch; lane c holds channel c: W4 f of the 32 nodes and the
// sums of dL/dpre4 over the envs stay in registers (FP64, as every sum over
// envs), the nodes' g are broadcast from LDS.  Thirteen VALU operations per env,
// passive node and channel; VALU-bound.
struct PassLds {
    int first[kMaxPatches + 1];
    float4 g[kWaves][2][32];
    double w5[kWaves][256];
};

__global__ __launch_bounds__(kWG) void k_adj_passive(AdjParams p) {
    __shared__ PassLds L;
    const StepParams &S = p.s;
    const MeshDev &M = S.mesh;
    const TileDev &T = S.tile;
    const int K = M.K, N = M.N, lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const size_t EN = (size_t)S.E * N;
    const float *phi = S.model.phi;
    const float w50 = phi[kW5 + lane], w51 = phi[kW5 + 64 + lane], w52 = phi[kW5 + 128 + lane];
    const int32_t *na = S.itm.n_act;
    const int EC = p.env_chunk;
    const int total = unit_prefix<kWaves>(K, L.first, [&](int kk) {
        const int k = M.order[kk], n = M.offset[k + 1] - M.offset[k];
        return ((live_count(S, k) + EC - 1) / EC) * ((n + 127) >> 7);
    });
    for (int q = blockIdx.x; q < total; q += gridDim.x) {
        const int kk = unit_rank(L.first, K, q), k = uniform(M.order[kk]);
        const int base = uniform(M.offset[k]), n = uniform(M.offset[k + 1]) - base;
        const int cnt = uniform(live_count(S, k)), chunks = (cnt + EC - 1) / EC;
        const int local = q - uniform(L.first[kk]), nb = local / chunks, ch = local - nb * chunks;
        const int hw = 4 * nb + wave, i0 = 32 * hw;
        const int w0 = uniform(T.word_off[k]), left = max(0, min(32, n - i0));
        const unsigned all = left >= 32 ? ~0u : (1u << left) - 1u;
        float z[32];
        double s[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            z[i] = S.tab.dec[(size_t)(base + min(i0 + i, n - 1)) * 64 + lane];
            s[i] = 0.0;
        }
        double w0s = 0.0, w1s = 0.0, w2s = 0.0, b0 = 0.0, b1 = 0.0, b2 = 0.0;
        const int q0 = ch * EC, q1 = left ? min(cnt, q0 + EC) : q0;      // a wave beyond the patch has nothing to add
        // the next env's operands are requested while this one's are used
        float g0, g1, g2, c4;
        unsigned act;
        int e;
        auto fetch = [&](int qq) {
            e = uniform(live_env(S, k, qq));
            const size_t at = (size_t)e * N + base + min(i0 + (lane & 31), n - 1);
            g0 = p.grad_u[at];
            g1 = p.grad_u[EN + at];
            g2 = p.grad_u[2 * EN + at];
            c4 = S.itm.c4[((size_t)e * K + k) * 64 + lane];
            act = (unsigned)(S.itm.mask[(size_t)e * T.NW + w0 + (hw >> 1)] >> (32 * (hw & 1)));
            if (S.dense && na[(size_t)e * K + k] == 0) act = ~0u;      // not in contact: nothing passive
        };
        if (q0 < q1) fetch(q0);
        for (int qq = q0; qq < q1; ++qq) {
            const unsigned pas = uniform(all & ~act);
            const int ce = e, buf = qq & 1;
            const float c = c4;
            if (lane < 32) {
                const bool on = (pas >> lane) & 1u;
                L.g[wave][buf][lane] = make_float4(g0, g1, g2, 0.0f);
                b0 += (double)(on ? g0 : 0.0f);
                b1 += (double)(on ? g1 : 0.0f);
                b2 += (double)(on ? g2 : 0.0f);
            }
            wave_sync();
            if (qq + 1 < q1) fetch(qq + 1);
            float s4 = 0.0f, a0 = 0.0f, a1 = 0.0f, a2 = 0.0f;      // over the nodes of one item
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                if (!((pas >> i) & 1u)) continue;      // wave-uniform
                const float4 g = L.g[wave][buf][i];
                const float t = z[i] + c;
                const float h = relu1(t);
                const float v = w50 * g.x + w51 * g.y + w52 * g.z;
                const float d = t > 0.0f ? v : 0.0f;
                s[i] += (double)d;
                s4 += d;
                a0 += g.x * h;
                a1 += g.y * h;
                a2 += g.z * h;
            }
            p.b.s4_part[((size_t)ce * 2 * T.NW + 2 * w0 + hw) * 64 + lane] = s4;
            w0s += (double)a0;
            w1s += (double)a1;
            w2s += (double)a2;
        }
        double *so = p.b.s4_node + ((size_t)ch * N + base + i0) * 64 + lane;
#pragma unroll
        for (int i = 0; i < 32; ++i)
            if (i < left) so[(size_t)i * 64] = s[i];
        // db5: sums over the 32 node lanes (lanes 32 .. 63 hold zeros)
        for (int off = 32; off >= 1; off >>= 1) {
            b0 += __shfl_xor(b0, off);
            b1 += __shfl_xor(b1, off);
            b2 += __shfl_xor(b2, off);
        }
        __syncthreads();      // the previous unit's sums are read
        L.w5[wave][lane] = w0s;
        L.w5[wave][64 + lane] = w1s;
        L.w5[wave][128 + lane] = w2s;
        L.w5[wave][192 + lane] = lane == 0 ? b0 : lane == 1 ? b1 : lane == 2 ? b2 : 0.0;
        __syncthreads();
        double v = L.w5[0][threadIdx.x];
        for (int w = 1; w < kWaves; ++w) v += L.w5[w][threadIdx.x];
        p.b.w5_part[((size_t)ch * T.NB5 + uniform(T.blk5_off[k]) + nb) * 256 + threadIdx.x] = v;
    }
}

// ---------------------------------------------------------------------------
// global MLP and max-pool routes of the items
// ---------------------------------------------------------------------------

// A wave per item.  Lane c first holds channel c: s4, dg' = W4[:, 64:]^T s4,
// dpre3 = dg' [g' > 0], dg = W3^T dpre3, and the inputs of the channel's
// arg-max node.  Then lane f holds feature f: h1 of every channel's node, and
// from dL/dpre2 = dg_c [g_c > 0] e_c its shares of dW2, dW1 and db1, summed in
// registers over the wave's items, in FP64.  Then again by channels: W1^T dL/dpre1
// reaches u_hat of active arg-max nodes.  An item is one dependent chain, so
// the weights are in LDS and everything it reads is requested first (4096
// hands: 161 us with weights from L2 and loads in turn, 102 us).
struct ItemLds {
    alignas(16) float w1u[64][4];     // W1[:, 6..8]
    float x[kWaves][64][12];          // inputs of the channels' nodes, then the routed gradient
    float d[kWaves][64][4];           // dL/du_hat of the channels' nodes, and the node
    unsigned long long gate[kWaves][64];   // features of a channel's node with h1 > 0
    union {
        struct {
            float w2[64][65];         // W2, rows and columns read without bank conflicts
            float w3[64][64], w4[64][64];      // W3, W4[:, 64:]
        };
        double sum[kRouteWords];      // after the items
    };
};
ETAC_LDS_ALIGNED(ItemLds, w1u);
ETAC_LDS_ALIGNED(ItemLds, x);
ETAC_LDS_ALIGNED(ItemLds, d);

// sum_c w[c][lane] x_c, four partial sums of 16 terms in order.
__device__ __forceinline__ float column_dot(const float (*w)[64], float x) {
    const int lane = lane_id();
    float s = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float a = 0.0f;
#pragma unroll
        for (int c = 0; c < 16; ++c)
            a += w[16 * q + c][lane] * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 16 * q + c));
        s += a;
        reload_fence();
    }
    return s;
}

__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(2))) void k_adj_item(AdjParams p) {
    __shared__ ItemLds L;
    __shared__ int first[kMaxPatches + 1];
    const StepParams &S = p.s;
    const MeshDev &M = S.mesh;
    const TileDev &T = S.tile;
    const int K = M.K, N = M.N, lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const size_t EN = (size_t)S.E * N;
    const float *phi = S.model.phi, *src = uhat_source(S);
    const int32_t *na = S.itm.n_act;
    const uint32_t *rec = S.recall ? S.recall : S.saved;
    for (int i = threadIdx.x; i < 4096; i += kWG) {
        L.w2[i >> 6][i & 63] = phi[kW2 + i];
        L.w3[i >> 6][i & 63] = phi[kW3 + i];
        L.w4[i >> 6][i & 63] = phi[kW4 + (i >> 6) * 128 + 64 + (i & 63)];
    }
    for (int i = threadIdx.x; i < 256; i += kWG) L.w1u[i >> 2][i & 3] = (i & 3) < 3 ? phi[kW1 + (i >> 2) * 9 + 6 + (i & 3)] : 0.0f;
    const int total = unit_prefix<kWaves>(K, first, [&](int kk) { return live_count(S, M.order[kk]); });
    float w1[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) w1[c] = phi[kW1 + lane * 9 + c];
    const float bias1 = phi[kB1 + lane];
    double acc2[64], accx[10], accb2 = 0.0;      // over the wave's items
#pragma unroll
    for (int c = 0; c < 64; ++c) acc2[c] = 0.0;
#pragma unroll
    for (int c = 0; c < 10; ++c) accx[c] = 0.0;
    for (int q = blockIdx.x * kWaves + wave; q < total; q += gridDim.x * kWaves) {
        const int kk = unit_rank(first, K, q), k = uniform(M.order[kk]);
        const int e = uniform(live_env(S, k, q - uniform(first[kk])));
        const size_t item = (size_t)e * K + k;
        if (S.dense && uniform(na[item]) == 0) continue;
        const int base = uniform(M.offset[k]), n = uniform(M.offset[k + 1]) - base;
        const int w0 = uniform(T.word_off[k]), hws = (n + 31) >> 5;
        // everything an item reads is requested before its first sums
        float *iv = p.b.ivec + item * 256 + lane;
        const float gp = iv[64], g = iv[192];
        const unsigned arg = rec[item * kSavedWords + 64 + lane];
        const float *sp = p.b.s4_part + ((size_t)e * 2 * T.NW + 2 * w0) * 64 + lane;
        float sv[32];
#pragma unroll
        for (int h = 0; h < 32; ++h) sv[h] = sp[(size_t)min(h, hws - 1) * 64];
        const bool ok = arg < (unsigned)n;      // a record not written for this item routes nothing
        const int a = ok ? (int)arg : 0, gi = base + a;
        float x[9];
        const unsigned long long am = S.itm.mask[(size_t)e * T.NW + w0 + (a >> 6)];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            x[c] = M.pos[(size_t)c * N + gi] - M.origin[3 * k + c];
            x[3 + c] = M.nrm[(size_t)c * N + gi];
            x[6 + c] = src[c * EN + (size_t)e * N + gi];
        }
        double sd = 0.0;
#pragma unroll
        for (int h = 0; h < 32; ++h) sd += h < hws ? (double)sv[h] : 0.0;
#pragma unroll 1
        for (int h0 = 32; h0 < hws; h0 += 32) {
#pragma unroll
            for (int h = 0; h < 32; ++h) sv[h] = sp[(size_t)min(h0 + h, hws - 1) * 64];
#pragma unroll
            for (int h = 0; h < 32; ++h) sd += h0 + h < hws ? (double)sv[h] : 0.0;
        }
        const float s4 = (float)sd;
        const float dgp = column_dot(L.w4, s4);
        const float dp3 = gp > 0.0f ? dgp : 0.0f;
        const float dg = column_dot(L.w3, dp3);
        iv[0] = s4;
        iv[128] = dp3;
        const float vr = (ok && g > 0.0f) ? dg : 0.0f;
        const bool act = ok && ((am >> (a & 63)) & 1ull);
        accb2 += (double)vr;
        wave_sync();
        {
            float *o = L.x[wave][lane];
            *reinterpret_cast<floatx4 *>(o) = floatx4{x[0], x[1], x[2], x[3]};
            *reinterpret_cast<floatx4 *>(o + 4) = floatx4{x[4], x[5], act ? x[6] : 0.0f, act ? x[7] : 0.0f};
            *reinterpret_cast<floatx2 *>(o + 8) = floatx2{act ? x[8] : 0.0f, vr};
        }
        wave_sync();
        float sx[10];      // this item's
#pragma unroll
        for (int c = 0; c < 10; ++c) sx[c] = 0.0f;
#pragma unroll
        for (int c = 0; c < 64; ++c) {
            const float w2c = L.w2[c][lane];      // read whether used or not: no branch
            const floatx4 xa = *reinterpret_cast<const floatx4 *>(&L.x[wave][c][0]);
            const floatx4 xb = *reinterpret_cast<const floatx4 *>(&L.x[wave][c][4]);
            const float x8 = L.x[wave][c][8], v = L.x[wave][c][9];
            float h = bias1;
            h += w1[0] * xa[0]; h += w1[1] * xa[1]; h += w1[2] * xa[2]; h += w1[3] * xa[3];
            h += w1[4] * xb[0]; h += w1[5] * xb[1]; h += w1[6] * xb[2]; h += w1[7] * xb[3];
            h += w1[8] * x8;
            acc2[c] += (double)(v * relu1(h));
            const float d = h > 0.0f ? v * w2c : 0.0f;
            sx[0] += d * xa[0]; sx[1] += d * xa[1]; sx[2] += d * xa[2]; sx[3] += d * xa[3];
            sx[4] += d * xb[0]; sx[5] += d * xb[1]; sx[6] += d * xb[2]; sx[7] += d * xb[3];
            sx[8] += d * x8;
            sx[9] += d;
            L.gate[wave][c] = __ballot(h > 0.0f);      // every lane stores the same value
            if ((c & 7) == 7) reload_fence();      // eight channels' operands in flight, not all 64
        }
#pragma unroll
        for (int c = 0; c < 10; ++c) accx[c] += (double)sx[c];
        if (__ballot(act && vr != 0.0f)) {
            wave_sync();
            const unsigned long long gate = L.gate[wave][lane];
            float d0 = 0.0f, d1 = 0.0f, d2 = 0.0f;
#pragma unroll 8
            for (int f = 0; f < 64; ++f) {
                const float w2f = L.w2[lane][f];
                const float d = (gate >> f) & 1ull ? vr * w2f : 0.0f;
                const floatx4 w = *reinterpret_cast<const floatx4 *>(&L.w1u[f][0]);
                d0 += w[0] * d;
                d1 += w[1] * d;
                d2 += w[2] * d;
            }
            // the lowest channel routed to a node adds all of its channels, in order
            *reinterpret_cast<floatx4 *>(&L.d[wave][lane][0]) = floatx4{d0, d1, d2, __int_as_float(ok ? a : -1)};
            wave_sync();
            bool own = act;
            float t0 = 0.0f, t1 = 0.0f, t2 = 0.0f;
#pragma unroll 8
            for (int c = 0; c < 64; ++c) {
                const floatx4 o = *reinterpret_cast<const floatx4 *>(&L.d[wave][c][0]);
                const bool same = __float_as_int(o[3]) == a;
                own = own && !(same && c < lane);
                t0 += same ? o[0] : 0.0f;
                t1 += same ? o[1] : 0.0f;
                t2 += same ? o[2] : 0.0f;
            }
            if (own) {
                float *gh = p.gh + (size_t)e * N + base + a;
                gh[0] += t0;
                gh[EN] += t1;
                gh[2 * EN] += t2;
            }
        }
    }
    // the workgroup's sums, waves in order
    __syncthreads();      // the weights are done with
    for (int w = 0; w < kWaves; ++w) {
        if (w == wave) {
#pragma unroll
            for (int c = 0; c < 64; ++c) L.sum[c * 64 + lane] = (w ? L.sum[c * 64 + lane] : 0.0) + acc2[c];
#pragma unroll
            for (int c = 0; c < 10; ++c)
                L.sum[4096 + c * 64 + lane] = (w ? L.sum[4096 + c * 64 + lane] : 0.0) + accx[c];
            L.sum[4736 + lane] = (w ? L.sum[4736 + lane] : 0.0) + accb2;
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i < kRouteWords; i += kWG) p.b.route[(size_t)blockIdx.x * kRouteWords + i] = L.sum[i];
}

// ---------------------------------------------------------------------------
// contact
// ---------------------------------------------------------------------------

// One half of the values of a lane added to another lane's, as halve_max.
template <int H, int CTRL>
__device__ __forceinline__ void halve_sum(double (&v)[16], bool bit) {
#pragma unroll
    for (int i = 0; i < H / 2; ++i) {
        const double keep = bit ? v[H / 2 + i] : v[i], give = bit ? v[i] : v[H / 2 + i];
        v[i] = keep + __hiloint2double(dpp<CTRL>(__double2hiint(give)), dpp<CTRL>(__double2loint(give)));
    }
}

// Sums of twelve values over the wave in a fixed order: lane l returns value l % 16.
__device__ __forceinline__ double wave_sums(const double (&x)[12]) {
    const int lane = lane_id();
    double v[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) v[c] = c < 12 ? x[c < 12 ? c : 0] : 0.0;
    halve_sum<16, kDppXor8>(v, lane & 8);
    halve_sum<8, kDppXor7>(v, lane & 4);
    halve_sum<4, kDppXor2>(v, lane & 2);
    halve_sum<2, kDppXor1>(v, lane & 1);
    double s = v[0];
    {      // rows 0 and 1, 2 and 3
        const auto l = __builtin_amdgcn_permlane16_swap(__double2loint(s), __double2loint(s), false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(__double2hiint(s), __double2hiint(s), false, false);
        s = __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
    }
    const auto l = __builtin_amdgcn_permlane32_swap(__double2loint(s), __double2loint(s), false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(__double2hiint(s), __double2hiint(s), false, false);
    return __hiloint2double(h[0], l[0]) + __hiloint2double(h[1], l[1]);
}

// A wave per chunk of kPoseWords words of an item: for every object that wins
// a node there, the sum over its nodes; exact zeros for the others.  An
// object's nodes are listed, so that every lane has one (a lane per node of a
// word left half of them idle in FP64), and the next 64 nodes' operands are
// requested while these are used.  4096 hands: 158 us a word at a time, 97 us.
__global__ __launch_bounds__(kWG) void k_adj_contact(AdjParams p) {
    __shared__ int first[kMaxPatches + 1];
    __shared__ uint16_t lists[kWaves][64 * kPoseWords];
    const StepParams &S = p.s;
    const MeshDev &M = S.mesh;
    const TileDev &T = S.tile;
    const SceneDev &C = S.scene;
    const int K = M.K, N = M.N, O = p.O, lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const size_t EN = (size_t)S.E * N;
    const int32_t *na = S.itm.n_act;
    uint16_t *list = lists[wave];
    const int total = unit_prefix<kWaves>(K, first, [&](int kk) {
        const int k = M.order[kk];
        return live_count(S, k) * (T.chunk_off[k + 1] - T.chunk_off[k]);
    });
    for (int q = blockIdx.x * kWaves + wave; q < total; q += gridDim.x * kWaves) {
        const int kk = unit_rank(first, K, q), k = uniform(M.order[kk]);
        const int c0 = uniform(T.chunk_off[k]), cnt_k = uniform(live_count(S, k));
        const int local = q - uniform(first[kk]), part = local / cnt_k, e = uniform(live_env(S, k, local - part * cnt_k));
        const size_t item = (size_t)e * K + k;
        if (S.dense && uniform(na[item]) == 0) continue;
        const int base = uniform(M.offset[k]), n = uniform(M.offset[k + 1]) - base;
        const int w0 = uniform(T.word_off[k]), nw = uniform(T.word_off[k + 1]) - w0;
        const int wf = part * kPoseWords, wl = min(nw, wf + kPoseWords);
        const size_t srow = scene_row(C, e, k), row = (size_t)e * N + base;
        const int no = min(uniform(C.n_obj[srow]), O);
        float *out = p.pose_part + ((size_t)e * T.NC + c0 + part) * O * 12;
        const unsigned long long *mask = S.itm.mask + (size_t)e * T.NW + w0;
        // this lane's winner in every word of the chunk, all requested at once (-1: not active)
        int win[kPoseWords];
        unsigned present = 0;
#pragma unroll
        for (int w = 0; w < kPoseWords; ++w) {
            const bool in = wf + w < wl;
            const unsigned long long act = mask[min(wf + w, nw - 1)];
            const int o = p.cobj[row + min(64 * (wf + w) + lane, n - 1)];
            win[w] = in && ((act >> lane) & 1ull) ? o : -1;
        }
#pragma unroll
        for (int w = 0; w < kPoseWords; ++w)
            if (win[w] >= 0) present |= 1u << (win[w] & 31);
        present = uniform(wave_or(present));
        for (int o = 0; o < O; ++o)
            if (o >= no || !((present >> o) & 1u))
                if (lane < 12) out[o * 12 + lane] = 0.0f;
        while (present) {
            const int o = __ffs(present) - 1;
            present &= present - 1;
            if (o >= no) continue;
            int cnt = 0;
            wave_sync();
#pragma unroll
            for (int w = 0; w < kPoseWords; ++w) {
                const unsigned long long bal = __ballot(win[w] == o);
                if (win[w] == o) list[cnt + lanes_below(bal)] = (uint16_t)(64 * w + lane);
                cnt += __popcll(bal);
            }
            wave_sync();
            double acc[12];
#pragma unroll
            for (int c = 0; c < 12; ++c) acc[c] = 0.0;
            const size_t eo = srow * C.O + o;
            const int ty = uniform(C.type[eo]);
            const float *sh = C.shape + 4 * eo, *R = C.rot + 9 * eo, *t = C.trans + 3 * eo;
            float g[3], x[3];
            auto fetch = [&](int t0) {      // beyond the list: its last node
                const int i = 64 * wf + list[min(t0 + lane, cnt - 1)];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    g[c] = p.gh[c * EN + row + i];
                    x[c] = M.pos[(size_t)c * N + base + i];
                }
            };
            fetch(0);
#pragma unroll 1
            for (int t0 = 0; t0 < cnt; t0 += 64) {
                const double gd[3] = {g[0], g[1], g[2]};
                const float px = x[0], py = x[1], pz = x[2];
                fetch(t0 + 64);
                if (t0 + lane < cnt) contact_adjoint_node(ty, sh, R, t, px, py, pz, gd, acc);
            }
            const double v = wave_sums(acc);
            if (lane < 12) out[o * 12 + lane] = (float)v;
        }
    }
}

// Pose gradients: sum over the env's parts in order.
__global__ __launch_bounds__(256) void k_pose(AdjParams p, float *grad_rot, float *grad_trans) {
    const TileDev &T = p.s.tile;
    const int K = p.s.mesh.K, O = p.O;
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (t >= p.s.E * O * 12) return;
    const int c = t % 12, eo = t / 12, o = eo % O, e = eo / O;
    double acc = 0.0;
    for (int k0 = 0; k0 < K; k0 += 8) {
        int n[8], h0[8], h1[8];      // eight patches' counts requested at once
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int k = min(k0 + t, K - 1);
            n[t] = p.s.itm.n_act[(size_t)e * K + k];
            h0[t] = T.chunk_off[k];
            h1[t] = T.chunk_off[k + 1];
        }
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if (n[t] == 0 || k0 + t >= K) continue;
            for (int h = h0[t]; h < h1[t]; ++h) acc += (double)p.pose_part[(((size_t)e * T.NC + h) * O + o) * 12 + c];
        }
    }
    if (c < 9) grad_rot[(size_t)eo * 9 + c] = (float)acc;
    else grad_trans[(size_t)eo * 3 + (c - 9)] = (float)acc;
}

// ---------------------------------------------------------------------------
// parameter sums
// ---------------------------------------------------------------------------

// Segment sums (FP64) of the reduction's columns: the node blocks' records,
// the routing workgroups' sums, the items' vectors (db4, db3, and the rank-one
// products dW4[:, 64:] = s4 g'^T, dW3 = dpre3 g^T), and dW5 / db5 by half word
// and chunk.  A block takes 256 columns of one kind and the entries of one
// segment, in ascending order.  The 8192 columns of the rank-one products are
// one block's, as matrix products in FP64 over the segment's items: a thread
// per column reads both vectors of every item for each of them (4096 hands, all
// columns: 170 us, 48 us as products).
__global__ __launch_bounds__(256) void k_phi_segments(AdjParams p, int route_groups, int segs) {
    __shared__ int list[1024];
    __shared__ int wsum[kWaves];
    const StepParams &S = p.s;
    const MeshDev &M = S.mesh;
    const TileDev &T = S.tile;
    const int K = M.K, s = blockIdx.y, lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    // one block for all columns of the items' vectors and their products
    const int first = blockIdx.x * 256 + (blockIdx.x > kRedItem / 256 ? kRedW5 - kRedRank : 0), col = first + threadIdx.x;
    double acc = 0.0;
    auto range = [&](long long n, long long &a, long long &b) {
        const long long per = (n + segs - 1) / segs;
        a = min(n, s * per);
        b = min(n, a + per);
    };
    long long a, b;
    if (first < kRedRoute) {
        range(T.NU, a, b);
        if (col < kNodeRecWords)
            for (long long u0 = a; u0 < b; u0 += 8) {
                bool live[8];      // eight blocks' flags requested at once
#pragma unroll
                for (int t = 0; t < 8; ++t) live[t] = u0 + t < b && live_count(S, T.block[min(u0 + t, b - 1)].x) > 0;
#pragma unroll
                for (int t = 0; t < 8; ++t)
                    if (live[t]) acc += (double)p.b.node_rec[(u0 + t) * kNodeRecWords + col];
            }
    } else if (first < kRedItem) {
        range(route_groups, a, b);
        const int c = col - kRedRoute;
        if (c < kRouteWords) {
#pragma unroll 4
            for (long long u = a; u < b; ++u) acc += p.b.route[u * kRouteWords + c];
        }
    } else if (first == kRedItem) {
        // items in contact, listed 1024 at a time
        range((long long)S.E * K, a, b);
        // wave w takes rows 32 (w & 1) .. + 31 of matrix w >> 1, and the sums of those rows' vector
        const int m = wave >> 1, l = lane & 15, sub = lane >> 4;
        const int ro = 128 * m + 32 * (wave & 1) + l, co = 64 + 128 * m + l;
        doublex4 d[2][5];
#pragma unroll
        for (int i = 0; i < 10; ++i) d[i / 5][i % 5] = doublex4{0.0, 0.0, 0.0, 0.0};
        for (long long c0 = a; c0 < b; c0 += 1024) {
            int cnt = 0;   // identical in every thread
            for (int j = 0; j < 4; ++j) {
                const long long it = c0 + j * 256 + threadIdx.x;
                const bool f = it < b && S.itm.n_act[it] > 0;
                const unsigned long long bal = __ballot(f);
                __syncthreads();   // the previous round's reads are done
                wsum[wave] = __popcll(bal);
                __syncthreads();
                int off = cnt, tot = 0;
                for (int v = 0; v < kWaves; ++v) {
                    if (v < wave) off += wsum[v];
                    tot += wsum[v];
                }
                if (f) list[off + lanes_below(bal)] = (int)(it - c0);
                cnt += uniform(tot);
            }
            __syncthreads();
            const float *iv = p.b.ivec + c0 * 256;
            for (int t = 0; t < cnt; t += 32) {      // eight steps of four items; lanes beyond the last hold zeros
                float x[8][2], y[8][4];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int at = t + 4 * u + sub;
                    const float *r = iv + (size_t)list[min(at, cnt - 1)] * 256;
#pragma unroll
                    for (int i = 0; i < 2; ++i) x[u][i] = r[ro + 16 * i];
#pragma unroll
                    for (int j = 0; j < 4; ++j) y[u][j] = r[co + 16 * j];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const bool in = t + 4 * u + sub < cnt;
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const double v = in ? (double)x[u][i] : 0.0;
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            d[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, in ? (double)y[u][j] : 0.0, d[i][j], 0, 0, 0);
                        d[i][4] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, 1.0, d[i][4], 0, 0, 0);
                    }
                }
            }
            __syncthreads();   // the list is rewritten
        }
        // register r of a lane: row 4 r + lane / 16, column lane % 16
        double *o = p.b.seg + (size_t)s * kRedCols + kRedRank + 4096 * m + (32 * (wave & 1) + sub) * 64 + l;
        double *sum = p.b.seg + (size_t)s * kRedCols + kRedItem + 64 * m + 32 * (wave & 1) + sub;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
#pragma unroll
                for (int j = 0; j < 4; ++j) o[(16 * i + 4 * r) * 64 + 16 * j] = d[i][j][r];
                sum[16 * i + 4 * r] = d[i][4][r];      // the same in every column
            }
        return;
    } else {
        range(T.NB5, a, b);
        const int c = col - kRedW5, EC = p.env_chunk;
        // the patch of the segment's first block
        int k = 0;
        for (int hi = K - 1; k < hi;) {
            const int mid = (k + hi + 1) >> 1;
            if (T.blk5_off[mid] <= a) k = mid;
            else hi = mid - 1;
        }
        for (long long h = a; h < b; ++h) {
            while (T.blk5_off[k + 1] <= h) ++k;
            const int chunks = (live_count(S, k) + EC - 1) / EC;
            const double *w = p.b.w5_part + (size_t)h * 256 + c;
#pragma unroll 8
            for (int t = 0; t < chunks; ++t) acc += w[(size_t)t * T.NB5 * 256];
        }
    }
    p.b.seg[(size_t)s * kRedCols + col] = acc;
}

// Slot of entry (row, col) of 16 x 16 block b in a node record (MFMA output order).
__device__ constexpr int rec_slot(int b, int row, int col) { return b * 256 + (16 * (row >> 2) + col) * 4 + (row & 3); }

// dL/dphi: the columns of each parameter over the segments, in order, B of them
// requested at once (4096 hands: 14.2 us eight at a time, 10.4 us at 32).
template <int B>
__global__ __launch_bounds__(256) void k_phi_final(const double *seg, int segs, float *grad_phi) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= kPhiN) return;
    int c1, c2 = -1;
    if (c < kB1) {
        const int o = c / 9, i = c % 9;
        c1 = rec_slot(32 + (o >> 4), o & 15, i);
        c2 = kRedRoute + 4096 + i * 64 + o;
    } else if (c < kW2) {
        const int o = c - kB1;
        c1 = rec_slot(32 + (o >> 4), o & 15, 9);
        c2 = kRedRoute + 4096 + 9 * 64 + o;
    } else if (c < kB2) {
        const int o = (c - kW2) >> 6, i = (c - kW2) & 63;
        c1 = rec_slot(16 + 4 * (o >> 4) + (i >> 4), o & 15, i & 15);
        c2 = kRedRoute + 64 * o + i;
    } else if (c < kW3) {
        c1 = 36 * 256 + (c - kB2);
        c2 = kRedRoute + 4736 + (c - kB2);
    } else if (c < kB3) {
        c1 = kRedRank + 4096 + (c - kW3);
    } else if (c < kW4) {
        c1 = kRedItem + 64 + (c - kB3);
    } else if (c < kB4) {
        const int o = (c - kW4) >> 7, i = (c - kW4) & 127;
        c1 = i < 64 ? rec_slot(4 * (o >> 4) + (i >> 4), o & 15, i & 15) : kRedRank + 64 * o + (i - 64);
    } else if (c < kW5) {
        c1 = kRedItem + (c - kB4);
    } else if (c < kB5) {
        c1 = kRedW5 + (c - kW5);
    } else {
        c1 = kRedW5 + 192 + (c - kB5);
    }
    double acc = 0.0, more = 0.0;
    const int cm = c2 >= 0 ? c2 : c1;
#pragma unroll 1
    for (int s0 = 0; s0 < segs; s0 += B) {
        double v[B], w[B];
#pragma unroll
        for (int t = 0; t < B; ++t) {
            const double *row = seg + (size_t)min(s0 + t, segs - 1) * kRedCols;
            v[t] = row[c1];
            w[t] = row[cm];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < B; ++t)
            if (s0 + t < segs) {
                acc += v[t];
                more += w[t];
            }
    }
    if (c2 >= 0) acc += more;
    grad_phi[c] = (float)acc;
}

__global__ __launch_bounds__(256) void k_zero(float *x, int n) {
    for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) x[i] = 0.0f;
}

// dL/dalpha_k: block (k, s) sums the parts of the envs of segment s, threads
// in turn, then a fixed tree; k_alpha_sum adds the segments.  Latency-bound:
// eight parts in flight (4096 hands: 18.6 us with their envs and values in turn,
// 8.0 us).
__global__ __launch_bounds__(256) void k_alpha(AdjParams p, float *grad_alpha, double *seg) {
    __shared__ double red[256];
    const StepParams &S = p.s;
    const TileDev &T = S.tile;
    const int k = blockIdx.x, cnt = live_count(S, k), off = T.part_off[k], parts = T.part_off[k + 1] - off;
    const int per = (cnt + gridDim.y - 1) / gridDim.y, q0 = blockIdx.y * per, q1 = min(cnt, q0 + per);
    double acc = 0.0;
    if (q0 < q1) {
        const int n = (q1 - q0) * parts;
        for (int i0 = threadIdx.x; i0 < n; i0 += 8 * 256) {      // eight parts in flight
            double v[8];
            int e[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) e[t] = live_env(S, k, q0 + min(i0 + 256 * t, n - 1) / parts);
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                v[t] = p.b.alpha_part[(size_t)e[t] * T.NP + off + min(i0 + 256 * t, n - 1) % parts];
                if (S.dense) v[t] = S.itm.n_act[(size_t)e[t] * S.mesh.K + k] == 0 ? 0.0 : v[t];
            }
#pragma unroll
            for (int t = 0; t < 8; ++t) acc += i0 + 256 * t < n ? v[t] : 0.0;
        }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (gridDim.y == 1) grad_alpha[k] = (float)red[0];
        else seg[(size_t)k * gridDim.y + blockIdx.y] = red[0];
    }
}

__global__ __launch_bounds__(256) void k_alpha_sum(const double *seg, int K, int segs, float *grad_alpha) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= K) return;
    double acc = 0.0;
#pragma unroll 8
    for (int s = 0; s < segs; ++s) acc += seg[(size_t)k * segs + s];
    grad_alpha[k] = (float)acc;
}

// ---------------------------------------------------------------------------
// host
// ---------------------------------------------------------------------------
static unsigned blocks(long long want, long long most) { return (unsigned)std::max<long long>(1, std::min(want, most)); }

hipError_t launch_backward(const Plan &pl, const SceneDev *s, const ModelDev &m, int n_envs, const int8_t *cobj_in,
                           const float *uhat_in, const float *grad_u, const uint32_t *saved, float *grad_uhat,
                           float *grad_rot, float *grad_trans, float *grad_alpha, float *grad_phi,
                           hipStream_t st, const SceneDev *world, const LinksDev *links, float *grad_link_rot,
                           float *grad_link_trans) {
    const bool res = m.mode != ETAC_DECAY_ONLY, dec = m.mode != ETAC_RESIDUAL_ONLY;
    if (grad_phi && (n_envs == 0 || !res))     // sums over no network adjoint
        hipLaunchKernelGGL(k_zero, dim3((kPhiN + 255) / 256), dim3(256), 0, st, grad_phi, kPhiN);
    if (n_envs == 0) {
        if (grad_alpha) hipLaunchKernelGGL(k_zero, dim3(1), dim3(256), 0, st, grad_alpha, pl.K);
        return hipGetLastError();
    }
    AdjParams p{};
    StepParams &f = p.s;
    f.scene = s ? *s : SceneDev{nullptr, nullptr, nullptr, nullptr, nullptr, 0, 1};
    f.model = m;
    f.E = n_envs;
    f.cobj_in = cobj_in;
    f.uhat_in = uhat_in;
    f.u = s ? pl.bwd.uhat_st : grad_uhat;
    f.scratch = s != nullptr;
    f.cobj_out = s ? pl.bwd.cobj_st : nullptr;
    f.adjoint = 1;
    f.ivec = pl.bwd.ivec;
    f.recall = saved;
    f.saved = saved ? nullptr : pl.bwd.record;
    shape_step(pl, f);
    p.b = pl.bwd;
    p.env_chunk = env_chunk(n_envs, pl.tile.NB5);
    p.O = s ? s->O : 1;
    p.grad_u = grad_u;
    p.gh = s ? pl.bwd.gh : grad_uhat;
    p.cobj = pl.bwd.cobj_st;
    // the hand's rows hold up to cap candidates: their own pose parts
    p.pose_part = links ? pl.hand->pose_part : pl.bwd.pose_part;
    const long long cus = f.cus, items = f.items;
    int slot = timer_begin(pl, ETAC_TIMER_BWD_DECAY, st);
    launch_front(pl, f, st);
    if (pl.tile.n_near) {
        // as in the forward: wide tiles once they give every CU work
        if (f.wide) hipLaunchKernelGGL(k_adj_wide, dim3(2 * f.cus), dim3(kWG), 0, st, p);
        else
            hipLaunchKernelGGL(k_adj_narrow, dim3(blocks((long long)((n_envs + 15) / 16) * pl.tile.near_rows, 4 * cus)),
                               dim3(kWG), 0, st, p);
    }
    if (pl.tile.n_far) {
        launch_far_lists(f, false, st);
        if (dec) launch_far_lists(f, true, st);
        hipLaunchKernelGGL(k_adj_far, dim3(blocks(f.words / 4 + items, 8 * cus)), dim3(kWG), 0, st, p);
    }
    timer_end(pl, ETAC_TIMER_BWD_DECAY, slot, st);
    slot = timer_begin(pl, ETAC_TIMER_BACKWARD, st);
    const int route_groups = (int)blocks((items + kWaves - 1) / kWaves, kRouteGroups * cus);
    if (res) {
        launch_pool(pl, f, st);
        hipLaunchKernelGGL(k_adj_passive, dim3(blocks((f.words / 2 + items) / p.env_chunk + pl.tile.NU + 1, 3 * cus)), dim3(kWG), 0, st, p);
        hipLaunchKernelGGL(k_adj_item, dim3(route_groups), dim3(kWG), 0, st, p);
        const hipError_t e = launch_adj_nodes(p, (int)blocks(pl.tile.NU, cus), st);
        if (e != hipSuccess) return e;
    }
    if (s) hipLaunchKernelGGL(k_adj_contact, dim3(blocks(((long long)n_envs * pl.tile.NC + 3) / 4, 8 * cus)), dim3(kWG), 0, st, p);
    timer_end(pl, ETAC_TIMER_BACKWARD, slot, st);
    slot = timer_begin(pl, ETAC_TIMER_REDUCE, st);
    if (res && grad_phi) {
        const int segs = f.dense && pl.tile.NU <= 64 ? 8 : kPhiSegs;
        hipLaunchKernelGGL(k_phi_segments, dim3((kRedCols - (kRedW5 - kRedRank)) / 256, segs), dim3(256), 0, st, p, route_groups, segs);
        if (segs <= 8)
            hipLaunchKernelGGL(k_phi_final<8>, dim3((kPhiN + 255) / 256), dim3(256), 0, st, pl.bwd.seg, segs, grad_phi);
        else
            hipLaunchKernelGGL(k_phi_final<32>, dim3((kPhiN + 255) / 256), dim3(256), 0, st, pl.bwd.seg, segs, grad_phi);
    }
    if (grad_alpha) {
        const int segs = f.dense ? 1 : kAlphaSegs;
        hipLaunchKernelGGL(k_alpha, dim3(pl.K, segs), dim3(256), 0, st, p, grad_alpha, pl.bwd.alpha_seg);
        if (segs > 1)
            hipLaunchKernelGGL(k_alpha_sum, dim3((pl.K + 255) / 256), dim3(256), 0, st, pl.bwd.alpha_seg, pl.K, segs, grad_alpha);
    }
    hipError_t e = hipSuccess;
    if (s && links) e = launch_pose_hand(pl, *world, *links, grad_rot, grad_trans, grad_link_rot, grad_link_trans, st);
    else if (s)
        hipLaunchKernelGGL(k_pose, dim3((n_envs * p.O * 12 + 255) / 256), dim3(256), 0, st, p, grad_rot, grad_trans);
    if (e == hipSuccess) e = hipGetLastError();
    timer_end(pl, ETAC_TIMER_REDUCE, slot, st);
    return e;
}

hipError_t launch_contact_backward(const Plan &pl, const SceneDev &s, const float *grad_uhat, float *grad_rot,
                                   float *grad_trans, hipStream_t st) {
    if (s.E == 0) return hipSuccess;
    AdjParams p{};
    StepParams &f = p.s;
    f.scene = s;
    f.model = ModelDev{ETAC_DECAY_ONLY, nullptr, nullptr};
    f.E = s.E;
    f.u = pl.bwd.uhat_st;
    f.scratch = 1;
    f.cobj_out = pl.bwd.cobj_st;
    f.adjoint = 1;
    shape_step(pl, f);
    f.matrix_units = 0;      // contact alone
    p.b = pl.bwd;
    p.O = s.O;
    p.gh = const_cast<float *>(grad_uhat);      // read only
    p.cobj = pl.bwd.cobj_st;
    p.pose_part = pl.bwd.pose_part;
    launch_front(pl, f, st);
    hipLaunchKernelGGL(k_adj_contact, dim3(blocks(((long long)s.E * pl.tile.NC + 3) / 4, 8 * (long long)f.cus)), dim3(kWG), 0, st, p);
    hipLaunchKernelGGL(k_pose, dim3((s.E * p.O * 12 + 255) / 256), dim3(256), 0, st, p, grad_rot, grad_trans);
    return hipGetLastError();
}

}  // namespace etac
