// Network adjoint's node pass on gfx950.
//
// At a passive node the encoder's features do not depend on the env, and its
// adjoint is linear in dL/dpre4.  So dL/dpre4, summed over the envs in contact
// (k_adj_passive), is carried through the encoder once per node and call:
//   dW4[:, :64] = sum_i dpre4_i (x) f_i,  dpre2 = (W4[:, :64]^T dpre4) [f > 0],
//   dW2, db2 from dpre2 and h1,  dpre1 = (W2^T dpre2) [h1 > 0],  dW1, db1.
// A workgroup takes kBlockNodes nodes of a patch at a time, a wave a 16-node
// tile of them, on split-FP16 MFMA, and writes the block's sums as a record.
//
// Built in a translation unit of its own, with MFMA results in VGPRs as well as
// AGPRs and instruction sinking: the accumulators and two tiles of activations
// take most of a lane's registers.
#include "etac_adjoint.h"

namespace etac {

constexpr int kTrRow = 20;     // padded row of the block transpose buffer: conflict-free stores, aligned loads

// ---------------------------------------------------------------------------
// wave-level tile algebra in two register layouts
//
// T form (the forward's): lane l holds node (l & 15) of a 16-node tile;
// register r of block b holds feature 16 b + 4 (l >> 4) + r.  It is the
// output of W X^T with the tile as the MFMA's B operand, and chains into the
// next layer as B.
// N form: lane l holds feature 16 b + (l & 15) of block b; register r holds
// node 4 (l >> 4) + r.  In N form the nodes sit in registers, so a weight
// gradient dW = sum_n a_n (x) b_n per 16 x 16 block takes both operands
// straight from the N-form registers.
// ---------------------------------------------------------------------------
typedef _Float16 half4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void split4(const floatx4 &v, half4 &hi, half4 &lo) {
    uint2t h, l;
    unsigned a, b, c, d;
    split2(v[0], v[1], a, b);
    split2(v[2], v[3], c, d);
    h[0] = a; h[1] = c;
    l[0] = b; l[1] = d;
    hi = __builtin_bit_cast(half4, h);
    lo = __builtin_bit_cast(half4, l);
}

// Weight-gradient operands: NB N-form blocks of a tile, split and packed as
// K = 32 MFMA operands (lane group q holds k = 8 q .. 8 q + 7; any k order
// contracts correctly as long as both operands use it).
// A operand h = [hi hi], l = [lo 0]; B operand h = [hi lo]; then A.h B.h =
// hi*hi + hi*lo and A.l B.h = lo*hi.
// Every accumulator sees only the 16x16x32 MFMA shape: chaining an
// accumulator from that shape into the 16x16x16 one gave wrong gradients
// with ROCm 7.2 hipcc for gfx950, so the 16x16x16 shape is not used.
template <int NB, bool A_ROLE>
struct WOp {
    half8 h[NB], l[NB];
    __device__ __forceinline__ void set(int j, const floatx4 &v) {
        half4 hi, lo;
        split4(v, hi, lo);
        if constexpr (A_ROLE) {
            h[j].lo = hi; h[j].hi = hi;
            l[j].lo = lo; l[j].hi = half4{0, 0, 0, 0};
        } else {
            h[j].lo = hi; h[j].hi = lo;
        }
    }
};

// acc[o][i] += sum over the tile's nodes of A[o] (x) B[i], split passes
// outermost.
template <int NO, int NI>
__device__ __forceinline__ void wgrad_tile(const WOp<NO, true> &A, const WOp<NI, false> &B, floatx4 (&acc)[NO][NI]) {
#pragma unroll
    for (int o = 0; o < NO; ++o)
#pragma unroll
        for (int i = 0; i < NI; ++i) acc[o][i] = mfma16(A.h[o], B.h[i], acc[o][i]);
#pragma unroll
    for (int o = 0; o < NO; ++o)
#pragma unroll
        for (int i = 0; i < NI; ++i) acc[o][i] = mfma16(A.l[o], B.h[i], acc[o][i]);
}

// N form of a T-form tile through the wave's LDS buffer, one 16 x 16 block
// at a time: value (feature 4 q + r, node c) of a block is stored at row
// 4 q + r, column c and read back as four consecutive columns of row c.  The
// wave's LDS operations execute in order, so the buffer is reused per block
// with no wait between blocks.
__device__ __forceinline__ void to_n_form(floatx4 *buf, const floatx4 t[4], floatx4 n[4]) {
    float *b = reinterpret_cast<float *>(buf);
    const int lane = lane_id(), gq = lane >> 4, col = lane & 15;
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
#pragma unroll
        for (int r = 0; r < 4; ++r) b[(4 * gq + r) * kTrRow + col] = t[ob][r];
        wave_sync();
        n[ob] = *reinterpret_cast<const floatx4 *>(&b[col * kTrRow + 4 * gq]);
        wave_sync();
    }
}

// T-form layers over NT tiles; each weight fragment is read from LDS once
// for all tiles.  Per tile and block the MFMA sequence is that of layer64:
// per K step hi*hi, hi*lo, lo*hi.  A tile's MFMAs of a K step are issued
// together, so the first tile's output is complete while the next tile's
// MFMAs still run and its ReLU and split overlap them.
template <int NT>
__device__ __forceinline__ void layer1_tiles(const NetLds &L, const half8 (&xh)[NT], const half8 (&xl)[NT],
                                             floatx4 (&h1)[NT][4]) {
    reload_fence();
    const int lane = lane_id(), gq = lane >> 4;
    half8 wh[4], wl[4];
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
        wh[ob] = L.w1h[ob * 64 + lane];
        wl[ob] = L.w1l[ob * 64 + lane];
        const floatx4 b = *reinterpret_cast<const floatx4 *>(&L.b1s[ob * 16 + 4 * gq]);
#pragma unroll
        for (int u = 0; u < NT; ++u) h1[u][ob] = b;
    }
#pragma unroll
    for (int u = 0; u < NT; ++u) {
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) h1[u][ob] = mfma16(wh[ob], xh[u], h1[u][ob]);
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) h1[u][ob] = mfma16(wh[ob], xl[u], h1[u][ob]);
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) h1[u][ob] = relu4(mfma16(wl[ob], xh[u], h1[u][ob]));
    }
}

// y[u] = W x[u] (+ bias), relu if RELU (T form in and out).
template <int NT, bool RELU>
__device__ __forceinline__ void layer64_tiles(const half8 *wh, const half8 *wl, const half8 (&xh)[NT][2],
                                              const half8 (&xl)[NT][2], const float *bias, floatx4 (&y)[NT][4]) {
    reload_fence();
    const int lane = lane_id(), gq = lane >> 4;
#pragma unroll
    for (int ob = 0; ob < 4; ++ob) {
        const floatx4 b = bias ? *reinterpret_cast<const floatx4 *>(&bias[ob * 16 + 4 * gq])
                               : floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int u = 0; u < NT; ++u) y[u][ob] = b;
    }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        half8 h[4], l[4];
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
            h[ob] = wh[(ob * 2 + s) * 64 + lane];
            l[ob] = wl[(ob * 2 + s) * 64 + lane];
        }
#pragma unroll
        for (int u = 0; u < NT; ++u) {
#pragma unroll
            for (int ob = 0; ob < 4; ++ob) y[u][ob] = mfma16(h[ob], xh[u][s], y[u][ob]);
#pragma unroll
            for (int ob = 0; ob < 4; ++ob) y[u][ob] = mfma16(h[ob], xl[u][s], y[u][ob]);
#pragma unroll
            for (int ob = 0; ob < 4; ++ob) y[u][ob] = mfma16(l[ob], xh[u][s], y[u][ob]);
        }
    }
    if (RELU)
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int ob = 0; ob < 4; ++ob) y[u][ob] = relu4(y[u][ob]);
}

// y[u] = x[u] W^T in N form from a split T-form input (no bias, no relu).
template <int NT>
__device__ __forceinline__ void layer64_tiles_n(const half8 *wh, const half8 *wl, const half8 (&xh)[NT][2],
                                                const half8 (&xl)[NT][2], floatx4 (&y)[NT][4]) {
    reload_fence();
    const int lane = lane_id();
#pragma unroll
    for (int ob = 0; ob < 4; ++ob)
#pragma unroll
        for (int u = 0; u < NT; ++u) y[u][ob] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        half8 h[4], l[4];
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
            h[ob] = wh[(ob * 2 + s) * 64 + lane];
            l[ob] = wl[(ob * 2 + s) * 64 + lane];
        }
#pragma unroll
        for (int u = 0; u < NT; ++u) {
#pragma unroll
            for (int ob = 0; ob < 4; ++ob) y[u][ob] = mfma16(xh[u][s], h[ob], y[u][ob]);
#pragma unroll
            for (int ob = 0; ob < 4; ++ob) y[u][ob] = mfma16(xh[u][s], l[ob], y[u][ob]);
#pragma unroll
            for (int ob = 0; ob < 4; ++ob) y[u][ob] = mfma16(xl[u][s], h[ob], y[u][ob]);
        }
    }
}

struct NodeLds {
    NetLds net;
    half8 w2th[4 * 2 * 64], w2tl[4 * 2 * 64];   // [it][s][lane] split fragments of W2^T
    half8 w4th[4 * 2 * 64], w4tl[4 * 2 * 64];   // [it][s][lane] split fragments of W4[:, :64]^T
    union {
        floatx4 red[kWaves][8][64];             // eight record blocks of every wave's accumulators
        struct {
            float x[6][kBlockNodes];            // [p - o_k, n] 2^ax of the block's nodes
            float s4[kBlockNodes][68];          // sum of dL/dpre4 over the envs
        };
    };
    floatx4 tr[kWaves][16 * kTrRow / 4];        // per-wave 16 x 16 block transpose buffer (rows of kTrRow floats)
    float mx[kWaves];
    float b2[kWaves][64];
};
ETAC_LDS_ALIGNED(NodeLds, s4);
ETAC_LDS_ALIGNED(NodeLds, tr);

// Transposed weight fragments for the adjoint layers, in the chain order of
// etac_device.h (K step s, lane group q, element e <-> output chain_k(s, q, e)),
// scaled by 2^s2t and 2^s4t (after stage_net).
__device__ void stage_net_t(NodeLds &S, const float *phi) {
    const float s2 = pow2(uniform(S.net.s2t)), s4 = pow2(uniform(S.net.s4t));
    for (int idx = threadIdx.x; idx < 4 * 2 * 64; idx += kWG) {
        const int lane = idx & 63, s = (idx >> 6) & 1, it = idx >> 7, q = lane >> 4;
        const int in = it * 16 + (lane & 15);
        float a[8], b[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int out = chain_k(s, q, e);
            a[e] = phi[kW2 + out * 64 + in] * s2;
            b[e] = phi[kW4 + out * 128 + in] * s4;
        }
        split8(a, S.w2th[idx], S.w2tl[idx]);
        split8(b, S.w4th[idx], S.w4tl[idx]);
    }
}

// This wave's accumulators, 16 x 16 blocks in MFMA output layout: lane l,
// register r holds row 4 (l >> 4) + r, column l & 15 of the block.
struct WGrad {
    floatx4 w4[4][4];    // dW4[:, :64]   [row block][column block]
    floatx4 w2[4][4];    // dW2
    floatx4 w1[4][1];    // dW1, columns = 16 padded inputs, column 9 = db1
    floatx4 b2;          // per-lane partial sums of dpre2 for feature 16 b + (l & 15), b = component
};

// One tile (nodes 16 t[0] ..) of the staged block of cnt nodes.  d4mul puts
// dL/dpre4 at 2^d4; accumulator scales: dW4 2^(d4 + af), dW2 2^(d2 + a1), db2
// 2^d2, dW1 2^(d1 + ax) with d2 = d4 + s4t, d1 = d2 + s2t.
__device__ __forceinline__ void node_tiles(NodeLds &S, WGrad &G, int cnt, const int (&t)[1], float d4mul, float one) {
    constexpr int NT = 1;
    const NetLds &L = S.net;
    const int wave = threadIdx.x >> 6;
    floatx4 *tb = S.tr[wave];
    const int lane = lane_id(), gq = lane >> 4, col = lane & 15;
    floatx4 xn[NT], d4T[NT][4];
    half8 xh[NT], xl[NT];
    // N-form inputs: feature col of nodes 4 gq + r (U_hat = 0; input 9 = 1)
    const int fcol = col < 6 ? col : 0;
    const float fsel = col < 6 ? 1.0f : 0.0f, fone = col == 9 ? one : 0.0f;
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        const int li = 16 * t[u] + col;
        const bool valid = li < cnt;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int lj = 16 * t[u] + 4 * gq + r;
            xn[u][r] = lj < cnt ? S.x[fcol][lj] * fsel + fone : 0.0f;
        }
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = e < 6 && valid && gq == 0 ? S.x[e < 6 ? e : 0][li] : 0.0f;
        split8(v, xh[u], xl[u]);
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
            const floatx4 d = *reinterpret_cast<const floatx4 *>(&S.s4[li][16 * ob + 4 * gq]);
            d4T[u][ob] = valid ? d * d4mul : floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        }
    }
    floatx4 h1T[NT][4], fT[NT][4];
    half8 sh[NT][2], sl[NT][2];
    layer1_tiles<NT>(L, xh, xl, h1T);
#pragma unroll
    for (int u = 0; u < NT; ++u) split_chain(h1T[u], sh[u], sl[u]);
    layer64_tiles<NT, true>(L.w2h, L.w2l, sh, sl, L.b2s, fT);
    // dW4[:, :64] += dpre4 (x) f; f > 0 kept as bits (4 block + register)
    unsigned fmask[NT];
    {
        WOp<4, true> A;
        WOp<4, false> B;
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            floatx4 d4N[4], fN[4];
            to_n_form(tb, d4T[u], d4N);
            to_n_form(tb, fT[u], fN);
            fmask[u] = 0u;
#pragma unroll
            for (int ob = 0; ob < 4; ++ob) {
#pragma unroll
                for (int r = 0; r < 4; ++r) fmask[u] |= (fT[u][ob][r] > 0.0f ? 1u : 0u) << (4 * ob + r);
                B.set(ob, fN[ob]);
                A.set(ob, d4N[ob]);
            }
        }
        wgrad_tile(A, B, G.w4);
    }
    // dL/df = W4[:, :64]^T dpre4
#pragma unroll
    for (int u = 0; u < NT; ++u) split_chain(d4T[u], sh[u], sl[u]);
    floatx4 dfT[NT][4];
    layer64_tiles<NT, false>(S.w4th, S.w4tl, sh, sl, nullptr, dfT);
    // dL/dpre2 = df [f > 0]; dL/dh1 = W2^T dpre2 (N form)
    floatx4 d2T[NT][4];
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
        for (int ob = 0; ob < 4; ++ob)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                d2T[u][ob][r] = ((fmask[u] >> (4 * ob + r)) & 1u) ? dfT[u][ob][r] : 0.0f;
#pragma unroll
    for (int u = 0; u < NT; ++u) split_chain(d2T[u], sh[u], sl[u]);
    floatx4 dh1N[NT][4];
    layer64_tiles_n<NT>(S.w2th, S.w2tl, sh, sl, dh1N);
    // dW2 += dpre2 (x) h1, db2; dW1 += dpre1 (x) x (db1 through input 9)
    WOp<4, true> A2, A1;
    WOp<4, false> B2;
    WOp<1, false> B1;
#pragma unroll
    for (int u = 0; u < NT; ++u) {
        floatx4 h1N[4], d2N[4];
        to_n_form(tb, h1T[u], h1N);
        to_n_form(tb, d2T[u], d2N);
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
            B2.set(ob, h1N[ob]);
            G.b2[ob] += (d2N[ob][0] + d2N[ob][1]) + (d2N[ob][2] + d2N[ob][3]);
            A2.set(ob, d2N[ob]);
            floatx4 d1;
#pragma unroll
            for (int r = 0; r < 4; ++r) d1[r] = h1N[ob][r] > 0.0f ? dh1N[u][ob][r] : 0.0f;
            A1.set(ob, d1);
        }
        B1.set(0, xn[u]);
    }
    wgrad_tile(A2, B2, G.w2);
    wgrad_tile(A1, B1, G.w1);
}

// Record blocks 8 C .. 8 C + 7 (C = 4: the four of dW1): every wave puts its
// accumulators in LDS, then each thread adds entries over the waves in order,
// unscales and stores them.
template <int C>
__device__ __forceinline__ void store_record_chunk(NodeLds &S, const WGrad &G, float *rec, float mul) {
    constexpr int NB = C < 4 ? 8 : 4;
    const int wave = threadIdx.x >> 6, lane = lane_id();
    __syncthreads();    // previous users of the buffer are done
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        floatx4 v;
        if constexpr (C == 0) v = G.w4[j >> 2][j & 3];
        else if constexpr (C == 1) v = G.w4[2 + (j >> 2)][j & 3];
        else if constexpr (C == 2) v = G.w2[j >> 2][j & 3];
        else if constexpr (C == 3) v = G.w2[2 + (j >> 2)][j & 3];
        else v = G.w1[j][0];
        S.red[wave][j][lane] = v;
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < NB * 64; idx += kWG) {
        const int j = idx >> 6, ln = idx & 63;
        floatx4 v = S.red[0][j][ln];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) v += S.red[w][j][ln];
        *reinterpret_cast<floatx4 *>(&rec[(8 * C + j) * 256 + 4 * ln]) = v * mul;
    }
}

__global__ __launch_bounds__(kWG) void k_adj_nodes(AdjParams p) {
    __shared__ NodeLds S;
    const MeshDev &M = p.s.mesh;
    const TileDev &T = p.s.tile;
    const int N = M.N, tid = threadIdx.x, lane = lane_id(), wave = uniform(tid >> 6);
    const float *phi = p.s.model.phi;
    stage_net(S.net, phi);
    stage_net_t(S, phi);
    __syncthreads();
    for (int b = blockIdx.x; b < T.NU; b += gridDim.x) {
        const int2 blk = T.block[b];
        const int k = uniform(blk.x), i0 = uniform(blk.y);
        const int live = uniform(live_count(p.s, k));
        if (live == 0) continue;      // its record is not read
        const int base = uniform(M.offset[k]), n = uniform(M.offset[k + 1]) - base, cnt = min(kBlockNodes, n - i0);
        const int chunks = (live + p.env_chunk - 1) / p.env_chunk;
        const ItemScale sc = item_scale(S.net, item_xbound(M, k, 0.0f));
        __syncthreads();              // the previous block is done with S
        item_biases(S.net, sc);
        for (int i = tid; i < 6 * kBlockNodes; i += kWG) {
            const int f = i / kBlockNodes, j = i % kBlockNodes, g = base + i0 + min(j, cnt - 1);
            S.x[f][j] = (f < 3 ? M.pos[(size_t)f * N + g] - M.origin[3 * k + f] : M.nrm[(size_t)(f - 3) * N + g]) * sc.xmul;
        }
        // the chunks' sums in order, and their largest component
        float mx = 0.0f;
        for (int i = tid; i < kBlockNodes * 16; i += kWG) {
            const int j = i >> 4, c = 4 * (i & 15);
            floatx4 o = {0.0f, 0.0f, 0.0f, 0.0f};
            if (j < cnt) {
                const double *src = p.b.s4_node + (size_t)(base + i0 + j) * 64 + c;
                double a[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
                for (int t = 0; t < chunks; ++t) {
#pragma unroll
                    for (int x = 0; x < 4; ++x) a[x] += src[(size_t)t * N * 64 + x];
                }
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    o[x] = (float)a[x];
                    mx = fmaxf(mx, fabsf(o[x]));
                }
            }
            *reinterpret_cast<floatx4 *>(&S.s4[j][c]) = o;
        }
        S.mx[wave] = wave_max(mx);
        __syncthreads();
        mx = fmaxf(fmaxf(S.mx[0], S.mx[1]), fmaxf(S.mx[2], S.mx[3]));
        const int d4 = uniform(range_exp(mx)), d2 = d4 + uniform(S.net.s4t), d1 = d2 + uniform(S.net.s2t);
        WGrad G;
        const floatx4 z = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int x = 0; x < 4; ++x) {
#pragma unroll
            for (int y = 0; y < 4; ++y) { G.w4[x][y] = z; G.w2[x][y] = z; }
            G.w1[x][0] = z;
        }
        G.b2 = z;
        const int tt[1] = {wave};
        node_tiles(S, G, cnt, tt, pow2(d4), sc.xmul);
        float *rec = p.b.node_rec + (size_t)b * kNodeRecWords;
        const float m4 = pow2(-(d4 + sc.af)), m2 = pow2(-(d2 + sc.a1));
        store_record_chunk<0>(S, G, rec, m4);
        store_record_chunk<1>(S, G, rec, m4);
        store_record_chunk<2>(S, G, rec, m2);
        store_record_chunk<3>(S, G, rec, m2);
        store_record_chunk<4>(S, G, rec, pow2(-(d1 + sc.ax)));
#pragma unroll
        for (int ob = 0; ob < 4; ++ob) {
            float v = G.b2[ob];
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);
            S.b2[wave][ob * 16 + (lane & 15)] = v;      // the same in the 4 lane groups
        }
        __syncthreads();
        if (tid < 64) rec[36 * 256 + tid] = (((S.b2[0][tid] + S.b2[1][tid]) + S.b2[2][tid]) + S.b2[3][tid]) * pow2(-d2);
    }
}

hipError_t launch_adj_nodes(const AdjParams &p, int grid, hipStream_t st) {
    hipLaunchKernelGGL(k_adj_nodes, dim3(grid), dim3(kWG), 0, st, p);
    return hipGetLastError();
}

}  // namespace etac
