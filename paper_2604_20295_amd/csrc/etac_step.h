// Pieces of the step's kernels that forward and adjoint share: launch
// parameters, the contact pass over node words, the tables of the undeformed
// surface, work units over the envs in contact, and the max-pool.
#pragma once

#include "etac_device.h"

namespace etac {

struct StepParams {
    MeshDev mesh;
    TileDev tile;
    TableDev tab;
    ItemDev itm;
    SceneDev scene;
    ModelDev model;
    int E;
    int splits;              // workgroups per env of the contact pass
    int dense;               // 1: every item is listed (no k_live), those without contact are passed over
    int table_units, matrix_units;
    int touched;             // 1: tables come after the contact pass, of the patches in contact alone
    int wide;                // 1: products of the decay matrices in wide tiles
    int cus;                 // compute units of the device
    long long items, words;  // E K, E NW
    const int8_t *cobj_in;   // propagate-only: given contact results
    const float *uhat_in;
    float *u;                // [3][E][N]
    int8_t *cobj_out;        // [E][N] (whole step)
    int32_t *n_active;       // [E][K]
    int32_t *n_touch;        // [E][K] active nodes won by external objects (hand), or null
    uint32_t *saved;         // [E K][kSavedWords] pooling record written for the adjoint, or null
    const uint32_t *recall;  // [E K][kSavedWords] pooling record of the forward, read instead of pooling, or null
    float *ivec;             // [E K][4][64] adjoint's vectors per item (s4, g', dpre3, g), or null
    int scratch;             // 1: u and cobj_out are scratch, read at active nodes only
    int adjoint;             // 1: the tables of the adjoint too; given contact results leave zeros in u
};

// Shapes of a call's launches from its sizes (host), its tables, contact pass
// and live lists, and its max-pool.
void shape_step(const Plan &pl, StepParams &p);
void launch_live(const int32_t *n_active, int E, int K, int *live, int *live_cnt, hipStream_t st);
void launch_front(const Plan &pl, StepParams p, hipStream_t st);
void launch_pool(const Plan &pl, const StepParams &p, hipStream_t st);
void launch_far_lists(const StepParams &p, bool passive, hipStream_t st);

__host__ __device__ inline bool step_residual(const StepParams &p) { return p.model.mode != ETAC_DECAY_ONLY; }
__host__ __device__ inline bool step_decay(const StepParams &p) { return p.model.mode != ETAC_RESIDUAL_ONLY; }

// Words of patch k, and its count of envs to visit.
__device__ __forceinline__ int live_count(const StepParams &p, int k) { return p.dense ? p.E : p.itm.live_cnt[k]; }
__device__ __forceinline__ int live_env(const StepParams &p, int k, int q) {
    return p.dense ? q : p.itm.live[(size_t)k * p.E + q];
}

constexpr int kScan = kWG;      // words listed at a time

constexpr int kRowCache = 64;
static_assert(ETAC_MAX_OBJ <= kRowCache, "the env's objects fit");

template <bool ROWS>
struct ContactLds {
    int cnt[kMaxPatches];
    unsigned cand[kMaxPatches];
    int wsum[kWaves];
    int list[kScan];
    ObjRow obj[ROWS ? kRowCache : ETAC_MAX_OBJ];      // the env's objects, or its patches' rows of candidates
    int tcnt[ROWS ? kMaxPatches : 1];
    int16_t at[ROWS ? kMaxPatches : 1];               // a patch's row in obj, -1: read from memory
    int rows;
};

constexpr int kDirectWords = 64;

// Stores of four consecutive values at any 4-byte (winners: 1-byte) address.
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned uint1u __attribute__((aligned(1)));

// Contact of env e, workgroup s of p.splits: first the empty results of every
// node of patches that no object reaches (five of six on a hand), four nodes a
// thread; then the words of the other patches, listed in LDS, a word per wave
// and a node per lane.  Winners and u_hat stream out, and a bit per node is
// kept in p.itm.mask (null for the contact pass alone).  Bound by the stores,
// 13 bytes a node: a lane's 16-byte stores issue a quarter of the instructions
// of a node per lane, which ran at half the rate a fill of the same bytes does.
// The adjoint, whose outputs are scratch, stores active nodes alone (4096 hands:
// 115 us with all nodes, 87 us).
// A surface of few words, or given contact results, has nothing to list: a wave
// takes its words as they come (DIRECT), the first one's geometry requested before the
// objects are read (16384 pads of 256 nodes: 51 us, 38 us).  Several workgroups of
// an env add to its counts (one of them that hands out their sum last needs no
// cleared counts, but 64 workgroups' turns at it take longer than that launch).
template <bool FROM_INPUT, bool ROWS, bool DIRECT>
__device__ void contact_env(const StepParams &p, ContactLds<ROWS> &L, int e, int s) {
    const MeshDev &M = p.mesh;
    const SceneDev &S = p.scene;
    const int N = M.N, K = M.K, NW = p.tile.NW, lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const size_t EN = (size_t)p.E * N, row = (size_t)e * N;
    static_assert(DIRECT || !FROM_INPUT, "given contact results are taken as they come");
    const int step = p.splits * kWaves;
    int4 inf{};
    float x[6];
    auto fetch = [&](int w) {
        inf = p.tile.word[w];
        if (!FROM_INPUT) {
            const int i = uniform(inf.y) + min(lane, uniform(inf.z) - 1);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                x[c] = M.pos[(size_t)c * N + i];
                x[3 + c] = M.nrm[(size_t)c * N + i];
            }
        }
    };
    if (DIRECT) fetch(min(s + p.splits * wave, NW - 1));
    int no = 0;
    if (!FROM_INPUT && !ROWS) {      // the env's objects: read once, then from LDS
        no = min(uniform(S.n_obj[e]), S.O);
        if ((int)threadIdx.x < no * 17) {
            const int o = threadIdx.x / 17, c = threadIdx.x - 17 * o;
            const size_t eo = (size_t)e * S.O + o;
            ObjRow &r = L.obj[o];
            if (c == 0) r.type = S.type[eo];
            else if (c < 5) r.shape[c - 1] = S.shape[4 * eo + c - 1];
            else if (c < 14) r.rot[c - 5] = S.rot[9 * eo + c - 5];
            else r.trans[c - 14] = S.trans[3 * eo + c - 14];
        }
        __syncthreads();
        if ((int)threadIdx.x < no) L.obj[threadIdx.x].reach2 = ball_reach2(L.obj[threadIdx.x].type, L.obj[threadIdx.x].shape);
    }
    if (ROWS) {
        if (threadIdx.x < 64) L.rows = 0;      // identical stores
        __syncthreads();
    }
    for (int k = threadIdx.x; k < K; k += kWG) {
        L.cnt[k] = 0;
        if (ROWS) L.tcnt[k] = 0;
        unsigned c = FROM_INPUT ? ~0u : 0u;
        if (!FROM_INPUT && ROWS) {      // a row holds candidates alone
            const int n = min(S.n_obj[scene_row(S, e, k)], S.O);
            c = n >= 32 ? ~0u : (1u << n) - 1u;
            const int at = n ? atomicAdd(&L.rows, n) : 0;
            L.at[k] = (int16_t)(at + n <= kRowCache ? at : -1);
        }
        if (!FROM_INPUT && !ROWS) {
            const float4 b = M.bound[k];
            for (int o = 0; o < no; ++o) {
                const ObjRow &r = L.obj[o];
                if ((unsigned)r.type <= (unsigned)ETAC_CAPSULE && ball_reaches(b, r.type, r.shape, r.trans)) c |= 1u << o;
            }
        }
        L.cand[k] = c;
    }
    __syncthreads();
    if (!FROM_INPUT && ROWS) {      // four patches' rows at a time, a wave each
        for (int k = wave; k < K; k += kWaves) {
            const unsigned c = uniform(L.cand[k]);
            const int n = __popc(c), at = uniform((int)L.at[k]);
            if (n == 0 || at < 0) continue;
            const size_t r0 = scene_row(S, e, k) * S.O;
            for (int t = lane; t < 17 * n; t += 64) {
                const int o = t / 17, f = t - 17 * o;
                ObjRow &r = L.obj[at + o];
                if (f == 0) r.type = S.type[r0 + o];
                else if (f < 5) r.shape[f - 1] = S.shape[4 * (r0 + o) + f - 1];
                else if (f < 14) r.rot[f - 5] = S.rot[9 * (r0 + o) + f - 5];
                else r.trans[f - 14] = S.trans[3 * (r0 + o) + f - 14];
            }
            wave_sync();
            if (lane < n) L.obj[at + lane].reach2 = ball_reach2(L.obj[at + lane].type, L.obj[at + lane].shape);
        }
        __syncthreads();
    }
    if (!DIRECT && !p.scratch) {
        const floatx4u zero = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int i = 4 * (s * kWG + threadIdx.x); i < N; i += 4 * kWG * p.splits) {
            unsigned c[4];
            bool none = i + 4 <= N;
            int k[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) k[x] = M.node_patch[min(i + x, N - 1)];
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                c[x] = L.cand[k[x]];
                none = none && c[x] == 0;
            }
            if (none) {
                if (p.cobj_out) __builtin_nontemporal_store(~0u, reinterpret_cast<uint1u *>(p.cobj_out + row + i));
                if (p.u)
#pragma unroll
                    for (int a = 0; a < 3; ++a)
                        __builtin_nontemporal_store(zero, reinterpret_cast<floatx4u *>(p.u + a * EN + row + i));
            } else {
#pragma unroll
                for (int x = 0; x < 4; ++x)
                    if (i + x < N && c[x] == 0) {
                        if (p.cobj_out) p.cobj_out[row + i + x] = -1;
                        if (p.u)
#pragma unroll
                            for (int a = 0; a < 3; ++a) p.u[a * EN + row + i + x] = 0.0f;
                    }
            }
        }
    }
    const bool residual = p.itm.mask && step_residual(p);
    // word w, whose geometry is in inf and x; `next`: the word to request meanwhile
    auto take = [&](int w, int next) {
        const int k = uniform(inf.x), i = uniform(inf.y) + lane;
        const bool valid = lane < uniform(inf.z);
        const float px = x[0], py = x[1], pz = x[2], nx = x[3], ny = x[4], nz = x[5];
        if (next >= 0) fetch(next);
        int best = -1;
        float u0 = 0.0f, u1 = 0.0f, u2 = 0.0f;
        int8_t id = -1;
        bool touch = false;
        if (FROM_INPUT) {
            if (valid && p.cobj_in[row + i] >= 0) {
                best = 0;
                u0 = p.uhat_in[row + i];
                u1 = p.uhat_in[EN + row + i];
                u2 = p.uhat_in[2 * EN + row + i];
            }
        } else if (valid) {
            const unsigned c = uniform(L.cand[k]);
            if (ROWS) {
                const size_t srow = scene_row(S, e, k);
                const int at = uniform((int)L.at[k]);
                best = at >= 0 ? contact_node(L.obj + at, c, px, py, pz, nx, ny, nz, u0, u1, u2)
                               : contact_node(S, srow, c, px, py, pz, nx, ny, nz, u0, u1, u2);
                if (best >= 0) touch = S.n_ext && best < S.n_ext[srow];
                id = best >= 0 && S.src ? S.src[srow * S.O + best] : (int8_t)best;
            } else {
                best = contact_node(L.obj, c, px, py, pz, nx, ny, nz, u0, u1, u2);
                id = (int8_t)best;
            }
        }
        if (FROM_INPUT && p.adjoint) {
            if (valid) {
                p.u[row + i] = 0.0f;
                p.u[EN + row + i] = 0.0f;
                p.u[2 * EN + row + i] = 0.0f;
            }
        } else if (valid && (best >= 0 || !p.scratch)) {
            if (!FROM_INPUT && p.cobj_out) __builtin_nontemporal_store(id, p.cobj_out + row + i);
            if (p.u) {
                __builtin_nontemporal_store(u0, p.u + row + i);
                __builtin_nontemporal_store(u1, p.u + EN + row + i);
                __builtin_nontemporal_store(u2, p.u + 2 * EN + row + i);
            }
        }
        const unsigned long long act = __ballot(best >= 0);
        if (p.itm.mask) p.itm.mask[(size_t)e * NW + w] = act;      // every lane stores the same value
        if (act) {                                                 // wave-uniform
            if (residual) {
                const float m = wave_max(fmaxf(fmaxf(fabsf(u0), fabsf(u1)), fabsf(u2)));
                p.itm.umax[(size_t)e * NW + w] = m;
            }
            const unsigned long long tb = ROWS ? __ballot(touch) : 0ull;
            if (lane == 0) {
                atomicAdd(&L.cnt[k], __popcll(act));
                if (ROWS) atomicAdd(&L.tcnt[k], __popcll(tb));
            }
        }
    };
    if (DIRECT)
        for (int w = s + p.splits * wave; w < NW; w += step) take(w, w + step < NW ? w + step : -1);
    for (int w0 = DIRECT ? NW : 0; w0 < NW; w0 += kScan * p.splits) {
        // words w0 + s, w0 + s + splits, ... of patches with candidates
        const int mine = w0 + s + p.splits * (int)threadIdx.x;
        const bool in = mine < NW;
        const bool hit = in && L.cand[p.tile.word[min(mine, NW - 1)].x] != 0;
        if (in && !hit && p.itm.mask) p.itm.mask[(size_t)e * NW + mine] = 0ull;
        const unsigned long long bal = __ballot(hit);
        L.wsum[wave] = __popcll(bal);      // identical in every lane
        __syncthreads();
        int off = 0, total = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            if (w < wave) off += L.wsum[w];
            total += L.wsum[w];
        }
        total = uniform(total);
        if (hit) L.list[off + lanes_below(bal)] = mine;
        __syncthreads();
        // the next word's geometry is requested while this one is tested
        if (wave < total) fetch(uniform(L.list[wave]));
        for (int t = wave; t < total; t += kWaves)
            take(uniform(L.list[t]), t + kWaves < total ? uniform(L.list[t + kWaves]) : -1);
        __syncthreads();      // the list is rewritten
    }
    if (DIRECT) __syncthreads();      // every wave has counted
    if (residual)
        for (int k = wave; k < K; k += kWaves)
            if (uniform(L.cnt[k])) p.itm.pool[((size_t)e * K + k) * 64 + lane] = 0ull;      // k_pool_* raise it
    int32_t *na = p.n_active ? p.n_active : p.itm.n_act;
    for (int k = threadIdx.x; k < K; k += kWG) {
        const size_t it = (size_t)e * K + k;
        if (p.splits == 1) {
            na[it] = L.cnt[k];
            if (ROWS && p.n_touch) p.n_touch[it] = L.tcnt[k];
        } else if (L.cnt[k]) {        // zero before this launch
            atomicAdd(&na[it], L.cnt[k]);
            if (ROWS && p.n_touch && L.tcnt[k]) atomicAdd(&p.n_touch[it], L.tcnt[k]);
        }
    }
}

// ---------------------------------------------------------------------------
// tables
// ---------------------------------------------------------------------------
struct TableLds {
    float part[kWaves][64];
    alignas(16) float bv[kWaves][64];
};
ETAC_LDS_ALIGNED(TableLds, bv);

// Split weight fragments of a 64-input layer (rows `stride` floats apart),
// straight from the packed parameters into registers.
__device__ __forceinline__ void load_frag64(const float *w, int stride, float mul, half8 (&h)[4][2], half8 (&l)[4][2]) {
    const int lane = lane_id(), q = lane >> 4;
#pragma unroll
    for (int ot = 0; ot < 4; ++ot)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const float *r = w + (size_t)(ot * 16 + (lane & 15)) * stride + 32 * s + 4 * q;
            floatx4 a, b;
            __builtin_memcpy(&a, r, 16);
            __builtin_memcpy(&b, r + 16, 16);
            const float x[8] = {a[0] * mul, a[1] * mul, a[2] * mul, a[3] * mul,
                                b[0] * mul, b[1] * mul, b[2] * mul, b[3] * mul};
            split8(x, h[ot][s], l[ot][s]);
        }
}

// Encoder weights of one wave in registers.  Layer 1 has nine inputs: the three
// products of its FP16 parts share the 32 slots of one K step (lane group 0
// hi W hi x, 2 hi W lo x, 3 lo W hi x of inputs 0-7; group 1 all three of input 8).
struct EncW {
    half8 w1[4], w2h[4][2], w2l[4][2];
};

__device__ __forceinline__ void load_encoder(const float *phi, int s1, int s2, EncW &W) {
    const int lane = lane_id(), q = lane >> 4;
    const float e1 = pow2(s1);
#pragma unroll
    for (int ot = 0; ot < 4; ++ot) {
        const float *row = phi + kW1 + (ot * 16 + (lane & 15)) * 9;
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = row[q == 1 ? 8 : e] * e1;
        half8 h, l;
        split8(x, h, l);
        const _Float16 zero = 0;
        const half8 ninth = {h[0], h[0], l[0], zero, zero, zero, zero, zero};
        W.w1[ot] = q == 1 ? ninth : (q == 3 ? l : h);
    }
    load_frag64(phi + kW2, 64, pow2(s2), W.w2h, W.w2l);
}

// Layer 1's B operand of a node (this lane's part).  x: inputs 0-7 of the node;
// in lane group 1 input 8 and zeros.
__device__ __forceinline__ half8 pack_inputs(const float (&x)[8]) {
    const int q = lane_id() >> 4;
    half8 h, l;
    split8(x, h, l);
    uint4t a = __builtin_bit_cast(uint4t, h), b = __builtin_bit_cast(uint4t, l);
#pragma unroll
    for (int e = 0; e < 4; ++e) b[e] = q == 2 ? b[e] : a[e];
    const unsigned lo = __builtin_bit_cast(uint4t, l)[0];
    b[0] = q == 1 ? (a[0] & 0xffffu) | (lo << 16) : b[0];
    b[1] = q == 1 ? a[0] & 0xffffu : b[1];
    return __builtin_bit_cast(half8, b);
}

// The encoder of NT 16-node tiles from register weights, without the last
// ReLU.  b1, b2: scaled biases in LDS.
template <int NT>
__device__ __forceinline__ void encode(const EncW &W, const float *b1, const float *b2, const half8 (&x)[NT],
                                       floatx4 (&f)[NT][4]) {
    const int gq = lane_id() >> 4;
    half8 bh[NT][2], bl[NT][2];
    {
        floatx4 h1[NT][4];
#pragma unroll
        for (int ot = 0; ot < 4; ++ot) {
            const floatx4 b = *reinterpret_cast<const floatx4 *>(&b1[ot * 16 + 4 * gq]);
#pragma unroll
            for (int u = 0; u < NT; ++u) h1[u][ot] = relu4(mfma16(W.w1[ot], x[u], b));
        }
#pragma unroll
        for (int u = 0; u < NT; ++u) split_chain(h1[u], bh[u], bl[u]);
    }
#pragma unroll
    for (int ot = 0; ot < 4; ++ot) {
        const floatx4 b = *reinterpret_cast<const floatx4 *>(&b2[ot * 16 + 4 * gq]);
#pragma unroll
        for (int u = 0; u < NT; ++u) f[u][ot] = b;
    }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int u = 0; u < NT; ++u) {
#pragma unroll
            for (int ot = 0; ot < 4; ++ot) f[u][ot] = mfma16(W.w2h[ot][s], bh[u][s], f[u][ot]);
#pragma unroll
            for (int ot = 0; ot < 4; ++ot) f[u][ot] = mfma16(W.w2h[ot][s], bl[u][s], f[u][ot]);
#pragma unroll
            for (int ot = 0; ot < 4; ++ot) f[u][ot] = mfma16(W.w2l[ot][s], bh[u][s], f[u][ot]);
        }
}

// Whether any env is in contact on patch k, where the contact pass came first
// (the same in every wave).
__device__ __forceinline__ bool table_wanted(const StepParams &p, int k) {
    if (!p.touched) return true;
    if (!p.dense) return uniform(p.itm.live_cnt[k]) > 0;
    const int32_t *na = p.n_active ? p.n_active : p.itm.n_act;
    bool any = false;
    for (int e = lane_id(); e < p.E; e += 64) any = any || na[(size_t)e * p.mesh.K + k] > 0;
    return __ballot(any) != 0ull;
}

// Features of the nodes of words w0, w0 + step, ...: a wave takes 16 nodes of
// the word.  Latency-bound: one dependent chain of three layers per word,
// spread over as many workgroups as there are words (up to two per CU).
struct FeatLds {
    TableLds t;
    alignas(16) float b1s[64], b2s[64];
};
ETAC_LDS_ALIGNED(FeatLds, t);
ETAC_LDS_ALIGNED(FeatLds, b1s);
ETAC_LDS_ALIGNED(FeatLds, b2s);

__device__ void table_words(const StepParams &p, FeatLds &L, int w0, int step) {
    const MeshDev &M = p.mesh;
    bool any = w0 == 0;      // the first block also writes what does not depend on the surface
    for (int w = w0; w < p.tile.NW && !any; w += step) any = table_wanted(p, uniform(p.tile.word[w].x));
    if (!any) return;
    const float *phi = p.model.phi;
    const int tid = threadIdx.x, lane = lane_id(), wave = uniform(tid >> 6), gq = lane >> 4, N = M.N;
    net_norms(L.t.part, phi);
    __syncthreads();
    int s1, s2, s4;
    {
        float v[kNorms];
#pragma unroll
        for (int j = 0; j < kNorms; ++j) {
            v[j] = L.t.part[0][j];
            for (int q = 1; q < kWaves; ++q) v[j] = fmaxf(v[j], L.t.part[q][j]);
        }
        net_scales(v, s1, s2, s4);
        s1 = uniform(s1); s2 = uniform(s2); s4 = uniform(s4);
    }
    if (w0 == 0) {
        if (tid < 64) {   // wave 0, identical values
            p.tab.scale[0] = s1;
            p.tab.scale[1] = s2;
            p.tab.scale[2] = s4;
        }
        for (int i = tid; i < 4096; i += kWG) {
            p.tab.w3t[i] = phi[kW3 + (i & 63) * 64 + (i >> 6)];
            p.tab.w4t[i] = phi[kW4 + (i & 63) * 128 + 64 + (i >> 6)];
        }
    }
    EncW W;
    load_encoder(phi, s1, s2, W);
    for (int w = w0; w < p.tile.NW; w += step) {
        const int4 inf = p.tile.word[w];
        const int k = uniform(inf.x), start = uniform(inf.y), cnt = uniform(inf.z);
        if (!table_wanted(p, k)) continue;
        const int ax = uniform(range_exp(fmaxf(M.xbound[k], 1.0f)));
        const int a1 = s1 + ax, af = s2 + a1;
        __syncthreads();
        if (tid < 64) {
            L.b1s[tid] = phi[kB1 + tid] * pow2(a1);
            L.b2s[tid] = phi[kB2 + tid] * pow2(af);
        }
        __syncthreads();
        const int j = 16 * wave + (lane & 15);
        const bool valid = j < cnt;
        float x[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = 0.0f;
        if (valid && gq != 1) {      // u_hat is zero
            const float xmul = pow2(ax);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                x[a] = (M.pos[(size_t)a * N + start + j] - M.origin[3 * k + a]) * xmul;
                x[3 + a] = M.nrm[(size_t)a * N + start + j] * xmul;
            }
        }
        const half8 in[1] = {pack_inputs(x)};
        floatx4 f[1][4];
        encode<1>(W, L.b1s, L.b2s, in, f);
#pragma unroll
        for (int ot = 0; ot < 4; ++ot) f[0][ot] = relu4(f[0][ot]);
        const float fmul = pow2(-af);
        if (valid)
#pragma unroll
            for (int ot = 0; ot < 4; ++ot)
                *reinterpret_cast<floatx4 *>(p.tab.feat + (size_t)(start + j) * 64 + 16 * ot + 4 * gq) = f[0][ot] * fmul;
        // largest features of eight nodes, then of the wave's sixteen
#pragma unroll
        for (int ot = 0; ot < 4; ++ot) {
            floatx4 v = valid ? f[0][ot] * fmul : floatx4{-1.0f, -1.0f, -1.0f, -1.0f};
#pragma unroll
            for (int off = 1; off <= 4; off <<= 1)
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], __shfl_xor(v[r], off));
            // the eight lanes of a group hold the same values (identical stores)
            *reinterpret_cast<floatx4 *>(p.tab.max8 + (size_t)(8 * w + 2 * wave + ((lane >> 3) & 1)) * 64 + 16 * ot + 4 * gq) = v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = fmaxf(v[r], __shfl_xor(v[r], 8));
            *reinterpret_cast<floatx4 *>(&L.t.bv[wave][16 * ot + 4 * gq]) = v;
        }
        // W4[:, :64] f: the decoder's part that no env changes
        half8 fh[2], fl[2], w4h[4][2], w4l[4][2];
        split_chain(f[0], fh, fl);
        load_frag64(phi + kW4, 128, pow2(s4), w4h, w4l);
        floatx4 z[4];
#pragma unroll
        for (int ot = 0; ot < 4; ++ot) {
            z[ot] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int s = 0; s < 2; ++s) z[ot] = mfma_split(w4h[ot][s], w4l[ot][s], fh[s], fl[s], z[ot]);
        }
        const float zmul = pow2(-(s4 + af));
        if (valid)
#pragma unroll
            for (int ot = 0; ot < 4; ++ot)
                *reinterpret_cast<floatx4 *>(p.tab.dec + (size_t)(start + j) * 64 + 16 * ot + 4 * gq) = z[ot] * zmul;
        __syncthreads();
        if (tid < 128) {      // half words 0 and 1: waves 0-1 and 2-3
            const int h = tid >> 6, c = tid & 63;
            p.tab.max32[(size_t)(2 * w + h) * 64 + c] = fmaxf(L.t.bv[2 * h][c], L.t.bv[2 * h + 1][c]);
        }
    }
}

// Decay matrices.  W = exp(-alpha |p_j - p_i|) of a near patch as three BF16
// parts whose sum is the FP32 value (24 bits: RNE of the value and of the two
// exact remainders; the products keep every product of parts down to 2^-24 of
// the whole, which leaves out at most 2^-26 of it), in the order the matrix
// cores take as A operand: row tile
// t (16 nodes i), K step s (32 nodes j), part c, lane l: row 16 t + (l & 15),
// columns 32 s + 8 (l >> 4) + 0..7 at 16-byte unit ((t KS + s) 3 + c) 64 + l.
// Entries beyond the patch are 0.  For the adjoint also d W.  A workgroup takes a row tile, its waves the
// K steps in turn.  The exponent keeps the remainders of the root and of the
// product, so a weight is good to the rounding of v_exp_f32.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

// x = b0 + b1 + b2 for eight values (24 bits; exact unless a part underflows).
__device__ __forceinline__ void split_bf16x3(const float (&x)[8], bf16x8 (&b)[3]) {
    uint4t o[3];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        floatx2 v = {x[2 * e], x[2 * e + 1]};
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const unsigned h = __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
            o[c][e] = h;
            if (c < 2) {
                v[0] -= __uint_as_float(h << 16);
                v[1] -= __uint_as_float(h & 0xffff0000u);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) b[c] = __builtin_bit_cast(bf16x8, o[c]);
}

// Distance d and exponent t + tl of a pair's weight 2^(t + tl), to 2^-24 of
// the weight: d + dl is the root of s, dl = (s - d^2) / (2 d).
__device__ __forceinline__ void decay_exponent(float dx, float dy, float dz, float nb_hi, float nb_lo, float &d, float &t,
                                               float &tl) {
    const float s = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
    d = __builtin_amdgcn_sqrtf(s);
    const float dl = d > 0.0f ? 0.5f * fmaf(-d, d, s) * __builtin_amdgcn_rcpf(d) : 0.0f;
    t = nb_hi * d;
    tl = fmaf(nb_hi, d, -t) + fmaf(nb_lo, d, nb_hi * dl);
}

__device__ __forceinline__ float decay_weight(float dx, float dy, float dz, float nb_hi, float nb_lo, float &d) {
    float t, tl;
    decay_exponent(dx, dy, dz, nb_hi, nb_lo, d, t, tl);
    const float w = __builtin_amdgcn_exp2f(t);
    return fmaf(w, 0.69314718f * tl, w);
}

// The same beyond FP32's range, for the pair-by-pair sums.
__device__ __forceinline__ double decay_weight_wide(float dx, float dy, float dz, float nb_hi, float nb_lo, float &d) {
    float t, tl;
    decay_exponent(dx, dy, dz, nb_hi, nb_lo, d, t, tl);
    const float ti = rintf(t), w = __builtin_amdgcn_exp2f(t - ti);
    return ldexp((double)fmaf(w, 0.69314718f * tl, w), (int)ti);
}

// -alpha log2(e) as a sum of two floats.
__device__ __forceinline__ void decay_rate(float alpha, float &hi, float &lo) {
    const double b = -(double)alpha * 1.4426950408889634;
    hi = (float)b;
    lo = (float)(b - (double)hi);
}

// Whether a weight could overflow (alpha < 0 on a wide patch: they grow up to
// 2^120 and more): the matrix then holds infinities, which a product would
// spread to nodes that have no such pair; such a patch is summed pair by pair.
__device__ __forceinline__ bool matrix_overflows(const MeshDev &M, float alpha, int k) {
    return alpha < 0.0f && -alpha * 1.4427f * 2.0f * M.bound[k].w > 120.0f;
}

__device__ void matrix_row_tile(const StepParams &p, int unit) {
    const MeshDev &M = p.mesh;
    const int lane = lane_id(), wave = uniform(threadIdx.x >> 6), N = M.N;
    const int2 rt = p.tile.row_tile[unit];
    const int k = uniform(rt.x);
    if (!table_wanted(p, k)) return;
    unit = uniform(rt.y);
    const int base = M.offset[k], n = M.offset[k + 1] - base, KS = (n + 31) >> 5;
    float hi, lo;
    decay_rate(p.model.alpha[k], hi, lo);
    const int i = 16 * unit + (lane & 15);
    const int gi = base + min(i, n - 1);
    const float px = M.pos[gi], py = M.pos[N + gi], pz = M.pos[2 * N + gi];
    const size_t at = p.tile.w_off[k] + (size_t)unit * KS * 3 * 64 + lane;
    uint4 *w = p.tab.w + at, *wd = p.tab.wd + at;
    auto store = [&](uint4 *o, int s, const float (&v)[8]) {
        bf16x8 b[3];
        split_bf16x3(v, b);
#pragma unroll
        for (int c = 0; c < 3; ++c) o[(size_t)(3 * s + c) * 64] = __builtin_bit_cast(uint4, b[c]);
    };
    for (int s = wave; s < KS; s += kWaves) {
        const int j0 = 32 * s + 8 * (lane >> 4);
        float x[8], y[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int gj = base + min(j0 + e, n - 1);
            float d;
            const float v = decay_weight(M.pos[gj] - px, M.pos[N + gj] - py, M.pos[2 * N + gj] - pz, hi, lo, d);
            x[e] = (i < n && j0 + e < n) ? v : 0.0f;
            y[e] = x[e] * d;
        }
        store(w, s, x);
        if (p.adjoint) store(wd, s, y);
    }
}

__device__ __forceinline__ void table_block(const StepParams &p, FeatLds &L, int b) {
    if (b < p.table_units) table_words(p, L, b, p.table_units);
    else matrix_row_tile(p, b - p.table_units);
}

// Units of the live lists: first unit of every patch (in queue order, largest
// patch first) given `per(k)` units each.  Whole workgroup of NW waves; ends
// with a barrier.  Returns the total.
template <int NWV, typename F>
__device__ int unit_prefix(int K, int *first, F per) {
    // K is small (16 on a hand): one wave scans 64 patches at a time
    if (threadIdx.x < 64) {
        int run = 0;
        for (int k0 = 0; k0 < K; k0 += 64) {
            const int kk = k0 + lane_id();
            const int c = kk < K ? per(kk) : 0;
            int inc = c;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) {
                const int o = __shfl_up(inc, off);
                if (lane_id() >= off) inc += o;
            }
            if (kk < K) first[kk] = run + inc - c;
            run += uniform(__shfl(inc, 63));
        }
        first[K] = run;     // identical stores
    }
    __syncthreads();
    return uniform(first[K]);
}

// Units of a product of a patch's decay matrix with the envs in contact: row
// blocks times groups of envs, the row blocks of a group after one another.
// Workgroups stride over the units of all patches, so no part of the chip runs
// dry before another, whatever the patches' sizes (dealt by residues of row block
// and group, six of the eight XCDs had none of one 256-node patch).  Workgroups go
// to the XCDs in turn: where a patch has a multiple of eight row blocks, an XCD
// keeps to an eighth of its matrix.  Shares of an XCD's own of row blocks and
// groups gain nothing on it (4096 hands, forward and transposed product: 419 and
// 669 us, 411 and 667 like this; 16384 hands, forward: 1528 and 1554, whose runs
// differ by 40).
struct ProductRef {
    int k, row_block, group;
};

// The units (whole workgroup; ends with a barrier).
__device__ int product_units(const StepParams &p, int (&first)[kMaxPatches + 1], int rows, int envs) {
    const MeshDev &M = p.mesh;
    return unit_prefix<kWaves>(M.K, first, [&](int kk) {
        const int k = M.order[kk], groups = (live_count(p, k) + envs - 1) / envs;
        if (p.tile.w_off[k] < 0) return 0;
        return (M.offset[k + 1] - M.offset[k] + rows - 1) / rows * groups;
    });
}

// Queue position (patch rank) of unit u: the last rank whose first unit is <= u.
__device__ __forceinline__ int unit_rank(const int *first, int K, int u) {
    int lo = 0, hi = K - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (first[mid] <= u) lo = mid;
        else hi = mid - 1;
    }
    return uniform(lo);
}

// Where Eq. 1 reads the active nodes' u_hat: the caller's own on given contact
// results, else the step's output, whose active entries are u_hat.
__device__ __forceinline__ const float *uhat_source(const StepParams &p) { return p.uhat_in ? p.uhat_in : p.u; }

__device__ __forceinline__ ProductRef product_ref(const StepParams &p, const int (&first)[kMaxPatches + 1], int q, int rows) {
    const int kk = unit_rank(first, p.mesh.K, q), k = uniform(p.mesh.order[kk]);
    const int blocks = (uniform(p.mesh.offset[k + 1]) - uniform(p.mesh.offset[k]) + rows - 1) / rows;
    const int local = q - uniform(first[kk]), group = local / blocks;
    return ProductRef{k, local - group * blocks, group};
}

// ---------------------------------------------------------------------------
// products of a decay matrix
// ---------------------------------------------------------------------------
__device__ __forceinline__ floatx4 mfma_bf16(const bf16x8 &a, const bf16x8 &b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

typedef double doublex4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ doublex4 widen(floatx4 v) { return __builtin_convertvector(v, doublex4); }

__device__ __forceinline__ void pin(doublex4 &v, int x) {
    double t = v[x];
    asm volatile("" : "+v"(t));
    v[x] = t;
}

// Whether a sum is infinite or NaN: the parts of an infinity, or of a value that
// rounds to one, are not finite, and their products with a weight's parts no
// longer add up to the product.  Such rows are summed pair by pair.
__device__ __forceinline__ bool not_finite(const doublex4 (&a)[3]) {
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int x = 0; x < 4; ++x) s += a[c][x];
    return !(fabs(s) <= 1.7976931348623157e308);
}

// acc + A B with three-part operands: every product of parts down to 2^-24 of
// the whole, smallest first.
__device__ __forceinline__ floatx4 mfma_bf16x3(const bf16x8 (&a)[3], const bf16x8 (&b)[3], floatx4 acc) {
    acc = mfma_bf16(a[2], b[0], acc);
    acc = mfma_bf16(a[0], b[2], acc);
    acc = mfma_bf16(a[1], b[1], acc);
    acc = mfma_bf16(a[1], b[0], acc);
    acc = mfma_bf16(a[0], b[1], acc);
    return mfma_bf16(a[0], b[0], acc);
}

// Eight consecutive values x[j0 .. j0 + 7] of a patch of n nodes (0 beyond it).
__device__ __forceinline__ void load8(const float *x, int j0, int n, float (&v)[8]) {
    if (j0 + 8 <= n) {
        floatx4 a, b;
        __builtin_memcpy(&a, x + j0, 16);
        __builtin_memcpy(&b, x + j0 + 4, 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[e] = a[e]; v[4 + e] = b[e]; }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = j0 + e < n ? x[j0 + e] : 0.0f;
    }
}

// A wave's share of a product of NA row tiles of decay matrices with 32 envs'
// values (two column tiles of three components): acc[m][t][c] over all K steps
// of 32 nodes, the FP32 sum of a step added in FP64.  The workgroup's four waves
// split the B fragments of two K steps (this wave's: step wave / 2, column tile
// wave % 2) into LDS while the MFMAs of the two before run.  An MFMA takes 16
// cycles, 12 of which a SIMD has for other instructions: a tile's sum is added
// under the next tile's MFMAs, and the splits are spread over the second step's.
// A fragments come from L2 AHEAD steps ahead, values two pairs ahead.  `mask`:
// this lane's env (has: there is one); PASSIVE takes the nodes without contact.
// Whole workgroup; ends before the last pair's reads of B are done.
using ProductB = uint4[2][2][6][3][64];      // [buffer][K step][3 column tile + component][part][lane]

template <int NA, bool PASSIVE, int AHEAD>
__device__ __forceinline__ void product_loop(ProductB &B, const uint4 *const (&wa)[NA], const float *src, size_t at, size_t EN,
                                             const unsigned long long *mask, bool has, int n, int KS,
                                             doublex4 (&acc)[NA][2][3]) {
    const int lane = lane_id(), wave = uniform(threadIdx.x >> 6), gq = lane >> 4;
    float raw[3][8];
    unsigned long long word = 0;
    int j0 = 0;
    auto fetch = [&](int s0) {
        j0 = 32 * (s0 + (wave >> 1)) + 8 * gq;
        const int j = min(j0, 32 * KS - 8);
        word = mask[j >> 6];
        // values beyond the patch are masked; past the array's end only the last env's last component could reach
        const size_t start = 2 * EN + at + j, safe = min(start, 3 * EN - 8);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float *x = src + (c < 2 ? c * EN + at + j : safe);
            floatx4 a, b;
            __builtin_memcpy(&a, x, 16);
            __builtin_memcpy(&b, x + 4, 16);
#pragma unroll
            for (int e = 0; e < 4; ++e) { raw[c][e] = a[e]; raw[c][4 + e] = b[e]; }
        }
        if (start != safe)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                float v = src[min(start + e, 3 * EN - 1)];
                asm volatile("" : "+v"(v));      // waited for here, not where the branches meet
                raw[2][e] = v;
            }
    };
    auto put = [&](int buf, int c) {
        const int left = has ? max(min(n - j0, 8), 0) : 0;
        const unsigned bits = (unsigned)((PASSIVE ? ~word : word) >> (j0 & 63)) & ((1u << left) - 1u);
        uint4(&o)[3][64] = B[buf][wave >> 1][3 * (wave & 1) + c];
#pragma unroll
        for (int x = 0; x < 8; ++x) raw[c][x] = (bits >> x) & 1u ? raw[c][x] : 0.0f;
        bf16x8 b[3];
        split_bf16x3(raw[c], b);
#pragma unroll
        for (int y = 0; y < 3; ++y) o[y][lane] = __builtin_bit_cast(uint4, b[y]);
    };
    uint4 ab[AHEAD][NA][3];
    auto fetch_a = [&](int s, uint4 (&a)[NA][3]) {
#pragma unroll
        for (int m = 0; m < NA; ++m)
#pragma unroll
            for (int c = 0; c < 3; ++c) a[m][c] = wa[m][(size_t)(s * 3 + c) * 64];
    };
    auto mul = [&](int buf, int ds, const uint4 (&a)[NA][3]) {
        uint4 b[2][3];
        floatx4 o[2][NA];
        auto fold = [&](int f) {
#pragma unroll
            for (int m = 0; m < NA; ++m) {
                doublex4 &s = acc[m][f / 3][f % 3];
                s += widen(o[f & 1][m]);
                // added here, not where the loop ends: the products of a step would all stay in registers
#pragma unroll
                for (int x = 0; x < 4; ++x) pin(s, x);
            }
        };
#pragma unroll
        for (int c = 0; c < 3; ++c) b[0][c] = B[buf][ds][0][c][lane];
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            if (f < 5)
#pragma unroll
                for (int c = 0; c < 3; ++c) b[(f + 1) & 1][c] = B[buf][ds][f + 1][c][lane];
#pragma unroll
            for (int m = 0; m < NA; ++m) {
                bf16x8 y[3], z[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    y[c] = __builtin_bit_cast(bf16x8, a[m][c]);
                    z[c] = __builtin_bit_cast(bf16x8, b[f & 1][c]);
                }
                o[f & 1][m] = mfma_bf16x3(y, z, floatx4{0.0f, 0.0f, 0.0f, 0.0f});
            }
            if (f) fold(f - 1);
            if (ds && !(f & 1)) put(buf ^ 1, f / 2);
#pragma unroll
            for (int i = 0; i < 6 * NA; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        fold(5);
    };
    fetch(0);
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) fetch_a(min(s, KS - 1), ab[s]);
#pragma unroll
    for (int c = 0; c < 3; ++c) put(0, c);
    fetch(2);
    for (int s0 = 0, buf = 0; s0 < KS; s0 += 2, buf ^= 1) {
        __syncthreads();          // this pair is in B[buf]; the other buffer is free
        // a step beyond the last has zeros in B
        mul(buf, 0, ab[0]);
        fetch_a(min(s0 + AHEAD, KS - 1), ab[0]);
        mul(buf, 1, ab[AHEAD - 1]);
        fetch_a(min(s0 + 1 + AHEAD, KS - 1), ab[AHEAD - 1]);
        fetch(s0 + 4);
    }
}

// The runs of 32 listed nodes whose boxes lie within the cutoff of the box of a
// wave's own nodes, in order; uniform over the wave.
struct NearRuns {
    const float4 *box;
    int count, b0 = -64;      // runs, first of the 64 that todo covers
    float lx, ly, lz, hx, hy, hz, cut2;
    unsigned long long todo = 0;

    __device__ __forceinline__ NearRuns(const float4 *boxes, int runs, bool on, float px, float py, float pz, float cut)
        : box(boxes), count(runs), cut2(cut) {
        lx = -wave_max(on ? -px : -3.0e38f); ly = -wave_max(on ? -py : -3.0e38f); lz = -wave_max(on ? -pz : -3.0e38f);
        hx = wave_max(on ? px : -3.0e38f); hy = wave_max(on ? py : -3.0e38f); hz = wave_max(on ? pz : -3.0e38f);
    }
    // The next run, -1 after the last.
    __device__ __forceinline__ int take() {
        while (!todo) {
            b0 += 64;
            if (b0 >= count) return -1;
            const int b = b0 + lane_id();
            const float4 bl = box[2 * min(b, count - 1)], bh = box[2 * min(b, count - 1) + 1];
            const float dx = fmaxf(fmaxf(bl.x - hx, lx - bh.x), 0.0f);
            const float dy = fmaxf(fmaxf(bl.y - hy, ly - bh.y), 0.0f);
            const float dz = fmaxf(fmaxf(bl.z - hz, lz - bh.z), 0.0f);
            todo = __ballot(b < count && !(dx * dx + dy * dy + dz * dz >= cut2));
        }
        const int b = b0 + __ffsll(todo) - 1;
        todo &= todo - 1;
        return uniform(b);
    }
};

// Two runs' nodes, one per lane: positions and values, requested a pair of
// runs ahead of their use (a run at a time, with its list and values read in
// turn before its 32 pairs, waits for memory as long as it computes).
struct RunPair {
    int r[2], c[2];      // runs (-1: none) and their node counts
    float x[6];

    __device__ __forceinline__ void fetch(NearRuns &runs, const MeshDev &M, const int *list, int nodes, int base,
                                          const float *v, size_t EN) {
        r[0] = runs.take();
        r[1] = r[0] >= 0 ? runs.take() : -1;
#pragma unroll
        for (int h = 0; h < 2; ++h) c[h] = r[h] >= 0 ? min(32, nodes - 32 * r[h]) : 0;
        if (r[0] < 0) return;
        const int lane = lane_id(), h = lane >> 5, run = h && c[1] ? r[1] : r[0], cnt = h && c[1] ? c[1] : c[0];
        const int i = list[32 * run + min(lane & 31, cnt - 1)], g = base + i;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            x[a] = M.pos[(size_t)a * M.N + g];
            x[3 + a] = v[a * EN + i];
        }
    }
};

}  // namespace etac
