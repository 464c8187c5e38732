// Forward kernels of the ETac step on gfx950:
// launches over (env, patch) items:
//   k_tables        : what the model gives on the undeformed surface, the same
//                     for every env: encoder features of passive nodes and
//                     their decoder part, and the decay matrices of Eq. 1
//   k_contact_items : contact of every node (or given contact results): winners,
//                     u_hat, and a bit per node for the kernels that follow
//                     (one launch with k_tables on small batches: k_front);
//                     also the contact pass alone
//   k_live          : the envs in contact on each patch
//   k_pool          : max-pool and global MLP of the items in contact
//   k_prop_wide / k_prop_narrow / k_prop_far : U of their passive nodes
//
// Passive nodes have U_hat = 0, so the network's encoder sees only the
// geometry there: its features are computed once per call and node instead of
// once per env, and with them W4[:, :64] f.  What is left per env and passive
// node is an addition, a ReLU and W5.  The decay weights exp(-alpha d) of a
// patch do not depend on the env either: Eq. 1 over the envs in contact is the
// product of a patch matrix with their u_hat columns, on the matrix cores.
#include <algorithm>

#include "etac_step.h"

namespace etac {

// ---------------------------------------------------------------------------
// contact pass
// ---------------------------------------------------------------------------
template <bool FROM_INPUT, bool ROWS, bool DIRECT>
__global__ __launch_bounds__(kWG) void k_contact_items(StepParams p) {
    __shared__ ContactLds<ROWS> L;
    const int e = blockIdx.x / p.splits;
    contact_env<FROM_INPUT, ROWS, DIRECT>(p, L, e, blockIdx.x - e * p.splits);
}

// The contact pass alone on small surfaces: a workgroup per env, a node per
// thread, the objects read where they are tested.  It keeps nothing for later
// kernels and has a third of k_contact_items' chain before the first node:
// 16384 pads of 256 nodes 27 us, 38 in words; 1024 hands of 64 64-node patches 13
// and 14; 256 pads of 4096 nodes 16, and 13 in words by several workgroups an env.
__global__ __launch_bounds__(kWG) void k_contact_small(StepParams p) {
    __shared__ int cnt[kMaxPatches];
    __shared__ unsigned cand[kMaxPatches];
    const MeshDev &M = p.mesh;
    const SceneDev &S = p.scene;
    const int e = blockIdx.x, N = M.N, K = M.K, no = min(S.n_obj[e], S.O);
    const size_t EN = (size_t)p.E * N, row = (size_t)e * N;
    for (int k = threadIdx.x; k < K; k += kWG) {
        const float4 b = M.bound[k];
        unsigned c = 0;
        for (int o = 0; o < no; ++o) {
            const size_t eo = (size_t)e * S.O + o;
            const int ty = S.type[eo];
            if ((unsigned)ty <= (unsigned)ETAC_CAPSULE && ball_reaches(b, ty, S.shape + 4 * eo, S.trans + 3 * eo)) c |= 1u << o;
        }
        cnt[k] = 0;
        cand[k] = c;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < N; i += kWG) {
        float u0 = 0.0f, u1 = 0.0f, u2 = 0.0f;
        const int k = M.node_patch[i];
        const unsigned c = cand[k];
        int best = -1;
        if (c) {
            best = contact_node(S, (size_t)e, c, M.pos[i], M.pos[N + i], M.pos[2 * N + i], M.nrm[i], M.nrm[N + i],
                                M.nrm[2 * N + i], u0, u1, u2);
            if (best >= 0) atomicAdd(&cnt[k], 1);
        }
        __builtin_nontemporal_store((int8_t)best, p.cobj_out + row + i);
        if (p.u) {
            __builtin_nontemporal_store(u0, p.u + row + i);
            __builtin_nontemporal_store(u1, p.u + EN + row + i);
            __builtin_nontemporal_store(u2, p.u + 2 * EN + row + i);
        }
    }
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += kWG) p.n_active[(size_t)e * K + k] = cnt[k];
}

// Zero counts where several workgroups an env add to them.
__device__ __forceinline__ void zero_counts(const StepParams &p) {
    int32_t *na = p.n_active ? p.n_active : p.itm.n_act;
    for (size_t i = (size_t)blockIdx.x * kWG + threadIdx.x; i < (size_t)p.E * p.mesh.K; i += (size_t)gridDim.x * kWG) {
        na[i] = 0;
        if (p.n_touch) p.n_touch[i] = 0;
    }
}

__global__ __launch_bounds__(kWG) void k_zero_counts(StepParams p) { zero_counts(p); }

__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(2))) void k_tables(StepParams p) {
    __shared__ FeatLds L;
    if (p.splits > 1 && !p.touched) zero_counts(p);
    if ((int)blockIdx.x < p.table_units + p.matrix_units) table_block(p, L, blockIdx.x);
}

// Tables and contact in one launch: on small batches neither fills the chip
// and a launch costs as much as either.
template <bool FROM_INPUT, bool ROWS>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(2))) void k_front(StepParams p) {
    __shared__ union {
        FeatLds feat;
        ContactLds<ROWS> contact;
    } L;
    const int nt = p.table_units + p.matrix_units;
    if ((int)blockIdx.x < nt) table_block(p, L.feat, blockIdx.x);
    else contact_env<FROM_INPUT, ROWS, true>(p, L.contact, blockIdx.x - nt, 0);
}

// Envs in contact on patch blockIdx.x, ascending.
__global__ __launch_bounds__(1024) void k_live(const int32_t *n_active, int E, int K, int *live, int *live_cnt) {
    __shared__ int wsum[16];
    const int k = blockIdx.x, wave = threadIdx.x >> 6;
    int run = 0;   // identical in every thread
    for (int e0 = 0; e0 < E; e0 += 1024) {
        const int e = e0 + threadIdx.x;
        const bool f = e < E && n_active[(size_t)e * K + k] > 0;
        const unsigned long long bal = __ballot(f);
        __syncthreads();   // the previous round's reads are done
        wsum[wave] = __popcll(bal);
        __syncthreads();
        int off = run, tot = 0;
        for (int w = 0; w < 16; ++w) {
            if (w < wave) off += wsum[w];
            tot += wsum[w];
        }
        if (f) live[(size_t)k * E + off + lanes_below(bal)] = e;
        run += uniform(tot);
    }
    if (threadIdx.x < 64) live_cnt[k] = run;     // identical stores
}

// ---------------------------------------------------------------------------
// max-pool and global MLP of the items in contact
// ---------------------------------------------------------------------------

// A pooled candidate: feature bits over the complement of the node, so that
// the larger key is the larger feature, the lowest node on ties (features are
// not negative).
__device__ __forceinline__ unsigned long long pool_key(float v, int node) {
    return ((unsigned long long)__float_as_uint(v) << 32) | (unsigned)~node;
}

// Words [w0, w0 + cw) of an item, at most PCW.
template <int PCW>
struct PassiveLds {
    uint16_t code[PCW * 56];       // at most seven single nodes per eight
};

// Largest feature of the passive nodes among `words` words from word wf of the
// item, lane c on channel c; 0 without any.  Eight or thirty-two consecutive
// passive nodes take one read of the table of their maxima, so a contact
// patch's surroundings cost about a seventh of their nodes' reads.  The reads
// are listed first, then issued sixteen at a time; the winner's node is looked
// up at the end.
template <int PCW>
__device__ unsigned long long pool_passive(const StepParams &p, PassiveLds<PCW> &L, int base, int n, int w0, int wf,
                                           int words, const unsigned long long *mask) {
    const int lane = lane_id();
    constexpr int OPL = PCW * 8 / 64 > 0 ? PCW * 8 / 64 : 1;      // octets per lane
    // this lane's octets
    unsigned pas[OPL];
    int kind[OPL], cnt = 0;
#pragma unroll
    for (int t = 0; t < OPL; ++t) {
        const int o = lane * OPL + t, w = o >> 3;
        pas[t] = 0;
        kind[t] = 0;
        if (w >= words) continue;
        const int left = n - 64 * (wf + w);            // nodes of the word (and beyond)
        const unsigned long long all = left >= 64 ? ~0ull : (1ull << left) - 1ull;
        const unsigned long long pw = all & ~mask[wf + w];
        const unsigned half = (unsigned)(pw >> (32 * ((o >> 2) & 1)));
        pas[t] = (unsigned)(pw >> (8 * (o & 7))) & 0xffu;
        if (half == ~0u) kind[t] = (o & 3) == 0 ? 2 : 3;         // 3: its half word's first octet reads for it
        else if (pas[t] == 0xffu) kind[t] = 1;
        cnt += kind[t] == 3 ? 0 : (kind[t] ? 1 : __popc(pas[t]));
    }
    int at = cnt;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(at, off);
        if (lane >= off) at += o;
    }
    const int total = uniform(__shfl(at, 63));
    at -= cnt;
    if (total == 0) return 0ull;
    wave_sync();
#pragma unroll
    for (int t = 0; t < OPL; ++t) {
        const int n0 = 8 * (lane * OPL + t);
        if (kind[t] == 1 || kind[t] == 2) L.code[at++] = (uint16_t)(n0 | (kind[t] << 12));
        else if (kind[t] == 0)
            for (unsigned b = pas[t]; b; b &= b - 1) L.code[at++] = (uint16_t)(n0 + __ffs(b) - 1);
    }
    wave_sync();
    const float *feat = p.tab.feat + (size_t)(base + 64 * wf) * 64 + lane;
    const float *m8 = p.tab.max8 + (size_t)8 * (w0 + wf) * 64 + lane, *m32 = p.tab.max32 + (size_t)2 * (w0 + wf) * 64 + lane;
    float best = -1.0f;
    int bc = 0;
    for (int i = 0; i < total; i += 16) {
        int c[16];
        float v[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) c[t] = uniform((int)L.code[min(i + t, total - 1)]);
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const int node = c[t] & 0xfff;
            const float *src = c[t] >> 13 ? m32 + (size_t)(node >> 5) * 64
                                          : (c[t] >> 12 ? m8 + (size_t)(node >> 3) * 64 : feat + (size_t)node * 64);
            v[t] = *src;
        }
#pragma unroll
        for (int t = 0; t < 16; ++t)
            if (v[t] > best) { best = v[t]; bc = c[t]; }
    }
    // the first node of the winning run with that value
    int node = bc & 0xfff;
    if (bc >> 13) {
        float v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = m8[(size_t)((node >> 3) + t) * 64];
        int f = 3;
#pragma unroll
        for (int t = 2; t >= 0; --t) f = v[t] == best ? t : f;
        node += 8 * f;
    }
    if (bc >> 12) {
        float v[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = feat[(size_t)(node + t) * 64];
        int f = 7;
#pragma unroll
        for (int t = 6; t >= 0; --t) f = v[t] == best ? t : f;
        node += f;
    }
    return pool_key(best, 64 * wf + node);
}

// Words of an active chunk.
constexpr int kActiveWords = 8;

struct ActiveLds {
    alignas(16) float b1s[64], b2s[64];
    float v[64];
    int ix[64];
    uint16_t slot[64 * kActiveWords];
};
ETAC_LDS_ALIGNED(ActiveLds, b1s);
ETAC_LDS_ALIGNED(ActiveLds, b2s);

// Largest of two (value, node) pairs, the lower node on ties.
__device__ __forceinline__ void take_max(float &v, int &ix, float v2, int i2) {
    const bool take = (v2 > v) | ((v2 == v) & (i2 < ix));
    v = take ? v2 : v;
    ix = take ? i2 : ix;
}

// A step of the reduction of H pairs per lane over 16 lanes: lanes keep the
// half of their pairs that their `bit` names and hand the other half to a lane
// of the other half.
template <int H, int CTRL>
__device__ __forceinline__ void halve_max(float (&v)[16], int (&ix)[16], bool bit) {
#pragma unroll
    for (int i = 0; i < H / 2; ++i) {
        const float keep = bit ? v[H / 2 + i] : v[i], give = bit ? v[i] : v[H / 2 + i];
        const int ikeep = bit ? ix[H / 2 + i] : ix[i], igive = bit ? ix[i] : ix[H / 2 + i];
        v[i] = keep;
        ix[i] = ikeep;
        take_max(v[i], ix[i], dpp<CTRL>(give), dpp<CTRL>(igive));
    }
}

// Largest feature of the active nodes among `words` words from word wf of the
// item: its active nodes in order, 32 at a time through the encoder on the
// matrix cores, weights in registers.  One wave; lane c returns channel c.
// Nodes beyond the last repeat it.  Bound by the VALU (splits and maxima, 9 per
// feature) and the dependent chain of a unit's start, so words and ranges are
// loaded at once, no load of the loop is under a branch, and the 16 lanes of a
// row are reduced by exchanging halves (15 exchanges of a pair instead of 64).
// 4096 hands (3.8 M active nodes): 317 us without these, 208 us.
__device__ unsigned long long pool_active(const StepParams &p, ActiveLds &L, const EncW &W, float rb1, float rb2, int s1,
                                          int s2, int k, int e, int base, int nw, int w0, int wf, int words) {
    const MeshDev &M = p.mesh;
    const int N = M.N, lane = lane_id(), gq = lane >> 4;
    const size_t EN = (size_t)p.E * N;
    const unsigned long long *mask = p.itm.mask + (size_t)e * p.tile.NW + w0;
    const float *um = p.itm.umax + (size_t)e * p.tile.NW + w0;
    const unsigned long long mine = mask[wf + min(lane, words - 1)];
    float umax = 0.0f;
    for (int w = lane; w < nw; w += 64) {
        const unsigned long long m = mask[w];
        const float v = um[w];      // stale in words without contact
        umax = m ? fmaxf(umax, v) : umax;
    }
    int total = 0;
    wave_sync();
#pragma unroll
    for (int t = 0; t < kActiveWords; ++t) {
        const unsigned long long act =
            t < words ? ((unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(mine >> 32), t) << 32) |
                            (unsigned)__builtin_amdgcn_readlane((int)mine, t)
                      : 0ull;
        if ((act >> lane) & 1ull) L.slot[total + lanes_below(act)] = (uint16_t)(64 * t + lane);
        total += __popcll(act);
    }
    if (total == 0) return 0ull;
    umax = wave_max(umax);
    const int ax = uniform(range_exp(fmaxf(item_xbound(M, k, umax), 1.0f)));
    const int a1 = s1 + ax, af = s2 + a1;
    L.b1s[lane] = rb1 * pow2(a1);
    L.b2s[lane] = rb2 * pow2(af);
    wave_sync();
    // input = raw * mul + add; lane group 1 holds the ninth input and zeros
    const float xmul = pow2(ax), mul = gq == 1 ? 0.0f : xmul;
    const float add[3] = {gq == 1 ? 0.0f : -M.origin[3 * k] * xmul, -M.origin[3 * k + 1] * mul, -M.origin[3 * k + 2] * mul};
    const float *uh = uhat_source(p) + (size_t)e * N + base + 64 * wf, *pos = M.pos + base + 64 * wf;
    const float *nrm = M.nrm + base + 64 * wf, *in0 = gq == 1 ? uh + 2 * EN : pos;
    float raw[2][8];
    int next[2];
    auto fetch = [&](int t0) {      // inputs of the next two tiles, requested while these run
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int g = next[u] = L.slot[min(t0 + 16 * u + (lane & 15), total - 1)];
            raw[u][0] = in0[g];
#pragma unroll
            for (int c = 1; c < 3; ++c) raw[u][c] = pos[(size_t)c * N + g];
#pragma unroll
            for (int c = 0; c < 3; ++c) raw[u][3 + c] = nrm[(size_t)c * N + g];
            raw[u][6] = uh[g];
            raw[u][7] = uh[EN + g];
        }
    };
    fetch(0);
    // a feature is at least 0 (ReLU), which every node without a larger one has
    float mx[16];
    int mi[16];
    const int first = uniform((int)L.slot[0]);
#pragma unroll
    for (int o = 0; o < 16; ++o) { mx[o] = 0.0f; mi[o] = first; }
    for (int t0 = 0; t0 < total; t0 += 32) {
        half8 in[2];
        int node[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            float x[8];
            x[0] = fmaf(raw[u][0], xmul, add[0]);
            x[1] = fmaf(raw[u][1], mul, add[1]);
            x[2] = fmaf(raw[u][2], mul, add[2]);
#pragma unroll
            for (int c = 3; c < 8; ++c) x[c] = raw[u][c] * mul;
            in[u] = pack_inputs(x);
            node[u] = next[u];
        }
        fetch(t0 + 32);
        floatx4 f[2][4];
        encode<2>(W, L.b1s, L.b2s, in, f);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int o = 0; o < 16; ++o) {
                const float v = f[u][o >> 2][o & 3];
                const bool take = v > mx[o];
                mx[o] = take ? v : mx[o];
                mi[o] = take ? node[u] : mi[o];
            }
    }
    // over the 16 nodes of a row, the lowest node on ties: lane l of the row
    // ends with output tile l / 4, row 4 gq + l % 4
    halve_max<16, kDppXor8>(mx, mi, lane & 8);
    halve_max<8, kDppXor7>(mx, mi, lane & 4);
    halve_max<4, kDppXor2>(mx, mi, lane & 2);
    halve_max<2, kDppXor1>(mx, mi, lane & 1);
    const int ch = ((lane >> 2) & 3) * 16 + 4 * gq + (lane & 3);
    L.v[ch] = mx[0];
    L.ix[ch] = mi[0];
    wave_sync();
    const unsigned long long key = pool_key(L.v[lane] * pow2(-af), 64 * wf + L.ix[lane]);
    wave_sync();
    return key;
}

// Pooled feature v of an item, the node it came from and g' (lane c on channel
// c) to its record and the adjoint's vectors.
__device__ __forceinline__ void keep_pool(const StepParams &p, size_t item, float v, unsigned node, float gp) {
    const int lane = lane_id();
    if (p.saved) {
        uint32_t *rec = p.saved + item * kSavedWords;
        rec[lane] = __float_as_uint(v);
        rec[64 + lane] = node;
    }
    if (p.ivec) {
        p.ivec[item * 256 + 64 + lane] = gp;
        p.ivec[item * 256 + 192 + lane] = v;
    }
}

// Partial product of a vector's C channels from c0 on (x: lane c holds channel
// c) with the weights w of this lane's row.
template <int C>
__device__ __forceinline__ float dot_lanes(const float (&w)[C], float x, int c0) {
    float a = 0.0f;
#pragma unroll
    for (int c = 0; c < C; ++c) a += w[c] * __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), c0 + c));
    return a;
}

// The item of live-list unit q, part by part of a patch's items: parts differ in
// their active nodes, and a workgroup that strides over the units would meet the
// same part of every item otherwise.
struct ItemRef {
    int k, e, part;
};

__device__ __forceinline__ ItemRef item_ref(const StepParams &p, const int *first, int q) {
    const int kk = unit_rank(first, p.mesh.K, q), k = uniform(p.mesh.order[kk]);
    const int cnt = uniform(live_count(p, k)), local = q - uniform(first[kk]), part = local / cnt;
    return ItemRef{k, uniform(live_env(p, k, local - part * cnt)), part};
}

__device__ __forceinline__ int item_units(const StepParams &p, const int *first, int words) {
    return unit_prefix<kWaves>(p.mesh.K, const_cast<int *>(first), [&](int kk) {
        const int k = p.mesh.order[kk];
        return live_count(p, k) * ((p.tile.word_off[k + 1] - p.tile.word_off[k] + words - 1) / words);
    });
}

// Max-pool over the items in contact, in two launches that raise the items'
// keys (a maximum: no order matters) and one that finishes them.  Passive
// nodes need few registers and many waves in flight (reads of the feature
// tables in L2), active nodes the encoder's weights in registers.
constexpr int kPassiveWords = 16;

__global__ __launch_bounds__(kWG) void k_pool_passive(StepParams p) {
    __shared__ int first[kMaxPatches + 1];
    __shared__ PassiveLds<kPassiveWords> L[kWaves];
    const int K = p.mesh.K, wave = uniform(threadIdx.x >> 6);
    const int total = item_units(p, first, kPassiveWords);
    const int32_t *na = p.n_active ? p.n_active : p.itm.n_act;
    for (int q = blockIdx.x * kWaves + wave; q < total; q += gridDim.x * kWaves) {
        const ItemRef it = item_ref(p, first, q);
        const size_t item = (size_t)it.e * K + it.k;
        if (p.dense && uniform(na[item]) == 0) continue;
        const int base = uniform(p.mesh.offset[it.k]), n = uniform(p.mesh.offset[it.k + 1]) - base;
        const int w0 = uniform(p.tile.word_off[it.k]), nw = uniform(p.tile.word_off[it.k + 1]) - w0;
        const int wf = it.part * kPassiveWords;
        const unsigned long long key = pool_passive(p, L[wave], base, n, w0, wf, min(kPassiveWords, nw - wf),
                                                    p.itm.mask + (size_t)it.e * p.tile.NW + w0);
        if (key) atomicMax(&p.itm.pool[item * 64 + lane_id()], key);
    }
}

__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(2))) void k_pool_active(StepParams p) {
    __shared__ int first[kMaxPatches + 1];
    __shared__ ActiveLds L[kWaves];
    const int K = p.mesh.K, lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const float *phi = p.model.phi;
    const int total = item_units(p, first, kActiveWords);
    const int32_t *na = p.n_active ? p.n_active : p.itm.n_act;
    const int s1 = uniform(p.tab.scale[0]), s2 = uniform(p.tab.scale[1]);
    EncW W;
    load_encoder(phi, s1, s2, W);
    const float rb1 = phi[kB1 + lane], rb2 = phi[kB2 + lane];
    for (int q = blockIdx.x * kWaves + wave; q < total; q += gridDim.x * kWaves) {
        const ItemRef it = item_ref(p, first, q);
        const size_t item = (size_t)it.e * K + it.k;
        if (p.dense && uniform(na[item]) == 0) continue;
        const int base = uniform(p.mesh.offset[it.k]), w0 = uniform(p.tile.word_off[it.k]);
        const int nw = uniform(p.tile.word_off[it.k + 1]) - w0, wf = it.part * kActiveWords;
        const unsigned long long key = pool_active(p, L[wave], W, rb1, rb2, s1, s2, it.k, it.e, base, nw, w0, wf,
                                                   min(kActiveWords, nw - wf));
        if (key) atomicMax(&p.itm.pool[item * 64 + lane], key);
    }
}

// Global MLP of the items, a wave at a time, the weights of both layers in
// registers: read again for every item they cost four trips to L2 a layer.
// 16384 hands (36000 items): 48 us like that, 40 us now; four pads in contact
// 10 and 5 us.
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(3))) void k_pool_finish(StepParams p) {
    __shared__ int first[kMaxPatches + 1];
    const int K = p.mesh.K, lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const float *phi = p.model.phi;
    float w3[8][8], w4[8][8];      // partial sums of eight channels, as k_pool's
#pragma unroll
    for (int c = 0; c < 64; ++c) w3[c / 8][c % 8] = p.tab.w3t[c * 64 + lane];
#pragma unroll
    for (int c = 0; c < 64; ++c) w4[c / 8][c % 8] = p.tab.w4t[c * 64 + lane];
    const float b3 = phi[kB3 + lane], b4 = phi[kB4 + lane];
    const int total = item_units(p, first, 1 << 20);
    const int32_t *na = p.n_active ? p.n_active : p.itm.n_act;
    for (int q = blockIdx.x * kWaves + wave; q < total; q += gridDim.x * kWaves) {
        const ItemRef it = item_ref(p, first, q);
        const size_t item = (size_t)it.e * K + it.k;
        if (p.dense && uniform(na[item]) == 0) continue;
        float v;
        unsigned node;
        if (p.recall) {      // the forward's record
            const uint32_t *rec = p.recall + item * kSavedWords;
            v = __uint_as_float(rec[lane]);
            node = rec[64 + lane];
        } else {
            const unsigned long long key = p.itm.pool[item * 64 + lane];
            v = __uint_as_float((unsigned)(key >> 32));
            node = ~(unsigned)key;
        }
        float s = b3;
#pragma unroll
        for (int g = 0; g < 8; ++g) s += dot_lanes<8>(w3[g], v, 8 * g);
        const float gp = fmaxf(s, 0.0f);
        s = b4;
#pragma unroll
        for (int g = 0; g < 8; ++g) s += dot_lanes<8>(w4[g], gp, 8 * g);
        p.itm.c4[item * 64 + lane] = s;
        keep_pool(p, item, v, node, gp);
    }
}

// The same in one launch, a workgroup of eight waves per item, in contact or not,
// for batches of few items, where a launch costs more than the idle waves (24
// hands, 384 items: 48 us in three launches, 19 us).  Latency-
// bound: the layers of the global MLP are split over the waves, their weights
// loaded at the start (one pad: 24.1 us with one wave reading them, 16.8 us).
constexpr int kPoolWaves = 8, kPoolWords = 4, kPoolItems = 1024;

struct PoolLds {
    unsigned long long key[64];
    float part[2][kPoolWaves][64];
    union {
        PassiveLds<kPoolWords> pas;
        ActiveLds act;
    } w[kPoolWaves];
};
ETAC_LDS_ALIGNED(PoolLds, w);

__global__ __launch_bounds__(64 * kPoolWaves) __attribute__((amdgpu_waves_per_eu(2))) void k_pool(StepParams p) {
    __shared__ PoolLds L;
    const MeshDev &M = p.mesh;
    const int K = M.K, lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const float *phi = p.model.phi;
    const int32_t *na = p.n_active ? p.n_active : p.itm.n_act;
    const int s1 = uniform(p.tab.scale[0]), s2 = uniform(p.tab.scale[1]);
    EncW W;
    load_encoder(phi, s1, s2, W);
    const float rb1 = phi[kB1 + lane], rb2 = phi[kB2 + lane], b3 = phi[kB3 + lane], b4 = phi[kB4 + lane];
    // the global MLP's layers are split over the waves by input channels
    constexpr int kShare = 64 / kPoolWaves;
    const int c0 = kShare * wave;
    float w3[kShare], w4[kShare];
#pragma unroll
    for (int c = 0; c < kShare; ++c) {
        w3[c] = p.tab.w3t[(c0 + c) * 64 + lane];
        w4[c] = p.tab.w4t[(c0 + c) * 64 + lane];
    }
    for (int q = blockIdx.x; q < p.E * K; q += gridDim.x) {
        const int e = q / K, k = q - e * K;
        const size_t item = (size_t)q;
        if (uniform(na[item]) == 0) continue;      // the same in every wave
        const int base = uniform(M.offset[k]), n = uniform(M.offset[k + 1]) - base;
        const int w0 = uniform(p.tile.word_off[k]), nw = uniform(p.tile.word_off[k + 1]) - w0;
        const int chunks = (nw + kPoolWords - 1) / kPoolWords;
        __syncthreads();          // the previous item is done with L
        if (threadIdx.x < 64) L.key[lane] = 0ull;
        __syncthreads();
        for (int t = wave; t < 2 * chunks; t += kPoolWaves) {
            const int wf = (t >> 1) * kPoolWords, words = min(kPoolWords, nw - wf);
            const unsigned long long key =
                (t & 1) ? pool_passive(p, L.w[wave].pas, base, n, w0, wf, words, p.itm.mask + (size_t)e * p.tile.NW + w0)
                        : pool_active(p, L.w[wave].act, W, rb1, rb2, s1, s2, k, e, base, nw, w0, wf, words);
            if (key) atomicMax(&L.key[lane], key);
        }
        __syncthreads();
        const unsigned long long key = L.key[lane];
        const float v = __uint_as_float((unsigned)(key >> 32));
        L.part[0][wave][lane] = dot_lanes<kShare>(w3, v, c0);
        __syncthreads();
        float s = b3;
#pragma unroll
        for (int w = 0; w < kPoolWaves; ++w) s += L.part[0][w][lane];
        const float gp = fmaxf(s, 0.0f);
        L.part[1][wave][lane] = dot_lanes<kShare>(w4, gp, c0);
        __syncthreads();
        if (wave == 0) {
            s = b4;
#pragma unroll
            for (int w = 0; w < kPoolWaves; ++w) s += L.part[1][w][lane];
            p.itm.c4[item * 64 + lane] = s;
            keep_pool(p, item, v, ~(unsigned)key, gp);
        }
    }
}

// ---------------------------------------------------------------------------
// U of the passive nodes: near patches
// ---------------------------------------------------------------------------
// Eq. 1 of one node over the active nodes of its item, pair by pair.
__device__ void pair_sum(const StepParams &p, int k, int e, int i, const float *src, double (&s)[3]) {
    const MeshDev &M = p.mesh;
    const int N = M.N, base = M.offset[k], n = M.offset[k + 1] - base;
    const size_t EN = (size_t)p.E * N;
    const unsigned long long *mask = p.itm.mask + (size_t)e * p.tile.NW + p.tile.word_off[k];
    const float *u = src + (size_t)e * N + base;
    float hi, lo;
    decay_rate(p.model.alpha[k], hi, lo);
    s[0] = s[1] = s[2] = 0.0;
    for (int j = 0; j < n; ++j) {
        if (!((mask[j >> 6] >> (j & 63)) & 1ull)) continue;
        float d;
        const double w = decay_weight_wide(M.pos[base + j] - M.pos[base + i], M.pos[N + base + j] - M.pos[N + base + i],
                                     M.pos[2 * N + base + j] - M.pos[2 * N + base + i], hi, lo, d);
        s[0] += w * u[j];
        s[1] += w * u[EN + j];
        s[2] += w * u[2 * EN + j];
    }
}

// Bit x: row i0 + x of an env's four rows is a passive node of the patch.
__device__ __forceinline__ unsigned passive_rows(const StepParams &p, int e, int w0, int i0, int n) {
    if (e < 0 || i0 >= n) return 0u;
    const unsigned act = (unsigned)(p.itm.mask[(size_t)e * p.tile.NW + w0 + (i0 >> 6)] >> (i0 & 63));
    return ~act & (n - i0 >= 4 ? 0xfu : (1u << (n - i0)) - 1u);
}

// The rows of `todo` summed pair by pair (no register indexed at run time).
__device__ void pair_rows(const StepParams &p, int k, int e, int i0, unsigned todo, const float *src, doublex4 (&a)[3]) {
    for (; todo; todo &= todo - 1) {
        const int row = __ffs(todo) - 1;
        double s[3];
        pair_sum(p, k, e, i0 + row, src, s);
#pragma unroll
        for (int x = 0; x < 4; ++x)
#pragma unroll
            for (int c = 0; c < 3; ++c) a[c][x] = x == row ? s[c] : a[c][x];
    }
}

// Residual of NT envs on the four nodes whose decoder rows z points at, over
// channels [c0, c1): r += W5 relu(z + c4).
template <int NT>
__device__ __forceinline__ void residual_rows(const float (*w5)[64], const float *const (&z)[4],
                                              const float *const (&c4)[NT], int c0, int c1, floatx4 (&r)[NT][3]) {
#pragma unroll 2
    for (int c = c0; c < c1; c += 4) {
        floatx4 zz[4], w[3];
#pragma unroll
        for (int x = 0; x < 4; ++x) zz[x] = *reinterpret_cast<const floatx4 *>(z[x] + c);
#pragma unroll
        for (int a = 0; a < 3; ++a) w[a] = *reinterpret_cast<const floatx4 *>(&w5[a][c]);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const floatx4 cc = *reinterpret_cast<const floatx4 *>(c4[t] + c);
#pragma unroll
            for (int h = 0; h < 4; ++h)
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const float v = relu1(zz[x][h] + cc[h]);
#pragma unroll
                    for (int a = 0; a < 3; ++a) r[t][a][x] += w[a][h] * v;
                }
        }
    }
}

// W5 and b5 to LDS (whole workgroup; the caller's next barrier publishes them).
__device__ __forceinline__ void stage_w5(const StepParams &p, float (*w5)[64], float *b5) {
    if (!step_residual(p)) return;
    for (int i = threadIdx.x; i < 192; i += blockDim.x) w5[i >> 6][i & 63] = p.model.phi[kW5 + i];
    if (threadIdx.x < 64) b5[threadIdx.x & 3] = p.model.phi[kB5 + min((int)(threadIdx.x & 3), 2)];
}

// U of four consecutive nodes of one env: decay part a, residual r; active
// nodes (their bits) and rows beyond the patch are left alone.
__device__ __forceinline__ void store_rows(float *o, size_t EN, unsigned act, int left, const doublex4 (&a)[3],
                                           const floatx4 (&r)[3], bool dec, bool res) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const floatx4 v = dec ? __builtin_convertvector(res ? a[c] + widen(r[c]) : a[c], floatx4) : r[c];
        if (act == 0 && left >= 4) {
            __builtin_memcpy(o + c * EN, &v, 16);
        } else {
#pragma unroll
            for (int x = 0; x < 4; ++x)
                if (x < left && !((act >> x) & 1u)) o[c * EN + x] = v[x];
        }
    }
}

// Wide tiles: 64 MT rows (a wave takes MT row tiles) times 32 envs (two column
// tiles per component: column l & 15 is an env).  Bound by the matrix cores in
// the loop (4096 hands: 17.8 M MFMAs, 116 us of all of them at full rate) and by
// the VALU: the FP64 sums there, and five operations per node, env and channel
// of the residual in the epilogue.  A taller tile reads and splits each env's
// values for more rows: 4096 hands 530 us at MT = 1 and 410 at MT = 2, 16384 hands
// 2020 and 1520 (three row tiles would not fit the registers).  Patches are padded
// to it and there are fewer units: see tall_tiles.
constexpr int kWideEnvs = 32;

struct WideLds {
    int first[kMaxPatches + 1];
    int env[kWideEnvs];
    union {
        ProductB b;
        struct {                      // after the K loop
            float c4[kWideEnvs][68];
            float w5[3][64], b5[4];
        };
    };
};
ETAC_LDS_ALIGNED(WideLds, c4);
ETAC_LDS_ALIGNED(WideLds, w5);

template <int MT>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(2))) void k_prop_wide(StepParams p) {
    __shared__ WideLds L;
    constexpr int kRows = 64 * MT;
    const MeshDev &M = p.mesh;
    const TileDev &T = p.tile;
    const int K = M.K, N = M.N, lane = lane_id(), wave = uniform(threadIdx.x >> 6), gq = lane >> 4, col = lane & 15;
    const size_t EN = (size_t)p.E * N;
    const bool dec = step_decay(p), res = step_residual(p);
    const float *src = uhat_source(p);
    const int32_t *na = p.n_active ? p.n_active : p.itm.n_act;
    const int total = product_units(p, L.first, kRows, kWideEnvs);
    for (int q = blockIdx.x; q < total; q += gridDim.x) {
        const ProductRef ref = product_ref(p, L.first, q, kRows);
        const int k = ref.k, rb = ref.row_block, g0 = ref.group * kWideEnvs;
        const int base = uniform(M.offset[k]), n = uniform(M.offset[k + 1]) - base, KS = (n + 31) >> 5;
        const int cnt = uniform(live_count(p, k));
        const int w0 = uniform(T.word_off[k]);
        __syncthreads();      // the previous unit is done with L
        if (threadIdx.x < kWideEnvs) {
            const int e = g0 + threadIdx.x < cnt ? live_env(p, k, g0 + threadIdx.x) : -1;
            L.env[threadIdx.x] = (e >= 0 && p.dense && na[(size_t)e * K + k] == 0) ? -1 : e;
        }
        __syncthreads();
        int env[2];
        env[0] = L.env[col];
        env[1] = L.env[16 + col];
        const int row0 = rb * kRows + wave * 16 * MT;
        doublex4 acc[MT][2][3];
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int c = 0; c < 3; ++c) acc[m][t][c] = doublex4{0.0, 0.0, 0.0, 0.0};
        const bool slow = matrix_overflows(M, p.model.alpha[k], k);
        if (dec && !slow) {
            const int mine = 16 * (wave & 1) + col, myenv = L.env[mine], safe = max(myenv, 0);
            const size_t at = (size_t)safe * N + base;
            const unsigned long long *mask = p.itm.mask + (size_t)safe * T.NW + w0;
            const uint4 *wa[MT];
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const int mt = min((row0 >> 4) + m, ((n + 15) >> 4) - 1);      // rows beyond the patch repeat its last tile
                wa[m] = p.tab.w + T.w_off[k] + (size_t)mt * KS * 3 * 64 + lane;
            }
            product_loop<MT, false, 1>(L.b, wa, src, at, EN, mask, myenv >= 0, n, KS, acc);
        }
        if (dec)
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int i0 = row0 + 16 * m + 4 * gq;
                    if (slow || not_finite(acc[m][t]))
                        pair_rows(p, k, env[t], i0, passive_rows(p, env[t], w0, i0, n), src, acc[m][t]);
                }
        __syncthreads();      // L.b is done with
        if (res) {
            stage_w5(p, L.w5, L.b5);
            for (int i = threadIdx.x; i < kWideEnvs * 64; i += kWG) {
                const int e = L.env[i >> 6];
                L.c4[i >> 6][i & 63] = e >= 0 ? p.itm.c4[((size_t)e * K + k) * 64 + (i & 63)] : 0.0f;
            }
        }
        __syncthreads();
        // residual and store: this lane holds rows row0 + 16 m + 4 gq + r of two envs
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const int i0 = row0 + 16 * m + 4 * gq;
            floatx4 r[2][3];
            if (res) {
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int c = 0; c < 3; ++c) r[t][c] = floatx4{L.b5[c], L.b5[c], L.b5[c], L.b5[c]};
                const float *z[4];
#pragma unroll
                for (int x = 0; x < 4; ++x) z[x] = p.tab.dec + (size_t)(base + min(i0 + x, n - 1)) * 64;
                const float *const c4[2] = {L.c4[col], L.c4[16 + col]};
                residual_rows<2>(L.w5, z, c4, 0, 64, r);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int e = env[t];
                if (e < 0 || i0 >= n) continue;
                const unsigned act = (unsigned)(p.itm.mask[(size_t)e * T.NW + w0 + (i0 >> 6)] >> (i0 & 63)) & 0xfu;
                store_rows(p.u + (size_t)e * N + base + i0, EN, act, n - i0, acc[m][t], r[t], dec, res);
            }
            __builtin_amdgcn_sched_barrier(0);      // one row tile's operands at a time
        }
    }
}

// Narrow tiles: 16 rows times 16 envs, the K steps split over the workgroup's
// four waves (each splits its own B fragments, no barrier in the loop), for
// batches whose wide tiles would leave the chip idle.
struct NarrowLds {
    int first[kMaxPatches + 1];
    alignas(16) float w5[3][64], b5[4];
    doublex4 part[kWaves][3][64];
    floatx4 rpart[kWaves][3][64];
};
ETAC_LDS_ALIGNED(NarrowLds, w5);

__global__ __launch_bounds__(kWG) void k_prop_narrow(StepParams p) {
    __shared__ NarrowLds L;
    const MeshDev &M = p.mesh;
    const TileDev &T = p.tile;
    const int K = M.K, N = M.N, lane = lane_id(), wave = uniform(threadIdx.x >> 6), gq = lane >> 4, col = lane & 15;
    const size_t EN = (size_t)p.E * N;
    const bool dec = step_decay(p), res = step_residual(p);
    const float *src = uhat_source(p);
    const int32_t *na = p.n_active ? p.n_active : p.itm.n_act;
    const int total = unit_prefix<kWaves>(K, L.first, [&](int kk) {
        const int k = M.order[kk], n = M.offset[k + 1] - M.offset[k];
        if (T.w_off[k] < 0) return 0;
        return ((live_count(p, k) + 15) >> 4) * ((n + 15) >> 4);
    });
    stage_w5(p, L.w5, L.b5);
    __syncthreads();
    for (int q = blockIdx.x; q < total; q += gridDim.x) {
        const int kk = unit_rank(L.first, K, q), k = uniform(M.order[kk]);
        const int base = uniform(M.offset[k]), n = uniform(M.offset[k + 1]) - base, KS = (n + 31) >> 5;
        const int cnt = uniform(live_count(p, k)), groups = (cnt + 15) >> 4;
        const int local = q - uniform(L.first[kk]), mt = local / groups, g0 = (local - mt * groups) * 16;
        const int w0 = uniform(T.word_off[k]);
        int e = g0 + col < cnt ? live_env(p, k, g0 + col) : -1;
        if (e >= 0 && p.dense && na[(size_t)e * K + k] == 0) e = -1;
        if (!__ballot(e >= 0)) continue;      // the same in every wave
        doublex4 acc[3];
        floatx4 r[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            acc[c] = doublex4{0.0, 0.0, 0.0, 0.0};
            r[c] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        const bool slow = matrix_overflows(M, p.model.alpha[k], k);
        if (dec && !slow) {
            const uint4 *wa = p.tab.w + T.w_off[k] + (size_t)mt * KS * 3 * 64 + lane;
            const int safe = max(e, 0);
            const float *me = src + (size_t)safe * N + base;
            const unsigned long long *mymask = p.itm.mask + (size_t)safe * T.NW + w0;
            // the next step's operands are requested before this one's are used
            uint4 a[3];
            float raw[3][8];
            unsigned bits = 0;
            auto fetch = [&](int s) {
                const int j0 = 32 * s + 8 * gq;
                const bool in = e >= 0 && j0 < n;
#pragma unroll
                for (int c = 0; c < 3; ++c) a[c] = wa[(size_t)(s * 3 + c) * 64];
                bits = in ? (unsigned)(mymask[j0 >> 6] >> (j0 & 63)) & 0xffu : 0u;
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    if (in) load8(me + c * EN, j0, n, raw[c]);
            };
            if (wave < KS) fetch(wave);
            for (int s = wave; s < KS; s += kWaves) {
                bf16x8 b[3][3], y[3];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    y[c] = __builtin_bit_cast(bf16x8, a[c]);
#pragma unroll
                    for (int x = 0; x < 8; ++x) raw[c][x] = (bits >> x) & 1u ? raw[c][x] : 0.0f;
                    split_bf16x3(raw[c], b[c]);
                }
                if (s + kWaves < KS) fetch(s + kWaves);
#pragma unroll
                for (int c = 0; c < 3; ++c) acc[c] += widen(mfma_bf16x3(y, b[c], floatx4{0.0f, 0.0f, 0.0f, 0.0f}));
            }
        }
        const int i0 = 16 * mt + 4 * gq;
        if (res) {
            const float *z[4];
#pragma unroll
            for (int x = 0; x < 4; ++x) z[x] = p.tab.dec + (size_t)(base + min(i0 + x, n - 1)) * 64;
            // columns without an env read their neighbour's row: some column has one
            const int ee = e >= 0 ? e : uniform(wave_max_int(e));
            const float *const c4[1] = {p.itm.c4 + ((size_t)ee * K + k) * 64};
            floatx4 rr[1][3] = {{r[0], r[1], r[2]}};
            residual_rows<1>(L.w5, z, c4, 16 * wave, 16 * wave + 16, rr);
#pragma unroll
            for (int c = 0; c < 3; ++c) r[c] = rr[0][c];
        }
        __syncthreads();          // the previous unit is done with L.part
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            L.part[wave][c][lane] = acc[c];
            L.rpart[wave][c][lane] = r[c];
        }
        __syncthreads();
        if (wave == 0 && e >= 0 && i0 < n) {
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float b = res ? L.b5[c] : 0.0f;
                acc[c] = L.part[0][c][lane];
                r[c] = L.rpart[0][c][lane] + b;
                for (int v = 1; v < kWaves; ++v) {
                    acc[c] += L.part[v][c][lane];
                    r[c] += L.rpart[v][c][lane];
                }
            }
            const unsigned act = (unsigned)(p.itm.mask[(size_t)e * T.NW + w0 + (i0 >> 6)] >> (i0 & 63)) & 0xfu;
            if (dec && (slow || not_finite(acc))) pair_rows(p, k, e, i0, passive_rows(p, e, w0, i0, n), src, acc);
            store_rows(p.u + (size_t)e * N + base + i0, EN, act, n - i0, acc, r, dec, res);
        }
    }
}

// ---------------------------------------------------------------------------
// U of the passive nodes: far patches
// ---------------------------------------------------------------------------

// Active nodes of every live far item in the patch's spatial order, with a box
// per 32 of them (in the adjoint its passive nodes: the sources of its sums
// are listed, PASSIVE).
template <bool PASSIVE>
__global__ __launch_bounds__(1024) void k_far_list(StepParams p) {
    __shared__ int first[kMaxPatches + 1];
    __shared__ int wsum[16];
    const MeshDev &M = p.mesh;
    const TileDev &T = p.tile;
    const int K = M.K, N = M.N, lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const int total = unit_prefix<16>(K, first, [&](int kk) { return T.w_off[M.order[kk]] < 0 ? live_count(p, M.order[kk]) : 0; });
    for (int q = blockIdx.x; q < total; q += gridDim.x) {
        const int kk = unit_rank(first, K, q), k = uniform(M.order[kk]), e = uniform(live_env(p, k, q - first[kk]));
        const int base = uniform(M.offset[k]), n = uniform(M.offset[k + 1]) - base;
        const unsigned long long *mask = p.itm.mask + (size_t)e * T.NW + T.word_off[k];
        int *list = (PASSIVE ? p.itm.plist : p.itm.alist) + (size_t)e * N + base;
        int run = 0;
        for (int i0 = 0; i0 < n; i0 += 1024) {
            const int i = i0 + threadIdx.x;
            const int node = i < n ? T.perm[base + i] : 0;
            const bool f = i < n && (((mask[node >> 6] >> (node & 63)) & 1ull) != 0ull) != PASSIVE;
            const unsigned long long bal = __ballot(f);
            __syncthreads();
            wsum[wave] = __popcll(bal);
            __syncthreads();
            int off = run, tot = 0;
            for (int w = 0; w < 16; ++w) {
                if (w < wave) off += wsum[w];
                tot += wsum[w];
            }
            if (f) list[off + lanes_below(bal)] = node;
            run += uniform(tot);
        }
        __threadfence_block();
        __syncthreads();
        float4 *box = (PASSIVE ? p.itm.pbox : p.itm.abox) + 2 * ((size_t)e * p.itm.NB + p.itm.box_off[k]);
        for (int t0 = 0; t0 < run; t0 += 1024) {
            const int t = t0 + threadIdx.x;
            const bool ok = t < run;
            const int g = base + (ok ? list[t] : list[0]);
            float lx = M.pos[g], ly = M.pos[N + g], lz = M.pos[2 * N + g];
            float hx = lx, hy = ly, hz = lz;
            if (!ok) { lx = ly = lz = 3.0e38f; hx = hy = hz = -3.0e38f; }
#pragma unroll
            for (int off = 16; off >= 1; off >>= 1) {
                lx = fminf(lx, __shfl_xor(lx, off)); ly = fminf(ly, __shfl_xor(ly, off)); lz = fminf(lz, __shfl_xor(lz, off));
                hx = fmaxf(hx, __shfl_xor(hx, off)); hy = fmaxf(hy, __shfl_xor(hy, off)); hz = fmaxf(hz, __shfl_xor(hz, off));
            }
            if (ok && (lane & 31) == 0) {
                box[2 * (t >> 5)] = make_float4(lx, ly, lz, 0.0f);
                box[2 * (t >> 5) + 1] = make_float4(hx, hy, hz, 0.0f);
            }
        }
        __syncthreads();
    }
}

// A workgroup takes 256 nodes of an item in the patch's spatial order, a wave
// 64 of them (a compact piece of the surface), a lane one node.  Runs of 32
// active nodes whose box lies beyond the cutoff of the wave's own box are
// passed over (64 boxes are tested at once, one per lane), the others are
// staged in LDS, two at a time, and summed pair by pair.  Bound by the VALU
// (sqrt and exp of every pair).  Units go tile by tile over a patch's items.
// 384 scenes of four 16384-node patches: 2690 us with runs read one at a time
// and units item by item, 1990 us.
struct FarLds {
    int first[kMaxPatches + 1];
    alignas(16) float w5[3][64], b5[4];
    float c4[64];
    float4 a[kWaves][64];
    float2 b[kWaves][64];
};
ETAC_LDS_ALIGNED(FarLds, w5);
ETAC_LDS_ALIGNED(FarLds, c4);

__global__ __launch_bounds__(kWG) void k_prop_far(StepParams p) {
    __shared__ FarLds L;
    const MeshDev &M = p.mesh;
    const TileDev &T = p.tile;
    const int K = M.K, N = M.N, lane = lane_id(), wave = uniform(threadIdx.x >> 6);
    const size_t EN = (size_t)p.E * N;
    const bool dec = step_decay(p), res = step_residual(p);
    const float *src = uhat_source(p);
    const int32_t *na = p.n_active ? p.n_active : p.itm.n_act;
    const int total = unit_prefix<kWaves>(K, L.first, [&](int kk) {
        const int k = M.order[kk];
        return T.w_off[k] < 0 ? live_count(p, k) * ((M.offset[k + 1] - M.offset[k] + kWG - 1) / kWG) : 0;
    });
    stage_w5(p, L.w5, L.b5);
    for (int q = blockIdx.x; q < total; q += gridDim.x) {
        const int kk = unit_rank(L.first, K, q), k = uniform(M.order[kk]);
        const int base = uniform(M.offset[k]), n = uniform(M.offset[k + 1]) - base;
        const int cnt = uniform(live_count(p, k)), local = q - uniform(L.first[kk]), tile = local / cnt;
        const int e = uniform(live_env(p, k, local - tile * cnt));
        const size_t item = (size_t)e * K + k;
        const int m = uniform(na[item]);
        __syncthreads();      // the previous unit is done with L
        if (res && threadIdx.x < 64) L.c4[lane] = p.itm.c4[item * 64 + lane];
        __syncthreads();
        const int s = tile * kWG + wave * 64 + lane;
        const int node = s < n ? T.perm[base + s] : 0;
        const bool pas = s < n && m > 0 &&
                         !((p.itm.mask[(size_t)e * T.NW + T.word_off[k] + (node >> 6)] >> (node & 63)) & 1ull);
        if (!__ballot(pas)) continue;
        const int g = base + node;
        const float px = M.pos[g], py = M.pos[N + g], pz = M.pos[2 * N + g];
        double a0 = 0.0, a1 = 0.0, a2 = 0.0;
        if (dec) {
            const float alpha = p.model.alpha[k], cut2 = cutoff_d2(alpha);
            float hi, lo;
            decay_rate(alpha, hi, lo);
            NearRuns runs(p.itm.abox + 2 * ((size_t)e * p.itm.NB + p.itm.box_off[k]), (m + 31) >> 5, pas, px, py, pz, cut2);
            const size_t row = (size_t)e * N + base;
            RunPair next;
            next.fetch(runs, M, p.itm.alist + row, m, base, src + row, EN);
            while (next.r[0] >= 0) {
                const int c[2] = {next.c[0], next.c[1]};
                wave_sync();
                L.a[wave][lane] = make_float4(next.x[0], next.x[1], next.x[2], next.x[3]);
                L.b[wave][lane] = make_float2(next.x[4], next.x[5]);
                wave_sync();
                next.fetch(runs, M, p.itm.alist + row, m, base, src + row, EN);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f;
#pragma unroll 4
                    for (int j = 32 * h; j < 32 * h + c[h]; ++j) {
                        const float4 pa = L.a[wave][j];
                        const float2 pb = L.b[wave][j];
                        const float dx = pa.x - px, dy = pa.y - py, dz = pa.z - pz;
                        const float d = __builtin_amdgcn_sqrtf(dx * dx + dy * dy + dz * dz);
                        const float w = __builtin_amdgcn_exp2f(hi * d);
                        s0 += w * pa.w; s1 += w * pb.x; s2 += w * pb.y;
                    }
                    a0 += s0; a1 += s1; a2 += s2;
                }
            }
        }
        float r0 = 0.0f, r1 = 0.0f, r2 = 0.0f;
        if (res) {
            const float *z = p.tab.dec + (size_t)g * 64;
            r0 = L.b5[0]; r1 = L.b5[1]; r2 = L.b5[2];
#pragma unroll 4
            for (int c = 0; c < 64; c += 4) {
                const floatx4 zz = *reinterpret_cast<const floatx4 *>(z + c);
                const floatx4 cc = *reinterpret_cast<const floatx4 *>(&L.c4[c]);
                const floatx4 wx = *reinterpret_cast<const floatx4 *>(&L.w5[0][c]);
                const floatx4 wy = *reinterpret_cast<const floatx4 *>(&L.w5[1][c]);
                const floatx4 wz = *reinterpret_cast<const floatx4 *>(&L.w5[2][c]);
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    const float v = relu1(zz[h] + cc[h]);
                    r0 += wx[h] * v; r1 += wy[h] * v; r2 += wz[h] * v;
                }
            }
        }
        if (pas) {
            float *o = p.u + (size_t)e * N + g;
            o[0] = (float)(a0 + (double)r0);
            o[EN] = (float)(a1 + (double)r1);
            o[2 * EN] = (float)(a2 + (double)r2);
        }
    }
}

template <bool FROM_INPUT, bool ROWS>
static void launch_contact_items(const StepParams &p, bool merged, int nt, hipStream_t st) {
    if (merged) {
        hipLaunchKernelGGL((k_front<FROM_INPUT, ROWS>), dim3(nt + p.E), dim3(kWG), 0, st, p);
        return;
    }
    const dim3 grid(p.E * p.splits);
    if constexpr (!FROM_INPUT) {
        if (p.tile.NW > kDirectWords) {
            hipLaunchKernelGGL((k_contact_items<FROM_INPUT, ROWS, false>), grid, dim3(kWG), 0, st, p);
            return;
        }
    }
    hipLaunchKernelGGL((k_contact_items<FROM_INPUT, ROWS, true>), grid, dim3(kWG), 0, st, p);
}

static void launch_contact_items(const StepParams &p, bool merged, int nt, hipStream_t st) {
    const bool rows = p.scene.rows_per_env != 0;
    if (p.cobj_in) launch_contact_items<true, false>(p, merged, nt, st);
    else if (rows) launch_contact_items<false, true>(p, merged, nt, st);
    else launch_contact_items<false, false>(p, merged, nt, st);
}

constexpr long long kAllPairs = 8 << 20;      // weights, words of surfaces that get every table
constexpr int kAllWords = 2048;

// Workgroups per env of the contact pass: enough to fill the chip.
static int contact_splits(const Plan &pl, int E) {
    int s = 1;
    while (E * s < kSplitEnvs * pl.cu_count && s * kWaves * 4 < pl.tile.NW) s *= 2;
    return s;
}

hipError_t launch_contact(const Plan &p, const SceneDev &s, int8_t *cobj, float *uhat, int32_t *n_active,
                          hipStream_t st) {
    return launch_contact_rows(p, s, cobj, uhat, n_active, nullptr, st);
}

hipError_t launch_contact_rows(const Plan &pl, const SceneDev &s, int8_t *cobj, float *uhat, int32_t *n_active,
                               int32_t *n_touch, hipStream_t st) {
    if (s.E == 0) return hipSuccess;
    StepParams p{};
    p.mesh = pl.mesh;
    p.tile = pl.tile;
    p.scene = s;
    p.model = ModelDev{ETAC_DECAY_ONLY, nullptr, nullptr};
    p.E = s.E;
    p.splits = contact_splits(pl, s.E);
    p.u = uhat;
    p.cobj_out = cobj;
    p.n_active = n_active;
    p.n_touch = n_touch;
    const int slot = timer_begin(pl, ETAC_TIMER_CONTACT, st);
    if (!s.rows_per_env && pl.tile.NW <= (p.splits == 1 ? kDirectWords : kDirectWords / 2)) {
        hipLaunchKernelGGL(k_contact_small, dim3(s.E), dim3(kWG), 0, st, p);
    } else {
        if (p.splits > 1) hipLaunchKernelGGL(k_zero_counts, dim3(64), dim3(kWG), 0, st, p);
        launch_contact_items(p, false, 0, st);
    }
    const hipError_t e = hipGetLastError();
    timer_end(pl, ETAC_TIMER_CONTACT, slot, st);
    return e;
}

void shape_step(const Plan &pl, StepParams &p) {
    p.mesh = pl.mesh;
    p.tile = pl.tile;
    p.tab = pl.tab;
    p.itm = pl.itm;
    p.cus = pl.cu_count;
    p.items = (long long)p.E * pl.K;
    p.words = (long long)p.E * pl.tile.NW;
    p.table_units = p.model.mode != ETAC_DECAY_ONLY ? std::min(pl.tile.NW, 2 * pl.cu_count) : 0;
    p.matrix_units = p.model.mode != ETAC_RESIDUAL_ONLY ? pl.tile.near_rows : 0;
    // Small batches: tables and contact share a launch and every item is
    // listed.  A launch costs 5-7 us; on one 32 x 32 pad the whole step takes
    // about 50, and the listing of 256 items would take as long as visiting them.
    p.dense = p.items <= 256;
    // Wide tiles from 128 envs on: below, they would leave compute units idle.
    p.wide = p.E >= 128;
    p.splits = contact_splits(pl, p.E);
}

void launch_live(const int32_t *n_active, int E, int K, int *live, int *live_cnt, hipStream_t st) {
    hipLaunchKernelGGL(k_live, dim3(K), dim3(1024), 0, st, n_active, E, K, live, live_cnt);
}

void launch_front(const Plan &pl, StepParams p, hipStream_t st) {
    const int nt = p.table_units + p.matrix_units;
    // On surfaces of up to 16 words tables and contact share a launch.  On large
    // ones contact comes first, and only patches in contact get tables: one hand
    // that touches one of 40 patches of 2048 nodes 316 us with all tables (the
    // matrices alone are 1 GB), 90 us; one of 400 patches of 256 nodes 150 and 65.
    // In between the tables are a launch's worth and clear the contact's counts,
    // which would take a launch of their own.
    const bool merged = p.dense && p.splits == 1 && nt > 0;
    p.touched = !merged && (pl.tile.pairs > kAllPairs || pl.tile.NW > kAllWords);
    if (!merged && (p.touched ? p.splits > 1 : nt > 0 || p.splits > 1)) {
        if (p.touched || nt == 0) hipLaunchKernelGGL(k_zero_counts, dim3(64), dim3(kWG), 0, st, p);
        else hipLaunchKernelGGL(k_tables, dim3(std::max(nt, 64)), dim3(kWG), 0, st, p);
    }
    launch_contact_items(p, merged, nt, st);
    const int32_t *na = p.n_active ? p.n_active : pl.itm.n_act;
    if (!p.dense) launch_live(na, p.E, pl.K, pl.itm.live, pl.itm.live_cnt, st);
    if (p.touched && nt > 0) hipLaunchKernelGGL(k_tables, dim3(nt), dim3(kWG), 0, st, p);
}

void launch_pool(const Plan &pl, const StepParams &p, hipStream_t st) {
    const long long cus = p.cus;
    if (!p.recall) {
        if (p.items <= kPoolItems && pl.tile.n_far == 0) {
            hipLaunchKernelGGL(k_pool, dim3((unsigned)std::min(p.items, cus)), dim3(64 * kPoolWaves), 0, st, p);
            return;
        }
        hipLaunchKernelGGL(k_pool_passive, dim3((unsigned)std::min((p.words / kPassiveWords + p.items) / kWaves + 1, 8 * cus)),
                           dim3(kWG), 0, st, p);
        hipLaunchKernelGGL(k_pool_active, dim3((unsigned)std::min((p.words / kActiveWords + p.items) / kWaves + 1, 2 * cus)),
                           dim3(kWG), 0, st, p);
    }
    hipLaunchKernelGGL(k_pool_finish, dim3((unsigned)std::min(p.items / kWaves + 1, 3 * cus)), dim3(kWG), 0, st, p);
}

void launch_far_lists(const StepParams &p, bool passive, hipStream_t st) {
    const dim3 grid((unsigned)std::min<long long>(p.items, 2 * p.cus));
    if (passive) hipLaunchKernelGGL(k_far_list<true>, grid, dim3(1024), 0, st, p);
    else hipLaunchKernelGGL(k_far_list<false>, grid, dim3(1024), 0, st, p);
}

// Tiles of 128 rows in the wide product where they give every CU a unit and more,
// if an object touches a patch, and are not padding: 1024 hands (342 units) 314
// us, 326 in tiles of 64 rows; 4096 pads of 1024 nodes (1024 units) 335 and 398; but
// 1024 of those pads (256 units) 158 and 150, 1024 hands of 64 64-node patches 105
// and 98, 128 envs on forty patches of 2048 nodes, three in contact on each, 700 and
// 660.
static bool tall_tiles(const Plan &pl, const StepParams &p) {
    const long long objects = std::min(p.cobj_in ? pl.max_obj : p.scene.O, pl.K);
    const long long envs = p.E * objects / pl.K, groups = (envs + kWideEnvs - 1) / kWideEnvs;
    return p.wide && envs >= kWideEnvs && pl.tile.near_blocks * groups > pl.cu_count && pl.tile.near_blocks * 128 <= pl.tile.near_rows * 20;
}

hipError_t launch_step(const Plan &pl, const SceneDev *s, const ModelDev &m, int n_envs,
                       const int8_t *cobj_in, const float *uhat_in, float *u, int8_t *cobj_out,
                       int32_t *n_active, uint32_t *saved, hipStream_t st, int32_t *n_touch) {
    if (n_envs == 0) return hipSuccess;
    StepParams p{};
    p.scene = s ? *s : SceneDev{nullptr, nullptr, nullptr, nullptr, nullptr, 0, 1};
    p.model = m;
    p.E = n_envs;
    p.cobj_in = cobj_in;
    p.uhat_in = uhat_in;
    p.u = u;
    p.cobj_out = cobj_out;
    p.n_active = n_active;
    p.n_touch = n_touch;
    p.saved = saved;
    shape_step(pl, p);
    const long long cus = p.cus;
    const int slot = timer_begin(pl, ETAC_TIMER_STEP, st);
    launch_front(pl, p, st);
    if (step_residual(p)) launch_pool(pl, p, st);
    if (pl.tile.n_near) {
        if (tall_tiles(pl, p)) hipLaunchKernelGGL(k_prop_wide<2>, dim3((unsigned)(2 * cus)), dim3(kWG), 0, st, p);
        else if (p.wide) hipLaunchKernelGGL(k_prop_wide<1>, dim3((unsigned)(2 * cus)), dim3(kWG), 0, st, p);
        else
            hipLaunchKernelGGL(k_prop_narrow, dim3((unsigned)std::min<long long>((long long)((n_envs + 15) / 16) * pl.tile.near_rows, 4 * cus)),
                               dim3(kWG), 0, st, p);
    }
    if (pl.tile.n_far) {
        if (step_decay(p)) launch_far_lists(p, false, st);
        hipLaunchKernelGGL(k_prop_far, dim3((unsigned)std::min(p.words / 4 + p.items, 8 * cus)), dim3(kWG), 0, st, p);
    }
    const hipError_t e = hipGetLastError();
    timer_end(pl, ETAC_TIMER_STEP, slot, st);
    return e;
}

}  // namespace etac
