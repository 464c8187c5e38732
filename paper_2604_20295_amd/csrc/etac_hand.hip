// Articulated hand on gfx950: every patch rides on one link of the hand, its
// nodes, normals, origin, u_hat and U given in that link's frame.  Contact
// of a patch covers the env's objects and the collision primitives of the
// other links it may touch (self-contact, Sec. III-A contact detection),
// all expressed in the patch's link frame; the contact reward of Sec. IV-B
// (contact-reward equation) comes from per-item counts the contact pass
// already produces.
//
//   k_hand_scene  : half a wave per (env, patch) item, a lane per object or
//                   link, fills the item's row of candidates (relative poses,
//                   FP64 then rounded to FP32, culled against the patch's
//                   bounding sphere);
//   k_hand_reward : one thread per env, n_a, touched links and r_contact;
//   k_pose_hand   : a wave per env, the chain rule from the rows' relative-pose
//                   gradients to object and link poses, summed in item and
//                   slot order in FP64.
// The step, the contact pass and the adjoint kernels run unchanged on
// the rows (SceneDev with one row per item).
#include "etac_device.h"

namespace etac {

// Relative pose of a world pose (Rw, tw) in the frame (Rl, tl):
//   R' = Rl^T Rw,  t' = Rl^T (tw - tl),
// every entry a sum of three products taken as (x0 y0 + x1 y1) + x2 y2 in
// FP64, no fused multiply-add, then rounded to FP32 (the values the contact
// test reads).
__device__ __forceinline__ void relative_pose(const double Rl[9], const double tl[3], const double Rw[9],
                                              const double tw[3], float Rr[9], float tr[3]) {
#pragma clang fp contract(off)
    const double d[3] = {tw[0] - tl[0], tw[1] - tl[1], tw[2] - tl[2]};
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            Rr[a * 3 + c] = (float)((Rl[0 * 3 + a] * Rw[0 * 3 + c] + Rl[1 * 3 + a] * Rw[1 * 3 + c]) +
                                    Rl[2 * 3 + a] * Rw[2 * 3 + c]);
#pragma unroll
    for (int c = 0; c < 3; ++c)
        tr[c] = (float)((Rl[0 * 3 + c] * d[0] + Rl[1 * 3 + c] * d[1]) + Rl[2 * 3 + c] * d[2]);
}

// World pose of link j's collision primitive: Rw = Rj C_R, tw = Rj C_t + tj
// (same summation order).
__device__ __forceinline__ void primitive_world(const double Rj[9], const double tj[3], const float *CR,
                                                const float *Ct, double Rw[9], double tw[3]) {
#pragma clang fp contract(off)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
            Rw[a * 3 + c] = (Rj[a * 3 + 0] * (double)CR[0 * 3 + c] + Rj[a * 3 + 1] * (double)CR[1 * 3 + c]) +
                            Rj[a * 3 + 2] * (double)CR[2 * 3 + c];
        tw[a] = ((Rj[a * 3 + 0] * (double)Ct[0] + Rj[a * 3 + 1] * (double)Ct[1]) + Rj[a * 3 + 2] * (double)Ct[2]) +
                tj[a];
    }
}

__device__ __forceinline__ void load_pose(const float *R, const float *t, double Rd[9], double td[3]) {
#pragma unroll
    for (int i = 0; i < 9; ++i) Rd[i] = R[i];
#pragma unroll
    for (int i = 0; i < 3; ++i) td[i] = t[i];
}

struct HandSceneParams {
    MeshDev mesh;
    SceneDev world;
    LinksDev links;
    HandDev hand;
    int n_items;
};

// Half a wave per item: lane t < O takes object t, lane O + j link j's
// primitive (O + L <= 32).  Candidates are those whose bounding ball may reach
// the patch, in lane order, objects first.  A thread per item went through them
// one after the other, each a round trip to memory (1024 hands of 16 patches:
// 25.6 us, 9.9 us now).
constexpr int kSceneLanes = 32;
static_assert(ETAC_MAX_OBJ + ETAC_MAX_LINKS <= kSceneLanes, "a lane per candidate");

__global__ __launch_bounds__(256) void k_hand_scene(HandSceneParams p, long long group0) {
    const int t = threadIdx.x & (kSceneLanes - 1);
    const long long at = (group0 + blockIdx.x) * (256 / kSceneLanes) + threadIdx.x / kSceneLanes;
    const int item = (int)min(at, (long long)p.n_items - 1);      // whole half waves beyond the last repeat it, without stores
    const MeshDev &M = p.mesh;
    const HandDev &H = p.hand;
    const int K = M.K, L = H.L, O = p.world.O;
    const int e = item / K, k = item - e * K;
    const int l = H.patch_link[k];
    const bool is_obj = t < O, is_link = !is_obj && t - O < L;
    const int j = is_link ? t - O : 0;
    const size_t eo = (size_t)e * O + (is_obj ? t : 0);
    const unsigned pairs = H.collide[l] & ~(1u << l);
    const int ty = is_obj ? p.world.type[eo] : H.ptype[j];
    bool in = is_obj ? t < min(p.world.n_obj[e], O) : is_link && ((pairs >> j) & 1u);
    in = in && (unsigned)ty <= (unsigned)ETAC_CAPSULE;
    const float4 b = M.bound[k];
    const float *sh = is_obj ? p.world.shape + 4 * eo : H.pshape + 4 * j;
    double Rl[9], tl[3], Rj[9], tj[3], Rw[9], tw[3];
    load_pose(p.links.rot + ((size_t)e * L + l) * 9, p.links.trans + ((size_t)e * L + l) * 3, Rl, tl);
    load_pose(is_obj ? p.world.rot + 9 * eo : p.links.rot + ((size_t)e * L + j) * 9,
              is_obj ? p.world.trans + 3 * eo : p.links.trans + ((size_t)e * L + j) * 3, Rj, tj);
    primitive_world(Rj, tj, H.prot + 9 * j, H.ptrans + 3 * j, Rw, tw);
#pragma unroll
    for (int i = 0; i < 9; ++i) Rw[i] = is_obj ? Rj[i] : Rw[i];
#pragma unroll
    for (int i = 0; i < 3; ++i) tw[i] = is_obj ? tj[i] : tw[i];
    float Rr[9], tr[3], shape[4];
    relative_pose(Rl, tl, Rw, tw, Rr, tr);
#pragma unroll
    for (int i = 0; i < 4; ++i) shape[i] = sh[i];
    const bool take = in && ball_reaches(b, in ? ty : ETAC_SPHERE, shape, tr);
    const unsigned long long both = __ballot(take);
    const unsigned mine = (unsigned)(both >> (lane_id() & kSceneLanes));
    if (at >= p.n_items) return;
    const size_t row = (size_t)item;
    if (take) {
        const size_t s = row * p.hand.cap + __popc(mine & ((1u << t) - 1u));
        p.hand.type[s] = ty;
        p.hand.src[s] = (int8_t)t;
#pragma unroll
        for (int i = 0; i < 4; ++i) p.hand.shape[4 * s + i] = shape[i];
#pragma unroll
        for (int i = 0; i < 9; ++i) p.hand.rot[9 * s + i] = Rr[i];
#pragma unroll
        for (int i = 0; i < 3; ++i) p.hand.trans[3 * s + i] = tr[i];
    }
    if (t == 0) {
        H.n_obj[row] = __popc(mine);
        H.n_ext[row] = __popc(mine & ((1u << O) - 1u));
    }
}

hipError_t launch_hand_scene(const Plan &pl, const SceneDev &world, const LinksDev &links, SceneDev *rows,
                             hipStream_t st) {
    const HandDev &H = *pl.hand;
    HandSceneParams p{pl.mesh, world, links, H, world.E * pl.K};
    *rows = SceneDev{H.n_obj, H.type, H.shape, H.rot, H.trans, world.E, H.cap};
    rows->rows_per_env = pl.K;
    rows->src = H.src;
    rows->n_ext = H.n_ext;
    if (p.n_items == 0) return hipSuccess;
    launch_slices(((long long)p.n_items + 256 / kSceneLanes - 1) / (256 / kSceneLanes), [&](long long first, dim3 grid) {
        hipLaunchKernelGGL(k_hand_scene, grid, dim3(256), 0, st, p, first);
    });
    return hipGetLastError();
}

// r_contact = (links touched by an object) / L + omega_a (n_a / N if n_a > 0,
// else -0.1), n_a the nodes won by objects over the hand.
__global__ __launch_bounds__(256) void k_hand_reward(int E, int K, int L, int N, const int *patch_link,
                                                     const int32_t *n_touch, float omega_a, int32_t *n_a,
                                                     uint32_t *link_mask, float *r_contact) {
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= E) return;
    long long s = 0;
    unsigned mask = 0;
    for (int k = 0; k < K; ++k) {
        const int t = n_touch[(size_t)e * K + k];
        s += t;
        if (t > 0) mask |= 1u << patch_link[k];
    }
    if (n_a) n_a[e] = (int32_t)s;
    if (link_mask) link_mask[e] = mask;
    if (r_contact) {
        const double ra = s > 0 ? (double)s / (double)N : -0.1;
        r_contact[e] = (float)((double)__popc(mask) / (double)L + (double)omega_a * ra);
    }
}

hipError_t launch_hand_reward(const Plan &pl, int n_envs, const int32_t *n_touch, float omega_a, int32_t *n_a,
                              uint32_t *link_mask, float *r_contact, hipStream_t st) {
    if (n_envs == 0 || (!n_a && !link_mask && !r_contact)) return hipSuccess;
    hipLaunchKernelGGL(k_hand_reward, dim3((n_envs + 255) / 256), dim3(256), 0, st, n_envs, pl.K, pl.hand->L, pl.N,
                       pl.hand->patch_link, n_touch, omega_a, n_a, link_mask, r_contact);
    return hipGetLastError();
}

// Chain rule of the hand's pose adjoint.  A row slot of item (e, k) on link
// l holds G' = dL/dR', g' = dL/dt' of its candidate's relative pose.  With the
// candidate's world pose (Rw, tw):
//   source : dL/dRw = Rl G',  dL/dtw = Rl g'
//            (link j's primitive: dL/dRj += dL/dRw C_R^T + dL/dtw C_t^T,
//             dL/dtj += dL/dtw);
//   frame  : dL/dRl += Rw G'^T + (tw - tl) g'^T,  dL/dtl -= Rl g'.
// A wave per env.  Its slots in contact are listed 64 at a time; a lane forms
// the two contributions of its slot, then a lane per component of a target (an
// object, t < O, or link t - O) adds those of its target in item and slot
// order, in FP64.  A thread per target that walked the slots itself waited for
// each (1024 hands: 121 us, 13.5 us now).
struct PoseHandParams {
    SceneDev world;
    LinksDev links;
    HandDev hand;
    const float *part;       // [E][NC][cap][12], written for items in contact
    const int *n_act;        // [E K]
    const int *chunk_off;    // [K+1]
    int NC;
    int E, K;
    float *grad_rot, *grad_trans, *grad_link_rot, *grad_link_trans;
};

struct PoseHandLds {
    double src[64][13], frame[64][13];      // contributions of a slot to its source and its frame
    double sum[ETAC_MAX_OBJ + ETAC_MAX_LINKS][12];
    unsigned long long slots[ETAC_MAX_OBJ + ETAC_MAX_LINKS][2];      // a target's slots, as frame and as source
    uint16_t list[64 * kMaxRowObj];         // slots of 64 patches
};

__global__ __launch_bounds__(64) void k_pose_hand(PoseHandParams p) {
    __shared__ PoseHandLds S;
    const HandDev &H = p.hand;
    const int O = p.world.O, L = H.L, T = O + L, e = blockIdx.x, lane = threadIdx.x;
    for (int i = lane; i < T * 12; i += 64) S.sum[i / 12][i % 12] = 0.0;
    for (int k0 = 0; k0 < p.K; k0 += 64) {
        // slots of the patches in contact, in order
        const int kl = min(k0 + lane, p.K - 1);
        const size_t rl = (size_t)e * p.K + kl;
        const int mine = k0 + lane < p.K && p.n_act[rl] > 0 ? min(H.n_obj[rl], H.cap) : 0;
        int inc = mine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(inc, off);
            if (lane >= off) inc += v;
        }
        const int total = uniform(__shfl(inc, 63));
        wave_sync();
        for (int s = 0; s < mine; ++s) S.list[inc - mine + s] = (uint16_t)(lane * kMaxRowObj + s);
        wave_sync();
        for (int c0 = 0; c0 < total; c0 += 64) {
            const int cnt = min(64, total - c0);
            int to = -1, frame = -1;      // the targets of this lane's contributions
            if (lane < cnt) {
                const int slot = S.list[c0 + lane], k = k0 + slot / kMaxRowObj, s = slot % kMaxRowObj;
                const size_t row = (size_t)e * p.K + k;
                const int l = H.patch_link[k], src = H.src[row * H.cap + s];
                double Rl[9], tl[3], Gp[9], tp[3];
                load_pose(p.links.rot + ((size_t)e * L + l) * 9, p.links.trans + ((size_t)e * L + l) * 3, Rl, tl);
#pragma unroll
                for (int i = 0; i < 9; ++i) Gp[i] = 0.0;
#pragma unroll
                for (int i = 0; i < 3; ++i) tp[i] = 0.0;
                for (int h = p.chunk_off[k]; h < p.chunk_off[k + 1]; ++h) {
                    const float *gp = p.part + (((size_t)e * p.NC + h) * H.cap + s) * 12;
#pragma unroll
                    for (int i = 0; i < 9; ++i) Gp[i] += gp[i];
#pragma unroll
                    for (int i = 0; i < 3; ++i) tp[i] += gp[9 + i];
                }
                double GRw[9], gtw[3];
#pragma unroll
                for (int a = 0; a < 3; ++a) {
#pragma unroll
                    for (int c = 0; c < 3; ++c)
                        GRw[a * 3 + c] = Rl[a * 3 + 0] * Gp[0 * 3 + c] + Rl[a * 3 + 1] * Gp[1 * 3 + c] +
                                         Rl[a * 3 + 2] * Gp[2 * 3 + c];
                    gtw[a] = Rl[a * 3 + 0] * tp[0] + Rl[a * 3 + 1] * tp[1] + Rl[a * 3 + 2] * tp[2];
                }
                double Rw[9], tw[3];
                if (src < O) {
                    load_pose(p.world.rot + ((size_t)e * O + src) * 9, p.world.trans + ((size_t)e * O + src) * 3, Rw, tw);
#pragma unroll
                    for (int i = 0; i < 9; ++i) S.src[lane][i] = GRw[i];
                } else {
                    const int j = src - O;
                    const float *CR = H.prot + 9 * j, *Ct = H.ptrans + 3 * j;
                    double Rj[9], tj[3];
                    load_pose(p.links.rot + ((size_t)e * L + j) * 9, p.links.trans + ((size_t)e * L + j) * 3, Rj, tj);
                    primitive_world(Rj, tj, CR, Ct, Rw, tw);
#pragma unroll
                    for (int a = 0; a < 3; ++a)
#pragma unroll
                        for (int b = 0; b < 3; ++b)
                            S.src[lane][a * 3 + b] = GRw[a * 3 + 0] * (double)CR[b * 3 + 0] + GRw[a * 3 + 1] * (double)CR[b * 3 + 1] +
                                                     GRw[a * 3 + 2] * (double)CR[b * 3 + 2] + gtw[a] * (double)Ct[b];
                }
#pragma unroll
                for (int a = 0; a < 3; ++a) {
#pragma unroll
                    for (int b = 0; b < 3; ++b)
                        S.frame[lane][a * 3 + b] = (Rw[a * 3 + 0] * Gp[b * 3 + 0] + Rw[a * 3 + 1] * Gp[b * 3 + 1] +
                                                    Rw[a * 3 + 2] * Gp[b * 3 + 2]) + (tw[a] - tl[a]) * tp[b];
                    S.frame[lane][9 + a] = -gtw[a];
                    S.src[lane][9 + a] = gtw[a];
                }
                to = src;
                frame = O + l;
            }
            unsigned long long as_frame = 0, as_src = 0;      // lane t: target t's slots
            for (int t = 0; t < T; ++t) {
                const unsigned long long f = __ballot(frame == t), o = __ballot(to == t && frame != t);
                as_frame = lane == t ? f : as_frame;
                as_src = lane == t ? o : as_src;
            }
            if (lane < T) {
                S.slots[lane][0] = as_frame;
                S.slots[lane][1] = as_src;
            }
            wave_sync();
            for (int i = lane; i < T * 12; i += 64) {
                const int t = i / 12, c = i - 12 * t;
                double v = S.sum[t][c];
                const unsigned long long f = S.slots[t][0];
                for (unsigned long long m = f | S.slots[t][1]; m; m &= m - 1) {
                    const int q = __ffsll(m) - 1;
                    v += (f >> q) & 1ull ? S.frame[q][c] : S.src[q][c];
                }
                S.sum[t][c] = v;
            }
            wave_sync();
        }
    }
    wave_sync();
    for (int i = lane; i < T * 12; i += 64) {
        const int t = i / 12, c = i - 12 * t;
        const float v = (float)S.sum[t][c];
        if (t < O) {
            if (c < 9) p.grad_rot[((size_t)e * O + t) * 9 + c] = v;
            else p.grad_trans[((size_t)e * O + t) * 3 + c - 9] = v;
        } else {
            if (c < 9) p.grad_link_rot[((size_t)e * L + t - O) * 9 + c] = v;
            else p.grad_link_trans[((size_t)e * L + t - O) * 3 + c - 9] = v;
        }
    }
}

hipError_t launch_pose_hand(const Plan &pl, const SceneDev &world, const LinksDev &links, float *grad_rot,
                            float *grad_trans, float *grad_link_rot, float *grad_link_trans, hipStream_t st) {
    if (world.E == 0) return hipSuccess;
    PoseHandParams p{world, links, *pl.hand, pl.hand->pose_part, pl.itm.n_act, pl.tile.chunk_off, pl.tile.NC,
                     world.E, pl.K, grad_rot, grad_trans, grad_link_rot, grad_link_trans};
    hipLaunchKernelGGL(k_pose_hand, dim3(world.E), dim3(64), 0, st, p);
    return hipGetLastError();
}

}  // namespace etac
