// Internal declarations shared by the host API and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/etac.h"

namespace etac {

constexpr int kWG = 256;           // threads per workgroup: 4 waves of 64
constexpr int kWaves = kWG / 64;
constexpr int kSavedWords = ETAC_SAVED_WORDS;   // pooling record per (env, patch) item
// parameter reduction: words of a node block's record (dW4[:, :64], dW2, dW1
// with db1 as input column 9 as 36 blocks of 16 x 16, db2), of a routing
// workgroup's (dW2, dW1 and db1 by input, db2), and all its columns
constexpr int kNodeRecWords = 36 * 256 + 64;
constexpr int kRouteWords = 4096 + 640 + 64;
constexpr int kRouteGroups = 2;                   // routing workgroups per compute unit
constexpr int kRedRoute = 37 * 256, kRedItem = kRedRoute + 19 * 256, kRedRank = kRedItem + 256,
              kRedW5 = kRedRank + 8192, kRedCols = kRedW5 + 256;
constexpr int kRegUnitNodes = 256;               // nodes of a regressor unit, the least of a plan
constexpr size_t kRegRows = 1 << 18;             // rows of 1 KB its units may take (or one per item)
constexpr int kAlphaSegs = 32;
constexpr int kPhiSegs = 64;                      // segments of the parameter reduction
constexpr int kMaxPatches = 1024;  // per-patch counters of the contact kernel live in LDS
constexpr int kSplitEnvs = 4;      // envs per compute unit up to which an env's contact takes several workgroups
constexpr int kDefaultWgPerCu = 2;
constexpr int kDefaultBatch = 4;   // default of the batch knobs
constexpr int kDefaultDecayWgPerCu = 3;
constexpr int kDefaultNetBatch = 2;

// Device view of the plan's mesh copy.
struct MeshDev {
    const float *pos;      // [3][N]
    const float *nrm;      // [3][N]
    const float *origin;   // [K][3]
    const int *offset;     // [K+1]
    const float4 *bound;   // [K] conservative bounding sphere (cx, cy, cz, radius)
    const int16_t *node_patch;  // [N] patch of each node
    const int *order;      // [K] patches sorted by node count, largest first
    const float *xbound;   // [K] largest |component| of p - o_k and of n over the patch's nodes (rounded up)
    int K, N, n_max;
};

// Objects the contact test sees, in rows of O candidates: one row per env
// (rows_per_env = 0), or one row per (env, patch) item (rows_per_env = K:
// the articulated hand, whose rows hold each patch's candidates in its link
// frame).  With `src`, contact_obj reports src[row][winner] instead of the
// winner's slot; with `n_ext`, slots below n_ext[row] are external objects
// (their nodes count towards the contact reward).
struct SceneDev {
    const int *n_obj;      // [rows]
    const int *type;       // [rows][O]
    const float *shape;    // [rows][O][4]
    const float *rot;      // [rows][O][9]
    const float *trans;    // [rows][O][3]
    int E, O;
    int rows_per_env = 0;
    const int8_t *src = nullptr;   // [rows][O]
    const int *n_ext = nullptr;    // [rows]
};

__host__ __device__ inline size_t scene_row(const SceneDev &S, int e, int k) {
    return S.rows_per_env ? (size_t)e * S.rows_per_env + k : (size_t)e;
}

// Articulated hand (etac_plan_set_hand): the link description on the device
// and the per-item candidate table its pre-pass fills.
constexpr int kMaxLinks = 24;
constexpr int kMaxRowObj = 32;     // candidates per item row (one bit each in a 32-bit mask)

struct HandDev {
    int L;
    int cap;                       // row capacity: plan max_obj + largest self-contact set
    const int *patch_link;         // [K]
    const unsigned *collide;       // [L]
    const int *ptype;              // [L] primitive type or -1
    const float *pshape;           // [L][4]
    const float *prot;             // [L][9] primitive pose in its link frame
    const float *ptrans;           // [L][3]
    // candidate table, one row per (env, patch) item
    int *n_obj;                    // [E K]
    int *n_ext;                    // [E K]
    int *type;                     // [E K][cap]
    float *shape;                  // [E K][cap][4]
    float *rot;                    // [E K][cap][9]
    float *trans;                  // [E K][cap][3]
    int8_t *src;                   // [E K][cap]
    float *pose_part;              // [E][NC][cap][12] relative-pose gradient parts (backward)
    int *n_touch;                  // [E K] reward counts when the caller passes none
};

// Per-step inputs of the hand: link poses.
struct LinksDev {
    const float *rot;              // [E][L][9]
    const float *trans;            // [E][L][3]
};

// Node words and decay tiles of the mesh (plan copies, fixed at creation).
// A word is up to 64 consecutive nodes of one patch, the unit of the contact
// masks.  Patches of at most kNearNodes nodes have a decay matrix; the others
// ("far") take Eq. 1 pair by pair in a spatial order of their nodes.
constexpr int kNearNodes = 2048;
constexpr size_t kDecayMatrixBytes = size_t(1) << 30;   // bound on all decay matrices of a plan

constexpr int kPoseWords = 16;     // words per pose part of the contact adjoint
constexpr int kBlockNodes = 64;    // nodes per unit of the network adjoint's node pass

struct TileDev {
    const int4 *word;          // [NW] patch, first node (index into the mesh), nodes, word of the patch
    const int2 *row_tile;      // [near_rows] near patch and tile of 16 of its nodes
    const int *word_off;       // [K+1] first word of each patch
    const long long *w_off;    // [K] the patch's decay matrix in w, in 16-byte units; -1: far patch
    const int *perm;           // [N] far patches: patch-local node of each position of the spatial order
    const int *part_off;       // [K+1] first Eq. 1 part of each patch: tiles of 16 rows (near), of 64 (far)
    const int *chunk_off;      // [K+1] first pose part of each patch: chunks of kPoseWords words
    const int2 *block;         // [NU] patch and first node (patch-local) of every kBlockNodes nodes
    const int *blk5_off;       // [K+1] first 128-node block of each patch
    int NW, NP, NC, NU, NB5;   // words, parts, chunks, blocks, 128-node blocks
    int n_near, n_far;         // patches of each kind
    int far_max;               // nodes of the largest far patch
    int near_rows;             // tiles of 16 nodes of the near patches
    long long pairs;           // weights of the near patches
    int near_blocks;           // 128-node blocks of the near patches
};

// What one model gives on the undeformed surface, whatever the env: rebuilt
// by every call that uses it (k_tables).
struct TableDev {
    float *feat;               // [N][64] encoder features of a passive node (U_hat = 0)
    float *dec;                // [N][64] W4[:, :64] feat
    float *max8, *max32;       // [8 NW][64], [2 NW][64] largest features of 8 and of 32 consecutive nodes of a word
    int *scale;                // [8] exponents of the network's weight scales (s1, s2, s4)
    float *w3t, *w4t;          // [64][64] W3 and W4[:, 64:] transposed
    uint4 *w, *wd;             // decay matrices W and, for the adjoint, d W (see matrix_row_tile)
};

// Results of the contact pass the later kernels of a call read.
struct ItemDev {
    unsigned long long *mask;  // [E][NW] active nodes of each word
    float *umax;               // [E][NW] largest |u_hat| component of each word
    int *n_act;                // [E][K] active counts where the caller takes none
    int *live, *live_cnt;      // [K][E] envs in contact on each patch, ascending; [K] how many
    unsigned long long *pool;  // [E K][64] max-pool of the items in contact: feature bits, then ~node (lowest node on ties)
    float *c4;                 // [E K][64] W4[:, 64:] g' + b4 of the items in contact
    int *alist;                // [E][N] far patches: active nodes in spatial order (patch-local)
    float4 *abox;              // [E][NB][2] boxes of 32 consecutive entries of alist
    int *plist;                // the same of the passive nodes (adjoint)
    float4 *pbox;
    const int *box_off;        // [K] first box of each patch
    int NB;                    // boxes per env
};

struct ModelDev {
    int mode;
    const float *alpha;    // [K]
    const float *phi;      // [17411] or null in decay-only mode
};

// Envs per chunk of the passive network adjoint, by the envs of the call and the
// surface's 128-node blocks.  A chunk's sums are written and read once, so long
// chunks move less, as long as there is a unit for every CU: 4096 hands, the
// pass and the one that reads its sums 315 us at 32, 302 at 48; 301 hands of 16
// patches 94 us at 32, 65 at 16.  Blocks alone fill the chip on large surfaces,
// and on the smallest ones the chunks have to.
inline int env_chunk(int E, int blocks) {
    if (E >= 1024 && blocks >= 32) return 48;
    return E >= 4096 ? 32 : E >= 256 || blocks >= 512 ? 16 : 8;
}

// Adjoint scratch (plan flag ETAC_PLAN_BACKWARD).
struct BwdScratch {
    int8_t *cobj_st;       // [E][N]    contact winners (step adjoint)
    float *uhat_st;        // [3][E][N] u_hat of active nodes (step adjoint)
    float *gh;             // [3][E][N] dL/du_hat of active nodes (step adjoint)
    double *alpha_part;    // [E][NP]   dL/dalpha of every part of Eq. 1
    float *s4_part;        // [E][2 NW][64] sum of dL/dpre4 over the passive nodes of a half word
    double *s4_node;       // [chunks][N][64] sum of dL/dpre4 over a chunk's envs, per node
    double *w5_part;       // [chunks][NB5][256] dW5 (192), db5 (3) of 128 nodes and a chunk
    float *ivec;           // [E K][4][64] s4, g', dpre3, g per item
    uint32_t *record;      // [E K][kSavedWords] the adjoint's own pooling record
    double *route;         // [workgroups][kRouteWords] parameter gradients of the max-pool's routes
    float *node_rec;       // [NU][kNodeRecWords] parameter gradients of a block of nodes
    double *alpha_seg;     // [K][kAlphaSegs]
    double *seg;           // [kPhiSegs][kRedCols] segment sums of the parameter reduction
    float *pose_part;      // [E][NC][O][12] pose-gradient parts
    int chunks;            // chunks s4_node and w5_part hold, of any batch the plan takes
};

// Event pairs bracketing kernel launches (etac_plan_set_timing).
struct Timers {
    bool on;
    hipEvent_t ev[ETAC_TIMER_COUNT][ETAC_TIMER_SLOTS][2];
    int n[ETAC_TIMER_COUNT];
};

struct Plan {
    int device;
    int cu_count;
    int wg_per_cu;
    int grid;              // cu_count x wg_per_cu
    int batch, bwd_batch, decay_wg_per_cu, net_batch;   // kept and reported; the kernels choose their own shape
    int n_envs, max_obj, K, N, n_max;
    uint32_t flags;
    MeshDev mesh;
    TileDev tile;
    TableDev tab;
    ItemDev itm;
    unsigned *counter;     // [4] regressor's work queue (self-resetting)
    BwdScratch bwd;
    bool has_bwd;
    void *mem;             // the plan's device block
    int64_t scratch_bytes;
    Timers *timers;        // null until timing is first turned on
    HandDev *hand;         // null until etac_plan_set_hand (host copy of the device view)
    void *hand_mem;        // the hand's device block (one allocation)
    float *reg_rest;       // [K][8] regressor outputs of the patches at U = 0
    int reg_unit;          // nodes of a regressor unit
    float *reg_pooled;     // [units][256] regressor: weighted sums of a unit of an item
    float2 *reg_ml;        // [units] their largest scores and sums of weights
    int *reg_live;         // [K][E] envs in contact of the call's n_active
    int *reg_cnt;          // [K]
};

// Workgroups of a launch whose grid grows with the batch: a launch holds fewer
// than 2^32 threads, so larger grids go in slices of this many.
constexpr long long kMostGroups = 1 << 23;
template <typename F>
inline void launch_slices(long long groups, F launch) {
    for (long long first = 0; first < groups; first += kMostGroups)
        launch(first, dim3((unsigned)(groups - first < kMostGroups ? groups - first : kMostGroups)));
}

// Open a timed span of timer k on stream st; returns the slot, or -1 when
// timing is off or the stream is being captured.
inline int timer_begin(const Plan &p, int k, hipStream_t st) {
    Timers *t = p.timers;
    if (!t || !t->on) return -1;
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &cs) != hipSuccess || cs != hipStreamCaptureStatusNone) return -1;
    const int slot = t->n[k] % ETAC_TIMER_SLOTS;
    return hipEventRecord(t->ev[k][slot][0], st) == hipSuccess ? slot : -1;
}

inline void timer_end(const Plan &p, int k, int slot, hipStream_t st) {
    if (slot < 0) return;
    if (hipEventRecord(p.timers->ev[k][slot][1], st) == hipSuccess) p.timers->n[k]++;
}

// Launchers (return hipError_t of the launch).
// Real-sensor regressor: taxels [E][K][8] from u [3][E][N] (n_envs = E).
hipError_t launch_regress(const Plan &p, const float *reg, int n_envs, const float *u, const int32_t *n_active,
                          float *taxels, hipStream_t st);
hipError_t launch_contact(const Plan &p, const SceneDev &s, int8_t *cobj, float *uhat, int32_t *n_active,
                          hipStream_t st);
hipError_t launch_contact_rows(const Plan &p, const SceneDev &s, int8_t *cobj, float *uhat, int32_t *n_active,
                               int32_t *n_touch, hipStream_t st);
hipError_t launch_step(const Plan &p, const SceneDev *s, const ModelDev &m, int n_envs,
                       const int8_t *cobj_in, const float *uhat_in, float *u, int8_t *cobj_out,
                       int32_t *n_active, uint32_t *saved, hipStream_t st, int32_t *n_touch = nullptr);
// hand: with `links`, pose partials are relative-pose gradients of the hand's
// candidate rows, chained to object and link poses (grad_link_rot/trans).
hipError_t launch_backward(const Plan &p, const SceneDev *s, const ModelDev &m, int n_envs,
                           const int8_t *cobj_in, const float *uhat_in, const float *grad_u,
                           const uint32_t *saved, float *grad_uhat, float *grad_rot, float *grad_trans,
                           float *grad_alpha, float *grad_phi, hipStream_t st, const SceneDev *world = nullptr,
                           const LinksDev *links = nullptr, float *grad_link_rot = nullptr,
                           float *grad_link_trans = nullptr);
// hand pre-pass: fills the candidate rows of every (env, patch) item from the
// world scene and the link poses; returns the row view in *rows.
hipError_t launch_hand_scene(const Plan &p, const SceneDev &world, const LinksDev &links, SceneDev *rows,
                             hipStream_t st);
hipError_t launch_hand_reward(const Plan &p, int n_envs, const int32_t *n_touch, float omega_a, int32_t *n_a,
                              uint32_t *link_mask, float *r_contact, hipStream_t st);
hipError_t launch_pose_hand(const Plan &p, const SceneDev &world, const LinksDev &links, float *grad_rot,
                            float *grad_trans, float *grad_link_rot, float *grad_link_trans, hipStream_t st);

hipError_t launch_contact_backward(const Plan &p, const SceneDev &s, const float *grad_uhat,
                                   float *grad_rot, float *grad_trans, hipStream_t st);

// Triangle meshes of rigid objects on the device (one etac_meshset).  The
// triangles of each mesh are stored in cluster order (clusters of at most 64
// spatially close triangles); `orig` keeps each triangle's index within its
// mesh as given, which breaks distance ties.
struct MeshSetDev {
    const int4 *mesh;        // [M] first triangle, end triangle, first cluster, end cluster
    const float *radius;     // [M] ball about the object origin holding the mesh (rounded up)
    const float *corner;     // [9][T] a.x a.y a.z b.x b.y b.z c.x c.y c.z per triangle
    const int *orig;         // [T] index of the triangle within its mesh, as given
    const double *pn;        // [T][7][3] pseudo-normals: face, edges ab bc ca, vertices a b c
    const double *box;       // [C][16] cluster bounding box: centre, three unit axes, half extents (with margin)
    // occupancy grid per mesh over its bounding box: bit (i, j, k) is clear
    // when every point of that cell is certainly outside the mesh
    const float4 *grid_lo;   // [M] box corner (object frame), 1 / cell size
    const int4 *grid_dim;    // [M] cells along x, y, z; first bit in grid_bits
    const unsigned *grid_bits;
    int M, T, C;
};

hipError_t launch_contact_mesh(const Plan &p, const MeshSetDev &ms, const SceneDev &s, int8_t *cobj, float *uhat,
                               int32_t *n_active, int32_t *hit, hipStream_t st);
hipError_t launch_contact_mesh_backward(const Plan &p, const MeshSetDev &ms, const SceneDev &s,
                                        const float *grad_uhat, const int8_t *cobj, const int32_t *hit,
                                        float *grad_rot, float *grad_trans, hipStream_t st);

}  // namespace etac

struct etac_meshset {
    int device;
    etac::MeshSetDev d;
    void *allocs[16];
    int n_allocs;
};
