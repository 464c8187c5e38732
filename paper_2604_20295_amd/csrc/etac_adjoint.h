// Launch parameters of the adjoint's kernels.
#pragma once

#include "etac_step.h"

namespace etac {

struct AdjParams {
    StepParams s;                 // contact, tables and lists as in the forward
    BwdScratch b;
    int env_chunk;                // envs per chunk of the passive network adjoint
    int O;                        // objects (candidates) per scene row
    const float *grad_u;          // [3][E][N]
    float *gh;                    // [3][E][N] dL/du_hat (written on active nodes)
    const int8_t *cobj;           // [E][N] winners' slots
    float *pose_part;             // [E][NC][O][12]
};

// The node pass: built on its own, see etac_backward.hip.
hipError_t launch_adj_nodes(const AdjParams &p, int grid, hipStream_t st);

}  // namespace etac
