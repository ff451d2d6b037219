// Arguments of the adjoint kernels (internal).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace lenia {

struct BwdArgs {
    const float* A;          // A_t    [C][H][W]
    const float* P;          // P_t    [3NK][H][W]
    const float* U;          // saved potentials [NK][H][W]
    const uint8_t* alpha;    // saved alpha [H][W]
    const float* gA1;        // gA_next [C][H][W]
    const float* gP1;        // gP_next [3NK][H][W] or null (zero)
    float* gA;               // gA_t (written by the cell pass, completed by the gather pass)
    float* gP;               // gP_t
    float* ubar;             // workspace [NK][H][W]
    float* numbar;           // workspace [3NK][H][W] (gene update only)
    float* part;             // workspace [n_tiles][NK][3]
    const float* wt;         // orbit weights [NO][C][8] in the step kernel's orbit order
    const float* bt;         // shell-height coefficients [NO][C][16] (slot j, shell i at
                             // j * 3 + i) in the same orbit order
    const float* shc;        // shell coefficients [C][KPS][8] (15-kernel table)
    const double* bcomb;     // shell-height combinations [NK][3][3] (15-kernel table)
    const int* n_shells;     // [NK]
    int H, W, tiles_x, n_tiles;
    float dt, eps;
    int mode;
};

// The adjoint of a gene-updating step of the 15-kernel table in quads
// (lenia_bwd_quad.hip) on worlds that quad_fits(R, 4, 64, H, W); part: at least
// 45 floats per 4 x 64 tile.
hipError_t launch_bwd_quad(int R, const BwdArgs& a, float* gbeta, hipStream_t s);

}  // namespace lenia
