// Device helpers that the batched products share.
#pragma once

#include <hip/hip_runtime.h>

#include "csb_internal.hpp"
#include "csb_kernels.hpp"

namespace csb {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// A value that is the same in every lane, in a scalar register.  Two kernel arguments between which a lane
// chooses (the strides of two sources) go through it: the compiler turns a choice between two arguments
// into a per-lane load of the chosen one, a trip to memory in front of every load that needs it.
// (24 of those per pair of passes in the kernels that take several products; without them, batch 64, us
// per step: two GRU layers of 1024 in 16-row blocks 32.6 -> 25.4, two LSTM layers in 32-row blocks 23.0 -> 20.0.)
__device__ __forceinline__ uint32_t uni_(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// Product of two 24-bit numbers, modulo 2^32.  (__umul24's result is a signed int: the byte offset of an input
// row 2 GiB and more into X must not be extended with its sign.)
__device__ __forceinline__ uint32_t mul24_(uint32_t a, uint32_t b) { return (uint32_t)__umul24(a, b); }

// First record segment of the rank-th row tile.  Where every tile's records fit one segment it is the rank
// itself: one dependent trip to memory less before a launch of a few microseconds has any work.
__device__ __forceinline__ uint32_t first_segment(const DevMat &m, uint32_t rank) { return m.one_seg ? rank : m.tile_seg0[rank]; }

// Element (column j of A, right-hand side n) of the input, from one of two sources; the right-hand
// sides of a column are contiguous.  Byte offsets fit 32 bits and the strides over j fit 24 bits
// (checked on the host).
struct XSrc {
    const float *p0;
    uint32_t n0;          // columns j < n0 come from p0, the rest from p1
    uint32_t sj0;         // stride over j
    const float *p1;
    uint32_t sj1;
};

// Several independent products in one launch (blockIdx.z picks the product): the per-step
// products of different layers of a batched recurrent model, each too small to fill the GPU.
struct SpmmJobs {
    DevMat m[kMaxJobsPerLaunch];
    XSrc X[kMaxJobsPerLaunch];
    float *Y[kMaxJobsPerLaunch];
    int64_t ldy[kMaxJobsPerLaunch];
};

// ---- products from the quad section (csb_spmm_quad.hip) -------------------------------------------------------
constexpr uint32_t kQuadMaxStride = 16383;               // right-hand sides from one column to the next (kQuadNoCol times that, in bytes, fits 32 bits)
struct QuadMat {
    const uint32_t *table;
    const void *recs;
    const uint8_t *vals;
    uint32_t vals_bytes, n_tiles, tile_rows, rows, cols, list_stride;
};
struct QuadJobs {
    QuadMat m[kMaxJobsPerLaunch];
    XSrc X[kMaxJobsPerLaunch];
    float *Y[kMaxJobsPerLaunch];
    int64_t ldy[kMaxJobsPerLaunch];
};
struct QuadShape {
    int columns;            // right-hand sides per workgroup: 32, 64 or 128
    int nw;                 // wavefronts per workgroup
    bool low;               // the section of 16-row tiles, where a matrix has it
    size_t lds;
    unsigned tiles, batch_tiles;
    double us;              // estimate of the launch's time
};
QuadMat quad_mat(const csb_matrix *m, bool low);
// Whether a product (checked by the caller) is for these kernels; its sources as they read them, and whether there are two.
bool quad_source(const SpmmCall &c, XSrc *X, bool *two);
// The same for 16-bit values times 16-bit right-hand sides (one source, `ldx` elements from one column to the next).
bool quad16_source(const csb_matrix *mat, int64_t ldx);
// The launch shape of n products that share a launch.
QuadShape quad_shape(const csb_matrix *const *mats, int n, int32_t batch);
const void *quad_kernel(const QuadShape &sh, bool two, bool multi);
// Such products in panels: rows of a tile, right-hand sides of a workgroup, wavefronts that share a list of passes.
struct PanelShape {
    int rows, columns, share;
    bool low;               // the section of 16-row tiles beside that of 32
    size_t lds;
    unsigned workgroups;
    int32_t batch;          // right-hand sides of the launch: all, or as many as a grid has threads for
};
PanelShape panel_shape(const csb_matrix *m, int32_t batch);
const void *panel16_kernel(const PanelShape &ps, bool half);

// csb_debug_spmm_force's choices
enum { kFormAuto = 0, kFormTiles = 1, kFormQuads = 2 };

}  // namespace csb
