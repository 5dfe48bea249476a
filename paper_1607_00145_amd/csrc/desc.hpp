// desc.hpp -- plain-data kernel descriptor shared by the host analyser and
// the device kernels.
//
// The macro-kernel computes a tile of the matrix view C[x][y] of C, where
//   x runs over I_x, the free indices of the "row" operand X, and
//   y runs over I_y, the free indices of the "column" operand Y;
// (X, Y) is (A, B) or, when the operands are exchanged, (B, A).  Each free
// set is linearised in the analyser's order (first index fastest), which is
// how the paper's single m- and n-loops of Listing 4 stand for several
// indices each (Sec. 3, identify_subtensor).  The contracted set is walked as
// a sequence of "K boxes": the first kj indices of I_k in full, a block of
// tj values of index kj, and one point of every later index -- a sub-tensor
// of fixed shape slid along the contracted indices (Sec. 3.2.1, Eq. 5-6).
#pragma once
#include <stdint.h>

#ifndef __HIP__
#define __host__
#define __device__
#endif

namespace gett {

constexpr int kMaxDims = 16;   // per index set (== GETT_MAX_RANK)
// Indices of the three sets together: each is in two of the three tensors
// (3 x 16 / 2), an empty set adds one, a split of one set up to four.
constexpr int kMaxIndices = 30;

// Gather modes of an operand tile (see kernel.hpp).
enum GatherMode : int {
    kGatherRowVec = 0,   // 16-byte vectors along the tile's free index (stride-one there)
    kGatherKVec = 1,     // 16-byte vectors along the contracted index (stride-one there)
    kGatherScalar = 2,   // one element per access
    // Column operand only: 16-byte vectors along the operand's stride-one
    // index when that index is the second of the tile's free indices (after
    // a block of C's stride-one index) or the second of the K box (after a
    // block of the row operand's stride-one index); consecutive elements of a
    // vector are KDesc::yes tile rows or K positions apart.
    kGatherRowVecStrided = 3,
    kGatherKVecStrided = 4
};

// Gather modes the direct-load kernel takes: vectors on both sides, Y's
// possibly strided by a split of the K box (X's then run along its block).
constexpr bool direct_modes(int xmode, int ymode)
{
    return (xmode <= kGatherKVec && ymode <= kGatherKVec) ||
           (xmode == kGatherKVec && ymode == kGatherKVecStrided);
}

// K slices of a tile that carries the direct-load kernel run on it when both
// operands gather in plain vectors.  After a K split they stay on the
// macro-kernel: the direct-load kernel returns to X's cache lines too late in
// the order of the boxes that slices take (fp32, 32 x 62 x 48 x 48 over 80 x 32
// in 4 slices: 381 us against 307).
constexpr bool direct_slices(bool carries, int xmode, int ymode)
{
    return carries && xmode <= kGatherKVec && ymode <= kGatherKVec;
}

// Division of v < 2^31 by a divisor known to the host: q = (v * mag) >> 32 >> sh
// with sh = ceil(log2 n) - 1 and mag = floor(2^(32 + sh) / n) + 1 (Granlund and
// Montgomery, "Division by Invariant Integers using Multiplication"; mag * n
// exceeds 2^(32 + sh) by at most n <= 2^(sh + 1), so the error v * n / 2^(32 +
// sh) / n stays below 1 / n).  n = 1 has no such multiplier below 2^32; it is
// left at mag = 0 (q = 0): an index of extent 1 stands for an empty set, whose
// only position is 0.  On the device it is a multiplication and a shift in
// place of the twenty-odd instructions of a division.
struct Recip {
    uint32_t mag = 0;
    uint32_t sh = 0;
};
inline Recip recip(int64_t n)
{
    Recip r;
    if (n < 2) return r;
    while (((int64_t)2 << r.sh) < n) ++r.sh;
    r.mag = (uint32_t)((((uint64_t)1 << (32 + r.sh)) / (uint64_t)n) + 1);
    return r;
}

// One index of a set: its extent with the reciprocal, and its strides in the
// two tensors that hold it -- the operand and C (free sets), X and Y (the
// contracted set).  Kept together, so that one wide scalar load fetches it.
struct KDim {
    int32_t ext;
    Recip inv;
    int32_t pad;
    int64_t s0, s1;
};

struct KDesc {
    // ---- free sets, linearised ----
    int64_t sizeX;                 // S_{I_x}
    int64_t sizeY;                 // S_{I_y}
    int32_t nx, ny;                // number of (merged) indices in each set
    // ---- contracted set, walked as K boxes ----
    int32_t nk;                    // number of (merged) contracted indices (>= 1)
    int32_t kj;                    // index that is blocked (earlier ones are whole)
    int32_t tj;                    // block length along index kj
    int32_t kbox;                  // elements in one box = prod(earlier extents) * tj
    int32_t nblk;                  // blocks along index kj = ceil(extent of kj / tj)
    Recip nblkInv;
    int32_t linK;                  // contracted positions, walked linearly by the
                                   // element-wise direct-load kernel (0: none)
    int64_t nsteps;                // boxes = nblk * prod(later extents); 0 = empty sum
    // ---- grid ----
    int32_t tilesX, tilesY;        // tiles along x and y
    int32_t group;                 // tiles along x that share a column band (L2 reuse)
    Recip tilesYInv, bandInv, groupInv;   // of tilesY, group * tilesY and group
    int32_t order;                 // 0: banded tile walk, 1: y-fastest walk (C stream order)
    int32_t xcdremap;              // 1: consecutive tiles on one XCD, 0: hardware order
                                   // (-1 in a plan: chosen per call)
    int32_t cvec;                  // 1: C is accessed in 16-byte vectors along y on the 16-byte
                                   // grid, 0: in vectors at any element address where columns
                                   // follow one another, -1: in single elements
    int32_t xscalar_kfast;         // scalar gather of X: 1 = contracted index fastest
    int32_t yscalar_kfast;         // scalar gather of Y: 1 = contracted index fastest
    int32_t yes;                   // strided vector gathers of Y: distance between the
                                   // elements of one vector (extent of the first index)
    int32_t kslices;               // workgroups per tile, each summing an equal share of
                                   // the K boxes (1: one per tile); their partial tiles
                                   // are summed in slice order through the workspace
    int32_t crun;                  // > 0: C's stride-one run along y, stored in C order
                                   // through LDS (E elements; 0: per-lane stores only)
    int32_t stepY;                 // columns from one tile to the next: the tile's NT, or
                                   // the whole runs of crun in it (the last columns idle)
    Recip piecesInv;               // of the 16-byte pieces per run
    int32_t xperm, yperm;          // > 0: element-wise gathers of X (Y) walk the tile rows
                                   // grouped by row mod this extent (0: in order)
    int32_t tile0;                 // first tile of the grid (> 0: a pass over tiles tile0..)
    // ---- stream-K tail (the tail kernel only) ----
    int32_t tailFull;              // tiles computed whole, one workgroup each
    int32_t tailWgs;               // workgroups that share the boxes of the other tiles
    int32_t tailLen;               // boxes per such workgroup
    // ---- the indices, one set after the other (first = fastest in the set's
    //      linear order): a kernel finds them in the first few cache lines of
    //      its arguments, and a launch copies no more than it has to ----
    KDim dim[kMaxIndices];
    __host__ __device__ const KDim *x() const { return dim; }            // s0: X, s1: C
    __host__ __device__ const KDim *y() const { return dim + nx; }       // s0: Y, s1: C
    __host__ __device__ const KDim *k() const { return dim + nx + ny; }  // s0: X, s1: Y
};

}  // namespace gett
