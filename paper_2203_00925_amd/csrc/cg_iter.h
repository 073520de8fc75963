// How the fused Jacobi-CG iteration (cg_iter.hip) splits a state's rows and
// vertices into blocks.
#pragma once
#include <cstdint>
#include <vector>

#include "mesh.h"

namespace mifvm {

// A block works on rows of one mesh only, `rows` consecutive ones, and
// writes one partial per dot product.  Every block of the next kernel adds
// all the partials of its mesh itself, so no mesh gets more than 1024 of them
// (1024 doubles are 8 KB, an L2 hit for all but the first block of an XCD):
// meshes of up to 1024 * 256 cells take one row per thread of a 256-thread
// block, larger ones several rows per thread of a 512-thread block.
constexpr int kCgMaxParts = 1024;
constexpr int kCgVertexLanes = 4;         // lanes that share a vertex list

struct CgPlan {
    int32_t threads = 256;
    int32_t rows = 256;                   // rows per block
    int32_t nblk = 0, vblk = 0;           // blocks of rows, blocks of vertices
    // per block its mesh and row (vertex) range, per mesh its first block
    // and block count; filled for several meshes only (one mesh: arithmetic)
    struct Item { int32_t mesh, begin, end, pad; };
    struct Range { int32_t first, count; };
    std::vector<Item> cells, vertices;
    std::vector<Range> parts;
};

CgPlan cg_plan(const Mesh& m);
// whether every vertex lies in one mesh: a vertex that two meshes share has
// no single beta for its value's recurrence
bool cg_meshes_apart(const Mesh& m);

}  // namespace mifvm
