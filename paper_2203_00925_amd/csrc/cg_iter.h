// How the fused Jacobi-CG iteration (cg_iter.hip) splits a state's rows and
// vertices into blocks.
#pragma once
#include <cstdint>
#include <vector>

#include "mesh.h"

namespace mifvm {

// A block works on rows of one mesh only and writes one partial per dot
// product; every block of the next kernel adds all the partials of its mesh
// itself.  The vector kernels take about 1024 blocks for the whole state (four
// a CU, so that the CUs stay even: 844 blocks made a product of 1.3M rows 18%
// slower than 5,063) and no more for any mesh, several rows a thread where 256
// each do not reach (cg_plan).
// The product's gathers want many short blocks instead: one row a thread up
// to 8192 blocks (their partials, 64 KB, come from L2 for all but the first
// block of an XCD).
constexpr int kCgMaxBlocks = 1024, kCgMaxProductBlocks = 8192;
constexpr int kCgVertexLanes = 4;         // lanes that share a vertex list

struct CgPlan {
    int32_t threads = 256, rows = 256;    // vector kernels: threads and rows of a block
    int32_t prows = 256;                  // product: rows of a 256-thread block
    int32_t nblk = 0, pblk = 0, vblk = 0; // blocks of rows, of product rows, of vertices
    // per block its mesh and row (vertex) range, per mesh its first block
    // and block count; filled for several meshes only (one mesh: arithmetic)
    struct Item { int32_t mesh, begin, end, lead; };
    struct Range { int32_t first, count, pfirst, pcount; };
    std::vector<Item> cells, product, vertices;
    std::vector<Range> parts;
};

CgPlan cg_plan(const Mesh& m);
// whether every vertex lies in one mesh: a vertex that two meshes share has
// no single beta for its value's recurrence
bool cg_meshes_apart(const Mesh& m);

}  // namespace mifvm
