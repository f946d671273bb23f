// d2q9.hpp -- launch interface of the D2Q9 step in tiles of one or more steps.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "kernels.hpp"

namespace lbm {

constexpr int kMaxTileSteps = 4;

// LDS entries of a workgroup with `threads` threads and `per` nodes per thread: per field (the
// nodes whose densities the first step takes) and per population (those it collides)
constexpr int d2_fields(int threads, int per) { return threads * per; }
constexpr int d2_pops(int threads, int per) { return threads * per * 13 / 16; }

// Workgroup shape, own nodes of a tile and the most steps per launch. per = 0 with 512 threads, 64 x 8
// nodes and one step: one thread per tile node.
struct D2Shape {
    int threads, per, tx, ty, steps;
};

// One launch: every tile of the grid advanced by nsteps steps.
struct D2Tiles {
    int tx, ty;        // own nodes of a tile
    int ntx, nty;      // tiles
    int nsteps;
    int first;         // 0: the step that pulls from the lattice
    int stream;        // one thread per node: non-temporal stores (d2_stream)
    int chunk;         // consecutive tiles dealt to one XCD at a time
    unsigned inv_chunk, inv_ntx;   // 2^32 / d of these: division by a multiplication
    unsigned inv[kMaxTileSteps];   // 2^20 / width + 1 of the region's width by steps still to come
    size_t lds;        // dynamic LDS bytes
};

D2Tiles d2_tiles(const Geom &g, bool fp64, const D2Shape &sh, int nsteps);

// Whether the kernel with a thread per node writes its lattice with non-temporal stores.
bool d2_stream(const Geom &g, bool fp64);

// whether a tile with its halo fits the workgroup's nodes and LDS
bool d2_fits(bool fp64, const D2Shape &sh);

using D2Launch = void (*)(hipStream_t, const void *A, void *B, const Geom &, const uint32_t *links, const void *params,
                          const D2Tiles &);

// kernel of a workgroup shape; nullptr when there is none
D2Launch d2_launcher(bool fp64, bool masked, const D2Shape &sh);

// the shape for launches of several steps (its `steps` at most), and for launches of one step
D2Shape d2_plan(const Geom &g, bool fp64, bool masked, int cus);
D2Shape d2_plan_one(const Geom &g, const D2Shape &plan);

// the kernel with a thread per tile node for far_arrays, which the tiles do not address
D2Launch d2_far_launcher(bool fp64, bool masked);

}  // namespace lbm
