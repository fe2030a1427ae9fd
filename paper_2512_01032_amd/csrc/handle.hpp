// handle.hpp -- the single-lattice handle behind the opaque lbm_handle of
// include/lbm.h, shared by the sources that implement its entry points.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

#include "../../include/lbm.h"
#include "lattice_host.hpp"
#include "pflbm.hpp"

struct lbm_handle {
    lbm_params p;
    lbm_geometry geo;
    int device = 0;
    hipStream_t stream = nullptr;
    char* base = nullptr;        // device arena
    bool own_arena = false;
    pflbm::LatticeLayout L;
    pflbm::Desc hdesc;           // host copy of the descriptor at creation
    pflbm::Desc* ddesc = nullptr;
    pflbm::Tile* dtiles = nullptr;
    pflbm::Tile* drtiles = nullptr;   // of the read pass
    int ntiles = 0;
    pflbm::GhostRef* dghosts = nullptr;
    int nghosts = 0;
    pflbm::WallRef* dwalls = nullptr;  // near-wall fluid nodes (wall pass)
    int nwalls = 0;
    int64_t step = 0;            // steps queued so far
    // stability flag copied back asynchronously after each lbm_step
    int* h_unstable = nullptr;   // pinned
    hipEvent_t unstable_ev = nullptr;
    bool unstable_pending = false;
    bool unstable = false;
    // per-kernel timing
    bool timing = false;
    std::vector<hipEvent_t> ev_pool;
    size_t ev_used = 0;
    double phi_ms = 0.0, sweep_ms = 0.0;
    int64_t steps_timed = 0;
    // replayed step sequences (captured on a private stream at the first untimed
    // lbm_step, in the fused layout the first long one): GRAPH_CHUNK steps without a
    // diagnostic step by starting parity, and, for separate passes, one step by
    // [parity][diagnostic]
    hipStream_t cap_stream = nullptr;
    bool graphs_ready = false;
    hipGraphExec_t one[2][2] = {{nullptr, nullptr}, {nullptr, nullptr}};
    hipGraphExec_t chunk[2] = {nullptr, nullptr};
};

// steps per replay of a chunk graph (even, so a chunk ends at the parity it
// started from)
constexpr int64_t GRAPH_CHUNK = 16;
// Shortest call in the fused layout that replays graphs.  Its steps are single kernels,
// and launches follow each other without a gap, so a graph changes little (us per step
// plain / replayed: FP64 droplet 32^3 8.05 / 8.15, FP16 g channel 1024 x 32 x 32 37.0 /
// 37.4, FP32 44.5 / 43.5), while the first capture of a process takes 3 ms and later ones
// 0.15: a first call of 20 steps went from 8.6 to 157 us a step.
constexpr int64_t GRAPH_MIN_STEPS = 64;
