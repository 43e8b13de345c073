// Context object behind the opaque swe_ctx of include/swe.h (internal).
#pragma once

#include <hip/hip_runtime.h>

#include <string>
#include <vector>

#include "swe_internal.h"
#include "swe_kernels.h"

namespace swe {
// Tile plan of one tile size (swe_plan.h): one allocation, arrays inside it
// with strides of hs halo cells and es edges per tile.
struct TilePlan {
    int tile = 0;  // cells per tile; 0: not built
    int hs = 0, es = 0, ntiles = 0;
    void *mem = nullptr;
    void *desc = nullptr, *halo = nullptr, *ent = nullptr, *nrm = nullptr, *wgt = nullptr, *gam = nullptr,
         *dfw = nullptr;
    // DEEP (a two-stage step in one launch): the plain plan's halo
    const void *base = nullptr;
    int base_hs = 0;
};
}  // namespace swe

constexpr size_t kHostClock = 64, kHostBytes = 4096;

struct swe_ctx {
    swe_config cfg{};
    int dev = 0;
    hipStream_t stream = nullptr;
    bool own_stream = true;  // false: borrowed from the caller (swe_config.stream)
    // around the steps of a call: its start, its end without and with a fence,
    // and the end that was recorded last
    hipEvent_t ev0 = nullptr, ev1 = nullptr, ev1_fence = nullptr, last_end = nullptr;
    std::string err;
    bool has_mesh = false, has_state = false, ran = false;
    int n_owned = 0, n_total = 0, n_scen = 1, n_send = 0, n_ghost = 0;
    int send_prefix = 0;  // the send cells are local cells [0, send_prefix)
    size_t tsize = 4;
    // device buffers
    void *nbr = nullptr, *cell = nullptr, *man2 = nullptr, *rad = nullptr, *he_geo = nullptr, *he_dist = nullptr;
    void *he_co = nullptr, *he_lam = nullptr, *he_gam = nullptr;  // tiled kernel's half-edge set
    void *he_dfw = nullptr;     // tiled WAF kernel: centroid distance per half-edge (WAF contexts)
    void *U[2] = {nullptr, nullptr}, *U1 = nullptr, *tmp3 = nullptr, *bed = nullptr;
    float *phi = nullptr;       // learned-limiter output, one per half-edge
    void *mlp = nullptr;        // learned-limiter weights (MlpDev, BF16)
    bool has_mlp = false;
    bool phi_stale = false;  // learned limiter: the next step evaluates phi whatever its index
    unsigned long long *clock = nullptr;  // 4 slots x (1 + ncopy) lines per scenario
    int ncopy = 64;
    swe::ScenParams *scen = nullptr;
    double *ser_t = nullptr, *ser_q = nullptr;
    swe::TilePlan plans[4];  // 64, 128, 256 and 512 cells per tile, built when first needed
    swe::TilePlan deep;      // of 64-cell tiles (tile -1: does not fit)
    int *health = nullptr, *flag = nullptr, *send_idx = nullptr;
    int *pk_off = nullptr, *pk_ent = nullptr;  // send entries per send cell (CSR)
    // page-locked: call number of a refused state, health bits, and from
    // kHostClock bytes on clock words that were asked for
    int *host = nullptr;
    int calls = 1;        // number of the last state set (k_check_state); 0 and 1 are none's
    // host mirrors
    std::vector<swe::ScenParams> h_scen;
    std::vector<std::pair<std::vector<double>, std::vector<double>>> series;  // per scenario
    std::vector<double> h_ser_t, h_ser_q;
    std::vector<int> scen_off;  // first cell of each scenario, n_scen + 1 entries
    // launch shape: by the configuration and the mesh's size, or what
    // swe_autotune chose, until the next mesh.  grid_persist: blocks of a
    // persistent launch (0 by size, -1 one tile per block)
    int grid_persist = 0;
    int wide = -1;  // tiled kernel: a thread per edge (1) or per cell (0), -1 by size
    int ncu = 0;    // compute units of the device
    double computed_inflow_len = 0.0, given_inflow_len = 0.0;
    long long step_count = 0;  // steps since set_state (selects clock slots and buffers)
    int block = 0;  // cells per tile or threads per block; 0: by size
    // graphs: chunks of kGraphSteps and kLongSteps steps starting at a step
    // index that is a multiple of kGraphSteps
    hipGraphExec_t graphs[2] = {nullptr, nullptr};
    double graph_dt = -1.0;
    bool use_graphs = true;
};


namespace swe {
// Learned limiter (swe_mlp.hip): phi of every half-edge of state U into
// out[3 * n_total], on the context stream.
int launch_limiter_phi(swe_ctx *c, const void *U, float *out);
// Clock slots of a freshly set state U[0] (time t, CFL minima); syncs.
int init_clock(swe_ctx *c, double t);
}  // namespace swe

// Device memory of a context: the configured allocator, else hipMalloc.
// Freed only once the context's stream has finished with it.
inline hipError_t dalloc(swe_ctx *c, void **p, size_t bytes)
{
    *p = nullptr;
    if (bytes == 0) return hipSuccess;
    if (!c->cfg.alloc) return hipMalloc(p, bytes);
    *p = c->cfg.alloc(bytes, c->cfg.alloc_user);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
inline void dfree(swe_ctx *c, void *&p)
{
    if (p) {
        if (c->cfg.free) c->cfg.free(p, c->cfg.alloc_user);
        else (void)hipFree(p);
    }
    p = nullptr;
}
