// Internal declarations shared by the host toolkit and the device runtime of
// libswe.so.  Not part of the public ABI (include/swe.h).
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/swe.h"

// A sub-domain as the host toolkit builds it (swe_subdomain_view gives the
// arrays): local numbering, ghost layers, neighbour table, peers and lists.
struct swe_subdomain {
    int32_t n_owned = 0, n_total = 0, n_peers = 0, n_send = 0;
    std::vector<int32_t> l2g, layer, owner, nbr, peers, recv_off, send_off, send_idx;
};

namespace swe {

// Packed per-cell word (4th int of the neighbour quad):
//   bits 0..5   local edge index, in the neighbour, of the shared edge (2 bits per edge)
//   bits 6..8   edge m is oriented with this cell as the L side (smaller global id)
//   bit  9      owned cell (counts in the CFL reduction)
//   bits 16..31 scenario index (batched ensembles; 0 otherwise)
constexpr int kOwnedBit = 9;
constexpr int kScenShift = 16;
constexpr int kMaxScenarios = 1 << 15;

// Geometry of one mesh prepared on the host in double precision.
struct HostGeometry {
    std::vector<double> cell;    // [4*n]  inv_area, inradius, manning^2, 0
    std::vector<double> he_geo;  // [12*n] per half-edge: nx, ny, L, d_mid
    std::vector<double> he_dist; // [12*n] per half-edge: 1/d_up, 1/d_fwd, 1/d_central, d_fwd
    std::vector<int32_t> nbr4;   // [4*n]  nbr0, nbr1, nbr2, packed word
    double inflow_length = 0.0;  // sum of SWE_BC_INFLOW edge lengths over owned cells
};

// Validates the mesh and fills g.  Returns SWE_OK or SWE_ERR_MESH with msg.
int prepare_geometry(const swe_mesh &m, int scenario, HostGeometry &g, std::string &msg);

// Steps of the next piece of a run: of the short graph, of the long one, or
// one.  left: steps still to take; asked: steps of the whole call, each of dt
// (0: CFL); has_long: a long graph exists, of steps of long_dt.  The long graph
// is built for a call that replays it at least twice.
constexpr int kGraphSteps = 6;  // lcm of the clock-slot (3) and buffer (2) periods
constexpr int kLongSteps = 24;
inline int steps_next(long long step_count, int left, int asked, double dt, bool has_long, double long_dt)
{
    if (step_count % kGraphSteps != 0 || left < kGraphSteps) return 1;
    if (left >= kLongSteps && ((has_long && long_dt == dt) || asked / 2 >= kLongSteps)) return kLongSteps;
    return kGraphSteps;
}

}  // namespace swe
