// resident.hpp -- the on-chip launch of the per-cycle engine (kernels_resident.hip):
// its launch shape and the kernel's argument.
#pragma once

#include "spkmc_device.hpp"

namespace spkmc {

// Lines per workgroup where the lattice needs more than one workgroup.
constexpr uint32_t kResidentLines = 32;

struct ResidentShape {
    bool ok;         // the lattice fits on chip
    int G, D;        // workgroups, domains per workgroup
    int gs, block;   // lanes per frequency line, threads per workgroup
    size_t lds;      // bytes of LDS per workgroup
    uint64_t min_cycles;  // shorter runs take the per-cycle kernels
};

struct ResidentArgs {
    Geom g;
    uint64_t *rec;   // 2 x lines: the event of each line, cycle + 1 in the upper half
    uint64_t *slot;  // 2 x G, `apart` words apart: R_max of each workgroup, generation bit 63
    uint64_t *part;  // 4 x G: counters of a cycle of each workgroup, generation bit 63
    uint64_t n0, ncycles;
    uint32_t obs_every, G, D;
    uint32_t ow, W;  // words (of four sites) per octant, and per lane of a line's group
    uint32_t hinv;   // ceil(2^32 / h)
    uint32_t apart;
};

bool resident_configure(const Geom &g, ResidentShape &out);
hipError_t launch_resident(const Geom &g, const ResidentShape &shape, uint64_t n0, uint64_t ncycles,
                           uint32_t obs_every, bool prep, hipStream_t stream);

}  // namespace spkmc
