// Maximin reconstruction by basins (basin.hip).
#pragma once
#include "ibip_internal.h"

namespace ibip {

// Capacities of a voxel: from a step image (0 on solid, infinity on uninvaded
// pore, the step on invaded voxels), or given.
struct CapSeq {
    const int32_t* seq;
    __device__ uint32_t operator()(int64_t v) const {
        int32_t s = seq[v];
        return s < 0 ? 0u : (s == 0 ? kInf32 : (uint32_t)s);
    }
};
struct CapU32 {
    const uint32_t* cap;
    __device__ uint32_t operator()(int64_t v) const { return cap[v]; }
};

constexpr int kBasinWg = 256;
constexpr uint32_t kBasinSlots = 64;  // lists of basins and of edges
constexpr uint32_t kBasinPad = 32;    // words between the lists' lengths (a line of their own)
constexpr int kBasinRounds = 32;      // a round at least halves the components with edges: 2^31 of them at most
constexpr int kBasinHops = 32;

struct BasinCtl {
    uint32_t abort;               // a list was too short (of the basins, of the edges): nothing
    uint32_t abort_edges;         // is reconstructed; two words, each read only after its writers' launch
    uint32_t pad[30];
    uint32_t climb[8];            // a labelling pass left climbs
    uint32_t live[kBasinRounds];  // the round had edges between components
    uint32_t deep[kBasinRounds];  // the round left chains
    uint32_t np[kBasinSlots * kBasinPad];
    uint32_t ne[kBasinSlots * kBasinPad];
};

struct BasinArgs {
    BasinCtl* ctl;   // zero before the launches
    uint64_t* H;     // [pall + 1] per basin (weight << 32 | basin above), itself at a root; O at pall
    uint64_t* best;  // [2][pall + 1] best edge offered (weight << 32 | edge), by the round's parity
    uint64_t* ends;  // [slots * ecap] an edge's basins
    uint32_t* wt;    // [slots * ecap] an edge's weight
    uint32_t* par;   // [n] climb, then label
    int64_t n;
    int X, Y, Z;
    int nty, ntz;    // tiles along y and z
    uint32_t pcap, pall, ecap;
};

// Sizes of the lists for an image; the scratch they take; its layout at `mem`
// (8-byte aligned).
void basin_caps(BasinArgs& a, ibip_dims d);
size_t basin_bytes(const BasinArgs& a);
void basin_carve(BasinArgs& a, void* mem);
// Basins and edges of a capacity image and its seeds w; rounds from..to-1; and,
// if the last of `rounds` rounds had no edge left, w = the reconstruction.
hipError_t launch_basin_graph(const BasinArgs& a, const int32_t* seq, const uint32_t* cap32, bool conn26,
                              const uint32_t* w, hipStream_t s);
hipError_t launch_basin_rounds(const BasinArgs& a, int from, int to, hipStream_t s);
hipError_t launch_basin_finish(const BasinArgs& a, const int32_t* seq, const uint32_t* cap32, uint32_t* w, int rounds,
                               hipStream_t s);

}  // namespace ibip
