// Maximin reconstruction by basins (basin.hip).
#pragma once
#include "ibip_internal.h"

namespace ibip {

// A voxel's word, its capacity in it, and whether the voxel has a neighbour at
// dx along x: from a step image (0 on solid, infinity on uninvaded pore, the step
// on invaded voxels), given, or the rank of a key word (images side by side along
// x in a common array, each ending where its neighbour bits say).
struct CapSeq {
    const int32_t* seq;
    static __device__ uint32_t rank(uint32_t w) { return w; }
    static __device__ bool open(uint32_t, int) { return true; }
    __device__ uint32_t operator()(int64_t v) const {
        int32_t s = seq[v];
        return s < 0 ? 0u : (s == 0 ? kInf32 : (uint32_t)s);
    }
};
struct CapU32 {
    const uint32_t* cap;
    static __device__ uint32_t rank(uint32_t w) { return w; }
    static __device__ bool open(uint32_t, int) { return true; }
    __device__ uint32_t operator()(int64_t v) const { return cap[v]; }
};
struct CapKey {
    const uint32_t* key;
    static __device__ uint32_t rank(uint32_t w) { return w & 0x00FFFFFFu; }
    static __device__ bool open(uint32_t w, int dx) { return dx == 0 || (w >> (dx < 0 ? 24 : 25) & 1u); }
    __device__ uint32_t operator()(int64_t v) const { return key[v]; }
};

constexpr int kBasinWg = 256;
constexpr uint32_t kBasinSlots = 64;  // lists of basins and of edges
constexpr uint32_t kBasinPad = 32;    // words between the lists' lengths (a line of their own)
constexpr int kBasinRounds = 32;      // a round at least halves the components with edges: 2^31 of them at most
constexpr int kBasinHops = 32;
constexpr uint32_t kBasinTop = 0x80000000u;   // in par: a label (basin), not a voxel
constexpr uint32_t kBasinNone = 0xffffffffu;  // in par: capacity 0

struct BasinCtl {
    uint32_t abort;               // a list was too short (of the basins, of the edges): nothing
    uint32_t abort_edges;         // is reconstructed; two words, each read only after its writers' launch
    uint32_t pad[30];
    uint32_t climb[8];            // a labelling pass left climbs
    uint32_t live[kBasinRounds];  // the round had edges between components
    uint32_t np[kBasinSlots * kBasinPad];
    uint32_t ne[kBasinSlots * kBasinPad];
};

struct BasinArgs {
    BasinCtl* ctl;   // zero before the launches
    uint64_t* H;     // [pall + 1] per basin (weight << 32 | basin above), itself at a root; O at pall
    uint64_t* best;  // [2][pall + 1] best edge offered (weight << 32 | edge), by the round's parity
    uint64_t* ends;  // [eall] an edge's basins
    uint32_t* wt;    // [eall] an edge's weight
    uint32_t* par;   // [n] climb, then label
    // for the component tree (else null): the edge by which a root was hooked
    // (weight << 32 | other root), and each basin's top voxel
    uint64_t* mst;
    uint32_t* topv;
    int64_t n;
    int X, Y, Z;
    int nty, ntz;    // tiles along y and z
    uint32_t pcap, pall, ecap, eall;  // places of a slot's list and of all: basins, edges
    bool whole;                       // one place for each voxel and four for its edges
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
// The same of the ranks in the key words, without seeds.
hipError_t launch_basin_graph_keys(const BasinArgs& a, const uint32_t* key, hipStream_t s);
hipError_t launch_basin_rounds(const BasinArgs& a, int from, int to, hipStream_t s);
hipError_t launch_basin_finish(const BasinArgs& a, const int32_t* seq, const uint32_t* cap32, uint32_t* w, int rounds,
                               hipStream_t s);

}  // namespace ibip
