// The invasion by levels of the component tree (tree.hip): data layout shared
// by the single-image path, the batch and the server.
#pragma once

#include "basin.h"

namespace ibip {

// Key words: bits 0..23 hold the rank of dt2 among the distinct pore values
// (0 on solid); bit 24 + d is set when the face neighbour in direction d
// (0 -x, 1 +x, 2 -y, 3 +y, 4 -z, 5 +z) lies inside the image; bit 31 marks
// a voxel claimed as a candidate. A claim thus returns, with the rank, what a
// later step needs to claim the voxel's own neighbours without dividing its
// index into coordinates.
constexpr uint32_t kClaim = 0x80000000u;
constexpr uint32_t kRankMask = 0x00FFFFFFu;
constexpr int kNbShift = 24;

// in-image neighbour bits of the voxel at (x, y, z)
__device__ inline uint32_t nb_bits(uint32_t x, uint32_t y, uint32_t z, int X, int Y, int Z) {
    return (x > 0 ? 1u : 0u) | (x + 1 < (uint32_t)X ? 2u : 0u) | (y > 0 ? 4u : 0u) |
           (y + 1 < (uint32_t)Y ? 8u : 0u) | (z > 0 ? 16u : 0u) | (z + 1 < (uint32_t)Z ? 32u : 0u);
}

// Counts of the voxels that a level's rounds over the whole GPU left: round r's in
// slot r % kTreeSlots (a round reads the one before it and clears the one after).
constexpr uint32_t kTreeSlots = 8;
// A level that leaves more voxels than this after its rounds over the whole GPU gets
// more of them, since one workgroup goes through what is left. How many rounds a
// level takes is known only as they go (a plateau, as between parallel plates, takes
// one per voxel of its length), so the launches that follow stop short and the host
// queues on (TreeStop). 512^3 blurred noise leaves at most 24 k in any level and
// never comes back. ms, at 2^17, 2^16, 2^15 and 2^14: 256^3 noise of sigma 2 27.8, 20.9,
// 16.7, 15.0; sigma 1 19.9, 16.2, 15.9, 16.0; plane 500^2 of sigma 1 15.5, 15.5, 4.3,
// 4.3; 256^3 noise of single voxels 46 with any of them, 5,309 without.
constexpr uint32_t kTreeStall = 1u << 15;
constexpr uint32_t kTreeMore = 4096;  // rounds queued at a time, at most
// Why the launches after a tree's kernel do nothing.
enum TreeStop : uint32_t {
    TREE_RUN = 0,
    TREE_GIVE_UP = 1,  // a capacity was exceeded: the step loop runs instead
    TREE_STALL = 2,    // level stall_t wants more rounds: launch_tree_more
};

// Counters of one tree, zeroed before its first kernel.
struct TreeCtl {
    uint32_t nmerge;  // merged peaks (their ids are 0..nmerge-1)
    uint32_t nroot;   // peaks never merged (ids nmerge..nmerge+nroot-1)
    uint32_t nev;     // events, the root event 0 included
    uint32_t nblk;    // blocks of events
    uint32_t ucnt[kTreeSlots];  // voxels that the rounds of the current level left
    uint32_t xcnt[2]; // candidates claimed at the current level; the two in turn
    uint32_t abort;   // TreeStop
    uint32_t stall_t, stall_r;  // the level that wants more rounds, and its rounds so far
    uint32_t pad;
    uint32_t popped[kCountSlots];  // centres, by block
};
static_assert(sizeof(TreeCtl) % 8 == 0, "the images' entries follow the control words");

// One image of a tree. A batch's images share one tree: they lie one after
// another along x in a common array of (sum of X) x Y x Z voxels (Y and Z those
// of the largest, the rest solid), take their ranks from one table, and each
// is entered as a thread of its own, so they are searched level by level
// together and numbered apart.
struct TreeJob {
    uint32_t vox;        // first voxel in the common array
    uint32_t m;          // first entry in M
    uint32_t max_steps;  // 0: no limit
    uint32_t K;          // out: steps
};

struct TreeArgs {
    TreeCtl* ctl;
    TreeJob* jobs;       // njobs; event j < njobs is the root of image j
    const uint32_t* key;
    const uint32_t* list;  // pore voxels by rank: rank r at off[r] .. off[r + 1]
    const uint32_t* off;
    uint32_t* uf;          // N: the voxels' basins
    uint32_t* top;         // N: the peak that labels a voxel's component at its own level
    uint32_t* idx;         // N: a voxel's place in the list (kTreeNone on solid), the step in the end
    // per place of the list
    uint4* rec;            // two each: the neighbours, the top, the voxel (see TreeRec)
    uint32_t* dist;        // the round within the level, then the event; kTreeClaimed before
    uint32_t* gu;          // the thread of the voxel's component at its level
    // per peak (pcap entries)
    uint2* cpm;            // (merge level, parent peak); level 0: never merged
    uint32_t *plo, *mark, *grp, *er, *head, *lcnt, *E;
    // per event (ecap entries; an event is also the thread that it starts):
    // (level, round) of its last event, first event of its current block, last
    // block; per block of events: thread, first event, events, level, the
    // thread's block before it
    uint32_t *gm, *gbase, *lastb, *bg, *bbase, *bcnt, *blev, *bprev;
    uint2 *rank0, *rank1;  // 2 ecap each: list ranking of the events' tour (next, steps); over rec, which
                           // phase 3 does not read
    uint32_t* blkoff;      // R + 2: first block of each level
    char* basin;           // the basins' scratch (phase 1, over what the others need later)
    // lists of one level: places that a round left (two in turn), places
    // popped, and candidates in components entered (three words each)
    uint32_t *U, *U2, *F, *X;
    uint32_t* nodes;       // next pointers, six per waiting voxel
    uint32_t* M;           // rank of each step (out)
    uint32_t pcap, ecap, lcap, xcap, ncap;
    uint32_t R;
    uint32_t kb;           // bits of a round in the (level, round) codes
    int32_t sx, sy;        // strides along x and y
    uint32_t n, n_pore, njobs;
};
constexpr uint32_t kTreeNone = 0xFFFFFFFFu;
constexpr uint32_t kTreeClaimed = 0x80000000u;

constexpr int kPeakWords = 9;   // words per peak: cpm 2, plo, mark, grp, er, head, lcnt, E
constexpr int kEventWords = 8;  // words per event: gm .. bprev
constexpr int kRankWords = 8;   // words per event in the list ranking, over the records (8 a pore voxel)
constexpr int kLevelWords = 3;  // words per voxel of the largest level: U, U2, F
// bytes of the control words and the images' entries, which start the scratch
inline size_t tree_head_bytes(uint32_t njobs) { return align256(sizeof(TreeCtl) + sizeof(TreeJob) * (size_t)njobs); }
// The basins of phase 1 (par in a.uf's memory) in the scratch at `mem`, which takes
// *bytes: the control words, the slices of the tree's edges by level (counts, which
// start as zero, and offsets), the edges, and the basins' own.
struct TreeBasins {
    BasinArgs b;
    uint32_t *cnt, *at;  // R + 2 each
    uint2* edge;         // [pall] the two basins
    uint32_t* pk;        // [pall] a basin's peak (in the memory of b.best)
};
inline TreeBasins tree_basins(const TreeArgs& a, char* mem, size_t* bytes) {
    TreeBasins t{};
    basin_caps(t.b, ibip_dims{(int32_t)(a.n / (uint32_t)a.sx), a.sx / a.sy, a.sy});
    char* m = mem;
    auto take = [&m](size_t k) {
        char* p = m;
        m += (k + 7) / 8 * 8;
        return p;
    };
    const size_t P = (size_t)t.b.pall + 1, E = (size_t)t.b.eall;
    t.b.ctl = (BasinCtl*)take(sizeof(BasinCtl));
    t.cnt = (uint32_t*)take(4 * ((size_t)a.R + 2));
    t.at = (uint32_t*)take(4 * ((size_t)a.R + 2));
    t.edge = (uint2*)take(8 * P);
    t.b.H = (uint64_t*)take(8 * P);
    t.b.best = (uint64_t*)take(16 * P);
    t.pk = (uint32_t*)t.b.best;
    t.b.mst = (uint64_t*)take(8 * P);
    t.b.topv = (uint32_t*)take(4 * P);
    t.b.ends = (uint64_t*)take(8 * E);
    t.b.wt = (uint32_t*)take(4 * E);
    t.b.par = a.uf;
    *bytes = (size_t)(m - mem);
    return t;
}
// words of the records, which the two rank arrays share
inline size_t tree_rec_words(const TreeArgs& a) {
    return std::max(8 * (size_t)a.n_pore, (size_t)kRankWords * a.ecap);
}
// words of scratch for the caps of `a`
inline size_t tree_words(const TreeArgs& a) {
    size_t basins;
    tree_basins(a, nullptr, &basins);
    const size_t later = tree_rec_words(a) + (a.n_pore + 1u) / 2 * 2 + (size_t)a.ecap * kEventWords + (a.R + 2) +
                         (size_t)a.lcap * kLevelWords + (size_t)a.xcap * 3;
    return tree_head_bytes(a.njobs) / 4 + (size_t)a.pcap * kPeakWords + 3 + std::max(later, basins / 4);
}
// lays the control words, peaks, and the rest out in w, and sets a.kb
inline void tree_carve(TreeArgs& a, uint32_t* w) {
    a.ctl = (TreeCtl*)w;
    a.jobs = (TreeJob*)(a.ctl + 1);
    w += tree_head_bytes(a.njobs) / 4;
    a.cpm = (uint2*)w;
    w += 2 * (size_t)a.pcap;
    for (uint32_t** p : {&a.plo, &a.mark, &a.grp, &a.er, &a.head, &a.lcnt, &a.E}) {
        *p = w;
        w += a.pcap;
    }
    w += (4 - (w - (uint32_t*)a.ctl) % 4) % 4;  // (the records are read by 16 bytes)
    a.basin = (char*)w;
    a.rec = (uint4*)w;
    a.rank0 = (uint2*)w;
    a.rank1 = a.rank0 + 2 * (size_t)a.ecap;
    w += tree_rec_words(a);
    a.dist = w;
    w += (a.n_pore + 1u) / 2 * 2;
    for (uint32_t** p : {&a.gm, &a.gbase, &a.lastb, &a.bg, &a.bbase, &a.bcnt, &a.blev, &a.bprev}) {
        *p = w;
        w += a.ecap;
    }
    a.blkoff = w;
    w += a.R + 2;
    for (uint32_t** p : {&a.U, &a.U2, &a.F}) {
        *p = w;
        w += a.lcap;
    }
    a.X = w;
    uint32_t levels = 0;
    while ((a.R >> levels) != 0) levels++;
    a.kb = 32 - levels;
}
// Whether an invasion is expected to take less time by the tree than by the step loop
// (largest: the voxels of the most frequent rank; max_steps 0: no limit), `loops` loops
// of other jobs running in the time of one tree beside it.
bool tree_pays(ibip_dims d, int64_t n_pore, uint32_t R, uint32_t largest, int64_t max_steps, double loops = 1.0);
// The same of an image of which nothing is known yet, taken as 60 % pore with 80 ranks.
constexpr double kGuessPore = 0.6;
constexpr uint32_t kGuessRanks = 80;
bool sizes_by_loop(ibip_dims d, int64_t max_steps);
bool tree_crowded(int64_t n_pore, uint32_t largest);  // one rank holds almost all of it
double loop_ms_expected(ibip_dims d, int64_t n_pore, uint32_t R, int64_t max_steps);
double tree_ms_expected(ibip_dims d, int64_t n_pore, uint32_t R);
// Levels of at most this many voxels are searched in one workgroup.
constexpr uint32_t kTreeSmall = 2048;

inline bool is_plane(ibip_dims d) { return d.X == 1 || d.Y == 1 || d.Z == 1; }
// The scratch's caps for n_pore pore voxels in njobs images (planes: one of them is
// one), the largest level of lcap voxels. More peaks, events or candidates than that
// and the tree gives up. Pore voxels per peak: 130 to 260 in volumes of blurred noise
// or grains, 50 to 100 in such planes, 9 to 25 in noise of single voxels. Pore voxels
// per event (step): 50 to 200 in volumes (16 and more in the smallest), but 9 to 16 in
// planes, 27 in plane noise of single voxels. An image has no more of either than pore
// voxels; the 4,096 are its own.
inline void tree_caps(TreeArgs& a, uint32_t n_pore, uint32_t njobs, uint32_t lcap, bool planes) {
    a.n_pore = n_pore;
    a.njobs = njobs;
    const uint64_t own = 4096 * (uint64_t)njobs;
    a.pcap = (uint32_t)std::min<uint64_t>(n_pore, n_pore / 8 + own);
    a.ecap = (uint32_t)std::min<uint64_t>(n_pore, n_pore / (planes ? 4 : 16) + own) + njobs;
    a.lcap = lcap;
    a.xcap = lcap + 4096;
    a.ncap = n_pore / 6;
}
// key (ranks and neighbour bits from dt2), uf and top of the voxels of an image
// of dims d at voxel `vox` of the common array, whose strides are a's.
hipError_t launch_tree_convert(const TreeArgs& a, uint32_t vox, const uint8_t* image, const uint32_t* dt2,
                               uint32_t* key, const uint32_t* present_scanned, ibip_dims d, uint32_t vlimit,
                               hipStream_t s);
// the pore voxels sorted by rank into a.list (cursors: the slice offsets), a.idx the inverse
hipError_t launch_tree_sort(const TreeArgs& a, uint32_t* cursor, uint32_t* list, hipStream_t s);
// The component tree and what the levels need of it.
hipError_t launch_tree_build(const TreeArgs& a, hipStream_t s);
// the seeds of the image of dims d at voxel `vox`
hipError_t launch_tree_seed(const TreeArgs& a, uint32_t vox, const uint8_t* inlets, ibip_dims d, bool mask,
                            hipStream_t s);
// The levels and the steps' numbers. Leaves the step of each centre in the
// memory of a.idx (0 elsewhere), the images' ranks per step in a.M, their steps
// in a.jobs (or ctl->abort), and seq (the memory of a.top) = INT_MAX on pore,
// -1 on solid.
hipError_t launch_tree_levels(const TreeArgs& a, const uint32_t* off_host, int32_t* seq, hipStream_t s);
// The same from the level on that `c`, the control words read back, says wants more
// rounds (TREE_STALL): four times its rounds so far, so that a level of many rounds
// comes back few times.
hipError_t launch_tree_more(const TreeArgs& a, const TreeCtl& c, const uint32_t* off_host, int32_t* seq, hipStream_t s);
// One job after job_setup_ranks, whose state and slice offsets the host has
// read: the tree's arguments (tree_carve lays its own scratch out, tree_words
// of them), the whole tree on s (head: zeroed control words and the job's
// entry, in pinned memory), and the start of the step loop after a tree that
// gave up.
TreeArgs job_tree_args(const JobBufs& j, const LoopState& hs, const uint32_t* off_host, ibip_dims d, int32_t* seq);
hipError_t job_tree(const JobBufs& j, const TreeArgs& ta, const TreeCtl* head, const uint32_t* off_host,
                    const uint8_t* image, const uint8_t* inlets, ibip_dims d, int32_t* seq, hipStream_t s);
hipError_t job_tree_undo(const JobBufs& j, const TreeArgs& ta, const uint8_t* inlets, ibip_dims d, int32_t* seq,
                         hipStream_t s);
// state (the memory of a.idx), seq and the slices as the step loop starts from
hipError_t launch_tree_undo(const TreeArgs& a, int32_t* seq, uint32_t* head, uint32_t* tail, hipStream_t s);

}  // namespace ibip
