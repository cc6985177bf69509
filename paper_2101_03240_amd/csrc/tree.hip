// The invasion of Section 2.1 (Figure 2(e)-(l)) by levels of the component
// tree of the distance transform, instead of one dependent step after another.
//
// The step loop pops, at every step, all candidates that hold the largest
// rank (rank = place of dt2 among the distinct pore values). Once it has
// entered a component of {rank >= t} it pops nothing below t until that
// component is exhausted. So the whole invasion nests by level, and at one
// level t everything follows from a breadth-first search:
//  * A "thread" is a set of components of {rank >= t} that were entered in
//    the same step, so the loop works on them together. Thread 0 is entered
//    by the seeds.
//  * Within a thread, the loop first exhausts the components of {rank > t}
//    that hold a candidate already ("marked" ones: round 0). Then it pops all
//    candidates of rank t in one step (round 1), exhausts the components of
//    {rank > t} that these entered, pops the next candidates of rank t (round
//    2), and so on. A voxel of rank t is popped in round 1 if it is a
//    candidate already or touches a marked component, otherwise one round
//    after the first of its neighbours: a neighbour of rank t in that
//    neighbour's round, a component of {rank > t} in the round that entered it.
//  * Every (thread, level, round) is one step of the loop: an "event". The
//    components that it enters form a new thread, named by the event; those
//    of round 0 stay in the thread.
// All threads of a level are searched at once, so the dependent chain is the
// sum over levels of the longest search instead of the number of steps: on
// 512^3 blurred noise 2,108 rounds in 304 levels instead of 367,318 steps.
//
// The steps' numbers come afterwards: the events form a tree (an event's
// children are the events of its thread) and the loop visits it in preorder,
// the children by descending level and, in a level, by round.
//
// Phases:
//  1. The component tree: the voxels climb to their basins' tops, and Boruvka
//     rounds on the basins leave the edges that hold their graph together (basin.hip);
//     level by level from the highest rank down, a union-find joins the basins of
//     the level's edges. The root of a component is its highest top, its peak (of
//     equal ones the larger basin's; no result depends on which); a peak whose
//     component joins a higher one at level t keeps (t, the other peak), so the
//     label of a voxel's component at any level is found by walking from the
//     voxel's peak.
//  2. The levels from the lowest rank up: the search above.
//  3. The numbers, and the step of every voxel.
// Levels of few voxels run in one workgroup, several levels per launch, the
// others over the whole GPU until few are left (kTreeStall).
#include <climits>

#include "tree.h"

namespace ibip {

namespace {

constexpr uint32_t kNone = kTreeNone;
constexpr uint32_t kUfPeak = 0x80000000u;  // the link of a peak (its target may be shortened)
constexpr int kWg = 1024;                  // threads of the one-workgroup kernels

// Words that other waves change during the same kernel are read and written
// at device scope (past the CU's cache).
__device__ inline uint32_t ld(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void st(uint32_t* p, uint32_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline uint32_t uniform(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }

__device__ inline uint32_t below_mask_count(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Places for the lanes with `want` in a list whose length is *cnt: one atomic
// per wave. Every lane of the wave must call it.
__device__ inline uint32_t wave_append(uint32_t* cnt, bool want) {
    const uint64_t m = __ballot(want);
    if (!m) return 0;
    const int leader = __ffsll((unsigned long long)m) - 1;
    uint32_t base = 0;
    if ((int)(threadIdx.x & 63) == leader) base = atomicAdd(cnt, (uint32_t)__popcll(m));
    base = __builtin_amdgcn_readlane(base, leader);
    return base + below_mask_count(m);
}

// Places for `mine` entries of each thread in a list whose length is *cnt; the
// thread's first place is returned. kGrid: one atomic per workgroup of kWg
// threads, which all call it (an atomic on a word that the whole GPU appends
// at takes 50 ns and more, one after another); else one per wave, on LDS.
template <bool kGrid>
__device__ inline uint32_t append(uint32_t* cnt, uint32_t mine) {
    const uint32_t lane = threadIdx.x & 63;
    uint32_t incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o, 64);
        if (lane >= (uint32_t)o) incl += t;
    }
    const uint32_t total = __builtin_amdgcn_readlane(incl, 63);
    uint32_t base = 0;
    if (kGrid) {
        __shared__ uint32_t wave[kWg / 64 + 1], first;
        const uint32_t w = threadIdx.x >> 6;
        __syncthreads();  // (the words may still be read for the append before)
        if (lane == 0) wave[w] = total;
        __syncthreads();
        uint32_t before = 0, all = 0;
#pragma unroll
        for (uint32_t q = 0; q < kWg / 64; q++) {
            const uint32_t c = wave[q];
            before += q < w ? c : 0u;
            all += c;
        }
        if (all) {  // (the same in every thread)
            if (threadIdx.x == 0) first = atomicAdd(cnt, all);
            __syncthreads();
            base = first + before;
        }
    } else if (total) {
        if (lane == 0) base = atomicAdd(cnt, total);
        base = uniform(base);
    }
    return base + incl - mine;
}

__device__ inline int32_t nb_off(const TreeArgs& a, int d) {
    const int32_t s = d < 2 ? a.sx : d < 4 ? a.sy : 1;
    return d & 1 ? s : -s;
}

// ---------------------------------------------------------------------------
// Setup
// ---------------------------------------------------------------------------
// c: a voxel of the image's part of the common array (X x CY x CZ, the image
// in its corner, solid around it)
__global__ __launch_bounds__(256) void k_tree_convert(TreeArgs a, uint32_t vox, const uint8_t* __restrict__ img,
                                                      const uint32_t* dt2, uint32_t* key,
                                                      const uint32_t* __restrict__ present_scanned, uint32_t n,
                                                      uint32_t vlimit, int X, int Y, int Z, FastDiv divCZ,
                                                      FastDiv divCY) {
    const uint32_t c = blockIdx.x * 256 + threadIdx.x;
    if (c >= n) return;
    const uint32_t q = fdiv(c, divCZ), x = fdiv(q, divCY), y = q - x * divCY.d, z = c - q * divCZ.d;
    const uint32_t g = vox + c;
    uint32_t k = 0;
    if (y < (uint32_t)Y && z < (uint32_t)Z) {
        const uint32_t v = (x * (uint32_t)Y + y) * (uint32_t)Z + z;
        if (img[v]) {
            const uint32_t d = dt2[v];
            // d >= vlimit only without any solid voxel; such images are rejected
            const uint32_t rk = d < vlimit ? present_scanned[d] + 1 : 0u;
            k = rk == 0 || rk > a.R ? 0u : rk | (nb_bits(x, y, z, X, Y, Z) << kNbShift);
        }
    }
    if (k == 0) a.idx[g] = kNone;
    key[g] = k;
}

// The pore voxels into their ranks' slices. A block counts the ranks of its
// chunk in LDS, reserves its part of each slice with one atomic per rank, and
// places the voxels: one atomic per voxel on a few hot slice cursors would
// queue. A slice holds a chunk's voxels together, so the voxels that a wave
// takes from the list later are near each other.
__global__ __launch_bounds__(256) void k_tree_sort(const uint32_t* __restrict__ key, uint32_t n, uint32_t chunk,
                                                   uint32_t R, uint32_t* cursor, uint32_t* list,
                                                   uint32_t* idx) {
    extern __shared__ uint32_t cnt[];  // R + 1
    for (uint32_t q = threadIdx.x; q <= R; q += 256) cnt[q] = 0;
    __syncthreads();
    const uint32_t b0 = blockIdx.x * chunk, b1 = min(n, b0 + chunk);
    for (uint32_t v = b0 + threadIdx.x; v < b1; v += 256) {
        const uint32_t r = key[v] & kRankMask;
        if (r) atomicAdd(&cnt[r], 1u);
    }
    __syncthreads();
    for (uint32_t q = 1 + threadIdx.x; q <= R; q += 256) {
        const uint32_t c = cnt[q];
        if (c) cnt[q] = atomicAdd(&cursor[q], c);
    }
    __syncthreads();
    for (uint32_t v = b0 + threadIdx.x; v < b1; v += 256) {
        const uint32_t r = key[v] & kRankMask;
        if (r) {
            const uint32_t i = atomicAdd(&cnt[r], 1u);
            list[i] = v;
            idx[v] = i;
        }
    }
}

// ---------------------------------------------------------------------------
// Phase 1: the component tree
// ---------------------------------------------------------------------------
// The union-find over basins, one word each: the rank of the basin's top << 32 |
// the basin that it is linked to. (The voxels' own words would lie a page apart:
// joining by them took 5.7 ms instead of 3.2 at 512^3.) A link without
// kUfPeak leads to a basin of the same rank and is never changed; the links of
// merged peaks are shortened on the way. Links always lead to a higher top (rank,
// then index), so the walk ends. Returns the root's word.
__device__ inline uint64_t ld64(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline uint32_t uf_link(uint64_t w) { return (uint32_t)w & ~kUfPeak; }
__device__ inline uint64_t uf_find(uint64_t* uf, uint32_t x) {
    for (;;) {
        const uint64_t v = ld64(&uf[x]);
        const uint32_t y = uf_link(v);
        if (y == x) return v;
        const uint64_t v2 = ld64(&uf[y]);
        const uint32_t y2 = uf_link(v2);
        if (y2 == y) return v2;
        if ((uint32_t)v & kUfPeak)
            __hip_atomic_store(&uf[x], (v >> 32 << 32) | y2 | kUfPeak, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x = y2;
    }
}

// Joins the components of roots p and q (found a moment ago) at level t: the
// lower root is linked to the higher one; a lost race looks both up again.
__device__ inline void uf_union(const TreeArgs& a, uint64_t* uf, uint64_t p, uint64_t q, uint32_t t) {
    while (p != q) {
        const uint64_t hi = max(p, q), lo = min(p, q);
        const uint32_t l = uf_link(lo), h = uf_link(hi);
        const bool peak = (uint32_t)(lo >> 32) > t;  // a peak's component ends here
        const uint64_t to = (lo >> 32 << 32) | h | (peak ? kUfPeak : 0u);
        if (atomicCAS((unsigned long long*)&uf[l], (unsigned long long)lo, (unsigned long long)to) == lo) {
            if (peak) {
                const uint32_t i = atomicAdd(&a.ctl->nmerge, 1u);
                if (i < a.pcap) {
                    a.plo[i] = l;  // (the basins for now)
                    a.cpm[i] = make_uint2(t, h);
                }
            }
            return;
        }
        p = uf_find(uf, h);
        q = uf_find(uf, l);
    }
}

// The edges between the basins that hold their graph together (a maximum spanning
// forest) into their levels' slices; a workgroup takes a slot's, counts them
// by level in LDS, and then reserves its part of each slice and places them. The
// count also starts the union-find, and says whether the basins came out.
template <bool kPlace>
__global__ __launch_bounds__(kWg) void k_tree_edges(TreeArgs a, TreeBasins t, int rounds) {
    if (t.b.ctl->abort || t.b.ctl->abort_edges || t.b.ctl->live[rounds - 1]) {
        if (threadIdx.x == 0) a.ctl->abort = TREE_GIVE_UP;
        return;
    }
    extern __shared__ uint32_t cnt[];  // R + 1
    for (uint32_t q = threadIdx.x; q <= a.R; q += kWg) cnt[q] = 0;
    __syncthreads();
    const uint32_t np = t.b.ctl->np[blockIdx.x * kBasinPad], p0 = blockIdx.x * t.b.pcap;
    for (uint32_t i = threadIdx.x; i < np; i += kWg) {
        const uint64_t e = t.b.mst[p0 + i];
        if (e) atomicAdd(&cnt[e >> 32], 1u);
        if (!kPlace) {
            t.b.H[p0 + i] = (uint64_t)(a.key[t.b.topv[p0 + i]] & kRankMask) << 32 | (p0 + i);
            t.pk[p0 + i] = kNone;
        }
    }
    __syncthreads();
    for (uint32_t q = threadIdx.x; q <= a.R; q += kWg) {
        const uint32_t c = cnt[q];
        if (c) cnt[q] = atomicAdd(kPlace ? &t.at[q] : &t.cnt[q], c);
    }
    if (!kPlace) return;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < np; i += kWg) {
        const uint64_t e = t.b.mst[p0 + i];
        if (e) t.edge[atomicAdd(&cnt[e >> 32], 1u)] = make_uint2(p0 + i, (uint32_t)e);
    }
}
// at[r] = the first edge of level r, the levels descending; one workgroup.
__global__ __launch_bounds__(kWg) void k_tree_slices(TreeArgs a, TreeBasins t) {
    __shared__ uint32_t part[kWg];
    if (a.ctl->abort) return;
    const uint32_t per = a.R / kWg + 1, b0 = threadIdx.x * per;
    uint32_t sum = 0;
    for (uint32_t q = b0; q < b0 + per && q < a.R; q++) sum += t.cnt[a.R - q];
    part[threadIdx.x] = sum;
    __syncthreads();
    for (uint32_t o = 1; o < (uint32_t)kWg; o <<= 1) {
        const uint32_t before = threadIdx.x >= o ? part[threadIdx.x - o] : 0u;
        __syncthreads();
        part[threadIdx.x] += before;
        __syncthreads();
    }
    uint32_t at = part[threadIdx.x] - sum;
    for (uint32_t q = b0; q < b0 + per && q < a.R; q++) {
        t.at[a.R - q] = at;
        at += t.cnt[a.R - q];
    }
}

// Phase 1's merges: level by level down, each level's edges join their basins'
// components; one workgroup, since a level has few (512^3 blurred noise: 0.4 M in
// 304 levels). (at[r] is the end of level r's slice now, cnt[r] its length.)
__global__ __launch_bounds__(kWg) void k_tree_merge(TreeArgs a, TreeBasins t) {
    if (a.ctl->abort) return;
    __shared__ uint32_t cnt[kWg], end[kWg];  // the slices of the next levels
    for (uint32_t r0 = a.R; r0 >= 1; r0 -= min(r0, (uint32_t)kWg)) {
        if (threadIdx.x < r0) {
            cnt[threadIdx.x] = t.cnt[r0 - threadIdx.x];
            end[threadIdx.x] = t.at[r0 - threadIdx.x];
        }
        __syncthreads();
        for (uint32_t q = 0; q < (uint32_t)kWg && q < r0; q++) {
            const uint32_t c = cnt[q], e1 = end[q];
            if (c == 0) continue;  // (the same in every thread)
            for (uint32_t i = e1 - c + threadIdx.x; i < e1; i += kWg) {
                const uint2 e = t.edge[i];
                uf_union(a, t.b.H, uf_find(t.b.H, e.x), uf_find(t.b.H, e.y), r0 - q);
            }
            __syncthreads();
        }
        __syncthreads();
    }
}

// ids of the peaks: the merged ones in the order of their log, then the others
__device__ inline void peak_init(const TreeArgs& a, uint32_t i) {
    a.mark[i] = 0;
    a.grp[i] = kNone;
    a.er[i] = kNone;
    a.head[i] = kNone;
    a.lcnt[i] = 0;
}
__global__ __launch_bounds__(256) void k_tree_peaks(TreeArgs a, TreeBasins t) {
    const uint32_t tid = blockIdx.x * 256 + threadIdx.x, nth = gridDim.x * 256;
    const uint32_t nm = a.ctl->nmerge;
    if (a.ctl->abort) return;
    if (nm > a.pcap) {
        if (tid == 0) a.ctl->abort = TREE_GIVE_UP;
        return;
    }
    for (uint32_t i = tid; i < nm; i += nth) {
        t.pk[a.plo[i]] = i;
        a.plo[i] = t.b.topv[a.plo[i]];
        peak_init(a, i);
    }
    const uint32_t slot = blockIdx.x % kBasinSlots, part = blockIdx.x / kBasinSlots, parts = gridDim.x / kBasinSlots;
    const uint32_t np = t.b.ctl->np[slot * kBasinPad];
    for (uint32_t q = part * 256; q < np; q += parts * 256) {
        const uint32_t p = slot * t.b.pcap + q + threadIdx.x;
        const bool root = q + threadIdx.x < np && uf_link(t.b.H[p]) == p;
        const uint32_t i = nm + wave_append(&a.ctl->nroot, root);
        if (root) {
            if (i < a.pcap) {
                t.pk[p] = i;
                a.plo[i] = t.b.topv[p];
                a.cpm[i] = make_uint2(0u, i);
                peak_init(a, i);
            } else {
                a.ctl->abort = TREE_GIVE_UP;
            }
        }
    }
}
__global__ __launch_bounds__(256) void k_tree_parents(TreeArgs a, TreeBasins t) {
    if (a.ctl->abort) return;
    const uint32_t nm = a.ctl->nmerge;
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < nm; i += gridDim.x * 256) a.cpm[i].y = t.pk[a.cpm[i].y];
}

// the peak labelling, at level `lvl`, the component that peak `pid` labels higher up
__device__ inline uint32_t label_at(const TreeArgs& a, uint32_t pid, uint32_t lvl) {
    for (;;) {
        const uint2 c = a.cpm[pid];
        if (c.x < lvl) return pid;
        pid = c.y;
    }
}

// top of every voxel: its basin leads to a peak (through basins of the same rank,
// if its top is none), then to the peak that labels that component at the voxel's
// level
__global__ __launch_bounds__(256) void k_tree_tops(TreeArgs a, TreeBasins t) {
    if (a.ctl->abort) return;
    const uint32_t v = blockIdx.x * 256 + threadIdx.x;
    if (v >= a.n) return;
    const uint32_t l = a.uf[v];
    if (l == kBasinNone) return;
    uint32_t p = l & ~kBasinTop, pid;
    while ((pid = t.pk[p]) == kNone) p = uf_link(t.b.H[p]);
    a.top[v] = label_at(a, pid, a.key[v] & kRankMask);
}

// What phase 2 needs of a voxel, looked up once in the voxels' own order (whose
// neighbours are near each other in memory) and kept at its place in the list
// (which a level reads through): neighbour d as kNone (outside, solid or of a
// lower rank), kEq | place (of the same rank) or the peak labelling its
// component one level up (of a higher rank).
constexpr uint32_t kEq = 0x80000000u;
struct Rec {
    uint32_t nb[6], top, v;
};
__device__ inline Rec load_rec(const TreeArgs& a, uint32_t i) {
    const uint4 p = a.rec[2 * (uint64_t)i], q = a.rec[2 * (uint64_t)i + 1];
    return Rec{{p.x, p.y, p.z, p.w, q.x, q.y}, q.z, q.w};
}
__device__ inline bool is_hi(uint32_t c) { return !(c & kEq); }
__device__ inline bool is_eq(uint32_t c) { return (c & kEq) && c != kNone; }
__device__ inline uint32_t eq_place(uint32_t c) { return c & ~kEq; }

__global__ __launch_bounds__(256) void k_tree_records(TreeArgs a) {
    if (a.ctl->abort) return;
    const uint32_t v = blockIdx.x * 256 + threadIdx.x;
    if (v < a.n_pore) a.dist[v] = 0;
    if (v >= a.n) return;
    const uint32_t kv = a.key[v], t = kv & kRankMask;
    if (t == 0) return;
    uint32_t c[6], kw[6], tp[6], open = 0;
#pragma unroll
    for (int d = 0; d < 6; d++) {
        const bool in = (kv >> (kNbShift + d)) & 1u;
        const uint32_t w = in ? v + (uint32_t)nb_off(a, d) : v;
        kw[d] = a.key[w] & kRankMask;
        tp[d] = a.top[w];
        c[d] = a.idx[w];
        kw[d] = in ? kw[d] : 0u;
    }
#pragma unroll
    for (int d = 0; d < 6; d++) {
        c[d] = kw[d] > t ? tp[d] : kw[d] == t ? kEq | c[d] : kNone;
        open |= (kw[d] > t ? 1u : 0u) << d;
    }
    // the walks to the labels side by side
    while (open) {
        uint2 m[6];
#pragma unroll
        for (int d = 0; d < 6; d++) m[d] = (open >> d) & 1u ? a.cpm[c[d]] : make_uint2(0u, 0u);
#pragma unroll
        for (int d = 0; d < 6; d++) {
            if (!((open >> d) & 1u)) continue;
            if (m[d].x <= t) open &= ~(1u << d);
            else c[d] = m[d].y;
        }
    }
    const uint64_t i = a.idx[v];
    a.rec[2 * i] = make_uint4(c[0], c[1], c[2], c[3]);
    a.rec[2 * i + 1] = make_uint4(c[4], c[5], a.top[v], v);
}

// ---------------------------------------------------------------------------
// Phase 2: the levels
// ---------------------------------------------------------------------------
// Candidate w (rank kw), claimed by an event of level t0: every component of
// a level above t0 that holds w is marked with the highest level at which it
// does.
__device__ inline void tree_mark(const TreeArgs& a, uint32_t w, uint32_t kw, uint32_t t0) {
    uint32_t pid = a.top[w], hi = kw;
    for (;;) {
        // marked from here on already? (read first: most candidates find it so)
        if (ld(&a.mark[pid]) >= hi || atomicMax(&a.mark[pid], hi) >= hi) return;
        const uint2 c = a.cpm[pid];
        if (c.x <= t0) return;
        hi = c.x;
        pid = c.y;
    }
}

__device__ inline void tree_candidate(const TreeArgs& a, uint32_t w, uint32_t t0) {
    const uint32_t i = a.idx[w];
    if (ld(&a.dist[i]) & kTreeClaimed) return;
    if (!(atomicOr(&a.dist[i], kTreeClaimed) & kTreeClaimed)) tree_mark(a, w, a.key[w] & kRankMask, t0);
}

// Seeds: Q0 = (inlets U their face neighbours) restricted to pore.
// mask: a solid inlet voxel (rank 0) seeds nothing (the masked reading).
__global__ __launch_bounds__(256) void k_tree_seed(TreeArgs a, uint32_t vox, const uint8_t* __restrict__ inlets,
                                                   uint32_t n, int X, int Y, int Z, FastDiv divZ, FastDiv divY,
                                                   bool mask) {
    if (a.ctl->abort) return;
    const uint32_t v = blockIdx.x * 256 + threadIdx.x;
    if (v >= n || inlets[v] == 0) return;
    const uint32_t t = fdiv(v, divZ), x = fdiv(t, divY), y = t - x * (uint32_t)Y, z = v - t * (uint32_t)Z;
    const uint32_t c = vox + x * (uint32_t)a.sx + y * (uint32_t)a.sy + z;
    if (mask && (a.key[c] & kRankMask) == 0) return;
    // (a solid inlet voxel's key holds no neighbour bits)
    const uint32_t nb = nb_bits(x, y, z, X, Y, Z);
#pragma unroll
    for (int j = 0; j < 7; j++) {
        if (j > 0 && !((nb >> (j - 1)) & 1u)) continue;
        const uint32_t u = j == 0 ? c : c + (uint32_t)nb_off(a, j - 1);
        if ((a.key[u] & kRankMask) != 0) tree_candidate(a, u, 0);
    }
}

// The images' threads: the components of the lowest level that hold a seed.
__global__ __launch_bounds__(256) void k_tree_start(TreeArgs a) {
    if (a.ctl->abort) return;
    const uint32_t tid = blockIdx.x * 256 + threadIdx.x, nth = gridDim.x * 256;
    const uint32_t nm = a.ctl->nmerge, nr = a.ctl->nroot;
    for (uint32_t i = nm + tid; i < nm + nr; i += nth) {
        if (a.mark[i] < 1u) continue;
        uint32_t lo = 0, hi = a.njobs;  // the last image that starts at or before the peak
        while (hi - lo > 1) {
            const uint32_t m = (lo + hi) / 2;
            if (a.jobs[m].vox <= a.plo[i]) lo = m;
            else hi = m;
        }
        a.grp[i] = lo;
    }
    for (uint32_t j = tid; j < a.njobs; j += nth) {
        a.lastb[j] = kNone;
        a.gm[j] = 0u;
    }
    if (tid == 0) {
        a.ctl->nev = a.njobs;
        a.blkoff[1] = 0;
    }
}

// round in which component `pid` (of level t + 1) was entered at level t,
// stored so that a later level's code is smaller (atomicMin)
__device__ inline uint32_t er_code(const TreeArgs& a, uint32_t t, uint32_t r) { return (a.R - t) << a.kb | r; }
// last round of a thread at a level
__device__ inline uint32_t gm_code(const TreeArgs& a, uint32_t t, uint32_t r) { return t << a.kb | r; }

// component pid is entered in round r of level t; true for the one that does it
__device__ inline bool tree_enter(const TreeArgs& a, uint32_t pid, uint32_t t, uint32_t r) {
    if (ld(&a.er[pid]) >> a.kb == a.R - t) return false;
    return atomicMin(&a.er[pid], er_code(a, t, r)) >> a.kb != a.R - t;
}

// Thread g has an event of code (level, round): its code is raised. True for
// the first event of a level, which lists the thread.
__device__ inline bool tree_thread(const TreeArgs& a, uint32_t g, uint32_t code) {
    if (ld(&a.gm[g]) >= code) return false;
    return atomicMax(&a.gm[g], code) >> a.kb != code >> a.kb;
}
__device__ inline void tree_block(const TreeArgs& a, uint32_t b, uint32_t g) {
    if (b < a.ecap) st(&a.bg[b], g);
    else st(&a.ctl->abort, (uint32_t)TREE_GIVE_UP);
}
// The same for the lanes with `want` of a whole wave: neighbouring lanes mostly
// share a thread, and the first of a run raises its code to the run's highest
// (one lane after another would queue on the thread's word). Every lane calls it.
__device__ inline bool wave_thread(const TreeArgs& a, bool want, uint32_t g, uint32_t code) {
    const int lane = threadIdx.x & 63;
    const uint32_t gp = __shfl_up(want ? g : kNone, 1, 64), cp = __shfl_up(want ? code : 0u, 1, 64);
    return want && (lane == 0 || gp != g || cp < code) && tree_thread(a, g, code);
}

// A candidate w in component pid, claimed by the event that enters it in
// thread g: entry x of the level's list.
__device__ inline void tree_edge(const TreeArgs& a, uint32_t x, uint32_t w, uint32_t pid, uint32_t g) {
    if (x >= a.xcap) {
        st(&a.ctl->abort, (uint32_t)TREE_GIVE_UP);
        return;
    }
    st(&a.X[3 * (uint64_t)x], w);
    st(&a.X[3 * (uint64_t)x + 1], pid);
    st(&a.X[3 * (uint64_t)x + 2], g);
}

// One workgroup's state of a level: list lengths, and the search in LDS.
constexpr uint32_t kLds = 6144;      // voxels of a search in LDS
constexpr uint32_t kLdsHash = 8192;  // components that it can tell apart
struct Lists {
    uint32_t u, u2, f, e, x, scan, over;
    uint32_t hkey[kLdsHash];     // component (kNone: free)
    uint16_t her[kLdsHash];      // the round that entered it (0: none yet)
    uint16_t dist[kLds];         // the round that popped a voxel (0: none yet)
    uint16_t nb[6][kLds];        // neighbours: voxel, kLdsComp | component, or kLdsNone
};
constexpr uint16_t kLdsComp = 0x8000u, kLdsNone = 0xFFFFu;

// Round 1 of level t over places lo..hi of the list. kGrid: by the whole GPU in
// workgroups of kWg threads, else by one (tid: the thread's number in the
// launch, nth: threads of the launch).
template <bool kGrid>
__device__ inline void tree_round1(const TreeArgs& a, uint32_t* ucnt, uint32_t* xcnt, uint32_t t, uint32_t lo,
                                   uint32_t hi, uint32_t tid, uint32_t nth) {
    for (uint32_t b = lo + (tid - threadIdx.x); b < hi; b += nth) {
        const uint32_t i = b + threadIdx.x;
        const bool act = i < hi;
        const Rec n = load_rec(a, act ? i : lo);
        const uint32_t dv = ld(&a.dist[act ? i : lo]);
        const uint32_t g = act ? ld(&a.grp[n.top]) : kNone;
        if (act) a.gu[i] = g;
        const bool in = g != kNone;  // (else the component is never entered)
        uint32_t mk = 0, hi_d = 0, mv[6];
#pragma unroll
        for (int d = 0; d < 6; d++) mv[d] = in && is_hi(n.nb[d]) ? ld(&a.mark[n.nb[d]]) : 0u;
#pragma unroll
        for (int d = 0; d < 6; d++) {
            hi_d |= (is_hi(n.nb[d]) ? 1u : 0u) << d;
            mk |= (mv[d] > t ? 1u : 0u) << d;
        }
        const bool set = in && ((dv & kTreeClaimed) || mk);
        const uint32_t fresh = set ? hi_d & ~mk : 0u;  // components that the voxel enters
        if (set) {
            st(&a.dist[i], 1u);
            // marked components stay in the thread
#pragma unroll
            for (int d = 0; d < 6; d++)
                if (((mk >> d) & 1u) && n.nb[d] != n.top && ld(&a.grp[n.nb[d]]) != g) st(&a.grp[n.nb[d]], g);
        }
        const bool won = wave_thread(a, set, g, gm_code(a, t, 1));
        const uint32_t nb = append<false>(&a.ctl->nblk, won ? 1u : 0u);
        if (won) tree_block(a, nb, g);
        uint32_t x = append<kGrid>(xcnt, (uint32_t)__popc(fresh));
        if (fresh) {
#pragma unroll
            for (int d = 0; d < 6; d++) {
                if (!((fresh >> d) & 1u)) continue;
                (void)tree_enter(a, n.nb[d], t, 1);
                tree_edge(a, x++, n.v + (uint32_t)nb_off(a, d), n.nb[d], g);
            }
        }
        const uint32_t q = append<kGrid>(ucnt, in && !set ? 1u : 0u);
        if (in && !set && q < a.lcap) st(&a.U[q], i);
    }
}

// Round r >= 2 of level t over the cnt voxels that the round before left: each
// looks at its neighbours. Those still left go to `out`; in one workgroup (not
// kGrid) they also wait in the lists of the components next to them, and the
// voxels popped and the components entered are listed for the next round.
template <bool kGrid>
__device__ inline void tree_pull(const TreeArgs& a, const uint32_t* in, uint32_t cnt, uint32_t* out, uint32_t* outcnt,
                                 uint32_t* fcnt, uint32_t* ecnt, uint32_t* xcnt, uint32_t t, uint32_t r, uint32_t tid,
                                 uint32_t nth) {
    const uint32_t want = er_code(a, t, r - 1);
    for (uint32_t b = tid - threadIdx.x; b < cnt; b += nth) {
        const uint32_t q0 = b + threadIdx.x;
        const bool act = q0 < cnt;
        const uint32_t i = ld(&in[act ? q0 : 0]);
        const Rec n = load_rec(a, i);
        uint32_t ev[6];
#pragma unroll
        for (int d = 0; d < 6; d++) {
            ev[d] = 0;
            if (act && is_hi(n.nb[d])) ev[d] = ld(&a.er[n.nb[d]]);
            if (act && is_eq(n.nb[d])) ev[d] = ld(&a.dist[eq_place(n.nb[d])]);
        }
        bool set = false;
        uint32_t fresh = 0;
#pragma unroll
        for (int d = 0; d < 6; d++) set |= ev[d] == (is_hi(n.nb[d]) ? want : r - 1);
        set = set && act;
        uint32_t g = 0;
        if (set) {
            st(&a.dist[i], r);
            g = a.gu[i];
            // the components next to it that were not entered before (none of
            // them is marked, or the voxel would have been popped in round 1)
#pragma unroll
            for (int d = 0; d < 6; d++) fresh |= (is_hi(n.nb[d]) && ev[d] != want ? 1u : 0u) << d;
        }
        const bool won = wave_thread(a, set, g, gm_code(a, t, r));
        const uint32_t nb = append<false>(&a.ctl->nblk, won ? 1u : 0u);
        if (won) tree_block(a, nb, g);
        if (!kGrid) {
            const uint32_t f = append<false>(fcnt, set ? 1u : 0u);
            if (set) st(&a.F[f], i);
        }
        uint32_t x = append<kGrid>(xcnt, (uint32_t)__popc(fresh));
        if (fresh) {
#pragma unroll
            for (int d = 0; d < 6; d++) {
                if (!((fresh >> d) & 1u)) continue;
                if (tree_enter(a, n.nb[d], t, r) && !kGrid) st(&a.E[atomicAdd(ecnt, 1u)], n.nb[d]);
                tree_edge(a, x++, n.v + (uint32_t)nb_off(a, d), n.nb[d], g);
            }
        }
        const bool left = act && !set;
        const uint32_t q = append<kGrid>(outcnt, left ? 1u : 0u);
        if (!left) continue;
        st(&out[q], i);
        if (!kGrid && q < a.ncap) {
#pragma unroll
            for (int d = 0; d < 6; d++) {
                bool first = is_hi(n.nb[d]);
#pragma unroll
                for (int e = 0; e < d; e++) first &= n.nb[e] != n.nb[d];
                if (!first) continue;
                const uint32_t k = 6 * q + d;
                st(&a.nodes[k], atomicExch(&a.head[n.nb[d]], k));
                atomicAdd(&a.lcnt[n.nb[d]], 1u);
            }
        }
    }
}

// The search of level t after round r0 over the n <= kLds places `in` that
// round r0 left (kWhole: over the whole level, r0 = 0, places lo..lo + n), with
// the rounds in LDS: every voxel's neighbours are named by 16-bit numbers (a
// voxel of the list, or a component by its slot in a hash table), and a round
// is then a few LDS reads and a barrier instead of a chain of memory round
// trips (1.3 us against 5 us). False, with nothing done, if the voxels touch
// more components than the table takes.
template <bool kWhole>
__device__ inline bool tree_search(const TreeArgs& a, Lists& s, const uint32_t* in, uint32_t lo, uint32_t n,
                                   uint32_t t, uint32_t r0) {
    constexpr uint32_t kItem = 0x40000000u;  // dist of a voxel of the list: its number in it
    const uint32_t tid = threadIdx.x;
    auto place = [&](uint32_t q) { return kWhole ? lo + q : ld(&in[q]); };
    for (uint32_t q = tid; q < kLdsHash; q += kWg) {
        s.hkey[q] = kNone;
        s.her[q] = 0;
    }
    if (tid == 0) s.over = 0;
    if (!kWhole)
        for (uint32_t q = tid; q < n; q += kWg) st(&a.dist[place(q)], kItem | q);
    __syncthreads();
    const uint32_t want = er_code(a, t, r0);
    for (uint32_t q = tid; q < n; q += kWg) {
        const uint32_t i = place(q);
        const Rec b = load_rec(a, i);
        bool act = true, hit = false;
        uint32_t g = 0;
        if (kWhole) {
            g = ld(&a.grp[b.top]);
            a.gu[i] = g;
            act = g != kNone;  // (else the component is never entered)
            hit = act && (ld(&a.dist[i]) & kTreeClaimed);
        }
        uint32_t ev[6];
#pragma unroll
        for (int d = 0; d < 6; d++) {
            ev[d] = 0;
            if (act && is_hi(b.nb[d])) ev[d] = ld(kWhole ? &a.mark[b.nb[d]] : &a.er[b.nb[d]]);
            if (!kWhole && is_eq(b.nb[d])) ev[d] = ld(&a.dist[eq_place(b.nb[d])]);
        }
#pragma unroll
        for (int d = 0; d < 6; d++) {
            uint16_t c = kLdsNone;
            if (act && is_hi(b.nb[d])) {
                if (kWhole ? ev[d] > t : ev[d] == want) {
                    hit = true;
                    // a marked component stays in the thread
                    if (kWhole && b.nb[d] != b.top && ld(&a.grp[b.nb[d]]) != g) st(&a.grp[b.nb[d]], g);
                } else {
                    uint32_t h = (b.nb[d] * 2654435761u) >> 19;  // 13 bits
                    for (uint32_t p = 0;; p++) {
                        if (p == kLdsHash) {
                            s.over = 1;
                            break;
                        }
                        const uint32_t old = atomicCAS(&s.hkey[h], kNone, b.nb[d]);
                        if (old == kNone || old == b.nb[d]) {
                            c = (uint16_t)(kLdsComp | h);
                            break;
                        }
                        h = (h + 1) & (kLdsHash - 1);
                    }
                }
            } else if (act && is_eq(b.nb[d])) {
                if (kWhole) {
                    c = (uint16_t)(eq_place(b.nb[d]) - lo);
                } else {
                    hit |= ev[d] == r0;
                    if (ev[d] & kItem) c = (uint16_t)(ev[d] & ~kItem);
                }
            }
            s.nb[d][q] = c;
        }
        s.dist[q] = hit ? (uint16_t)(r0 + 1) : (uint16_t)0;
    }
    __syncthreads();
    if (uniform(s.over)) {
        if (!kWhole)
            for (uint32_t q = tid; q < n; q += kWg) st(&a.dist[place(q)], 0u);
        __syncthreads();
        return false;
    }
    for (uint32_t q = tid; q < n; q += kWg) {
        if (s.dist[q] == 0) continue;
#pragma unroll
        for (int d = 0; d < 6; d++) {
            const uint16_t c = s.nb[d][q];
            if (c != kLdsNone && (c & kLdsComp)) s.her[c & ~kLdsComp] = (uint16_t)(r0 + 1);
        }
    }
    __syncthreads();
    // one barrier a round: a voxel popped or a component entered in this round
    // holds r, which no test of this round takes. (At most n rounds.)
    for (uint32_t r = r0 + 2;; r++) {
        bool any = false;
        for (uint32_t q = tid; q < n; q += kWg) {
            if (s.dist[q] != 0) continue;
            bool hit = false;
            uint16_t cs[6];
#pragma unroll
            for (int d = 0; d < 6; d++) cs[d] = s.nb[d][q];
#pragma unroll
            for (int d = 0; d < 6; d++) {
                if (cs[d] == kLdsNone) continue;
                const uint16_t v = cs[d] & kLdsComp ? s.her[cs[d] & ~kLdsComp] : s.dist[cs[d]];
                hit |= v != 0 && v < r;
            }
            if (!hit) continue;
            any = true;
            s.dist[q] = (uint16_t)r;
#pragma unroll
            for (int d = 0; d < 6; d++)
                if (cs[d] != kLdsNone && (cs[d] & kLdsComp) && s.her[cs[d] & ~kLdsComp] == 0)
                    s.her[cs[d] & ~kLdsComp] = (uint16_t)r;
        }
        if (!uniform((uint32_t)__syncthreads_or(any))) break;
    }
    for (uint32_t q = tid; q < kLdsHash; q += kWg)
        if (s.hkey[q] != kNone && s.her[q] != 0) st(&a.er[s.hkey[q]], er_code(a, t, s.her[q]));
    for (uint32_t b = tid & ~63u; b < n; b += kWg) {
        const uint32_t q = b + (tid & 63u);
        const uint32_t d0 = q < n ? s.dist[q] : 0u;  // (0: only in components never entered)
        const uint32_t i = d0 ? place(q) : 0u, g = d0 ? a.gu[i] : 0u;
        if (d0) st(&a.dist[i], d0);
        const bool won = wave_thread(a, d0 != 0, g, gm_code(a, t, d0));
        const uint32_t nb = append<false>(&a.ctl->nblk, won ? 1u : 0u);
        if (won) tree_block(a, nb, g);
        if (!d0) continue;
        uint32_t edges = 0;
#pragma unroll
        for (int d = 0; d < 6; d++) {
            const uint16_t c = s.nb[d][q];
            edges |= (c != kLdsNone && (c & kLdsComp) && s.her[c & ~kLdsComp] == d0 ? 1u : 0u) << d;
        }
        if (!edges) continue;
        const uint32_t v = a.rec[2 * (uint64_t)i + 1].w;
#pragma unroll
        for (int d = 0; d < 6; d++)
            if ((edges >> d) & 1u)
                tree_edge(a, atomicAdd(&s.x, 1u), v + (uint32_t)nb_off(a, d), s.hkey[s.nb[d][q] & ~kLdsComp], g);
    }
    __syncthreads();
    return true;
}

// The same without LDS, for more voxels: the rounds of level t from round r on
// in one workgroup, after round r - 1 with its lists (s.u2 voxels wait, in
// `wait`), each in two halves. First the voxels popped in the last round pop
// their neighbours of the same rank, and the components entered in it the
// voxels that wait next to them: from the component's list, or, where a list
// is long, by a scan of all waiting voxels (a list is walked link by link, the
// scan takes all lanes; it costs as much as there are voxels waiting and takes
// at least the long list's voxels off, so the scans of a level stay within a
// constant factor of its voxels). Then the popped voxels enter the components
// next to them. A lane takes one (voxel, direction) pair.
__device__ inline void tree_rounds(const TreeArgs& a, Lists& s, const uint32_t* wait, uint32_t t, uint32_t r) {
    const uint32_t tid = threadIdx.x;
    const uint32_t u2 = uniform(s.u2);
    const uint32_t limit = (1u << a.kb) - 1u;
    const uint32_t longest = max(8u, u2 / 256u);
    uint32_t f0 = 0, e0 = 0;
    auto take = [&](uint32_t i, uint32_t r) {
        if (ld(&a.dist[i]) == 0 && atomicCAS(&a.dist[i], 0u, r) == 0) st(&a.F[atomicAdd(&s.f, 1u)], i);
    };
    for (;; r++) {
        const uint32_t f1 = uniform(s.f), e1 = uniform(s.e);
        if (f0 == f1 && e0 == e1) break;
        if (r >= limit) {
            if (tid == 0) st(&a.ctl->abort, (uint32_t)TREE_GIVE_UP);
            break;
        }
        __syncthreads();  // every wave has read the lengths
        for (uint32_t q = tid; q < 6 * (f1 - f0); q += kWg) {
            const uint32_t p = q / 6u, d = q - 6u * p;
            const uint32_t c = ((const uint32_t*)a.rec)[8 * (uint64_t)ld(&a.F[f0 + p]) + d];
            if (is_eq(c)) take(eq_place(c), r);
        }
        for (uint32_t q = e0 + tid; q < e1; q += kWg) {
            const uint32_t pid = ld(&a.E[q]);
            uint32_t k = ld(&a.head[pid]);
            if (ld(&a.lcnt[pid]) > longest) {
                s.scan = 1;
            } else {
                while (k != kNone) {
                    const uint32_t next = ld(&a.nodes[k]);
                    take(ld(&wait[k / 6u]), r);
                    k = next;
                }
            }
            st(&a.head[pid], kNone);
            st(&a.lcnt[pid], 0u);
        }
        __syncthreads();
        if (uniform(s.scan) || (u2 > a.ncap && e0 != e1)) {
            const uint32_t want = er_code(a, t, r - 1);
            for (uint32_t q = tid; q < u2; q += kWg) {
                const uint32_t i = ld(&wait[q]);
                if (ld(&a.dist[i]) != 0) continue;
                const Rec n = load_rec(a, i);
                bool hit = false;
#pragma unroll
                for (int d = 0; d < 6; d++)
                    if (is_hi(n.nb[d])) hit |= ld(&a.er[n.nb[d]]) == want;
                if (hit) take(i, r);
            }
            __syncthreads();
            if (tid == 0) s.scan = 0;
        }
        const uint32_t f2 = uniform(s.f);
        for (uint32_t q = tid; q < 6 * (f2 - f1); q += kWg) {
            const uint32_t p = q / 6u, d = q - 6u * p;
            const uint32_t i = ld(&a.F[f1 + p]), g = a.gu[i];
            const uint32_t c = ((const uint32_t*)a.rec)[8 * (uint64_t)i + d];
            if (d == 0 && tree_thread(a, g, gm_code(a, t, r))) tree_block(a, atomicAdd(&a.ctl->nblk, 1u), g);
            if (!is_hi(c)) continue;
            const uint32_t er = ld(&a.er[c]);
            // (none of the components next to it is marked, see tree_pull)
            if (er >> a.kb == a.R - t && er != er_code(a, t, r)) continue;
            if (tree_enter(a, c, t, r)) st(&a.E[atomicAdd(&s.e, 1u)], c);
            tree_edge(a, atomicAdd(&s.x, 1u), a.rec[2 * (uint64_t)i + 1].w + (uint32_t)nb_off(a, (int)d), c, g);
        }
        f0 = f1;
        e0 = e1;
        __syncthreads();
    }
    __syncthreads();
}

// The events of level t: one per thread and round, a block per thread.
__device__ inline void tree_events(const TreeArgs& a, uint32_t t) {
    const uint32_t b0 = a.blkoff[t], b1 = min(uniform(ld(&a.ctl->nblk)), a.ecap), rm = (1u << a.kb) - 1u;
    for (uint32_t b = b0 + threadIdx.x; b < b1; b += kWg) {
        const uint32_t g = ld(&a.bg[b]), cnt = ld(&a.gm[g]) & rm;
        const uint32_t base = atomicAdd(&a.ctl->nev, cnt);
        if (base > a.ecap || cnt > a.ecap - base) {
            st(&a.ctl->abort, (uint32_t)TREE_GIVE_UP);
            continue;
        }
        a.bbase[b] = base;
        a.bcnt[b] = cnt;
        a.blev[b] = t;
        a.bprev[b] = ld(&a.lastb[g]);
        st(&a.lastb[g], b);
        st(&a.gbase[g], base);
        for (uint32_t q = 0; q < cnt; q++) {
            st(&a.lastb[base + q], kNone);
            st(&a.gm[base + q], 0u);
        }
    }
}

// The candidates that the events of level t claim in the components that they
// enter, and these components' threads.
__device__ inline void tree_claim(const TreeArgs& a, uint32_t t, uint32_t nx, uint32_t tid, uint32_t nth) {
    const uint32_t rm = (1u << a.kb) - 1u;
    for (uint32_t x = tid; x < nx; x += nth) {
        const uint32_t w = ld(&a.X[3 * (uint64_t)x]), pid = ld(&a.X[3 * (uint64_t)x + 1]),
                       g = ld(&a.X[3 * (uint64_t)x + 2]);
        const uint32_t ev = ld(&a.gbase[g]) + (ld(&a.er[pid]) & rm) - 1;
        if (ld(&a.grp[pid]) != ev) st(&a.grp[pid], ev);
        tree_candidate(a, w, t);
    }
}

// The voxels of a level from rounds to events.
__device__ inline void tree_rounds_to_events(const TreeArgs& a, uint32_t lo, uint32_t hi, uint32_t tid, uint32_t nth) {
    for (uint32_t i = lo + tid; i < hi; i += nth) {
        const uint32_t d = ld(&a.dist[i]);
        if (d) st(&a.dist[i], ld(&a.gbase[a.gu[i]]) + d - 1);
    }
}

// A level of many voxels over the whole GPU: round 1, further rounds, then
// (after the rest of the search and the events, in one workgroup) the
// candidates and the voxels' events.
__global__ __launch_bounds__(kWg) void k_tree_round1(TreeArgs a, uint32_t t, uint32_t side, uint32_t lo, uint32_t hi) {
    if (a.ctl->abort) return;
    tree_round1<true>(a, &a.ctl->ucnt[1], &a.ctl->xcnt[side], t, lo, hi, blockIdx.x * kWg + threadIdx.x,
                      gridDim.x * kWg);
}

__global__ __launch_bounds__(kWg) void k_tree_pull(TreeArgs a, uint32_t t, uint32_t side, uint32_t r) {
    if (a.ctl->abort) return;
    TreeCtl* c = a.ctl;
    if (blockIdx.x == 0 && threadIdx.x == 0) st(&c->ucnt[(r + 1) % kTreeSlots], 0u);
    tree_pull<true>(a, r & 1u ? a.U2 : a.U, c->ucnt[(r - 1) % kTreeSlots], r & 1u ? a.U : a.U2,
                    &c->ucnt[r % kTreeSlots], nullptr, nullptr, &c->xcnt[side], t, r,
                    blockIdx.x * kWg + threadIdx.x, gridDim.x * kWg);
}

__global__ void k_tree_go_on(TreeArgs a) {
    if (a.ctl->abort == TREE_STALL) a.ctl->abort = TREE_RUN;
}

__global__ __launch_bounds__(256) void k_tree_claim(TreeArgs a, uint32_t t, uint32_t side, uint32_t lo, uint32_t hi) {
    if (a.ctl->abort) return;
    const uint32_t tid = blockIdx.x * 256 + threadIdx.x, nth = gridDim.x * 256;
    tree_claim(a, t, a.ctl->xcnt[side], tid, nth);
    tree_rounds_to_events(a, lo, hi, tid, nth);
}

// One workgroup: levels t_lo..t_hi, or (r0 > 0) the rest of the search of
// level t_lo after its first r0 rounds, and its events.
__device__ inline void tree_levels(const TreeArgs& a, Lists& s, uint32_t t_lo, uint32_t t_hi, uint32_t r0,
                                   uint32_t side) {
    const uint32_t tid = threadIdx.x;
    TreeCtl* c = a.ctl;
    for (uint32_t t = t_lo; t <= t_hi; t++) {
        if (uniform(ld(&c->abort))) return;
        if (tid == 0) {
            s.u = r0 ? c->ucnt[r0 % kTreeSlots] : 0u;
            s.x = r0 ? c->xcnt[side] : 0u;
            s.u2 = s.f = s.e = s.scan = 0;
        }
        __syncthreads();
        if (uniform(s.u) > kTreeStall) {
            if (tid == 0) {
                c->stall_t = t;
                c->stall_r = r0;
                // (the codes of rounds to come have to fit)
                st(&c->abort, (uint32_t)(r0 + kTreeMore < (1u << a.kb) - 1u ? TREE_STALL : TREE_GIVE_UP));
            }
            return;
        }
        const uint32_t i0 = a.off[t], i1 = a.off[t + 1];
        uint32_t r = r0;
        bool found = false;
        if (!r0) {
            found = i1 - i0 <= kLds && tree_search<true>(a, s, nullptr, i0, i1 - i0, t, 0);
            if (!found) {
                tree_round1<false>(a, &s.u, &s.x, t, i0, i1, tid, kWg);
                __syncthreads();
                r = 1;
            }
        }
        const uint32_t u = uniform(s.u);
        uint32_t* const in = r & 1u ? a.U : a.U2;
        // (the search in LDS holds rounds in 16 bits, and adds at most kLds of them)
        if (!found && u && !(u <= kLds && r <= 32768u && tree_search<false>(a, s, in, 0, u, t, r))) {
            uint32_t* const out = r & 1u ? a.U2 : a.U;
            tree_pull<false>(a, in, u, out, &s.u2, &s.f, &s.e, &s.x, t, r + 1, tid, kWg);
            __syncthreads();
            tree_rounds(a, s, out, t, r + 2);
        }
        tree_events(a, t);
        __syncthreads();
        if (uniform(ld(&c->abort))) return;
        if (!r0) {
            tree_claim(a, t, uniform(s.x), tid, kWg);
            tree_rounds_to_events(a, i0, i1, tid, kWg);
        }
        if (tid == 0) {
            a.blkoff[t + 1] = ld(&c->nblk);
            if (r0) {
                // (the next such level counts from 0; this one's candidates
                // are claimed by the next launch)
                c->xcnt[side] = s.x;
                c->xcnt[side ^ 1u] = 0;
                for (uint32_t q = 0; q < kTreeSlots; q++) c->ucnt[q] = 0;
            }
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(kWg) void k_tree_levels(TreeArgs a, uint32_t t_lo, uint32_t t_hi, uint32_t r0,
                                                     uint32_t side) {
    __shared__ Lists s;
    tree_levels(a, s, t_lo, t_hi, r0, side);
}

// ---------------------------------------------------------------------------
// Phase 3: the steps' numbers
// ---------------------------------------------------------------------------
// The events' tour: down into an event, through its children (its thread's
// blocks from the last, which is of the highest level, to the first, each
// block by round), up again. The number of an event is the number of "down"s
// before its own; a list ranking by pointer jumping counts those after it, in
// 1 + log2(2 events) passes over all events (levels of parents and children one
// after another took 3.8 ms on 512^3 blurred noise).
// rank[2e]: down of event e, rank[2e + 1]: up; x = the next of the tour
// (itself at the end, the up of the image's root), y = downs from here to
// before x.
__global__ __launch_bounds__(256) void k_tree_tour(TreeArgs a) {
    if (a.ctl->abort) return;
    const uint32_t nb = a.ctl->nblk;
    for (uint32_t b = blockIdx.x * 256 + threadIdx.x; b < nb + a.njobs; b += gridDim.x * 256) {
        // (each image's root event stands in for a block of its own)
        const uint32_t base = b < nb ? a.bbase[b] : b - nb, cnt = b < nb ? a.bcnt[b] : 1u;
        for (uint32_t q = 0; q < cnt; q++) {
            const uint32_t e = base + q, child = a.lastb[e];
            a.rank0[2 * e] = make_uint2(child != kNone ? 2 * a.bbase[child] : 2 * e + 1, 1u);
            uint32_t next = 2 * e + 1;
            if (q + 1 < cnt) next = 2 * (e + 1);
            else if (b < nb) next = a.bprev[b] != kNone ? 2 * a.bbase[a.bprev[b]] : 2 * a.bg[b] + 1;
            a.rank0[2 * e + 1] = make_uint2(next, 0u);
        }
    }
}
__global__ __launch_bounds__(256) void k_tree_jump(TreeArgs a, const uint2* __restrict__ in, uint2* __restrict__ out) {
    if (a.ctl->abort) return;
    const uint32_t n = 2 * a.ctl->nev;
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) {
        const uint2 p = in[i], q = in[p.x];
        out[i] = make_uint2(q.x, p.x == i ? p.y : p.y + q.y);
    }
}
// an event's image and step, from the list ranking
__device__ inline uint32_t event_step(const TreeArgs& a, const uint2* rank, uint32_t e, uint32_t& job) {
    const uint2 r = rank[2 * (uint64_t)e];
    job = r.x >> 1;
    return rank[2 * (uint64_t)job].y - r.y;
}

// the ranks per step
__global__ __launch_bounds__(256) void k_tree_steps(TreeArgs a, const uint2* __restrict__ rank) {
    if (a.ctl->abort) return;
    const uint32_t nb = a.ctl->nblk, tid = blockIdx.x * 256 + threadIdx.x, nth = gridDim.x * 256;
    for (uint32_t j = tid; j < a.njobs; j += nth) {
        const uint32_t K = rank[2 * (uint64_t)j].y - 1, lim = a.jobs[j].max_steps;
        a.jobs[j].K = lim ? min(K, lim) : K;
    }
    for (uint32_t b = tid; b < nb; b += nth) {
        const uint32_t base = a.bbase[b], cnt = a.bcnt[b], t = a.blev[b];
        for (uint32_t q = 0; q < cnt; q++) {
            uint32_t j;
            const uint32_t k = event_step(a, rank, base + q, j), lim = a.jobs[j].max_steps;
            if (lim == 0 || k <= lim) a.M[a.jobs[j].m + k - 1] = t;
        }
    }
}

// idx becomes the steps (0 past the step limit); seq: INT_MAX on pore, -1 on solid
__global__ __launch_bounds__(256) void k_tree_finish(TreeArgs a, const uint2* __restrict__ rank, int32_t* seq) {
    if (a.ctl->abort) return;
    uint32_t centres = 0;
    for (uint32_t v = blockIdx.x * 256 + threadIdx.x; v < a.n; v += gridDim.x * 256) {
        const uint32_t i = a.idx[v];
        // (a candidate's flag is gone once it is popped, as every candidate is;
        // the images' roots, events below njobs, hold no voxel)
        const uint32_t e = i != kNone ? a.dist[i] : 0u;
        uint32_t k = 0;
        if (e) {
            uint32_t j;
            k = event_step(a, rank, e, j);
            const uint32_t lim = a.jobs[j].max_steps;
            if (lim && k > lim) k = 0;
        }
        centres += k ? 1u : 0u;
        a.idx[v] = k;
        seq[v] = i != kNone ? INT_MAX : -1;
    }
    block_add_slots(a.ctl->popped, centres);
}

__global__ __launch_bounds__(256) void k_tree_undo(TreeArgs a, int32_t* seq, uint32_t* head, uint32_t* tail) {
    const uint32_t v = blockIdx.x * 256 + threadIdx.x;
    if (v >= 1 && v <= a.R) head[v] = tail[v] = a.off[v];
    if (v >= a.n) return;
    a.idx[v] = 0;
    seq[v] = (a.key[v] & kRankMask) ? INT_MAX : -1;
}

inline unsigned blocks(uint64_t n, unsigned t = 256) { return (unsigned)((n + t - 1) / t); }

}  // namespace

hipError_t launch_tree_convert(const TreeArgs& a, uint32_t vox, const uint8_t* image, const uint32_t* dt2,
                               uint32_t* key, const uint32_t* present_scanned, ibip_dims d, uint32_t vlimit,
                               hipStream_t s) {
    const uint32_t n = (uint32_t)d.X * (uint32_t)a.sx;
    hipLaunchKernelGGL(k_tree_convert, dim3(blocks(n)), dim3(256), 0, s, a, vox, image, dt2, key, present_scanned, n,
                       vlimit, d.X, d.Y, d.Z, make_fastdiv((uint32_t)a.sy), make_fastdiv((uint32_t)(a.sx / a.sy)));
    return hipGetLastError();
}

hipError_t launch_tree_sort(const TreeArgs& a, uint32_t* cursor, uint32_t* list, hipStream_t s) {
    const uint32_t chunk = a.n > (1u << 24) ? 16384u : a.n > (1u << 21) ? 4096u : 1024u;
    hipLaunchKernelGGL(k_tree_sort, dim3(blocks(a.n, chunk)), dim3(256), sizeof(uint32_t) * (a.R + 1), s, a.key, a.n,
                       chunk, a.R, cursor, list, a.idx);
    return hipGetLastError();
}

hipError_t launch_tree_build(const TreeArgs& a, hipStream_t s) {
    size_t bytes;
    const TreeBasins t = tree_basins(a, a.basin, &bytes);
    // a round at least halves the components with edges, and mostly leaves a
    // tenth; an image of more than 2^16 basins that takes more rounds than this
    // runs the step loop
    int rounds = 1;
    while (rounds < 16 && (a.n_pore >> rounds) != 0) rounds++;
    hipError_t e;
    if ((e = hipMemsetAsync(t.b.ctl, 0, (size_t)((char*)t.at - (char*)t.b.ctl), s)) != hipSuccess) return e;
    if ((e = launch_basin_graph_keys(t.b, a.key, s)) != hipSuccess) return e;
    if ((e = launch_basin_rounds(t.b, 0, rounds, s)) != hipSuccess) return e;
    const size_t lds = sizeof(uint32_t) * ((size_t)a.R + 1);
    hipLaunchKernelGGL(k_tree_edges<false>, dim3(kBasinSlots), dim3(kWg), lds, s, a, t, rounds);
    hipLaunchKernelGGL(k_tree_slices, dim3(1), dim3(kWg), 0, s, a, t);
    hipLaunchKernelGGL(k_tree_edges<true>, dim3(kBasinSlots), dim3(kWg), lds, s, a, t, rounds);
    hipLaunchKernelGGL(k_tree_merge, dim3(1), dim3(kWg), 0, s, a, t);
    const unsigned few = kBasinSlots * std::min(std::max(blocks(a.pcap, 1u << 14), 1u), 16u);
    hipLaunchKernelGGL(k_tree_peaks, dim3(few), dim3(256), 0, s, a, t);
    hipLaunchKernelGGL(k_tree_parents, dim3(few), dim3(256), 0, s, a, t);
    hipLaunchKernelGGL(k_tree_tops, dim3(blocks(a.n)), dim3(256), 0, s, a, t);
    hipLaunchKernelGGL(k_tree_records, dim3(blocks(a.n)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_tree_seed(const TreeArgs& a, uint32_t vox, const uint8_t* inlets, ibip_dims d, bool mask,
                            hipStream_t s) {
    const uint32_t n = (uint32_t)nvox(d);
    hipLaunchKernelGGL(k_tree_seed, dim3(blocks(n)), dim3(256), 0, s, a, vox, inlets, n, d.X, d.Y, d.Z,
                       make_fastdiv((uint32_t)d.Z), make_fastdiv((uint32_t)d.Y), mask);
    return hipGetLastError();
}

// Levels t0.. and phase 3; r > 0: level t0 has had r rounds and gets `more`.
static hipError_t levels_from(const TreeArgs& a, const uint32_t* off, int32_t* seq, uint32_t t0, uint32_t r,
                              uint32_t more, hipStream_t s) {
    auto size = [&](uint32_t t) { return off[t + 1] - off[t]; };
    uint32_t side = 0;
    for (uint32_t t = 1; t < t0; t++) side ^= size(t) > kTreeSmall ? 1u : 0u;
    for (uint32_t t = t0; t <= a.R;) {
        if (size(t) > kTreeSmall) {
            // further rounds over the whole GPU where round 1 may leave many
            const uint32_t n = size(t);
            uint32_t r0 = n > (1u << 19) ? 7u : n > (1u << 17) ? 5u : n > (1u << 15) ? 4u : n > (1u << 13) ? 2u : 1u;
            if (r) r0 = r + more;
            else
                hipLaunchKernelGGL(k_tree_round1, dim3(std::min(blocks(n, kWg), 4096u)), dim3(kWg), 0, s, a, t, side,
                                   off[t], off[t + 1]);
            for (uint32_t q = r ? r + 1 : 2; q <= r0; q++)
                hipLaunchKernelGGL(k_tree_pull, dim3(std::min(blocks(n, 4 * kWg), 512u)), dim3(kWg), 0, s, a, t,
                                   side, q);
            r = 0;
            hipLaunchKernelGGL(k_tree_levels, dim3(1), dim3(kWg), 0, s, a, t, t, r0, side);
            hipLaunchKernelGGL(k_tree_claim, dim3(std::min(blocks(size(t)), 4096u)), dim3(256), 0, s, a, t, side,
                               off[t], off[t + 1]);
            side ^= 1u;
            t++;
        } else {
            uint32_t q = t;
            while (q < a.R && size(q + 1) <= kTreeSmall) q++;
            hipLaunchKernelGGL(k_tree_levels, dim3(1), dim3(kWg), 0, s, a, t, q, 0u, 0u);
            t = q + 1;
        }
    }
    // phase 3
    const unsigned ge = std::min(blocks(a.ecap), 2048u);
    hipLaunchKernelGGL(k_tree_tour, dim3(ge), dim3(256), 0, s, a);
    uint2 *in = a.rank0, *out = a.rank1;
    for (uint64_t span = 1; span < 2 * (uint64_t)a.ecap; span *= 2) {
        hipLaunchKernelGGL(k_tree_jump, dim3(ge), dim3(256), 0, s, a, in, out);
        std::swap(in, out);
    }
    hipLaunchKernelGGL(k_tree_steps, dim3(ge), dim3(256), 0, s, a, in);
    hipLaunchKernelGGL(k_tree_finish, dim3(std::min(blocks(a.n), 8192u)), dim3(256), 0, s, a, in, seq);
    return hipGetLastError();
}

hipError_t launch_tree_levels(const TreeArgs& a, const uint32_t* off, int32_t* seq, hipStream_t s) {
    hipLaunchKernelGGL(k_tree_start, dim3(64), dim3(256), 0, s, a);
    return levels_from(a, off, seq, 1, 0, 0, s);
}

hipError_t launch_tree_more(const TreeArgs& a, const TreeCtl& c, const uint32_t* off, int32_t* seq, hipStream_t s) {
    hipLaunchKernelGGL(k_tree_go_on, dim3(1), dim3(1), 0, s, a);
    return levels_from(a, off, seq, c.stall_t, c.stall_r, std::min(std::max(4 * c.stall_r, 64u), kTreeMore), s);
}

hipError_t launch_tree_undo(const TreeArgs& a, int32_t* seq, uint32_t* head, uint32_t* tail, hipStream_t s) {
    hipLaunchKernelGGL(k_tree_undo, dim3(blocks(std::max<uint64_t>(a.n, (uint64_t)a.R + 1))), dim3(256), 0, s, a, seq,
                       head, tail);
    return hipGetLastError();
}

}  // namespace ibip
