// Maximin reconstruction by basins.
//
//   W(v) = max over paths from the seeds to v of the smallest capacity on the path
//
// Each voxel climbs to the neighbour of largest (capacity, index) until it
// reaches a voxel that has none larger, its basin's top. The climb never goes
// below cap(v), so W(v) = min(cap(v), B(top)) with B the maximin of the tops, and
// the problem shrinks to the graph of the basins: an edge (a, b, w) for
// neighbours u, v of basins a and b, w = min(cap(u), cap(v)), and an edge to a node
// O of capacity infinity for each seed voxel. On 512^3 blurred noise 67 M pore
// voxels have 0.4 M basins by squared distance, 2 M by step.
//
// Boruvka rounds on that graph: every component but O's takes its best edge
// (largest (w, place in the list), so that no cycle longer than two arises) and
// hooks its root under the root at the other end, H[root] = (w, other root); of two
// that chose the same edge the larger index hooks. Inside a component the
// roots reach each other by edges no worse than the best edge that leaves it, so
// B(root) = min(w, B(other root)), and compressing H by (min of w, root) gives B
// once no edge is left between components: 6 to 8 rounds on the images above.
//
// Against relaxing tiles to the fixed point (trap.hip), which took 176 sweeps
// with the front crossing the image: MEASURED
#include "basin.h"

namespace ibip {

namespace {

constexpr uint32_t kTop = 0x80000000u;    // in par: a label (basin), not a voxel
constexpr uint32_t kNone = 0xffffffffu;   // in par: capacity 0

__device__ inline uint64_t ld64(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ inline uint32_t to(uint64_t h) { return (uint32_t)h; }
__device__ inline uint64_t hook(uint32_t w, uint32_t t) { return (uint64_t)w << 32 | t; }

// Places for `mine` entries of each thread in the list of slot s: one atomic per
// workgroup of 256 threads, which all call it; kBasinSlots lists, since an atomic on
// a word that the whole GPU appends at takes 50 ns, one after another.
__device__ inline uint32_t slot_append(uint32_t* cnt, uint32_t mine) {
    __shared__ uint32_t wave[kBasinWg / 64 + 1], first;
    const uint32_t lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t t = __shfl_up(incl, o, 64);
        if (lane >= (uint32_t)o) incl += t;
    }
    const uint32_t total = __builtin_amdgcn_readlane(incl, 63);
    if (lane == 0) wave[w] = total;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (uint32_t q = 0; q < (kBasinWg + 63) / 64; q++) {
        const uint32_t c = wave[q];
        before += q < w ? c : 0u;
        all += c;
    }
    if (all == 0) return 0;  // (the same in every thread)
    if (threadIdx.x == 0) first = atomicAdd(cnt, all);
    __syncthreads();
    return first + before + incl - mine;
}

struct Place {
    int64_t v;
    int x, y, z;
    bool in;
};
__device__ inline Place place(const BasinArgs& a) {
    Place p;
    const int64_t v = (int64_t)blockIdx.x * kBasinWg + threadIdx.x;
    p.in = v < a.n;
    p.v = p.in ? v : 0;
    const uint32_t t = fdiv((uint32_t)p.v, a.divZ), xx = fdiv(t, a.divY);
    p.z = (int)((uint32_t)p.v - t * (uint32_t)a.Z);
    p.y = (int)(t - xx * (uint32_t)a.Y);
    p.x = (int)xx;
    return p;
}
__device__ inline bool inside(const BasinArgs& a, int x, int y, int z) {
    return (unsigned)x < (unsigned)a.X && (unsigned)y < (unsigned)a.Y && (unsigned)z < (unsigned)a.Z;
}

// par[v] = the neighbour to climb to, or kTop | label where v is a top. All
// neighbours are loaded before the first is used (an outside one reads v).
template <class Cap, bool kConn26>
__global__ __launch_bounds__(kBasinWg) void k_basin_up(BasinArgs a, Cap cap) {
    const Place p = place(a);
    const int64_t yz = (int64_t)a.Y * a.Z;
    const uint32_t c = p.in ? cap(p.v) : 0u;
    uint64_t best = (uint64_t)c << 32 | (uint32_t)p.v;
    if (kConn26) {
        if (c) {
#pragma unroll
            for (int j = 0; j < 27; j++) {
                const int dx = j / 9 - 1, dy = j / 3 % 3 - 1, dz = j % 3 - 1;
                if (j == 13) continue;
                const int64_t u = inside(a, p.x + dx, p.y + dy, p.z + dz) ? p.v + dx * yz + dy * a.Z + dz : p.v;
                best = max(best, (uint64_t)cap(u) << 32 | (uint32_t)u);
            }
        }
    } else {
        const int64_t u[6] = {p.x > 0 ? p.v - yz : p.v,  p.x < a.X - 1 ? p.v + yz : p.v,
                              p.y > 0 ? p.v - a.Z : p.v, p.y < a.Y - 1 ? p.v + a.Z : p.v,
                              p.z > 0 ? p.v - 1 : p.v,   p.z < a.Z - 1 ? p.v + 1 : p.v};
        uint32_t cu[6];
#pragma unroll
        for (int j = 0; j < 6; j++) cu[j] = cap(u[j]);
#pragma unroll
        for (int j = 0; j < 6; j++) best = max(best, (uint64_t)cu[j] << 32 | (uint32_t)u[j]);
    }
    const uint32_t up = (uint32_t)best;
    const bool top = c != 0 && up == (uint32_t)p.v;
    const uint32_t slot = blockIdx.x % kBasinSlots;
    const uint32_t i = slot_append(&a.ctl->np[slot * kBasinPad], top ? 1u : 0u);
    uint32_t val = c == 0 ? kNone : up;
    if (top) {
        if (i < a.pcap) {
            const uint32_t id = slot * a.pcap + i;
            a.H[id] = hook(0xffffffffu, id);
            a.best[id] = 0;
            a.best[a.pall + 1 + id] = 0;
            val = kTop | id;
        } else {
            val = kNone;
            a.ctl->abort = 1;
        }
    }
    if (p.in) a.par[p.v] = val;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.H[a.pall] = hook(0xffffffffu, a.pall);
}

// par[v] = the label at the end of v's climb. A launch makes up to `hops` hops
// and writes where it got, so the next launch's hops are that much longer (any
// value read is further up the climb); it runs if the one before left some.
__global__ __launch_bounds__(256) void k_basin_label(BasinArgs a, int hops, int pass) {
    if (a.ctl->abort || (pass > 0 && !a.ctl->climb[pass - 1])) return;
    bool left = false;
    for (int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x; v < a.n; v += (int64_t)gridDim.x * 256) {
        const uint32_t p0 = a.par[v];
        if (p0 & kTop) continue;
        uint32_t p = p0;
        for (int h = 0; h < hops && !(p & kTop); h++) p = a.par[p];
        a.par[v] = p;
        left |= !(p & kTop);
    }
    if (left) a.ctl->climb[pass] = 1;
}

// The edges between basins, and to O from the seeds. Of the edges between two
// basins only the best matters, so an edge goes into the list only if the pair
// of voxels one step aside, between the same two basins, is not better (of equals
// the one at the larger index is): on the images above 8 to 17 % of all voxels.
template <class Cap, bool kConn26>
__global__ __launch_bounds__(kBasinWg) void k_basin_edges(BasinArgs a, Cap cap, const uint32_t* w0) {
    if (a.ctl->abort) return;
    const Place p = place(a);
    const int64_t yz = (int64_t)a.Y * a.Z;
    const uint32_t la = p.in ? a.par[p.v] : kNone;
    constexpr int kDirs = kConn26 ? 13 : 3;
    uint32_t eb[kDirs + 1], ew[kDirs + 1];
    uint32_t mine = 0;
    const uint32_t c = la == kNone ? 0u : cap(p.v);
    const int64_t st[6] = {-yz, yz, -(int64_t)a.Z, (int64_t)a.Z, -1, 1};
    bool side[6];  // v has a neighbour there
    side[0] = p.x > 0; side[1] = p.x < a.X - 1;
    side[2] = p.y > 0; side[3] = p.y < a.Y - 1;
    side[4] = p.z > 0; side[5] = p.z < a.Z - 1;
#pragma unroll
    for (int d = 0; d < kDirs; d++) {
        const int j = kConn26 ? d + 14 : d == 0 ? 22 : d == 1 ? 16 : 14;  // the later half of the 3 x 3 x 3
        const int dx = j / 9 - 1, dy = j / 3 % 3 - 1, dz = j % 3 - 1;
        eb[d] = kNone;
        ew[d] = 0;
        if (la == kNone || !inside(a, p.x + dx, p.y + dy, p.z + dz)) continue;
        const int64_t u = p.v + dx * yz + dy * a.Z + dz;
        const uint32_t lb = a.par[u];
        if (lb == kNone || lb == la) continue;
        const uint32_t w = min(c, cap(u));
        bool best = true;
#pragma unroll
        for (int j2 = 0; j2 < 6; j2++) {
            const int e = j2 & 1 ? 1 : -1;
            const int ux = p.x + dx + (j2 < 2 ? e : 0), uy = p.y + dy + (j2 >> 1 == 1 ? e : 0), uz = p.z + dz + (j2 > 3 ? e : 0);
            if (!kConn26 && ((j2 < 2 && dx) || (j2 >> 1 == 1 && dy) || (j2 > 3 && dz))) continue;
            const bool ok = side[j2] && inside(a, ux, uy, uz);
            const int64_t v2 = ok ? p.v + st[j2] : p.v, u2 = ok ? u + st[j2] : u;
            const bool same = ok && a.par[v2] == la && a.par[u2] == lb;
            const uint32_t w2 = min(cap(v2), cap(u2));
            best = best && !(same && (w2 > w || (w2 == w && e > 0)));
        }
        if (best) {
            eb[d] = lb;
            ew[d] = w;
            mine++;
        }
    }
    eb[kDirs] = kNone;
    ew[kDirs] = la == kNone ? 0u : w0[p.v];
    if (ew[kDirs]) {
        bool best = true;
#pragma unroll
        for (int j2 = 0; j2 < 6; j2++) {
            const int64_t v2 = side[j2] ? p.v + st[j2] : p.v;
            const uint32_t w2 = w0[v2];
            best = best && !(side[j2] && a.par[v2] == la && (w2 > ew[kDirs] || (w2 == ew[kDirs] && (j2 & 1))));
        }
        if (best) {
            eb[kDirs] = kTop | a.pall;
            mine++;
        }
    }
    const uint32_t slot = blockIdx.x % kBasinSlots;
    uint32_t i = slot_append(&a.ctl->ne[slot * kBasinPad], mine);
    if (i + mine > a.ecap) {
        if (mine) a.ctl->abort_edges = 1;
        return;
    }
#pragma unroll
    for (int d = 0; d <= kDirs; d++) {
        if (eb[d] == kNone) continue;
        const uint32_t k = slot * a.ecap + i++;
        a.ends[k] = (uint64_t)(eb[d] & ~kTop) << 32 | (la & ~kTop);
        a.wt[k] = ew[d];
    }
}

// best[r] = max(best[r], key). The edges of one component are many in the late
// rounds: lanes that share the first lane's component send one atomic.
__device__ inline void offer(uint64_t* best, uint32_t r, uint64_t key, bool want) {
    const uint64_t wm = __ballot(want);
    if (!wm) return;
    const int lead = __ffsll((unsigned long long)wm) - 1;
    const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)r, lead);
    const uint64_t m = __ballot(want && r == r0);
    if (__popcll(m) > 4) {
        uint64_t k = want && r == r0 ? key : 0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) k = max(k, (uint64_t)__shfl_xor((unsigned long long)k, o, 64));
        if (r == r0) {
            want = want && (int)(threadIdx.x & 63) == lead;
            key = max(key, k);
        }
    }
    if (want && ld64(&best[r]) < key) atomicMax((unsigned long long*)&best[r], (unsigned long long)key);
}

// A round: the edges' ends become their components' roots; an edge inside a
// component is done with; the others are offered to both ends.
__global__ __launch_bounds__(256) void k_basin_offer(BasinArgs a, int round) {
    if (a.ctl->abort || a.ctl->abort_edges || (round > 0 && !a.ctl->live[round - 1])) return;
    const uint32_t slot = blockIdx.x % kBasinSlots, part = blockIdx.x / kBasinSlots, parts = gridDim.x / kBasinSlots;
    const uint32_t ne = a.ctl->ne[slot * kBasinPad];
    uint64_t* best = a.best + (round & 1 ? a.pall + 1 : 0u);
    bool live = false;
    for (uint32_t i0 = part * 256; i0 < ne; i0 += parts * 256) {
        const uint32_t i = i0 + threadIdx.x;
        const uint32_t k = slot * a.ecap + i;
        const uint64_t e = i < ne ? a.ends[k] : 0;
        uint32_t x = (uint32_t)e, y = (uint32_t)(e >> 32);
        bool on = x != y;
        if (on) {
            for (uint32_t t; (t = to(a.H[x])) != x;) x = t;
            for (uint32_t t; (t = to(a.H[y])) != y;) y = t;
            const uint64_t f = (uint64_t)y << 32 | x;
            if (f != e) a.ends[k] = f;
            on = x != y;
        }
        const uint64_t key = on ? hook(a.wt[k], k) : 0;
        live |= on;
        offer(best, x, key, on && x != a.pall);
        offer(best, y, key, on && y != a.pall);
    }
    if (live) a.ctl->live[round] = 1;
}

// Every root with an edge hooks under the root at its best edge's other end.
// The other round's offers are cleared for the next.
__global__ __launch_bounds__(256) void k_basin_hook(BasinArgs a, int round) {
    if (a.ctl->abort || a.ctl->abort_edges || !a.ctl->live[round]) return;
    const uint32_t slot = blockIdx.x % kBasinSlots, part = blockIdx.x / kBasinSlots, parts = gridDim.x / kBasinSlots;
    const uint32_t np = a.ctl->np[slot * kBasinPad];
    uint64_t* best = a.best + (round & 1 ? a.pall + 1 : 0u);
    uint64_t* next = a.best + (round & 1 ? 0u : a.pall + 1);
    for (uint32_t i = part * 256 + threadIdx.x; i < np; i += parts * 256) {
        const uint32_t p = slot * a.pcap + i;
        const uint64_t key = best[p];  // 0: not a root, or no edge
        if (key) {
            const uint64_t e = a.ends[(uint32_t)key];
            const uint32_t o = (uint32_t)e == p ? (uint32_t)(e >> 32) : (uint32_t)e;
            if (!(o != a.pall && best[o] == key && p < o)) a.H[p] = hook((uint32_t)(key >> 32), o);
        }
        next[p] = 0;
    }
}

// H[p] = (smallest weight on the way to p's root, that root), as far as `hops`
// hops go. The offers follow what is left of a longer chain.
__global__ __launch_bounds__(256) void k_basin_flat(BasinArgs a, int hops, int round) {
    if (a.ctl->abort || a.ctl->abort_edges || !a.ctl->live[round] || (hops > kBasinHops && !a.ctl->deep[round])) return;
    const uint32_t slot = blockIdx.x % kBasinSlots, part = blockIdx.x / kBasinSlots, parts = gridDim.x / kBasinSlots;
    const uint32_t np = a.ctl->np[slot * kBasinPad];
    bool left = false;
    for (uint32_t i = part * 256 + threadIdx.x; i < np; i += parts * 256) {
        const uint32_t p = slot * a.pcap + i;
        uint64_t h = ld64(&a.H[p]);
        if (to(h) == p) continue;
        const uint32_t t0 = to(h);
        int q = 0;
        for (; q < hops; q++) {
            const uint64_t g = ld64(&a.H[to(h)]);
            if (to(g) == to(h)) break;
            h = hook(min((uint32_t)(h >> 32), (uint32_t)(g >> 32)), to(g));
        }
        if (to(h) != t0) __hip_atomic_store(&a.H[p], h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        left |= q == hops;
    }
    if (left) a.ctl->deep[round] = 1;
}

// w[v] = min(cap(v), B(label)).
template <class Cap>
__global__ __launch_bounds__(256) void k_basin_finish(BasinArgs a, Cap cap, uint32_t* w, int rounds) {
    if (a.ctl->abort || a.ctl->abort_edges || a.ctl->live[rounds - 1]) return;
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (v >= a.n) return;
    const uint32_t l = a.par[v];
    uint32_t r = 0;
    if (l != kNone) {
        uint64_t h = a.H[l & ~kTop];
        uint32_t b = (uint32_t)(h >> 32);
        while (to(h) != a.pall) {
            const uint64_t g = a.H[to(h)];
            if (to(g) == to(h)) {
                b = 0;
                break;
            }
            b = min(b, (uint32_t)(g >> 32));
            h = g;
        }
        r = min(cap(v), b);
    }
    w[v] = r;
}

inline unsigned blocks(int64_t n, unsigned t = 256) { return (unsigned)((n + t - 1) / t); }

template <class Cap, bool kConn26>
hipError_t start(const BasinArgs& a, Cap cap, const uint32_t* w, hipStream_t s) {
    const unsigned nb = blocks(a.n, kBasinWg), few = std::min<unsigned>(blocks(a.n, 256), 2048);
    hipLaunchKernelGGL((k_basin_up<Cap, kConn26>), dim3(nb), dim3(kBasinWg), 0, s, a, cap);
    int pass = 0;
    // climbs of up to 2^5, 2^13, 2^21, 2^29 and 2^37 voxels
    for (int64_t reach = kBasinHops; pass == 0 || reach < 256 * a.n; reach *= 256, pass++)
        hipLaunchKernelGGL(k_basin_label, dim3(few), dim3(256), 0, s, a, pass ? 256 : kBasinHops, pass);
    hipLaunchKernelGGL((k_basin_edges<Cap, kConn26>), dim3(nb), dim3(kBasinWg), 0, s, a, cap, w);
    return hipGetLastError();
}

}  // namespace

void basin_caps(BasinArgs& a, int64_t n) {
    // each slot takes every kBasinSlots-th workgroup's voxels
    const int64_t per = ((n + kBasinWg - 1) / kBasinWg + kBasinSlots - 1) / kBasinSlots * kBasinWg;
    const bool all = n <= (1 << 20);  // room for whatever the image holds
    a.pcap = (uint32_t)(all ? per : per / 8);
    a.ecap = (uint32_t)(all ? 4 * per : per / 2);
    a.pall = a.pcap * kBasinSlots;
    a.n = n;
}

size_t basin_bytes(const BasinArgs& a) {
    return sizeof(BasinCtl) + 8 * (3 * ((size_t)a.pall + 1) + (size_t)a.ecap * kBasinSlots) +
           4 * ((size_t)a.ecap * kBasinSlots + (size_t)a.n);
}

void basin_carve(BasinArgs& a, void* mem) {
    char* m = (char*)mem;
    a.ctl = (BasinCtl*)m;
    m += sizeof(BasinCtl);
    a.H = (uint64_t*)m;
    a.best = a.H + a.pall + 1;
    a.ends = a.best + 2 * ((size_t)a.pall + 1);
    a.wt = (uint32_t*)(a.ends + (size_t)a.ecap * kBasinSlots);
    a.par = a.wt + (size_t)a.ecap * kBasinSlots;
}

hipError_t launch_basin_graph(const BasinArgs& a, const int32_t* seq, const uint32_t* cap32, bool conn26,
                              const uint32_t* w, hipStream_t s) {
    if (cap32) return conn26 ? start<CapU32, true>(a, CapU32{cap32}, w, s) : start<CapU32, false>(a, CapU32{cap32}, w, s);
    return conn26 ? start<CapSeq, true>(a, CapSeq{seq}, w, s) : start<CapSeq, false>(a, CapSeq{seq}, w, s);
}

hipError_t launch_basin_rounds(const BasinArgs& a, int from, int to, hipStream_t s) {
    // (workgroups by the image's size: a slot's list is read by 1 to 32 of them)
    const unsigned g = kBasinSlots * (unsigned)std::min<int64_t>(std::max<int64_t>(a.n >> 18, 1), 32);
    for (int r = from; r < to; r++) {
        hipLaunchKernelGGL(k_basin_offer, dim3(g), dim3(256), 0, s, a, r);
        hipLaunchKernelGGL(k_basin_hook, dim3(g), dim3(256), 0, s, a, r);
        hipLaunchKernelGGL(k_basin_flat, dim3(g), dim3(256), 0, s, a, kBasinHops, r);
        hipLaunchKernelGGL(k_basin_flat, dim3(g), dim3(256), 0, s, a, 32 * kBasinHops, r);
    }
    return hipGetLastError();
}

hipError_t launch_basin_finish(const BasinArgs& a, const int32_t* seq, const uint32_t* cap32, uint32_t* w, int rounds,
                               hipStream_t s) {
    if (cap32)
        hipLaunchKernelGGL(k_basin_finish<CapU32>, dim3(blocks(a.n)), dim3(256), 0, s, a, CapU32{cap32}, w, rounds);
    else
        hipLaunchKernelGGL(k_basin_finish<CapSeq>, dim3(blocks(a.n)), dim3(256), 0, s, a, CapSeq{seq}, w, rounds);
    return hipGetLastError();
}

}  // namespace ibip
