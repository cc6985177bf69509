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
// once no edge is left between components: 6 to 9 rounds on such images.
//
// Against relaxing tiles to the fixed point (trap.hip), 64 to 184 sweeps while the
// front crosses the image: trapping of 512^3 19.2 -> 6.3 ms (climbs 0.73, labels 0.53,
// edges 0.85, rounds 2.5, result 0.34), of 230 x 171 x 199 2.31 -> 0.72 ms; opening of
// 512^3 20.0 -> 7.4 ms. Bound by gathers at the edges' ends and best edges.
#include "basin.h"

namespace ibip {

namespace {

constexpr uint32_t kTop = kBasinTop, kNone = kBasinNone;

__device__ inline uint64_t ld64(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ inline uint32_t to(uint64_t h) { return (uint32_t)h; }
__device__ inline uint64_t hook(uint32_t w, uint32_t t) { return (uint64_t)w << 32 | t; }

// Sets a flag that most waves set: read first, by one lane of each.
__device__ inline void raise(uint32_t* flag, bool want) {
    const uint64_t m = __ballot(want);
    if (m && (int)(threadIdx.x & 63) == __ffsll((unsigned long long)m) - 1 &&
        __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)
        __hip_atomic_store(flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

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

// A tile of 2048 voxels, 32 along z: 8 x 8 x 32, or 64 x 32 of a plane (kFlat, for
// images of one plane, which fill an eighth of the former), with a halo of one.
// A thread has the voxels of one z and every eighth row.
template <bool kFlat>
struct Tile {
    static constexpr int TX = kFlat ? 1 : 8, TY = kFlat ? 64 : 8, TZ = 32;
    static constexpr int HX = kFlat ? 1 : TX + 2, HY = TY + 2, HZ = TZ + 2, HN = HX * HY * HZ;
    int x0, y0, z0;
    __device__ Tile(const BasinArgs& a) {
        const uint32_t t = blockIdx.x / (uint32_t)a.ntz;
        z0 = (int)(blockIdx.x - t * (uint32_t)a.ntz) * TZ;
        x0 = (int)(t / (uint32_t)a.nty) * TX;
        y0 = (int)(t % (uint32_t)a.nty) * TY;
    }
    // voxel i of the tile (z fastest): its place, its place in the halo's box
    __device__ static int lx(int i) { return kFlat ? 0 : i / (TY * TZ); }
    __device__ static int ly(int i) { return kFlat ? i / TZ : i / TZ % TY; }
    __device__ static int lz(int i) { return i % TZ; }
    __device__ static int halo(int i) { return ((lx(i) + (kFlat ? 0 : 1)) * HY + ly(i) + 1) * HZ + lz(i) + 1; }
    __device__ bool in(const BasinArgs& a, int i) const { return x0 + lx(i) < a.X && y0 + ly(i) < a.Y && z0 + lz(i) < a.Z; }
    __device__ int64_t voxel(const BasinArgs& a, int i) const {
        return ((int64_t)(x0 + lx(i)) * a.Y + y0 + ly(i)) * a.Z + z0 + lz(i);
    }
    // f of the tile and its halo into LDS (0 or `out` outside the image): all
    // loads are issued before the first is used, from clamped places
    template <class F>
    __device__ void load(const BasinArgs& a, F f, uint32_t* lds, uint32_t out) const {
        constexpr int kPer = (HN + kBasinWg - 1) / kBasinWg;
        uint32_t h[kPer];
#pragma unroll
        for (int q = 0; q < kPer; q++) {
            const int i = min((int)threadIdx.x + q * kBasinWg, HN - 1);
            const int hz = i % HZ, hy = i / HZ % HY, hx = i / (HZ * HY);
            const int gx = x0 + hx - (kFlat ? 0 : 1), gy = y0 + hy - 1, gz = z0 + hz - 1;
            const bool ok = (unsigned)gx < (unsigned)a.X && (unsigned)gy < (unsigned)a.Y && (unsigned)gz < (unsigned)a.Z;
            const int64_t v = ((int64_t)min(max(gx, 0), a.X - 1) * a.Y + min(max(gy, 0), a.Y - 1)) * a.Z + min(max(gz, 0), a.Z - 1);
            const uint32_t val = f(v);
            h[q] = ok ? val : out;
        }
#pragma unroll
        for (int q = 0; q < kPer; q++) {
            const int i = (int)threadIdx.x + q * kBasinWg;
            if (i < HN) lds[i] = h[q];
        }
    }
};
constexpr int kTileVoxels = 2048, kOwn = kTileVoxels / kBasinWg;

// par[v] = the end of v's climb inside its tile: kTop | label at a top, else
// the voxel outside the tile that it goes on to.
template <class Cap, bool kConn26, bool kFlat>
__global__ __launch_bounds__(kBasinWg) void k_basin_up(BasinArgs a, Cap cap) {
    using T = Tile<kFlat>;
    __shared__ uint32_t hw[T::HN];
    __shared__ uint16_t up[kTileVoxels];  // the tile's voxel to climb to (itself at a top), or kOut | direction
    constexpr uint32_t kOut = 0x8000u;
    const T t(a);
    const int tid = threadIdx.x;
    t.load(a, cap, hw, 0u);
    __syncthreads();
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < kOwn; j++) {
        const int i = tid + j * kBasinWg, h = T::halo(i);
        // directions 0..26 are in the order of the neighbours' indices; 13 is v itself
        const uint32_t me = hw[h];
        uint64_t best = (uint64_t)Cap::rank(me) << 5 | 13u;
#pragma unroll
        for (int q = 0; q < 27; q++) {
            const int dx = q / 9 - 1, dy = q / 3 % 3 - 1, dz = q % 3 - 1;
            if (q == 13 || (kFlat && dx) || (!kConn26 && (dx != 0) + (dy != 0) + (dz != 0) > 1)) continue;
            const uint32_t c = Cap::rank(hw[h + (dx * T::HY + dy) * T::HZ + dz]);
            best = max(best, (uint64_t)(Cap::open(me, dx) ? c : 0u) << 5 | (uint32_t)q);
        }
        const int q = (int)((uint32_t)best & 31u);
        const int x = T::lx(i) + q / 9 - 1, y = T::ly(i) + q / 3 % 3 - 1, z = T::lz(i) + q % 3 - 1;
        const bool stay = (unsigned)x < (unsigned)T::TX && (unsigned)y < (unsigned)T::TY && (unsigned)z < (unsigned)T::TZ;
        up[i] = (uint16_t)(stay ? (uint32_t)((x * T::TY + y) * T::TZ + z) : kOut | (uint32_t)q);
        mine += q == 13 && Cap::rank(me) != 0;  // (outside the image the capacity is 0)
    }
    __syncthreads();
    uint32_t end[kOwn];
#pragma unroll
    for (int j = 0; j < kOwn; j++) {
        const int i = tid + j * kBasinWg;
        uint32_t e = (uint32_t)i;
        if (Cap::rank(hw[T::halo(i)]))
            for (uint32_t n; (n = up[e]) != e && !(n & kOut);) e = n;
        end[j] = e;
    }
    const uint32_t slot = blockIdx.x % kBasinSlots;
    uint32_t k = slot_append(&a.ctl->np[slot * kBasinPad], mine);
    // the tops' labels, in place of their capacities
    uint32_t own[kOwn];
#pragma unroll
    for (int j = 0; j < kOwn; j++) own[j] = Cap::rank(hw[T::halo(tid + j * kBasinWg)]);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kOwn; j++) {
        const int i = tid + j * kBasinWg;
        if (!own[j] || up[i] != i) continue;
        uint32_t id = kNone;
        if (k < a.pcap) {
            id = slot * a.pcap + k;
            a.H[id] = hook(0xffffffffu, id);
            a.best[id] = 0;
            a.best[a.pall + 1 + id] = 0;
            if (a.mst) {
                a.mst[id] = 0;
                a.topv[id] = (uint32_t)t.voxel(a, i);
            }
            id |= kTop;
        } else {
            a.ctl->abort = 1;
        }
        k++;
        hw[T::halo(i)] = id;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kOwn; j++) {
        const int i = tid + j * kBasinWg;
        if (!t.in(a, i)) continue;
        uint32_t val = kNone;
        if (own[j]) {
            const uint32_t e = end[j], n = up[e];
            if (n & kOut) {
                const int q = (int)(n & 31u);
                val = (uint32_t)(t.voxel(a, (int)e) + ((int64_t)(q / 9 - 1) * a.Y + (q / 3 % 3 - 1)) * a.Z + q % 3 - 1);
            } else {
                val = hw[T::halo((int)e)];
            }
        }
        a.par[t.voxel(a, i)] = val;
    }
    if (blockIdx.x == 0 && tid == 0) a.H[a.pall] = hook(0xffffffffu, a.pall);
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
    raise(&a.ctl->climb[pass], left);
}

// The edges between basins, and to O from the seeds. Of the edges between two
// basins only the best matters, so an edge goes into the list only if the pair
// of voxels one step aside, between the same two basins, is not better (of equals
// the one at the larger index is): on the images above 8 to 17 % of all voxels.
template <class Cap, bool kConn26, bool kFlat>
__global__ __launch_bounds__(kBasinWg) void k_basin_edges(BasinArgs a, Cap cap, const uint32_t* w0) {
    if (a.ctl->abort) return;
    using T = Tile<kFlat>;
    __shared__ uint32_t hl[T::HN], hc[T::HN];
    const T t(a);
    const int tid = threadIdx.x;
    t.load(a, [&](int64_t v) { return a.par[v]; }, hl, kNone);
    t.load(a, cap, hc, 0u);
    __syncthreads();
    constexpr int kDirs = kConn26 ? 13 : 3;
    uint32_t take[kOwn], seed[kOwn];  // bit d: the edge in direction d; the seed's weight
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < kOwn; j++) {
        const int i = tid + j * kBasinWg, h = T::halo(i);
        const uint32_t la = hl[h];
        take[j] = seed[j] = 0;
        const int64_t v = t.in(a, i) ? t.voxel(a, i) : 0;
        uint32_t s0 = w0 ? w0[v] : 0u;
        if (la == kNone) s0 = 0;
        uint32_t mask = 0;
#pragma unroll
        for (int d = 0; d < kDirs; d++) {
            const int q = kConn26 ? d + 14 : d == 0 ? 22 : d == 1 ? 16 : 14;  // the later half of the neighbours
            const int dx = q / 9 - 1, dy = q / 3 % 3 - 1, dz = q % 3 - 1;
            if (kFlat && dx) continue;
            const int off = (dx * T::HY + dy) * T::HZ + dz;
            const uint32_t lb = hl[h + off];
            if (la != kNone && lb != kNone && lb != la && Cap::open(hc[h], dx)) {
                const uint32_t w = min(Cap::rank(hc[h]), Cap::rank(hc[h + off]));
                uint32_t better = 0;
#pragma unroll
                for (int b = 0; b < 6; b++) {
                    const int e = b & 1 ? 1 : -1;
                    const int ex = b < 2 ? e : 0, ey = b >> 1 == 1 ? e : 0, ez = b > 3 ? e : 0;
                    // (inside the halo; along the edge itself there is no such pair)
                    if ((kFlat && ex) || (!kConn26 && (ex * dx || ey * dy || ez * dz)) || dx + ex > 1 || dx + ex < -1 ||
                        dy + ey > 1 || dy + ey < -1 || dz + ez > 1 || dz + ez < -1)
                        continue;
                    const int side = h + (ex * T::HY + ey) * T::HZ + ez;
                    const uint32_t w2 = min(Cap::rank(hc[side]), Cap::rank(hc[side + off]));
                    better |= (uint32_t)(hl[side] == la) & (uint32_t)(hl[side + off] == lb) &
                              (uint32_t)(e > 0 ? w2 >= w : w2 > w);
                }
                mask |= (1u - better) << d;
            }
        }
        take[j] = mask;
        mine += (uint32_t)__popc(mask);
        if (s0) {
#pragma unroll
            for (int b = 0; b < 6; b++) {
                const int e = b & 1 ? 1 : -1;
                const int ex = b < 2 ? e : 0, ey = b >> 1 == 1 ? e : 0, ez = b > 3 ? e : 0;
                if (kFlat && ex) continue;
                if (hl[h + (ex * T::HY + ey) * T::HZ + ez] != la) continue;  // (so it is inside the image)
                const uint32_t w2 = w0[v + ((int64_t)ex * a.Y + ey) * a.Z + ez];
                if (w2 > s0 || (w2 == s0 && e > 0)) {
                    s0 = 0;
                    break;
                }
            }
            seed[j] = s0;
            mine += s0 != 0;
        }
    }
    const uint32_t slot = blockIdx.x % kBasinSlots;
    uint32_t i = slot_append(&a.ctl->ne[slot * kBasinPad], mine);
    if (i + mine > a.ecap) {
        if (mine) a.ctl->abort_edges = 1;
        return;
    }
    uint32_t k = slot * a.ecap + i;
#pragma unroll
    for (int j = 0; j < kOwn; j++) {
        const int h = T::halo(tid + j * kBasinWg);
        const uint32_t la = hl[h] & ~kTop;
#pragma unroll
        for (int d = 0; d < kDirs; d++) {
            if (!(take[j] >> d & 1u)) continue;
            const int q = kConn26 ? d + 14 : d == 0 ? 22 : d == 1 ? 16 : 14;
            const int off = ((q / 9 - 1) * T::HY + (q / 3 % 3 - 1)) * T::HZ + q % 3 - 1;
            a.ends[k] = (uint64_t)(hl[h + off] & ~kTop) << 32 | la;
            a.wt[k++] = min(Cap::rank(hc[h]), Cap::rank(hc[h + off]));
        }
        if (seed[j]) {
            a.ends[k] = (uint64_t)a.pall << 32 | la;
            a.wt[k++] = seed[j];
        }
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
    raise(&a.ctl->live[round], live);
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
            if (!(o != a.pall && best[o] == key && p < o)) {
                a.H[p] = hook((uint32_t)(key >> 32), o);
                if (a.mst) a.mst[p] = hook((uint32_t)(key >> 32), o);
            }
        }
        next[p] = 0;
    }
}

// H[p] = (smallest weight on the way to p's root, that root), as far as `hops`
// hops go. The offers follow what is left of a longer chain.
__global__ __launch_bounds__(256) void k_basin_flat(BasinArgs a, int hops, int round) {
    if (a.ctl->abort || a.ctl->abort_edges || !a.ctl->live[round]) return;
    const uint32_t slot = blockIdx.x % kBasinSlots, part = blockIdx.x / kBasinSlots, parts = gridDim.x / kBasinSlots;
    const uint32_t np = a.ctl->np[slot * kBasinPad];
    for (uint32_t i = part * 256 + threadIdx.x; i < np; i += parts * 256) {
        const uint32_t p = slot * a.pcap + i;
        uint64_t h = ld64(&a.H[p]);
        if (to(h) == p) continue;
        const uint32_t t0 = to(h);
        for (int q = 0; q < hops; q++) {
            const uint64_t g = ld64(&a.H[to(h)]);
            if (to(g) == to(h)) break;
            h = hook(min((uint32_t)(h >> 32), (uint32_t)(g >> 32)), to(g));
        }
        if (to(h) != t0) __hip_atomic_store(&a.H[p], h, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
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

template <bool kFlat>
int64_t tiles(const BasinArgs& a) {
    return (int64_t)((a.X + Tile<kFlat>::TX - 1) / Tile<kFlat>::TX) * a.nty * a.ntz;
}

inline unsigned blocks(int64_t n, unsigned t = 256) { return (unsigned)((n + t - 1) / t); }

template <class Cap, bool kConn26, bool kFlat>
hipError_t start(const BasinArgs& a, Cap cap, const uint32_t* w, hipStream_t s) {
    const unsigned nb = (unsigned)(tiles<kFlat>(a)), few = std::min<unsigned>(blocks(a.n), 2048);
    hipLaunchKernelGGL((k_basin_up<Cap, kConn26, kFlat>), dim3(nb), dim3(kBasinWg), 0, s, a, cap);
    int pass = 0;
    // climbs of up to 2^5, 2^13, 2^21, 2^29 and 2^37 tiles
    for (int64_t reach = kBasinHops; pass == 0 || reach < 256 * a.n; reach *= 256, pass++)
        hipLaunchKernelGGL(k_basin_label, dim3(few), dim3(256), 0, s, a, pass ? 256 : kBasinHops, pass);
    hipLaunchKernelGGL((k_basin_edges<Cap, kConn26, kFlat>), dim3(nb), dim3(kBasinWg), 0, s, a, cap, w);
    return hipGetLastError();
}
template <class Cap>
hipError_t start(const BasinArgs& a, Cap cap, bool conn26, const uint32_t* w, hipStream_t s) {
    if (a.X == 1) return conn26 ? start<Cap, true, true>(a, cap, w, s) : start<Cap, false, true>(a, cap, w, s);
    return conn26 ? start<Cap, true, false>(a, cap, w, s) : start<Cap, false, false>(a, cap, w, s);
}

}  // namespace

void basin_caps(BasinArgs& a, ibip_dims d) {
    a.X = d.X;
    a.Y = d.Y;
    a.Z = d.Z;
    a.n = nvox(d);
    const int ty = a.X == 1 ? Tile<true>::TY : Tile<false>::TY;
    a.nty = (a.Y + ty - 1) / ty;
    a.ntz = (a.Z + Tile<true>::TZ - 1) / Tile<true>::TZ;
    // Each slot takes every kBasinSlots-th tile's voxels, those of the image: a tile
    // of an image one or a few voxels thick holds that share of its 2,048, and an
    // image of few tiles uses that many slots. So the lists have room for an eighth
    // and half of the voxels, 1.8 times that at most where the last tiles are mostly
    // outside, and places in them fit 32 bits for any image (fewer than 2^31 voxels).
    const int64_t nt = a.X == 1 ? tiles<true>(a) : tiles<false>(a);
    const int64_t held = (int64_t)std::min(a.X, a.X == 1 ? 1 : Tile<false>::TX) * std::min(a.Y, ty) *
                         std::min(a.Z, Tile<true>::TZ);
    const int64_t slots = std::min<int64_t>(nt, kBasinSlots);
    const int64_t per = (nt + slots - 1) / slots * held;
    a.whole = per * slots <= 1 << 20;
    a.pcap = (uint32_t)(a.whole ? per : per / 8);
    a.ecap = (uint32_t)(a.whole ? 4 * per : per / 2);
    a.pall = a.pcap * (uint32_t)slots;
    a.eall = a.ecap * (uint32_t)slots;
}

size_t basin_bytes(const BasinArgs& a) {
    return sizeof(BasinCtl) + 8 * (3 * ((size_t)a.pall + 1) + (size_t)a.eall) + 4 * ((size_t)a.eall + (size_t)a.n);
}

void basin_carve(BasinArgs& a, void* mem) {
    char* m = (char*)mem;
    a.ctl = (BasinCtl*)m;
    m += sizeof(BasinCtl);
    a.H = (uint64_t*)m;
    a.best = a.H + a.pall + 1;
    a.ends = a.best + 2 * ((size_t)a.pall + 1);
    a.wt = (uint32_t*)(a.ends + (size_t)a.eall);
    a.par = a.wt + (size_t)a.eall;
}

hipError_t launch_basin_graph(const BasinArgs& a, const int32_t* seq, const uint32_t* cap32, bool conn26,
                              const uint32_t* w, hipStream_t s) {
    return cap32 ? start(a, CapU32{cap32}, conn26, w, s) : start(a, CapSeq{seq}, conn26, w, s);
}

hipError_t launch_basin_graph_keys(const BasinArgs& a, const uint32_t* key, hipStream_t s) {
    const CapKey cap{key};
    return a.X == 1 ? start<CapKey, false, true>(a, cap, nullptr, s) : start<CapKey, false, false>(a, cap, nullptr, s);
}

hipError_t launch_basin_rounds(const BasinArgs& a, int from, int to, hipStream_t s) {
    // (workgroups by the image's size: a slot's list is read by 1 to 32 of them)
    const unsigned g = kBasinSlots * (unsigned)std::min<int64_t>(std::max<int64_t>(a.n >> 18, 1), 32);
    for (int r = from; r < to; r++) {
        hipLaunchKernelGGL(k_basin_offer, dim3(g), dim3(256), 0, s, a, r);
        hipLaunchKernelGGL(k_basin_hook, dim3(g), dim3(256), 0, s, a, r);
        hipLaunchKernelGGL(k_basin_flat, dim3(g), dim3(256), 0, s, a, 8 * kBasinHops, r);
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
