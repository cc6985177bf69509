// Pressure-based drainage by morphological image opening (Section 2.4.1),
// used for the equal-saturation comparison of Section 3.1.1.
//
// For a squared radius T: eroding the pore space by B(., T) leaves the
// centres c with dt2[c] >= T (a ball around c is free of solid exactly when
// the nearest solid is at squared distance >= T); trimming keeps the eroded
// components that touch the inlet candidates Q0 (inlets and their face
// neighbours, pore only); dilating by B(., T) gives
//   D_T = {v : some kept c has |v - c|^2 < T}.
// The kept sets are nested in T, and c is kept at T exactly when
// K(c) >= T, where K(c) is the maximin of dt2 over paths from Q0 to c. So one
// maximin reconstruction gives every trim at once, and each dilation is a
// distance transform of {K >= T} thresholded at T.
#include "ibip_internal.h"

namespace ibip {

namespace {

// K0(v) = dt2(v) on Q0, 0 elsewhere; also counts pore voxels.
// Seeds of the opening: pore voxels in Q0 (an inlet voxel or a face
// neighbour of one); with kMask, only pore inlet voxels count.
// A workgroup takes kSeedChunk voxels, so that it adds its count once: with 256
// voxels a workgroup and the image loaded at all seven places also without kMask,
// 512^3 took 2.47 ms; now 0.33.
constexpr int kSeedChunk = 2048;
template <bool kMask>
__global__ __launch_bounds__(256) void k_mio_seed(const uint8_t* img, const uint8_t* inlets, const uint32_t* dt2,
                                                  int X, int Y, int Z, FastDiv divZ, FastDiv divY, uint32_t* k0,
                                                  uint32_t* n_pore) {
    const int64_t yz = (int64_t)Y * Z;
    const int64_t n = (int64_t)X * yz;
    uint32_t pores = 0;
    for (int64_t v = (int64_t)blockIdx.x * kSeedChunk + threadIdx.x, end = min(v + kSeedChunk, n); v < end; v += 256) {
        // the seven positions are loaded together (an outside neighbour reads
        // v itself): a chain of conditional loads would wait for each in turn
        // coordinates by multiplicative division (indices fit 31 bits)
        const uint32_t t = fdiv((uint32_t)v, divZ), xx = fdiv(t, divY);
        const int z = (int)((uint32_t)v - t * (uint32_t)Z), y = (int)(t - xx * (uint32_t)Y), x = (int)xx;
        const int64_t nb[7] = {v, x > 0 ? v - yz : v, x < X - 1 ? v + yz : v, y > 0 ? v - Z : v,
                               y < Y - 1 ? v + Z : v, z > 0 ? v - 1 : v, z < Z - 1 ? v + 1 : v};
        const uint32_t d = dt2[v];
        uint8_t in[7], im[7];
#pragma unroll
        for (int j = 0; j < 7; j++) {
            in[j] = inlets[nb[j]];
            im[j] = kMask || j == 0 ? img[nb[j]] : 1;
        }
        bool any = false;
#pragma unroll
        for (int j = 0; j < 7; j++) any |= in[j] != 0 && (!kMask || im[j] != 0);
        const bool pore = im[0] != 0;
        pores += pore;
        k0[v] = pore && any ? d : 0u;
    }
    block_add_slots(n_pore, pores);
}

// Voxels of the intermediate images that a set of launches holds.
constexpr int64_t kLevelVoxels = 1 << 23;

// counts[i * kCountSlots + slot] += the voxels with mio_r2 = T[i] (T decreasing).
constexpr int kCountLevels = 4096;  // levels whose table LDS holds
__global__ __launch_bounds__(256) void k_mio_count(const uint32_t* mio_r2, int64_t n, const uint32_t* T, int nT,
                                                   uint32_t* counts) {
    extern __shared__ uint32_t lds[];  // T, then the counts
    uint32_t* cnt = lds + nT;
    for (int i = threadIdx.x; i < nT; i += 256) {
        lds[i] = T[i];
        cnt[i] = 0;
    }
    __syncthreads();
    const int64_t per = (n + gridDim.x - 1) / gridDim.x, v0 = blockIdx.x * per, v1 = min(v0 + per, n);
    for (int64_t base = v0; base < v1; base += 4 * 256) {
        uint32_t r[4];
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int64_t v = base + q * 256 + threadIdx.x;
            const uint32_t x = mio_r2[min(v, n - 1)];
            r[q] = v < v1 ? x : 0u;
        }
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const uint64_t m = __ballot(r[q] != 0);
            if (!m) continue;
            int lo = 0, hi = nT - 1;  // the first level with T <= r
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (lds[mid] > r[q]) lo = mid + 1;
                else hi = mid;
            }
            // most lanes of a wave share their level
            const int l0 = __builtin_amdgcn_readlane(lo, __ffsll((unsigned long long)m) - 1);
            const bool first = r[q] != 0 && lo == l0;
            const uint64_t same = __ballot(first);
            if ((int)(threadIdx.x & 63) == __ffsll((unsigned long long)same) - 1)
                atomicAdd(&cnt[l0], (uint32_t)__popcll(same));
            if (r[q] != 0 && !first) atomicAdd(&cnt[lo], 1u);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nT; i += 256)
        if (cnt[i]) atomicAdd(&counts[(size_t)i * kCountSlots + blockIdx.x % kCountSlots], cnt[i]);
}

inline unsigned blocks(int64_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

ibip_status run_mio(ibip_ctx* ctx, const uint8_t* image, const uint8_t* inlets, ibip_dims d, const uint32_t* T,
                    int32_t nT, uint32_t* mio_r2, double* mio_sat) {
    hipStream_t s = ctx->stream;
    const int64_t n = nvox(d);
    uint32_t* dt2 = (uint32_t*)ensure(ctx, B_KEY, sizeof(uint32_t) * n);
    uint32_t* kmap = (uint32_t*)ensure(ctx, B_STATE, sizeof(uint32_t) * n);
    // Several levels share their launches where the image alone does not fill the
    // GPU: 226 levels of 500 x 500, one by one, took 13.5 ms (16 workgroups in pass
    // y, 27 + 25 + 8 us a level), 32 at a time 0.58 (43 + 28 us for 32
    // levels). From 2^22 voxels on a level's launches fill it by themselves.
    const EdtTiles tiles = edt_tiles(ctx->tuning);
    const bool levels = nT > 0 && nT <= kCountLevels && opening_levels_ok(d, T[0], tiles);
    const int64_t stride = (n + 7) / 8 * 8;
    const int at_once = (int)std::max<int64_t>(std::min<int64_t>({(int64_t)kOpeningLevels, (int64_t)nT, kLevelVoxels / n}), 1);
    const int64_t held = levels ? stride * at_once : n;
    uint16_t* g16 = (uint16_t*)ensure(ctx, B_TMP0, sizeof(uint16_t) * held);
    uint32_t* tmp32 = (uint32_t*)ensure(ctx, B_TMP1, std::max(sizeof(uint32_t) * n, sizeof(uint16_t) * held));
    // per-level counts and the pore count, kCountSlots words each
    const size_t ncount = (size_t)kCountSlots * ((size_t)nT + 1);
    uint32_t* counts = (uint32_t*)ensure(ctx, B_MIOCNT, sizeof(uint32_t) * (ncount + nT));
    uint32_t* dT = counts + ncount;
    uint8_t* misc = (uint8_t*)ensure(ctx, B_MISC, 4096);
    uint32_t* h = (uint32_t*)pinned(ctx, 4096 + sizeof(uint32_t) * ncount);
    if (!dt2 || !kmap || !g16 || !tmp32 || !counts || !misc || !h)
        return fail(ctx, IBIP_ENOMEM, "opening_drainage: allocation failed");
    uint32_t* flags = (uint32_t*)(misc + 3584);  // [0] solid seen, [2] scratch flag
    uint32_t* pore_slots = counts + (size_t)kCountSlots * nT;
    ibip_status rc;
    ctx->timer.mark(10, s);
    if ((rc = hip_check(ctx, hipMemsetAsync(flags, 0, 16, s), "memset")) != IBIP_OK) return rc;
    if ((rc = hip_check(ctx, hipMemsetAsync(counts, 0, sizeof(uint32_t) * ncount, s), "memset")) != IBIP_OK)
        return rc;
    if ((rc = hip_check(ctx, hipMemsetAsync(mio_r2, 0, sizeof(uint32_t) * n, s), "memset")) != IBIP_OK) return rc;
    if ((rc = hip_check(ctx, launch_edt(image, nullptr, 0, 0, d, g16, tmp32, dt2, &flags[0], s, nullptr, nullptr,
                                        edt_tiles(ctx->tuning)), "edt")) != IBIP_OK)
        return rc;
    const unsigned seed_blocks = (unsigned)((n + kSeedChunk - 1) / kSeedChunk);
    const FastDiv fz = make_fastdiv((uint32_t)d.Z), fy = make_fastdiv((uint32_t)d.Y);
    if (ctx->readings & IBIP_READ_MASK_INLETS)
        hipLaunchKernelGGL(k_mio_seed<true>, dim3(seed_blocks), dim3(256), 0, s, image, inlets, dt2, d.X, d.Y, d.Z, fz,
                           fy, kmap, pore_slots);
    else
        hipLaunchKernelGGL(k_mio_seed<false>, dim3(seed_blocks), dim3(256), 0, s, image, inlets, dt2, d.X, d.Y, d.Z, fz,
                           fy, kmap, pore_slots);
    if ((rc = hip_check(ctx, hipMemcpyAsync(h, flags, 4, hipMemcpyDeviceToHost, s), "copy")) != IBIP_OK) return rc;
    if ((rc = hip_check(ctx, hipMemcpyAsync(h + 64, pore_slots, sizeof(uint32_t) * kCountSlots,
                                            hipMemcpyDeviceToHost, s), "copy")) != IBIP_OK)
        return rc;
    if ((rc = hip_check(ctx, hipStreamSynchronize(s), "sync")) != IBIP_OK) return rc;
    if (!h[0]) return fail(ctx, IBIP_ENOSOLID, "opening_drainage: image holds no solid voxel");
    uint64_t n_pore = 0;
    for (int q = 0; q < kCountSlots; q++) n_pore += h[64 + q];
    int iters = 0;
    if ((rc = reconstruct(ctx, nullptr, dt2, false, d, kmap, &iters)) != IBIP_OK) return rc;
    if (levels) {
        for (int32_t i = 0; i < nT; i += at_once)
            if ((rc = hip_check(ctx, launch_opening_levels(kmap, T + i, std::min(at_once, nT - i), stride, d, g16,
                                                           (uint16_t*)tmp32, &flags[2], mio_r2, s, tiles),
                                "opening levels")) != IBIP_OK)
                return rc;
        if (mio_sat) {
            uint32_t* hT = h + 1024;  // (the counts' place, copied back after)
            std::copy(T, T + nT, hT);
            if ((rc = hip_check(ctx, hipMemcpyAsync(dT, hT, sizeof(uint32_t) * nT, hipMemcpyHostToDevice, s), "copy")) !=
                IBIP_OK)
                return rc;
            hipLaunchKernelGGL(k_mio_count, dim3((unsigned)std::max<int64_t>(std::min<int64_t>(n / 8192, 1024), 1)),
                               dim3(256), sizeof(uint32_t) * 2 * nT, s, mio_r2, n, dT, nT, counts);
        }
    }
    for (int32_t i = levels ? nT : 0; i < nT; i++) {
        // distance to the kept centres, capped at T; the last pass writes T
        // into mio_r2 where it is still 0 and the distance is below T
        if ((rc = hip_check(ctx, launch_edt(nullptr, kmap, T[i], T[i], d, g16, tmp32, nullptr, &flags[2], s, mio_r2,
                                            counts + (size_t)kCountSlots * i, edt_tiles(ctx->tuning)),
                                 "edt")) != IBIP_OK)
            return rc;
    }
    if ((rc = hip_check(ctx, hipGetLastError(), "mio launch")) != IBIP_OK) return rc;
    uint32_t* hc = h + 1024;
    if ((rc = hip_check(ctx, hipMemcpyAsync(hc, counts, sizeof(uint32_t) * kCountSlots * nT, hipMemcpyDeviceToHost,
                                            s), "copy")) != IBIP_OK)
        return rc;
    ctx->timer.mark(11, s);
    if ((rc = hip_check(ctx, hipStreamSynchronize(s), "sync")) != IBIP_OK) return rc;
    if (ctx->timer.on) {
        ctx->timing.mio_ms += ctx->timer.ms(10, 11);
        ctx->timing.relax_sweeps += iters;
    }
    if (mio_sat) {
        uint64_t c = 0;
        for (int32_t i = 0; i < nT; i++) {
            if (!levels) c = 0;  // (counted per level; else the voxels first reached at each)
            for (int q = 0; q < kCountSlots; q++) c += hc[(size_t)kCountSlots * i + q];
            mio_sat[i] = n_pore ? (double)c / (double)n_pore : 0.0;
        }
    }
    return IBIP_OK;
}

}  // namespace ibip
