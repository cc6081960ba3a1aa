// Gather rows on their way to a pass: index rows tiled through LDS and the
// partners' records loaded ahead.
#pragma once

#include "crk_internal.h"

namespace crk {

// wait for the loads
__device__ __forceinline__ void stage_wait() {
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    __builtin_amdgcn_sched_barrier(0);
}

// Tiles of the gather rows of a wavefront's 64 / G groups in LDS. Read from
// memory as the loop goes, every step of many rows would meet the first line
// of some row's next 32 entries, and a wavefront's loads complete in order,
// so that each step would wait for HBM whatever is prefetched. One load
// instruction brings the next 4 G entries of each row.
template <int G, int Loads = G < 16 ? 8 : 128 / G>
struct RowTile {
    static constexpr int kLoads = Loads;
    static constexpr int kTile = 4 * G * kLoads - (G < 2 ? 4 : 2 * G);   // entries used: any alignment, whole steps
    __align__(16) int32_t e[kLoads * 256];
};

// the tile from entry k0 (a multiple of four) of the row at gidx + b4 + al of
// this lane's group, b4 a multiple of four; up to three entries past the row
// are read
template <int G, int Loads>
__device__ __forceinline__ void fetch_tile(RowTile<G, Loads> &t, const int32_t *__restrict__ gidx, int64_t b4, int end,
                                           int k0, int l) {
    const int32_t *p = gidx + b4 + k0 + 4 * l;
    int o = k0 + 4 * l;
#pragma unroll
    for (int q = 0; q < Loads; q++, p += 4 * G, o += 4 * G)
        if (o < end)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)p,
                                             (__attribute__((address_space(3))) void *)(t.e + q * 256), 16, 0, 0);
    stage_wait();
}

// word of the tile, from its group's first on, that holds entry x (counted from
// its first, aligned, entry)
template <int G>
__device__ __forceinline__ uint32_t tile_word(uint32_t x) {
    return x / (4 * G) * 256 + x % (4 * G);
}

// The entries l, l + G, ... below cnt of a row: term(load(k)) for each in
// turn, the next D (1 or 2) partners' records loading meanwhile (load takes
// any k). With two ahead four entries a step, each record in registers of its
// own: were they moved on at the end of a step, the move would wait for all
// that is on its way (FP64 moments, one lane a row: 32^3 with 268 neighbours
// 0.81 and 0.63 ms so, 64^3 0.208 and 0.193; FP32 gradient of 128^3, 0.66 and
// 0.61). One ahead (FP64 gradient) has no registers to spare for it.
template <int G, int D, typename Load, typename Term>
__device__ __forceinline__ void row_terms(int l, int cnt, Load &&load, Term &&term) {
    if constexpr (D == 1) {
        auto r0 = load(l);
        for (int k = l; k < cnt; k += G) {
            const auto a = r0;
            r0 = load(k + G);
            term(a);
        }
    } else {
        auto r0 = load(l), r1 = load(l + G);
        for (int k = l; k < cnt; k += 4 * G) {
            const auto r2 = load(k + 2 * G);
            term(r0);
            const auto r3 = load(k + 3 * G);
            if (k + G < cnt) term(r1);
            r0 = load(k + 4 * G);
            if (k + 2 * G < cnt) term(r2);
            r1 = load(k + 5 * G);
            if (k + 3 * G < cnt) term(r3);
        }
    }
}

// The sum over the row gidx[b .. b + cnt) of this lane's group: term(load(j))
// over the lane's entries j, the next D (1 or 2) partners' records loading
// meanwhile. self: any particle, loaded past the end.
template <int G, int D, int Loads, typename Load, typename Term>
__device__ __forceinline__ void row_sum(RowTile<G, Loads> &t, const int32_t *__restrict__ gidx, int64_t b, int cnt,
                                        int32_t self, int lane, Load &&load, Term &&term) {
    const int al = (int)(b & 3), l = lane % G;
    for (int k0 = 0; k0 < cnt; k0 += RowTile<G, Loads>::kTile) {
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): the last tile's reads are done
        __builtin_amdgcn_sched_barrier(0);
        fetch_tile(t, gidx, b - al, cnt + al, k0, l);
        const int end = min(cnt - k0, RowTile<G, Loads>::kTile);
        const int32_t *const e = t.e + (lane - l) * 4;
        row_terms<G, D>(l, end, [&](int k) { return load(k < end ? e[tile_word<G>(k + al)] : self); }, term);
    }
}

}  // namespace crk
