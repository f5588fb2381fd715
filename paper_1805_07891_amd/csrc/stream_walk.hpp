// Walk over a wave's tiles (or remainders) as one stream of load blocks, the
// worker count a run-time number (fused_many.hip, fused_stream.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "device.hpp"
#include "kernels.hpp"

namespace phub {

namespace {

// One run of up to 256 float4 of a key: a full tile or a remainder's whole
// float4s.
struct Unit {
    const float* const* row;  // the key's gradient pointers
    int64_t base;             // element of the state arenas that byte offset 0 stands for
    uint32_t vlo;             // float4 index of the unit's first, beside vhi
    uint32_t vhi;             // float4 index folded into the gradient bases
    uint32_t nvec;
};

// The units of a bin: its full tiles (DevTile) or its remainders (DevRem;
// those shorter than a float4 have no unit), each descriptor fetched one
// unit before its own is decoded.
template <typename DESC>
struct UnitList {
    const DESC* desc;
    int32_t i, end;  // the fetched descriptor's index, the bin's end
    DESC d;

    __device__ __forceinline__ void fetch() {
        if constexpr (sizeof(DESC) == sizeof(DevRem))
            while (i < end && desc[i].count < 4) ++i;
        if (i < end) d = desc[i];
    }
    __device__ __forceinline__ UnitList(const DESC* all, int32_t b, int32_t e)
        : desc(all), i(b), end(e) {
        fetch();
    }
    __device__ __forceinline__ bool more() const { return i < end; }
    __device__ __forceinline__ const float* const* row(const float* const* grads, int n) const {
        return grads + int64_t(d.key) * n;
    }
    __device__ __forceinline__ Unit take(const float* const* grads, int n) {
        Unit u;
        uint64_t vec;
        if constexpr (sizeof(DESC) == sizeof(DevRem)) {
            vec = uint64_t(d.offset) / 4;
            u.nvec = uint32_t(d.count) >> 2;
        } else {
            vec = d.vec;
            u.nvec = uint32_t(kTileElems / 4);
        }
        u.vlo = uint32_t(vec) & kVecLowMask;
        u.vhi = uint32_t(vec) & ~kVecLowMask;
        u.base = d.arena_offset - int64_t(u.vlo) * 4;
        u.row = row(grads, n);
        ++i;
        fetch();
        return u;
    }
};

// Byte offset of the lane's float4 of piece u; lanes past the unit's end
// repeat its last float4.
__device__ __forceinline__ uint32_t lane_off(const Unit& c, uint32_t u) {
    const uint32_t v = u * 64u + (threadIdx.x & 63u);
    return (c.vlo + (v < c.nvec ? v : c.nvec - 1)) * 16u;
}

// Gradient bases of the block whose first worker is w0, lane j holding
// worker w0 + j's (past the last worker, the last one's): one vector load,
// issued one block before its first use, so that it returns with the data
// loads issued around it.
template <int B>
__device__ __forceinline__ uint64_t block_pointers(const float* const* row, int w0, int n) {
    const int l = int(threadIdx.x & 63u);
    const int w = w0 + (l < B ? l : B - 1);
    return ((const PHUB_GLOBAL uint64_t*)row)[uint32_t(w < n ? w : n - 1)];
}

__device__ __forceinline__ const float* lane_base(uint64_t p, int j) {
    const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(p)), j));
    const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(p >> 32)), j));
    return reinterpret_cast<const float*>((uint64_t(hi) << 32) | lo);
}

// Burst write-back of the streamed tiles' state, as in tile_walk.hpp: a
// finished piece's state goes to a stash in LDS (P pieces per wave, lane l
// holding entry l of every 64), and the wave writes the stash back in one run
// of stores when the chip-wide write window is open (looked at after every
// block of loads), when the stash is full, or after its last piece.  Each
// lane reads back only what it wrote: no barrier.
template <int S>
struct Stash {
    PHUB_LDS f4* lds;  // the lane's entry of the wave's first piece
    uint32_t lo = 0;   // lane k: where piece k's state goes (element index
    uint32_t hi = 0;   // in the state arenas)
    int count = 0;

    __device__ __forceinline__ void put(const f4 (&st)[S], int64_t elem) {
        lo = lane == uint32_t(count) ? uint32_t(elem) : lo;
        hi = lane == uint32_t(count) ? uint32_t(uint64_t(elem) >> 32) : hi;
#pragma unroll
        for (int i = 0; i < S; ++i) lds[(count * S + i) * 64] = st[i];
        ++count;
    }
    template <bool RES>
    __device__ __forceinline__ void write_back(float* const* state) {
#pragma unroll
        for (int i = 0; i < S; ++i) {
            for (int k0 = 0; k0 < count; k0 += kVecPerLane) {
                f4 r[kVecPerLane];
#pragma unroll
                for (int k = 0; k < kVecPerLane; ++k) r[k] = lds[((k0 + k) * S + i) * 64];
#pragma unroll
                for (int k = 0; k < kVecPerLane; ++k) {
                    if (k0 + k < count) {
                        const uint32_t l = uint32_t(__builtin_amdgcn_readlane(int(lo), k0 + k));
                        const uint32_t h = uint32_t(__builtin_amdgcn_readlane(int(hi), k0 + k));
                        float* const a = state[i] + int64_t((uint64_t(h) << 32) | l);
                        if constexpr (RES)
                            store_wm<true>(a, lane * 16u, r[k]);
                        else
                            store_wb(a, lane * 16u, r[k]);
                    }
                }
            }
        }
        count = 0;
    }
    uint32_t lane = threadIdx.x & 63u;
};

template <int B, int OPT, bool RES, int P, typename DESC>
__device__ __forceinline__ void walk_units(const DESC* desc, int32_t begin, int32_t end,
                                           const float* const* grads, int n, float* const* state,
                                           OptArgs o, PHUB_LDS f4* stash_lds) {
    constexpr int S = kStates<OPT>;
    constexpr bool STASH = sizeof(DESC) == sizeof(DevTile);
    static_assert(P >= 1 && P <= 64 && P % kVecPerLane == 0, "a lane holds one piece's place");
    Stash<S> stash{stash_lds};
    UnitList<DESC> list(desc, begin, end);
    if (!list.more()) return;
    const int last = (n - 1) / B * B;  // first worker of the last block
    const int tail = n - last;         // its workers
    const uint32_t lane = threadIdx.x & 63u;
    Unit c = list.take(grads, n);
    f4 v[B];
    uint32_t u = 0;
    uint32_t off = lane_off(c, 0);
    uint64_t p = block_pointers<B>(c.row, 0, n) + uint64_t(c.vhi) * 16u;
    uint64_t q = block_pointers<B>(c.row, B, n);
#pragma unroll
    for (int j = 0; j < B; ++j) v[j] = load_stream(lane_base(p, j), off);
    f4 acc, st[S];
    auto load_state = [&]() {
#pragma unroll
        for (int i = 0; i < S; ++i) st[i] = load_wm<RES>(state[i] + c.base, off);
    };
    auto finish = [&](int64_t base, uint32_t vlo, uint32_t nvec, uint32_t u, uint32_t off) {
        update4<OPT, false>(acc, st, o);
        if constexpr (STASH) {
            stash.put(st, base + int64_t(vlo + u * 64u) * 4);
        } else if (u * 64u + lane < nvec) {
#pragma unroll
            for (int i = 0; i < S; ++i) store_wm<RES>(state[i] + base, off, st[i]);
        }
    };
    for (;;) {
        const bool same = (u + 1) * 64u < c.nvec;
        const bool has = same || list.more();
        acc = -0.0f;  // -0 + x is x, bit for bit
        // All but the last block: issue the next block of this piece.  p:
        // the bases of the block being issued; q: of the one after it.
        for (int w0 = 0; w0 < last; w0 += B) {
            if constexpr (STASH) {
                if (stash.count && (stash.count == P ||
                                    in_write_window(o.wb_period, o.wb_window)))
                    stash.template write_back<RES>(state);
            }
            p = q + uint64_t(c.vhi) * 16u;
            if (w0 + B < last)
                q = block_pointers<B>(c.row, w0 + 2 * B, n);
            else
                q = block_pointers<B>(same || !has ? c.row : list.row(grads, n), 0, n);
            // the loads of the next block past the last worker: one line only
            const int real = w0 + B < last ? B : tail;
            const uint32_t spare = uint32_t(__builtin_amdgcn_readfirstlane(int(off)));
#pragma unroll
            for (int j = 0; j < B; ++j) {
                acc = acc + v[j];
                asm volatile("" : "+v"(acc));  // keep the wait for load j here
                v[j] = load_stream(lane_base(p, j), j < real ? off : spare);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (!has) break;
        // The last block: issue the piece's state loads, then the first
        // block of the next piece.
        load_state();
        const int64_t base = c.base;
        const uint32_t vlo = c.vlo, nvec = c.nvec, pu = u, poff = off;
        if (!same) c = list.take(grads, n);
        u = same ? u + 1 : 0;
        off = lane_off(c, u);
        p = q + uint64_t(c.vhi) * 16u;
        q = block_pointers<B>(c.row, B, n);
#pragma unroll
        for (int j = 0; j < B; ++j) {
            const f4 sum = acc + v[j];
            acc = j < tail ? sum : acc;
            asm volatile("" : "+v"(acc));
            v[j] = load_stream(lane_base(p, j), off);
            __builtin_amdgcn_sched_barrier(0);
        }
        finish(base, vlo, nvec, pu, poff);
        __builtin_amdgcn_sched_barrier(0);
    }
    // the last block of the last piece
    load_state();
#pragma unroll
    for (int j = 0; j < B; ++j) {
        const f4 sum = acc + v[j];
        acc = j < tail ? sum : acc;
    }
    finish(c.base, c.vlo, c.nvec, u, off);
    if constexpr (STASH) stash.template write_back<RES>(state);
}

}  // namespace

}  // namespace phub
