// The K loop of a workgroup whose waves share pixel tiles (each wave has output channels of its own): gathered operands through LDS.
//
// A wave that gathers the MFMA operands of its own 32 pixels asks for 32 different lines per load instruction, which occupies the
// compute unit's vector memory path for 64 clocks per KB (device_utils.h, quad gathers), and waves that share a tile each fetch the same
// pixels: four waves on a 3x3 256->256 tile took 384 clocks a K-step, 256 of them for gathers.  Here a group of four K-steps -- a
// 128-byte line of one window tap -- is fetched ONCE per tile, its loads dealt over the SH waves that share it and every quad
// of lanes on one line (16 clocks a load), and left in LDS in operand order: 16 clocks of gathers a K-step and tile for all of
// them, and no vector instructions to deal the vectors out.  LDS holds two groups: while one is multiplied the next is stored, and the
// vectors of RD further ones are in registers or on their way.  Weights come straight from L2, WS K-steps ahead, each in place of the one just
// multiplied.  One workgroup barrier per group where tiles are
// shared, so all waves walk the union of the workgroup's window taps.
#pragma once

#include "conv_plan.h"
#include "kstep.h"

namespace dcnn {

// A layer's weights into the L2 of every XCD while its list is formed: each workgroup touches a share of their 64-byte pieces (8 rounds: 1 MB of
// weights on the 64 workgroups of a small map).  Workgroups on short lists all walk the weights in the same order, so without it they share one stream of
// misses.  It asks before the list's length is known, for a list that may be empty: a ResNet-50-shaped step of 8 streams takes 1032 us without it, 1023
// with it and 1040 where it waits for the length; of a still scene 367, 370 and 368.  Layers stepped alone, whose weights are in L2, no flags / 1 / 2 / 10 %,
// without -> with: 3x3 256->256 + ReLU on 8 streams of 16x16 35.8 / 38.4 / 39.2 / 40.0 -> 33.9 / 38.6 / 39.5 / 40.1, 128->64 on 8 of 128x128 35.2 / 40.4 / 44.6 / 60.7 ->
// 33.3 / 40.6 / 44.5 / 60.5.  Pieces of 128 bytes, half as many, and leaving without a wait where the list is empty: the same times.
struct WarmL2 {
    static constexpr int kRounds = 8;
    uint32_t v[kRounds];
    template <int NT> __device__ __forceinline__ void request(const void* p, uint64_t bytes) {
        const __amdgpu_buffer_rsrc_t rs = ws_rsrc(p, bytes);
        const uint32_t n = gridDim.x / kXcd > 0 ? gridDim.x / kXcd : 1, i = blockIdx.x / kXcd, pieces = (uint32_t)(bytes / 64);
#pragma unroll
        for (int k = 0; k < kRounds; ++k) {
            const uint32_t first = ((uint32_t)k * n + i) * NT, at = first + threadIdx.x;
            v[k] = 0;
            if (first < pieces) v[k] = __builtin_amdgcn_raw_buffer_load_b32(rs, at < pieces ? (int)(at * 64u) : (int)kOob, 0, 0);
        }
    }
    __device__ __forceinline__ void arrived() {
#pragma unroll
        for (int k = 0; k < kRounds; ++k) asm volatile("" ::"v"(v[k]));
    }
};

constexpr int kGatherGroup = 4;                                // K-steps of a group
constexpr int kGatherTile = kGatherGroup * kWave * 16;         // bytes of one tile's group: [K-step][half][pixel ^ K-step][16]

// loads per wave and group; load i of wave `part` fetches pixel 4 * (lane % 32 / 4) + gather_pixel(i) of tile gather_tile(i)
template <int TI, int SH> struct GatherShare {
    static constexpr int kLoads = TI * kGatherGroup / SH;
    static constexpr int kWords = (kLoads + 2) / 3;            // tap words of up to nine bits, three to a register
    static_assert(TI * kGatherGroup % SH == 0, "loads dealt out evenly");
    static __device__ __forceinline__ int tile(int part, int i) { return (part * kLoads + i) / kGatherGroup; }
    static __device__ __forceinline__ int pixel(int part, int i) { return (part * kLoads + i) % kGatherGroup; }
};

// What a wave multiplies: acc[ti][b] += W[column block b] * X[tile ti] over the taps of `taps` (the workgroup's union, in ascending order).
// base / need: byte offset of window tap (0,0) and tap word of the pixels this wave fetches; wlane: this lane's place in the wave's first
// K-step; buf: [2][TI][kGatherTile] of the SH waves; mine: false for a wave without pixels, which only keeps the barriers.
template <typename T, int NB, int KS, int TI, int SH, int RD, int WS>
__device__ __forceinline__ void gather_tiles(f32x16 (&acc)[TI][NB], __amdgpu_buffer_rsrc_t rs_in, __amdgpu_buffer_rsrc_t rs_w,
                                             const uint32_t (&base)[GatherShare<TI, SH>::kLoads], const uint32_t (&need)[GatherShare<TI, SH>::kWords],
                                             uint32_t taps, int kch, int cin_bytes, int line_bytes, uint32_t wlane, uint32_t wstep,
                                             unsigned char* buf, int part, int lane, bool mine) {
    typedef typename Mma<T>::Vec Vec;
    constexpr int N = GatherShare<TI, SH>::kLoads, GK = kGatherGroup, kNoTap = 31;
    static_assert(RD * GK % WS == 0, "weights in step with the unrolled groups");
    const int kgroups = (kch + GK - 1) / GK;
    const int groups = __popc(taps) * kgroups;
    if (groups == 0) return;
    auto sync = [&]() __attribute__((always_inline)) {         // (a wave with tiles of its own waits for nobody)
        if constexpr (SH == 1) lds_wave_sync(); else lds_block_sync();
    };
    if (!mine) {
        if constexpr (SH > 1)
            for (int s = 0; s <= groups; ++s) sync();
        return;
    }
    const int g = lane / 32, r = lane % 4;
    const uint32_t place = (uint32_t)(r * 32 + g * 16);
    // (one wave per SIMD waits for its own instructions: cursors move once per group, by selects)
    struct Cur { uint32_t rest; int t, kg; };                  // t == kNoTap: past the end
    auto advance = [&](Cur& cu) __attribute__((always_inline)) {
        const bool wrap = cu.kg + 1 == kgroups;
        cu.kg = wrap ? 0 : cu.kg + 1;
        cu.rest = wrap ? cu.rest & (cu.rest - 1) : cu.rest;
        cu.t = __builtin_ctz(cu.rest | 1u << kNoTap);
    };
    // Every load is issued unconditionally: a pixel whose tap is not flagged, channel padding and groups past the end read zeros from
    // an offset outside the descriptor.
    auto request_x = [&](const Cur& cu, Vec (&x)[N]) __attribute__((always_inline)) {
        const bool live = cu.t != kNoTap;
        const int t = live ? cu.t : 0, dy = t / KS, dx = t - dy * KS;
        const uint32_t at = (uint32_t)(dy * line_bytes + dx * cin_bytes + cu.kg * (GK * 32)) + place;
        const uint32_t tbit = live && (int)place < cin_bytes - cu.kg * (GK * 32) ? 1u << t : 0u;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            uint32_t off = (need[i / 3] & (tbit << (9 * (i % 3)))) ? base[i] + at : kOob;
            asm volatile("" : "+v"(off));                      // one load at a computed offset, not a load per case
            x[i] = ws_load16<Vec>(rs_in, off);
        }
    };
    auto request_w = [&](const Cur& cu, int u, Vec (&w)[NB]) __attribute__((always_inline)) {
        const int kc = cu.kg * GK + u;                         // (a group's last steps may be padding, which meets zeros)
        const uint32_t voff = kc < kch ? wlane : kOob, soff = (uint32_t)weight_step(cu.t == kNoTap ? 0 : cu.t, kch, kc) * wstep;
#pragma unroll
        for (int b = 0; b < NB; ++b) w[b] = ws_load16<Vec>(rs_w, voff + (uint32_t)b * (32u * 16u), soff);
    };
    // (pixel p of K-step u lies at p ^ u: the four lanes of a quad write to four bank groups)
    const int first = part * N;
    unsigned char* put = buf + (size_t)(first / GK) * kGatherTile + (r * kWave + g * 32 + ((lane % 32 / 4 * 4 + first % GK) ^ r)) * 16;
    constexpr uint32_t kFlip = (uint32_t)TI * kGatherTile;
    auto store_x = [&](uint32_t half, const Vec (&x)[N]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uintptr_t at = (uintptr_t)(put - buf);       // (buf is a multiple of 128 bytes into LDS)
            *reinterpret_cast<Vec*>(buf + half + ((at ^ (uintptr_t)(i % GK * 16)) + (size_t)(i / GK) * kGatherTile)) = x[i];
        }
    };

    Vec x[RD][N], w[WS][NB];
    Cur cx{taps, __builtin_ctz(taps), 0};
    Cur cw = cx;
#pragma unroll
    for (int d = 0; d < RD; ++d) { request_x(cx, x[d]); advance(cx); }
    __builtin_amdgcn_sched_barrier(0);                         // (loads in the order of their use: a wait counts those behind it)
#pragma unroll
    for (int d = 0; d < WS; ++d) {
        request_w(cw, d % GK, w[d]);
        if (d % GK == GK - 1) advance(cw);
        __builtin_amdgcn_sched_barrier(0);
    }
    store_x(0, x[0]);
    request_x(cx, x[0]); advance(cx);
    sync();
    uint32_t half = 0;
    auto group = [&](auto jc) __attribute__((always_inline)) {
        constexpr int j = decltype(jc)::value;
        store_x(half ^ kFlip, x[(j + 1) % RD]);
        request_x(cx, x[(j + 1) % RD]); advance(cx);
        __builtin_amdgcn_sched_barrier(0);
        // operands in the order of their use, requested AHEAD of it (one tile: the whole group at once), K-step by K-step
        constexpr int Q = GK * TI, AHEAD = TI == 1 ? GK : 2;
        auto operand = [&](int q) { return *reinterpret_cast<const Vec*>(buf + half + q % TI * kGatherTile + q / TI * (kWave * 16) + ((lane ^ (q / TI)) * 16)); };
        Vec v[AHEAD];
#pragma unroll
        for (int q = 0; q < AHEAD; ++q) v[q] = operand(q);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int u = q / TI, ti = q % TI;
#pragma unroll
            for (int b = 0; b < NB; ++b) Mma<T>::run(acc[ti][b], w[(j * GK + u) % WS][b], v[q % AHEAD]);
            if (q + AHEAD < Q) v[q % AHEAD] = operand(q + AHEAD);
            if (ti == TI - 1) {
                request_w(cw, (u + WS) % GK, w[(j * GK + u) % WS]);
                if ((u + WS) % GK == GK - 1) advance(cw);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        half ^= kFlip;
        sync();
    };
    // (no way out of the middle of the loop: with one the compiler's waits at its head left half as many loads in flight)
    int s = 0;
    for (; s + RD <= groups; s += RD) {
        group(std::integral_constant<int, 0>{});
        if constexpr (RD > 1) {
            static_assert(RD == 1 || RD == 4);
            group(std::integral_constant<int, 1>{});
            group(std::integral_constant<int, 2>{});
            group(std::integral_constant<int, 3>{});
        }
    }
    if constexpr (RD > 1) {
        if (s < groups) group(std::integral_constant<int, 0>{});
        if (s + 1 < groups) group(std::integral_constant<int, 1>{});
        if (s + 2 < groups) group(std::integral_constant<int, 2>{});
    }
}

}  // namespace dcnn
