// The dense first frame of a convolution with dense weights: an implicit GEMM over every output pixel, with bias, the
// optional residual or projection of a second input, and the first-frame form of the activation (x^A <- v, x^T <- 0, output
// f(v); Fig. 2).  No pixel is decided on, so the output channels need not meet and the work splits freely over
// pixels AND channels -- which is what the sparse kernels, whose tail wants the whole pixel, cannot do.
//
// A wave owns 64 pixels x 64 output channels (2 x 2 MFMA 32x32 blocks; x 32 where the last tile would be half empty or compute units idle:
// first_narrow, first_halves), operands straight from global memory / L2 into registers.  Four K-steps of a pixel -- a 128-byte line of one
// tap -- are fetched by quads of lanes (quad_transpose: a load instruction then takes 16 clocks of the memory path instead of 64, and
// the gathers of a K-step 32 beside 32 of weights instead of 128).  Once a group's vectors are dealt out the next group's travel in
// their place, and its weights in place of each K-step's as it is multiplied: 64 sums, 64 vectors of pixels and 32 of weights fit two
// waves per SIMD (two whole sets of both spilled: 64->64 on 64 streams of 128x128 3x3 478 us, not 223).  With enough such
// tiles the four waves of a workgroup take four pixel tiles of the same channels (they share the weights in the
// vector cache); with too few -- the deep stages of a backbone: 512 pixels, K = 4608 -- they split the K-steps of ONE
// tile and add their partial sums in LDS in a fixed order.
// Bound: 64 streams of 128x128, 64->256 with its projection, x^A and O (rows of x^T that hold zeros stay): 1.07 GB written and 0.27 GB read in
// 480 us, 2.8 TB/s of the 5.3 that a copy reaches -- sums of one group leave nothing to ask for ahead, so a tile's operands, the projection's and its
// stores follow each other on two waves per SIMD.  Memory latency for the deep layers.  Kernels with a lane per pixel and a ring of four
// K-steps -> quads, us: 3x3 256->256 on 8 streams of 64x64 104 -> 64, 512->512 on 512 pixels 29 -> 17, 1x1 64->64 and 3x3 64->64 on 64
// streams of 128x128 together 321 -> 255.
#include "conv_plan.h"
#include "kstep.h"

namespace dcnn {

constexpr int kFirstWaves = 4;
constexpr int kFirstPx = 64;                                   // tile of a wave: pixels; its channels are 32 * TC
constexpr int kFirstGroup = 4;                                 // K-steps whose operands are requested together (quad_transpose); two groups in registers or on their way
constexpr int kFirstRing = 4;                                  // where every lane fetches its own pixel: K-steps in registers or on their way

struct FirstArgs {
    int nb;                        // column blocks per packed channel group (the layer's plan)
    int ngroups;                   // packed channel groups
    int wc;                        // waves of a workgroup side by side over the channels (1, 2 or 4), the others over pixels
    int cgroups;                   // channel tiles per pixel, in groups of wc
    int64_t units;                 // workgroups: groups of pixel tiles x groups of channel tiles
    int64_t pixels;
    const void* bias2;             // bias of the projection
};

template <typename T> constexpr int first_stage_stride(int channels) { return channels * (int)sizeof(T) + kStagePad; }

// STEPS: K-steps of a tap's group that can hold channels.  4 or 2 (rows of up to 64 bytes): a group is a 128-byte line of one tap.
// 1: single K-steps, of which every lane fetches its own pixel's 16 bytes, kFirstRing of them in registers or on their way: three waves per SIMD
// instead of two, and none of the work on the padding of a group (first_by_lanes has the rule and both sides of it).
template <typename T, int SPLIT, int TC, bool XT, int STEPS>
__global__ __launch_bounds__(kFirstWaves* kWave, 2) void conv_first_kernel(ConvArgs c, EpilogueArgs e, FirstArgs f) {
    typedef typename Mma<T>::Vec Vec;
    constexpr int V = Elem<T>::VEC;
    typedef typename RawOf<T, V>::type Raw;
    constexpr int ES = (int)sizeof(T);
    constexpr int TP = kFirstPx / 32, kFirstCh = TC * 32;
    constexpr int stage_stride = first_stage_stride<T>(kFirstCh);
    static_assert(SPLIT == 1 || SPLIT == kFirstWaves, "one tile per wave or one tile per workgroup");
    static_assert(SPLIT == 1 || TP * TC <= kFirstWaves, "after a split a wave sums one block");
    extern __shared__ __align__(16) unsigned char smem[];

    // One tile per wave: pixel groups in launch order, the channel groups of one behind each other on one XCD (workgroup b runs
    // on XCD b % 8): they gather the same pixels and, where rows are no multiple of a cache line, write parts of the same lines
    // (8 streams of 128x128, 1x1 256->320: 99 us with the channel groups on different XCDs, now 70).  (A contiguous eighth of the
    // pixels per XCD spreads the eight fronts over memory a power of two apart: 563 -> 530 us for the layer above without it.)
    // One tile per workgroup: the XCDs do take an eighth each, so that a weight slice is fetched by few L2s.
    const int64_t in_xcd = blockIdx.x / kXcd, xcd = blockIdx.x % kXcd;
    const int64_t per = (f.units + kXcd - 1) / kXcd;
    const int64_t unit = SPLIT == 1 ? (in_xcd / f.cgroups * kXcd + xcd) * f.cgroups + in_xcd % f.cgroups : xcd * per + in_xcd;
    if ((SPLIT != 1 && in_xcd >= per) || unit >= f.units) return;   // uniform for the workgroup
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int col = lane % 32, g = lane / 32;
    const uint32_t place = (uint32_t)(lane % 4) * 32u + (uint32_t)g * 16u;   // this lane's 16 bytes of a group, load 0
    const int64_t pg = unit / f.cgroups;
    const int cg = (int)(unit - pg * f.cgroups);
    const int64_t pt = SPLIT == 1 ? pg * (kFirstWaves / f.wc) + wave / f.wc : pg;
    const int ct = SPLIT == 1 ? cg * f.wc + wave % f.wc : cg;
    const int64_t px0 = pt * kFirstPx;
    const int ch0 = ct * kFirstCh;
    if (SPLIT == 1 && (px0 >= f.pixels || ch0 >= e.c)) return;   // (no workgroup barrier below in this case)
    const int cols = f.nb * 32;
    // x^T row flags of the tile's pixels, one per lane: rows that hold zeros already are not written again
    static_assert(kFirstPx == kWave, "a pixel's flag per lane");
    int xt_row = 1;
    if constexpr (XT) xt_row = e.xt_flags[px0 + lane < f.pixels ? px0 + lane : px0];

    // the lane's pixels: origin of their windows
    struct Px { int iy0, ix0; uint32_t base, base2; bool on; };
    Px px[TP];
    const int cin_bytes = c.cin * ES, cin2_bytes = c.cin2 * ES;
#pragma unroll
    for (int i = 0; i < TP; ++i) {
        const int64_t p = px0 + i * 32 + col;
        px[i].on = p < f.pixels;
        const uint32_t pu = px[i].on ? (uint32_t)p : 0u;
        const uint32_t t1 = fast_div(pu, c.div_ow);
        const int ox = (int)(pu - t1 * (uint32_t)c.ow);
        const uint32_t n = fast_div(t1, c.div_oh);
        const int oy = (int)(t1 - n * (uint32_t)c.oh);
        px[i].iy0 = px[i].on ? oy * c.stride - c.pad : INT32_MIN / 2;   // (off: outside the map at every tap)
        px[i].ix0 = ox * c.stride - c.pad;
        px[i].base = (uint32_t)(((int)n * c.h + oy * c.stride - c.pad) * c.w + px[i].ix0) * (uint32_t)cin_bytes;
        px[i].base2 = (uint32_t)(((int)n * c.h2 + oy * c.stride2) * c.w2 + ox * c.stride2) * (uint32_t)cin2_bytes;
    }
    // column blocks of the tile in the packed weights (a block past the last one repeats it; its channels are not stored)
    auto block_of = [&](int b) {
        const int cb = ch0 / 32 + b, last = f.ngroups * f.nb - 1;
        return cb < last ? cb : last;
    };

    f32x16 acc[TP][TC];
    auto zero_acc = [&]() {
#pragma unroll
        for (int i = 0; i < TP; ++i)
#pragma unroll
            for (int b = 0; b < TC; ++b)
#pragma unroll
                for (int q = 0; q < 16; ++q) acc[i][b][q] = 0.0f;
    };
    // acc += window of `data` x packed weights, over this wave's share of the groups of K-steps.  `proj`: the 1x1 second input.
    auto k_loop = [&](auto pc) __attribute__((always_inline)) {
        constexpr bool proj = decltype(pc)::value;
        const int ksz = proj ? 1 : c.k, kch = proj ? c.kch2 : c.kch;
        const int rowb = proj ? cin2_bytes : cin_bytes, iw = proj ? c.w2 : c.w;
        const int ksteps = ksz * ksz * kch;
        const __amdgpu_buffer_rsrc_t rs_in = proj ? ws_rsrc(c.in2_data, (uint64_t)c.n * c.h2 * c.w2 * cin2_bytes)
                                                  : ws_rsrc(c.in_data, (uint64_t)c.n * c.h * c.w * cin_bytes);
        const __amdgpu_buffer_rsrc_t rs_w = ws_rsrc(proj ? c.wpacked2 : c.wpacked, (uint64_t)f.ngroups * ksteps * 2 * cols * 16);
        uint32_t wlane[TC];
#pragma unroll
        for (int b = 0; b < TC; ++b) {
            const int cb = block_of(b);
            wlane[b] = ((uint32_t)(cb / f.nb) * (uint32_t)ksteps * 2u * (uint32_t)cols + (uint32_t)g * (uint32_t)cols +
                        (uint32_t)(cb % f.nb) * 32u + (uint32_t)col) * 16u;
        }
        const uint32_t wrow = (uint32_t)(2 * cols * 16);       // weights of one K-step
        const int share = SPLIT == 1 ? 0 : wave;
        const int k_first = (int)((int64_t)ksteps * share / SPLIT), k_last = (int)((int64_t)ksteps * (share + 1) / SPLIT);
        if (k_first == k_last) return;
        if constexpr (STEPS == 1) {
            constexpr int D = kFirstRing;
            int s_next = k_first, kc, dy, dx;                  // the K-step to ask for
            {
                const int tap = k_first / kch;
                kc = k_first - tap * kch;
                dy = tap / ksz; dx = tap - dy * ksz;
            }
            // Every load is issued unconditionally: a pixel outside the map, padding channels and steps past the end read zeros
            // from an offset outside the descriptor, so the number of loads in flight at each wait is known.
            auto issue = [&](Vec (&x)[TP], Vec (&w)[TC]) __attribute__((always_inline)) {
                const bool live = s_next < k_last;
                const bool chan_ok = live && (2 * kc + g) * 16 < rowb;
                const uint32_t uni = (uint32_t)((dy * iw + dx) * rowb + kc * 32 + g * 16);
#pragma unroll
                for (int i = 0; i < TP; ++i) {
                    const bool in = (unsigned)(px[i].iy0 + dy) < (unsigned)c.h && (unsigned)(px[i].ix0 + dx) < (unsigned)c.w;
                    uint32_t off = chan_ok && in ? px[i].base + uni : kOob;
                    asm volatile("" : "+v"(off));
                    x[i] = ws_load16<Vec>(rs_in, off);
                }
                const uint32_t step = (uint32_t)weight_step(0, k_last, s_next) * wrow;
#pragma unroll
                for (int b = 0; b < TC; ++b) w[b] = ws_load16<Vec>(rs_w, live ? wlane[b] : kOob, step);
                ++s_next;
                if (++kc == kch) {
                    kc = 0;
                    if (++dx == ksz) { dx = 0; ++dy; }
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            Vec x[D][TP], w[D][TC];
#pragma unroll
            for (int j = 0; j < D - 1; ++j) issue(x[j], w[j]);
            for (int s = k_first; s < k_last; s += D) {
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    issue(x[(j + D - 1) % D], w[(j + D - 1) % D]);
#pragma unroll
                    for (int b = 0; b < TC; ++b)
#pragma unroll
                        for (int i = 0; i < TP; ++i) Mma<T>::run(acc[i][b], w[j][b], x[j][i]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            return;
        }
        // The groups that hold this wave's K-steps (a group at either end may hold another wave's too).
        const int kgroups = (kch + kFirstGroup - 1) / kFirstGroup;
        auto group_of = [&](int k) { return k / kch * kgroups + k % kch / kFirstGroup; };
        const int first = group_of(k_first), last = group_of(k_last - 1) + 1;
        int kg, dy, dx;
        {
            const int tap = k_first / kch;
            kg = k_first % kch / kFirstGroup;
            dy = tap / ksz; dx = tap - dy * ksz;
        }
        struct Part { int lo, hi; };                           // the K-steps of the current group that are this wave's
        auto part_of = [&]() {
            const int base = (dy * ksz + dx) * kch + kg * kFirstGroup, end = kch - kg * kFirstGroup;
            if constexpr (SPLIT == 1) return Part{0, end};
            return Part{k_first - base, min(k_last - base, end)};
        };
        // Every load is issued unconditionally: a pixel outside the map and padding channels read zeros from an offset outside
        // the descriptor, so the number of loads in flight at each wait is known.
        Vec x[TP][kFirstGroup], w[STEPS][TC];
        auto request_x = [&]() __attribute__((always_inline)) {
            const int left = rowb - kg * (kFirstGroup * 32);
            const uint32_t uni = (uint32_t)((dy * iw + dx) * rowb + kg * (kFirstGroup * 32));
#pragma unroll
            for (int i = 0; i < TP; ++i) {
                uint32_t off;
                if constexpr (proj) off = px[i].on ? px[i].base2 + uni : kOob;
                else off = ((unsigned)(px[i].iy0 + dy) < (unsigned)c.h && (unsigned)(px[i].ix0 + dx) < (unsigned)c.w) ? px[i].base + uni : kOob;
                auto load = [&](auto jc) __attribute__((always_inline)) {
                    constexpr int J = decltype(jc)::value;
                    const uint32_t at = quad_place<J>(place, 32u);
                    uint32_t o = quad_bcast<J>(off) + at;
                    o = (int)at < left ? o : kOob;
                    asm volatile("" : "+v"(o));                // one load at a computed offset, not a load per case
                    x[i][J] = ws_load16<Vec>(rs_in, o);
                };
                load(std::integral_constant<int, 0>{}); load(std::integral_constant<int, 1>{});
                load(std::integral_constant<int, 2>{}); load(std::integral_constant<int, 3>{});
            }
        };
        auto request_w = [&](int u) __attribute__((always_inline)) {
            const int at = kg * kFirstGroup + u;
            const uint32_t step = (uint32_t)weight_step(dy * ksz + dx, kch, at) * wrow;
#pragma unroll
            for (int b = 0; b < TC; ++b) w[u][b] = ws_load16<Vec>(rs_w, at < kch ? wlane[b] : kOob, step);
        };
        auto mma = [&](int u, const Part& part, const Vec (&v)[TP][kFirstGroup]) __attribute__((always_inline)) {
            if (SPLIT != 1 && (u < part.lo || u >= part.hi)) return;
            if (SPLIT == 1 && STEPS == kFirstGroup && u > 0 && u >= part.hi) return;   // (a group's last steps may be padding, which meets zeros)
#pragma unroll
            for (int b = 0; b < TC; ++b)
#pragma unroll
                for (int i = 0; i < TP; ++i) Mma<T>::run(acc[i][b], w[u][b], v[i][u]);
        };
        request_x();
#pragma unroll
        for (int u = 0; u < STEPS; ++u) request_w(u);
        for (int s = first + 1; s < last; ++s) {
            // the next group's pixels take the place of the vectors as fetched, its weights that of the ones just multiplied
            Vec xt[TP][kFirstGroup];
#pragma unroll
            for (int i = 0; i < TP; ++i) {
                quad_transpose(x[i], lane);
#pragma unroll
                for (int u = 0; u < kFirstGroup; ++u) xt[i][u] = x[i][u];
            }
            const Part part = part_of();
            if (++kg == kgroups) {
                kg = 0;
                if (++dx == ksz) { dx = 0; ++dy; }
            }
            request_x();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < STEPS; ++u) {
                mma(u, part, xt);
                request_w(u);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int i = 0; i < TP; ++i) quad_transpose(x[i], lane);
        const Part part = part_of();
#pragma unroll
        for (int u = 0; u < STEPS; ++u) mma(u, part, x);
    };

    // staging tile [pixel][channel] in the storage type: one per wave, or one for the workgroup behind the partial sums
    unsigned char* stage = smem + (SPLIT == 1 ? (size_t)wave * kFirstPx * stage_stride : (size_t)kFirstWaves * TP * TC * 4 * kWave * 16);
    f32x4* partial = reinterpret_cast<f32x4*>(smem);
    // sums (+ bias) of one 32x32 block -> rounded to the storage type -> staging tile; with `add` onto what it holds
    typedef T Quad __attribute__((ext_vector_type(4)));
    auto stage_block = [&](const f32x16& a, int i, int b, const T* bias, bool add) __attribute__((always_inline)) {
        unsigned char* row = stage + (size_t)(i * 32 + col) * stage_stride;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int ch = ch0 + b * 32 + 8 * q + 4 * g;       // (channels are a multiple of 4: all four exist or none)
            Quad* dst = reinterpret_cast<Quad*>(reinterpret_cast<T*>(row) + b * 32 + 8 * q + 4 * g);
            Quad bv, v, old;
#pragma unroll
            for (int k = 0; k < 4; ++k) { bv[k] = (T)0.0f; old[k] = (T)0.0f; }
            if (bias != nullptr && ch < e.c) bv = *reinterpret_cast<const Quad*>(bias + ch);
            if (add) old = *dst;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[k] = (T)(a[4 * q + k] + (float)bv[k]);
                if (add) v[k] = (T)((float)old[k] + (float)v[k]);
            }
            *dst = v;
        }
    };
    auto deliver = [&](const T* bias, bool add) __attribute__((always_inline)) {
        if constexpr (SPLIT == 1) {
#pragma unroll
            for (int i = 0; i < TP; ++i)
#pragma unroll
                for (int b = 0; b < TC; ++b) stage_block(acc[i][b], i, b, bias, add);
        } else {
            // partial sums meet in LDS: wave w adds block w of all waves, in wave order
#pragma unroll
            for (int i = 0; i < TP; ++i)
#pragma unroll
                for (int b = 0; b < TC; ++b)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        f32x4 v;
#pragma unroll
                        for (int k = 0; k < 4; ++k) v[k] = acc[i][b][4 * q + k];
                        partial[((wave * (TP * TC) + i * TC + b) * 4 + q) * kWave + lane] = v;
                    }
            lds_block_sync();
            if (wave < TP * TC) {
                f32x16 sum;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    f32x4 v = partial[(wave * 4 + q) * kWave + lane];
#pragma unroll
                    for (int o = 1; o < kFirstWaves; ++o) {
                        const f32x4 u = partial[((o * (TP * TC) + wave) * 4 + q) * kWave + lane];
#pragma unroll
                        for (int k = 0; k < 4; ++k) v[k] += u[k];
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) sum[4 * q + k] = v[k];
                }
                stage_block(sum, wave / TC, wave % TC, bias, add);
            }
            lds_block_sync();                                  // (the partial sums may be overwritten, the staged tile may be read)
        }
    };

    zero_acc();
    k_loop(std::false_type{});
    deliver(static_cast<const T*>(e.bias), false);
    if (STEPS != 1 && c.in2_data != nullptr) {                 // the projection: rounded on its own, then added
        zero_acc();
        k_loop(std::true_type{});
        deliver(static_cast<const T*>(f.bias2), true);
    }
    lds_wave_sync();

    // tail: the tile's channels of a pixel are NV vectors, neighbouring lanes hold neighbouring vectors
    constexpr int NV = kFirstCh / V;
    constexpr int NLANES = SPLIT == 1 ? kWave : kFirstWaves * kWave;
    constexpr int PPI = NLANES / NV, NIT = kFirstPx / PPI;
    const int me = SPLIT == 1 ? lane : (int)threadIdx.x;
    const int sub = me % NV, grp = me / NV;
    const int ch = ch0 + sub * V;
    const bool stateful = e.act != DCNN_ACT_NONE;
    Raw lo_v, hi_v;
#pragma unroll
    for (int k = 0; k < V; ++k) { lo_v[k] = (T)0.0f; hi_v[k] = (T)act_hi(e.act); }
    const T* res = static_cast<const T*>(e.res_data);
    T* xA = static_cast<T*>(e.xA);
    T* xT = static_cast<T*>(e.xT);
    T* out = static_cast<T*>(e.out_data);
    const bool ch_on = ch < e.c;                               // (channels are a multiple of V; the flags are handed on by all lanes)
    constexpr int HB = NIT < 8 ? NIT : 8;                      // residual rows requested together
#pragma unroll
    for (int it0 = 0; it0 < NIT; it0 += HB) {
        Raw rr[HB];
        int xt_on[HB];
#pragma unroll
        for (int h = 0; h < HB; ++h) {
            const int64_t p = px0 + (it0 + h) * PPI + grp;
            xt_on[h] = XT ? __shfl(xt_row, (it0 + h) * PPI + grp, kWave) : 1;
            rr[h] = raw_zero<T, V>();
            if (res != nullptr && p < f.pixels && ch_on) rr[h] = raw_load<T, V>(res + p * e.c + ch);
        }
#pragma unroll
        for (int h = 0; h < HB; ++h) {
            const int row = (it0 + h) * PPI + grp;
            const int64_t p = px0 + row;
            if (p >= f.pixels || !ch_on) continue;
            const Raw d0 = raw_load<T, V>(reinterpret_cast<const T*>(stage + (size_t)row * stage_stride) + sub * V);
            Raw o_a = d0;
            if (res != nullptr) {
#pragma unroll
                for (int k = 0; k < V; ++k) raw_set<T, V>(o_a, k, raw_get<T, V>(d0, k) + raw_get<T, V>(rr[h], k));
            }
            // f of a stored value is exact in the storage type: clamped there, two elements an instruction in fp16
            const Raw o_y = stateful ? __builtin_elementwise_min(__builtin_elementwise_max(o_a, lo_v), hi_v) : o_a;
            const int64_t off = p * e.c + ch;
            if (stateful) {
                __builtin_nontemporal_store(o_a, reinterpret_cast<Raw*>(xA + off));
                if (xT != nullptr && xt_on[h]) __builtin_nontemporal_store(raw_zero<T, V>(), reinterpret_cast<Raw*>(xT + off));
            }
            raw_store<T, V>(out + off, o_y);
        }
    }
}

// Input bytes of one stream that a launch must reach with 32-bit offsets.
static uint64_t first_stream_bytes(size_t es, const ConvArgs& c) {
    const uint64_t a = (uint64_t)c.h * c.w * c.cin * es, b = c.in2_data ? (uint64_t)c.h2 * c.w2 * c.cin2 * es : 0;
    return a > b ? a : b;
}

// The waves of a workgroup share a tile's K-steps where ONE stream has fewer tiles than the chip has compute units (256) and K
// is long enough to be worth cutting.  The number of streams stays out of the rule on purpose: the order of the sum
// must not depend on it (a stream gives the same bits alone and in a batch).  Measured against the sum in one chain over 80
// shapes: the distance from the 64-bit result is the same in fp16 (rounding to storage) and half as large in fp32.
static bool first_splits(const ConvArgs& c) {
    return cdiv((int64_t)c.oh * c.ow, kFirstPx) * cdiv(c.cout, 64) < 256 && c.k * c.k * c.kch >= 8 * kFirstWaves;
}
// Tiles of 32 channels for layers of up to 32: the other half of a tile of 64 would be padding (fp32, 4 streams of 128x128, 32
// channels: 5x5 128->32 240 us, now 154, plain kernel 178).
static bool first_narrow(const ConvArgs& c) { return c.cout <= 32; }

// Whole long sums whose workgroups (tiles of 64 channels) fill at least half of the compute units, one each.
constexpr int kFirstLongSum = 45;                              // K-steps; see first_halves for both sides
static bool first_single(const ConvArgs& c, int64_t workgroups, int num_cu) {
    return workgroups > num_cu / 2 && workgroups <= num_cu && c.k * c.k * c.kch >= kFirstLongSum;
}

// Where every lane fetches its own pixel (STEPS 1) instead of a quad of lanes a line: where much of a line is nothing, and where a third wave per
// SIMD hides more than the quads save.  First frames of one layer with its input layer, MI355X, us, quads -> lanes:
// * windows over few channels: on 16 streams of 128x128 3x3 24->24 31.2 -> 25.5, 24->64 46.5 -> 40.8, 40->64 51 -> 49, 16->256 91 -> 80; on 12 of 120x128
//   5x5 24->96 95 -> 78, 7x7 24->256 260 -> 219.  Not for whole K-steps (3x3 32->96 65 -> 72) nor 40 channels to one block (3x3 40->32 27.6 -> 29.7).
// * `padded` lines, a K-step in four and more empty: split sums over 3x3 on 4 of 64x66 72->64 17.4 -> 16.5, 72->128 24.3 -> 23.6, and whatever the
//   window where no compute unit has two workgroups: 5x5 72->96 on 2 of 60x50 20.1 -> 17.2 (but 5x5 72->96 on 4 of 64x66 35.9 -> 37.7).
//   fp32, whose sums the matrix cores bound and whose quads only add to: 5x5 36->64 35.7 -> 31.3, 100->64 66 -> 61, 3x3 52->64 23.5 -> 21.5.
// * wide fp16 layers, whose stores want the third wave: on 12 of 120x128 1x1 40->192 49.8 -> 45, 72->512 201 -> 188, 96->512 324 -> 314, 3x3 72->256
//   182 -> 163, 48->512 383 -> 353, 5x5 48->256 224 -> 199; and 1x1 layers whose workgroups are one round of three per compute unit but
//   not of two: 56->64 28.9 -> 27.5, 96->64 36.3 -> 34.6.  (Not 3x3 72->128 nor 56->192: 100.7 and 111 by quads, 101 and 122.)
static bool first_by_lanes(const ConvArgs& c, size_t es, bool split, int64_t tiles, int num_cu) {
    if (c.in2_data != nullptr) return false;
    const int kch = c.kch, kgroups = (int)cdiv(kch, kFirstGroup);
    const bool half_words = es == 2, padded = kFirstGroup * kgroups - kch >= kgroups;
    if (c.k > 1 && (kch == 1 || (half_words && (size_t)c.cin * es % 32 != 0 && (kch == 2 || (kch == 3 && c.cout > 32))))) return true;
    if ((size_t)c.cin * es % 128 == 0) return false;
    if (split) return half_words ? padded && ((c.k == 3 && kch == 5) || tiles <= num_cu) : kch % 2 == 1 && kch <= 13;
    if (!half_words) return false;
    const int64_t workgroups = cdiv(tiles, kFirstWaves);
    if (padded && first_single(c, workgroups, num_cu)) return true;
    if (c.k == 1 && kch >= 3 && kch <= 9 && (c.cout >= 512 || (workgroups > 2 * num_cu && workgroups <= 3 * num_cu))) return true;
    return c.cout >= 128 && (kch == 3 || (c.k == 1 && kch == 4) || (kch == 5 && (c.k == 1 || cdiv(c.cout, 64) % 4 == 0)));
}

// Tiles of 32 channels also where tiles of 64 leave compute units idle, if those of 32 are one round of workgroups (split sums) or a second one does not
// wait behind long sums (whole ones, first_single): their width changes no sum.  64 -> 32 channels a tile, us: 3x3 512->512 on 512 pixels 30.5 -> 28.0,
// 128->128 on 100x100 32.3 -> 26.6, 1x1 64->256 on 64x64 17.4 -> 14.9, fp32 3x3 256->256 on 2048 pixels 59.9 -> 44.5; the first frame of a
// ResNet-50-shaped network of 8 streams 757 -> 692.  But split 5x5 72->128 on 2 of 60x50 (188 tiles, 376 of half the width) 17.7 -> 20.9, and whole sums of
// between half a workgroup and one per compute unit: 5x5 144->256 on 96x97 61 -> 71, 128->384 52 -> 55; short ones 3x3 32->384 20 -> 19.2, 1x1 128->384 17.6 -> 16.1;
// by lanes also above that: 5x5 72->256 on 4 of 64x66 59 -> 64.
// And 96 channels over short sums: three tiles instead of two with half of the last one padding (16 streams of 128x128: 1x1 48->96 52.7 -> 48.0, 72->96
// 59.5 -> 53.5, 3x3 32->96 of 12 of 120x128 49 -> 48; not 5x5 32->96 90 -> 96, 3x3 112->96 116 -> 121, nor lanes over 24 and 40 channels;
// not 160: 3x3 96->160 on 8 streams 113 -> 126; nor rows that tiles of 32 cut within 64-byte pieces: 1x1 64->72 66 -> 82).
static bool first_halves(const ConvArgs& c, bool split, bool lanes, int64_t tiles, int64_t halves, int num_cu) {
    if (split) return halves <= num_cu;
    const bool long_sum = c.k * c.k * c.kch >= kFirstLongSum;
    if (c.cout < 128 && c.cout % 64 == 32 && (!lanes || c.kch == 1) && !long_sum) return true;
    const int64_t workgroups = cdiv(tiles, kFirstWaves);
    if (lanes && long_sum && workgroups > num_cu / 2) return false;
    return workgroups < 2 * num_cu && !first_single(c, workgroups, num_cu);
}

// (What decides between sums in one chain and split ones looks at one stream; kernels that sum in one chain give the same bits.)
bool conv_first_supported(int dtype, const ConvArgs& c, const ConvPlan& p) {
    const size_t es = dtype_size(dtype);
    const int vec = dtype == DCNN_F16 ? 8 : 4;
    if (p.flat || p.w_bytes > kWsMaxBytes || c.cout % vec != 0 || ((size_t)c.cin * es) % 16 != 0) return false;
    if (first_stream_bytes(es, c) > kWsMaxBytes || (c.in2_data != nullptr && ((size_t)c.cin2 * es) % 16 != 0)) return false;
    const int64_t ctiles = first_narrow(c) ? 1 : cdiv(c.cout, 64), tiles = cdiv((int64_t)c.n * c.oh * c.ow, kFirstPx) * ctiles;
    if (c.in2_data != nullptr || first_narrow(c) || first_splits(c) || tiles < 1024) return true;
    // Matrix work bounds long sums over enough tiles to fill the chip, and there the plain kernel's plan is the better one where it
    // pads the channels to fewer blocks than tiles of 64 do, or, on large maps, where the number of tiles leaves waves of a workgroup
    // to gather for themselves: 8 streams of 128x128, fp16, 3x3 256->96 193 us against 152, 5x5 256->160 957 against 714 (but one
    // stream of the former 48 against 73, 4 streams of 96x96 of the latter 241 against 364, and 3x3 64->96 54 against 58: short sums
    // are bound by the gathers); fp32, whose K-steps take 16 times as long, 1x1 32->72 41 against 38 and on 96x96 18 against 21.
    const bool uneven = ctiles > 2 && ctiles % 4 != 0;
    const int long_sum = dtype == DCNN_F16 ? 64 : (tiles < 4096 ? 32 : 4);     // K-steps
    if ((ctiles * 64 > p.cout_pad || (uneven && tiles >= 4096)) && c.k * c.k * c.kch >= long_sum) return false;
    // Stores bound short sums on large maps, and whole rows are the better ones where the tiles' parts of a row share 64-byte pieces:
    // 1x1 64->328 on the same maps 111 us against 77, 64->136 50 against 46 (but on 4 of 96x96 34 against 37 and 16 against 29,
    // 256->328 100 against 150, and with whole pieces 64->160 30 against 46).
    return c.k * c.k * c.kch > 8 || tiles < 4096 || ((size_t)c.cout * es) % 64 == 0 || !(uneven || ctiles > 4);
}

template <typename T>
static dcnn_status launch_conv_first_t(dcnn_ctx* ctx, const ConvArgs& c, const EpilogueArgs& e, const ConvPlan& p, const void* bias2) {
    FirstArgs f{};
    f.nb = p.nb; f.ngroups = p.npass * p.cs;
    f.pixels = (int64_t)c.n * c.oh * c.ow;
    f.bias2 = bias2;
    const int64_t ptiles = cdiv(f.pixels, kFirstPx);
    const int64_t tiles = ptiles * cdiv(c.cout, 64), halves = ptiles * cdiv(c.cout, 32);
    const bool split = first_splits(c), lanes = first_by_lanes(c, sizeof(T), split, tiles, ctx->num_cu);
    const bool narrow = first_narrow(c) || first_halves(c, split, lanes, tiles, halves, ctx->num_cu);
    const int ctiles = (int)cdiv(e.c, narrow ? 32 : 64);
    f.wc = split ? 1 : (ctiles % 4 == 0 ? 4 : (ctiles % 2 == 0 ? 2 : 1));      // (no wave without channels)
    f.cgroups = (int)cdiv(ctiles, f.wc);
    f.units = (split ? ptiles : cdiv(ptiles, kFirstWaves / f.wc)) * f.cgroups;
    const size_t stage = (size_t)kFirstPx * first_stage_stride<T>(narrow ? 32 : 64);
    const size_t lds = split ? (size_t)kFirstWaves * (narrow ? 2 : 4) * 4 * kWave * 16 + stage : kFirstWaves * stage;
    const int64_t grid = split ? cdiv(f.units, kXcd) * kXcd : cdiv(f.units / f.cgroups, kXcd) * kXcd * f.cgroups;
    if (grid > INT32_MAX) return fail(ctx, DCNN_ESHAPE, "first frame: %lld workgroups", (long long)grid);
    hipError_t err = hipSuccess;
    const bool thin = c.kch <= 2 && (c.in2_data == nullptr || c.kch2 <= 2);
#define DCNN_FIRST_LAUNCH_X(SPLIT, TC, XT, STEPS)                                                                        \
    do {                                                                                                         \
        auto kern = conv_first_kernel<T, SPLIT, TC, XT, STEPS>;                                                          \
        static bool attr_set = false;                                                                            \
        if (!attr_set) {                                                                                         \
            err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsBytes); \
            attr_set = (err == hipSuccess);                                                                      \
        }                                                                                                        \
        if (err == hipSuccess) hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kFirstWaves * kWave), lds, ctx->stream, c, e, f); \
    } while (0)
#define DCNN_FIRST_LAUNCH(SPLIT, TC, STEPS) do { if (e.xt_flags) DCNN_FIRST_LAUNCH_X(SPLIT, TC, true, STEPS); else DCNN_FIRST_LAUNCH_X(SPLIT, TC, false, STEPS); } while (0)
#define DCNN_FIRST_STEPS(SPLIT, TC) do { if (lanes) DCNN_FIRST_LAUNCH(SPLIT, TC, 1); else if (thin) DCNN_FIRST_LAUNCH(SPLIT, TC, 2); else DCNN_FIRST_LAUNCH(SPLIT, TC, kFirstGroup); } while (0)
    if (split) { if (narrow) DCNN_FIRST_STEPS(kFirstWaves, 1); else DCNN_FIRST_STEPS(kFirstWaves, 2); }
    else { if (narrow) DCNN_FIRST_STEPS(1, 1); else DCNN_FIRST_STEPS(1, 2); }
#undef DCNN_FIRST_STEPS
#undef DCNN_FIRST_LAUNCH
#undef DCNN_FIRST_LAUNCH_X
    if (err != hipSuccess) return check_hip(ctx, err, "hipFuncSetAttribute(conv_first_kernel)");
    return check_hip(ctx, hipGetLastError(), "conv_first_kernel launch");
}

dcnn_status launch_conv_first(dcnn_ctx* ctx, int dtype, const ConvArgs& c_all, const EpilogueArgs& e_all, const ConvPlan& p, const void* bias2) {
    // Inputs past 2 GiB go through in slices of whole streams: the kernel that serves a layer, and with it the order of its
    // sums, is the same however many streams there are.
    const size_t es = dtype_size(dtype);
    const uint64_t slice = kWsMaxBytes / first_stream_bytes(es, c_all);
    auto at = [](const void* base, uint64_t bytes) -> const void* { return base ? static_cast<const char*>(base) + bytes : nullptr; };
    auto at_mut = [](void* base, uint64_t bytes) -> void* { return base ? static_cast<char*>(base) + bytes : nullptr; };
    for (int first = 0; first < c_all.n;) {
        ConvArgs c = c_all;
        EpilogueArgs e = e_all;
        c.n = (uint64_t)(c_all.n - first) < slice ? c_all.n - first : (int)slice;
        const uint64_t out = (uint64_t)first * c.oh * c.ow * e.c * es;
        c.in_data = at(c.in_data, (uint64_t)first * c.h * c.w * c.cin * es);
        c.in2_data = at(c.in2_data, (uint64_t)first * c.h2 * c.w2 * c.cin2 * es);
        e.res_data = at(e.res_data, out);
        e.xA = at_mut(e.xA, out); e.xT = at_mut(e.xT, out); e.out_data = at_mut(e.out_data, out);
        if (e.xt_flags) e.xt_flags += (int64_t)first * c.oh * c.ow;
        const dcnn_status st = dtype == DCNN_F16 ? launch_conv_first_t<f16>(ctx, c, e, p, bias2) : launch_conv_first_t<float>(ctx, c, e, p, bias2);
        if (st != DCNN_OK) return st;
        first += c.n;
    }
    return DCNN_OK;
}

}  // namespace dcnn
