// Sparse delta convolution on small maps with weights too large for LDS: one wave per (pixel tile, 32 output channels).
//
// The deep layers of a backbone multiply a few hundred listed pixels with megabytes of weights.  What sets the pace there
// is the vector memory path of the compute units that take part, so a 3x3 512->512 layer on 16 tiles that ran on 32 workgroups of four waves,
// each pulling 0.9 MB, took 54 us.  Here the work is cut as fine as it goes without splitting a sum -- the order of
// every sum is tap by tap, as in the other kernels that serve such layers, so a stream gives the same bits whichever its batch size
// selects (but for the register-blocked kernel's row gathers in fp32, on lists of tens of thousands of pixels with most taps flagged) --
// and spread over the chip: unit u = (tile u / G, channel group u % G), and since workgroup b runs on XCD b % 8, a group's
// weights are fetched into the L2 of one XCD only (of 8 / G, for fewer than 8 groups).  A layer that compacts blocks in place does so
// by runs of 256 pixels (local_run): tiles of 32 pixels as they lie hold a few listed ones each when flags are scattered and cost their
// weights all the same.  One layer between an input and an output layer, f16, us, 2 / 10 / 30 % of the pixels flagged at random, tiles as they lie ->
// runs: 1x1 512->2048 on 16 K pixels 91 / 119 / 138 -> 52 / 63 / 105, 256->1024 on 6272 26 / 30 / 33 -> 20 / 24 / 30; the layer alone, 3x3 128->512 on
// 8192 21 / 28 / 32 -> 15 / 24 / 31.  3x3 256->256 on 4096 12.6 / 14.7 / 15.9 -> 11.4 / 15.3 / 16.2, with a quarter of it in one region 11.6 -> 14.0:
// there every tile has a SIMD to itself.
//
// fp16 workgroups of four waves fetch their tile's operands once and share them through LDS (gather_tiles.h).  A wave each, a pixel
// per lane -> shared, us a step with input and output layer, 2 / 10 / 50 / 100 % flagged at random: 3x3 128->512 on 8 streams of 32x32
// 25 / 37 / 54 / 69 -> 23 / 32 / 42 / 43, 72->392 on 2 of 60x60 24 / 35 / 44 / 44 -> 22 / 30 / 38 / 37, 1x1 512->2048 on 2 of 64x64
// 27 / 36 / 80 / 124 -> 26 / 30 / 57 / 84, 256->1024 on 8 of 16x16 18 / 19 / 23 / 25 -> 18 / 18 / 21 / 22.  Smaller workgroups are those of layers
// that give a SIMD a wave or two, which wait for each other and for LDS: there every wave gathers for itself.  A wave each -> shared: two waves,
// 3x3 128->512 on 56x56 19 / 25 / 33 / 40 -> 21 / 30 / 35 / 35, 72->392 on 50x50 19 / 22 / 25 / 26 -> 20 / 23 / 30 / 30, 1x1 256->512 on 8 of 16x16
// 17 / 17 / 19 / 21 -> 17 / 18 / 21 / 22; one wave, 3x3 512->512 on 16x16 29 / 30 / 33 / 37 -> 38 / 39 / 40 / 40.  (These with two register sets of
// eight K-steps a wave; now eight sets of two, see the kernel.  Through LDS a single wave has sixteen K-steps of weights in flight at all times: three
// ResNet-50-shaped networks of 8 streams stepped in turn 1075 us a step, 1081 this way, but one alone 1025 and 1014, of 1 stream 920 and 914.)
//
// Layers without an activation only: a decision needs all channels of a pixel.  (Groups that leave their sums in memory and
// a tail done by the last of a tile to arrive were built: the device-scope release and acquire that it takes cost
// ~15 us a layer, 3x3 256->256 44 us against 32 in one workgroup.)
#include "conv_plan.h"
#include "conv_ws_impl.h"
#include "gather_tiles.h"
#include "self_list.h"

namespace dcnn {

// Where every wave gathers for itself: K-steps whose operands are requested together, and groups in registers or on their way -- sixteen K-steps either way.
constexpr int kUnitGroup(int es) { return es == 2 ? 2 : 8; }
constexpr int kUnitSets(int es) { return es == 2 ? 8 : 2; }
constexpr int kUnitMaxWaves = 4;

struct UnitArgs {
    int nb;                        // column blocks per packed channel group (the layer's plan)
    int blocks;                    // 32-channel blocks of the output
    int groups;                    // groups of one block per wave of the workgroup
    int waves;                     // waves with a block (a workgroup that writes lists has more)
    uint32_t map_bytes, out_pixels;
};

// LDS: gathered operands of the tile (where shared) | staging rows per wave | flags and prefix sums of a list built here
constexpr int kUnitStageRow(int es) { return 32 * es + kStagePad; }
constexpr int kUnitOperands(int sh) { return sh > 0 ? 2 * kGatherTile : 0; }
inline bool unit_shares(int waves, int es) { return es == 2 && waves == kUnitMaxWaves; }
inline size_t unit_stage_bytes(int waves, int es) {
    return (size_t)kUnitOperands(unit_shares(waves, es) ? waves : 0) + (size_t)waves * kTile * kUnitStageRow(es);
}

// SH: the waves of the workgroup, which share the gathered operands of their tile (gather_tiles.h); 0: every wave gathers for itself (fp32,
// and fewer than four waves)
template <typename T, int KS, int SH>
__global__ __launch_bounds__(kUnitMaxWaves* kWave) void conv_unit_kernel(ListArgs l, ConvArgs c, EpilogueArgs e, UnitArgs a) {
    typedef typename Mma<T>::Vec Vec;
    constexpr int V = Elem<T>::VEC;
    typedef typename RawOf<T, V>::type Raw;
    constexpr int ES = (int)sizeof(T);
    constexpr int kNoTap = 31;
    constexpr int stage_row = kUnitStageRow(ES);
    static_assert(SH == 0 || (SH == kUnitMaxWaves && ES == 2), "as unit_shares");
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int nwaves = a.waves;
    const int col = lane % 32, g = lane / 32;
    unsigned char* stage = smem + kUnitOperands(SH) + (size_t)wave * kTile * stage_row;

    // Units of this workgroup: u = first, first + step, ... below end.  Where blocks are compacted here they are the tiles of its share
    // of a run's entries, `tile_px` each, for one group of channels.
    int count, first = blockIdx.x, step = gridDim.x, tile_px = kTile;
    const int32_t* run_px = nullptr;
    const uint32_t* run_taps = nullptr;
    if (l.self) {
        static_assert(kUnitMaxWaves * kWave == kRunPixels, "a pixel per thread");
        if (first < l.writers) {
            local_write<kUnitMaxWaves * kWave>(l, smem);
            return;
        }
        first -= l.writers;
        const int group = first % a.groups;
        const RunPart rp = run_part(first / a.groups, (l.m_out_px + kRunPixels - 1) / kRunPixels, l.run_parts);
        const int all = local_run(l, smem + l.lds_list, rp.run, group == 0 && rp.part == 0, run_px, run_taps);
        const int share = run_share(all, l.run_parts, l.run_even), from = rp.part * share;
        count = min(all - from, share);
        if (wave >= nwaves || count <= 0) return;
        run_px += from;
        run_taps += from;
        const int tiles = (count + kTile - 1) / kTile;
        tile_px = (count + tiles - 1) / tiles;
        first = group;
        step = a.groups;
    } else {
        count = (int)list_count(l);
    }
    const int end = (count + kTile - 1) / kTile * a.groups;
    const int kch = c.kch, ksteps = KS * KS * kch, cols = a.nb * 32;
    const int cin_bytes = c.cin * ES;
    const __amdgpu_buffer_rsrc_t rs_in = ws_rsrc(c.in_data, (uint64_t)c.n * c.h * c.w * cin_bytes);
    const __amdgpu_buffer_rsrc_t rs_w = ws_rsrc(c.wpacked, (uint64_t)(c.cout_pad / cols) * ksteps * 2 * cols * 16);
    const __amdgpu_buffer_rsrc_t rs_out = ws_rsrc(e.out_data, a.map_bytes), rs_res = ws_rsrc(e.res_data, a.map_bytes);
    const __amdgpu_buffer_rsrc_t rs_rmask = ws_rsrc(e.res_mask, a.out_pixels);
    const uint32_t wstride = (uint32_t)(2 * cols * 16);        // weights of one K-step
    const uint32_t row_bytes = (uint32_t)e.c * ES;

    for (int u = first; u < end; u += step) {
        const int tile = u / a.groups;
        const int cb = (u - tile * a.groups) * nwaves + wave;  // this wave's channel block
        const bool cb_on = cb < a.blocks;
        const int j = tile * tile_px + col;
        int p = -1, rflag = 1;
        uint32_t taps = 0;
        if (col < tile_px && j < count) {
            if (l.self) {
                p = run_px[j];
                taps = run_taps[j];
                rflag = (taps & kLocalSecond) != 0;
            } else {
                p = l.list ? l.list[j] : j;
                taps = l.taps ? l.taps[j] & ((1u << (KS * KS)) - 1u) : 1u;
            }
        }
        if (!l.self && e.res_mask) rflag = __builtin_amdgcn_raw_buffer_load_b8(rs_rmask, p >= 0 ? p : (int)kOob, 0, 0);
        uint32_t base;                                         // this lane's 16 bytes of tap (0,0), K-step 0
        {
            const uint32_t pu = p >= 0 ? (uint32_t)p : 0u;
            const uint32_t t1 = fast_div(pu, c.div_ow);
            const int ox = (int)(pu - t1 * (uint32_t)c.ow);
            const uint32_t n = fast_div(t1, c.div_oh);
            const int oy = (int)(t1 - n * (uint32_t)c.oh);
            base = (uint32_t)(((int)n * c.h + oy * c.stride - c.pad) * c.w + ox * c.stride - c.pad) * (uint32_t)cin_bytes + (SH > 0 ? 0u : (uint32_t)g * 16u);
        }
        uint32_t wave_taps = 0;                                // taps any lane of the wave needs
#pragma unroll
        for (int t = 0; t < KS * KS; ++t)
            if (__ballot((taps >> t) & 1)) wave_taps |= 1u << t;
        const uint32_t wlane = ((uint32_t)(cb_on ? cb / a.nb : 0) * (uint32_t)ksteps * 2u * (uint32_t)cols + (uint32_t)g * (uint32_t)cols +
                                (uint32_t)(cb_on ? cb % a.nb : 0) * 32u + (uint32_t)col) * 16u;
        f32x16 acc[1][1];
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[0][0][i] = 0.0f;
        if constexpr (SH > 0) {
            // the pixels this wave fetches, from the lanes whose columns they are
            typedef GatherShare<1, SH> Share;
            uint32_t from[Share::kLoads], need[Share::kWords];
#pragma unroll
            for (int i = 0; i < Share::kWords; ++i) need[i] = 0;
#pragma unroll
            for (int i = 0; i < Share::kLoads; ++i) {
                const int at = col / 4 * 4 + Share::pixel(wave, i);
                from[i] = (uint32_t)__shfl((int)base, at, kWave);
                need[i / 3] |= ((uint32_t)__shfl((int)taps, at, kWave) & ((1u << (KS * KS)) - 1u)) << (9 * (i % 3));
            }
            gather_tiles<T, 1, KS, 1, SH, 4, 16>(acc, rs_in, rs_w, from, need, wave_taps, kch, cin_bytes, c.w * cin_bytes, cb_on ? wlane : kOob, wstride,
                                                 smem, wave, lane, true);
        } else {
        // Groups of K-steps of one tap, in a ring of register sets.  One wave per SIMD has its own instructions to wait for
        // (4-8 clocks each), so a group's addresses are formed once: the gathers of its steps differ by an immediate, the
        // weights by a scalar offset, and the cursor moves by selects.  fp16: eight sets of two steps, of which seven are on their way at any wait, not eight of
        // sixteen steps as with two sets of eight.  Two of eight -> eight of two, us a step: three ResNet-50-shaped networks of 8 streams in turn, whose
        // weights leave every cache between steps, 1095 -> 1081, one alone 1019 -> 1014, three of 3 streams 1032 -> 1021, HRNet-shaped 989 -> 985, 1x1
        // 2048->512 on 512 pixels 36 / 39 / 45 / 53 -> 36 / 38 / 44 / 51 (2 / 10 / 50 / 100 % flagged); but 3x3 512->512 on 512 pixels stepped alone, its weights in L2,
        // 27 / 28 / 31 / 35 -> 33 / 33 / 34 / 35, for the address arithmetic.  Four of four, sixteen single steps, and twenty or twenty-four steps (200 and 232
        // registers) were slower in networks: 1036, 1057, 1020-1025.  Lines touched ahead by a load of their own 1025.  fp32, which the matrix cores bound: two of eight.
        constexpr int G = kUnitGroup(ES), SETS = kUnitSets(ES);
        const int kgroups = (kch + G - 1) / G;
        const bool whole_groups = kch % G == 0 && kch * 32 == cin_bytes;   // no K-step of a group reaches past the pixel's channels
        struct Cur { uint32_t rest; int t, kg; };
        auto advance = [&](Cur& q) __attribute__((always_inline)) {
            const bool wrap = q.kg + 1 == kgroups;
            q.kg = wrap ? 0 : q.kg + 1;
            q.rest = wrap ? q.rest & (q.rest - 1) : q.rest;
            q.t = __builtin_ctz(q.rest | 1u << kNoTap);
        };
        struct Set { Vec x[G], w[G]; };
        // Every load is issued unconditionally: a lane whose tap is not flagged, channel padding and groups past the end
        // read zeros from an offset outside the descriptor.
        auto issue = [&](const Cur& q, Set& st) __attribute__((always_inline)) {
            const bool live = q.t != kNoTap;
            const int t = live ? q.t : 0;
            const int dy = t / KS, dx = t - dy * KS;
            uint32_t off = (live && ((taps >> t) & 1u)) ? base + (uint32_t)((dy * c.w + dx) * cin_bytes + q.kg * (G * 32)) : kOob;
            asm volatile("" : "+v"(off));                      // one load at a computed offset, not a load per case
            uint32_t wstep = (uint32_t)(t * kch + q.kg * G) * wstride;
            if (whole_groups) {
#pragma unroll
                for (int i = 0; i < G; ++i) {
                    st.x[i] = ws_load16<Vec>(rs_in, off + (uint32_t)i * 32u);
                    st.w[i] = ws_load16<Vec>(rs_w, wlane, wstep);
                    wstep += wstride;
                }
            } else {
#pragma unroll
                for (int i = 0; i < G; ++i) {
                    const int kc = q.kg * G + i;
                    st.x[i] = ws_load16<Vec>(rs_in, (2 * kc + g) * 16 < cin_bytes ? off + (uint32_t)i * 32u : kOob);
                    st.w[i] = ws_load16<Vec>(rs_w, wlane, wstep);
                    if (kc + 1 < kch) wstep += wstride;        // (a step past the last one repeats its weights and meets zeros)
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto mma = [&](const Set& st) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < G; ++i) Mma<T>::run(acc[0][0], st.w[i], st.x[i]);
            __builtin_amdgcn_sched_barrier(0);
        };
        if (cb_on && wave_taps) {
            Set st[SETS];
            Cur cg{wave_taps, __builtin_ctz(wave_taps), 0};
#pragma unroll
            for (int d = 0; d < SETS - 1; ++d) { issue(cg, st[d]); advance(cg); }
            for (int left = __popc(wave_taps) * kgroups; left > 0; left -= SETS) {
#pragma unroll
                for (int d = 0; d < SETS; ++d) {
                    issue(cg, st[(d + SETS - 1) % SETS]); advance(cg);
                    mma(st[d]);
                }
            }
        }
        }
        // rounded sums -> staging rows -> the pixels' rows, 16 bytes per lane
        stage_accumulators<T, 1>(acc[0], stage + (size_t)col * stage_row, g);
        lds_wave_sync();
        constexpr int LPB = 32 / V;                            // lanes per pixel
#pragma unroll
        for (int it = 0; it < kTile * LPB / kWave; ++it) {
            const int ent = it * (kWave / LPB) + lane / LPB, vi = lane % LPB;
            const int pe = __shfl(p, ent, kWave), rf = __shfl(rflag, ent, kWave);
            const int ch = cb * 32 + vi * V;
            const uint32_t o = (pe >= 0 && cb_on && ch < e.c) ? (uint32_t)pe * row_bytes + (uint32_t)ch * ES : kOob;
            Raw d = raw_load<T, V>(reinterpret_cast<const T*>(stage + (size_t)ent * stage_row) + vi * V);
            if (e.res_data != nullptr) {
                const Raw rr = ws_load16<Raw>(rs_res, rf ? o : kOob);
#pragma unroll
                for (int k = 0; k < V; ++k) raw_set<T, V>(d, k, raw_get<T, V>(d, k) + raw_get<T, V>(rr, k));
            }
            ws_store16<Raw>(rs_out, o, d);
        }
        lds_wave_sync();                                       // (the staging rows are free again)
    }
}

// Fewer waves per workgroup (finer units) until the chip has two workgroups per compute unit.
static int unit_waves(const dcnn_ctx* ctx, int64_t tiles, int blocks) {
    int w = kUnitMaxWaves;
    while (w > 1 && (w > blocks || tiles * cdiv(blocks, w) < 2 * (int64_t)ctx->num_cu)) w >>= 1;
    return w;
}

// The length of a list is known on the device only, so the rule looks at the map's: units if every pixel is listed, K-steps of a
// sum and passes over the channels.  A unit fetches its weights for 32 pixels, the register-blocked kernel and the streamed one for
// more, so long sums over full lists of large maps are theirs.  Kernels on lists in memory, whose tiles are full, us, other kernel -> units, all pixels / 30 % / 10 % listed:
//   up to a wave per SIMD:   3x3 256->256 on 4096 pixels 41 -> 29 / 32 -> 20 / .., 1x1 1024->256 17.5 -> 15 / 17 -> 9 / ..
//   beyond, one pass:        3x3 256->256 on 6272 43 -> 48, 1x1 1024->256 18 -> 24: no
//   several passes, K <= 32: 1x1 256->1024 on 6272 34 -> 25 / 18 -> 10 / 17 -> 7, 512->2048 on 16 K 153 -> 160 / 79 -> 56 / 75 -> 9
//                            (stride 2, whose lists cost more: 256->1024 on 4096 outputs 32 -> 33 / 21 -> 22 / 20 -> 19, 512->2048 57 -> 76: no)
//   3x3, K <= 72:            128->512 on 8192 51 -> 52 / 44 -> 37 / 42 -> 24, on 16 K 84 -> 96: no
//   longer:                  3x3 256->512 on 4096 43 -> 47, 1x1 1024->512 20 -> 24: no (at 10 % 34 -> 26 and 18 -> 13)
static int64_t unit_limit(const dcnn_ctx* ctx, const ConvArgs& c, const ConvPlan& p) {
    const int ksteps = c.k * c.k * c.kch;
    if (p.npass > 1 && ksteps <= 32) return c.stride == 1 ? INT64_MAX : (int64_t)ctx->num_cu * 16;
    if (p.npass > 1 && c.k == 3 && ksteps <= 72) return (int64_t)ctx->num_cu * 16;
    return (int64_t)ctx->num_cu * 4;
}

bool conv_unit_supported(const dcnn_ctx* ctx, int dtype, const ListArgs& l, const ConvArgs& c, const EpilogueArgs& e, const ConvPlan& p) {
    const size_t es = dtype_size(dtype);
    const int vec = dtype == DCNN_F16 ? 8 : 4;
    if ((!p.stream && conv_ws_lds_bytes(p, dtype, c.k, e.c) != 0) || p.flat || (c.k != 1 && c.k != 3) || e.c % vec != 0 || ((size_t)c.cin * es) % 16 != 0) return false;
    if (e.act != DCNN_ACT_NONE || c.in2_data != nullptr || e.accum_O != nullptr || e.xt_flags != nullptr) return false;
    if (!l.self && l.taps == nullptr && !(c.k == 1 && c.stride == 1 && l.list != nullptr)) return false;
    const int64_t out_px = (int64_t)c.n * c.oh * c.ow;
    return out_px <= kUnitMaxPixels && cdiv(out_px, kTile) * cdiv(e.c, 32) <= unit_limit(ctx, c, p) && (uint64_t)c.n * c.h * c.w * c.cin * es <= kWsMaxBytes && (uint64_t)out_px * e.c * es <= kWsMaxBytes &&
           p.w_bytes <= kWsMaxBytes;
}

template <typename T>
static dcnn_status launch_conv_unit_t(dcnn_ctx* ctx, const ListArgs& l_in, const ConvArgs& c, const EpilogueArgs& e, const ConvPlan& p) {
    ListArgs l = l_in;
    const int64_t out_px = (int64_t)c.n * c.oh * c.ow, tiles = cdiv(out_px, kTile);
    UnitArgs a{};
    a.nb = p.nb;
    a.blocks = (int)cdiv(e.c, 32);
    const int waves = unit_waves(ctx, tiles, a.blocks);
    a.groups = (int)cdiv(a.blocks, waves);
    a.map_bytes = (uint32_t)((uint64_t)out_px * e.c * sizeof(T));
    a.out_pixels = (uint32_t)out_px;
    a.waves = waves;
    const int64_t want = tiles * a.groups, cap = (int64_t)ctx->num_cu * 8;
    int grid = (int)(cdiv(want < cap ? want : cap, kXcd) * kXcd);
    size_t lds = unit_stage_bytes(waves, (int)sizeof(T));
    if (l.self) {
        // (multiples of 8 keep a channel group on its XCD; writers form the flags of the whole map: four waves.  LDS: entries behind
        // the staging rows; a writer uses the space from 0 on)
        l.writers = (int)cdiv(local_writers(l), kXcd) * kXcd;
        l.run_parts = run_parts(out_px, a.groups, 4 * (int64_t)ctx->num_cu);
        l.run_even = cdiv(out_px, kRunPixels) * l.run_parts * a.groups * waves <= 4 * (int64_t)ctx->num_cu;
        l.lds_list = (int)align_up(lds, 16);
        lds = (size_t)l.lds_list + kRunLds;
        grid = (int)(cdiv(out_px, kRunPixels) * l.run_parts * a.groups) + l.writers;
        const size_t scratch = self_scratch_bytes(l.m_in_px, l.m_out_px);
        if (scratch > lds) lds = scratch;
    }
    const dim3 g(grid), b((l.self ? kUnitMaxWaves : waves) * kWave);
#define DCNN_UNIT_LAUNCH(SH)                                                                                     \
    do {                                                                                                         \
        if (c.k == 1) hipLaunchKernelGGL((conv_unit_kernel<T, 1, SH>), g, b, lds, ctx->stream, l, c, e, a);      \
        else hipLaunchKernelGGL((conv_unit_kernel<T, 3, SH>), g, b, lds, ctx->stream, l, c, e, a);               \
    } while (0)
    bool shared = false;
    if constexpr (sizeof(T) == 2) {
        shared = unit_shares(waves, (int)sizeof(T));
        if (shared) DCNN_UNIT_LAUNCH(kUnitMaxWaves);
    }
    if (!shared) DCNN_UNIT_LAUNCH(0);
#undef DCNN_UNIT_LAUNCH
    return check_hip(ctx, hipGetLastError(), "conv_unit_kernel launch");
}

dcnn_status launch_conv_unit(dcnn_ctx* ctx, int dtype, const ListArgs& l, const ConvArgs& c, const EpilogueArgs& e, const ConvPlan& p) {
    return dtype == DCNN_F16 ? launch_conv_unit_t<f16>(ctx, l, c, e, p) : launch_conv_unit_t<float>(ctx, l, c, e, p);
}

}  // namespace dcnn
