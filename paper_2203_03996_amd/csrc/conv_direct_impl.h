// Sparse delta convolution whose weights do not fit LDS, long work lists: register-blocked gather-GEMM.
//
// When a layer's packed weights exceed LDS, every wave that multiplies a pixel tile has to fetch the weight operands of all K-steps from
// L2.  fp16 (conv_direct_body): the waves of a tile share its gathered operands through LDS (gather_tiles.h), on long lists two or four
// tiles per wave, so that every weight operand is multiplied with all of them.  What bounds it: the vector memory path of a compute unit
// with weights (short lists: 22 clocks per KB, 16 in flight per wave; 777 clocks per four K-steps of a 3x3 256->256 tile, 1047 before the
// cursors moved by selects and the loop had one way out), the matrix cores and LDS about equally on long ones.  Kernels whose waves gathered for
// themselves, a pixel per lane -> this, us a step with input and output layer: 3x3 256->256 + ReLU on 8 streams of 16x16, all / a tenth
// flagged 56 / 48 -> 45 / 44, 1x1 1024->256 there 51 / 43 -> 46 / 39, 3x3 128->128 on 8 of 256x256 439 / 242 -> 375 / 217, with ReLU
// 542 / 306 -> 484 / 287, 256->512 on 16 of 64x64 404 / 250 -> 313 / 223.  128->64 on 8 of 128x128 with 1 / 2 /
// 10 % flagged 43.5 / 45.2 / 67.7 -> 40.6 / 44.5 / 60.5.  Known cost: lines that are mostly padding on short lists, 3x3 72->256 + ReLU on 8 of 96x100 with 2 % flagged 56 -> 58,
// 104->192 57 -> 60 (with half of them flagged they gain).
// fp32 (conv_lane_body): every wave for itself.
//
// Addressing is by 32-bit byte offsets against buffer descriptors (tensors below 2 GiB): a lane whose tap is not
// flagged, whose entry lies beyond the list or whose K-step is channel padding gets an offset outside the
// descriptor and reads zeros, so unflagged memory is never touched and the loop has no branches.  Window taps
// that no pixel of the wave or workgroup needs are skipped altogether.  Sparse steps of 1x1 / 3x3 layers with 16-byte aligned
// channels only; which taps an entry needs comes with the work list (one word per entry).
#pragma once

#include "conv_plan.h"
#include "gather_tiles.h"
#include "self_list.h"

namespace dcnn {

constexpr int kDirectWaves = 4;
constexpr int direct_pow2_ceil(int v) { int p = 1; while (p < v) p <<= 1; return p; }
// pixel tiles per wave on long lists (a register block of 128 sums; 64 where an fp16 tile has one wave, whose operands nobody shares)
__host__ __device__ constexpr int direct_tiles(int nb, int es, int sh) { return nb <= 2 && (es > 2 || sh > 1) ? 4 : 2; }
// LDS: operands of the tiles, then their rounded sums in the same space (a wave with tiles of its own waits for nobody before it puts
// them there: it has a part of the space to itself) | partial maxima | a tap word per wave | an iteration's entries
__host__ __device__ constexpr int direct_space(int nb, int es, int ti, int sh) {
    const int x = kDirectWaves / sh * 2 * ti * kGatherTile, y = kDirectWaves * ti * kTile * (nb * 32 * es + kStagePad);
    return x > y ? x : y;
}
inline size_t direct_lds_bytes(int nb, int es, int sh, bool self) {
    if (es > 2) return (size_t)kDirectWaves * kTile * (nb * 32 * es + kStagePad) + conv_xchg_bytes(kDirectWaves);
    return (size_t)direct_space(nb, es, self ? 1 : direct_tiles(nb, es, sh), sh) + conv_xchg_bytes(kDirectWaves) + 2 * kDirectWaves * sizeof(uint32_t) * (1 + 3 * kWave);
}

// The work of one workgroup with TI pixel tiles per wave; SH waves (the plan's `cs`) share a tile and split its output channels.
template <typename T, int NB, int KS, int TI, int SH, bool SELF>
__device__ __forceinline__ void conv_direct_body(const ListParam<SELF>& l, const ConvArgs& c, const EpilogueArgs& e, int npass,
                                                 int64_t count, unsigned char* smem, const int32_t* self_px, const uint32_t* self_tap) {
    typedef typename Mma<T>::Vec Vec;
    constexpr int V = Elem<T>::VEC;
    typedef typename RawOf<T, V>::type Raw;
    constexpr int COLS = NB * 32;
    constexpr int ES = (int)sizeof(T);
    constexpr int NW = kDirectWaves, SLOTS = NW / SH;
    constexpr int N = GatherShare<TI, SH>::kLoads;
    constexpr int LP = direct_pow2_ceil(COLS / V), NIT = kTile / (kWave / LP);   // lanes per pixel of the tail, rows of a tile per lane
    constexpr int UB = TI == 1 || NIT < 4 ? 2 : 4;              // rows of a batch (of a single tile two: less code)
    constexpr int PIECES = COLS * ES / 64;                     // 64-byte pieces of a row of this wave's channels
    // K-steps of weights in flight (more spill: eight of two blocks beside the sixteen vectors of a tile that a wave fetches alone)
    constexpr int kAheadW = TI == 4 ? 2 : TI == 1 && NB <= 2 && NB <= SH ? 8 : 4;
    static_assert(LP >= 2 && LP <= kWave, "a pixel's channels on neighbouring lanes");
    static_assert(sizeof(Vec) == 16, "16-byte operand vectors");

    const int64_t ntiles = (count + kTile - 1) / kTile;
    // tile slots in use: as few as go round the grid once (a compute unit's memory path is what a short list waits for)
    const int slots = TI > 1 ? SLOTS : SELF ? (int)min(ntiles, (int64_t)SLOTS) : ws_slots((uint32_t)ntiles, gridDim.x, SLOTS);
    const int64_t groups = (ntiles + slots * TI - 1) / (slots * TI);
    const WgTileRange r = SELF ? WgTileRange{0, groups, 1} : wg_tile_range(groups);
    if (r.begin >= r.end) return;

    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int col = lane % 32, g = lane / 32;
    const int slot = wave / SH, part = wave % SH;
    const int kch = c.kch;
    const int ksteps = KS * KS * kch;
    const bool full_tail = npass == 1;
    constexpr int stage_stride = COLS * ES + kStagePad;
    // (a tile's rounded sums wait in the space of its operands)
    constexpr int space = direct_space(NB, ES, TI, SH);
    unsigned char* buf = smem + (SH == 1 ? (size_t)wave * (space / NW) : (size_t)slot * 2 * TI * kGatherTile);
    unsigned char* stage = SH == 1 ? buf : smem + (size_t)wave * TI * kTile * stage_stride;
    unsigned char* behind = smem + space;
    float* xchg = reinterpret_cast<float*>(behind) + (size_t)slot * 2 * SH * kTile;
    uint32_t* wave_words;
    // [3][a thread each]; these and the words twice: a wave may be an iteration ahead of one that still reads them
    int32_t* entries;
    int phase = 0;

    const int cin_bytes = c.cin * ES;
    const __amdgpu_buffer_rsrc_t rs_in = ws_rsrc(c.in_data, (uint64_t)c.n * c.h * c.w * cin_bytes);
    const __amdgpu_buffer_rsrc_t rs_w = ws_rsrc(c.wpacked, (uint64_t)npass * SH * ksteps * 2 * COLS * 16);

    auto origin = [&](int p32) {
        // pixel index of tap (0,0) of the entry's window (only used when that tap is in bounds)
        const uint32_t pu = p32 >= 0 ? (uint32_t)p32 : 0u;
        const uint32_t t1 = fast_div(pu, c.div_ow);
        const int ox = (int)(pu - t1 * (uint32_t)c.ow);
        const uint32_t n = fast_div(t1, c.div_oh);
        const int oy = (int)(t1 - n * (uint32_t)c.oh);
        return ((int)n * c.h + oy * c.stride - c.pad) * c.w + ox * c.stride - c.pad;
    };
    auto tile_of = [&](int64_t wt, int ti) { return (wt * slots + slot) * TI + ti; };
    const int mine_n = slots * TI * kTile;                     // entries of an iteration
    // An iteration's entries, one per thread, are requested an iteration ahead -- entry after entry by the lanes that need them, a wait
    // each, 16384 tiles of a 3x3 128->128 layer spent half their time on lists -- and meet in LDS: pixel, offset of its window, tap word.
    static_assert(SLOTS * TI * kTile <= NW * kWave, "an entry per thread");
    struct Entry { int p; uint32_t tap; };
    const __amdgpu_buffer_rsrc_t rs_list = ws_rsrc(l.list, SELF ? 0 : (uint64_t)count * 4), rs_taps = ws_rsrc(l.taps, SELF ? 0 : (uint64_t)count * 4);
    const int me = threadIdx.x;
    auto request_entry = [&](int64_t wt) -> Entry {
        const int64_t j = wt * mine_n + me;
        const bool on = wt < r.end && me < mine_n && j < count;
        if constexpr (SELF) return on ? Entry{self_px[j], self_tap ? self_tap[j] : 1u} : Entry{-1, 0u};
        const uint32_t off = on ? (uint32_t)j * 4u : kOob;
        return Entry{(int)__builtin_amdgcn_raw_buffer_load_b32(rs_list, (int)off, 0, 0), (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs_taps, (int)off, 0, 0)};
    };
    Entry ahead = request_entry(r.begin);

    int survivors = 0;
    for (int64_t wt = r.begin; wt < r.end; wt += r.step) {
        uint32_t any;
        wave_words = reinterpret_cast<uint32_t*>(behind + conv_xchg_bytes(NW)) + phase * NW;
        entries = reinterpret_cast<int32_t*>(behind + conv_xchg_bytes(NW)) + 2 * NW + phase * 3 * NW * kWave;
        phase ^= 1;
        {
            const int64_t j = wt * mine_n + me;
            const bool on = me < mine_n && j < count;   // (what lies behind belongs to the run's next workgroup)
            const int p32 = !on ? -1 : (SELF || l.list != nullptr) ? ahead.p : (int)j;
            any = !on ? 0u : (SELF || l.taps != nullptr) ? ahead.tap & ((1u << (KS * KS)) - 1u) : 1u;   // (no words: a 1x1 layer on its input's own list)
            if (me < mine_n) {
                entries[me] = p32;
                entries[NW * kWave + me] = (int)((uint32_t)origin(p32) * (uint32_t)cin_bytes);
                entries[2 * NW * kWave + me] = (int)any;
            }
        }
        // window taps that a pixel of the workgroup needs; a slot without entries only keeps the barriers
        if constexpr (SH > 1) {
            uint32_t wave_taps = 0;
#pragma unroll
            for (int t = 0; t < KS * KS; ++t)
                if (__ballot((any >> t) & 1)) wave_taps |= 1u << t;
            if (lane == 0) wave_words[wave] = wave_taps;
        }
        lds_block_sync();
        ahead = request_entry(wt + r.step);
        uint32_t taps = 0;
        if constexpr (SH > 1) {
#pragma unroll
            for (int i = 0; i < NW; ++i) taps |= (uint32_t)__builtin_amdgcn_readfirstlane((int)wave_words[i]);
        }
        const bool mine = slot < slots && tile_of(wt, 0) * kTile < count;
        uint32_t base[N], need[GatherShare<TI, SH>::kWords];    // the pixels this wave fetches
#pragma unroll
        for (int i = 0; i < GatherShare<TI, SH>::kWords; ++i) need[i] = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int at = (slot * TI + GatherShare<TI, SH>::tile(part, i)) * kTile + col / 4 * 4 + GatherShare<TI, SH>::pixel(part, i);
            base[i] = (uint32_t)entries[NW * kWave + at];
            need[i / 3] |= (uint32_t)entries[2 * NW * kWave + at] << (9 * (i % 3));
        }
        if constexpr (SH == 1) {
            uint32_t own = 0;
#pragma unroll
            for (int i = 0; i < N; ++i) own |= need[i / 3] >> (9 * (i % 3)) & 0x1ffu;
#pragma unroll
            for (int t = 0; t < KS * KS; ++t)
                if (__ballot((own >> t) & 1)) taps |= 1u << t;
        }

        for (int pass = 0; pass < npass; ++pass) {
            const int cgroup = pass * SH + part;               // which group of COLS output channels
            const int ch0 = cgroup * COLS;
            int nch = e.c - ch0;
            nch = nch < 0 ? 0 : (nch > COLS ? COLS : nch);
            f32x16 acc[TI][NB];
#pragma unroll
            for (int ti = 0; ti < TI; ++ti)
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[ti][b][i] = 0.0f;

            if (pass > 0) lds_block_sync();                    // (the tail before has left the space)
            // The tail's batches wait for their state rows one after the other: a word of every 64 bytes of them is touched ahead of the
            // sums, x^A by the lower half of the wave, x^T by the upper one.  (Lists with several tiles per wave have others' sums to wait behind.)
            uint32_t touched[PIECES];
            auto touch_rows = [&](int ti) {
                const unsigned char* rows = static_cast<const unsigned char*>(g == 0 ? e.xA : e.xT);
                const int p32 = mine ? entries[(slot * TI + ti) * kTile + col] : -1;
#pragma unroll
                for (int i = 0; i < PIECES; ++i) {
                    touched[i] = 0;
                    if (rows != nullptr && p32 >= 0 && i * 64 < nch * ES)
                        touched[i] = *reinterpret_cast<const uint32_t*>(rows + ((int64_t)p32 * e.c + ch0) * ES + i * 64);
                }
            };
            auto rows_arrived = [&]() {
#pragma unroll
                for (int i = 0; i < PIECES; ++i) asm volatile("" ::"v"(touched[i]));
            };
            if constexpr (TI == 1) touch_rows(0);
            gather_tiles<T, NB, KS, TI, SH, (TI == 1 ? 4 : 1), kAheadW>(
                acc, rs_in, rs_w, base, need, taps, kch, cin_bytes, c.w * cin_bytes,
                (uint32_t)cgroup * (uint32_t)ksteps * (uint32_t)(2 * COLS * 16) + (uint32_t)(g * COLS + col) * 16u, (uint32_t)(2 * COLS * 16),
                buf, part, lane, mine);
            if constexpr (TI == 1) rows_arrived();

            // ---- tail: this wave's channel slice of each of its tiles -------------------------------
            // (all tiles are staged first: their sums leave the registers to the state rows)
            if constexpr (SH > 1) lds_block_sync(); else lds_wave_sync();   // (operands and staged sums share the space)
            int tlane = lane;
            if constexpr (TI == 4 || SH == 1) asm volatile("" : "+v"(tlane));   // (what the tail derives from it is formed here, not kept through the sums)
            const int tcol = tlane % 32;
#pragma unroll
            for (int ti = 0; ti < TI; ++ti) stage_accumulators<T, NB>(acc[ti], stage + (size_t)(ti * kTile + tcol) * stage_stride, tlane / 32);
            lds_wave_sync();
            if (e.act == DCNN_ACT_NONE && e.res_data == nullptr) {   // nothing to do to the sums
                const int nvec = (nch + V - 1) / V, sub = tlane % LP, grp = tlane / LP;
#pragma unroll 1
                for (int ti = 0; ti < TI; ++ti) {
#pragma unroll
                    for (int it = 0; it < NIT; ++it) {
                        const int ent = it * (kWave / LP) + grp, pe = mine ? entries[(slot * TI + ti) * kTile + ent] : -1;
                        if (pe >= 0 && sub < nvec)
                            raw_store<T, V>(static_cast<T*>(e.out_data) + (int64_t)pe * e.c + ch0 + sub * V,
                                            raw_load<T, V>(reinterpret_cast<const T*>(stage + (size_t)(ti * kTile + ent) * stage_stride) + sub * V));
                    }
                }
                continue;
            }
            const MaxExchange mx{xchg, SH, part};
            const bool exchange = SH > 1 && full_tail && e.act != DCNN_ACT_NONE;
#pragma unroll 1
            for (int ti = 0; ti < TI; ++ti) {
                const int p32 = mine ? entries[(slot * TI + ti) * kTile + tcol] : -1;
                auto dx = [&](int ent, int64_t, int c0) -> Raw {
                    return raw_load<T, V>(reinterpret_cast<const T*>(stage + (size_t)(ti * kTile + ent) * stage_stride) + (c0 - ch0));
                };
                uint32_t bits;
                if (SH > 1 && exchange) bits = act_trunc_tile<T, V, 1, UB, true>(e, false, p32, tlane, dx, ch0, nch, COLS, mx);
                else bits = act_trunc_tile<T, V, 1, UB, false>(e, false, p32, tlane, dx, ch0, nch, COLS, mx);
                const int64_t tile = tile_of(wt, ti);
                if (mine && full_tail && part == 0 && tile * kTile < count) {
                    if (e.surv) { if (tlane == 0) e.surv[tile] = bits; }
                    else survivors += __popc(bits);
                }
            }
        }
    }
    // one atomic per wave: a counter bumped once per tile by every wave serialises in L2
    if (e.out_count && !e.surv && lane == 0 && survivors) atomicAdd(e.out_count, survivors);
}

// fp32: the matrix cores take sixteen times as long over a K-step as the vector memory path over its gathers, so every wave gathers for itself and
// none waits for another (3x3 64->64 on 87 K pixels, a tenth flagged: 101 us, with shared operands 111).
// The work of one workgroup with TI pixel tiles per wave and a ring of D operand sets (D - 1 K-steps in flight).
// ROW (3x3, stride 1, padding 1): one gather per window ROW instead of one per tap.  The work list is ascending and
// holds every output pixel with a flagged tap, so if an entry's left tap (dy, 0) is flagged, the output pixel to its
// left is listed too and is the entry just before it -- the lane below holds that very input pixel as ITS centre tap
// (dy, 1).  Left and right operands are therefore the centre column moved by one lane (a DPP wave shift); only the
// first and the last column of a tile, whose neighbours sit in other tiles, fetch theirs, both through ONE extra load
// per tile (the two edges are different lanes).  A third of the gather traffic of a kernel that L2 bounds, and the
// weight operands of a row's three taps are multiplied with the same gathered registers.
template <typename T, int NB, int KS, int TI, int D, bool ROW, bool SELF>
__device__ __forceinline__ void conv_lane_body(const ListParam<SELF>& l, const ConvArgs& c, const EpilogueArgs& e, int npass, int cs,
                                                 int64_t count, unsigned char* smem, const int32_t* self_px, const uint32_t* self_tap) {
    typedef typename Mma<T>::Vec Vec;
    constexpr int V = Elem<T>::VEC;
    typedef typename RawOf<T, V>::type Raw;
    constexpr int COLS = NB * 32;
    constexpr int ES = (int)sizeof(T);
    constexpr int NW = kDirectWaves;
    constexpr int kNoTap = 31;
    static_assert(sizeof(Vec) == 16, "16-byte operand vectors");

    const int units_per_iter = NW / cs;                        // groups of TI tiles per workgroup iteration
    const int64_t ntiles = (count + kTile - 1) / kTile;
    const int64_t groups = (ntiles + units_per_iter * TI - 1) / (units_per_iter * TI);
    const WgTileRange r = SELF ? WgTileRange{0, groups, 1} : wg_tile_range(groups);
    if (r.begin >= r.end) return;

    const int lane = threadIdx.x % kWave;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int col = lane % 32, g = lane / 32;
    const int slot = wave / cs, part = wave % cs;
    const int kch = c.kch;
    const int ksteps = KS * KS * kch;
    const bool full_tail = npass == 1;
    constexpr int stage_stride = COLS * ES + kStagePad;
    unsigned char* stage = smem + (size_t)wave * kTile * stage_stride;
    float* xchg = reinterpret_cast<float*>(smem + (size_t)NW * kTile * stage_stride) + (size_t)slot * 2 * cs * kTile;

    const int cin_bytes = c.cin * ES;
    const __amdgpu_buffer_rsrc_t rs_in = ws_rsrc(c.in_data, (uint64_t)c.n * c.h * c.w * cin_bytes);
    const __amdgpu_buffer_rsrc_t rs_w = ws_rsrc(c.wpacked, (uint64_t)npass * cs * ksteps * 2 * COLS * 16);
    const uint32_t wlane = (uint32_t)(g * COLS + col) * 16u;   // this lane's place in a K-step's weight block
    const bool k_exact = kch * 32 == cin_bytes;                // no K-step reaches past the pixel's channels

    auto origin = [&](int p32) {
        // pixel index of tap (0,0) of the entry's window (only used when that tap is in bounds)
        const uint32_t pu = p32 >= 0 ? (uint32_t)p32 : 0u;
        const uint32_t t1 = fast_div(pu, c.div_ow);
        const int ox = (int)(pu - t1 * (uint32_t)c.ow);
        const uint32_t n = fast_div(t1, c.div_oh);
        const int oy = (int)(t1 - n * (uint32_t)c.oh);
        return ((int)n * c.h + oy * c.stride - c.pad) * c.w + ox * c.stride - c.pad;
    };
    auto tile_of = [&](int64_t wt, int ti) { return (wt * units_per_iter + slot) * TI + ti; };
    auto entry = [&](int64_t wt, int ti) {
        const int64_t j = tile_of(wt, ti) * kTile + col;
        if (wt >= r.end) return -1;
        if constexpr (SELF) return j < count ? self_px[j] : -1;   // (what lies behind belongs to the run's next workgroup)
        return list_pixel(l.list, j, count);
    };
    auto tap_word = [&](int64_t wt, int ti, int p32) -> uint32_t {
        if (SELF && self_tap != nullptr) return p32 >= 0 ? self_tap[tile_of(wt, ti) * kTile + col] & ((1u << (KS * KS)) - 1u) : 0u;
        if (l.taps == nullptr) return p32 >= 0 ? 1u : 0u;      // a 1x1 layer on its input's own list: its one tap
        const int64_t j = tile_of(wt, ti) * kTile + col;
        return (wt < r.end && j < count) ? (l.taps[j] & ((1u << (KS * KS)) - 1u)) : 0u;
    };

    int survivors = 0;
    for (int64_t wt = r.begin; wt < r.end; wt += r.step) {
        int p32[TI];
        uint32_t tb[TI], base00[TI];
        uint32_t any = 0;
#pragma unroll
        for (int ti = 0; ti < TI; ++ti) {
            p32[ti] = entry(wt, ti);
            tb[ti] = tap_word(wt, ti, p32[ti]);
            base00[ti] = (uint32_t)origin(p32[ti]) * (uint32_t)cin_bytes + (uint32_t)g * 16u;
            any |= tb[ti];
        }
        uint32_t wave_taps = 0;                                // taps any lane of the wave needs
#pragma unroll
        for (int t = 0; t < KS * KS; ++t)
            if (__ballot((any >> t) & 1)) wave_taps |= 1u << t;
        const int nsteps = __popc(wave_taps) * kch;

        for (int pass = 0; pass < npass; ++pass) {
            const int cgroup = pass * cs + part;               // which group of COLS output channels
            const int ch0 = cgroup * COLS;
            int nch = e.c - ch0;
            nch = nch < 0 ? 0 : (nch > COLS ? COLS : nch);
            f32x16 acc[TI][NB];
#pragma unroll
            for (int ti = 0; ti < TI; ++ti)
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[ti][b][i] = 0.0f;

            const uint32_t wpass = (uint32_t)cgroup * (uint32_t)ksteps;
            if constexpr (ROW) {
                static_assert(KS == 3 && D == 2, "row gathers: 3x3 windows, two operand sets");
                uint32_t rows = 0;                             // window rows any lane of the wave needs
#pragma unroll
                for (int dy = 0; dy < 3; ++dy)
                    if ((wave_taps >> (3 * dy)) & 7u) rows |= 1u << dy;
                const int rsteps = __popc(rows) * kch;
                struct RCur { uint32_t rest; int dy, kc; };    // dy == 3: past the end (gathers zeros, multiplies nothing)
                auto advance = [&](RCur& cu) {
                    if (cu.dy < 3 && ++cu.kc == kch) {
                        cu.kc = 0;
                        cu.rest &= cu.rest - 1;
                        cu.dy = cu.rest ? __builtin_ctz(cu.rest) : 3;
                    }
                };
                const bool first_col = col == 0, last_col = col == kTile - 1;
                struct RSet { Vec xc[TI], xe[TI], wv[3][NB]; };
                auto issue = [&](const RCur& cu, RSet& st) {
                    const bool live = cu.dy < 3;
                    const int dy = live ? cu.dy : 0;
                    const uint32_t uni = (uint32_t)(dy * c.w * cin_bytes + cu.kc * 32);
                    const bool chan_ok = live && (k_exact || (2 * cu.kc + g) * 16 < cin_bytes);
#pragma unroll
                    for (int ti = 0; ti < TI; ++ti) {
                        const uint32_t three = (tb[ti] >> (3 * dy)) & 7u;
                        const uint32_t row0 = base00[ti] + uni;
                        uint32_t offc = (chan_ok && (three & 2u)) ? row0 + (uint32_t)cin_bytes : kOob;
                        uint32_t offe = !chan_ok ? kOob
                                        : (first_col && (three & 1u)) ? row0
                                        : (last_col && (three & 4u)) ? row0 + 2u * (uint32_t)cin_bytes : kOob;
                        asm volatile("" : "+v"(offc));
                        asm volatile("" : "+v"(offe));
                        st.xc[ti] = ws_load16<Vec>(rs_in, offc);
                        st.xe[ti] = ws_load16<Vec>(rs_in, offe);
                    }
                    const uint32_t wave_three = live ? (wave_taps >> (3 * dy)) & 7u : 0u;
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx) {
                        const uint32_t woff = ((wave_three >> dx) & 1u)
                                                  ? wlane + (wpass + (uint32_t)((3 * dy + dx) * kch + cu.kc)) * (uint32_t)(2 * COLS * 16)
                                                  : kOob;
#pragma unroll
                        for (int b = 0; b < NB; ++b)
                            st.wv[dx][b] = ws_load16<Vec>(rs_w, woff == kOob ? kOob : woff + (uint32_t)b * (32u * 16u));
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                // the centre column moved by one lane: lane l takes lane l-1 (from_below) or lane l+1; the tile's
                // edge lanes take what they fetched themselves; a lane whose tap is not flagged takes zeros
                auto moved = [&](const Vec& v, bool from_below, bool take, bool edge, const Vec& ev) -> Vec {
                    const u32x4 w = __builtin_bit_cast(u32x4, v), o = __builtin_bit_cast(u32x4, ev);
                    u32x4 rr;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int sft = from_below ? __builtin_amdgcn_update_dpp(0, (int)w[i], 0x138, 0xf, 0xf, true)    // wave_shr:1
                                                   : __builtin_amdgcn_update_dpp(0, (int)w[i], 0x130, 0xf, 0xf, true);   // wave_shl:1
                        rr[i] = edge ? o[i] : (take ? (uint32_t)sft : 0u);
                    }
                    return __builtin_bit_cast(Vec, rr);
                };
                auto mma = [&](const RCur& cu, const RSet& st) {
                    const bool live = cu.dy < 3;
                    const int dy = live ? cu.dy : 0;
                    const uint32_t wave_three = live ? (wave_taps >> (3 * dy)) & 7u : 0u;
#pragma unroll
                    for (int ti = 0; ti < TI; ++ti) {
                        const uint32_t three = live ? (tb[ti] >> (3 * dy)) & 7u : 0u;
                        const Vec xl = moved(st.xc[ti], true, three & 1u, first_col, st.xe[ti]);
                        const Vec xr = moved(st.xc[ti], false, three & 4u, last_col, st.xe[ti]);
#pragma unroll
                        for (int dx = 0; dx < 3; ++dx) {
                            if (!((wave_three >> dx) & 1u)) continue;
#pragma unroll
                            for (int b = 0; b < NB; ++b)
                                Mma<T>::run(acc[ti][b], st.wv[dx][b], dx == 0 ? xl : (dx == 1 ? st.xc[ti] : xr));
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                RSet sa, sb;
                RCur cg{rows, rows ? __builtin_ctz(rows) : 3, 0};
                RCur cm = cg;
                issue(cg, sa); advance(cg);
                for (int s = 0; s < rsteps; s += 2) {
                    issue(cg, sb); advance(cg);
                    mma(cm, sa); advance(cm);
                    issue(cg, sa); advance(cg);
                    mma(cm, sb); advance(cm);
                }
            } else {
            // Wave-uniform cursor over the K-steps that matter: (flagged tap, channel group) pairs in order.
            // Past the end a step gathers zeros and multiplies them with the (valid) first weight block.
            // Every load is issued unconditionally (a lane with nothing to fetch gets an offset outside the
            // descriptor), so the number of loads in flight at each wait is known at compile time.
            struct Cur { uint32_t rest; int t, kc; };
            auto issue = [&](Cur& cu, Vec (&x)[TI], Vec (&wv)[NB]) {
                const bool live = cu.t != kNoTap;
                const int t = live ? cu.t : 0;
                const uint32_t tbit = live ? 1u << t : 0u;
                const int dy = t / KS, dx = t - dy * KS;
                const uint32_t uni = (uint32_t)((dy * c.w + dx) * cin_bytes + cu.kc * 32);
                const bool chan_ok = k_exact || (2 * cu.kc + g) * 16 < cin_bytes;
#pragma unroll
                for (int ti = 0; ti < TI; ++ti) {
                    uint32_t off = (chan_ok && (tb[ti] & tbit)) ? base00[ti] + uni : kOob;
                    asm volatile("" : "+v"(off));              // one load at a computed offset, not a load per case
                    x[ti] = ws_load16<Vec>(rs_in, off);
                }
                const uint32_t woff = wlane + (wpass + (uint32_t)(t * kch + cu.kc)) * (uint32_t)(2 * COLS * 16);
#pragma unroll
                for (int b = 0; b < NB; ++b) wv[b] = ws_load16<Vec>(rs_w, woff + (uint32_t)b * (32u * 16u));
                if (live && ++cu.kc == kch) {
                    cu.kc = 0;
                    cu.rest &= cu.rest - 1;
                    cu.t = cu.rest ? __builtin_ctz(cu.rest) : kNoTap;
                }
                __builtin_amdgcn_sched_barrier(0);             // the scheduler must not sink the loads below the MFMAs
            };
            auto mma = [&](const Vec (&x)[TI], const Vec (&wv)[NB]) {
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int ti = 0; ti < TI; ++ti) Mma<T>::run(acc[ti][b], wv[b], x[ti]);
                __builtin_amdgcn_sched_barrier(0);
            };
            // ring of D register sets: the operands of D - 1 K-steps travel while one step is multiplied
            Vec x[D][TI], w[D][NB];
            Cur cu{wave_taps, wave_taps ? __builtin_ctz(wave_taps) : kNoTap, 0};
#pragma unroll
            for (int i = 0; i < D - 1; ++i) issue(cu, x[i], w[i]);
            for (int s = 0; s < nsteps; s += D) {
#pragma unroll
                for (int j = 0; j < D; ++j) {
                    issue(cu, x[(j + D - 1) % D], w[(j + D - 1) % D]);
                    mma(x[j], w[j]);
                }
            }
            }

            // ---- tail: this wave's channel slice of each of its tiles -------------------------------
            const MaxExchange mx{xchg, cs, part};
            const bool exchange = cs > 1 && full_tail && e.act != DCNN_ACT_NONE;
#pragma unroll
            for (int ti = 0; ti < TI; ++ti) {
                stage_accumulators<T, NB>(acc[ti], stage + (size_t)col * stage_stride, g);
                lds_wave_sync();
                auto dx = [&](int ent, int64_t, int c0) -> Raw {
                    return raw_load<T, V>(reinterpret_cast<const T*>(stage + (size_t)ent * stage_stride) + (c0 - ch0));
                };
                uint32_t bits;
                if (exchange) bits = act_trunc_tile<T, V, 1, 2, true>(e, false, p32[ti], lane, dx, ch0, nch, COLS, mx);
                else bits = act_trunc_tile<T, V, 1, 2, false>(e, false, p32[ti], lane, dx, ch0, nch, COLS, mx);
                const int64_t tile = tile_of(wt, ti);
                if (full_tail && part == 0 && tile * kTile < count) {
                    if (e.surv) { if (lane == 0) e.surv[tile] = bits; }
                    else survivors += __popc(bits);
                }
                lds_wave_sync();
            }
        }
    }
    // one atomic per wave: a counter bumped once per tile by every wave serialises in L2
    if (e.out_count && !e.surv && lane == 0 && survivors) atomicAdd(e.out_count, survivors);
}

// Lists too short to keep the chip busy with TI tiles per wave run one tile per wave and a deeper ring instead
// (more waves, more loads in flight); the length of the list is only known on the device.
// SH (fp16): the waves that share a tile, the plan's `cs`, one kernel each: with the bodies of all three in one kernel it spilled (28-36 bytes
// of scratch a lane for two column blocks, 100 KB of code); 3x3 128->128 on 8 streams of 256x256 with a tenth of the pixels new, a
// step 204 us -> 201, 128->64 on 8 of 128x128 with 2 % flagged 60 -> 58.  fp32, whose waves share nothing: 0, and `cs` as the kernel finds it.
template <typename T, int NB, int KS, int SH, bool SELF>
__global__ __launch_bounds__(kDirectWaves* kWave, 2) void conv_direct_kernel(ListParam<SELF> l, ConvArgs c, EpilogueArgs e, int npass, int cs,
                                                                             int blocked_min_tiles) {
    static_assert((SH == 0) == (sizeof(T) == 4), "fp16 tiles are shared by a fixed number of waves");
    extern __shared__ __align__(16) unsigned char smem[];
    clear_ahead(e);
    WarmL2 warm;
    warm.request<kDirectWaves * kWave>(c.wpacked, (uint64_t)npass * cs * KS * KS * c.kch * (2 * NB * 32 * 16));
    if constexpr (SELF) {
        if ((int)blockIdx.x < l.writers) {
            local_write<kDirectWaves * kWave>(l, smem + l.lds_scratch);
            return;
        }
        // Maps whose lists are built here are too small for more than one tile per wave.  The layer's weights are fetched for every
        // tile, so tiles are filled from a run of pixels (local_run) and each workgroup of the run takes its share of them.  2 / 10 /
        // 30 % of the pixels flagged at random, a workgroup per 32 pixels as they lie -> runs: 3x3 128->128 + ReLU on 128x128 pixels
        // 19.3 / 21.2 / 22.4 -> 17.7 / 20.5 / 21.4 us, 256->256 on 8 streams of 28x28 24.2 / 25.5 / 26.1 -> 23.3 / 24.5 / 25.4.
        static_assert(kDirectWaves * kWave == kRunPixels, "a pixel per thread");
        const RunPart rp = run_part((int)blockIdx.x - l.writers, (l.m_out_px + kRunPixels - 1) / kRunPixels, l.run_parts);
        const int32_t* px;
        const uint32_t* tap;
        const int all = local_run(l, smem + l.lds_list, rp.run, rp.part == 0, px, tap);
        const int share = run_share(all, l.run_parts, l.run_even), from = rp.part * share;
        const int count = min(all - from, share);              // (none where the run lists fewer)
        warm.arrived();
        if (count <= 0) return;
        px += from;
        tap = l.want_taps ? tap + from : nullptr;
        if constexpr (sizeof(T) == 4) conv_lane_body<T, NB, KS, 1, (NB >= 4 ? 6 : 8), false, SELF>(l, c, e, npass, cs, count, smem, px, tap);
        else conv_direct_body<T, NB, KS, 1, SH, true>(l, c, e, npass, count, smem, px, tap);
    } else {
        const int64_t count = list_count(l);
        warm.arrived();
        const bool blocked = count >= (int64_t)blocked_min_tiles * kTile;
        if constexpr (sizeof(T) == 4) {
            if (blocked) {
                if constexpr (KS == 3 && NB <= 2) {
                    // Row gathers pay when most taps of the listed windows are flagged.  Every flagged input pixel is a tap
                    // of (up to) nine listed outputs, so flagged inputs / listed outputs IS the mean fraction of flagged taps
                    // per window; three quarters, as measured when fp16 layers took them too (halves: 4 % slower).
                    // (an input that comes without a count: the rule of the resident-weight kernel, most of the map listed)
                    const bool dense_taps = c.in_count ? (int64_t)*c.in_count * 4 >= count * 3
                                                       : count * 4 >= (int64_t)c.n * c.oh * c.ow * 3;
                    if (c.stride == 1 && c.pad == 1 && dense_taps) {
                        conv_lane_body<T, NB, KS, 3, 2, true, SELF>(l, c, e, npass, cs, count, smem, nullptr, nullptr);   // 3 tiles: two operand sets of 12 vectors fit beside 96 accumulators
                        return;
                    }
                }
                conv_lane_body<T, NB, KS, direct_tiles(NB, 4, 4), 3, false, SELF>(l, c, e, npass, cs, count, smem, nullptr, nullptr);
            } else {
                conv_lane_body<T, NB, KS, 1, (NB >= 4 ? 6 : 8), false, SELF>(l, c, e, npass, cs, count, smem, nullptr, nullptr);
            }
        } else if (blocked) {
            conv_direct_body<T, NB, KS, direct_tiles(NB, 2, SH), SH, false>(l, c, e, npass, count, smem, nullptr, nullptr);
        } else {
            conv_direct_body<T, NB, KS, 1, SH, false>(l, c, e, npass, count, smem, nullptr, nullptr);
        }
    }
}

}  // namespace dcnn
