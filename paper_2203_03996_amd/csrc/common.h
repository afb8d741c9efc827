// Internal declarations shared by the translation units of libdeltacnn (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <type_traits>

#include "../../include/deltacnn.h"

namespace dcnn {

constexpr int kWave = 64;            // gfx950 wavefront
constexpr int kTile = 32;            // list entries one wave processes at a time (= MFMA N)
constexpr int kChunk = 2048;         // pixels per workgroup in the pixel-space mask passes
constexpr int kXcd = 8;              // accelerator complex dies, each with its own L2
constexpr size_t kAlign = 256;

inline size_t align_up(size_t v, size_t a = kAlign) { return (v + a - 1) / a * a; }
inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t dtype_size(int dt) { return dt == DCNN_F16 ? 2 : 4; }

// Division of a 31-bit unsigned number by a constant known on the host: q = (mulhi(n, m) + n) >> s
// with s = ceil(log2 d), m = ceil(2^(32+s) / d) - 2^32.  Exact for 0 <= n < 2^31.
struct FastDiv {
    uint32_t m, s, d;
};
inline FastDiv make_fastdiv(uint32_t d) {
    FastDiv f;
    f.d = d;
    f.s = 0;
    while ((1ull << f.s) < d) ++f.s;
    f.m = (uint32_t)((((1ull << (32 + f.s)) + d - 1) / d) - (1ull << 32));
    return f;
}

}  // namespace dcnn

struct dcnn_ctx {
    hipStream_t stream;
    int device;              // HIP device that was current when the context was created
    char* ws;
    size_t ws_bytes;
    int num_cu;
    size_t max_lds;
    char err[512];
};

namespace dcnn {

dcnn_status fail(dcnn_ctx* ctx, dcnn_status s, const char* fmt, ...);
dcnn_status check_hip(dcnn_ctx* ctx, hipError_t e, const char* what);

// Workspace carve-up (all offsets 256-byte aligned).
struct Workspace {
    int32_t* chunk_counts;   // one per kChunk pixels
    uint32_t* surv;          // one survivor word per kTile list entries
    uint8_t* scratch_mask;   // mask of a pass whose caller only wants the list
    uint8_t* scratch_mask2;  // second intermediate mask (separable dilation of the input mask)
    int64_t max_pixels;
};
size_t workspace_bytes(int64_t max_pixels);
dcnn_status workspace_view(dcnn_ctx* ctx, int64_t pixels, Workspace* out);

// ---- kernel launchers (defined in the *.hip files) -------------------------------------------
struct MaskPassArgs {
    const uint8_t* mask_in;      // [n,h,w] or nullptr (treated as all zero)
    const uint8_t* mask_b;       // [n,oh,ow] or nullptr
    uint8_t* mask_out;           // [n,oh,ow] or nullptr
    int32_t* idx_out;            // may be nullptr (then only mask_out is written)
    int32_t* count_out;
    int n, h, w, oh, ow, k, stride, pad;
    int up;                      // > 1: nearest upsampling of the input mask by this factor (k = 1)
    int bilinear;                // with up > 1: bilinear upsampling instead (sources that carry weight)
    int emit_only;               // 1: mask_in is final and its flags have been counted: counts_per_chunk numbers per chunk of
    const int32_t* counts;       //    pixels, in `counts`
    int counts_per_chunk;
    uint32_t* taps_out;          // optional [n*oh*ow]: per list entry, which window taps are flagged (k*k <= 25 bits);
                                 // bit 30: the entry's pixel is flagged in mask_b
    int b_stride, b_h, b_w;      // b_stride > 0: mask_b is [n,b_h,b_w] and output pixel (y,x) looks at (y,x)*b_stride
    int kw, pad_w;               // kw > 0: the window is k rows x kw columns with padding pad / pad_w (stride 1)
};
dcnn_status launch_mask_compact(dcnn_ctx* ctx, const MaskPassArgs& a);
// Resolves the device address of the library's static scratch array for HIP device `dev`, which must be the
// current device (set-up step of dcnn_mask_compact_static; called by dcnn_ctx_create).
hipError_t static_scratch_setup(int dev);

// Ordered compaction of the entries of a work list that survived (bit set in surv).
dcnn_status launch_emit_sublist(dcnn_ctx* ctx, const int32_t* list, const int32_t* count, int64_t max_count,
                                const uint32_t* surv, int32_t* idx_out, int32_t* count_out);
dcnn_status launch_fill_i32(dcnn_ctx* ctx, int32_t* p, int32_t v, int64_t n);
// Statistics (never on a timed path): *out = number of non-zero bytes among mask[0 .. pixels).
dcnn_status launch_mask_sum(dcnn_ctx* ctx, const uint8_t* mask, int64_t pixels, int32_t* out);
// flags[p] = 1 iff row p of `data` ([pixels, c] elements) has a non-zero bit.
dcnn_status launch_row_flags(dcnn_ctx* ctx, int dtype, const void* data, uint8_t* flags, int64_t pixels, int c);
// Zeroes a set of 16-byte aligned pieces of device memory (lengths are rounded up to 16 bytes): the mask, count and flag
// arrays of one layer or of a whole network, one launch for up to kClearPieces of them.
struct ClearPiece {
    void* p;
    int64_t bytes;
};
constexpr int kClearPieces = 120;
dcnn_status launch_clear(dcnn_ctx* ctx, const ClearPiece* pieces, int n);

// Element-wise tail shared by CONV / ACT: (+bias) (+residual) activation, truncation, state.
struct EpilogueArgs {
    int c;                       // channels of the output pixel
    int act;                     // dcnn_act
    float eps;
    const void* bias;            // [c] or nullptr (first frame only)
    const void* res_data;        // second delta stream (output shape) or nullptr
    const uint8_t* res_mask;     // nullptr in the first frame (dense residual)
    void* xA;                    // nullptr when act == NONE
    void* xT;
    void* out_data;
    uint8_t* out_mask;           // written at every visited pixel (0 or 1); nullptr: not written
    uint32_t* surv;              // survivor word per tile; nullptr: not written
    int32_t* out_count;          // when surv is null: survivors are added here, one atomic per wave.  The layer code
                                 // passes nullptr: atomics on one address are served one after the other, and a
                                 // few thousand of them at the end of a kernel cost 10-20 us (see dcnn_layer_step)
    uint8_t* xt_flags;           // optional, per output pixel: 0 = the pixel's x^T row is all zero bits in memory and is
                                 // not read; 1 = it may hold values.  Kept up to date by the wave-specialised kernel only.
                                 // First frame: rows whose flag is 0 are not cleared again (null: every row is).
    void* accum_O;               // fused final accumulation: dense output O (output shape); the emitted delta is
                                 // added to it and not stored (sparse steps of layers with an activation only)
    int carry;                   // 1: an update leaves the rounding residue of x^A in x^T (s - round(s)) instead of 0
    uint8_t* clear_mask;         // optional: a byte array every workgroup of the grid zeroes a share of before anything else
    int64_t clear_bytes;         // (the output mask of the layer's NEXT step, see dcnn_layer_step)
};

struct StoredList {
    const int32_t* list;         // nullptr: identity (entry j is pixel j)
    const int32_t* count;        // nullptr: use count_host
    int64_t count_host;
    int64_t max_count;           // upper bound used to size the grid
    const uint32_t* taps;        // optional, per entry: bit t set iff window tap t of the entry's pixel is in
                                 // bounds and flagged in the input mask (written with the list by the mask pass)
};
// ... or built by the kernel itself from the masks (self_list.h); list, count and taps are then null.
struct ListArgs : StoredList {
    int self;
    int want_taps;               // ... with the entries' tap words (bit 30: flagged in m_b)
    const uint8_t* m_in;         // input mask [n, m_h, m_w]
    const uint8_t* m_b;          // second mask, as in MaskPassArgs, or nullptr
    int m_in_px, m_out_px, m_h, m_w, m_oh, m_ow, m_k, m_stride, m_pad, m_up;
    int b_stride, b_h, b_w;
    FastDiv div_ow, div_oh, div_iw, div_ih, div_up;
    uint8_t* mask_out;           // what the kernel writes for others, each may be null: the flags of the list,
    int32_t* idx_out;            // the ascending list,
    int32_t* count_out;          // its length
    int32_t* in_idx_out;         // the ascending list of the INPUT's flagged pixels and its length, on behalf of a producer that
    int32_t* in_count_out;       //    leaves it to this kernel, or both null
    uint8_t* mask_zero;          // 0 at every pixel that is not listed (the kernel itself writes the decision at those that are)
    int lds_scratch, lds_list;   // byte offsets into the kernel's dynamic LDS (set by the launchers)
    int lds_entries;             // room for this many entries
    // Kernels whose workgroups compact blocks of pixels of their own (local_build) instead of cutting up the map's list:
    int writers;                 // the first workgroups of the grid write what belongs to the whole map
    union { int local_shift;     // a block is 1 << local_shift pixels
            int run_even; };     // or, where workgroups share runs of pixels (local_run): how (run_share)
    union { int local_slots;     // pixels per workgroup: its blocks, whole
            int run_parts; };    // or the workgroups that share a run
};
// What a kernel takes: the five words of a stored list where it walks one.  (All of ListArgs on every launch, 250 bytes of
// arguments more, cost 0.4 us a launch: activations of 5-11 us 5-8 % slower.)
template <bool SELF> using ListParam = std::conditional_t<SELF, ListArgs, StoredList>;

// ---- work lists built by the kernel itself (host side; self_list.h has the device side) ---------------------------
constexpr int64_t kListMaxPixels = 65536;    // mask_list_kernel: input and output pixels (positions are kept in 16 bits)
// Layers in whose kernel some workgroup forms all of the map's flags on the way: plain convolutions of windows other than 1x1 and 3x3,
// upsampling (its writers), and kernels that fetch the weights for every tile (register-blocked, units, plain).  Forming them costs
// 3-4 us up to 16 K pixels and 5-8 beyond, against ~6 us for a launch of mask_list_kernel.
constexpr int64_t kSelfMaxPixels = 16384;
// Layers whose workgroups compact blocks of their own (local_build; activations, depthwise and wave-specialised convolutions): as far as
// the writers' 16-bit positions reach.  Steps with this limit at 16 K pixels -> here, 8 streams: HRNet-shaped 1126 -> 1012 us,
// ResNet-50-shaped 1250 -> 1213.  Nearest upsampling stays at 16 K: its writers expand the flags, 18 us on 55 K pixels against 11 on a
// stored list.
constexpr int64_t kLocalMaxPixels = kListMaxPixels;
constexpr int64_t kLocalMaxSampled = 49152;  // outputs whose second mask is sampled (layer_lists_itself)
inline size_t self_scratch_bytes(int64_t in_px, int64_t out_px) {
    return align_up(128 + 4 * (size_t)(2 * cdiv(in_px, 32) + cdiv(out_px, 32)) + 2 * (size_t)cdiv(out_px, 32), 16);
}
// How a list is cut into groups of entries and the groups are dealt out.  Kernels walk by these rules and launchers size the
// room of lists built in place by them, so there is one of each.  Activation and depthwise kernels walk whole tiles -- every
// part of a survivor word gets written -- and may own up to three groups of eight entries behind a list's last one.
constexpr int kTileWaves = 4;                                  // waves per workgroup of the activation and depthwise kernels
constexpr int kWideRun = 8;                                    // entries per workgroup and step of act_wide_kernel (a quarter tile)
__host__ __device__ inline int64_t wide_groups(int64_t count) { return (count + kTile - 1) / kTile * (kTile / kWideRun); }
__host__ __device__ inline int64_t run_groups(int64_t count, int run) {        // kTileWaves runs of `run` entries
    return ((count + kTile - 1) / kTile * (kTile / run) + kTileWaves - 1) / kTileWaves;
}
// Groups begin, begin + step, ... below end are workgroup `block`'s: consecutive groups stay on one XCD and share its L2
// (workgroup b runs on XCD b % 8; an XCD owns a contiguous range, its workgroups stride through it).
struct WgTileRange { int64_t begin, end, step; };
__host__ __device__ inline WgTileRange tile_range(int64_t groups, uint32_t block, uint32_t grid) {
    const int64_t per = (groups + kXcd - 1) / kXcd, xcd = block % kXcd;
    const int64_t end = (xcd + 1) * per;
    return {xcd * per + block / kXcd, end < groups ? end : groups, grid / kXcd};
}
// Tiles per round of a workgroup of the wave-specialised convolution that has room for `slots` of them: as few as go round the grid
// once.  The vector memory path of one compute unit is what a short list waits for (64-72 clocks per load instruction, ~50 of them
// per 3x3 tile of 64 channels): with always eight tiles to a workgroup a list of 4000 entries ran on 16 of 256 compute units.  Spread:
// fp32 3x3 32->32 + ReLU on 64x64 27.6 -> 21.8 us with its input layer, the bottleneck block on one 128x128 stream 53.1 -> 47.5,
// a four-resolution network on 8 streams 1399 -> 1325; lists that fill the chip anyway (64 streams) the same.
__host__ __device__ inline int ws_slots(uint32_t tiles, uint32_t grid, int slots) {
    const int each = (int)((tiles + grid - 1) / grid);
    return each < 1 ? 1 : (each < slots ? each : slots);
}
// entries of the groups that one workgroup of `grid` owns at most (tile_range)
inline int64_t self_local_entries(int64_t out_px, int64_t entries_per_group, int grid) {
    const int64_t groups = cdiv(out_px, entries_per_group);
    const int64_t mine = cdiv(cdiv(groups, kXcd), grid / kXcd);
    return (mine < 1 ? 1 : mine) * entries_per_group;
}

// Blocks that workgroups compact for themselves (local_build in self_list.h).  Workgroups of one launch: the writers of what
// belongs to the whole map, then the owners of pixels.
constexpr int kLocalHeader = 64;                               // bytes of counts ahead of a workgroup's entries
inline int local_writers(const ListArgs& l) {
    // (only the ascending list is shared out; the input's list and the lengths are the first one's)
    if (l.idx_out == nullptr) return l.count_out != nullptr || l.in_idx_out != nullptr ? 1 : 0;
    const int64_t px = l.m_in_px > l.m_out_px ? l.m_in_px : l.m_out_px, w = cdiv(px, 8192);
    return (int)(w < 8 ? w : 8);
}
struct LocalShape { int owners, slots, entries; };             // workgroups with pixels, pixels of each, room for entries
// `group`: entries that a workgroup walks per iteration; owners_cap: workgroups that are worth having
inline LocalShape local_shape(int64_t out_px, int local_shift, int64_t owners_cap, int group) {
    const int64_t blocks = cdiv(out_px, 1 << local_shift);
    LocalShape s;
    s.owners = (int)(blocks < owners_cap ? blocks : owners_cap);
    s.slots = (int)cdiv(blocks, s.owners) << local_shift;
    s.entries = (int)(cdiv(s.slots, group) * group);
    return s;
}

// Activation, depthwise and upsampling kernels: a block per workgroup, of as many pixels as it walks in one iteration (`group`
// entries), 32 at most -- or 64 on maps that would have more than 1024 blocks, of which four fit a compute unit.
inline int tile_local_shift(int64_t out_px, int group) {
    int shift = 3;
    while (shift < 6 && ((1 << shift) < (group < 32 ? group : 32) || cdiv(out_px, 1 << shift) > 1024)) ++shift;
    return shift;
}

// Runs of consecutive pixels that `parts` workgroups compact, each for itself, and divide among themselves (local_run in self_list.h).
constexpr int kRunPixels = 256, kRunTiles = kRunPixels / kTile;
constexpr int kRunLds = kLocalHeader + kRunPixels * 8;
// as many workgroups as a run has tiles, or fewer (a power of two) where `chip` of them are there as it is; `rest`: workgroups per tile
inline int run_parts(int64_t out_px, int64_t rest, int64_t chip) {
    const int64_t want = cdiv(chip, cdiv(out_px, kRunPixels) * rest);
    int parts = 1;
    while (parts < want && parts < kRunTiles) parts *= 2;
    return parts;
}
// Workgroup `item` of the owners' -> run and part.  A scattered update lists a part or two of each run, a clustered one all parts of
// some: first parts lie ahead of second ones, and each lot is turned against the one before, so that either way the workgroups with
// work are spread over XCDs and compute units (not turned, a clustered 3x3 256->256 on 4096 pixels had two on some units and none on
// others).
struct RunPart { int run, part; };
__host__ __device__ inline RunPart run_part(int item, int runs, int parts) {
    const int part = item / runs, run = item - part * runs - part * runs / parts;
    return {run < 0 ? run + runs : run, part};
}
// A workgroup's share of a run's entries: whole tiles, or (`even`) the same number for each, 16 at least -- a tile takes as long
// as its pixels' lines do, so where every part has a SIMD to itself full tiles on some of them are the slower way.
__host__ __device__ inline int run_share(int count, int parts, int even) {
    if (!even) return ((count + kTile - 1) / kTile + parts - 1) / parts * kTile;
    const int each = (count + parts - 1) / parts;
    return each > kTile / 2 ? each : kTile / 2;
}

// Statistics (never on a timed path): x^T rows a convolution that keeps row flags reads and writes in one step.
// phase 0, before the step's kernel: before[j] = flag of list entry j's pixel, io[0] = their number (rows read);
// phase 1, after it: io[1] = entries whose row held values before or holds values now (rows written).
dcnn_status launch_xt_row_count(dcnn_ctx* ctx, int phase, const ListArgs& l, const uint8_t* flags, uint8_t* before,
                                unsigned long long* io);

struct ConvArgs {
    const void* in_data;
    const uint8_t* in_mask;      // nullptr: every in-bounds pixel is flagged (first frame)
    const int32_t* in_count;     // optional, device: number of flagged input pixels (how dense the window taps are)
    const void* wpacked;
    const void* zero_page;       // >= 16 bytes of zeros: what lanes read instead of an unflagged / padded input
    int n, h, w, cin, oh, ow, cout, cout_pad, k, stride, pad, kch;
    int depthwise;
    int flat;                    // filled by launch_conv: kch counts K-steps over the flat (tap, channel) dimension
    FastDiv div_ow, div_oh;      // filled by launch_conv
    // optional projection: a 1x1 convolution (stride2, no padding) of a second input [n,h2,w2,cin2] whose
    // result is added to this one's before the epilogue; its update flag is bit 30 of the list's tap words
    const void* in2_data;        // nullptr: none
    const void* wpacked2;
    const void* bias2;           // first frame only
    int h2, w2, cin2, stride2, kch2;
};
dcnn_status launch_conv(dcnn_ctx* ctx, int dtype, bool init, const ListArgs& l, const ConvArgs& c,
                        const EpilogueArgs& e);
size_t conv_packed_weight_bytes(int dtype, int k, int cin, int cout, int depthwise, bool fused);
dcnn_status launch_pack_weights(dcnn_ctx* ctx, int dtype, const void* w, void* wpacked, int k, int cin, int cout,
                                int depthwise, bool fused);
bool conv_supported(const dcnn_ctx* ctx, int dtype, int k, int cin, int cout, int depthwise, bool fused,
                    char* why, size_t why_len);
// Convolution + activation with a fused 1x1 projection of a second input (cin2 channels): supported when the
// sparse step can run on the wave-specialised kernel with both weight tensors resident in LDS.
// Convolution + activation whose sparse step runs on the wave-specialised kernel (needed for a fused final
// accumulation).
bool conv_ws_supported(const dcnn_ctx* ctx, int dtype, int k, int cin, int cout, int64_t in_elems, int64_t out_elems);
bool conv_proj_supported(const dcnn_ctx* ctx, int dtype, int k, int cin, int cin2, int cout, int64_t in_elems,
                         int64_t in2_elems, int64_t out_elems);
// Maps on which layers with streamed weights run one wave per (tile, channel block) (conv_unit.hip).
constexpr int64_t kUnitMaxPixels = 16384;
// Can the sparse steps of this convolution build their work list in the kernel, and is it the better way?  (LDS room in every kernel
// that may serve them.)
bool conv_self_fits(const dcnn_ctx* ctx, int dtype, int k, int cin, int cout, bool fused, int cin2, int64_t in_px,
                    int64_t out_px);
size_t conv_proj_weight_bytes(int dtype, int k, int cin, int cin2, int cout);
// Packs the projection's [cin2][cout] weights in the column grouping of the main convolution's plan.
dcnn_status launch_pack_weights_proj(dcnn_ctx* ctx, int dtype, const void* w2, void* wpacked2, int k, int cin, int cin2,
                                     int cout);

struct ActArgs {
    const void* in_data;         // first delta stream
    const uint8_t* in_mask;      // nullptr: always valid (single input: the list is its mask)
};
dcnn_status launch_act(dcnn_ctx* ctx, int dtype, bool init, const ListArgs& l, const ActArgs& a,
                       const EpilogueArgs& e);
dcnn_status launch_dwconv(dcnn_ctx* ctx, int dtype, bool init, const ListArgs& l, const ConvArgs& c,
                          const EpilogueArgs& e);
// Do the sparse steps of such a layer run on a kernel that can build its work list?
bool act_self_fits(int dtype, int channels, int64_t pixels);
bool dwconv_self_fits(int dtype, int k, int channels, int64_t in_px, int64_t out_px);

struct DeltaGenArgs {
    const void* frame;
    void* P;
    void* out_data;
    uint8_t* out_mask;
    int32_t* out_idx;
    int32_t* out_count;
    int64_t pixels;
    int n, h, w, c;
    float eps;
    int dilate_r;
    int mask_only;               // 1: nobody walks the list, only mask and values are written (dilate_r == 0)
};
dcnn_status launch_deltagen(dcnn_ctx* ctx, int dtype, const DeltaGenArgs& a);
dcnn_status launch_copy(dcnn_ctx* ctx, void* dst, const void* src, size_t bytes);

struct AccumArgs {
    const void* in_data;
    void* O;
    int c;
};
dcnn_status launch_accum(dcnn_ctx* ctx, int dtype, const ListArgs& l, const AccumArgs& a);

struct PoolArgs {
    const void* in_data;         // delta at flagged input pixels
    const uint8_t* in_mask;
    void* xA;                    // accumulated dense input [n,h,w,c]
    void* out_data;              // [n,oh,ow,c]
    int n, h, w, c, oh, ow, k, stride, pad;
};
// work list = flagged OUTPUT pixels; a second pass over the flagged INPUT pixels folds the delta into xA
dcnn_status launch_maxpool_out(dcnn_ctx* ctx, int dtype, bool init, const ListArgs& l, const PoolArgs& a);
dcnn_status launch_maxpool_commit(dcnn_ctx* ctx, int dtype, const ListArgs& l_in, const PoolArgs& a);

struct ConcatArgs {
    const void* a_data;          // [pixels, ca]
    const void* b_data;          // [pixels, cb]
    const uint8_t* a_mask;       // nullptr: dense (first frame)
    const uint8_t* b_mask;
    void* out_data;              // [pixels, ca + cb]
    int ca, cb;
};
dcnn_status launch_concat(dcnn_ctx* ctx, int dtype, const ListArgs& l, const ConcatArgs& a);

struct UpsampleArgs {
    const void* in_data;
    void* out_data;
    int n, h, w, c, factor;
    int bilinear;                // 0: nearest neighbour; 1: bilinear, half-pixel centres
    const uint8_t* in_mask;      // bilinear: unflagged sources count as zero (nullptr: all flagged)
};

// Global average pooling: one list entry per stream with an update; out[n, c] = sum over the stream's flagged
// pixels / (h * w).
struct GapArgs {
    const void* in_data;         // [n, h*w, c]
    const uint8_t* in_mask;      // nullptr: every pixel counts (first frame)
    void* out_data;              // [n, c]
    int hw, c;
};
dcnn_status launch_gavgpool(dcnn_ctx* ctx, int dtype, const ListArgs& l_out, const GapArgs& a);
dcnn_status launch_upsample(dcnn_ctx* ctx, int dtype, const ListArgs& l_out, const UpsampleArgs& a);

}  // namespace dcnn
