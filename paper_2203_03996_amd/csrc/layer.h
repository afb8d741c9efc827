// Internal layout of a layer object (shared by layer.hip and net.hip).
#pragma once

#include <utility>
#include <vector>

#include "common.h"

struct dcnn_layer {
    dcnn_ctx* ctx;
    dcnn_layer_desc d;
    int oh, ow, oc;
    int64_t in_pixels, out_pixels;
    bool inited;
    bool alias_mask;            // output mask / index list are those of input 0
    bool has_bias;
    bool self = false;          // sparse steps build their work list in the layer's own kernel (self_list.h)
    bool skip_list = false;     // input layer of a network whose list is written by a consumer's kernel (in_idx_out), not by its own
    int32_t* in_idx_out = nullptr;      // such a consumer: where the input layer's list and its length go
    int32_t* in_count_out = nullptr;
    bool has_bias2 = false;     // bias of the fused projection
    size_t state_bytes;
    // pieces of the caller-provided state memory
    void* buf0; size_t buf0_bytes;      // x^A | stored input frame | dense output
    void* buf1; size_t buf1_bytes;      // x^T
    void* buf2; size_t buf2_bytes;      // dense accumulated output of a layer with fuse_accum
    void* out_data;
    uint8_t* out_mask;
    int32_t* out_idx;
    int32_t* out_count;
    uint8_t* out_mask_alt;              // second output mask of a layer that alternates between two (see dcnn_layer_step)
    int mask_phase;                     // which of the two the NEXT step writes
    int32_t* list;                      // work list when the layer builds its own
    int32_t* list_count;
    uint32_t* taps;                     // per work-list entry: flagged window taps (dense convolutions, 1x1 / 3x3)
    uint8_t* xt_flags;                  // per output pixel: 0 = its x^T row is all zero and need not be read (layers whose
                                        // sparse steps run on the wave-specialised kernel); nullptr: none
    bool counting = false, counted = false;   // statistics mode (dcnn_layer_set_counting); the last step was counted
    mutable bool xt_flags_stale = false;  // the state memory was handed out: the flags are rebuilt from x^T before the next step
    // The row flags describe x^T as it lies in memory: a first frame has gone through and nobody outside can write x^T, so the next
    // first frame clears the rows that hold values only.  From 64 MB of x^T on: there the stores count (64 streams of 128x128, 64 to 256
    // channels, 134-537 MB a layer: first frame 906 -> 844 us when no row holds any, 901 -> 855 after 1 to 64 sparse steps), below it reading the flags and a clearing launch of
    // their own do (layers of 4-16 MB, ResNet-50-shaped: 947 -> 959 us).
    bool xt_flags_hold = false;
    mutable bool xt_shared = false;       // x^T was handed out once (dcnn_layer_state): whoever has it may write it at any time
    void* wpacked;
    void* bias;
    void* wpacked2;                     // fused projection: weights in the main plan's column grouping
    void* bias2;
    int32_t* counters;
    // bookkeeping of the last step
    dcnn_delta view;
    const int32_t* last_in_count;
    const int32_t* last_work_count;
    const int32_t* last_in2_count;
    const uint8_t* last_in_mask;        // for statistics of inputs that come without a count
    const uint8_t* last_in2_mask;
    // optional kernel timing
    std::vector<std::pair<hipEvent_t, hipEvent_t>> events;
    size_t events_used = 0;
};

namespace dcnn {
// dcnn_layer_create with the weights and bias of a fused projection passed on their own.
dcnn_status layer_create(dcnn_ctx* ctx, const dcnn_layer_desc* desc, const void* weights_dev, const void* bias_dev,
                         const void* proj_weights_dev, const void* proj_bias_dev, void* state_dev, size_t state_bytes,
                         bool self, dcnn_layer** out);
// Can the layer's sparse steps build their work list in their own kernel, so that nobody has to hand one over?  `walker`:
// also if the layer would otherwise walk its input's list.  (Not if the ordered list of the pixels that stayed flagged
// is wanted: that is compacted from a stored list.)
bool layer_lists_itself(const dcnn_ctx* ctx, const dcnn_layer_desc& d, bool walker);
// dcnn_layer_init; with clear = false the caller has cleared the layer's pieces (collect_clears) itself.
dcnn_status layer_init(dcnn_layer* L, const void* const* dense_in, int32_t n_in, void* dense_out, bool clear);
// The pieces of the layer's state that are zero before its first sparse step: masks, counts, x^T row flags.
constexpr int kMaxLayerClears = 5;
int collect_clears(const dcnn_layer* L, bool with_flags, ClearPiece* out);
constexpr size_t kXtSparseClear = 64ull << 20;
inline bool clears_rows_by_flag(const dcnn_layer* L) { return L->xt_flags && !L->xt_shared && L->buf1_bytes >= kXtSparseClear; }
// The row flags alone, of a layer whose first frame reads them: a network clears them behind its first frame.
int collect_flag_clear(const dcnn_layer* L, ClearPiece* out);
// Host-side bookkeeping that goes with cleared pieces.
void sparse_output_cleared(dcnn_layer* L);
}  // namespace dcnn
