// Work lists that a kernel builds for itself, on small maps.
//
// On maps of up to 64 K pixels the mask pass, the list emission and the compaction of survivors cost more than
// what they serve: each is a launch of its own with two or three dependent round trips to memory (4-6 us; a layer of a
// network of small maps took 12-20 us, half of it spent on lists).  Ways out, all with the entries' results unchanged:
//   local_build  a workgroup compacts blocks of pixels of its own.  Most kernels, up to kLocalMaxPixels or kSelfMaxPixels.
//   local_run    several workgroups compact the same run of pixels and divide its entries.  Kernels in which every tile fetches
//                the layer's weights: register-blocked convolution, units.
//   self_build   a mask of 16 K pixels is 2 KB of bits, so a workgroup can hold ALL flags in LDS: it reads the input mask
//                (one round trip of 16-byte loads), forms the flagged output pixels as bits (a 3x3 window on whole words) and
//                takes the prefix sums of the words' counts -- the position of every pixel in the ascending list.  The plain
//                convolution kernel on windows other than 1x1 and 3x3, which keeps the entries of its own tiles; the list kernel
//                (mask_kernels.hip); and the few workgroups that write what belongs to the whole map beside the other ways.
// Every workgroup of a layer's kernel went the second way once: 3-5 us of the 11-18 that such a kernel took.  Step, all of
// them -> blocks: bottleneck block on one 128x128 stream 47.5 -> 41.1 us, 3x3 fp32 32->32 + ReLU on 64x64 21.7 -> 19.7, 8 streams
// of a ResNet-50-shaped network 1450 -> 1250, HRNet-shaped 1306 -> 1126, MobileNet-shaped 512 -> 413 (half of the last from
// runs of one batch, tail_shape).
#pragma once

#include "device_utils.h"

namespace dcnn {

// 32 mask bytes -> 32 bits, any non-zero byte counts
__device__ __forceinline__ uint32_t self_pack(const uint4& a, const uint4& b) {
    auto pack8 = [](uint64_t v) -> uint32_t {
        v |= v >> 4; v |= v >> 2; v |= v >> 1;
        v &= 0x0101010101010101ull;
        return (uint32_t)((v * 0x0102040810204080ull) >> 56);
    };
    return pack8((uint64_t)a.x | (uint64_t)a.y << 32) | pack8((uint64_t)a.z | (uint64_t)a.w << 32) << 8 |
           pack8((uint64_t)b.x | (uint64_t)b.y << 32) << 16 | pack8((uint64_t)b.z | (uint64_t)b.w << 32) << 24;
}
// flags of pixels 32*w .. 32*w+31 of a mask (16-byte aligned) that holds them all
__device__ __forceinline__ uint32_t self_mask_word(const uint8_t* mask, int w) {
    return self_pack(*reinterpret_cast<const uint4*>(mask + w * 32), *reinterpret_cast<const uint4*>(mask + w * 32 + 16));
}
// The last word of a mask of `px` bytes that ends inside it: a byte per lane, by a whole wave, all lanes get the word.  (Byte after
// byte by the lane whose word it is, each load waited for, a map of 100 x 100 pixels cost every kernel that builds its list 4-5 us
// over one of 96 x 104: add + ReLU, 64 channels, 14.8 us, now 11.4.  With dwords and bytes requested together by that lane the
// code alone cost all maps 0.4 us a launch.)
__device__ __forceinline__ uint32_t self_mask_tail(const uint8_t* mask, int px) {
    const int at = (px & ~31) + (int)(threadIdx.x % kWave);
    return (uint32_t)__ballot(at < px && mask[min(at, px - 1)] != 0);
}

// 32 bits from bit position `pos` on; positions outside the array read some word of it (callers mask those bits)
__device__ __forceinline__ uint32_t self_bits32(const uint32_t* words, int nwords, int pos) {
    const int i = pos >> 5, sh = pos & 31;
    const int lo = min(max(i, 0), nwords - 1), hi = min(max(i + 1, 0), nwords - 1);
    return (uint32_t)((((uint64_t)words[hi] << 32) | words[lo]) >> sh);
}

struct SelfSpan { int begin, end, step, entries; };            // this workgroup's groups of `entries` list entries

// floor(a / b) for 0 <= a < 2^17, 0 < b < 2^12 (the quotient's distance from the next integer exceeds the rounding error)
__device__ __forceinline__ int self_div(int a, float inv_b) { return (int)(((float)a + 0.5f) * inv_b); }

// Window taps of output pixel p, bit ky*k+kx, from the bits of the input mask.
__device__ __forceinline__ uint32_t self_taps(const ListArgs& l, const uint32_t* ibits, int in_words, int p) {
    const uint32_t t1 = fast_div((uint32_t)p, l.div_ow);
    const int ox = p - (int)t1 * l.m_ow;
    const int n = (int)fast_div(t1, l.div_oh);
    const int oy = (int)t1 - n * l.m_oh;
    const int iy0 = oy * l.m_stride - l.m_pad, ix0 = ox * l.m_stride - l.m_pad;
    uint32_t cols = (1u << l.m_k) - 1u;                        // window columns inside the map
    if (ix0 < 0) cols &= ~((1u << -ix0) - 1u);
    if (ix0 + l.m_k > l.m_w) cols &= (1u << (l.m_w - ix0)) - 1u;
    uint32_t taps = 0;
    for (int ky = 0; ky < l.m_k; ++ky) {
        const int iy = iy0 + ky;
        if (iy < 0 || iy >= l.m_h) continue;
        taps |= (self_bits32(ibits, in_words, (n * l.m_h + iy) * l.m_w + ix0) & cols) << (l.m_k > 5 ? 0 : ky * l.m_k);   // (windows above 5x5 are only asked whether any tap is set)
    }
    return taps;
}

__device__ __forceinline__ bool self_b_flag(const ListArgs& l, int p) {
    if (l.b_stride <= 0) return l.m_b[p] != 0;
    const uint32_t t1 = fast_div((uint32_t)p, l.div_ow);
    const int ox = p - (int)t1 * l.m_ow;
    const int n = (int)fast_div(t1, l.div_oh);
    const int oy = (int)t1 - n * l.m_oh;
    return l.m_b[((int64_t)n * l.b_h + oy * l.b_stride) * l.b_w + ox * l.b_stride] != 0;
}

// Inclusive sums over the 16 lanes of a row / the 64 lanes of the wave, by DPP lane shifts (register to register).
template <int CTRL, int ROWS> __device__ __forceinline__ int self_dpp_add(int v) {
    return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int self_row_scan(int v) {
    v = self_dpp_add<0x111, 0xf>(v);        // row_shr:1
    v = self_dpp_add<0x112, 0xf>(v);        // row_shr:2
    v = self_dpp_add<0x114, 0xf>(v);        // row_shr:4
    return self_dpp_add<0x118, 0xf>(v);     // row_shr:8
}
__device__ __forceinline__ int self_scan(int v) {
    v = self_row_scan(v);
    v = self_dpp_add<0x142, 0xa>(v);        // row_bcast:15 into rows 1 and 3
    return self_dpp_add<0x143, 0xc>(v);     // row_bcast:31 into rows 2 and 3
}

constexpr int kSelfTail = 31;                                  // where SelfBits::red keeps the second mask's incomplete last word
struct SelfBits {
    uint32_t* ibits;
    uint32_t* obits;
    uint32_t* dil;             // strided 3x3: the flags dilated at the input's resolution
    uint16_t* prefix;          // flagged pixels before each word of obits
    int* red;
    int in_words, out_words;
    int top;                   // power of two, at least out_words
};
__device__ __forceinline__ SelfBits self_carve(const ListArgs& l, unsigned char* scratch) {
    SelfBits s;
    s.in_words = (l.m_in_px + 31) / 32;
    s.out_words = (l.m_out_px + 31) / 32;
    s.top = 1;
    while (s.top < s.out_words) s.top <<= 1;
    s.red = reinterpret_cast<int*>(scratch);                   // 128 bytes
    s.ibits = reinterpret_cast<uint32_t*>(scratch + 128);
    s.obits = s.ibits + s.in_words;
    s.dil = s.obits + s.out_words;
    s.prefix = reinterpret_cast<uint16_t*>(s.dil + (l.m_stride == 2 ? s.in_words : 0));
    return s;
}

// 3x3 dilation of the bits of the input map, whole words: the rows above, at and below, each OR-ed with itself moved by
// one column; what lies beyond a border of the map is masked out by the columns and rows the word's pixels are in.
__device__ __forceinline__ uint32_t self_dilate_word(const ListArgs& l, const SelfBits& s, int w, const FastDiv& div_w, const FastDiv& div_h) {
    const int p0 = w * 32;
    const uint32_t t1 = fast_div((uint32_t)p0, div_w);
    int x = p0 - (int)t1 * l.m_w;
    int y = (int)t1 - (int)fast_div(t1, div_h) * l.m_h;
    uint32_t first_col = 0, last_col = 0, first_row = 0, last_row = 0;
    for (int pos = 0; pos < 32;) {
        const int run = min(l.m_w - x, 32 - pos);
        const uint32_t seg = (run == 32 ? 0xffffffffu : ((1u << run) - 1u)) << pos;
        if (x == 0) first_col |= 1u << pos;
        if (x + run == l.m_w) last_col |= 1u << (pos + run - 1);
        if (y == 0) first_row |= seg;
        if (y == l.m_h - 1) last_row |= seg;
        pos += run;
        x = 0;
        if (++y == l.m_h) y = 0;
    }
    uint32_t hit = 0;
#pragma unroll
    for (int dy = -1; dy <= 1; ++dy) {
        const int pos = p0 + dy * l.m_w;
        uint32_t row = self_bits32(s.ibits, s.in_words, pos) | (self_bits32(s.ibits, s.in_words, pos - 1) & ~first_col) |
                       (self_bits32(s.ibits, s.in_words, pos + 1) & ~last_col);
        if (dy < 0) row &= ~first_row;
        if (dy > 0) row &= ~last_row;
        hit |= row;
    }
    if (p0 + 32 > l.m_in_px) hit &= (1u << (l.m_in_px - p0)) - 1u;
    return hit;
}

// The input mask on its way: requested before the kernel does anything else that waits (two words per thread of a
// workgroup of 1024; an incomplete last word is read in self_build).
constexpr int kSelfAhead = 2;
struct SelfAhead { uint4 a[kSelfAhead], b[kSelfAhead]; };
__device__ __forceinline__ void self_request(const ListArgs& l, SelfAhead& v) {
#pragma unroll
    for (int i = 0; i < kSelfAhead; ++i) {
        const int p0 = ((int)threadIdx.x + i * 1024) * 32;
        v.a[i] = v.b[i] = make_uint4(0u, 0u, 0u, 0u);
        if (p0 + 32 <= l.m_in_px) {
            v.a[i] = *reinterpret_cast<const uint4*>(l.m_in + p0);
            v.b[i] = *reinterpret_cast<const uint4*>(l.m_in + p0 + 16);
        }
    }
}

// Phase 1: all flags and list positions.  Returns the length of the list.  Every thread
// of the workgroup (NT of them) calls it; ends with a barrier.
template <int NT>
__device__ __forceinline__ int self_build(const ListArgs& l, const SelfBits& s, const SelfAhead* ahead = nullptr) {
    constexpr int NWV = NT / kWave;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const bool copy = l.m_k == 1 && l.m_stride == 1 && l.m_up == 1;
    const bool win3 = l.m_k == 3 && l.m_stride == 1 && l.m_pad == 1 && l.m_up == 1;   // (up > 1 comes with k = 1)
    static_assert(NT == 1024 || NT <= 512, "self_request assumes 1024 threads");
    const bool b_words = l.m_b != nullptr && l.b_stride <= 0;  // the second mask has the output's shape
    int i = 0;
#pragma unroll 2
    for (int w = tid; w < l.m_in_px / 32; w += NT, ++i) {
        uint32_t v;
        if (ahead != nullptr) v = i == 0 ? self_pack(ahead->a[0], ahead->b[0]) : self_pack(ahead->a[1], ahead->b[1]);
        else v = self_mask_word(l.m_in, w);
        s.ibits[w] = v;
        if (copy) s.obits[w] = v | (b_words ? self_mask_word(l.m_b, w) : 0u);
    }
    if (wave == NWV - 1) {                                     // incomplete last words (the last wave has the fewest whole ones)
        uint32_t b = 0;
        if (b_words && l.m_out_px % 32 != 0) {
            b = self_mask_tail(l.m_b, l.m_out_px);
            if (lane == 0) s.red[kSelfTail] = (int)b;
        }
        if (l.m_in_px % 32 != 0) {
            const uint32_t v = self_mask_tail(l.m_in, l.m_in_px);
            if (lane == 0) {
                s.ibits[s.in_words - 1] = v;
                if (copy) s.obits[s.in_words - 1] = v | b;
            }
        }
    }
    lds_block_sync();
    if (win3) {
        for (int w = tid; w < s.out_words; w += NT) {
            uint32_t hit = self_dilate_word(l, s, w, l.div_ow, l.div_oh);      // (input and output maps have one shape)
            if (b_words) hit |= w * 32 + 32 <= l.m_out_px ? self_mask_word(l.m_b, w) : (uint32_t)s.red[kSelfTail];
            s.obits[w] = hit;
        }
    } else if (l.m_up > 1) {
        // nearest upsampling: runs of equal flags, cut at words and rows
        for (int w = tid; w < s.out_words; w += NT) {
            const int p0 = w * 32;
            const uint32_t t1 = fast_div((uint32_t)p0, l.div_ow);
            int x = p0 - (int)t1 * l.m_ow;
            int n = (int)fast_div(t1, l.div_oh);
            int y = (int)t1 - n * l.m_oh;
            uint32_t bits = 0;
            int q = (n * l.m_h + (int)fast_div((uint32_t)y, l.div_up)) * l.m_w + (int)fast_div((uint32_t)x, l.div_up);
            int left = l.m_up - (x - (int)fast_div((uint32_t)x, l.div_up) * l.m_up);     // pixels until the next source
            const int end = min(32, l.m_out_px - p0);
            for (int pos = 0; pos < end;) {
                const int run = min(left, end - pos);
                if ((s.ibits[q >> 5] >> (q & 31)) & 1u) bits |= (uint32_t)(((1ull << run) - 1ull) << pos);
                pos += run;
                x += run;
                ++q;
                left = l.m_up;
                if (x >= l.m_ow) {                             // next row: a source row further every m_up of them
                    x = 0;
                    if (++y == l.m_oh) { y = 0; ++n; }
                    q = (n * l.m_h + (int)fast_div((uint32_t)y, l.div_up)) * l.m_w;
                }
            }
            s.obits[w] = bits;
        }
    } else if (!copy) {
        // stride 2: the flags dilated at the input's resolution, then one bit per output pixel; any other window: its
        // taps pixel by pixel.  A pixel per lane, 64 flags per wave and step.
        const bool sample = l.m_stride == 2 && ((l.m_k == 3 && l.m_pad == 1) || (l.m_k == 1 && l.m_pad == 0));
        if (sample && l.m_k == 3) {
            for (int w = tid; w < s.in_words; w += NT) s.dil[w] = self_dilate_word(l, s, w, l.div_iw, l.div_ih);
            lds_block_sync();
        }
        const uint32_t* from = l.m_k == 3 ? s.dil : s.ibits;
        for (int base = wave * kWave; base < l.m_out_px; base += NT) {
            const int p = base + lane;
            bool f = false;
            if (p < l.m_out_px) {
                if (sample) {
                    const uint32_t t1 = fast_div((uint32_t)p, l.div_ow);
                    const int ox = p - (int)t1 * l.m_ow;
                    const int n = (int)fast_div(t1, l.div_oh);
                    const int oy = (int)t1 - n * l.m_oh;
                    const int q = (n * l.m_h + 2 * oy) * l.m_w + 2 * ox;
                    f = (from[q >> 5] >> (q & 31)) & 1u;
                } else {
                    f = self_taps(l, s.ibits, s.in_words, p) != 0;
                }
                if (l.m_b && l.b_stride <= 0) f = f || l.m_b[p] != 0;
            }
            const uint64_t bits = __ballot(f);
            if (lane == 0) s.obits[base / 32] = (uint32_t)bits;
            if (lane == 1 && base / 32 + 1 < s.out_words) s.obits[base / 32 + 1] = (uint32_t)(bits >> 32);
        }
    }
    if (l.m_b && l.b_stride > 0) {                             // a second mask of another size: sampled pixel by pixel
        // (eight loads of a lane in flight: a 3x3 layer on 61 K pixels whose length was counted here 36 -> 32 us, most of it this)
        lds_block_sync();
        constexpr int B = 8;
        for (int base0 = wave * kWave; base0 < l.m_out_px; base0 += B * NT) {
            bool f[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int p = base0 + u * NT + lane;
                const bool flag = self_b_flag(l, p < l.m_out_px ? p : 0);
                f[u] = p < l.m_out_px && flag;
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const int base = base0 + u * NT;
                const uint64_t bits = __ballot(f[u]);
                if (lane == 0 && base / 32 < s.out_words) s.obits[base / 32] |= (uint32_t)bits;
                if (lane == 1 && base / 32 + 1 < s.out_words) s.obits[base / 32 + 1] |= (uint32_t)(bits >> 32);
            }
        }
    }
    lds_block_sync();
    // exclusive prefix over the words: W consecutive words per thread, a scan over threads, then within them
    const int W = (s.out_words + NT - 1) / NT;
    int mine = 0;
    for (int i = 0; i < W; ++i) {
        const int w = tid * W + i;
        if (w < s.out_words) mine += __popc(s.obits[w]);
    }
    const int inc = self_scan(mine);
    if (lane == kWave - 1) s.red[wave] = inc;
    lds_block_sync();
    // (at most 16 waves: their totals fit one row of lanes, every wave scans them again)
    const int waves = self_row_scan(lane < NWV ? s.red[lane] : 0);
    const int total = __builtin_amdgcn_readlane(waves, NWV - 1);
    const int before = wave == 0 ? 0 : __builtin_amdgcn_readlane(waves, __builtin_amdgcn_readfirstlane(wave > 0 ? wave - 1 : 0));
    int run = before + inc - mine;
    for (int i = 0; i < W; ++i) {
        const int w = tid * W + i;
        if (w < s.out_words) { s.prefix[w] = (uint16_t)run; run += __popc(s.obits[w]); }
    }
    lds_block_sync();
    return total;
}

// Pixel of list entry j (below the list's length): the last word with no more than j flagged pixels before it, then the
// bit of that rank in it.
__device__ __forceinline__ int self_select(const SelfBits& s, int j) {
    int w = 0;
    for (int half = s.top >> 1; half >= 1; half >>= 1) {
        const int m = w + half;
        if (m < s.out_words && (int)s.prefix[m] <= j) w = m;
    }
    uint32_t bits = s.obits[w];
    int rank = j - (int)s.prefix[w], at = 0;
#pragma unroll
    for (int half = 16; half >= 1; half >>= 1) {
        const int below = __popc(bits & ((1u << half) - 1u));
        if (rank >= below) { rank -= below; bits >>= half; at += half; }
    }
    return w * 32 + at;
}

// Phase 2: the entries of this workgroup's groups -> px in LDS, group after group; the shared outputs.
// Ends with a barrier, after which the scratch memory of phase 1 is free.
template <int NT>
__device__ __forceinline__ void self_emit(const ListArgs& l, const SelfBits& s, int count, SelfSpan span, int32_t* px) {
    const int tid = threadIdx.x;
    const int groups = span.begin < span.end ? (span.end - span.begin + span.step - 1) / span.step : 0;
    const int nloc = groups * span.entries;
    const float inv_e = 1.0f / (float)span.entries;
    for (int i = tid; i < nloc; i += NT) {
        const int q = self_div(i, inv_e);
        const int j = (span.begin + q * span.step) * span.entries + (i - q * span.entries);
        px[i] = j < count ? self_select(s, j) : -1;
    }
    // shares of what other kernels read
    if (blockIdx.y == 0) {
        const int per = (s.out_words + (int)gridDim.x - 1) / (int)gridDim.x;
        const int w1 = min(((int)blockIdx.x + 1) * per, s.out_words);
        if (l.mask_out != nullptr) {
            for (int i = (int)blockIdx.x * per * 8 + tid; i < w1 * 8; i += NT) {     // four pixels per step
                const uint32_t f = (s.obits[i / 8] >> (4 * (i % 8))) & 15u;
                const uint32_t v = (f & 1u) | (f & 2u) << 7 | (f & 4u) << 14 | (f & 8u) << 21;
                if (i * 4 + 4 <= l.m_out_px) *reinterpret_cast<uint32_t*>(l.mask_out + i * 4) = v;
                else for (int k = 0; i * 4 + k < l.m_out_px; ++k) l.mask_out[i * 4 + k] = (uint8_t)((f >> k) & 1u);
            }
        }
        if (l.mask_zero != nullptr) {
            for (int i = (int)blockIdx.x * per * 8 + tid; i < w1 * 8; i += NT) {     // (a listed pixel's byte is its tile's business)
                const uint32_t f = (s.obits[i / 8] >> (4 * (i % 8))) & 15u;
                if (f == 0 && i * 4 + 4 <= l.m_out_px) *reinterpret_cast<uint32_t*>(l.mask_zero + i * 4) = 0u;
                else for (int k = 0; k < 4 && i * 4 + k < l.m_out_px; ++k) if (!((f >> k) & 1u)) l.mask_zero[i * 4 + k] = 0;
            }
        }
        if (l.idx_out != nullptr) {
            for (int w = (int)blockIdx.x * per + tid; w < w1; w += NT) {
                int j = s.prefix[w];
                for (uint32_t rest = s.obits[w]; rest; rest &= rest - 1) l.idx_out[j++] = w * 32 + __builtin_ctz(rest);
            }
        }
        if (l.count_out != nullptr && blockIdx.x == 0 && tid == 0) *l.count_out = count;
        if (l.in_idx_out != nullptr) {                         // (uniform for the grid)
            // a run of words per workgroup: the flags before it are summed by all threads, those within it by each for itself
            constexpr int NWV = NT / kWave;
            const int share = (s.in_words + (int)gridDim.x - 1) / (int)gridDim.x;
            const int w0 = min((int)blockIdx.x * share, s.in_words), w2 = min(w0 + share, s.in_words);
            int part = 0;
            for (int w = tid; w < w0; w += NT) part += __popc(s.ibits[w]);
            part = self_scan(part);
            if (tid % kWave == kWave - 1) s.red[tid / kWave] = part;
            lds_block_sync();
            int before = 0;
            for (int i = 0; i < NWV; ++i) before += s.red[i];
            for (int w = w0 + tid; w < w2; w += NT) {
                int j = before;
                for (int v = w0; v < w; ++v) j += __popc(s.ibits[v]);
                for (uint32_t rest = s.ibits[w]; rest; rest &= rest - 1) l.in_idx_out[j++] = w * 32 + __builtin_ctz(rest);
                if (w == s.in_words - 1) *l.in_count_out = j;
            }
        }
    }
    lds_block_sync();
}

// ---- blocks of pixels that a workgroup compacts for itself ----------------------------------------------------------------
// A kernel does not need the map's list to know its work, only some cut of it.  Here the map is cut into blocks of 8 .. 64
// pixels that are dealt to the workgroups in turn; a workgroup tests the windows of its own pixels (a byte per tap and lane,
// one round trip), packs the flagged ones together in LDS and walks those.  No workgroup repeats another's work and none
// waits for a scan of the map.  What belongs to the whole map -- the ascending list, its length, the input's list -- is
// written by `writers` workgroups at the front of the grid that form all flags, beside the others and not ahead of them.
// An output pixel's sums do not depend on its neighbours in a tile, so results are those of the stored list.

// Window taps of output pixel p (windows up to 3x3), bit ky*k+kx, and bit 30: the second mask's flag.  All loads go out together.
constexpr uint32_t kLocalSecond = 1u << 30;
__device__ __forceinline__ uint32_t local_taps(const ListArgs& l, int p, bool live) {
    const uint32_t pu = live ? (uint32_t)p : 0u;
    const uint32_t t1 = fast_div(pu, l.div_ow);
    const int ox = (int)pu - (int)t1 * l.m_ow;
    const int n = (int)fast_div(t1, l.div_oh);
    const int oy = (int)t1 - n * l.m_oh;
    uint8_t fb = 0;
    if (l.m_b != nullptr) fb = l.m_b[l.b_stride > 0 ? ((int64_t)n * l.b_h + oy * l.b_stride) * l.b_w + ox * l.b_stride : (int64_t)pu];
    uint32_t taps = 0;
    if (l.m_k == 1) {
        const int iy = l.m_up > 1 ? (int)fast_div((uint32_t)oy, l.div_up) : oy * l.m_stride;
        const int ix = l.m_up > 1 ? (int)fast_div((uint32_t)ox, l.div_up) : ox * l.m_stride;
        taps = l.m_in[(n * l.m_h + iy) * l.m_w + ix] ? 1u : 0u;
    } else {
        const int iy0 = oy * l.m_stride - l.m_pad, ix0 = ox * l.m_stride - l.m_pad;
        uint8_t f[9];
        bool in[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            const int iy = iy0 + t / 3, ix = ix0 + t % 3;
            in[t] = t / 3 < l.m_k && t % 3 < l.m_k && (unsigned)iy < (unsigned)l.m_h && (unsigned)ix < (unsigned)l.m_w;
            f[t] = l.m_in[in[t] ? (n * l.m_h + iy) * l.m_w + ix : 0];
        }
#pragma unroll
        for (int t = 0; t < 9; ++t)
            if (in[t] && f[t]) taps |= 1u << ((t / 3) * l.m_k + t % 3);
    }
    if (fb) taps |= kLocalSecond;
    return live ? taps : 0u;
}
// The flags of a workgroup's own pixels that others read: the output mask, or its zeros where nothing is listed.
__device__ __forceinline__ void local_mask(const ListArgs& l, int p, bool listed) {
    if (l.mask_out != nullptr) l.mask_out[p] = listed ? 1 : 0;
    if (l.mask_zero != nullptr && !listed) l.mask_zero[p] = 0;
}
// The flagged pixels of this workgroup's blocks -> px and tap words in LDS, padded with -1 / 0 to l.lds_entries; returns their
// number.  Every thread of the workgroup (NT of them) calls it; ends with a barrier.
template <int NT>
__device__ __forceinline__ int local_build(const ListArgs& l, unsigned char* at, int32_t*& px, uint32_t*& taps) {
    constexpr int NWV = NT / kWave;
    int* red = reinterpret_cast<int*>(at);                     // 64 bytes
    px = reinterpret_cast<int32_t*>(at + 64);
    taps = reinterpret_cast<uint32_t*>(px + l.lds_entries);
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int owner = (int)blockIdx.x - l.writers, owners = (int)gridDim.x - l.writers;
    int count = 0;
    for (int s0 = 0; s0 < l.local_slots; s0 += NT) {
        const int slot = s0 + tid;
        const int p = ((owner + (slot >> l.local_shift) * owners) << l.local_shift) + (slot & ((1 << l.local_shift) - 1));
        const bool live = slot < l.local_slots && p < l.m_out_px;
        uint32_t t = 0;
        if (s0 + wave * kWave < l.local_slots) t = local_taps(l, p, live);
        const uint64_t hit = __ballot(t != 0);
        if (live) local_mask(l, p, t != 0);
        if (s0 > 0) lds_block_sync();                          // (the counts of the step before have been read)
        if (lane == 0) red[wave] = __popcll(hit);
        lds_block_sync();
        int before = count;
#pragma unroll
        for (int i = 0; i < NWV; ++i) {
            const int c = red[i];
            if (i < wave) before += c;
            count += c;
        }
        if (t != 0) {
            const int j = before + __popcll(hit & ((1ull << lane) - 1ull));
            px[j] = p;
            taps[j] = t;
        }
    }
    for (int j = count + tid; j < l.lds_entries; j += NT) { px[j] = -1; taps[j] = 0; }
    lds_block_sync();
    return count;
}
// The flagged pixels of run `run` (kRunPixels consecutive pixels, one per thread) -> px and tap words in LDS; returns their number.
// For kernels in which a tile costs its weights: every workgroup of the run's has the same entries and takes its own share of them.
// A run's tiles hold as many listed pixels as there are, where tiles of pixels as they lie each hold a few when flags are scattered.
__device__ __forceinline__ int local_run(const ListArgs& l, unsigned char* at, int run, bool write_masks, const int32_t*& px_out,
                                         const uint32_t*& taps_out) {
    constexpr int NWV = kRunPixels / kWave;
    int* red = reinterpret_cast<int*>(at);
    int32_t* px = reinterpret_cast<int32_t*>(at + kLocalHeader);
    uint32_t* taps = reinterpret_cast<uint32_t*>(px + kRunPixels);
    px_out = px; taps_out = taps;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int p = run * kRunPixels + tid;
    const bool live = p < l.m_out_px;
    const uint32_t t = local_taps(l, p, live);
    const uint64_t hit = __ballot(t != 0);
    if (write_masks && live) local_mask(l, p, t != 0);
    if (lane == 0) red[wave] = __popcll(hit);
    lds_block_sync();
    int before = 0, count = 0;
#pragma unroll
    for (int i = 0; i < NWV; ++i) {
        const int c = red[i];
        if (i < wave) before += c;
        count += c;
    }
    if (t != 0) {
        const int j = before + __popcll(hit & ((1ull << lane) - 1ull));
        px[j] = p;
        taps[j] = t;
    }
    lds_block_sync();
    return count;
}
// What belongs to the whole map, by writer blockIdx.x of l.writers.
template <int NT>
__device__ __forceinline__ void local_write(const ListArgs& l, unsigned char* scratch) {
    const SelfBits s = self_carve(l, scratch);
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int share = blockIdx.x;
    if (l.idx_out == nullptr && share > 0) return;             // (a launcher's multiple of eight)
    if (l.idx_out == nullptr && l.in_idx_out == nullptr && l.m_k == 1 && l.m_stride == 1 && l.m_up == 1 && l.b_stride <= 0) {
        // only the length is wanted and the flags are the masks': their sum, eight words a thread in flight
        constexpr int NWV = NT / kWave;
        const int whole = l.m_out_px / 32;
        int sum = 0;
#pragma unroll 8
        for (int w = tid; w < whole; w += NT) {
            uint32_t v = self_mask_word(l.m_in, w);
            if (l.m_b != nullptr) v |= self_mask_word(l.m_b, w);
            sum += __popc(v);
        }
        if (wave == NWV - 1 && l.m_out_px % 32 != 0) {
            uint32_t v = self_mask_tail(l.m_in, l.m_out_px);
            if (l.m_b != nullptr) v |= self_mask_tail(l.m_b, l.m_out_px);
            if (lane == 0) sum += __popc(v);
        }
        sum = self_scan(sum);
        if (lane == kWave - 1) s.red[wave] = sum;
        lds_block_sync();
        if (share == 0 && tid == 0 && l.count_out != nullptr) {
            int total = 0;
            for (int i = 0; i < NWV; ++i) total += s.red[i];
            *l.count_out = total;
        }
        return;
    }
    const int count = self_build<NT>(l, s);
    if (l.count_out != nullptr && share == 0 && tid == 0) *l.count_out = count;
    if (l.idx_out != nullptr) {
        // two words of flags per wave and step, a pixel per lane
        const int per = (s.out_words + l.writers - 1) / l.writers, w_end = min((share + 1) * per, s.out_words);
        for (int w0 = share * per + 2 * wave; w0 < w_end; w0 += 2 * NT / kWave) {
            const int w = w0 + lane / 32;
            if (w >= w_end) continue;
            const uint32_t bits = s.obits[w];
            if ((bits >> (lane & 31)) & 1u) l.idx_out[(int)s.prefix[w] + __popc(bits & ((1u << (lane & 31)) - 1u))] = w * 32 + (lane & 31);
        }
    }
    if (l.in_idx_out != nullptr && share == 0) {
        // consecutive words per thread, a scan over threads
        constexpr int NWV = NT / kWave;
        const int W = (s.in_words + NT - 1) / NT;
        int mine = 0;
        for (int i = 0; i < W; ++i)
            if (tid * W + i < s.in_words) mine += __popc(s.ibits[tid * W + i]);
        const int inc = self_scan(mine);
        lds_block_sync();                                      // (self_build's sums have been read)
        if (lane == kWave - 1) s.red[wave] = inc;
        lds_block_sync();
        int j = inc - mine, total = 0;
        for (int i = 0; i < NWV; ++i) {
            const int c = s.red[i];
            if (i < wave) j += c;
            total += c;
        }
        for (int i = 0; i < W; ++i) {
            const int w = tid * W + i;
            if (w < s.in_words)
                for (uint32_t rest = s.ibits[w]; rest; rest &= rest - 1) l.in_idx_out[j++] = w * 32 + __builtin_ctz(rest);
        }
        if (tid == 0) *l.in_count_out = total;
    }
}

}  // namespace dcnn
