// The activation + truncation tail of the sparse steps that reach memory through buffer descriptors, shared by the
// activation and depthwise kernels.
#pragma once

#include "device_utils.h"

namespace dcnn {

// ---- sparse-step tail with buffer addressing ---------------------------------------------------
// Activation + truncation (Eqs. 4-6) of one run of tile entries, for the sparse steps of layers whose channel
// count is a multiple of the vector width and whose tensors stay below 2 GiB.  Same arithmetic, rounding and
// decisions as act_trunc_tile; what differs is how memory is reached: every flag a load depends on has been
// fetched for the whole tile beforehand (one round trip, entry lane%32 per lane), and every load and store
// goes through a buffer descriptor with an out-of-range offset where a lane has nothing to do.  A batch of
// UB iterations therefore issues all its loads back to back and costs one round trip to memory.
//
// `Src` delivers the first delta stream: select(ub, ent) runs in wave-uniform control flow and picks the
// per-entry values of iteration ub (lane shuffles); issue(ub, v, c0, on, off) requests the values of the
// lane's vector v; finish(ub, v, c0) returns them, rounded to the storage type.
struct TailRsrc {
    __amdgpu_buffer_rsrc_t res, xA, xT, out, omask;
};

template <typename T, int V, int VPL, int UB, class Src>
__device__ __forceinline__ uint32_t sparse_tile_tail(const EpilogueArgs& e, const TailRsrc& rs, Src& src, int LP, int p_mine,
                                                    int rflag_mine, int ent_first, int ent_end, int nbatch, int lane) {
    typedef typename RawOf<T, V>::type Raw;
    constexpr uint32_t ES = sizeof(T);
    const int PPI = kWave / LP;
    const int sub = lane % LP, grp = lane / LP;
    const int nvec = e.c / V;
    const uint32_t row_bytes = (uint32_t)e.c * ES;
    const bool stateful = e.act != DCNN_ACT_NONE;
    const bool has_res = e.res_data != nullptr;
    const float hi = act_hi(e.act);
    uint32_t bits = 0;
    for (int b = 0; b < nbatch; ++b) {
        int pix[UB];
        uint32_t off[UB][VPL];
        Raw rr[UB][VPL], ra[UB][VPL], rt[UB][VPL];
        // ---- phase 1: every load of the batch ----------------------------------------------------
#pragma unroll
        for (int ub = 0; ub < UB; ++ub) {
            const int ent = ent_first + (b * UB + ub) * PPI + grp;
            const int p_any = __shfl(p_mine, ent & (kTile - 1), kWave);
            const int rf = __shfl(rflag_mine, ent & (kTile - 1), kWave);
            src.select(ub, ent & (kTile - 1));
            const int p = ent < ent_end ? p_any : -1;
            pix[ub] = p;
#pragma unroll
            for (int v = 0; v < VPL; ++v) {
                const int vi = sub + v * LP;
                const bool on = p >= 0 && vi < nvec;
                const int c0 = vi * V;
                const uint32_t o = on ? (uint32_t)p * row_bytes + (uint32_t)c0 * ES : kOob;
                off[ub][v] = o;
                src.issue(ub, v, c0, on, o);
                rr[ub][v] = ws_load16<Raw>(rs.res, rf ? o : kOob);          // empty descriptor without a second stream
                ra[ub][v] = ws_load16_nt<Raw>(rs.xA, o);                     // empty descriptors without an activation
                rt[ub][v] = ws_load16_nt<Raw>(rs.xT, o);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // ---- phase 2: arithmetic, per-pixel maximum, decision, stores -----------------------------
#pragma unroll
        for (int ub = 0; ub < UB; ++ub) {
            Raw o_a[VPL], o_t[VPL], o_y[VPL], o_r[VPL];
            float u = 0.0f;
#pragma unroll
            for (int v = 0; v < VPL; ++v) {
                const Raw d0 = src.finish(ub, v, (sub + v * LP) * V);
                o_r[v] = raw_zero<T, V>();
#pragma unroll
                for (int i = 0; i < V; ++i) {
                    float d = raw_get<T, V>(d0, i);
                    if (has_res) d = round_store<T>(d + raw_get<T, V>(rr[ub][v], i));
                    if (stateful) {
                        const float a = raw_get<T, V>(ra[ub][v], i), t = raw_get<T, V>(rt[ub][v], i);
                        const float sum = (a + t) + d;
                        const float dy = act_clamp(sum, hi) - act_clamp(a, hi);
                        u = fmaxf(u, fabsf(dy));
                        raw_set<T, V>(o_a[v], i, sum);
                        raw_set<T, V>(o_t[v], i, t + d);                       // x^T if the pixel is truncated
                        raw_set<T, V>(o_y[v], i, dy);
                        if (e.carry) raw_set<T, V>(o_r[v], i, round_residue<T>(sum));   // x^T if it is updated and keeps the residue
                    } else {
                        raw_set<T, V>(o_y[v], i, d);
                    }
                }
            }
            bool upd = true;
            if (stateful) {
                for (int m = LP >> 1; m >= 1; m >>= 1) u = fmaxf(u, __shfl_xor(u, m, kWave));
                upd = u >= e.eps;
            }
#pragma unroll
            for (int v = 0; v < VPL; ++v) {
                const uint32_t o = off[ub][v];
                if (stateful) {
                    const uint32_t o_upd = upd ? o : kOob;
                    ws_store16_nt<Raw>(rs.xA, o_upd, o_a[v]);
                    // (an x^T that already is all zero bits is not rewritten by an update that leaves zeros)
                    ws_store16_nt<Raw>(rs.xT, (upd && all_bits_zero(rt[ub][v]) && all_bits_zero(o_r[v])) ? kOob : o, upd ? o_r[v] : o_t[v]);
                    ws_store16<Raw>(rs.out, o_upd, o_y[v]);
                } else {
                    ws_store16<Raw>(rs.out, o, o_y[v]);
                }
            }
            const bool lead = pix[ub] >= 0 && sub == 0;
            if (stateful) __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(upd ? 1 : 0), rs.omask, lead ? pix[ub] : (int)kOob, 0, 0);
            const int ent = ent_first + (b * UB + ub) * PPI + grp;
            if (lead && upd) bits |= 1u << (ent & (kTile - 1));
        }
    }
#pragma unroll
    for (int m = kWave >> 1; m >= 1; m >>= 1) bits |= __shfl_xor(bits, m, kWave);
    return bits;
}

// How the entries of a tile are spread over waves and batches for a pixel of `nvec` vectors.
struct TailShape {
    int lp;        // lanes per pixel
    int run;       // consecutive tile entries per wave (1 .. 32)
    int nbatch;    // batches of UB iterations per wave
};
// A run is one batch: a second one starts behind the first one's stores, 3-4 us later.  (min_run = 8 where survivor words are
// wanted, which waves fill by the byte.)
inline TailShape tail_shape(int nvec, int vpl, int ub, int min_run) {
    TailShape s;
    int lp = 1;
    while (lp < (int)cdiv(nvec, vpl)) lp <<= 1;
    s.lp = lp < 2 ? 2 : (lp > kWave ? kWave : lp);
    const int per_batch = ub * (kWave / s.lp);                 // entries one batch covers
    s.run = per_batch < min_run ? min_run : (per_batch > kTile ? kTile : per_batch);
    s.nbatch = (int)cdiv(s.run, per_batch);
    return s;
}

__device__ __forceinline__ void store_survivors(uint32_t* surv, int64_t tile, int part, int parts, uint32_t bits) {
    if (parts == 1) surv[tile] = bits;
    else if (parts == 2) reinterpret_cast<uint16_t*>(surv)[tile * 2 + part] = (uint16_t)(bits >> (16 * part));
    else reinterpret_cast<uint8_t*>(surv)[tile * 4 + part] = (uint8_t)(bits >> (8 * part));
}

// Activation + truncation (+ add) of a sparse step: the first stream is a stored delta map.
template <typename T, int V, int VPL, int UB> struct ActSrc {
    typedef typename RawOf<T, V>::type Raw;
    __amdgpu_buffer_rsrc_t in;
    int flag_mine;                       // update flag of the first stream at entry lane%32
    int flag[UB];
    Raw d[UB][VPL];
    __device__ __forceinline__ void select(int ub, int ent) { flag[ub] = __shfl(flag_mine, ent, kWave); }
    __device__ __forceinline__ void issue(int ub, int v, int, bool, uint32_t o) { d[ub][v] = ws_load16<Raw>(in, flag[ub] ? o : kOob); }
    __device__ __forceinline__ Raw finish(int ub, int v, int) const { return d[ub][v]; }
};

}  // namespace dcnn
