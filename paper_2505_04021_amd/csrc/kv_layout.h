// Where an element of a K or V tile sits inside a block (gfx950 operand order).
//
// A block holds, per kv head, the K tile followed by the V tile, T = 16 tokens each;
// e4m3 blocks start with a 128-byte header (fp32 sK[Hkv], fp32 sV[Hkv]).  Tiles are stored
// in the lane order of the MFMA operands the attention kernels feed them to:
//   bf16 K: 16-byte unit (c, t)      = K[t][8c .. 8c+7]                  at ((c*16)+t)*16
//   bf16 V: 16-byte unit (jp, G, dl) = V[4G..4G+3][32jp+dl] ,
//                                      V[4G..4G+3][32jp+16+dl]           at ((jp*4+G)*16+dl)*16
//   e4m3 K: 16-byte unit (j2, G, t)  = K[t][8(8j2+G)+0..7] , K[t][8(8j2+4+G)+0..7]
//   e4m3 V: 16-byte unit (jq, G, dl) = V[4G..4G+3][64jq+16u+dl], u = 0..3
// The functions return the offset in elements from the start of the tile.
#pragma once
#include "pkv_internal.h"

constexpr int PKV_T = 16;   // tokens per block the kernels are built for

template <int DT>
__device__ __forceinline__ size_t k_elem_off(int t, int dd) {
    if (DT == PKV_BF16) return ((size_t)((dd >> 3) * 16 + t)) * 8 + (dd & 7);
    const int c8 = dd >> 3, j = c8 >> 2, Gk = c8 & 3, j2 = j >> 1, hf = j & 1;
    return ((size_t)((j2 * 4 + Gk) * 16 + t)) * 16 + hf * 8 + (dd & 7);
}

template <int DT>
__device__ __forceinline__ size_t v_elem_off(int t, int dd) {
    const int G = t >> 2, e = t & 3;
    if (DT == PKV_BF16) {
        const int jp = dd >> 5, half = (dd >> 4) & 1, dl = dd & 15;
        return ((size_t)((jp * 4 + G) * 16 + dl)) * 8 + half * 4 + e;
    }
    const int jq = dd >> 6, u = (dd >> 4) & 3, dl = dd & 15;
    return ((size_t)((jq * 4 + G) * 16 + dl)) * 16 + u * 4 + e;
}

// Has what every wave uses of a model's descriptor (kernel arguments) asked for here, in one go.  Left to itself the compiler reads a few
// arguments where they are first used, each time a cache line that has not been read before, one memory trip after the
// other in front of the kernel's own: a chunk append waited ten times in a row for its first rows, so three times.  With
// the rows asked for ahead of the block id (page_bf16 and its like), us a pass: append of 8 x 512 tokens into an e4m3 cache
// 24.3 -> 22.8, ragged prompts (append and prefill) 72.2 -> 68.4.
// `also`, `and_also`: two further arguments of the launch, addresses or whole numbers.  (What is used at the end only, or not at all
// in an ordinary call, is left out - out, ws, cnt, err, safe -: it would hold registers meanwhile.)
template <typename A, typename B>
__device__ __forceinline__ void ask_arguments(const AttnDesc &d, A also, B and_also) {
    asm volatile("" ::"s"(also), "s"(and_also), "s"(d.pool_base), "s"(d.q), "s"(d.table), "s"(d.ctx_lens), "s"(d.row_len),
                 "s"(d.frame_bytes), "s"(d.block_bytes), "s"(d.slots_div.d), "s"(d.slots_div.mul), "s"(d.slots_div.sh1),
                 "s"(d.slots_div.sh2), "s"(d.max_block_id), "s"(d.row_stride), "s"(d.Hq), "s"(d.Hkv), "s"(d.g), "s"(d.D), "s"(d.cols),
                 "s"(d.scale_log2));
}

// start of a block in the pool
__device__ __forceinline__ uint8_t *block_ptr(const AttnDesc &d, uint32_t id) {
    const uint32_t f = fastdiv_div(id, d.slots_div);
    const uint32_t s = id - f * d.slots_div.d;
    return const_cast<uint8_t *>(d.pool_base) + (uint64_t)f * d.frame_bytes + (uint64_t)s * d.block_bytes;
}

// The unit u of a chunk launch: which sequence it belongs to (counted from plan.seq0), its number among that
// sequence's units, the sequence's first packed row, its rows and the parts of the context its groups come in.
struct PlanUnit {
    int seq, unit, row, rows, parts;
};

// One read of the plan for all 64 lanes (the constructor) and no further memory trip: the sequence is the last one that
// begins at or before u in the order of the units (sequences without units share their start with the next one).
template <int SEQS>
struct PlanLanes {
    static constexpr int PER_LANE = (SEQS + 1) / 64;
    static_assert(PER_LANE * 64 == SEQS + 1, "whole entries per lane");
    uint32_t unit[PER_LANE], row[PER_LANE];

    __device__ __forceinline__ explicit PlanLanes(const PlanOf<SEQS> &plan) {
#pragma unroll
        for (int k = 0; k < PER_LANE; ++k) {
            const int i = (threadIdx.x & 63) + 64 * k;
            unit[k] = plan.s[i].unit;
            row[k] = plan.s[i].row;
        }
    }
    static __device__ __forceinline__ uint32_t pick(const uint32_t *x, int i) {
        uint32_t v = 0;
#pragma unroll
        for (int k = 0; k < PER_LANE; ++k) v = i >> 6 == k ? (uint32_t)__builtin_amdgcn_readlane((int)x[k], i & 63) : v;
        return v;
    }
    __device__ __forceinline__ uint32_t units(const PlanOf<SEQS> &plan) const { return pick(unit, plan.n_seqs); }
    __device__ __forceinline__ PlanUnit find(const PlanOf<SEQS> &plan, uint32_t u) const {
        const int n = plan.n_seqs;
        int at = -1;
#pragma unroll
        for (int k = 0; k < PER_LANE; ++k) at += __popcll(__ballot((int)(threadIdx.x & 63) + 64 * k < n && (unit[k] & PKV_PLAN_UNITS) <= u));
        PlanUnit r;
        const uint32_t entry = pick(unit, at);
        const int seq = (int)(entry >> PKV_PLAN_SEQ_SHIFT);
        const uint32_t first = pick(row, seq);
        r.seq = plan.seq0 + seq;
        r.unit = (int)(u - (entry & PKV_PLAN_UNITS));
        r.row = (int)(first & PKV_PLAN_ROWS);
        r.rows = (int)(pick(row, seq + 1) & PKV_PLAN_ROWS) - r.row;
        r.parts = (int)(first >> PKV_PLAN_PART_SHIFT);
        return r;
    }
};
