// Paged GQA decode attention over the shared pool (gfx950 / CDNA4).
//
// Defines out = softmax(q K^T / sqrt(D)) V per sequence and query head, with K and V
// read through the sequence's block-table row (paper: Background, "KV cache and
// PagedAttention"; the balloon driver leaves attention semantics untouched, Sec. 4.2
// R4/D4).  The path is bound by HBM reads of K and V, each byte exactly once.
//
// Mapping to the hardware
//   * one wavefront (64 lanes) per work item; the pages of all (sequence, kv head)
//     pairs are laid end to end and cut into shares of equal expected time (pages plus
//     an allowance per segment, scaled by a weight per XCD), whatever the mix of
//     context lengths; where a share boundary
//     cuts a sequence, the wave that finishes it last merges the pieces with the
//     online-softmax rule inside the same kernel (partials and arrival counters sit in
//     uncached memory: no cache flush, no second launch).  Launches of few pages, whose
//     rows suit it, run k_attention_small instead: a work-group per (sequence, kv head)
//     or per part of a long one;
//   * K and V tiles are stored inside a block in the lane order of the MFMA operands,
//     so each 16-byte global load is fully coalesced (64 lanes x 16 B = 1 KiB
//     contiguous) and lands directly in operand registers — no LDS round trip, no
//     shuffles between load and matrix op;
//   * the g query heads that share a kv head are padded to the 16 columns of one
//     MFMA tile: S[token][head] = K . q^T is a 16x16x32 bf16 MFMA per 32 elements of
//     head_dim; pages are taken two at a time, so out^T[d][head] += V^T . P contracts
//     over 32 tokens (4 + 4 per lane, one half from each page) in one 16x16x32 bf16
//     MFMA per 16 elements of head_dim, with P split into bf16 high and low parts (two
//     MFMAs) so that the probabilities keep 16 significant bits; accumulation is fp32;
//   * the softmax runs on the MFMA accumulator layout (lane = 4 tokens x 1 head, per
//     page): in-lane max / sum, then lane-permute swaps across the four lane rows,
//     once per page pair; no LDS in the streaming loop.
//
// In-block layout (per kv head: K tile then V tile, T = 16 tokens):
//   bf16 K: 16-byte unit (c, t)      = K[t][8c .. 8c+7]                 at ((c*16)+t)*16
//   bf16 V: 16-byte unit (jp, G, dl) = V[4G..4G+3][32jp+dl] ,
//                                      V[4G..4G+3][32jp+16+dl]          at ((jp*4+G)*16+dl)*16
//   e4m3 K: 16-byte unit (j2, G, t)  = K[t][8(8j2+G)+0..7] , K[t][8(8j2+4+G)+0..7]
//   e4m3 V: 16-byte unit (jq, G, dl) = V[4G..4G+3][64jq+16u+dl], u = 0..3
//   e4m3 blocks start with a 128-byte header: fp32 sK[Hkv], fp32 sV[Hkv].
#include "mfma_util.h"

namespace {

constexpr int T = PKV_T;

template <int D, int DT>
struct Tile {
    static constexpr int E = DT == PKV_BF16 ? 2 : 1;
    static constexpr int TILE_BYTES = T * D * E;           // one K or V tile
    static constexpr int NL = TILE_BYTES / 1024;           // 16-byte loads per lane per tile
    static constexpr int NK = D / 32;                      // QK^T MFMAs per page
    static constexpr int NV = D / 16;                      // d-tiles of the output
};

template <int D, int DT>
struct PageRegs {
    u32x4 k[Tile<D, DT>::NL];
    u32x4 v[Tile<D, DT>::NL];
    float sk, sv;
};

// Block ids of a page pair.  They are read through the scalar cache one step before the
// loads that need them are issued, so the latency of this dependent access (block table
// -> address -> K/V load) is covered by the arithmetic of the step in between.
struct PairIds {
    uint32_t a, b;
};

__device__ __forceinline__ PairIds fetch_ids(const AttnDesc &d, const int32_t *row, int page) {
    const int last = d.row_stride - 1;
    // wave-uniform, and said to be: the ids come through the scalar cache (a vector load would wait for all K and V in flight)
    row = reinterpret_cast<const int32_t *>((uint32_t)__builtin_amdgcn_readfirstlane((int)(uintptr_t)row) |
                                            (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)((uintptr_t)row >> 32)) << 32);
    const int ia = page < last ? page : last, ib = page + 1 < last ? page + 1 : last;
    PairIds ids;
    ids.a = (uint32_t)__builtin_amdgcn_readfirstlane(PKV_CONST(int32_t, row)[ia]);
    ids.b = (uint32_t)__builtin_amdgcn_readfirstlane(PKV_CONST(int32_t, row)[ib]);
    return ids;
}

// Issue the loads of one page (K tile, V tile) of one kv head.  Buffer loads with a
// per-page resource descriptor: a page beyond the chunk (live == false) gets a
// descriptor of zero records, so its loads return zeros without touching memory.
// That keeps every load of the software pipeline unconditional, which lets the
// compiler count outstanding loads exactly (s_waitcnt vmcnt(N) with N > 0) instead of
// draining the queue at each control-flow join.
template <int D, int DT>
__device__ __forceinline__ void load_page(PageRegs<D, DT> &r, const AttnDesc &d, uint32_t id, bool live, int kvh,
                                          int lane, uint32_t &bad) {
    using TL = Tile<D, DT>;
    if (id >= d.max_block_id) {          // never dereference an id outside the pool
        bad |= live ? 1u : 0u;           // reported once, after the last load (no store inside the loop)
        id = 0;
        live = false;                    // the page is skipped: frame 0 need not even be backed by memory
    }
    const uint8_t *blk = block_ptr(d, id);
    if (DT == PKV_E4M3) {
        // A dead page's id is whatever the table holds past the row's end: possibly a block of a
        // frame that was given back and, in an elastic pool, is no longer backed by memory.
        // Its header must not be read (the tile loads below are harmless: zero records).
        const float *hdr = reinterpret_cast<const float *>(live ? blk : reinterpret_cast<const uint8_t *>(d.safe));
        r.sk = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(PKV_CONST(float, hdr)[kvh])));
        r.sv = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(PKV_CONST(float, hdr)[d.Hkv + kvh])));
        if (!live) r.sk = r.sv = 0.f;
        blk += PKV_FP8_HEADER;
    }
    const uint8_t *tiles = blk + (size_t)kvh * 2 * TL::TILE_BYTES;
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(tiles), 0, live ? 2 * TL::TILE_BYTES : 0, 0x00020000);
    const int voff = lane * 16;
#pragma unroll
    for (int j = 0; j < TL::NL; ++j)
        r.k[j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff + j * 1024, 0, 2 /* non-temporal */);
#pragma unroll
    for (int j = 0; j < TL::NL; ++j)
        r.v[j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff + j * 1024, TL::TILE_BYTES, 2);
}

template <int D, int DT>
struct State {
    f32x4 acc[Tile<D, DT>::NV];   // out^T tiles: acc[jt][i] = out[16jt + 4G + i][head n]
    float m, l;                   // running max (log2 domain) and this lane's share of the sum
};

// Two consecutive pages of a piece travel and are processed together (32 tokens): one
// max / rescale step per 32 tokens and 16x16x32 MFMAs for the PV product.
template <int D, int DT>
struct PairRegs {
    PageRegs<D, DT> a, b;
};

template <int D, int DT>
__device__ __forceinline__ void load_pair(PairRegs<D, DT> &r, const AttnDesc &d, PairIds ids, bool live_a, bool live_b,
                                          int kvh, int lane, uint32_t &bad) {
    load_page<D, DT>(r.a, d, ids.a, live_a, kvh, lane, bad);
    load_page<D, DT>(r.b, d, ids.b, live_b, kvh, lane, bad);
}

// S[token][head] of one page: K (A operand, row = token) times q (B operand)
template <int D, int DT>
__device__ __forceinline__ f32x4 qk_page(const PageRegs<D, DT> &r, const bf16x8 *qf) {
    using TL = Tile<D, DT>;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (DT == PKV_BF16) {
#pragma unroll
        for (int j = 0; j < TL::NK; ++j) {
            u32x4 kv = r.k[j];
            s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8 *>(&kv), qf[j], s, 0, 0, 0);
        }
    } else {
#pragma unroll
        for (int j2 = 0; j2 < TL::NL; ++j2) {
            const u32x4 kv = r.k[j2];
            const u32x2 a0 = fp8x4_to_bf16x4(kv.x), a1 = fp8x4_to_bf16x4(kv.y);
            const u32x2 b0 = fp8x4_to_bf16x4(kv.z), b1 = fp8x4_to_bf16x4(kv.w);
            u32x4 ka = mk4(a0.x, a0.y, a1.x, a1.y);
            u32x4 kb = mk4(b0.x, b0.y, b1.x, b1.y);
            s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8 *>(&ka), qf[2 * j2], s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*reinterpret_cast<bf16x8 *>(&kb), qf[2 * j2 + 1], s, 0, 0, 0);
        }
    }
    return s;
}

// V of one page for output tile jt as four bf16: V[4G..4G+3][16jt + (lane & 15)]
template <int D, int DT>
__device__ __forceinline__ u32x2 v_half(const PageRegs<D, DT> &r, int jt) {
    if (DT == PKV_BF16) {
        const u32x4 vv = r.v[jt >> 1];
        return (jt & 1) ? mk2(vv.z, vv.w) : mk2(vv.x, vv.y);
    }
    const u32x4 vv = r.v[jt >> 2];
    const uint32_t w = (jt & 3) == 0 ? vv.x : (jt & 3) == 1 ? vv.y : (jt & 3) == 2 ? vv.z : vv.w;
    return fp8x4_to_bf16x4(w);
}

// bf16 hi + lo of four probabilities: 16 significant bits reach the matrix unit
__device__ __forceinline__ void split_p(const float *p, u32x2 &hi, u32x2 &lo) {
    const uint32_t h01 = pack_bf16_rne(p[0], p[1]), h23 = pack_bf16_rne(p[2], p[3]);
    const float l0 = p[0] - __uint_as_float(h01 << 16), l1 = p[1] - __uint_as_float(h01 & 0xffff0000u);
    const float l2 = p[2] - __uint_as_float(h23 << 16), l3 = p[3] - __uint_as_float(h23 & 0xffff0000u);
    hi = mk2(h01, h23);
    lo = mk2(pack_bf16_rne(l0, l1), pack_bf16_rne(l2, l3));
}

// Blanks the tokens of a V tile past the context, which may hold anything (even NaN); live of the four that this lane holds count.
template <int D, int DT>
__device__ __forceinline__ void blank_v(u32x4 *v, int live) {
    const uint32_t m01 = live >= 2 ? 0xffffffffu : (live == 1 ? 0x0000ffffu : 0u), m23 = live >= 4 ? 0xffffffffu : (live == 3 ? 0x0000ffffu : 0u);
    const uint32_t m = live >= 4 ? 0xffffffffu : (live <= 0 ? 0u : (1u << (8 * live)) - 1u);      // codes
#pragma unroll
    for (int j = 0; j < Tile<D, DT>::NL; ++j) v[j] &= DT == PKV_BF16 ? mk4(m01, m23, m01, m23) : mk4(m, m, m, m);
}

// Small launches: the reference point, the sums and the probabilities of one online-softmax step, as process_pair below takes them,
// from scaled and masked logits s; but logits of -inf may be all that a column has seen so far, and weigh nothing.
template <int D, int DT>
__device__ __forceinline__ void softmax_pair(State<D, DT> &st, const float *s, float sva, float svb, bf16x8 &phv, bf16x8 &plv) {
    using TL = Tile<D, DT>;
    float mx = fmaxf(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])), fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7])));
    mx = rows_max(mx);
    const float m_new = fmaxf(st.m, mx);
    // wave-uniform: the reference point of the exponentials moves, and the sums are rescaled, only when some
    // column's maximum has run ahead of it by more than kRescaleSlack (probabilities stay below 2^kRescaleSlack)
    if (__any(m_new > st.m + kRescaleSlack)) {
        const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(st.m - m_new);
        st.l *= alpha;
#pragma unroll
        for (int jt = 0; jt < TL::NV; ++jt) st.acc[jt] *= alpha;
        st.m = m_new;
    }
    float p[8];
    const float m_ref = st.m == -INFINITY ? 0.f : st.m;      // then every s is -inf and every p is 0
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i] = __builtin_amdgcn_exp2f(s[i] - m_ref);
    st.l += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
    if (DT == PKV_E4M3) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] *= sva;
            p[4 + i] *= svb;
        }
    }
    // B operand of the PV product: lane (G, head) holds P for tokens 4G..4G+3 of page a, then of page b
    u32x2 ha, la, hb, lb;
    split_p(p, ha, la);
    split_p(p + 4, hb, lb);
    u32x4 ph = mk4(ha.x, ha.y, hb.x, hb.y), pl = mk4(la.x, la.y, lb.x, lb.y);
    phv = *reinterpret_cast<bf16x8 *>(&ph);
    plv = *reinterpret_cast<bf16x8 *>(&pl);
}

// One online-softmax step over the 32 tokens of a page pair.  valid_a is 1..16,
// valid_b 0..16 (0: the pair has no second page; its registers hold zeros).  Whether the
// pair needs masks is decided at run time inside (one code path with selects: the kernel is
// bound by memory).
template <int D, int DT>
__device__ __forceinline__ void process_pair(State<D, DT> &st, const PairRegs<D, DT> &r, const bf16x8 *qf,
                                             float scale_log2, int valid_a, int valid_b, int G) {
    using TL = Tile<D, DT>;
    const bool tail = valid_a < T || valid_b < T;
    f32x4 sa = qk_page<D, DT>(r.a, qf);
    f32x4 sb = qk_page<D, DT>(r.b, qf);
    const float sca = DT == PKV_E4M3 ? scale_log2 * r.a.sk : scale_log2;
    const float scb = DT == PKV_E4M3 ? scale_log2 * r.b.sk : scale_log2;
    float s[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        s[i] = sa[i] * sca;
        s[4 + i] = sb[i] * scb;
        if (tail) {                                        // select, so a NaN logit of a dead token cannot leak
            if (4 * G + i >= valid_a) s[i] = -INFINITY;
            if (4 * G + i >= valid_b) s[4 + i] = -INFINITY;
        }
    }
    float mx = fmaxf(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])), fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7])));
    mx = rows_max(mx);
    const float m_new = fmaxf(st.m, mx);
    // wave-uniform: the reference point of the exponentials moves, and the sums are rescaled, only when some
    // column's maximum has run ahead of it by more than kRescaleSlack (probabilities stay below 2^kRescaleSlack)
    if (__any(m_new > st.m + kRescaleSlack)) {
        const float alpha = __builtin_amdgcn_exp2f(st.m - m_new);
        st.l *= alpha;
#pragma unroll
        for (int jt = 0; jt < TL::NV; ++jt) st.acc[jt] *= alpha;
        st.m = m_new;
    }
    float p[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i] = __builtin_amdgcn_exp2f(s[i] - st.m);
    st.l += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
    if (DT == PKV_E4M3) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] *= r.a.sv;
            p[4 + i] *= r.b.sv;
        }
    }
    // B operand of the PV product: lane (G, head) holds P for tokens 4G..4G+3 of page a, then of page b
    u32x2 ha, la, hb, lb;
    split_p(p, ha, la);
    split_p(p + 4, hb, lb);
    u32x4 ph = mk4(ha.x, ha.y, hb.x, hb.y), pl = mk4(la.x, la.y, lb.x, lb.y);
    const bf16x8 phv = *reinterpret_cast<bf16x8 *>(&ph), plv = *reinterpret_cast<bf16x8 *>(&pl);
    // tokens past the context length may hold anything (even NaN): blank their V
    uint32_t ma01 = 0xffffffffu, ma23 = 0xffffffffu, mb01 = 0xffffffffu, mb23 = 0xffffffffu;
    if (tail) {
        const int la_ = valid_a - 4 * G, lb_ = valid_b - 4 * G;
        ma01 = la_ >= 2 ? 0xffffffffu : (la_ == 1 ? 0x0000ffffu : 0u);
        ma23 = la_ >= 4 ? 0xffffffffu : (la_ == 3 ? 0x0000ffffu : 0u);
        mb01 = lb_ >= 2 ? 0xffffffffu : (lb_ == 1 ? 0x0000ffffu : 0u);
        mb23 = lb_ >= 4 ? 0xffffffffu : (lb_ == 3 ? 0x0000ffffu : 0u);
    }
#pragma unroll
    for (int jt = 0; jt < TL::NV; ++jt) {
        // A operand: V^T, row = output element 16jt + (lane & 15), k = the same eight tokens
        const u32x2 va = v_half<D, DT>(r.a, jt), vb = v_half<D, DT>(r.b, jt);
        u32x4 vv = tail ? mk4(va.x & ma01, va.y & ma23, vb.x & mb01, vb.y & mb23) : mk4(va.x, va.y, vb.x, vb.y);
        const bf16x8 av = *reinterpret_cast<bf16x8 *>(&vv);
        st.acc[jt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, phv, st.acc[jt], 0, 0, 0);
        st.acc[jt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, plv, st.acc[jt], 0, 0, 0);
    }
}

constexpr int FLIGHT_KIB_2WAVES = 16;      // bytes in flight per wave, two waves per SIMD
// Page pairs resident per wave: one in use, the rest in flight.  In the form with two waves per
// SIMD every shape keeps the same number of bytes in flight (FLIGHT_KIB_2WAVES), small pages
// through a deeper ring; otherwise waves of a small-page model would fall behind the others in
// a grouped launch.
template <int D, int DT, int FLIGHT_KIB = FLIGHT_KIB_2WAVES>
struct Ring {
    static constexpr int PAIR_BYTES = 4 * Tile<D, DT>::TILE_BYTES;        // K and V tiles of two pages
    static constexpr int N = 1 + (FLIGHT_KIB * 1024 + PAIR_BYTES - 1) / PAIR_BYTES;
};
// The second form of the kernel: one wave per SIMD, the host launching only as many waves as it
// takes to keep the memory system busy (512 for bf16 pages of 8 KiB).  A wave alone on its SIMD
// turns a page pair over in 0.7-1.1 us whatever it has in flight, so one pair in use and one
// travelling is all the ring needs (8 KiB covers a pair of every shape but bf16 with 128-wide
// heads, whose pair of 16 KiB is the one in flight anyway); more bytes outstanding only lengthen
// the queues in front of the memory channels, and the launch as a whole gets slower.
constexpr int FLIGHT_KIB_1WAVE = 8;
constexpr int MAX_PIECES = 64;   // pieces of one (sequence, kv head) the merge stages in LDS

__device__ __forceinline__ int ctx_clamped(const AttnDesc &d, int seq) {
    int L = PKV_CONST(int32_t, d.ctx_lens)[seq];
    const int cap = (d.row_len ? PKV_CONST(int32_t, d.row_len)[seq] : d.row_stride) * T;
    return L < 0 ? 0 : (L > cap ? cap : L);
}

// Length a segment is given on the line the shares are cut from: its pages plus a fixed
// allowance for what every segment costs besides its pages (the turn it does not fill,
// the gap in the stream at its boundary, writing its result), at least 1 so that an
// empty sequence still has an owner who writes its zero row.
__device__ __forceinline__ int planned(const AttnDesc &d, int n_pages) {
    const int pl = n_pages + d.seg_cost;
    return pl > 0 ? pl : 1;
}

// A piece: the pages [pb, pe) of one (sequence, kv head) segment that fall into this
// wave's share.  All fields are wave-uniform.
struct Piece {
    int valid;                  // 0 past the end of the share
    int seq, kvh;
    int P;                      // planned pages of all earlier sequences
    int L, n_pages, pl;         // context length, its pages, planned pages (>= 1)
    int pb, pe;                 // page range of the piece inside the segment
    uint32_t g0;                // where the segment starts on the line of page units
};

__device__ __forceinline__ void piece_set_seq(Piece &pc, const AttnDesc &d, int seq, int P) {
    pc.seq = seq;
    pc.P = P;
    pc.L = seq < d.batch ? __builtin_amdgcn_readfirstlane(ctx_clamped(d, seq < d.batch ? seq : 0)) : 0;
    pc.n_pages = (pc.L + T - 1) / T;
    pc.pl = planned(d, pc.n_pages);
}

// clip segment (seq, kvh) against the share [gbeg, gend)
__device__ __forceinline__ void piece_clip(Piece &pc, const AttnDesc &d, uint32_t gbeg, uint32_t gend) {
    pc.g0 = (uint32_t)pc.P * d.Hkv + (uint32_t)pc.kvh * pc.pl;
    pc.valid = (pc.seq < d.batch && pc.g0 < gend) ? 1 : 0;
    pc.pb = gbeg > pc.g0 ? (int)(gbeg - pc.g0) : 0;
    pc.pe = gend - pc.g0 < (uint32_t)pc.pl ? (int)(gend - pc.g0) : pc.pl;
    // the allowance past the last page holds no work; an empty sequence has the one unit [0, 1)
    const int real = pc.n_pages > 0 ? pc.n_pages : 1;
    pc.pe = pc.pe < real ? pc.pe : real;
}

__device__ __forceinline__ Piece piece_next(const Piece &c, const AttnDesc &d, uint32_t gbeg, uint32_t gend) {
    Piece nx = c;
    if (c.kvh + 1 < d.Hkv) {
        nx.kvh = c.kvh + 1;
    } else {
        nx.kvh = 0;
        piece_set_seq(nx, d, c.seq + 1, c.P + c.pl);
    }
    piece_clip(nx, d, gbeg, gend);
    return nx;
}

// Whether MFMA column n is a query head at all.  Worked out anew for every piece: known to be the same throughout,
// the compiler splits the streaming loop on it and loses count of the loads in flight (full waits inside the loop).
__device__ __forceinline__ bool column_live(const AttnDesc &d, int n) {
    asm volatile("" : "+v"(n));
    return n < d.g;
}

// q as the B operand (column n: head n of the kv head's group): lane (G, n) holds q[column n][8(4j+G) .. +7] for each k-step j
template <int D>
__device__ __forceinline__ void load_q(bf16x8 *qf, const AttnDesc &d, int seq, int kvh, int lane) {
    const int G = lane >> 4, n = lane & 15;
    const uint16_t *qrow = d.q + ((size_t)seq * d.Hq + kvh * d.g + n) * D;
    const bool live = column_live(d, n);
#pragma unroll
    for (int j = 0; j < D / 32; ++j) {
        u32x4 v = mk4(0, 0, 0, 0);
        if (live) v = *reinterpret_cast<const u32x4 *>(qrow + 8 * (4 * j + G));
        qf[j] = *reinterpret_cast<bf16x8 *>(&v);
    }
}

// What is left to do for a piece whose segment is shared with other waves: once the
// arrival count is back, the wave that came last merges.
struct Pending {
    int valid, seq, kvh;
    uint32_t k0, k1, arrived;
};

// online-softmax merge of the pieces of one segment: M = max m_c,
// out = sum_c 2^(m_c-M) a_c / sum_c 2^(m_c-M) l_c.  Piece c of the segment sits in
// share k0 + c: slot b of that share for c = 0, slot a otherwise.
// The partials come from uncached memory, so the cost is memory round trips: each lane
// owns EPL groups of four consecutive output elements and fetches the accumulators of
// 32 / EPL pieces per trip; the maxima and sums of all pieces travel with the first trip
// and are staged in LDS.
template <int D, int EPL>
__device__ __forceinline__ void merge_rows(const AttnDesc &d, const Pending &pd, int lane, float *s_m, float *s_l,
                                           const float *base, int n_pc) {
    constexpr int D4 = D / 4;
    constexpr int PB = 32 / EPL;                      // pieces per trip
    const int g = d.g, pf = partial_floats(g, D);
    const int E = g * D4;
    int hn[EPL], x[EPL];
#pragma unroll
    for (int k = 0; k < EPL; ++k) {
        const int e = lane + 64 * k;
        const int ee = e < E ? e : E - 1;             // idle lanes shadow a valid element
        hn[k] = ee / D4;
        x[k] = ee - hn[k] * D4;
    }
    // first trip: the accumulators of the first PB pieces travel together with all maxima and sums
    f32x4 v[PB][EPL];
#pragma unroll
    for (int u = 0; u < PB; ++u) {
        const int c = u < n_pc ? u : n_pc - 1;
        const float *wc = base + (size_t)(2 * c + (c == 0 ? 1 : 0)) * pf;
#pragma unroll
        for (int k = 0; k < EPL; ++k) v[u][k] = *reinterpret_cast<const f32x4 *>(wc + hn[k] * D + 4 * x[k]);
    }
    for (int i = lane; i < n_pc * g; i += 64) {
        const int c = i / g, h = i - c * g;
        const float *wc = base + (size_t)(2 * c + (c == 0 ? 1 : 0)) * pf + g * D;
        s_m[i] = wc[h];
        s_l[i] = wc[g + h];
    }
    __builtin_amdgcn_wave_barrier();     // one wave per work-group: program order is enough
    float M[EPL], den[EPL];
    f32x4 num[EPL];
#pragma unroll
    for (int k = 0; k < EPL; ++k) {
        float mm = -INFINITY;
        for (int c = 0; c < n_pc; ++c) mm = fmaxf(mm, s_m[c * g + hn[k]]);
        M[k] = mm;
        den[k] = 0.f;
        num[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    for (int c0 = 0; c0 < n_pc; c0 += PB) {
        if (c0 > 0) {
#pragma unroll
            for (int u = 0; u < PB; ++u) {
                const int c = c0 + u < n_pc ? c0 + u : n_pc - 1;
                const float *wc = base + (size_t)(2 * c + (c == 0 ? 1 : 0)) * pf;
#pragma unroll
                for (int k = 0; k < EPL; ++k) v[u][k] = *reinterpret_cast<const f32x4 *>(wc + hn[k] * D + 4 * x[k]);
            }
        }
#pragma unroll
        for (int u = 0; u < PB; ++u) {
            if (c0 + u < n_pc) {
#pragma unroll
                for (int k = 0; k < EPL; ++k) {
                    const float f = __builtin_amdgcn_exp2f(s_m[(c0 + u) * g + hn[k]] - M[k]);
                    den[k] += f * s_l[(c0 + u) * g + hn[k]];
                    num[k] += f * v[u][k];
                }
            }
        }
    }
#pragma unroll
    for (int k = 0; k < EPL; ++k) {
        if (lane + 64 * k < E)
            *reinterpret_cast<f32x4 *>(d.out + ((size_t)pd.seq * d.Hq + pd.kvh * g + hn[k]) * D + 4 * x[k]) = num[k] * (1.0f / den[k]);
    }
    __builtin_amdgcn_wave_barrier();
}

template <int D>
__device__ __forceinline__ void merge_segment(const AttnDesc &d, const Pending &pd, int lane, float *s_m, float *s_l) {
    const int g = d.g, pf = partial_floats(g, D);
    const int n_pc = (int)(pd.k1 - pd.k0) + 1;
    const float *base = d.ws + (size_t)(2 * pd.k0) * pf;
    const int groups = (g * (D / 4) + 63) / 64;       // element groups per lane
    if (groups <= 1) merge_rows<D, 1>(d, pd, lane, s_m, s_l, base, n_pc);
    else if (groups <= 2) merge_rows<D, 2>(d, pd, lane, s_m, s_l, base, n_pc);
    else if (groups <= 4) merge_rows<D, 4>(d, pd, lane, s_m, s_l, base, n_pc);
    else merge_rows<D, 8>(d, pd, lane, s_m, s_l, base, n_pc);
}

// Work split ("stream-K" over pages): the (sequence, kv head) segments of a model are
// laid end to end, a segment being the pages of one sequence for one kv head; the
// resulting line of W page units is cut into equal shares, one per wave.  A wave's
// share may end inside a segment and start inside another: such pieces leave a partial
// (accumulators, max, sum) in uncached memory, and the wave that completes a segment
// last merges its pieces with the online-softmax rule.  Segments that lie inside one
// share are finished directly.  Every wave derives the split from ctx_lens itself, so
// the split follows the real context lengths and needs no host-side plan.
//
// Inside a share the pages of consecutive pieces form ONE stream through the register
// ring: pages travel and are processed in pairs (32 tokens), work proceeds in turns of
// RING pairs, every piece is padded to whole turns with dead pages (no traffic, no
// math), and during the last turn of a piece the loads already fetch the first pairs of
// the next piece.
// Where the shares of the work items begin on the line of page units.  Items come in
// blocks of eight (one per XCD); a block spans 8 * share units and is cut at
// cum[j] / 65536 of its length (cum[0] = 0, cum[8] = 65536), or evenly without weights.
constexpr uint32_t WEIGHTED_SHARE_MIN = 16;     // below this, uneven cuts could leave a share empty
struct Cut {
    uint32_t share;
    const uint32_t *cum;        // kernel-argument memory, or NULL for even cuts

    __device__ __forceinline__ uint32_t begin(uint32_t item) const {
        if (!cum) return item * share;
        const uint32_t blk = item >> 3, j = item & 7u;
        return blk * 8u * share + (uint32_t)(((uint64_t)(8u * share) * PKV_CONST(uint32_t, cum)[j]) >> 16);
    }
    // the item whose share holds line position x
    __device__ __forceinline__ uint32_t index(uint32_t x) const {
        if (!cum) return x / share;
        const uint32_t s8 = 8u * share, blk = x / s8, rem = x - blk * s8;
        uint32_t j = 0;
#pragma unroll
        for (uint32_t t = 1; t < 8; ++t)
            j += rem >= (uint32_t)(((uint64_t)s8 * PKV_CONST(uint32_t, cum)[t]) >> 16) ? 1u : 0u;
        return blk * 8u + j;
    }
};


// CACHED: the partials and arrival counters sit in ordinary (cached) device memory instead of
// uncached memory.  The L2 caches of the eight XCDs are not coherent with each other for such
// memory, so the hand-over of a partial follows the memory model by the book: partial stores,
// release fence, arrival atomic (agent scope) on the writer's side; arrival atomic, acquire fence,
// partial loads on the merger's side.
template <int D, int DT, int FLIGHT_KIB = FLIGHT_KIB_2WAVES, bool CACHED = false>
__device__ __forceinline__ void attn_wave(const AttnDesc &d, const AttnTune &w, int item, float *s_m, float *s_l) {
    using TL = Tile<D, DT>;
    const int lane = threadIdx.x;
    __builtin_amdgcn_s_setprio(3);      // from the first instruction: a wave still setting up must not wait behind streaming ones
    const int G = lane >> 4, n = lane & 15;
    const int g = d.g, Hkv = d.Hkv, B = d.batch;
    const uint64_t t_begin = w.stat ? wall_clock64() : 0;

    // --- planned pages per sequence, prefix sums across the wave.  Batches of up to
    // 64 * LINE_REGS sequences keep every context length in registers, so that finding
    // the first segment costs no further memory access.
    constexpr int LINE_REGS = 4;
    const int K = (B + 63) >> 6;                    // sequences per lane
    int Lc[LINE_REGS];
    int my_sum = 0, my_max = 0;
#pragma unroll
    for (int k = 0; k < LINE_REGS; ++k) {
        const int sq = lane * K + k;
        Lc[k] = (k < K && sq < B) ? ctx_clamped(d, sq) : -1;
    }
    if (K <= LINE_REGS) {
#pragma unroll
        for (int k = 0; k < LINE_REGS; ++k) {
            if (Lc[k] >= 0) {
                const int np = (Lc[k] + T - 1) / T;
                const int pl = planned(d, np);
                my_sum += pl;
                my_max = pl > my_max ? pl : my_max;
            }
        }
    } else {
        for (int k = 0; k < K; ++k) {
            const int sq = lane * K + k;
            if (sq < B) {
                const int np = (ctx_clamped(d, sq) + T - 1) / T;
                const int pl = planned(d, np);
                my_sum += pl;
                my_max = pl > my_max ? pl : my_max;
            }
        }
    }
    int incl = my_sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o);
        if (lane >= o) incl += v;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int v = __shfl_xor(my_max, o);
        my_max = v > my_max ? v : my_max;
    }
    const int total = __builtin_amdgcn_readlane(incl, 63);
    const uint32_t W = (uint32_t)total * (uint32_t)Hkv;
    // Shares: equal in the mean, but never so small that a segment falls into more pieces
    // than the merge can stage.  Eight consecutive items run on the eight XCDs (work-groups
    // are dealt to them in turn), and XCDs do not all get the same memory bandwidth; so a
    // block of eight shares is cut at the caller's cumulative weights instead of evenly.
    uint32_t share = (W + (uint32_t)d.n_items - 1) / (uint32_t)d.n_items;
    const uint32_t floor_share = ((uint32_t)my_max + (MAX_PIECES - 24) - 1) / (MAX_PIECES - 24);
    share = share < floor_share ? floor_share : share;
    share = share < (uint32_t)d.min_share ? (uint32_t)d.min_share : share;
    share = (uint32_t)__builtin_amdgcn_readfirstlane((int)share);
    const Cut cut = Cut{share, (share >= WEIGHTED_SHARE_MIN && d.weighted) ? w.cum : nullptr};
    const uint32_t gbeg = cut.begin((uint32_t)item);
    uint32_t gend = cut.begin((uint32_t)item + 1);
    if (gbeg >= W) return;
    gend = gend < W ? gend : W;

    // --- which segment holds line position x: the lane whose sequences span x walks them (from
    // registers for batches that fit there)
    auto locate = [&](uint32_t x, int &seq, int &P, int &L) {
        const uint32_t lo = (uint32_t)(incl - my_sum) * Hkv, hi = (uint32_t)incl * Hkv;
        const unsigned long long own = __ballot(lo <= x && x < hi);
        const int owner = __ffsll(own) - 1;
        int fs = 0, fp = incl - my_sum, fl = 0;     // sequence, pages before it, its context length
        if (K <= LINE_REGS) {
            bool found = false;
#pragma unroll
            for (int k = 0; k < LINE_REGS; ++k) {
                if (!found && Lc[k] >= 0) {
                    const int np = (Lc[k] + T - 1) / T;
                    const int pl = planned(d, np);
                    if ((uint32_t)(fp + pl) * Hkv <= x) fp += pl;
                    else { fs = lane * K + k; fl = Lc[k]; found = true; }
                }
            }
        } else {
            for (int k = 0; k < K; ++k) {           // only the owner's walk matters
                const int sq = lane * K + k;
                if (sq < B) {
                    const int L1 = ctx_clamped(d, sq);
                    const int np = (L1 + T - 1) / T;
                    const int pl = planned(d, np);
                    if ((uint32_t)(fp + pl) * Hkv <= x) fp += pl; else { fs = sq; fl = L1; break; }
                }
            }
        }
        seq = __builtin_amdgcn_readfirstlane(__shfl(fs, owner));
        P = __builtin_amdgcn_readfirstlane(__shfl(fp, owner));
        L = __builtin_amdgcn_readfirstlane(__shfl(fl, owner));
    };
    auto piece_at = [&](uint32_t x) {
        Piece pc;
        locate(x, pc.seq, pc.P, pc.L);
        pc.n_pages = (pc.L + T - 1) / T;
        pc.pl = planned(d, pc.n_pages);
        pc.kvh = (int)((x - (uint32_t)pc.P * Hkv) / (uint32_t)pc.pl);
        piece_clip(pc, d, gbeg, gend);
        return pc;
    };

    // --- the first piece: the segment that contains gbeg
    Piece cur = piece_at(gbeg);
    // a share may begin in the allowance behind a segment's last page: nothing to do there
    if (cur.pb >= cur.pe) cur = piece_next(cur, d, gbeg, gend);
    if (!cur.valid) return;

    uint32_t bad = 0;
    const int pf = partial_floats(g, D);
    float *ws_a = d.ws + (size_t)(2 * item) * pf;       // piece of a segment that began in an earlier share
    float *ws_b = ws_a + pf;                            // piece of a segment that begins in this share
    Pending pend_a, pend_b;
    pend_a.valid = pend_b.valid = 0;
    pend_a.arrived = pend_b.arrived = 0;

    // prologue of the stream: the first page pairs of the first piece, and its q
    constexpr int RING = Ring<D, DT, FLIGHT_KIB>::N;
    PairRegs<D, DT> ring[RING];
    PairIds pre;                            // block ids of the next pair to be requested
    {
        const int32_t *row = d.table + (size_t)cur.seq * d.row_stride;
        const int live_n = cur.n_pages > 0 ? cur.pe - cur.pb : 0;
#pragma unroll
        for (int r = 0; r < RING - 1; ++r)
            load_pair<D, DT>(ring[r], d, fetch_ids(d, row, cur.pb + 2 * r), 2 * r < live_n, 2 * r + 1 < live_n,
                             cur.kvh, lane, bad);
        pre = fetch_ids(d, row, cur.pb + 2 * (RING - 1));
    }
    bf16x8 qf[TL::NK], qn[TL::NK];
    load_q<D>(qf, d, cur.seq, cur.kvh, lane);

    State<D, DT> st;
    // Instruction issue favours the older wave of a SIMD, and at two waves per SIMD the
    // younger one can starve for tens of microseconds before it gets its turn.  A wave
    // therefore starts at the highest priority and steps down as its share proceeds, so
    // whichever wave is behind is the one that is favoured.
    const uint32_t prio_total = gend - gbeg + 1;
    uint32_t prio_done = 0;
    int prio_lvl = 0;
    while (cur.valid) {
        const Piece nxt = piece_next(cur, d, gbeg, gend);
        const int seq_n = __builtin_amdgcn_readfirstlane(nxt.valid ? nxt.seq : cur.seq);
        // q of the next piece travels while this piece streams (of this piece again if there is no next)
        load_q<D>(qn, d, seq_n, nxt.valid ? nxt.kvh : cur.kvh, lane);
#pragma unroll
        for (int jt = 0; jt < TL::NV; ++jt) st.acc[jt] = f32x4{0.f, 0.f, 0.f, 0.f};
        st.m = -INFINITY;
        st.l = 0.f;

        const int32_t *row_c = d.table + (size_t)__builtin_amdgcn_readfirstlane(cur.seq) * d.row_stride;
        const int32_t *row_n = d.table + (size_t)seq_n * d.row_stride;
        const bool col_live = column_live(d, n);
        const int n_live = cur.n_pages > 0 ? cur.pe - cur.pb : 0;       // pages to read and process
        const int n_next = (nxt.valid && nxt.n_pages > 0) ? nxt.pe - nxt.pb : 0;
        const int n_pairs = n_live > 0 ? (n_live + 1) >> 1 : 1;         // an empty segment still takes a turn
        const int last_valid = cur.L - (cur.n_pages - 1) * T;
        for (int t0 = 0; t0 < n_pairs; t0 += RING) {
            const bool last_turn = t0 + RING >= n_pairs;
#pragma unroll
            for (int r = 0; r < RING; ++r) {
                {
                    const int lvl = (int)(prio_done * 4u / prio_total) & 3;
                    if (lvl != prio_lvl) {
                        prio_lvl = lvl;
                        if (lvl == 1) __builtin_amdgcn_s_setprio(2);
                        else if (lvl == 2) __builtin_amdgcn_s_setprio(1);
                        else __builtin_amdgcn_s_setprio(0);
                    }
                }
                // request: position RING-1 of this turn (r == 0), else position r-1 of the next
                // turn, which belongs to the next piece when this is the piece's last turn
                {
                    const bool of_next = r > 0 && last_turn;
                    const int i = r == 0 ? 2 * (t0 + RING - 1) : (last_turn ? 2 * (r - 1) : 2 * (t0 + RING + r - 1));
                    const int lim = of_next ? n_next : n_live;
                    load_pair<D, DT>(ring[(r + RING - 1) % RING], d, pre, i < lim, i + 1 < lim,
                                     of_next ? nxt.kvh : cur.kvh, lane, bad);
                }
                // ids of the request after this one: the next step of this turn, or the first
                // step of the turn that follows (this piece's next turn, else the next piece's first)
                {
                    const int32_t *row;
                    int page;
                    if (r + 1 < RING) {
                        row = last_turn ? row_n : row_c;
                        page = last_turn ? nxt.pb + 2 * r : cur.pb + 2 * (t0 + RING + r);
                    } else {
                        row = last_turn ? row_n : row_c;
                        page = last_turn ? nxt.pb + 2 * (RING - 1) : cur.pb + 2 * (t0 + 2 * RING - 1);
                    }
                    pre = fetch_ids(d, row, page);
                }
                const int i = 2 * (t0 + r);
                if (i < n_live) {
                    const int pa = cur.pb + i;                                  // absolute page of the pair's first half
                    const int va = pa == cur.n_pages - 1 ? last_valid : T;
                    const int vb = i + 1 < n_live ? (pa + 1 == cur.n_pages - 1 ? last_valid : T) : 0;
                    process_pair<D, DT>(st, ring[r], qf, d.scale_log2, va, vb, G);
                    prio_done += 2;
                }
            }
        }

        // --- the piece is done: finish the segment or park a partial
        float *out_row = d.out + ((size_t)cur.seq * d.Hq + cur.kvh * g + n) * D;
        if (cur.n_pages == 0) {                  // empty context: the row is defined as zero
            if (cur.pb == 0 && col_live) {
#pragma unroll
                for (int jt = 0; jt < TL::NV; ++jt)
                    *reinterpret_cast<f32x4 *>(out_row + 16 * jt + 4 * G) = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        } else {
            float l = st.l;
            l += __shfl_xor(l, 16);
            l += __shfl_xor(l, 32);
            const uint32_t k0 = cut.index(cur.g0), k1 = cut.index(cur.g0 + (uint32_t)cur.n_pages - 1);
            if (k0 == k1) {                      // the whole segment was ours
                if (col_live) {
                    const float inv = 1.0f / l;
#pragma unroll
                    for (int jt = 0; jt < TL::NV; ++jt)
                        *reinterpret_cast<f32x4 *>(out_row + 16 * jt + 4 * G) = st.acc[jt] * inv;
                }
            } else {
                float *w = cur.pb == 0 ? ws_b : ws_a;
                if (col_live) {
#pragma unroll
                    for (int jt = 0; jt < TL::NV; ++jt)
                        *reinterpret_cast<f32x4 *>(w + n * D + 16 * jt + 4 * G) = st.acc[jt];
                    if (G == 0) {
                        w[g * D + n] = st.m;
                        w[g * D + g + n] = l;
                    }
                }
                // The partials and the arrival counters live in uncached device memory, so every
                // access goes to memory itself and is visible to all XCDs without flushing an L2.
                // Order is all that is left to enforce: the partial must have landed before the
                // counter moves.  The count itself is looked at only when the share is finished.
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                if (CACHED) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                uint32_t arrived = 0;
                if (lane == 0) arrived = atomicAdd(d.cnt + (size_t)cur.seq * Hkv + cur.kvh, 1u);
                Pending &pd = cur.pb == 0 ? pend_b : pend_a;
                pd.valid = 1;
                pd.seq = cur.seq;
                pd.kvh = cur.kvh;
                pd.k0 = k0;
                pd.k1 = k1;
                pd.arrived = arrived;
            }
        }
        cur = nxt;
#pragma unroll
        for (int j = 0; j < TL::NK; ++j) qf[j] = qn[j];
    }

    // --- merges this wave owes: it arrived last at a segment shared with other waves
    if (w.stat && lane == 0) {          // tuning launches only: when did this XCD's waves finish streaming
        const unsigned xcd = blockIdx.x & 7u;
        atomicAdd(reinterpret_cast<unsigned long long *>(w.stat) + 2 * xcd, (unsigned long long)(wall_clock64() - t_begin));
        atomicAdd(reinterpret_cast<unsigned long long *>(w.stat) + 2 * xcd + 1, 1ull);
    }
    asm volatile("" ::: "memory");
    if (pend_a.valid) {
        const uint32_t arrived = (uint32_t)__builtin_amdgcn_readfirstlane((int)pend_a.arrived);
        if (arrived == pend_a.k1 - pend_a.k0) {
            // ready for the next launch (cached counters are cleared by the host before every launch instead)
            if (!CACHED && lane == 0) d.cnt[(size_t)pend_a.seq * Hkv + pend_a.kvh] = 0u;
            if (CACHED) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            merge_segment<D>(d, pend_a, lane, s_m, s_l);
        }
    }
    if (pend_b.valid) {
        const uint32_t arrived = (uint32_t)__builtin_amdgcn_readfirstlane((int)pend_b.arrived);
        if (arrived == pend_b.k1 - pend_b.k0) {
            if (!CACHED && lane == 0) d.cnt[(size_t)pend_b.seq * Hkv + pend_b.kvh] = 0u;
            if (CACHED) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            merge_segment<D>(d, pend_b, lane, s_m, s_l);
        }
    }
    if (bad && lane == 0) atomicOr(d.err, 1u);
}

__global__ __launch_bounds__(64, 2) void k_attention(const AttnGroup grp) {
    __shared__ float s_m[MAX_PIECES * 16], s_l[MAX_PIECES * 16];
    const int gi = blockIdx.x;
    int mi = 0;
    for (int i = 1; i < grp.n; ++i)
        if (gi >= grp.m[i].item_begin) mi = i;
    const AttnDesc &d = grp.m[mi];
    const int item = gi - d.item_begin;
    if (d.dtype == PKV_BF16) {
        if (d.D == 128) attn_wave<128, PKV_BF16>(d, grp.tune, item, s_m, s_l);
        else attn_wave<64, PKV_BF16>(d, grp.tune, item, s_m, s_l);
    } else {
        if (d.D == 128) attn_wave<128, PKV_E4M3>(d, grp.tune, item, s_m, s_l);
        else attn_wave<64, PKV_E4M3>(d, grp.tune, item, s_m, s_l);
    }
}

__global__ __launch_bounds__(64, 1) void k_attention_deep(const AttnGroup grp) {
    __shared__ float s_m[MAX_PIECES * 16], s_l[MAX_PIECES * 16];
    const int gi = blockIdx.x;
    int mi = 0;
    for (int i = 1; i < grp.n; ++i)
        if (gi >= grp.m[i].item_begin) mi = i;
    const AttnDesc &d = grp.m[mi];
    const int item = gi - d.item_begin;
    if (d.dtype == PKV_BF16) {
        if (d.D == 128) attn_wave<128, PKV_BF16, FLIGHT_KIB_1WAVE>(d, grp.tune, item, s_m, s_l);
        else attn_wave<64, PKV_BF16, FLIGHT_KIB_1WAVE>(d, grp.tune, item, s_m, s_l);
    } else {
        if (d.D == 128) attn_wave<128, PKV_E4M3, FLIGHT_KIB_1WAVE>(d, grp.tune, item, s_m, s_l);
        else attn_wave<64, PKV_E4M3, FLIGHT_KIB_1WAVE>(d, grp.tune, item, s_m, s_l);
    }
}

// The decode kernel for callers that may not allocate: the same code with its split-K partials and
// arrival counters in the library's file-scope scratch array (ordinary cached memory).
__global__ __launch_bounds__(64, 2) void k_attention_static(const AttnGroup grp) {
    __shared__ float s_m[MAX_PIECES * 16], s_l[MAX_PIECES * 16];
    const AttnDesc &d = grp.m[0];
    const int item = blockIdx.x;
    if (d.dtype == PKV_BF16) {
        if (d.D == 128) attn_wave<128, PKV_BF16, FLIGHT_KIB_2WAVES, true>(d, grp.tune, item, s_m, s_l);
        else attn_wave<64, PKV_BF16, FLIGHT_KIB_2WAVES, true>(d, grp.tune, item, s_m, s_l);
    } else {
        if (d.D == 128) attn_wave<128, PKV_E4M3, FLIGHT_KIB_2WAVES, true>(d, grp.tune, item, s_m, s_l);
        else attn_wave<64, PKV_E4M3, FLIGHT_KIB_2WAVES, true>(d, grp.tune, item, s_m, s_l);
    }
}

// Small launches: one work-group of SMALL_WAVES waves per part of a (sequence, kv head).
//
// Such a launch is bound by the number of dependent memory trips, not by bytes: the kernels above find their share from
// all context lengths, then its block ids, then the pages, and hand every cut segment over through memory (partial,
// arrival, partials of the others: three more trips of about 1 us).  Here the block index alone names the segment and
// the part, so block ids, context length and queries are asked for together and the pages behind them; the waves of
// the work-group take the part's page pairs in turn and join their sums through LDS.  Only segments longer than
// `part_pages` pages come in several parts, whose partials the last to arrive joins.  The host sizes the parts
// (plan_small); a context that has outgrown them (a launch replayed from a graph) gets longer parts here.
//
// A wave alone on its SIMD issues an instruction every four or five cycles, so once its pages are there it is bound by how many a
// page pair costs: with the addresses of both pages worked out by scalar instructions and masks in every pair some 410 (bf16) and
// 510 (e4m3, 128-wide heads), so 308 and 328 (cold branches included).  Us a launch, caches cold, with parts as they were and are
// chosen: 1 x 9735 tokens of 4/1/128 bf16 12.4, 11.8; 3 x 1717 of 2/1/128 e4m3 9.2, 8.1; 7 x 573 of 16/8/64 e4m3 7.3, 6.1; rows in one part
// 0.85 to 0.95 of the time before.  Eight waves a work-group instead of four take longer everywhere (2 x 767 of 16/4/128 9.2, 9.9).
constexpr int SMALL_WAVES = 4;

// Weight of a wave's sums with maximum m beside a joint maximum of M.  A wave that has seen nothing but logits of -inf has
// m = -inf and sums of zero (four waves each begin somewhere in the row, so that is not only the row's own start); so may
// have all waves of a part.
__device__ __forceinline__ float merge_weight(float m, float M) { return m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M); }

template <int D, int DT>
__device__ __forceinline__ void attn_part(const AttnDesc &d, int wg, float *s_acc, float *s_m, float *s_l, uint32_t *s_arrived) {
    using TL = Tile<D, DT>;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int G = lane >> 4, n = lane & 15, g = d.g;
    // Work-groups are dealt to the eight XCDs in turn.  With a multiple of eight kv heads these come fastest (each XCD
    // keeps its heads), then the parts of the row, then rows: eight lognormal rows of 2048 tokens take 22 us a launch, 27
    // with the parts slowest.  Otherwise parts come slowest, so that the first parts, which every row has, fall on all
    // XCDs (100 rows of 2 kv heads, parts before rows: 40 us, twice the ordinary form).
    int seq, kvh, part;
    if ((d.Hkv & 7) == 0) {
        const int per_row = d.Hkv * d.parts, rest = wg % per_row;
        seq = wg / per_row;
        part = rest / d.Hkv;
        kvh = rest - part * d.Hkv;
    } else {
        const int n_segs = d.batch * d.Hkv, at = wg % n_segs;
        part = wg / n_segs;
        seq = at / d.Hkv;
        kvh = at - seq * d.Hkv;
    }
    const int seg = seq * d.Hkv + kvh;
    const int32_t *row = d.table + (size_t)seq * d.row_stride;
    bf16x8 qf[TL::NK];
    load_q<D>(qf, d, seq, kvh, lane);
    // This wave's pairs: pages page0 + STEP k and the one behind it, k = 0, 1, ...  The ids of the first come by themselves, those of
    // the next 32 in one read, for any row; lane i works out where page i & 1 of pair 1 + (i >> 1) is, if there is a second pair.
    // All are asked for with the context length and the queries.
    constexpr int STEP = 2 * SMALL_WAVES;
    const int ahead = STEP * (lane >> 1) + (lane & 1);
    auto id_of = [&](int page) __attribute__((always_inline)) { return (uint32_t)row[page < d.row_stride ? page : d.row_stride - 1]; };
    int page0 = part * d.part_pages + 2 * w;
    PairIds ids = fetch_ids(d, row, page0);
    uint32_t id = id_of(page0 + STEP + ahead);
    const int L = __builtin_amdgcn_readfirstlane(ctx_clamped(d, seq));
    const int n_pages = (L + T - 1) / T;
    int size = d.part_pages;
    if (n_pages > d.parts * size) {                       // longer than the host knew
        size = (n_pages + d.parts - 1) / d.parts;
        size = (size + STEP - 1) / STEP * STEP;
        page0 = part * size + 2 * w;
        ids = fetch_ids(d, row, page0);
        id = id_of(page0 + STEP + ahead);
    }
    const int n_parts = n_pages > size ? (n_pages + size - 1) / size : 1;
    if (part >= n_parts) return;
    const int pe = (part + 1) * size < n_pages ? (part + 1) * size : n_pages;
    const int last_valid = L - (n_pages - 1) * T;
    State<D, DT> st;
#pragma unroll
    for (int jt = 0; jt < TL::NV; ++jt) st.acc[jt] = f32x4{0.f, 0.f, 0.f, 0.f};
    st.m = -INFINITY;
    st.l = 0.f;

    // where the tiles of this lane's page are, in how many bytes (none: the page is beyond the part, or its id outside the
    // pool, and is never read), and its scales
    bool bad = false;
    uint32_t addr_lo = 0, addr_hi = 0, records = 0;
    float page_sk = 0.f, page_sv = 0.f;
    auto locate = [&](int page, uint32_t id) __attribute__((always_inline)) {
        const bool in_pool = id < d.max_block_id, live = page < pe;
        bad |= live && !in_pool;
        const uint8_t *blk = block_ptr(d, id);
        if (DT == PKV_E4M3) {
            const float *hdr = reinterpret_cast<const float *>(live && in_pool ? blk : reinterpret_cast<const uint8_t *>(d.safe));
            page_sk = hdr[kvh];
            page_sv = hdr[d.Hkv + kvh];
            blk += PKV_FP8_HEADER;
        }
        blk += (size_t)kvh * 2 * TL::TILE_BYTES;
        addr_lo = (uint32_t)(uintptr_t)blk;
        addr_hi = (uint32_t)((uintptr_t)blk >> 32);
        records = live && in_pool ? 2 * TL::TILE_BYTES : 0;
    };
    int window = 1;                                       // the lanes' pages are those of pairs window .. window + 31
    auto lane_of = [&](uint32_t x, int at) __attribute__((always_inline)) { return (uint32_t)__builtin_amdgcn_readlane((int)x, at); };
    auto tiles = [&](int k, int half) __attribute__((always_inline)) {
        const int at = 2 * (k - window) + half;
        return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<uint8_t *>(lane_of(addr_lo, at) | (uint64_t)lane_of(addr_hi, at) << 32), 0,
                                                 (int)lane_of(records, at), 0x00020000);
    };
    auto first_tiles = [&](uint32_t id, bool live, float &sk, float &sv) __attribute__((always_inline)) {
        const bool in_pool = id < d.max_block_id;
        bad |= live && !in_pool;
        live = live && in_pool;
        const uint8_t *blk = block_ptr(d, id);
        if (DT == PKV_E4M3) {
            const float *hdr = reinterpret_cast<const float *>(live ? blk : reinterpret_cast<const uint8_t *>(d.safe));
            sk = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(PKV_CONST(float, hdr)[kvh])));
            sv = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(PKV_CONST(float, hdr)[d.Hkv + kvh])));
            blk += PKV_FP8_HEADER;
        }
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(blk + (size_t)kvh * 2 * TL::TILE_BYTES), 0, live ? 2 * TL::TILE_BYTES : 0, 0x00020000);
    };
    const int voff = lane * 16;
    auto load = [&](u32x4 *r, __amdgpu_buffer_rsrc_t rsrc, int at) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TL::NL; ++j) r[j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voff + j * 1024, at, 2 /* non-temporal */);
        asm volatile("" ::: "memory");                    // in this order everywhere: loads in flight are counted
    };
    auto load_pages = [&](PairRegs<D, DT> &r, __amdgpu_buffer_rsrc_t a, __amdgpu_buffer_rsrc_t b) __attribute__((always_inline)) {
        load(r.a.k, a, 0);
        load(r.a.v, a, TL::TILE_BYTES);
        load(r.b.k, b, 0);
        load(r.b.v, b, TL::TILE_BYTES);
    };
    auto scales = [&](PairRegs<D, DT> &r, int k) __attribute__((always_inline)) {
        if (DT != PKV_E4M3) return;
        const int at = 2 * (k - window);
        r.a.sk = __uint_as_float(lane_of(__float_as_uint(page_sk), at));
        r.a.sv = __uint_as_float(lane_of(__float_as_uint(page_sv), at));
        r.b.sk = __uint_as_float(lane_of(__float_as_uint(page_sk), at + 1));
        r.b.sv = __uint_as_float(lane_of(__float_as_uint(page_sv), at + 1));
    };
    // Pair k; `more`: pair k + 1 is asked for ahead of it.  (Asked for earlier, K of pair k + 2 behind the scores and V behind the
    // products of pair k, launches took 2 to 10 % longer: 8 lognormal rows of 2048 tokens of 32/8/128 bf16 19.0, 20.0 us, 16 of 4717
    // of 10/2/128 25.3, 27.2, 30 of 366 of 40/8/128 7.7, 8.5.  Whole pages one after the other, K and V, cost 1 to 3 % less than K of
    // both and then V.)
    auto step = [&](PairRegs<D, DT> &r, PairRegs<D, DT> &o, int k, bool more) __attribute__((always_inline)) {
        if (more) {
            load_pages(o, tiles(k + 1, 0), tiles(k + 1, 1));
            scales(o, k + 1);
        }
        const int p = page0 + STEP * k;
        const int valid_a = p == n_pages - 1 ? last_valid : T;
        const int valid_b = p + 1 < pe ? (p + 1 == n_pages - 1 ? last_valid : T) : 0;
        const bool tail = valid_a < T || valid_b < T;
        const float sca = DT == PKV_E4M3 ? d.scale_log2 * r.a.sk : d.scale_log2, scb = DT == PKV_E4M3 ? d.scale_log2 * r.b.sk : d.scale_log2;
        const f32x4 sa = qk_page<D, DT>(r.a, qf), sb = qk_page<D, DT>(r.b, qf);
        float s[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s[i] = sa[i] * sca;
            s[4 + i] = sb[i] * scb;
        }
        // only a row's last pair holds tokens past its context: a branch of its own, not selects in every step
        if (tail) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (4 * G + i >= valid_a) s[i] = -INFINITY;
                if (4 * G + i >= valid_b) s[4 + i] = -INFINITY;
            }
            blank_v<D, DT>(r.a.v, valid_a - 4 * G);
            blank_v<D, DT>(r.b.v, valid_b - 4 * G);
        }
        bf16x8 phv, plv;
        softmax_pair<D, DT>(st, s, r.a.sv, r.b.sv, phv, plv);
#pragma unroll
        for (int jt = 0; jt < TL::NV; ++jt) {
            const u32x2 va = v_half<D, DT>(r.a, jt), vb = v_half<D, DT>(r.b, jt);
            const bf16x8 av = as_bf16x8(mk4(va.x, va.y, vb.x, vb.y));
            st.acc[jt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, phv, st.acc[jt], 0, 0, 0);
            st.acc[jt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, plv, st.acc[jt], 0, 0, 0);
        }
    };
    const int n_pairs = page0 < pe ? (pe - page0 + STEP - 1) / STEP : 0;
    if (n_pairs > 0) {
        PairRegs<D, DT> ring[2];
        const __amdgpu_buffer_rsrc_t a = first_tiles(ids.a, true, ring[0].a.sk, ring[0].a.sv);
        const __amdgpu_buffer_rsrc_t b = first_tiles(ids.b, page0 + 1 < pe, ring[0].b.sk, ring[0].b.sv);
        load_pages(ring[0], a, b);
        // (The loads in flight are counted along every way the compiler sees: the loop is entered from here only, two whole steps
        // a turn with no way out between them, the odd step by itself.)
        int k = 0;
        if (n_pairs > 1) {
            locate(page0 + STEP + ahead, id);
            do {
                if (k + 2 - window >= 32) {
                    window = k + 1;
                    locate(page0 + STEP * window + ahead, id_of(page0 + STEP * window + ahead));
                }
                step(ring[0], ring[1], k, true);
                step(ring[1], ring[0], k + 1, true);
                k += 2;
            } while (k + 2 <= n_pairs);
        }
        if (k < n_pairs) step(ring[0], ring[1], k, false);
    }
    float l = st.l;
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (n < g) {
        float *a = s_acc + (w * g + n) * D;
#pragma unroll
        for (int jt = 0; jt < TL::NV; ++jt) *reinterpret_cast<f32x4 *>(a + 16 * jt + 4 * G) = st.acc[jt];
        if (G == 0) {
            s_m[w * 16 + n] = st.m;
            s_l[w * 16 + n] = l;
        }
    }
    if (__any(bad) && lane == 0) atomicOr(d.err, 1u);
    __syncthreads();
    // the sums of the work-group: lane by lane four output elements of one head
    const int quads = g * (D / 4), pf = partial_floats(g, D);
    const bool whole = n_parts == 1;
    float *mine = d.ws + (size_t)(seg * d.parts + part) * pf;
    for (int i = threadIdx.x; i < quads; i += 64 * SMALL_WAVES) {
        const int hn = i / (D / 4), x = i - hn * (D / 4);
        float M = s_m[hn];
#pragma unroll
        for (int v = 1; v < SMALL_WAVES; ++v) M = fmaxf(M, s_m[v * 16 + hn]);
        float den = 0.f;
        f32x4 num = {0.f, 0.f, 0.f, 0.f};
        if (n_pages > 0) {                                // an empty context: the row is defined as zero
#pragma unroll
            for (int v = 0; v < SMALL_WAVES; ++v) {
                const float f = merge_weight(s_m[v * 16 + hn], M);
                den += f * s_l[v * 16 + hn];
                num += f * *reinterpret_cast<const f32x4 *>(s_acc + (v * g + hn) * D + 4 * x);
            }
        }
        if (whole) {
            *reinterpret_cast<f32x4 *>(d.out + ((size_t)seq * d.Hq + kvh * g + hn) * D + 4 * x) = n_pages > 0 ? num * (1.0f / den) : num;
        } else {
            *reinterpret_cast<f32x4 *>(mine + hn * D + 4 * x) = num;
            if (x == 0) {
                mine[g * D + hn] = M;
                mine[g * D + g + hn] = den;
            }
        }
    }
    if (whole) return;
    // Hand-over as in attn_wave: partials and counters are in uncached memory, so the order of a wave's own accesses is
    // all there is to enforce; every wave's stores have landed when the counter moves.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) *s_arrived = atomicAdd(d.cnt + seg, 1u);
    __syncthreads();
    if (*s_arrived != (uint32_t)(n_parts - 1)) return;
    if (threadIdx.x == 0) d.cnt[seg] = 0u;                // ready for the next launch
    const float *base = d.ws + (size_t)seg * d.parts * pf;
    // All maxima and sums travel together with the sums of the first eight parts: one trip to uncached memory instead of two.
    // Us a launch, rows in many parts: 1 x 32000 tokens of 8/1/128 17.5 -> 15.4, 1 x 12000 of 64/8/128 14.6 -> 13.6, 3 x 6000 of
    // 28/4/128 12.6 -> 12.0, 2 x 9000 of 32/8/128 e4m3 15.7 -> 15.2; with its append 8 x 2048 of 32/8/128 16.8 -> 16.4; rows in one
    // part (4 x 128 of 8/2/64) the same.  (The read is there twice, 7 KB more over all variants.)
    auto part_sums = [&](f32x4 *v, int c0, int hn, int x) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 8; ++u)
            v[u] = *reinterpret_cast<const f32x4 *>(base + (size_t)(c0 + u < n_parts ? c0 + u : n_parts - 1) * pf + hn * D + 4 * x);
    };
    f32x4 first[8];
    {
        const int i = (int)threadIdx.x < quads ? (int)threadIdx.x : quads - 1, hn = i / (D / 4);
        part_sums(first, 0, hn, i - hn * (D / 4));
    }
    for (int i = threadIdx.x; i < n_parts * g; i += 64 * SMALL_WAVES) {
        const int c = i / g, hn = i - c * g;
        s_acc[i] = base[(size_t)c * pf + g * D + hn];
        s_acc[MAX_PIECES * 16 + i] = base[(size_t)c * pf + g * D + g + hn];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < quads; i += 64 * SMALL_WAVES) {
        const int hn = i / (D / 4), x = i - hn * (D / 4);
        float M = -INFINITY, den = 0.f;
        f32x4 num = {0.f, 0.f, 0.f, 0.f};
        for (int c = 0; c < n_parts; ++c) M = fmaxf(M, s_acc[c * g + hn]);
        for (int c0 = 0; c0 < n_parts; c0 += 8) {
            if (c0 > 0 || i >= 64 * SMALL_WAVES) part_sums(first, c0, hn, x);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (c0 + u < n_parts) {
                    const float f = __builtin_amdgcn_exp2f(s_acc[(c0 + u) * g + hn] - M);
                    den += f * s_acc[MAX_PIECES * 16 + (c0 + u) * g + hn];
                    num += f * first[u];
                }
        }
        *reinterpret_cast<f32x4 *>(d.out + ((size_t)seq * d.Hq + kvh * g + hn) * D + 4 * x) = num * (1.0f / den);
    }
}

// One model's launch carries 200 bytes of arguments instead of the group's 3.4 KB (a decode step of four layers, eight
// launches: 98.7 -> 97.2 us).
struct AttnOne {
    AttnDesc m[1];
    static constexpr int n = 1;
};

template <typename GROUP>
__global__ __launch_bounds__(64 * SMALL_WAVES, 2) void k_attention_small(const GROUP grp) {
    __shared__ __align__(16) float s_acc[SMALL_WAVES * 16 * 128];
    __shared__ float s_m[SMALL_WAVES * 16], s_l[SMALL_WAVES * 16];
    __shared__ uint32_t s_arrived;
    static_assert(2 * MAX_PIECES * 16 <= SMALL_WAVES * 16 * 128, "maxima and sums of all parts fit where the accumulators were");
    const int gi = blockIdx.x;
    int mi = 0;
    for (int i = 1; i < grp.n; ++i)
        if (gi >= grp.m[i].item_begin) mi = i;
    const AttnDesc &d = grp.m[mi];
    const int wg = gi - d.item_begin;
    if (d.dtype == PKV_BF16) {
        if (d.D == 128) attn_part<128, PKV_BF16>(d, wg, s_acc, s_m, s_l, &s_arrived);
        else attn_part<64, PKV_BF16>(d, wg, s_acc, s_m, s_l, &s_arrived);
    } else {
        if (d.D == 128) attn_part<128, PKV_E4M3>(d, wg, s_acc, s_m, s_l, &s_arrived);
        else attn_part<64, PKV_E4M3>(d, wg, s_acc, s_m, s_l, &s_arrived);
    }
}

__global__ void k_clear_words(uint32_t *p, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = 0u;
}

// Read ceilings for comparison.  granule == 0: plain streaming read of the buffer,
// 16 bytes per lane.  granule > 0 (a power-of-two number of KiB): each wave reads
// whole granules of that size picked in a scrambled order, which is the access pattern
// of paged KV (contiguous inside a tile, scattered between tiles) without any math.
__global__ __launch_bounds__(256) void k_stream_read(const u32x4 *src, size_t n16, uint32_t granule16, uint32_t *sink) {
    u32x4 acc = {0, 0, 0, 0};
    if (granule16 == 0) {
        const size_t stride = (size_t)gridDim.x * blockDim.x;
        size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
        for (; i + 3 * stride < n16; i += 4 * stride) {
            const u32x4 a = __builtin_nontemporal_load(src + i), b = __builtin_nontemporal_load(src + i + stride);
            const u32x4 c = __builtin_nontemporal_load(src + i + 2 * stride),
                        e = __builtin_nontemporal_load(src + i + 3 * stride);
            acc ^= a ^ b ^ c ^ e;
        }
        for (; i < n16; i += stride) acc ^= __builtin_nontemporal_load(src + i);
    } else {
        const size_t n_gran = n16 / granule16;               // a power of two (checked by the host)
        const size_t waves = (size_t)gridDim.x * (blockDim.x / 64);
        const int lane = threadIdx.x & 63;
        for (size_t w = blockIdx.x * (size_t)(blockDim.x / 64) + (threadIdx.x >> 6); w < n_gran; w += waves) {
            const size_t gidx = (w * 0x9E3779B1ull + 12345ull) & (n_gran - 1);   // odd multiplier: a permutation
            const u32x4 *g = src + gidx * granule16 + lane;
            if (granule16 >= 8 * 64) {
                for (uint32_t k = 0; k < granule16; k += 8 * 64) {
#pragma unroll
                    for (int u = 0; u < 8; ++u) acc ^= __builtin_nontemporal_load(g + k + u * 64);
                }
            } else {
                for (uint32_t k = 0; k < granule16; k += 64) acc ^= __builtin_nontemporal_load(g + k);
            }
        }
    }
    if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9e3779b9u) *sink = 1;   // keeps the loads alive
}

}  // namespace

hipError_t pkv_launch_attention(const AttnGroup &grp, AttnForm form, hipStream_t s, hipEvent_t *ev) {
    int items = 0;
    for (int i = 0; i < grp.n; ++i) items += form == AttnForm::small ? grp.m[i].batch * grp.m[i].Hkv * grp.m[i].parts : grp.m[i].n_items;
    if (items == 0) return hipSuccess;
    hipError_t e;
    if (ev && (e = hipEventRecord(ev[0], s)) != hipSuccess) return e;
    if (form == AttnForm::deep) hipLaunchKernelGGL(k_attention_deep, dim3(items), dim3(64), 0, s, grp);
    else if (form == AttnForm::small && grp.n == 1) {
        AttnOne one;
        one.m[0] = grp.m[0];
        hipLaunchKernelGGL(k_attention_small<AttnOne>, dim3(items), dim3(64 * SMALL_WAVES), 0, s, one);
    } else if (form == AttnForm::small) hipLaunchKernelGGL(k_attention_small<AttnGroup>, dim3(items), dim3(64 * SMALL_WAVES), 0, s, grp);
    else hipLaunchKernelGGL(k_attention, dim3(items), dim3(64), 0, s, grp);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (ev && (e = hipEventRecord(ev[1], s)) != hipSuccess) return e;
    return hipSuccess;
}

// ---- scratch of the entry point that allocates nothing ------------------------------------------
// Arrival counters first, split-K partials behind them.  Every GPU holds its own copy of the array
// at its own address; in host code the array's name is only a handle for hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[PKV_STATIC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
void *g_scratch_ptr[kMaxDevices];     // per device: the address of its copy of `scratch`, once resolved
}  // namespace

// Address of the current device's copy of the scratch array (resolved once per device).
hipError_t pkv_static_scratch(void **ptr) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

// One model, the ordinary kernel form; d.ws and d.cnt point into the scratch array.  The counters the
// launch uses are cleared first (by a kernel: a caller may be capturing the stream into a graph).
hipError_t pkv_launch_attention_static(const AttnGroup &grp, uint32_t *cnt, size_t n_cnt, hipStream_t s) {
    if (grp.n != 1 || grp.m[0].n_items <= 0) return hipErrorInvalidValue;
    const unsigned blocks = (unsigned)((n_cnt + 255) / 256);
    hipLaunchKernelGGL(k_clear_words, dim3(blocks < 64 ? (blocks ? blocks : 1) : 64), dim3(256), 0, s, cnt, n_cnt);
    hipLaunchKernelGGL(k_attention_static, dim3(grp.m[0].n_items), dim3(64), 0, s, grp);
    return hipGetLastError();
}

hipError_t pkv_launch_stream_read(const void *src, size_t bytes, size_t granule_bytes, uint32_t *sink, hipStream_t s) {
    hipLaunchKernelGGL(k_stream_read, dim3(256 * 16), dim3(256), 0, s, (const u32x4 *)src, bytes / 16,
                       (uint32_t)(granule_bytes / 16), sink);
    return hipGetLastError();
}
