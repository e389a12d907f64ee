// Chunked prefill over the shared pool (gfx950 / CDNA4): causal attention of a group of consecutive
// query tokens against the paged cache (paper Sec. 5.2).
//
// One work-group of four waves per (group, kv head).  Every wave owns a tile of 32 MFMA columns (query
// tokens x the g heads of the kv head) and walks the context a page pair (32 tokens) at a time:
//   scores   S[token][column] = K . q^T          D / 16 products 32x32x16, K as the row operand
//   output   O^T[d][column] += V^T . P           2 * D / 32 products per half of P (hi, lo)
// The accumulator layout of the first is the column-operand layout of the second once the eight tokens a
// lane holds of a page are taken as the eight contraction slots of its lane half, so probabilities never
// change lanes.  K and V tiles travel from the pool into LDS in the byte order they have in the block
// (kv_layout.h), one tile of the pair per wave.
//
// What bounds it: power, then the latency of a step.  On bf16 caches with 128-wide heads a wave's step is 24
// products (768 matrix cycles, a third of them the low half of the probabilities) and some 105 other vector
// instructions (8 more with a maximum per step instead of the sum as the sign that the reference point has to move:
// 228 -> 225 us a pass with its append, all shapes 0.7 to 1.3 % faster); by the counters of a launch a step takes a
// wave 2250 cycles, 1000 of them waiting, and the matrix units are busy 58 % of the launch at 1.85 GHz; with all
// operands zero the same kernel runs 25 % faster, and a plain 8192^3 matrix product loses as much to random data.  Why
// this shape: 32x32x16 products read half as many operand registers and LDS bytes per flop as 16x16x32, need one lane
// exchange instead of two per maximum (and that only when the reference point moves), and fill 32 columns better for
// odd g.  The step is software-pipelined by one pair: scores of pair p + 1 and the V reads of pair p are issued before
// the output products of pair p, between which the softmax of pair p + 1 runs.  The waves meet once in two pairs, four on
// e4m3 caches (every pair: 2 % slower).  8 sequences x (2048 cached + 512 new) of 32/8/128, a maximum in every step, arguments read where they are
// used and no priority levels, and with these mended: bf16 221.9, 213.3 us, e4m3 180.6, 171.8; of 32/8/64: bf16 140.1, 137.1, e4m3
// 131.2, 127.2.
#include "mfma_util.h"

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int PF_WAVES = PKV_PREFILL_WAVES;
constexpr int PF_COLS = 32;     // MFMA columns per wave
static_assert(PF_WAVES * PF_COLS == PKV_PREFILL_COLS, "host and kernel must agree on the group size");

// Where the reference point of the exponentials starts: finite, so that a column that has seen no token yet needs no
// special case (its probabilities are exp2(-inf) = 0), and the lowest number there is, so that the first visible token's
// score, whatever it is, lies above it and replaces it.
constexpr float PF_M0 = -3.402823466e+38f;
// Sum of a lane's sixteen probabilities of a page pair beyond which the reference point moves.
constexpr float kSumBar = 256.f;
// Scores (log2 domain) beyond this are rounded to more than one.
constexpr float PF_FAR = 0x1p24f;

template <int D, int DT>
struct PfTile {
    static constexpr int E = DT == PKV_BF16 ? 2 : 1;
    static constexpr int BYTES = PKV_T * D * E;            // one K or V tile
    static constexpr int NL = BYTES / 1024;                // 1 KiB requests per tile
    static constexpr int NU = BYTES / 512;                 // 16-byte LDS reads per lane for the K operands of a pair
    static constexpr int NK = D / 16;                      // score products per pair
    static constexpr int ND = D / 32;                      // tiles of 32 output elements
};

// NL x 1 KiB from the pool straight into LDS: lane l's 16 bytes at src + 1024 j + 16 l land at dst + 1024 j + 16 l.
// Written as assembly so that the compiler does not drain all requests in flight before every LDS read;
// the waits are counted by hand (s_waitcnt vmcnt).  src and dst are wave-uniform.
template <int NL>
__device__ __forceinline__ void lds_fill(const uint8_t *src, uint32_t dst, uint32_t lane16) {
    if (NL == 1)
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(lane16), "s"(src), "s"(dst) : "memory", "m0");
    else if (NL == 2)
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1\n\tglobal_load_lds_dwordx4 %0, %1 offset:1024" ::"v"(lane16),
                     "s"(src), "s"(dst)
                     : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1\n\tglobal_load_lds_dwordx4 %0, %1 offset:1024\n\t"
                     "global_load_lds_dwordx4 %0, %1 offset:2048\n\tglobal_load_lds_dwordx4 %0, %1 offset:3072" ::"v"(lane16),
                     "s"(src), "s"(dst)
                     : "memory", "m0");
    static_assert(NL == 1 || NL == 2 || NL == 4, "tile sizes of 1, 2 or 4 KiB");
}

template <int NL>
__device__ __forceinline__ void wait_requests(int ahead) {      // all but the `ahead` most recent requests have landed
    if (ahead >= 4) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * NL) : "memory");
    else if (ahead == 3) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(3 * NL) : "memory");
    else if (ahead == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NL) : "memory");
    else if (ahead == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// One unit of the launch: the query tokens of a group (rows q0 .. q0 + ntok - 1 of the packed q and out, followed by
// `back` more of the sequence's chunk) and which of `parts` parts of the context it walks.
struct GroupInfo {
    int seq, q0, ntok, back, part, parts;
};

template <int SEQS>
__device__ __forceinline__ GroupInfo group_info(const AttnDesc &d, const PlanOf<SEQS> &plan, const PlanLanes<SEQS> &lanes, int unit) {
    const PlanUnit pu = lanes.find(plan, (uint32_t)unit);
    const int size = PF_WAVES * (d.cols / d.g), groups = (pu.rows + size - 1) / size;
    const int rank = pu.parts > 1 ? pu.unit / pu.parts : pu.unit;
    const int t0 = (groups - 1 - rank) * size;
    GroupInfo g;
    g.seq = pu.seq;
    g.q0 = pu.row + t0;
    g.ntok = pu.rows - t0 < size ? pu.rows - t0 : size;
    g.back = pu.rows - t0 - g.ntok;
    g.parts = pu.parts;
    g.part = pu.unit - rank * pu.parts;
    return g;
}

// The waves meet once in MEET pairs, and no wave runs further ahead than that.  An e4m3 cache leaves room in LDS for twice the
// slots that bf16 has (two work-groups a CU, three with 64-wide heads).  Us a pass, met in two and in four pairs: 8 x (2048 + 512)
// tokens of 32/8/128 179.3, 176.0; 8192 + 256 58.4, 56.5; ragged prompts 76.2, 75.1.  (Short walks: meets_often_in below.)
template <int D, int DT, int SEQS, int MEET>
__global__ __launch_bounds__(64 * PF_WAVES, 2) void k_prefill(const AttnDesc d, const PlanOf<SEQS> plan) {
    using TL = PfTile<D, DT>;
    constexpr int SLOT = 2 * TL::BYTES;                    // the K (or V) tiles of a pair
    constexpr int PF_SLOTS = 2 * MEET;                     // page pairs per ring (K and V have a ring each)
    __shared__ __align__(16) uint8_t ring[2 * PF_SLOTS * SLOT];   // K slots, then V slots
    const PlanLanes<SEQS> lanes(plan);
    ask_arguments(d, plan.n_seqs, plan.seq0);
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int h = lane >> 5, n = lane & 31, c16 = lane & 15, hi16 = (lane >> 4) & 1;
    const int group = blockIdx.x / d.Hkv, kvh = blockIdx.x - group * d.Hkv;

    // groups of a sequence come longest context first; a group of few query tokens in front of a long context comes
    // as several work-groups, each with a part of the context, that leave partial results for k_prefill_merge
    const GroupInfo gi = group_info(d, plan, lanes, group);
    const int seq = gi.seq, q0 = gi.q0, ntok = gi.ntok, split = gi.part, n_split = gi.parts;
    const int tile_tok = d.cols / d.g;                     // query tokens per wave
    const int tok = n / d.g, head = n - tok * d.g;         // this lane's column
    // the block ids of the first 64 pairs are asked for along with the context length, not behind it
    const int32_t *row = d.table + (size_t)seq * d.row_stride;
    auto table_id = [&](int page) __attribute__((always_inline)) { return (uint32_t)row[page < d.row_stride ? page : d.row_stride - 1]; };
    const uint32_t first_id = table_id(2 * lane + (w >> 1));
    // e4m3: of both pages of the pair, for their scales
    const uint32_t first_a = DT == PKV_E4M3 ? table_id(2 * lane) : 0u, first_b = DT == PKV_E4M3 ? table_id(2 * lane + 1) : 0u;

    // this wave's tile: the group's tokens [w * tile_tok, ...)
    const int t0 = w * tile_tok;
    int my_tok = ntok - t0;
    my_tok = my_tok < 0 ? 0 : (my_tok > tile_tok ? tile_tok : my_tok);
    const bool col_live = n < d.cols && tok < my_tok;

    // q as the column operand: lane (h, n) holds q[column n][16 kk + 8 h .. + 7], zeros in a column that stands for no query
    u32x4 qf[TL::NK];
    {
        const uint16_t *qrow = d.q + ((size_t)(q0 + (col_live ? t0 + tok : 0)) * d.Hq + kvh * d.g + (col_live ? head : 0)) * D + 8 * h;
#pragma unroll
        for (int kk = 0; kk < TL::NK; ++kk) qf[kk] = *reinterpret_cast<const u32x4 *>(qrow + 16 * kk);
    }

    // tokens the group's last query sees, never beyond what the row holds
    int L = PKV_CONST(int32_t, d.ctx_lens)[seq];
    int cap = PKV_CONST(int32_t, d.row_len)[seq];
    asm volatile("" : "+s"(L), "+s"(cap));                 // both at once
    L -= gi.back;
    cap *= PKV_T;
    L = L < 0 ? 0 : (L > cap ? cap : L);
    const int n_pages = (L + PKV_T - 1) / PKV_T, n_pairs = (n_pages + 1) >> 1;
    // the pairs this work-group walks
    const int per = n_split > 1 ? (n_pairs + n_split - 1) / n_split : n_pairs;
    const int p_begin = n_split > 1 ? (split * per < n_pairs ? split * per : n_pairs) : 0;
    const int p_end = p_begin + per < n_pairs ? p_begin + per : n_pairs;
    const int np = p_end - p_begin;
    // pairs below it hold only tokens that every column sees
    const int causal_from = L - (ntok - 1);
    const int p_plain = causal_from > 0 ? causal_from >> 5 : 0;

    const int col_lim = col_live ? L - (ntok - 1 - (t0 + tok)) : L;          // tokens this column sees
    const int tile_lim = my_tok > 0 ? L - (ntok - t0 - my_tok) : 0;          // tokens some column of the tile sees

    f32x16 acc[TL::ND];
#pragma unroll
    for (int dt = 0; dt < TL::ND; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[dt][i] = 0.f;
    float m = PF_M0, l = 0.f;

    // ---- requests.  Wave 0: K of page a, wave 1: V of page a, wave 2: K of page b, wave 3: V of page b.
    // The addresses of 64 pairs are worked out at a time, one pair per lane, and handed out by lane reads;
    // e4m3: so are the scales of both pages of 64 pairs.
    const bool is_v = w & 1;
    uint32_t bad = 0;
    const uint32_t lane16 = lane * 16;
    const uint32_t lds_tile = (uint32_t)(size_t)(__attribute__((address_space(3))) uint8_t *)ring + (is_v ? PF_SLOTS * SLOT : 0) +
                              (w >> 1) * TL::BYTES;
    // a page past the end of the context, or an id outside the pool, is never dereferenced: zeros stand in
    auto block_of = [&](int page, uint32_t id, uint64_t offset) __attribute__((always_inline)) {
        const bool in_pool = id < d.max_block_id;
        const bool live = page < n_pages;
        bad |= live && !in_pool ? 1u : 0u;
        const uint32_t f = fastdiv_div(id, d.slots_div);
        const uint32_t sl = id - f * d.slots_div.d;
        const uint8_t *blk = d.pool_base + (uint64_t)f * d.frame_bytes + (uint64_t)sl * d.block_bytes + offset;
        return live && in_pool ? blk : reinterpret_cast<const uint8_t *>(d.safe);
    };
    const uint64_t tile_offset = (DT == PKV_E4M3 ? PKV_FP8_HEADER : 0) + ((uint64_t)kvh * 2 + (is_v ? 1 : 0)) * TL::BYTES;
    uint32_t addr_lo = 0, addr_hi = 0;
    int addr_win = 0;
    auto load_addr = [&](int p) __attribute__((always_inline)) {
        addr_win = p;
        const int page = 2 * (p + lane) + (w >> 1);
        const uint8_t *src = block_of(page, p == 0 ? first_id : table_id(page), tile_offset);
        addr_lo = (uint32_t)(uintptr_t)src;
        addr_hi = (uint32_t)((uintptr_t)src >> 32);
        asm volatile("" ::"v"(addr_lo), "v"(addr_hi));     // waited for here, not where they are used
    };
    auto fetch = [&](int r) __attribute__((always_inline)) {                              // request this wave's tile of pair p_begin + r
        const int p = p_begin + r;
        const int at = p - addr_win;
        const uint64_t src = (uint32_t)__builtin_amdgcn_readlane((int)addr_lo, at) |
                             ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)addr_hi, at) << 32);
        lds_fill<TL::NL>(reinterpret_cast<const uint8_t *>(src), lds_tile + (uint32_t)(r & (PF_SLOTS - 1)) * SLOT, lane16);
    };
    float w_ska = 1.f, w_skb = 1.f, w_sva = 1.f, w_svb = 1.f;
    int scale_win = -64;
    float sva = 1.f, svb = 1.f, sva_n = 1.f, svb_n = 1.f, sca = d.scale_log2, scb = d.scale_log2;
    auto scales = [&](int p) __attribute__((always_inline)) {                             // e4m3: the scales of pair p (K into sca / scb, V into sv*_n)
        if (DT != PKV_E4M3) return;
        if (p - scale_win >= 64) {
            scale_win = p;
            const int page = 2 * (p + lane);
            uint32_t ida = first_a, idb = first_b;
            if (p > 0) {
                ida = table_id(page);
                idb = table_id(page + 1);
            }
            const float *ha = reinterpret_cast<const float *>(block_of(page, ida, 0));
            const float *hb = reinterpret_cast<const float *>(block_of(page + 1, idb, 0));
            w_ska = ha[kvh]; w_sva = ha[d.Hkv + kvh];
            w_skb = hb[kvh]; w_svb = hb[d.Hkv + kvh];
            asm volatile("" ::"v"(w_ska), "v"(w_sva), "v"(w_skb), "v"(w_svb));
        }
        const int at = p - scale_win;
        auto lane_of = [&](float x) __attribute__((always_inline)) { return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), at)); };
        sca = lane_of(w_ska) * d.scale_log2;
        scb = lane_of(w_skb) * d.scale_log2;
        sva_n = lane_of(w_sva);
        svb_n = lane_of(w_svb);
    };

    // ---- operands.  K: lane (h, n) reads token n & 15 of page n >> 4, units h and h + 2, ... (512 bytes apart)
    u32x4 kr[TL::NU];
    const uint8_t *k_lane = ring + hi16 * TL::BYTES + h * 256 + c16 * 16;
    auto read_k = [&](int r) __attribute__((always_inline)) {
        const uint8_t *src = k_lane + (r & (PF_SLOTS - 1)) * SLOT;
#pragma unroll
        for (int u = 0; u < TL::NU; ++u) kr[u] = *reinterpret_cast<const u32x4 *>(src + u * 512);
    };
    // V: one output element of tokens 4h..4h+3 and 8+4h..8+4h+3 of a page (lane row groups h and 2 + h).  Which element is row
    // n of tile dt is free: it is chosen so that 16 lanes in a row read all of 128 bytes (no two of them share a bank) and four rows in a
    // row, which one lane sums up, are four elements in a row (with elements in the order in which they lie in LDS the lanes had to
    // exchange their sums at the end: 311 x 5 new tokens of 16/4/128 16.7 us, 16.1; 237 x (22 + 5) of 8/8/128 21.5, 20.6).
    //   e4m3, D = 128: element 64 (n >> 4) + 16 dt + (n & 15), whole units, the words of one for the four tiles
    //   otherwise: half `half` of unit `unit`, element V_BASE dt + V_STEP half + unit
    constexpr bool UNITS = DT == PKV_E4M3 && D == 128;
    constexpr int V_BASE = DT == PKV_BF16 ? 32 : 16, V_STEP = DT == PKV_BF16 ? 16 : 32;
    constexpr int VW = DT == PKV_BF16 ? 2 : 1;             // words per token group
    uint32_t vr[TL::ND][2][2 * VW];
    const int unit = 8 * hi16 + (n & 7), half = (n >> 3) & 1;
    const uint8_t *v_lane = ring + PF_SLOTS * SLOT + h * 256 + (UNITS ? hi16 * 1024 + c16 * 16 : unit * 16 + half * 8);
    auto read_v = [&](int r) __attribute__((always_inline)) {
        const uint8_t *src = v_lane + (r & (PF_SLOTS - 1)) * SLOT;
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if constexpr (DT == PKV_BF16) {
#pragma unroll
                for (int dt = 0; dt < TL::ND; ++dt) {
                    const uint8_t *at = src + k * TL::BYTES + dt * 1024;
                    const u32x2 a = *reinterpret_cast<const u32x2 *>(at), b = *reinterpret_cast<const u32x2 *>(at + 512);
                    vr[dt][k][0] = a.x; vr[dt][k][1] = a.y; vr[dt][k][2] = b.x; vr[dt][k][3] = b.y;
                }
            } else {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    typedef uint32_t words __attribute__((ext_vector_type(TL::ND)));
                    const words a = *reinterpret_cast<const words *>(src + k * TL::BYTES + q * 512);
#pragma unroll
                    for (int dt = 0; dt < TL::ND; ++dt) vr[dt][k][q] = a[dt];
                }
            }
    };
    auto k_op = [&](int kk) __attribute__((always_inline)) {
        if constexpr (DT == PKV_BF16) return as_bf16x8(kr[kk]);
        else {
            const u32x4 u = kr[2 * (kk >> 2) + (kk & 1)];
            const u32x2 a = fp8x4_to_bf16x4((kk & 2) ? u.z : u.x), b = fp8x4_to_bf16x4((kk & 2) ? u.w : u.y);
            return as_bf16x8(mk4(a.x, a.y, b.x, b.y));
        }
    };
    auto v_op = [&](int dt, int k) __attribute__((always_inline)) {
        if constexpr (DT == PKV_BF16) return as_bf16x8(mk4(vr[dt][k][0], vr[dt][k][1], vr[dt][k][2], vr[dt][k][3]));
        else {
            const u32x2 a = fp8x4_to_bf16x4(vr[dt][k][0]), b = fp8x4_to_bf16x4(vr[dt][k][1]);
            return as_bf16x8(mk4(a.x, a.y, b.x, b.y));
        }
    };
    // tokens past the context may hold anything (even NaN): blank their V (their probabilities are 0)
    auto blank_v = [&](int p) __attribute__((always_inline)) {
        const int left = L - 32 * p - 4 * h;               // tokens of the pair before the end, from this half's first
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int v = left - 16 * k - 8 * q;       // live tokens of this group of four
                if constexpr (DT == PKV_BF16) {
                    const uint32_t m01 = v >= 2 ? 0xffffffffu : (v == 1 ? 0x0000ffffu : 0u);
                    const uint32_t m23 = v >= 4 ? 0xffffffffu : (v == 3 ? 0x0000ffffu : 0u);
#pragma unroll
                    for (int dt = 0; dt < TL::ND; ++dt) {
                        vr[dt][k][2 * q] &= m01;
                        vr[dt][k][2 * q + 1] &= m23;
                    }
                } else {
                    const uint32_t mm = v >= 4 ? 0xffffffffu : (v <= 0 ? 0u : (1u << (8 * v)) - 1u);
#pragma unroll
                    for (int dt = 0; dt < TL::ND; ++dt) vr[dt][k][q] &= mm;
                }
            }
    };

    // ---- one pair's softmax, in two parts.  Arguments: t = score * scale - m (log2 domain) against the reference
    // point m as it stands.  m need not be the column's maximum, only near it: it moves, and the sums are
    // rescaled, when a lane's sum of the pair's probabilities exceeds kSumBar, so that no probability does.
    // An argument takes the score before it is rounded, m is a rounded one: where that difference is no longer small
    // (some |m| beyond PF_FAR), every step is settled (bar -1), with arguments that take the rounded score too.
    f32x16 s;
    float bar = kSumBar;                                   // wave-uniform
    f32x16 pr;
    auto args = [&](int p, bool masked, bool far = false) __attribute__((always_inline)) {
        if (far) {
#pragma clang fp contract(off)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float x = s[i] * (i < 8 ? sca : scb);
                pr[i] = x - m;
            }
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) pr[i] = __builtin_fmaf(s[i], i < 8 ? sca : scb, -m);
        }
        if (masked) {
            const int rel = col_lim - 32 * p - 4 * h;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float x = pr[i];
                pr[i] = 16 * (i >> 3) + 8 * ((i >> 2) & 1) + (i & 3) < rel ? x : -INFINITY;
            }
        }
    };
    // p = exp2(t) and their sum over this lane's tokens.  No probability is larger than the sum, so the sum tells when the
    // reference point has to move: no maximum is taken in an ordinary step.
    auto take = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) pr[i] = __builtin_amdgcn_exp2f(pr[i]);
        return (((pr[0] + pr[1]) + (pr[2] + pr[3])) + ((pr[4] + pr[5]) + (pr[6] + pr[7]))) +
               (((pr[8] + pr[9]) + (pr[10] + pr[11])) + ((pr[12] + pr[13]) + (pr[14] + pr[15])));
    };
    auto settle = [&](int p, bool masked) __attribute__((always_inline)) {
        float sum = take();
        if (__builtin_expect(__any(sum > bar), 0)) {
            // the column's maximum from the scores themselves (arguments are inexact when m is far off)
            const int rel = col_lim - 32 * p - 4 * h;
            float top = -INFINITY;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const float x = s[i] * (i < 8 ? sca : scb);
                const bool dead = masked && 16 * (i >> 3) + 8 * ((i >> 2) & 1) + (i & 3) >= rel;
                top = fmaxf(top, dead ? -INFINITY : x);
            }
            top = halves_max(top);
            const float m_new = fmaxf(m, top);
            const float alpha = __builtin_amdgcn_exp2f(m - m_new);
            l *= alpha;
#pragma unroll
            for (int dt = 0; dt < TL::ND; ++dt) acc[dt] *= alpha;
            m = m_new;
            const bool far = __any(fabsf(m) > PF_FAR && m > PF_M0);
            bar = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(far ? -1.0f : kSumBar)));
            args(p, masked, far);
            sum = take();
        }
        l += sum;
    };
    auto scores = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
        for (int kk = 0; kk < TL::NK; ++kk)
            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_op(kk), as_bf16x8(qf[kk]), s, 0, 0, 0);
    };
    u32x4 ph[2], pl[2];
    auto probabilities = [&]() __attribute__((always_inline)) {
        if (DT == PKV_E4M3) {
#pragma unroll
            for (int i = 0; i < 16; ++i) pr[i] *= i < 8 ? sva : svb;
        }
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e) ph[k][e] = pack_bf16_rne(pr[8 * k + 2 * e], pr[8 * k + 2 * e + 1]);
    };
    auto low_halves = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                pl[k][e] = pack_bf16_rne(pr[8 * k + 2 * e] - __uint_as_float(ph[k][e] << 16),
                                         pr[8 * k + 2 * e + 1] - __uint_as_float(ph[k][e] & 0xffff0000u));
    };
    auto accumulate = [&](const u32x4 *p) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int dt = 0; dt < TL::ND; ++dt)
                acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_op(dt, k), as_bf16x8(p[k]), acc[dt], 0, 0, 0);
    };

    // 128-wide heads, two work-groups a CU: issue favours the older of the two waves of a SIMD.  Of the 512 work-groups of 512
    // tokens behind 15872 of 64/8/128, which all start together, half end within 236 to 291 us and half within 291 to 349, alone
    // from then on.  So a wave steps down a priority level in the course of its walk, and whichever work-group is behind is
    // favoured until it reaches the same level.  On it the older one draws ahead again, by some 0.4 of the level's length, and its lead
    // on the last level is how long the other one is alone at the end: so each level is half as long as the one before (8, 4, 2 and 1
    // fifteenths of the walk).  With four equal levels the two of a CU ended 32 us apart.  Us a pass without and with equal levels:
    // that pass 361.1, 358.1; 8 x (2048 + 512) of 32/8/128 bf16 223.8, 222.3, e4m3 183.0, 181.2; 8 x (1024 + 512) 136.2, 133.8 and 118.3,
    // 112.9.  Without and with halved ones: 8 x (2048 + 512) bf16 218.4, 213.4, e4m3 174.2, 168.3; 8 x (1024 + 512) 131.6, 127.9 and 107.3,
    // 104.2 (last levels of 1/24 or 1/8 of the walk instead of 1/15: 0.2 to 1.2 % more).  Within 256 work-groups, one a CU, bf16 launches lose
    // 1 % to the code of the levels, whether they are taken or not (2 x (768 + 256) 27.4 without it, 27.8); fresh prompts of very many
    // work-groups lose too (4 x 1024 66.0, 69.4, e4m3 56.8, 60.9).  64-wide heads have three work-groups a CU, which even out by
    // themselves: they go without (8 x (1024 + 512) of 32/8/64 bf16 86.5, 95.8, e4m3 80.3, 90.2).  A decode step of another model on a stream
    // beside it takes as long either way (16 x 2048 beside 8 x (2048 + 512) 218.5, 217.0; 4 x 300 beside 1 x (3968 + 128) 15.9, 15.5).
    // (The waves meet in every second or fourth step, for the last time in step np - 2 or before.  Rounded to such a step the last one
    // never comes in walks of up to 29 and odd numbers up to 43 pairs (bf16), of up to 17 and half of those up to 57 (e4m3): these end a level
    // or two above 0.  Moved to the last meeting, so that all end on it, launches take as long or up to 1 % longer.)
    constexpr bool LEVELS = D == 128;
    const int first_step = (np / 2 + np / 32 + MEET / 2) & -MEET, second_step = (np - np / 5 + MEET / 2) & -MEET, third_step = (np - np / 15 + MEET / 2) & -MEET;
    if constexpr (LEVELS) __builtin_amdgcn_s_setprio(3);

    // the meeting point of the steps r to r + MEET - 1, in the middle of step r: all requests under way have landed; behind
    // it K of pairs r + 2 to r + MEET + 1 and V of pairs r + 1 to r + MEET are visible to all waves, and the slots read up to now
    // take the next MEET pairs
    auto meet = [&](int r) __attribute__((always_inline)) {
        if constexpr (LEVELS) {
            if (r == first_step) __builtin_amdgcn_s_setprio(2);
            if (r == second_step) __builtin_amdgcn_s_setprio(1);
            if (r == third_step) __builtin_amdgcn_s_setprio(0);
        }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        const int next = r + MEET + 2 - (is_v ? 1 : 0);
        if (next < np && p_begin + next + MEET - 1 - addr_win >= 64) load_addr(p_begin + next);
#pragma unroll
        for (int i = 0; i < MEET; ++i)
            if (next + i < np) fetch(next + i);
    };

    if (np > 0) {
        load_addr(p_begin);
        const int ahead = MEET + 2 - (is_v ? 1 : 0), first = ahead < np ? ahead : np;
        for (int r = 0; r < first; ++r) fetch(r);
#pragma unroll
        for (int kk = 0; kk < TL::NK; ++kk)
            if (!col_live) qf[kk] = mk4(0, 0, 0, 0);
        wait_requests<TL::NL>(first - 2);                  // K 0, K 1 and V 0, V 1
        __builtin_amdgcn_s_barrier();
        const bool live = my_tok > 0;
        if (live) read_k(0);
        if (live) {
            scales(p_begin);
            scores();
            sva = sva_n; svb = svb_n;
            if (np > 1) read_k(1);
            const bool masked = p_begin >= p_plain;
            args(p_begin, masked);
            settle(p_begin, masked);
        }
        int r = 0;
        // pairs in front of pairs without masks: straight-line steps
        const int plain = live ? (np < p_plain - p_begin ? np : p_plain - p_begin) - 1 : 0;
        if (plain > 0) {
            do {
                read_v(r);
                scales(p_begin + r + 1);
                scores();
                probabilities();
                if (!(r & (MEET - 1))) meet(r);
                if (r + 2 < np) read_k(r + 2);
                sva = sva_n; svb = svb_n;
                accumulate(ph);
                if (DT == PKV_BF16) {
                    low_halves();
                    accumulate(pl);
                }
                args(p_begin + r + 1, false);
                settle(p_begin + r + 1, false);
            } while (++r < plain);
        }
        for (; r < np; ++r) {
            const int p = p_begin + r;
            const bool now = 32 * p < tile_lim, next = (r + 1 < np) & (32 * (p + 1) < tile_lim);     // (neither where no token is the wave's)
            if (now) {
                read_v(r);
                probabilities();
            }
            if (next) {
                scales(p + 1);
                scores();
            }
            if (r + 1 < np && !(r & (MEET - 1))) meet(r);
            if (next && r + 2 < np) read_k(r + 2);
            if (now) {
                if (32 * (p + 1) > L) blank_v(p);
                accumulate(ph);
                if (DT == PKV_BF16) {
                    low_halves();
                    accumulate(pl);
                }
            }
            if (next) {
                sva = sva_n; svb = svb_n;
                const bool masked = p + 1 >= p_plain;
                args(p + 1, masked);
                settle(p + 1, masked);
            }
        }
    }

    l += __shfl_xor(l, 32);
    // this lane's sums of its column, four elements at a time
    auto put_sums = [&](float *row, float f) __attribute__((always_inline)) {
#pragma unroll
        for (int dt = 0; dt < TL::ND; ++dt)
#pragma unroll
            for (int j = 0; j < 4; ++j)                    // rows 8 j + 4 h to 8 j + 4 h + 3
                *reinterpret_cast<f32x4 *>(row + (UNITS ? 64 * (j >> 1) + 16 * dt + 8 * (j & 1) : V_BASE * dt + V_STEP * (j & 1) + 8 * (j >> 1)) + 4 * h) =
                    f32x4{acc[dt][4 * j], acc[dt][4 * j + 1], acc[dt][4 * j + 2], acc[dt][4 * j + 3]} * f;
    };
    if (n_split > 1) {
        // a part of the context: the unnormalised sums, the reference point and the denominator of every column
        float *part = d.ws + (((size_t)group * d.Hkv + kvh) * PKV_PREFILL_COLS + w * PF_COLS + n) * (D + 4);
        put_sums(part, 1.f);
        if (h == 0) {
            part[D] = m;
            part[D + 1] = l;
        }
    } else if (col_live) {
        float *out_row = d.out + ((size_t)(q0 + t0 + tok) * d.Hq + kvh * d.g + head) * D;
        const float inv = l > 0.f ? 1.0f / l : 0.f;        // no visible token: the row is defined as zero
        put_sums(out_row, inv);
    }
    if (__any(bad != 0) && lane == 0) atomicOr(d.err, 1u);
}

// Joins the parts of a group whose context was walked by several work-groups of k_prefill (consecutive units):
// out = sum_i 2^(m_i - M) acc_i / sum_i 2^(m_i - M) l_i with M = max_i m_i, per column.  One work-group per eight
// columns, 32 lanes a column.  Bound by memory round trips: all maxima and denominators of a column travel at once,
// its sums eight parts a trip (one part after the other, 32 parts of one group took 80 of a call's 101 us).
constexpr int MERGE_COLS = 8;

template <int SEQS>
__global__ __launch_bounds__(32 * MERGE_COLS) void k_prefill_merge(const AttnDesc d, const PlanOf<SEQS> plan) {
    __shared__ float s_f[MERGE_COLS][PKV_PLAN_MAX_PARTS];
    constexpr int BLOCKS = PKV_PREFILL_COLS / MERGE_COLS;
    const int sub = threadIdx.x & 31, cc = threadIdx.x >> 5;
    const int x = blockIdx.x / BLOCKS, rank = x / d.Hkv, kvh = x - rank * d.Hkv;
    const int c = (blockIdx.x - x * BLOCKS) * MERGE_COLS + cc;
    const uint32_t entry = plan.s[blockIdx.y].unit, seq = entry >> PKV_PLAN_SEQ_SHIFT, first = plan.s[seq].row;
    const int parts = (int)(first >> PKV_PLAN_PART_SHIFT), row0 = (int)(first & PKV_PLAN_ROWS);
    const int rows = (int)(plan.s[seq + 1].row & PKV_PLAN_ROWS) - row0;
    const int tile_tok = d.cols / d.g, size = PF_WAVES * tile_tok, groups = (rows + size - 1) / size;
    if (parts <= 1 || rank >= groups) return;
    const int t0 = (groups - 1 - rank) * size;
    const int n = c & (PF_COLS - 1), tok = t0 + (c / PF_COLS) * tile_tok + n / d.g;      // this column's query token
    if (__syncthreads_or(n < d.cols && tok < rows) == 0) return;
    const int D = d.D, stride = D + 4;       // D sums, the reference point, the denominator, two unused (16-byte rows)
    const size_t step = (size_t)d.Hkv * PKV_PREFILL_COLS * stride;
    const float *part = d.ws + (((size_t)(entry & PKV_PLAN_UNITS) + (size_t)rank * parts) * d.Hkv + kvh) * PKV_PREFILL_COLS * stride + (size_t)c * stride;
    float m[2], l[2], M = PF_M0;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int i = sub + 32 * k;
        m[k] = i < parts ? part[i * step + D] : PF_M0;
        l[k] = i < parts ? part[i * step + D + 1] : 0.f;
        M = fmaxf(M, m[k]);
    }
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) M = fmaxf(M, __shfl_xor(M, o));
    float den = 0.f;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int i = sub + 32 * k;
        const float f = i < parts ? __builtin_amdgcn_exp2f(m[k] - M) : 0.f;
        s_f[cc][i] = f;
        den += f * l[k];
    }
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) den += __shfl_xor(den, o);
    __syncthreads();
    if (n >= d.cols || tok >= rows || 4 * sub >= D) return;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int i0 = 0; i0 < parts; i0 += 8) {
        f32x4 v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = *reinterpret_cast<const f32x4 *>(part + (i0 + u < parts ? i0 + u : parts - 1) * step + 4 * sub);
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (i0 + u < parts) acc += v[u] * s_f[cc][i0 + u];
    }
    const float inv = den > 0.f ? 1.0f / den : 0.f;
    *reinterpret_cast<f32x4 *>(d.out + ((size_t)(row0 + tok) * d.Hq + kvh * d.g + (n - (n / d.g) * d.g)) * D + 4 * sub) = acc * inv;
}

template <int SEQS>
void launch(const AttnDesc &d, const PlanOf<SEQS> &plan, int split_groups, bool meets_often, hipStream_t s) {
    const dim3 grid(plan.s[plan.n_seqs].unit * (unsigned)d.Hkv), wg(64 * PF_WAVES);
    if (d.dtype == PKV_BF16) {
        if (d.D == 128) hipLaunchKernelGGL((k_prefill<128, PKV_BF16, SEQS, 2>), grid, wg, 0, s, d, plan);
        else hipLaunchKernelGGL((k_prefill<64, PKV_BF16, SEQS, 2>), grid, wg, 0, s, d, plan);
    } else {
        if (d.D == 64) hipLaunchKernelGGL((k_prefill<64, PKV_E4M3, SEQS, 4>), grid, wg, 0, s, d, plan);
        else if (meets_often) hipLaunchKernelGGL((k_prefill<128, PKV_E4M3, SEQS, 2>), grid, wg, 0, s, d, plan);
        else hipLaunchKernelGGL((k_prefill<128, PKV_E4M3, SEQS, 4>), grid, wg, 0, s, d, plan);
    }
    if (split_groups > 0)
        hipLaunchKernelGGL(k_prefill_merge<SEQS>, dim3((unsigned)(split_groups * d.Hkv * (PKV_PREFILL_COLS / MERGE_COLS)), (unsigned)plan.n_seqs),
                           dim3(32 * MERGE_COLS), 0, s, d, plan);
}

}  // namespace

// Whether the waves of an e4m3 launch with 128-wide heads meet once in two pairs.  A work-group's LDS is given back when its last wave
// ends, its registers wave by wave: with the rings for four pairs (64 KiB) a third work-group of a CU waits for the LDS, with those for
// two (32 KiB) it starts beside the last waves.  That counts where more work-groups come than two a CU and walks are short.  Us,
// met in four and in two pairs: 92 x 5 new tokens of 32/8/128 (736 work-groups of one pair) 11.0, 10.2; 128 x (176 + 5) of 16/8/128 (1024 of
// six) 22.5, 21.3.  180 launches of short chunks: one to two pairs 1.074 (513 to 768 work-groups), up to eight 1.007 to 1.026; but nine to
// sixteen 0.97 to 0.99, and within 512 work-groups 0.95 to 1.00 of any length.  64-wide heads, three a CU: 0.99 to 1.01.
static bool meets_often_in(const AttnDesc &d, const ChunkPlan &plan, int longest_walk) {
    return longest_walk <= 8 && plan.s[plan.n_seqs].unit * (unsigned)d.Hkv > 512u;
}

hipError_t pkv_launch_prefill(const AttnDesc &d, const ChunkPlan &plan, int split_groups, int longest_walk, hipStream_t s) {
    if (plan.s[plan.n_seqs].unit == 0) return hipSuccess;
    const bool meets_often = meets_often_in(d, plan, longest_walk);
    if (plan.n_seqs <= PKV_PLAN_FEW) launch(d, few_of(plan), split_groups, meets_often, s);
    else launch(d, plan, split_groups, meets_often, s);
    return hipGetLastError();
}
