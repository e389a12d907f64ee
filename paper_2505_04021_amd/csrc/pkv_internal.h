// Internal declarations shared by the host API and the HIP kernels of libprismkv.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// built with hidden visibility: only what the public header declares is exported
#pragma GCC visibility push(default)
#include "../../include/prism_kv.h"
#include "../../include/prism_kv_tuning.h"
#pragma GCC visibility pop

#define PKV_MAX_POOLS 8
#define PKV_MAX_MODELS 64
#define PKV_FP8_HEADER 128   // bytes in front of an e4m3 block: fp32 sK[Hkv], fp32 sV[Hkv]
#define PKV_MAX_BATCH_OPS 4096   // entries of one reserve call (the growth rounds of a whole admission)
#define PKV_MAX_ROW_BLOCKS (1 << 20)   // blocks a row can hold at most (the reserve kernel packs a row position into 20 bits)
#define PKV_MAX_SEQS 4096
#define PKV_BOOK_THREADS 1024
// The file-scope scratch array of decode_attention_static: arrival counters, then split-K partials.
#define PKV_STATIC_COUNTERS 32768
#define PKV_STATIC_SCRATCH_BYTES ((size_t)20 << 20)

// Unsigned division by an invariant divisor with one multiply-high and two shifts
// (Granlund & Montgomery, "Division by invariant integers using multiplication").
// Exact for every 32-bit numerator.
struct FastDiv {
    uint32_t d, mul, sh1, sh2;
};

static inline FastDiv fastdiv_make(uint32_t d) {
    FastDiv f;
    f.d = d;
    uint32_t l = 0;
    while ((1ull << l) < d) ++l;                   // l = ceil(log2 d)
    f.mul = (uint32_t)(((1ull << 32) * ((1ull << l) - d)) / d + 1);
    f.sh1 = l < 1 ? l : 1;
    f.sh2 = l < 1 ? 0 : l - 1;
    return f;
}

__host__ __device__ static inline uint32_t fastdiv_div(uint32_t n, const FastDiv &f) {
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t t = __umulhi(n, f.mul);
#else
    uint32_t t = (uint32_t)(((uint64_t)n * f.mul) >> 32);
#endif
    return (t + ((n - t) >> f.sh1)) >> f.sh2;
}

// Result slot in pinned host memory, written by the bookkeeping kernels.
struct BookResult {
    int64_t value;     // count or negative PKV_E_* code
    int64_t aux0, aux1;
};

// Device-resident pool state.
struct PoolDev {
    int32_t *owner;        // [n_frames] model id or -1
    uint32_t *free_stack;  // [n_frames], [0] bottom .. [n_free-1] top
    int32_t *pos;          // [n_frames] position of the frame in its owner's list
    int64_t *n_free;       // [1]
    int64_t n_frames;
};

// Floats per split-K partial of decode attention: g rows of D accumulators, then g maxima, then g sums, in whole 16-byte
// units (the kernels read and write the accumulators in those, and a workspace holds partial after partial).
__host__ __device__ constexpr int partial_floats(int g, int D) { return (g * (D + 2) + 3) & ~3; }
static_assert(partial_floats(1, 128) * sizeof(float) % 16 == 0 && partial_floats(3, 64) * sizeof(float) % 16 == 0 &&
                  partial_floats(16, 128) == 16 * 130 && partial_floats(5, 64) >= 5 * 66,
              "whole units, nothing lost");

// Device-resident per-model bookkeeping state.
struct ModelDev {
    uint32_t *frames;      // [n_frames] acquisition order
    uint32_t *bits;        // [n_frames][wpf] slot bits of the frame at that position
    uint8_t *mark;         // [n_frames] scratch for deflate
    int32_t *rows;         // [max_seqs][max_blocks] block ids
    int32_t *row_len;      // [max_seqs]
    int64_t *counters;     // [0] owned frames, [1] free slots
    int32_t model_id;
    int32_t slots, wpf;    // slots per frame, 32-bit words per frame in `bits`
    int32_t max_seqs, max_blocks, page_tokens;
    FastDiv slots_div;     // division by `slots`
    FastDiv wpf_div;       // division by `wpf`
};

// What one attention work-group needs to know about its model.
struct AttnDesc {
    const uint8_t *pool_base;
    const uint16_t *q;          // bf16 [B][Hq][D]
    const int32_t *table;       // [B][row_stride]
    const int32_t *ctx_lens;    // [B]
    const int32_t *row_len;     // library table: [max_seqs] blocks reserved per row; NULL for a caller's table
    float *out;                 // [B][Hq][D]
    float *ws;                  // split-K partials: two per work item (uncached memory)
    uint32_t *cnt;              // [B][Hkv] arrival counters of the split-K merge, zero between launches
    uint32_t *err;              // device error flags
    const void *safe;           // 16 KiB of zeros owned by the library: stands in for blocks that must not be read
    uint64_t frame_bytes, block_bytes;
    FastDiv slots_div;
    uint32_t max_block_id;      // n_frames * slots
    int32_t batch, row_stride;
    int32_t Hq, Hkv, g, D, dtype;
    int32_t cols;               // prefill: MFMA columns in use of a wave's tile, (query tokens) * g, at most 32
    int32_t item_begin;         // first work item of this model in a grouped launch
    int32_t n_items;            // work items (waves) of this model
    int32_t min_share;          // smallest share of pages a wave may get
    int32_t weighted;           // items come in whole blocks of eight aligned with the XCDs
    int32_t seg_cost;           // what a segment costs besides its pages, in pages (for the split only)
    int32_t max_pages;          // longest row, as far as the host knows
    int32_t parts, part_pages;  // small launches: work-groups per (sequence, kv head), pages of each (item_begin then counts
                                // work-groups)
    float scale_log2;           // log2(e) / sqrt(D)
};

// How a chunk call (prefill_attention, kv_append_chunk) falls into units of work, as far as the host decides it: per
// sequence where its units and its packed rows begin.  Units may come in another order of the sequences than rows.  It travels in the kernel's arguments, so a call copies
// nothing to the device and needs no buffer.  A kernel's arguments end at 4 KB: a launch holds at most PKV_PLAN_SEQS
// sequences, and every work-group reads the plan, so that few sequences come with a shorter one (an append of 17 tokens each
// for 127 sequences 7.3 us, for 128 8.0).  With launches of 127 sequences, the last one often small, 128 x (1000 cached + 17
// new) tokens of 32/8/128 took 151 us (one launch 128), 447 x (200 + 3) of 8/2/128 41 (24.5), their append 18 (7).
#define PKV_PLAN_FEW 127
#define PKV_PLAN_SEQS 447
#define PKV_PLAN_SEQ_SHIFT 23        // of `unit`: the entry's sequence above, its first unit (fewer than 2^22) below
#define PKV_PLAN_UNITS 0x7fffffu
#define PKV_PLAN_PART_SHIFT 25       // of `row`: parts of the context per group above, first packed row (at most 2^24) below
#define PKV_PLAN_ROWS 0x1ffffffu
#define PKV_PLAN_MAX_PARTS 64
template <int SEQS>
struct PlanOf {
    int32_t n_seqs, seq0;                 // sequences seq0 .. seq0 + n_seqs - 1
    struct {
        uint32_t unit;                    // entry i in the order of the units: its first one | its sequence << PKV_PLAN_SEQ_SHIFT
        uint32_t row;                     // sequence i: its first packed row | parts of the context per group << PKV_PLAN_PART_SHIFT
    } s[SEQS + 1];                        // [n_seqs]: the totals
};
typedef PlanOf<PKV_PLAN_SEQS> ChunkPlan;

// The same plan of at most PKV_PLAN_FEW sequences.
inline PlanOf<PKV_PLAN_FEW> few_of(const ChunkPlan &plan) {
    PlanOf<PKV_PLAN_FEW> few;
    few.n_seqs = plan.n_seqs;
    few.seq0 = plan.seq0;
    for (int i = 0; i <= plan.n_seqs; ++i) {
        few.s[i].unit = plan.s[i].unit;
        few.s[i].row = plan.s[i].row;
    }
    return few;
}

#define PKV_MAX_GROUP 16
#define PKV_PREFILL_WAVES 4     // waves of a prefill work-group
#define PKV_PREFILL_COLS 128    // MFMA columns (query tokens x heads of the kv head) of a prefill work-group, 32 per wave

// How a launch cuts each block of eight consecutive shares among the eight XCDs.
struct AttnTune {
    uint32_t cum[9];            // cumulative weights in 1/65536: cum[0] = 0 <= ... <= cum[8] = 65536
    uint64_t *stat;             // NULL, or [8][2]: per XCD the sum of its waves' streaming times
                                // (100 MHz ticks) and their number; set in tuning launches only
};

struct AttnGroup {
    AttnDesc m[PKV_MAX_GROUP];
    AttnTune tune;
    int32_t n;
};

// ---- launch wrappers implemented in the .hip files ----------------------------
hipError_t pkv_launch_pool_init(const PoolDev &p, const uint32_t *perm_dev, hipStream_t s);
// Bookkeeping kernels: the result goes to *res (pinned host memory); a refused call also sets bit 2 of *err.
hipError_t pkv_launch_resize(const PoolDev &p, const ModelDev &m, int64_t target, BookResult *res, uint32_t *err, hipStream_t s);
// A call's list: in pinned host memory (ops), or, where it is short, in the kernel's arguments (ops NULL: a read of host
// memory is the longest trip such a kernel makes).
#define PKV_BOOK_LIST 192
struct BookList {
    int32_t v[PKV_BOOK_LIST];
};
// list: n sequence ids, n context lengths, then per entry the largest want (blocks) among
// the earlier entries of its sequence in the list (n <= PKV_MAX_BATCH_OPS)
hipError_t pkv_launch_reserve(const PoolDev &p, const ModelDev &m, int n, const int32_t *ops, const BookList &list, BookResult *res,
                              uint32_t *err, hipStream_t s);
// list: n sequence ids (n <= PKV_MAX_SEQS)
hipError_t pkv_launch_release(const PoolDev &p, const ModelDev &m, int n, const int32_t *ops, const BookList &list, BookResult *res,
                              uint32_t *err, hipStream_t s);

hipError_t pkv_launch_kv_write(const AttnDesc &d, int seq, int tok_begin, int n_tok, const void *k, const void *v,
                               const float *ks, const float *vs, int page_tokens, hipStream_t s);
hipError_t pkv_launch_kv_read(const AttnDesc &d, int seq, int tok_begin, int n_tok, void *k, void *v, float *ks, float *vs,
                              hipStream_t s);
// d.batch sequences, d.ctx_lens / d.row_len / d.table as for attention
hipError_t pkv_launch_kv_append(const AttnDesc &d, const void *k_new, const void *v_new, hipStream_t s);
// plan: per sequence one unit for every page its new tokens may touch
hipError_t pkv_launch_kv_append_chunk(const AttnDesc &d, const ChunkPlan &plan, const void *k_new, const void *v_new, hipStream_t s);
// ev: NULL or two events recorded before and after the attention kernel
enum class AttnForm { ordinary, deep, small };
hipError_t pkv_launch_attention(const AttnGroup &grp, AttnForm form, hipStream_t s, hipEvent_t *ev);
// the entry point that allocates nothing: the current device's copy of the library's scratch array
hipError_t pkv_static_scratch(void **ptr);
hipError_t pkv_launch_attention_static(const AttnGroup &grp, uint32_t *cnt, size_t n_cnt, hipStream_t s);
// chunked prefill: a unit is a group of up to PKV_PREFILL_WAVES * (d.cols / d.g) query tokens, or one of the parts
// of its context; split_groups: most groups of a sequence whose groups come in parts (0: none does);
// longest_walk: page pairs that a unit walks at most, as far as the host knows
hipError_t pkv_launch_prefill(const AttnDesc &d, const ChunkPlan &plan, int split_groups, int longest_walk, hipStream_t s);
hipError_t pkv_launch_stream_read(const void *src, size_t bytes, size_t granule_bytes, uint32_t *sink, hipStream_t s);
