// Page-pool / balloon bookkeeping kernels (gfx950).
//
// All state (free stack, frame ownership, per-model frame lists, slot bitmaps,
// block tables) lives in HBM and is changed only here.  The operations follow the
// balloon driver's contract in the paper (Sec. 4.2): D1 — a model's share grows and
// shrinks, memory only changes hands; D2 — token blocks fill slots of the model's
// own pages; D3 — partially filled pages are used first.  Results must be identical
// from run to run and equal to a sequential execution, so every ordering decision
// is taken with prefix sums inside ONE work-group of 1024 lanes; no atomics decide
// an order.  The data moved per call is a few KB, the cost is launch latency.
#include "pkv_internal.h"

#include <type_traits>

namespace {

constexpr int NT = PKV_BOOK_THREADS;
constexpr int NW = NT / 64;

// Work-group barrier for exchanges through LDS only: it waits for this wave's LDS traffic, not for its
// global stores to be acknowledged (__syncthreads does, and a store's round trip costs about as much as
// everything else such a kernel does between two barriers).
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Inclusive prefix sum over a wave, by lane moves inside the vector unit: 1, 2, 4 and 8 lanes up within a row of 16, then
// the last lane of a row to the next one, then of the lower half to the upper one.
__device__ inline int wave_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

// Exclusive prefix sums of N ints per lane over the work-group, side by side; the totals are uniform.  s_wave: N * NW ints.
template <int N>
__device__ inline void block_excl_scans(int *v, int *total, int *s_wave) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int inc[N];
#pragma unroll
    for (int c = 0; c < N; ++c) inc[c] = wave_scan(v[c]);
    lds_barrier();                   // protect s_wave from the previous call's readers
    if (lane == 63) {
#pragma unroll
        for (int c = 0; c < N; ++c) s_wave[c * NW + wave] = inc[c];
    }
    lds_barrier();
#pragma unroll
    for (int c = 0; c < N; ++c) {
        int before = 0, sum = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const int x = s_wave[c * NW + w];
            if (w < wave) before += x;
            sum += x;
        }
        total[c] = sum;
        v[c] = before + inc[c] - v[c];
    }
}
__device__ inline int block_excl_scan(int v, int &total, int *s_wave) {
    block_excl_scans<1>(&v, &total, s_wave);
    return v;
}

__global__ void k_pool_init(PoolDev p, const uint32_t *perm) {
    const int64_t n = p.n_frames;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        p.owner[i] = -1;
        p.pos[i] = -1;
        // pops take from the top (the end): frame perm[0] (or 0) must be last
        p.free_stack[n - 1 - i] = perm ? perm[i] : (uint32_t)i;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) *p.n_free = n;
}

// A call's result goes to its slot in pinned host memory; a refused call also raises the sticky
// device flag (bit 2), so that a caller who only enqueues learns of it without reading every slot.
__device__ inline void book_finish(BookResult *res, uint32_t *err, int64_t value) {
    if (value < 0 && err) atomicOr(err, 4u);
    __threadfence_system();
    res->value = value;
}

// inflate: pop `need` frames, append them to the model's list, all or nothing.
__device__ inline void inflate_body(const PoolDev &p, const ModelDev &m, int64_t target, int64_t owned, int64_t n_free, int64_t spare,
                                    BookResult *res, uint32_t *err) {
    const int64_t need = target - owned;
    if (need > n_free) {
        if (threadIdx.x == 0) book_finish(res, err, PKV_E_NOMEM);
        return;
    }
    for (int64_t k = threadIdx.x; k < need; k += NT) {
        const uint32_t f = p.free_stack[n_free - 1 - k];
        const int64_t at = owned + k;
        p.owner[f] = m.model_id;
        p.pos[f] = (int32_t)at;
        m.frames[at] = f;
        for (int w = 0; w < m.wpf; ++w) m.bits[at * m.wpf + w] = 0u;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        *p.n_free = n_free - need;
        m.counters[0] = target;
        m.counters[1] = spare + need * m.slots;
        res->aux0 = need;
        book_finish(res, err, target);
    }
}

// deflate: hand back empty frames, newest first, until `target` is met (clamp at
// frames that still hold blocks); then close the gaps in the frame list and bitmap
// keeping the order of what stays.
__device__ inline void deflate_body(const PoolDev &p, const ModelDev &m, int64_t target, int64_t owned, int64_t n_free, int64_t spare,
                                    BookResult *res, uint32_t *err, int *s_wave) {
    const int tid = threadIdx.x;
    const int64_t want = owned - target;
    const int wpf = m.wpf;
    int64_t reclaimed = 0, lo = owned;
    for (int64_t base = owned - 1; base >= 0 && reclaimed < want; base -= NT) {
        const int64_t i = base - tid;
        uint32_t used = 0u, f = 0u;
        if (i >= 0) {
            f = m.frames[i];                                       // along with the words, not behind them
            for (int w = 0; w < wpf; ++w) used |= m.bits[i * wpf + w];
        }
        const int empty = i >= 0 && used == 0u;
        int total;
        const int excl = block_excl_scan(empty, total, s_wave);   // rank in newest-first order
        const bool take = empty && (reclaimed + excl < want);
        if (i >= 0) m.mark[i] = take ? 1 : 0;
        if (take) {
            p.free_stack[n_free + reclaimed + excl] = f;           // pushed in scan order
            p.owner[f] = -1;
            p.pos[f] = -1;
        }
        reclaimed += (total < want - reclaimed) ? total : (want - reclaimed);
        lo = (base - (NT - 1) > 0) ? base - (NT - 1) : 0;
    }
    __syncthreads();
    // compaction of positions [lo, owned): column by column, read - barrier - write.
    // A kept entry only moves down, onto a slot whose old content was read in this
    // or an earlier round.  Where every position looked at was given back (a model that falls idle gives all it has), nothing is
    // left to move.
    int64_t w_at = lo;
    for (int64_t base = reclaimed < owned - lo ? lo : owned; base < owned; base += NT) {
        const int64_t i = base + tid;
        const uint32_t f = i < owned ? m.frames[i] : 0u;
        const int keep = (i < owned) && !m.mark[i];
        int total;
        const int excl = block_excl_scan(keep, total, s_wave);
        const int64_t to = w_at + excl;
        __syncthreads();
        if (keep) {
            m.frames[to] = f;
            p.pos[f] = (int32_t)to;
        }
        for (int w = 0; w < wpf; ++w) {
            uint32_t b = 0;
            if (keep) b = m.bits[i * wpf + w];
            __syncthreads();
            if (keep) m.bits[to * wpf + w] = b;
        }
        w_at += total;
        __syncthreads();
    }
    if (tid == 0) {
        *p.n_free = n_free + reclaimed;
        m.counters[0] = owned - reclaimed;
        m.counters[1] = spare - reclaimed * m.slots;
        res->aux0 = reclaimed;
        book_finish(res, err, owned - reclaimed);
    }
}

// balloon_resize: the direction is decided here, from the device's own count of owned frames, so
// that a caller can enqueue the call without knowing how earlier enqueued calls ended.  All counts are asked for at once, for
// both directions; a deflate reads frames along with their words and compacts only if something stays (us, in turn on one
// machine: inflate of 170 frames 2.3 -> 2.2, deflate of as many that are all empty 4.8 -> 3.0).
__global__ __launch_bounds__(NT) void k_resize(PoolDev p, ModelDev m, int64_t target, BookResult *res, uint32_t *err) {
    __shared__ int s_wave[NW];
    const int64_t owned = m.counters[0], spare = m.counters[1], n_free = *p.n_free;          // uniform: every lane takes the same branch
    if (target > owned) inflate_body(p, m, target, owned, n_free, spare, res, err);
    else if (target < owned) deflate_body(p, m, target, owned, n_free, spare, res, err, s_wave);
    else if (threadIdx.x == 0) book_finish(res, err, owned);
}

// reserve (batched): rows grow to ceil(ctx / T) blocks; the new blocks of the whole
// batch take the lowest free slots in frame-list order, entry by entry — the same
// state a sequential loop of single reserves leaves.  A sequence may appear several
// times (the growth rounds of an admission in one call): entry i then needs what its
// row lacks after the earlier entries, i.e. its want minus the largest want among the
// earlier entries of the same sequence (and the row's length before the call).
// list (kernel arguments or pinned host memory): n sequence ids, then n context lengths, then for each entry the largest want
// (in blocks) among the earlier entries of its sequence in this list, 0 if there is none.
constexpr int RESERVE_WIN = 8192;       // ranks whose blocks k_reserve collects in LDS at a time

__global__ __launch_bounds__(NT) void k_reserve(PoolDev p, ModelDev m, int n, const int32_t *host_ops, const BookList list,
                                                BookResult *res, uint32_t *err) {
    const int32_t *ops = host_ops ? host_ops : list.v;
    __shared__ int s_wave[4 * NW];
    __shared__ int s_cur[PKV_MAX_SEQS];             // row lengths: as the call finds them, then with its wants
    __shared__ int s_start[PKV_MAX_BATCH_OPS + 1];  // first rank of entry i
    __shared__ uint32_t s_ent[PKV_MAX_BATCH_OPS];   // entry i: sequence << 20 | row length before the entry
    __shared__ uint32_t s_free[NT], s_id[NT];       // placement: free bits of word j of the turn, the block id of its slot 0
    __shared__ int s_rank[NT];                      // placement: rank of the first free slot of that word
    __shared__ uint32_t s_blk[RESERVE_WIN];         // placement: the blocks of a window of ranks
    __shared__ int s_fail;
    const int tid = threadIdx.x;
    // Everything the kernel will read is asked for here, before the first answer is needed: the list
    // (host memory, the longest trip), the rows' lengths, the counters and the lane's own word of the
    // first turn of the placement.  The call then costs one such trip instead of five in a row.
    constexpr int CHUNKS = PKV_MAX_BATCH_OPS / NT;
    int o_seq[CHUNKS], o_ctx[CHUNKS], o_ear[CHUNKS];
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        const int i = c * NT + tid;
        o_seq[c] = i < n ? ops[i] : 0;
        o_ctx[c] = i < n ? ops[n + i] : 0;
        o_ear[c] = i < n ? ops[2 * n + i] : 0;
    }
    const int64_t owned = m.counters[0], spare = m.counters[1];
    const int wpf = m.wpf, slots = m.slots;
    // (words and list positions that the model does not own yet are read too, and never looked at: the addresses then do
    // not wait for the count of owned frames to arrive)
    const uint32_t first_frame = fastdiv_div((uint32_t)tid, m.wpf_div);
    const uint32_t first_word = first_frame < p.n_frames ? m.bits[tid] : 0u, first_id = first_frame < p.n_frames ? m.frames[first_frame] : 0u;
    for (int s = tid; s < m.max_seqs; s += NT) s_cur[s] = m.row_len[s];
    if (tid == 0) s_fail = 0x7fffffff;
    __syncthreads();
    const int T = m.page_tokens;
    // Row length before an entry = the larger of the row's length when the call began and the largest want
    // among the earlier entries of its sequence.  The second is a property of the list alone and comes
    // with it; the first is read here, for every entry, before any entry's want reaches s_cur.
    int e_seq[CHUNKS], e_want[CHUNKS], e_prev[CHUNKS];
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
        const int i = c * NT + tid;
        e_seq[c] = -1;
        e_want[c] = e_prev[c] = 0;
        if (i < n) {
            const int s_ = o_seq[c], cl = o_ctx[c];
            if (s_ < 0 || s_ >= m.max_seqs || cl < 0) {
                atomicMin(&s_fail, i * 2);                       // the first refused entry decides the code
            } else {
                const int64_t w = ((int64_t)cl + T - 1) / T;
                if (w > m.max_blocks) atomicMin(&s_fail, i * 2 + 1);
                else {
                    e_seq[c] = s_;
                    e_want[c] = (int)w;
                    const int before = s_cur[s_];
                    e_prev[c] = before > o_ear[c] ? before : o_ear[c];
                }
            }
        }
    }
    __syncthreads();
    int total = 0;
    auto rank_chunks = [&](auto count) __attribute__((always_inline)) {       // the first `count` chunks, side by side
        constexpr int N = decltype(count)::value;
        int rank[N], sum[N];
#pragma unroll
        for (int c = 0; c < N; ++c) {
            if (e_seq[c] >= 0) atomicMax(&s_cur[e_seq[c]], e_want[c]);       // the row's length after the call
            rank[c] = e_seq[c] >= 0 && e_want[c] > e_prev[c] ? e_want[c] - e_prev[c] : 0;
        }
        block_excl_scans<N>(rank, sum, s_wave);
#pragma unroll
        for (int c = 0; c < N; ++c) {
            const int i = c * NT + tid;
            if (i < n) {
                s_start[i] = total + rank[c];
                s_ent[i] = ((uint32_t)(e_seq[c] >= 0 ? e_seq[c] : 0) << 20) | (uint32_t)e_prev[c];
            }
            total += sum[c];
        }
    };
    static_assert(CHUNKS == 4, "chunks of the list");
    if (n <= NT) rank_chunks(std::integral_constant<int, 1>{});
    else if (n <= 2 * NT) rank_chunks(std::integral_constant<int, 2>{});
    else rank_chunks(std::integral_constant<int, 4>{});
    if (tid == 0) s_start[n] = total;
    __syncthreads();
    int status = 0;
    if (s_fail != 0x7fffffff) status = (s_fail & 1) ? PKV_E_RANGE : PKV_E_ARG;
    else if ((int64_t)total > spare) status = PKV_E_BALLOON;
    if (status != 0 || total == 0) {
        if (tid == 0) book_finish(res, err, status);
        return;
    }
    // Placement.  Free slots are ranked in frame-list order, ascending slot inside a frame; rank r goes to
    // the entry e with s_start[e] <= r < s_start[e + 1].  A lane per 32-slot word of the bitmap counts the word's free slots (a
    // prefix sum gives the rank of its first one) and publishes it; then a lane per (word, slot) takes over: a free slot knows
    // its rank from the bits below it and puts its block id there, in LDS.  The entries then copy their ranks into their rows,
    // `group` lanes each (a search for the entry of every slot took 4 of this kernel's 13 us).  The word's lane sets the bits
    // that were taken.
    // A turn is 1024 words.  A lane per frame instead, one word of the frame after the other, leaves most lanes idle and takes
    // two barriers a word: slower for every model, also where turns are many and a list is short.  Us of a release and a reserve
    // of all rows, and of one row at the far end of the list, a lane per frame and so: 39 frames of 31 words 146 -> 78 and
    // 34 -> 13; 462 of 8 572 -> 382 and 29 -> 15; 8339 of 2 3821 -> 3359 and 28 -> 26; 137 of one 18.2 -> 16.8 and 13.0 -> 12.0.
    // Four look-ups are on the way at a time while all four are live (dead ones among them: 151 us of this kernel for the
    // first model, where one at a time takes 98).  Reading a turn's words ahead of the turn before made it 2 to 8 % slower.
    int group = 4;
    while (group < NT && group * 2 * n <= NT) group *= 2;
    const int sub = tid & (group - 1);
    int running = 0;
    const int64_t words = owned * wpf;
    for (int64_t base = 0; base < words && running < total; base += NT) {
        const int64_t i = base + tid;
        const uint32_t frame = fastdiv_div((uint32_t)i, m.wpf_div);
        const uint32_t word = base == 0 ? first_word : i < words ? m.bits[i] : 0u;
        const uint32_t f = base == 0 ? first_id : i < words ? m.frames[frame] : 0u;
        const int first_slot = 32 * (int)((uint32_t)i - frame * (uint32_t)wpf), nb = slots - first_slot;
        const uint32_t freeb = i < words ? ~word & (nb >= 32 ? 0xffffffffu : (1u << nb) - 1u) : 0u;
        const int zeros = __popc(freeb);
        int turn_total;
        const int rank0 = running + block_excl_scan(zeros, turn_total, s_wave);     // rank of this word's first free slot
        if (turn_total == 0) continue;                       // (uniform)
        s_free[tid] = freeb;
        s_rank[tid] = rank0;
        s_id[tid] = f * (uint32_t)slots + (uint32_t)first_slot;
        lds_barrier();
        const int lookups = 32 * (int)(words - base < NT ? words - base : NT);
        const int turn_end = running + turn_total < total ? running + turn_total : total;
        for (int win0 = running; win0 < turn_end; win0 += RESERVE_WIN) {
            const int win1 = win0 + RESERVE_WIN < turn_end ? win0 + RESERVE_WIN : turn_end;
            auto place = [&](int idx, auto count) __attribute__((always_inline)) {       // look-ups idx, idx + NT, ...
                constexpr int N = decltype(count)::value;
                uint32_t fr[N], id[N];
                int first[N];
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    const int j = (idx + u * NT) >> 5;
                    fr[u] = s_free[j];
                    first[u] = s_rank[j];
                    id[u] = s_id[j];
                }
                const int bit = idx & 31;
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    const int r = first[u] + __popc(fr[u] & ((1u << bit) - 1u));
                    if (((fr[u] >> bit) & 1u) && r >= win0 && r < win1) s_blk[r - win0] = id[u] + (uint32_t)bit;
                }
            };
            int from = 0;
            for (; from + 4 * NT <= lookups; from += 4 * NT) place(from + tid, std::integral_constant<int, 4>{});
            for (; from + tid < lookups; from += NT) place(from + tid, std::integral_constant<int, 1>{});
            lds_barrier();
            for (int e = tid / group; e < n; e += NT / group) {
                const int st = s_start[e], en = s_start[e + 1];
                const int lo = st > win0 ? st : win0, hi = en < win1 ? en : win1;
                if (lo >= hi) continue;
                const uint32_t ent = s_ent[e];
                int32_t *row = m.rows + (int64_t)(ent >> 20) * m.max_blocks + (ent & 0xfffffu);
                for (int r = lo + sub; r < hi; r += group) row[r - st] = (int32_t)s_blk[r - win0];
            }
            lds_barrier();
        }
        if (zeros && rank0 < total) {
            const int take = total - rank0;
            uint32_t mask = freeb;                           // the lowest `take` free bits
            if (take < zeros) {
                mask = 0u;
                uint32_t rest = freeb;
                for (int k = 0; k < take; ++k) {
                    mask |= rest & (0u - rest);
                    rest &= rest - 1u;
                }
            }
            m.bits[i] = word | mask;
        }
        running += turn_total;
    }
    __syncthreads();
    for (int s = tid; s < m.max_seqs; s += NT) m.row_len[s] = s_cur[s];
    if (tid == 0) {
        m.counters[1] = spare - total;
        book_finish(res, err, total);
    }
}

constexpr int RELEASE_WIN = 6144;      // words of a model's slot bitmap that k_release collects in LDS at a time

// release (batched): clear the slot bits of every block of the listed rows; the same state as single
// releases in order (a sequence listed twice is empty the second time).
// list: n sequence ids, checked by the host; in the kernel's arguments up to PKV_BOOK_LIST words (reading 32 of them from
// host memory and comparing them pairwise for repetitions took 3 of the kernel's 10.6 us), else in pinned host memory.
__global__ __launch_bounds__(NT) void k_release(PoolDev p, ModelDev m, int n, const int32_t *host_ops, const BookList list,
                                                BookResult *res, uint32_t *err) {
    const int32_t *ops = host_ops ? host_ops : list.v;
    __shared__ int s_wave[NW];
    __shared__ uint32_t s_seen[PKV_MAX_SEQS / 32];
    __shared__ int s_start[PKV_MAX_SEQS + 1];
    __shared__ int s_seq[PKV_MAX_SEQS];
    __shared__ uint32_t s_win[RELEASE_WIN];
    const int tid = threadIdx.x;
    for (int i = tid; i < PKV_MAX_SEQS / 32; i += NT) s_seen[i] = 0u;
    const int64_t words_total = m.counters[0] * m.wpf, spare = m.counters[1];
    // (also where no frame of the model's lies: not looked at then)
    const uint32_t first_word = tid < p.n_frames * m.wpf ? m.bits[tid] : 0u;
    __syncthreads();
    int total = 0;
    for (int c0 = 0; c0 < n; c0 += NT) {
        const int i = c0 + tid;
        int len = 0;
        if (i < n) {
            int s_ = ops[i];
            s_ = (s_ >= 0 && s_ < m.max_seqs) ? s_ : -1;
            // a sequence listed twice is freed once, whichever of its entries does it
            if (s_ >= 0) {
                len = m.row_len[s_];
                if ((atomicOr(&s_seen[s_ >> 5], 1u << (s_ & 31)) >> (s_ & 31)) & 1u) len = 0;
            }
            s_seq[i] = s_;
        }
        int chunk_total;
        const int excl = block_excl_scan(len, chunk_total, s_wave);
        if (i < n) s_start[i] = total + excl;
        total += chunk_total;
    }
    if (tid == 0) s_start[n] = total;
    __syncthreads();
    // Every block costs two dependent reads (its id in the row, then the list position of its frame)
    // before its bit can be cleared; a lane takes RELEASE_BATCH blocks at a time and issues each kind of
    // read for all of them before it needs the first answer, so a pass costs two memory round trips.
    // The bits to clear are collected in LDS, a window of WIN words of the model's slot bitmap at a
    // time (one window covers the bitmap of all but very large models), and each word that lost bits is
    // then rewritten once by one lane: thirty atomics on the same word in memory cost more than the
    // rest of the kernel.
    constexpr int RELEASE_BATCH = 8;
    for (int64_t win0 = 0; win0 < words_total && total > 0; win0 += RELEASE_WIN) {
        for (int i = tid; i < RELEASE_WIN; i += NT) s_win[i] = 0u;
        lds_barrier();
        for (int x0 = 0; x0 < total; x0 += NT * RELEASE_BATCH) {
            uint32_t id[RELEASE_BATCH], frame[RELEASE_BATCH];
            int64_t at[RELEASE_BATCH];
#pragma unroll
            for (int u = 0; u < RELEASE_BATCH; ++u) {
                const int x = x0 + u * NT + tid;
                id[u] = 0xffffffffu;
                if (x < total) {
                    // last entry with s_start <= x (all eight searches at once and the reads behind them: 0.9 us more for
                    // 5411 blocks of 32 rows, 2.7 for 7000 of 64)
                    int lo = 0, hi = n;
                    while (hi - lo > 1) {
                        const int mid = (lo + hi) >> 1;
                        if (s_start[mid] <= x) lo = mid; else hi = mid;
                    }
                    id[u] = (uint32_t)m.rows[(int64_t)s_seq[lo] * m.max_blocks + (x - s_start[lo])];
                }
            }
#pragma unroll
            for (int u = 0; u < RELEASE_BATCH; ++u) {
                frame[u] = fastdiv_div(id[u], m.slots_div);
                at[u] = id[u] != 0xffffffffu ? p.pos[frame[u]] : 0;
            }
#pragma unroll
            for (int u = 0; u < RELEASE_BATCH; ++u)
                if (id[u] != 0xffffffffu) {
                    const uint32_t sl = id[u] - frame[u] * (uint32_t)m.slots;
                    const int64_t word = at[u] * m.wpf + (sl >> 5) - win0;
                    if (word >= 0 && word < RELEASE_WIN) atomicOr(&s_win[word], 1u << (sl & 31));
                }
        }
        lds_barrier();
        for (int i = tid; i < RELEASE_WIN && win0 + i < words_total; i += NT) {
            const uint32_t gone = s_win[i];
            if (gone) m.bits[win0 + i] = (win0 + i == tid ? first_word : m.bits[win0 + i]) & ~gone;
        }
        lds_barrier();
    }
    __syncthreads();
    for (int i = tid; i < n; i += NT)
        if (s_seq[i] >= 0) m.row_len[s_seq[i]] = 0;
    if (tid == 0) {
        m.counters[1] = spare + total;
        book_finish(res, err, total);
    }
}

}  // namespace

hipError_t pkv_launch_pool_init(const PoolDev &p, const uint32_t *perm_dev, hipStream_t s) {
    int blocks = (int)((p.n_frames + 255) / 256);
    if (blocks > 2048) blocks = 2048;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_pool_init, dim3(blocks), dim3(256), 0, s, p, perm_dev);
    return hipGetLastError();
}
hipError_t pkv_launch_resize(const PoolDev &p, const ModelDev &m, int64_t target, BookResult *res, uint32_t *err, hipStream_t s) {
    hipLaunchKernelGGL(k_resize, dim3(1), dim3(NT), 0, s, p, m, target, res, err);
    return hipGetLastError();
}
hipError_t pkv_launch_reserve(const PoolDev &p, const ModelDev &m, int n, const int32_t *ops, const BookList &list, BookResult *res,
                              uint32_t *err, hipStream_t s) {
    hipLaunchKernelGGL(k_reserve, dim3(1), dim3(NT), 0, s, p, m, n, ops, list, res, err);
    return hipGetLastError();
}
hipError_t pkv_launch_release(const PoolDev &p, const ModelDev &m, int n, const int32_t *ops, const BookList &list, BookResult *res,
                              uint32_t *err, hipStream_t s) {
    hipLaunchKernelGGL(k_release, dim3(1), dim3(NT), 0, s, p, m, n, ops, list, res, err);
    return hipGetLastError();
}
