// The write path of the shared pool (gfx950): bulk fill, the decode step's append of one
// new token per sequence, and a read-back in the logical layout.
//
// Paper: Sec. 4.2, D2 — a growing sequence takes its next token block from the slots of
// its model's pages; these kernels put K and V of the new tokens into that block, in the
// operand order the attention kernels read (kv_layout.h).
#include "mfma_util.h"

#include <type_traits>

namespace {

// kv_read: the inverse gather, plus the scale of each token's block.
template <int DT>
__global__ void k_kv_read(AttnDesc d, const int32_t *row, int tok_begin, int n_tok, uint8_t *k, uint8_t *v, float *ks,
                          float *vs) {
    constexpr int E = DT == PKV_BF16 ? 2 : 1;
    const int D = d.D, Hkv = d.Hkv;
    const int64_t total = (int64_t)n_tok * Hkv * D;
    const int64_t idx = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (idx >= total) return;
    const int dd = (int)(idx % D);
    const int h = (int)((idx / D) % Hkv);
    const int ti = (int)(idx / ((int64_t)D * Hkv));
    const int tok = tok_begin + ti;
    const int page = tok / PKV_T, t = tok % PKV_T;
    const uint8_t *blk = block_ptr(d, (uint32_t)row[page]);
    if (DT == PKV_E4M3) {
        if (dd == 0) {
            ks[(size_t)ti * Hkv + h] = reinterpret_cast<const float *>(blk)[h];
            vs[(size_t)ti * Hkv + h] = reinterpret_cast<const float *>(blk)[Hkv + h];
        }
        blk += PKV_FP8_HEADER;
    }
    const size_t tile = (size_t)PKV_T * D * E;
    const uint8_t *kt = blk + (size_t)h * 2 * tile, *vt = kt + tile;
    if (DT == PKV_BF16) {
        reinterpret_cast<uint16_t *>(k)[idx] = reinterpret_cast<const uint16_t *>(kt)[k_elem_off<DT>(t, dd)];
        reinterpret_cast<uint16_t *>(v)[idx] = reinterpret_cast<const uint16_t *>(vt)[v_elem_off<DT>(t, dd)];
    } else {
        k[idx] = kt[k_elem_off<DT>(t, dd)];
        v[idx] = vt[v_elem_off<DT>(t, dd)];
    }
}

// fp32 -> OCP E4M3 code: nearest value, ties to the even code, saturating at 448.
// Integer arithmetic on the bit pattern, so the result does not depend on a rounding
// mode or on how a conversion instruction treats the top of the range.
__device__ __forceinline__ uint32_t e4m3_encode(float y) {
    const uint32_t u = __float_as_uint(y);
    const uint32_t sign = (u >> 24) & 0x80u;
    const uint32_t a = u & 0x7fffffffu;
    if (a > 0x7f800000u) return 0x7fu;                    // NaN
    if (a >= 0x43e00000u) return sign | 0x7eu;            // |y| >= 448
    if (a < 0x3c800000u) {                                // |y| < 2^-6: subnormal codes, step 2^-9
        const float q = rintf(__uint_as_float(a) * 512.0f);   // exact scaling; ties to even
        return sign | (uint32_t)q;                        // 0 .. 8 (8 is the smallest normal)
    }
    uint32_t r = a + 0x7ffffu + ((a >> 20) & 1u);         // round to nearest even at mantissa bit 20
    r >>= 20;                                             // (biased exponent << 3) | 3 mantissa bits
    return sign | (r - ((127u - 7u) << 3));
}

__device__ __forceinline__ float e4m3_decode(uint32_t code) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f32x2 p = __builtin_amdgcn_cvt_pk_f32_fp8((int)code, false);
    return p[0];
}

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = fmaxf(x, __shfl_xor(x, o));
    return x;
}

// One K or V row of an e4m3 model: the running-maximum scale of its (block, kv head),
// re-encoding what the block already holds when the scale grows.  All arithmetic is
// fp32 with IEEE rounding (explicit _rn operations: nothing may be fused or reordered,
// the codes are compared bit for bit).
template <bool IS_V>
__device__ __forceinline__ void append_row_e4m3(uint8_t *tile, float *scale_p, int slot, int D, const uint32_t *x_bf16,
                                                int lane) {
    float x[2];
    float amax = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i) {                          // this lane's elements lane, lane + 64 (0 past the head's width)
        x[i] = __uint_as_float(x_bf16[i] << 16);
        amax = fmaxf(amax, fabsf(x[i]));
    }
    amax = wave_max(amax);
    const float cand = __fdiv_rn(amax, 448.0f);
    float scale;
    if (slot == 0) {
        scale = amax > 0.f ? cand : 1.0f;
    } else {
        scale = *scale_p;
        if (cand > scale) {
            for (int t = 0; t < slot; ++t) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int dd = lane + 64 * i;
                    if (dd < D) {
                        uint8_t *c = tile + (IS_V ? v_elem_off<PKV_E4M3>(t, dd) : k_elem_off<PKV_E4M3>(t, dd));
                        const float v = __fmul_rn(e4m3_decode(*c), scale);
                        *c = (uint8_t)e4m3_encode(__fdiv_rn(v, cand));
                    }
                }
            }
            scale = cand;
        }
    }
    if (lane == 0) *scale_p = scale;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int dd = lane + 64 * i;
        if (dd < D)
            tile[IS_V ? v_elem_off<PKV_E4M3>(slot, dd) : k_elem_off<PKV_E4M3>(slot, dd)] =
                (uint8_t)e4m3_encode(__fdiv_rn(x[i], scale));
    }
}


// ---- whole pages -----------------------------------------------------------------------------------
// One wave writes consecutive tokens of one page (slots s0 .. s0 + n - 1) into the K or the V tile of one kv head, in
// whole 16-byte units.  Lane layout of all of it: token t = lane & 15, column group c = lane >> 4, so that a wave's
// store is one contiguous KiB.  Bound by memory: every byte of the source is read once and every unit written once
// (kv_write of 8192 tokens of 8 heads x 128 in bf16, 67 MB: 32 us element by element with 2-byte stores).  A V unit holds four consecutive
// tokens: the four lanes of a quad hold one token each, and exchange elements by quad broadcasts.

struct PageRows {           // where the tokens come from and go to
    const uint8_t *src;     // first token's row of this head
    size_t stride;          // bytes from token to token
    int s0, n;              // slots written
    bool aligned;           // src may be read in 16-byte pieces
};

// N bytes of slot t's row from byte `at`; a slot that is not written takes the nearest one that is (what it holds is never
// stored), so that all lanes read and no branch parts the requests.
template <int N, int E, bool ALIGNED>
__device__ __forceinline__ void row_bytes(uint32_t *w, const PageRows &p, int t, int at) {
    int r = t - p.s0;
    r = r < 0 ? 0 : (r < p.n ? r : p.n - 1);
    const uint8_t *q = p.src + (size_t)r * p.stride + at;
    if constexpr (ALIGNED) {
        if constexpr (N == 16) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(q);
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = v[i];
        } else if constexpr (N == 8) {
            const u32x2 v = *reinterpret_cast<const u32x2 *>(q);
            w[0] = v.x;
            w[1] = v.y;
        } else {
            w[0] = *reinterpret_cast<const uint32_t *>(q);
        }
    } else {
#pragma unroll
        for (int i = 0; i < N / 4; ++i) w[i] = 0u;
#pragma unroll
        for (int i = 0; i < N / E; ++i) {
            const uint32_t x = E == 2 ? reinterpret_cast<const uint16_t *>(q)[i] : q[i];
            w[i * E / 4] |= x << (8 * (i * E % 4));
        }
    }
}

// The same reads for rows that may be read in 16-byte pieces and for those that may not: read(std::true_type) or (false_type).
template <typename READ>
__device__ __forceinline__ void read_rows(const PageRows &p, const READ &read) {
    if (p.aligned) read(std::true_type{});
    else read(std::false_type{});
}

template <int R>
__device__ __forceinline__ uint32_t quad_bcast(uint32_t x) {          // lane R of the quad, in all four
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, R * 0x55, 0xf, 0xf, true);
}

// Four lanes of a quad hold four bytes each (one token's elements d .. d + 3): lane e receives element d + e of all
// four tokens.  Its own inverse.
__device__ __forceinline__ uint32_t transpose_bytes(uint32_t w, int e) {
    const uint32_t lo = 0x0c0c0400u + (uint32_t)e * 0x0101u, hi = 0x04000c0cu + (uint32_t)e * 0x01010000u;
    return __builtin_amdgcn_perm(quad_bcast<1>(w), quad_bcast<0>(w), lo) | __builtin_amdgcn_perm(quad_bcast<3>(w), quad_bcast<2>(w), hi);
}

// The same for four 16-bit elements in two words.
__device__ __forceinline__ u32x2 transpose_halves(uint32_t w0, uint32_t w1, int e) {
    // (all broadcasts first: a conditional one would run without the lanes it reads from)
    const uint32_t a0 = quad_bcast<0>(w0), a1 = quad_bcast<1>(w0), a2 = quad_bcast<2>(w0), a3 = quad_bcast<3>(w0);
    const uint32_t b0 = quad_bcast<0>(w1), b1 = quad_bcast<1>(w1), b2 = quad_bcast<2>(w1), b3 = quad_bcast<3>(w1);
    const bool up = e & 2;
    const uint32_t z0 = up ? b0 : a0, z1 = up ? b1 : a1, z2 = up ? b2 : a2, z3 = up ? b3 : a3;
    const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
    return mk2(__builtin_amdgcn_perm(z1, z0, sel), __builtin_amdgcn_perm(z3, z2, sel));
}

// A V unit holds the four tokens of slots 4 * group .. + 3; those of slots first .. last - 1 are stored.  A unit that
// is written in part is stored by elements and never read back: another call, on another stream, may be writing the other
// tokens of the group.  e4m3: word u, byte k = token k of element 16 u; bf16: two words, then two words, two tokens each.
template <int E>
__device__ __forceinline__ void put_v_unit(uint8_t *unit, u32x4 v, int group, int first, int last) {
    const int k0 = first - 4 * group, k1 = last - 4 * group;
    if (k0 <= 0 && k1 >= 4) {
        *reinterpret_cast<u32x4 *>(unit) = v;
        return;
    }
    if (k0 >= 4 || k1 <= 0) return;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (k >= k0 && k < k1) {
            if constexpr (E == 2) {
                reinterpret_cast<uint16_t *>(unit)[k] = (uint16_t)(v[k >> 1] >> (16 * (k & 1)));
                reinterpret_cast<uint16_t *>(unit)[4 + k] = (uint16_t)(v[2 + (k >> 1)] >> (16 * (k & 1)));
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) unit[4 * u + k] = (uint8_t)(v[u] >> (8 * k));
            }
        }
}

// The three writers below ask for all of a wave's rows before they ask where the rows go (tile_of(), which waits for a
// block id and may say nowhere): the two trips then overlap.
__device__ __forceinline__ void asked_for() { asm volatile("" ::: "memory"); }      // the compiler would put the reads where they are used

// bf16 values into a bf16 tile
template <int D, bool IS_V, typename TILE_OF>
__device__ __forceinline__ void page_bf16(const TILE_OF &tile_of, const PageRows &p) {
    const int lane = threadIdx.x & 63, t = lane & 15, c = lane >> 4, G = t >> 2, e = t & 3;
    uint32_t w[D / 32][4];
    read_rows(p, [&](auto a) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < D / 32; ++i) {
            if constexpr (!IS_V) {
                row_bytes<16, 2, decltype(a)::value>(w[i], p, t, 16 * (4 * i + c));
            } else {
                row_bytes<8, 2, decltype(a)::value>(w[i], p, t, 2 * (32 * i + 4 * c));
                row_bytes<8, 2, decltype(a)::value>(w[i] + 2, p, t, 2 * (32 * i + 16 + 4 * c));
            }
        }
    });
    asked_for();
    uint8_t *tile = tile_of();
    if (!tile) return;
#pragma unroll
    for (int i = 0; i < D / 32; ++i) {
        if constexpr (!IS_V) {
            if (t >= p.s0 && t < p.s0 + p.n) *reinterpret_cast<u32x4 *>(tile + ((4 * i + c) * 16 + t) * 16) = mk4(w[i][0], w[i][1], w[i][2], w[i][3]);
        } else {
            const u32x2 ta = transpose_halves(w[i][0], w[i][1], e), tb = transpose_halves(w[i][2], w[i][3], e);
            put_v_unit<2>(tile + ((i * 4 + G) * 16 + 4 * c + e) * 16, mk4(ta.x, ta.y, tb.x, tb.y), G, p.s0, p.s0 + p.n);
        }
    }
}

// e4m3 codes as they are into an e4m3 tile
template <int D, bool IS_V, typename TILE_OF>
__device__ __forceinline__ void page_codes(const TILE_OF &tile_of, const PageRows &p) {
    const int lane = threadIdx.x & 63, t = lane & 15, c = lane >> 4, G = t >> 2, e = t & 3;
    uint32_t w[D / 64][4];
    read_rows(p, [&](auto a) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < D / 64; ++j) {
            if constexpr (!IS_V) {
                row_bytes<8, 1, decltype(a)::value>(w[j], p, t, 8 * (8 * j + c));
                row_bytes<8, 1, decltype(a)::value>(w[j] + 2, p, t, 8 * (8 * j + 4 + c));
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u) row_bytes<4, 1, decltype(a)::value>(w[j] + u, p, t, 64 * j + 16 * u + 4 * c);
            }
        }
    });
    asked_for();
    uint8_t *tile = tile_of();
    if (!tile) return;
#pragma unroll
    for (int j = 0; j < D / 64; ++j) {
        if constexpr (!IS_V) {
            if (t >= p.s0 && t < p.s0 + p.n) *reinterpret_cast<u32x4 *>(tile + ((j * 4 + c) * 16 + t) * 16) = mk4(w[j][0], w[j][1], w[j][2], w[j][3]);
        } else {
#pragma unroll
            for (int u = 0; u < 4; ++u) w[j][u] = transpose_bytes(w[j][u], e);
            put_v_unit<1>(tile + ((j * 4 + G) * 16 + 4 * c + e) * 16, mk4(w[j][0], w[j][1], w[j][2], w[j][3]), G, p.s0, p.s0 + p.n);
        }
    }
}

// Four values over one scale as e4m3 codes, bit for bit e4m3_encode(v / scale) with the correctly rounded quotient.
// The quotient is first taken between two products, v * lo and v * hi with lo < 1 / scale < hi (2^-21 either side of
// v_rcp_f32, which is within 2^-23): where both round to the same code the exact quotient does too (rounding is
// monotonic; the conversion instruction equals e4m3_encode for every float below 464 in magnitude: a sweep over all of
// them found no other; the tests compare the codes that calls write with the plain division).  Where they differ, or the code
// is a NaN, or the scale is out of the range in which this holds, the division is done.
struct Divisor {
    float scale, r, lo, hi;
    bool plain;             // the scale is small or large: always divide
};
__device__ __forceinline__ Divisor divisor(float scale) {
    const float r = __builtin_amdgcn_rcpf(scale);
    return Divisor{scale, r, r * (1.0f - 0x1p-21f), r * (1.0f + 0x1p-21f), !(scale > 0x1p-100f && scale < 0x1p100f)};
}
// The correctly rounded quotient of a bf16 value and a scale that is some bf16 value / 448, rounded: a first quotient within
// two units and one correction by its exact remainder (Markstein).  In general the outcome may be a unit off where the exact
// quotient all but lies between two floats; of these quotients, of 8 by 8 digits, none does (all pairs are tried in a test, with
// every reciprocal that v_rcp_f32's error allows).  Signs of zeros are kept: the remainder is taken negative.
__device__ __forceinline__ float quotient(float v, const Divisor &s) {
    const float q = v * s.r;
    return __builtin_fmaf(__builtin_fmaf(q, s.scale, -v), -s.r, q);
}
__device__ __forceinline__ uint32_t pack4(float a, float b, float c, float d) {
    const int x = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
    return (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(c, d, x, true);
}
__device__ __forceinline__ uint32_t divide4(float a, float b, float c, float d, float s) {
    uint32_t z = 0u;
#pragma unroll 1
    for (int k = 0; k < 4; ++k) {                        // (a rare path, which comes up to sixteen times: kept short)
        z = z >> 8 | e4m3_encode(__fdiv_rn(a, s)) << 24;
        a = b;
        b = c;
        c = d;
    }
    return z;
}
constexpr uint32_t SIGNS = 0x80808080u;
__device__ __forceinline__ uint32_t nan_codes(uint32_t w) { return (w & ~SIGNS) + 0x01010101u; }      // sign bit of a byte: its code is a NaN
__device__ __forceinline__ uint32_t encode4(float a, float b, float c, float d, const Divisor &s) {
    const uint32_t x = pack4(a * s.lo, b * s.lo, c * s.lo, d * s.lo), y = pack4(a * s.hi, b * s.hi, c * s.hi, d * s.hi);
    const bool odd = s.plain || x != y || (nan_codes(x) & SIGNS) != 0;
    if (__any(odd)) {
        const uint32_t z = divide4(a, b, c, d, s.scale);
        return odd ? z : x;
    }
    return x;
}

// What a raise of the scale from s to r > s does to a code, encode(decode(c) * s / r), depends on its three mantissa bits
// alone as long as code and outcome are normal numbers: both roundings are to a relative step, whatever the exponent.  The
// code then falls by a number of steps that a table of eight bytes holds (lo: mantissas 0 to 3, hi: 4 to 7), and two raises
// one after the other are one table again.  Four codes at a time, one byte permute.  A byte of `fit` keeps its sign bit
// where the outcome is normal.  With at most 60 steps an entry no byte borrows from the next one; entries above that are
// possible, and then neither result counts: the lane's `far` has been set when the first entry passed 60, stays set, and has all
// its words looked at again.
__device__ __forceinline__ uint32_t lower_codes(uint32_t w, uint32_t lo, uint32_t hi, uint32_t &fit) {
    const uint32_t y = (w | SIGNS) - __builtin_amdgcn_perm(hi, lo, w & 0x07070707u);
    fit &= y - 0x08080808u;
    return (y & ~SIGNS) | (w & SIGNS);
}

// bf16 values into an e4m3 tile under its running scale, with the outcome, bit for bit, of append_row_e4m3 called for
// each token in turn.  The scale after a token is the largest amax / 448 so far, so all 16 are known at once from one
// prefix maximum; a token is encoded under the scale of its own step and then re-encoded at every later step that raises
// the scale (for 16 like tokens between two and three times), by the table of those raises taken together (lower_codes):
// each lane works two entries of its token's table out with the divisions that define it.  Codes that a table does not
// cover (zeros, subnormals, and raises by more than 2^7) are looked at again: of N(0, 1) values one in some ten thousand,
// of rectified or sparse rows, rows with a channel far above the others or tokens that keep growing a good part.  Where few lanes
// hold such codes, the words that do are re-encoded raise by raise.  Where more do, zeros are put back first (no raise changes
// them) and the words left go together, raise by raise: each by itself they are a chain of divisions, which with the table's work
// made such rows slower than no table at all.  8 x 512 tokens of 8 heads x 128, us a call, without a table, each word by itself,
// so: N(0, 1) 25.3, 10.0, 10.1; one channel x 100 26.3, 20.8, 19.7; rectified 24.5, 25.1, 10.6; one value in ten 22.6, 25.7, 10.2;
// each token sqrt 2 times the one before 54.4, 58.2, 50.1; lognormal magnitudes (sigma 1.5) 25.6, 24.4, 22.8.  With all lanes put
// on the second way N(0, 1) takes 10.3; with 8 and 16 lanes as the line rectified rows take 13.4 and 15.3.
// Bound by memory trips and vector instructions alike: 8 x 512 tokens of 8 heads x 128, K and V, us a call: 65 with the
// tokens one after the other, a wave maximum through LDS and two divisions an element each; 22.8 with every raise worked
// out code by code and quotients between two products (1315 vector instructions a wave, half of them for quotients that fall
// on the border of two codes, as two of three waves hold some); 10.0 so (517).
constexpr int FEW_LANES = 4;

template <int D, bool IS_V, typename TILE_OF>
__device__ __forceinline__ void page_quantise(const TILE_OF &tile_of, const PageRows &p) {
    constexpr int NW = D / 16;                           // words of codes per lane
    const int lane = threadIdx.x & 63, t = lane & 15, c = lane >> 4, G = t >> 2, e = t & 3;
    const int s0 = p.s0, end = p.s0 + p.n;
    uint32_t x[2 * NW];                                  // this lane's values, two per word
    read_rows(p, [&](auto a) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < D / 64; ++i) {
            if constexpr (!IS_V) {                       // elements of units (i, c): 8 (8 i + c) .. + 7 and 8 (8 i + 4 + c) .. + 7
                row_bytes<16, 2, decltype(a)::value>(x + 8 * i, p, t, 16 * (8 * i + c));
                row_bytes<16, 2, decltype(a)::value>(x + 8 * i + 4, p, t, 16 * (8 * i + 4 + c));
            } else {                                     // elements 64 i + 16 u + 4 c .. + 3
#pragma unroll
                for (int u = 0; u < 4; ++u) row_bytes<8, 2, decltype(a)::value>(x + 8 * i + 2 * u, p, t, 2 * (64 * i + 16 * u + 4 * c));
            }
        }
    });
    asked_for();
    float *scale_p;
    uint8_t *tile = tile_of(scale_p);
    if (!tile) return;
    // what the tile holds: codes of the slots before
    u32x4 old[D / 64];
    u32x4 *unit = reinterpret_cast<u32x4 *>(tile + (IS_V ? (G * 16 + 4 * c + e) * 16 : (c * 16 + t) * 16));
    if (s0 > 0) {
#pragma unroll
        for (int i = 0; i < D / 64; ++i) old[i] = unit[64 * i];
    }
    const float kept_scale = s0 > 0 ? *scale_p : 1.0f;
    float amax = 0.f;
#pragma unroll
    for (int i = 0; i < 2 * NW; ++i)
        amax = fmaxf(fmaxf(amax, fabsf(__uint_as_float(x[i] << 16))), fabsf(__uint_as_float(x[i] & 0xffff0000u)));
    amax = rows_max(amax);                               // over the four column groups: lanes t, t + 16, t + 32, t + 48
    const float cand = __fdiv_rn(amax, 448.0f);
    // largest candidate up to this token, from the first new one on
    float top = t >= s0 && t < end ? cand : 0.f;
    auto up = [&](float v, int ctrl) __attribute__((always_inline)) {
        int r;
        switch (ctrl) {                                  // row_shr:n, zeros shifted in
            case 1: r = __builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x111, 0xf, 0xf, false); break;
            case 2: r = __builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x112, 0xf, 0xf, false); break;
            case 4: r = __builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x114, 0xf, 0xf, false); break;
            default: r = __builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x118, 0xf, 0xf, false); break;
        }
        return __uint_as_float((uint32_t)r);
    };
    top = fmaxf(top, up(top, 1));
    top = fmaxf(top, up(top, 2));
    top = fmaxf(top, up(top, 4));
    top = fmaxf(top, up(top, 8));
    auto of_lane = [&](float v, int l) __attribute__((always_inline)) {
        return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), l));
    };
    // slot 0 starts afresh: the scale of its token, 1 if that is all zero; else the scale the block has
    const float amax0 = of_lane(amax, 0), start = s0 > 0 ? kept_scale : (amax0 > 0.f ? of_lane(cand, 0) : 1.0f);
    const float scale = top > start ? top : start;       // after this lane's token
    float before = up(scale, 1);
    before = t == s0 ? start : before;
    const uint32_t events = (uint32_t)__ballot(t >= s0 && t > 0 && t < end && scale > before) & 0xffffu;
    const bool raised = events != 0u;

    uint32_t w[NW];
    {
        // a page's first token comes with its scale, so all scales here are bf16 amax / 448 (or 1 = 448 / 448, the scale of zeros);
        // behind tokens that the page holds already it may be any number
        const Divisor own = divisor(scale);
        auto value = [&](int i) __attribute__((always_inline)) { return __uint_as_float((i & 1) ? x[i >> 1] & 0xffff0000u : x[i >> 1] << 16); };
        uint32_t nan = 0u;
        bool plain = s0 > 0 || !(scale > 0x1p-60f && scale < 0x1p100f);
        if (!__any(plain)) {
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                w[i] = pack4(quotient(value(4 * i), own), quotient(value(4 * i + 1), own), quotient(value(4 * i + 2), own),
                             quotient(value(4 * i + 3), own));
                nan |= nan_codes(w[i]);
            }
            plain = (nan & SIGNS) != 0u;
        }
        if (__any(plain)) {
#pragma unroll
            for (int i = 0; i < NW; ++i) w[i] = encode4(value(4 * i), value(4 * i + 1), value(4 * i + 2), value(4 * i + 3), own);
        }
    }
    if (s0 > 0) {
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            uint32_t held = old[i / 4][i & 3];
            if constexpr (IS_V) held = transpose_bytes(held, e);
            w[i] = t < s0 ? held : w[i];
        }
    }
    if (raised) {                                        // wave-uniform
        // entries 2 c and 2 c + 1 of the table of this token's raise, from codes of exponent 14
        uint32_t two = 0u;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const uint32_t mant = 2u * (uint32_t)c + (uint32_t)k;
            const float v = __fmul_rn((float)(128u + 16u * mant), before);
            const uint32_t a = __float_as_uint(__fdiv_rn(v, scale));
            const uint32_t code = ((a + 0x7ffffu + ((a >> 20) & 1u)) >> 20) - ((127u - 7u) << 3);       // e4m3_encode of a normal outcome
            uint32_t steps = (0x70u | mant) - code;
            if (!(before > 0x1p-100f && scale < 0x1p100f) || steps > 60u) steps = 127u;
            two |= steps << (8 * k);
        }
        // all raises behind this lane's token as one table
        uint32_t lo = 0u, hi = 0u, far = 0u;
        for (uint32_t rest = events; rest; rest &= rest - 1u) {       // in the order of the tokens
            const int u = __ffs((int)rest) - 1;
            auto entries = [&](int l) __attribute__((always_inline)) { return (uint32_t)__builtin_amdgcn_readlane((int)two, l); };
            const uint32_t d0 = entries(u) | entries(u + 16) << 16, d1 = entries(u + 32) | entries(u + 48) << 16;
            const uint32_t lo_n = lo + __builtin_amdgcn_perm(d1, d0, (0x83828180u - lo) & 0x07070707u);
            const uint32_t hi_n = hi + __builtin_amdgcn_perm(d1, d0, (0x87868584u - hi) & 0x07070707u);
            if (t < u) {
                lo = lo_n;
                hi = hi_n;
                far |= (lo_n + 0x43434343u) | (hi_n + 0x43434343u);   // sign bit: more than 60 steps
            }
        }
        // a token of zeros stays as it is; any other code that the table does not cover is looked at again
        const bool zeros = t >= s0 && !(amax > 0.f);
        const bool lowered = t < 31 - __clz((int)events) && !zeros;
        if (zeros) lo = hi = 0u;
        uint32_t low[NW], fit = SIGNS, nan = 0u;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            low[i] = lower_codes(w[i], lo, hi, fit);
            nan |= nan_codes(w[i]);
        }
        auto uncovered = [&](uint32_t f, uint32_t n) __attribute__((always_inline)) { return __ballot(lowered && ((far | n | ~f) & SIGNS) != 0u); };
        auto each_raise = [&](const auto &f) __attribute__((always_inline)) {
            for (uint32_t rest = events; rest; rest &= rest - 1u) {
                const int u = __ffs((int)rest) - 1;
                f(u, of_lane(before, u), divisor(of_lane(scale, u)));
            }
        };
        auto again = [&](uint32_t x, int u, float was, const Divisor &now) __attribute__((always_inline)) {
            const f32x2 l2 = __builtin_amdgcn_cvt_pk_f32_fp8((int)x, false), h2 = __builtin_amdgcn_cvt_pk_f32_fp8((int)x, true);
            const uint32_t z = encode4(__fmul_rn(l2[0], was), __fmul_rn(l2[1], was), __fmul_rn(h2[0], was), __fmul_rn(h2[1], was), now);
            return t < u ? z : x;
        };
        const uint64_t missed = uncovered(fit, nan);
        if (missed != 0u && __popcll(missed) < FEW_LANES) {
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                uint32_t f = SIGNS;
                (void)lower_codes(w[i], lo, hi, f);
                if (uncovered(f, nan_codes(w[i])) == 0u) continue;
                low[i] = w[i];
                each_raise([&](int u, float was, const Divisor &now) __attribute__((always_inline)) { low[i] = again(low[i], u, was, now); });
            }
        } else if (missed != 0u) {
            uint32_t todo = 0u;
#pragma unroll
            for (int i = 0; i < NW; ++i) {
                const uint32_t zero = ~((w[i] & ~SIGNS) + 0x7f7f7f7fu) & SIGNS, same = (zero >> 7) * 0xffu;
                uint32_t f = SIGNS;
                (void)lower_codes(w[i], lo, hi, f);
                low[i] = (low[i] & ~same) | (w[i] & same);
                if (uncovered(f | zero, nan_codes(w[i])) != 0u) {
                    low[i] = w[i];
                    todo |= 1u << i;
                }
            }
            if (todo)
                each_raise([&](int u, float was, const Divisor &now) __attribute__((always_inline)) {
#pragma unroll
                    for (int i = 0; i < NW; ++i)
                        if (todo >> i & 1u) low[i] = again(low[i], u, was, now);
                });
        }
#pragma unroll
        for (int i = 0; i < NW; ++i) w[i] = low[i];
    }
    if (lane == 0) *scale_p = of_lane(scale, end - 1);
    const int first = raised ? 0 : s0;                   // slots below it still hold what memory holds
#pragma unroll
    for (int i = 0; i < D / 64; ++i) {
        if constexpr (!IS_V) {
            if (t >= first && t < end) unit[64 * i] = mk4(w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]);
        } else {
            const u32x4 v = mk4(transpose_bytes(w[4 * i], e), transpose_bytes(w[4 * i + 1], e), transpose_bytes(w[4 * i + 2], e),
                          transpose_bytes(w[4 * i + 3], e));
            put_v_unit<1>(reinterpret_cast<uint8_t *>(unit + 64 * i), v, G, first, end);
        }
    }
}

// One wave's share of a page: the K (which = 0) or V (1) tile of kv head h.  QUANT: bf16 values into an e4m3 block.
// block_of(): the block, or NULL where nothing may be written.
template <int DT, bool QUANT, typename BLOCK_OF>
__device__ __forceinline__ void page_tile(const AttnDesc &d, const BLOCK_OF &block_of, int h, int which, const PageRows &p) {
    constexpr int E = DT == PKV_BF16 ? 2 : 1;
    const size_t offset = (DT == PKV_E4M3 ? PKV_FP8_HEADER : 0) + ((size_t)h * 2 + which) * PKV_T * d.D * E;
    auto go = [&](auto dim, auto is_v) __attribute__((always_inline)) {
        constexpr int D = decltype(dim)::value;
        constexpr bool IS_V = decltype(is_v)::value;
        auto tile_of = [&]() __attribute__((always_inline)) {
            uint8_t *blk = block_of();
            return blk ? blk + offset : blk;
        };
        if constexpr (DT == PKV_BF16) page_bf16<D, IS_V>(tile_of, p);
        else if constexpr (!QUANT) page_codes<D, IS_V>(tile_of, p);
        else
            page_quantise<D, IS_V>([&](float *&scale_p) __attribute__((always_inline)) {
                uint8_t *blk = block_of();
                scale_p = reinterpret_cast<float *>(blk) + (IS_V ? d.Hkv : 0) + h;
                return blk ? blk + offset : blk;
            }, p);
    };
    if (d.D == 128) {
        if (which) go(std::integral_constant<int, 128>{}, std::true_type{});
        else go(std::integral_constant<int, 128>{}, std::false_type{});
    } else {
        if (which) go(std::integral_constant<int, 64>{}, std::true_type{});
        else go(std::integral_constant<int, 64>{}, std::false_type{});
    }
}

constexpr int PAGE_WAVES = 4;       // waves of a work-group; wave x of the launch: K or V, kv head, page, fastest first

// kv_write: logical [n_tok][Hkv][D] values (bf16) or codes with their scales (e4m3) -> the in-block operand layouts.
// Rows first, then the block: us a launch on 8 x 128 heads, element loops that wait for the block first and now: one token 3.3 ->
// 2.6 bf16, 3.3 -> 2.4 e4m3, 8192 bf16 tokens 11.8 -> 12.0, 16000 21.0 -> 21.5, 32000 49.7 -> 39.6.  All arguments at once pay off
// for bf16 and for few e4m3 tokens (0.1 us), but cost many e4m3 tokens more than they had gained: 8192 10.0 and 9.6 without, 12000 14.1
// and 12.5 (13.0 before), 32000 28.5 and 26.8.
template <int DT>
__global__ __launch_bounds__(64 * PAGE_WAVES) void k_kv_write(const AttnDesc d, const int32_t *row, int tok_begin, int n_tok,
                                                              const uint8_t *k, const uint8_t *v, const float *ks, const float *vs) {
    constexpr int E = DT == PKV_BF16 ? 2 : 1;
    if constexpr (DT == PKV_BF16) {                        // (e4m3: see above)
        ask_arguments(d, k, v);
        asm volatile("" ::"s"(row), "s"(tok_begin), "s"(n_tok));
    }
    const int x = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * PAGE_WAVES + (threadIdx.x >> 6)));
    const int which = x & 1, hp = x >> 1, j = hp / d.Hkv, h = hp - j * d.Hkv;
    const int page = tok_begin / PKV_T + j, end = tok_begin + n_tok;
    const int lo = page * PKV_T > tok_begin ? page * PKV_T : tok_begin, hi = (page + 1) * PKV_T < end ? (page + 1) * PKV_T : end;
    if (lo >= hi) return;
    const uint32_t id = (uint32_t)PKV_CONST(int32_t, row)[page];
    const uint8_t *src = which ? v : k;
    PageRows p;
    p.stride = (size_t)d.Hkv * d.D * E;
    p.src = src + (size_t)(lo - tok_begin) * p.stride + (size_t)h * d.D * E;
    p.s0 = lo % PKV_T;
    p.n = hi - lo;
    p.aligned = (reinterpret_cast<uintptr_t>(src) & 15) == 0;
    float scale = 0.f;
    if (DT == PKV_E4M3) scale = (which ? vs : ks)[(size_t)j * d.Hkv + h];
    page_tile<DT, false>(d, [&]() __attribute__((always_inline)) {
        uint8_t *blk = block_ptr(d, id);
        if (DT == PKV_E4M3 && (threadIdx.x & 63) == 0) reinterpret_cast<float *>(blk)[(which ? d.Hkv : 0) + h] = scale;
        return blk;
    }, h, which, p);
}

// kv_append, the decode step: one wave per (sequence, kv head) writes the token with index ctx_lens[seq] - 1 from row
// `seq` of k_new / v_new (bf16 [batch][Hkv][D]).  A context length outside what the row holds is skipped and reported
// through the device error flags (bit 1).
template <int DT>
__global__ __launch_bounds__(64) void k_kv_append(const AttnDesc d, const uint16_t *k_new, const uint16_t *v_new) {
    const int lane = threadIdx.x;
    ask_arguments(d, k_new, v_new);
    const int seq = blockIdx.x / d.Hkv, h = blockIdx.x - seq * d.Hkv;
    const int D = d.D;
    // The new token's values are asked for along with the context length: the launch is bound by its dependent memory
    // trips (context length, block id, the block), not by what it moves.
    const size_t src = ((size_t)seq * d.Hkv + h) * D + lane;
    const size_t second = src + (D > 64 ? 64 : 0);         // (no branch: it would wait for the first loads)
    uint32_t kx[2] = {k_new[src], k_new[second]}, vx[2] = {v_new[src], v_new[second]};
    asm volatile("" ::: "memory");                         // issued here: the compiler would put them where they are used
    const int ctx = PKV_CONST(int32_t, d.ctx_lens)[seq];
    const int cap = PKV_CONST(int32_t, d.row_len)[seq] * PKV_T;
    if ((ctx < 1) | (ctx > cap)) {
        if (lane == 0) atomicOr(d.err, 2u);
        return;
    }
    const uint32_t id = (uint32_t)PKV_CONST(int32_t, d.table)[(size_t)seq * d.row_stride + (ctx - 1) / PKV_T];
    if (id >= d.max_block_id) {
        if (lane == 0) atomicOr(d.err, 1u);
        return;
    }
    uint8_t *blk = block_ptr(d, id);
    const int slot = (ctx - 1) % PKV_T;
    if (DT == PKV_BF16) {
        const size_t tile = (size_t)PKV_T * D * 2;
        uint16_t *kt = reinterpret_cast<uint16_t *>(blk + (size_t)h * 2 * tile);
        uint16_t *vt = reinterpret_cast<uint16_t *>(blk + (size_t)h * 2 * tile + tile);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int dd = lane + 64 * i;
            if (dd < D) {
                kt[k_elem_off<PKV_BF16>(slot, dd)] = (uint16_t)kx[i];
                vt[v_elem_off<PKV_BF16>(slot, dd)] = (uint16_t)vx[i];
            }
        }
    } else {
        float *hdr = reinterpret_cast<float *>(blk);
        const size_t tile = (size_t)PKV_T * D;
        uint8_t *kt = blk + PKV_FP8_HEADER + (size_t)h * 2 * tile, *vt = kt + tile;
        if (D == 64) kx[1] = vx[1] = 0u;
        append_row_e4m3<false>(kt, hdr + h, slot, D, kx, lane);
        append_row_e4m3<true>(vt, hdr + d.Hkv + h, slot, D, vx, lane);
    }
}

// kv_append_chunk: the sequence's new tokens, at indices ctx_lens[seq] - tokens .. ctx_lens[seq] - 1, come from
// consecutive rows, each written exactly as a single append would; one wave per (sequence, j-th page the chunk touches,
// kv head, K or V).  Where the chunk starts is known only here (ctx_lens is device data), so the plan has one page more
// than the chunk can touch and a wave whose page holds none of the chunk leaves.  Tokens of one page go in order (the
// e4m3 scale rule is sequential within a block by definition); pages do not depend on each other (a block's scale
// starts afresh at its first slot).
template <int DT, int SEQS>
__global__ __launch_bounds__(64 * PAGE_WAVES) void k_kv_append_chunk(const AttnDesc d, const PlanOf<SEQS> plan, const uint16_t *k_new,
                                                                     const uint16_t *v_new) {
    const int lane = threadIdx.x & 63;
    const PlanLanes<SEQS> lanes(plan);
    ask_arguments(d, k_new, v_new);
    asm volatile("" ::"s"(plan.n_seqs), "s"(plan.seq0));
    const int x = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * PAGE_WAVES + (threadIdx.x >> 6)));
    const int which = x & 1, hp = x >> 1, unit = hp / d.Hkv, h = hp - unit * d.Hkv;
    if ((uint32_t)unit >= lanes.units(plan)) return;                 // the last work-group may have waves to spare
    const PlanUnit pu = lanes.find(plan, (uint32_t)unit);
    const int ctx = PKV_CONST(int32_t, d.ctx_lens)[pu.seq], cap = PKV_CONST(int32_t, d.row_len)[pu.seq] * PKV_T;
    if ((ctx < pu.rows) | (ctx < 1) | (ctx > cap)) {
        if (lane == 0) atomicOr(d.err, 2u);
        return;
    }
    const int tok0 = ctx - pu.rows, page = tok0 / PKV_T + pu.unit;
    const int lo = tok0 > page * PKV_T ? tok0 : page * PKV_T, hi = ctx < (page + 1) * PKV_T ? ctx : (page + 1) * PKV_T;
    if (lo >= hi) return;
    const uint32_t id = (uint32_t)PKV_CONST(int32_t, d.table)[(size_t)pu.seq * d.row_stride + page];
    const uint16_t *src = which ? v_new : k_new;
    PageRows p;
    p.stride = (size_t)d.Hkv * d.D * 2;
    p.src = reinterpret_cast<const uint8_t *>(src) + (size_t)(pu.row + (lo - tok0)) * p.stride + (size_t)h * d.D * 2;
    p.s0 = lo % PKV_T;
    p.n = hi - lo;
    p.aligned = (reinterpret_cast<uintptr_t>(src) & 15) == 0;
    page_tile<DT, true>(d, [&]() __attribute__((always_inline)) -> uint8_t * {
        if (id >= d.max_block_id) {
            if (lane == 0) atomicOr(d.err, 1u);
            return nullptr;
        }
        return block_ptr(d, id);
    }, h, which, p);
}

}  // namespace

hipError_t pkv_launch_kv_write(const AttnDesc &d, int seq, int tok_begin, int n_tok, const void *k, const void *v,
                               const float *ks, const float *vs, int page_tokens, hipStream_t s) {
    (void)page_tokens;
    if (n_tok == 0) return hipSuccess;
    const int32_t *row = d.table + (size_t)seq * d.row_stride;
    const int pages = (tok_begin + n_tok - 1) / PKV_T - tok_begin / PKV_T + 1;
    const unsigned waves = (unsigned)pages * (unsigned)d.Hkv * 2u, blocks = (waves + PAGE_WAVES - 1) / PAGE_WAVES;
    if (d.dtype == PKV_BF16)
        hipLaunchKernelGGL(k_kv_write<PKV_BF16>, dim3(blocks), dim3(64 * PAGE_WAVES), 0, s, d, row, tok_begin, n_tok,
                           (const uint8_t *)k, (const uint8_t *)v, ks, vs);
    else
        hipLaunchKernelGGL(k_kv_write<PKV_E4M3>, dim3(blocks), dim3(64 * PAGE_WAVES), 0, s, d, row, tok_begin, n_tok,
                           (const uint8_t *)k, (const uint8_t *)v, ks, vs);
    return hipGetLastError();
}

hipError_t pkv_launch_kv_read(const AttnDesc &d, int seq, int tok_begin, int n_tok, void *k, void *v, float *ks, float *vs,
                              hipStream_t s) {
    const int64_t total = (int64_t)n_tok * d.Hkv * d.D;
    if (total == 0) return hipSuccess;
    const int32_t *row = d.table + (size_t)seq * d.row_stride;
    const unsigned blocks = (unsigned)((total + 255) / 256);
    if (d.dtype == PKV_BF16)
        hipLaunchKernelGGL(k_kv_read<PKV_BF16>, dim3(blocks), dim3(256), 0, s, d, row, tok_begin, n_tok, (uint8_t *)k,
                           (uint8_t *)v, ks, vs);
    else
        hipLaunchKernelGGL(k_kv_read<PKV_E4M3>, dim3(blocks), dim3(256), 0, s, d, row, tok_begin, n_tok, (uint8_t *)k,
                           (uint8_t *)v, ks, vs);
    return hipGetLastError();
}

hipError_t pkv_launch_kv_append(const AttnDesc &d, const void *k_new, const void *v_new, hipStream_t s) {
    if (d.batch == 0) return hipSuccess;
    const unsigned blocks = (unsigned)(d.batch * d.Hkv);
    if (d.dtype == PKV_BF16)
        hipLaunchKernelGGL(k_kv_append<PKV_BF16>, dim3(blocks), dim3(64), 0, s, d, (const uint16_t *)k_new,
                           (const uint16_t *)v_new);
    else
        hipLaunchKernelGGL(k_kv_append<PKV_E4M3>, dim3(blocks), dim3(64), 0, s, d, (const uint16_t *)k_new,
                           (const uint16_t *)v_new);
    return hipGetLastError();
}

hipError_t pkv_launch_kv_append_chunk(const AttnDesc &d, const ChunkPlan &plan, const void *k_new, const void *v_new, hipStream_t s) {
    const unsigned waves = plan.s[plan.n_seqs].unit * (unsigned)d.Hkv * 2u, blocks = (waves + PAGE_WAVES - 1) / PAGE_WAVES;
    if (blocks == 0) return hipSuccess;
    const dim3 grid(blocks), wg(64 * PAGE_WAVES);
    const uint16_t *k = (const uint16_t *)k_new, *v = (const uint16_t *)v_new;
    if (plan.n_seqs <= PKV_PLAN_FEW) {
        if (d.dtype == PKV_BF16) hipLaunchKernelGGL((k_kv_append_chunk<PKV_BF16, PKV_PLAN_FEW>), grid, wg, 0, s, d, few_of(plan), k, v);
        else hipLaunchKernelGGL((k_kv_append_chunk<PKV_E4M3, PKV_PLAN_FEW>), grid, wg, 0, s, d, few_of(plan), k, v);
    } else {
        if (d.dtype == PKV_BF16) hipLaunchKernelGGL((k_kv_append_chunk<PKV_BF16, PKV_PLAN_SEQS>), grid, wg, 0, s, d, plan, k, v);
        else hipLaunchKernelGGL((k_kv_append_chunk<PKV_E4M3, PKV_PLAN_SEQS>), grid, wg, 0, s, d, plan, k, v);
    }
    return hipGetLastError();
}
