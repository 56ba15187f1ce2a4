// usp_device.h -- device code that the kernels of the library share: the decode
// of a tile record into MFMA operands, the fused epilogue and output stores, the
// arrival protocol of split row sets, and record transfers into LDS.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "usp_internal.h"

namespace usp {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t v4u32 __attribute__((ext_vector_type(4)));

// Word 3 of a raw buffer resource on gfx9-class targets (untyped 32-bit data).
constexpr int kBufferRsrcWord3 = 0x00020000;
// Cache policy of loads whose data is used once (the non-temporal bit): tile
// records read by a single wavefront. They then no longer push X, which every
// unit re-reads, out of L2: the 70B FFN layer at 16 tokens takes 57.2 instead of
// 59.2 us, 13B attention 12.6 instead of 13.2. Records that several token
// groups read in turn keep the default policy, which lets the later groups find
// them in L2 (128 tokens: 166 against 170 us with the bit set).
constexpr int kCachePolicyStream = 2;
// Cache policy with the device-scope bit (sc1): coherent across the XCDs' L2s.
constexpr int kCachePolicyDevice = 16;

// Rows m .. m + 3 of the bias or of a token's residual (m a multiple of 4), those
// < M; vec: 8-byte aligned. Requested ahead of what they are added to (a split
// row set's partials), so that their latency is not paid after it.
__device__ inline uint2 load_quad(const uint16_t *p, int64_t m, int64_t M, bool vec) {
    if (!p) return make_uint2(0, 0);
    if (vec && m + 4 <= M) return *reinterpret_cast<const uint2 *>(p + m);
    const uint32_t h0 = m < M ? p[m] : 0, h1 = m + 1 < M ? p[m + 1] : 0;
    const uint32_t h2 = m + 2 < M ? p[m + 2] : 0, h3 = m + 3 < M ? p[m + 3] : 0;
    return make_uint2(h0 | (h1 << 16), h2 | (h3 << 16));
}
template <class Args>
__device__ inline uint2 bias_quad(const Args &a, int64_t m) {
    return load_quad(a.bias, m, a.M, a.e_flags & kEpiBiasVec);
}
template <class Args>
__device__ inline uint2 residual_quad(const Args &a, int n, int64_t m) {
    return load_quad(a.res ? a.res + (int64_t)n * a.ldr : nullptr, m, a.M, a.e_flags & kEpiResVec);
}

__device__ inline floatx4 add_quad(floatx4 v, uint2 q) {
    typedef _Float16 half2 __attribute__((ext_vector_type(2)));
    const half2 lo = __builtin_bit_cast(half2, q.x), hi = __builtin_bit_cast(half2, q.y);
    return floatx4{v[0] + (float)lo[0], v[1] + (float)lo[1], v[2] + (float)hi[0], v[3] + (float)hi[1]};
}

// The fused epilogue of four outputs, in fp32: + bias, the activation, +
// residual. The branches are on arguments, so uniform.
template <class Args>
__device__ inline floatx4 epilogue(const Args &a, floatx4 v, uint2 bias, uint2 res) {
    if (a.bias) v = add_quad(v, bias);
    if (a.act == 1) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = v[i] > 0.f ? v[i] : 0.f;
    } else if (a.act == 2) {  // tanh form of GELU; sqrt(2 / pi) = 0.7978845608...
#pragma unroll
        for (int i = 0; i < 4; ++i)
            v[i] = 0.5f * v[i] * (1.f + tanhf(0.7978845608028654f * (v[i] + 0.044715f * v[i] * v[i] * v[i])));
    } else if (a.act == 3) {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = v[i] / (1.f + expf(-v[i]));
    }
    if (a.res) v = add_quad(v, res);
    return v;
}

template <class Args>
__device__ inline bool has_epilogue(const Args &a) {
    return a.e_flags & kEpiAny;
}

// Rows m .. m + 3 of token n, rounded to fp16, those < M.
template <class Args>
__device__ inline void store_rounded4(const Args &a, int n, int64_t m, floatx4 v) {
    const uint16_t h0 = __builtin_bit_cast(uint16_t, (_Float16)v[0]);
    const uint16_t h1 = __builtin_bit_cast(uint16_t, (_Float16)v[1]);
    const uint16_t h2 = __builtin_bit_cast(uint16_t, (_Float16)v[2]);
    const uint16_t h3 = __builtin_bit_cast(uint16_t, (_Float16)v[3]);
    uint16_t *dst = a.Y + (int64_t)n * a.ldy + m;
    if (a.y_vec && m + 4 <= a.M) {
        *reinterpret_cast<uint2 *>(dst) = make_uint2(h0 | ((uint32_t)h1 << 16), h2 | ((uint32_t)h3 << 16));
    } else {
        if (m < a.M) dst[0] = h0;
        if (m + 1 < a.M) dst[1] = h1;
        if (m + 2 < a.M) dst[2] = h2;
        if (m + 3 < a.M) dst[3] = h3;
    }
}

// The same after the fused epilogue, if any, its operands at hand or read here.
template <class Args>
__device__ inline void store_rows4(const Args &a, int n, int64_t m, floatx4 v, uint2 bias, uint2 res) {
    if (has_epilogue(a)) v = epilogue(a, v, bias, res);
    store_rounded4(a, n, m, v);
}
template <class Args>
__device__ inline void store_rows4(const Args &a, int n, int64_t m, floatx4 v) {
    if (has_epilogue(a)) v = epilogue(a, v, bias_quad(a, m), residual_quad(a, n, m));
    store_rounded4(a, n, m, v);
}

// How a kernel's stores take the fused epilogue.
enum EpilogueMode {
    kEpiNone,    // not at all: the kernel runs for calls without one
    kEpiInline,  // operands read as they are used
    kEpiAhead,   // operands requested for several outputs first, and before a split row set's partials
};

// Selector pair for expanding nibble `n` (positions 0..3) from the 4 packed
// halfs (c0,c1 | c2,c3) held in x0 | x1: output half j takes c_rank(j) when bit
// j is set and zero (selector byte 0x0c) otherwise.
__device__ inline uint2 nibble_selectors(uint32_t n) {
    uint32_t sel[2] = {0x0c0c0c0cu, 0x0c0c0c0cu};
    uint32_t r = 0;
    for (int j = 0; j < 4; ++j) {
        if (n & (1u << j)) {
            const uint32_t pair = (2 * r) | ((2 * r + 1) << 8);
            const int sh = 16 * (j & 1);
            sel[j >> 1] = (sel[j >> 1] & ~(0xFFFFu << sh)) | (pair << sh);
            ++r;
        }
    }
    return make_uint2(sel[0], sel[1]);
}

// The LDS words one step's decode needs: for each of the two nibbles, the three
// dwords holding its packed values and its selector pair, plus the byte
// offsets of both starts. Reading them for step s + 1 before finishing step s
// hides the LDS latency.
struct StepWords {
    uint32_t e[6];
    uint2 sel[2];
    uint32_t hb[2];
};

typedef const __attribute__((address_space(3))) uint32_t lds_u32;

// An LDS array seen as 32-bit words. Indexing the array itself (rather than an
// integer address) lets the compiler tell LDS arrays apart, which its waits for
// direct-to-LDS loads rely on.
__device__ inline lds_u32 *as_lds(const void *p) {
    return (lds_u32 *)(const __attribute__((address_space(3))) void *)p;
}

// region: the staged values. hb is the nibble's first byte (even); the three
// dwords from its dword hold its up to 4 values whatever its alignment. A read
// may run up to 12 bytes past the record's values, which every region leaves
// room for.
__device__ inline void read_nibble(lds_u32 *region, uint32_t hb, uint32_t idx8, const uint8_t *lut,
                                   uint32_t *e, uint2 &sel) {
    typedef const __attribute__((address_space(3))) uint8_t lds_u8;
    typedef volatile const __attribute__((address_space(3))) uint32_t lds_vu32;
    lds_vu32 *d = (lds_vu32 *)((lds_u8 *)region + (hb & ~3u));
    e[0] = d[0];
    e[1] = d[1];
    e[2] = d[2];
    sel = *reinterpret_cast<const uint2 *>(lut + idx8);
}

// Expands one nibble whose packed values start at byte hb (even) from its three
// dwords: a funnel shift aligns the 4 candidate halfs, then two byte permutes
// place them (or zeros) at the nibble's 4 positions.
__device__ inline void finish_nibble(const uint32_t *e, uint2 sel, uint32_t hb, uint32_t &o0, uint32_t &o1) {
    const uint32_t x0 = __builtin_amdgcn_alignbyte(e[1], e[0], hb);  // uses hb & 3 (0 or 2)
    const uint32_t x1 = __builtin_amdgcn_alignbyte(e[2], e[1], hb);
    o0 = __builtin_amdgcn_perm(x1, x0, sel.x);
    o1 = __builtin_amdgcn_perm(x1, x0, sel.y);
}

// Inclusive prefix sum over the 64 lanes of a wavefront (DPP row shifts and
// row broadcasts, 6 adds).
__device__ inline uint32_t wave_inclusive_scan(uint32_t v) {
    v += __builtin_amdgcn_update_dpp(0u, v, 0x111, 0xF, 0xF, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0u, v, 0x112, 0xF, 0xF, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0u, v, 0x114, 0xF, 0xF, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0u, v, 0x118, 0xF, 0xF, true);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0u, v, 0x142, 0xA, 0xF, false);  // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0u, v, 0x143, 0xC, 0xF, false);  // row_bcast:31
    return v;
}

// Number of set bits of each 4-bit nibble of x, one count per nibble.
__device__ inline uint32_t nibble_popcounts(uint32_t x) {
    x = x - ((x >> 1) & 0x55555555u);
    return (x & 0x33333333u) + ((x >> 2) & 0x33333333u);
}

// Per-record decode state of one lane, from its mask word (byte s = step s).
// The record's values are 16 blocks, b = 2 s + h for step s and nibble half h
// (h = 0: positions 0-3, h = 1: positions 4-7), each holding the 64 lanes'
// values of that nibble in lane order. A lane's nibble (s, h) therefore starts
// at the block's start plus the lane's exclusive prefix of the block's kept
// counts: four DPP scans over 8-bit fields give every lane its prefix for all
// 16 blocks (at most 63 x 4 = 252, so the fields never carry), and lane 63's
// prefix plus its own count gives each block's size.
struct RecState {
    uint32_t excl[4];            // prefixes: [2 (s / 4) + h], field s % 4
    uint32_t base2[2 * kSteps];  // byte offset of block b (wavefront-uniform)
    uint32_t t[4];               // selector-table offsets (nibble x 8): [2 (s / 4) + h], byte s % 4
};

// start: LDS byte offset of the record's values from the region that read_step
// is given (a multiple of 4).
__device__ inline RecState rec_state(uint2 msk, uint32_t start = 0) {
    const uint32_t nx = nibble_popcounts(msk.x), ny = nibble_popcounts(msk.y);
    const uint32_t w[4] = {nx & 0x0F0F0F0Fu, (nx >> 4) & 0x0F0F0F0Fu, ny & 0x0F0F0F0Fu, (ny >> 4) & 0x0F0F0F0Fu};
    RecState o;
    uint32_t tot[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t inc = wave_inclusive_scan(w[i]);
        asm("" : "+v"(inc));     // keeps the scan's last add a DPP add (the optimizer would split it)
        o.excl[i] = inc - w[i];  // exact: lane 63's inclusive sum may carry, the difference does not
        // Block sizes: lane 63's prefix plus its own count, per field (up to 256), in 16-bit halves.
        const uint32_t x = __builtin_amdgcn_readlane(o.excl[i], 63), c = __builtin_amdgcn_readlane(w[i], 63);
        const uint32_t even = (x & 0x00FF00FFu) + (c & 0x00FF00FFu), odd = ((x >> 8) & 0x00FF00FFu) + ((c >> 8) & 0x00FF00FFu);
        tot[i][0] = even & 0xFFFFu;
        tot[i][1] = odd & 0xFFFFu;
        tot[i][2] = even >> 16;
        tot[i][3] = odd >> 16;
    }
    uint32_t run = 0;
#pragma unroll
    for (int st = 0; st < kSteps; ++st) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            o.base2[2 * st + h] = start + 2 * run;
            run += tot[2 * (st >> 2) + h][st & 3];
        }
    }
    uint32_t t0 = (msk.x << 3) & 0x78787878u, t1 = (msk.x >> 1) & 0x78787878u;
    uint32_t t2 = (msk.y << 3) & 0x78787878u, t3 = (msk.y >> 1) & 0x78787878u;
    // Opaque to the optimizer: a step's selector index is then one bit-field
    // extract of these words instead of a shift and a mask of the raw mask.
    asm("" : "+v"(t0), "+v"(t1), "+v"(t2), "+v"(t3));
    o.t[0] = t0;
    o.t[1] = t1;
    o.t[2] = t2;
    o.t[3] = t3;
    return o;
}

// Issues the LDS reads of step s of the staged record.
__device__ inline StepWords read_step(lds_u32 *region, const uint8_t *lut, const RecState &rs, int s) {
    StepWords w;
    const int f = 8 * (s & 3), q = 2 * (s >> 2);
    w.hb[0] = 2 * ((rs.excl[q] >> f) & 0xFFu) + rs.base2[2 * s];
    w.hb[1] = 2 * ((rs.excl[q + 1] >> f) & 0xFFu) + rs.base2[2 * s + 1];
    read_nibble(region, w.hb[0], (rs.t[q] >> f) & 0xFFu, lut, w.e, w.sel[0]);
    read_nibble(region, w.hb[1], (rs.t[q + 1] >> f) & 0xFFu, lut, w.e + 3, w.sel[1]);
    return w;
}

// The A operand (8 halfs) of a step from its LDS words.
__device__ inline half8 finish_step(const StepWords &w) {
    uint4 a;
    finish_nibble(w.e, w.sel[0], w.hb[0], a.x, a.y);
    finish_nibble(w.e + 3, w.sel[1], w.hb[1], a.z, a.w);
    return __builtin_bit_cast(half8, a);
}

__device__ inline half8 decode_step(lds_u32 *region, const uint8_t *lut, const RecState &rs, int s) {
    return finish_step(read_step(region, lut, rs, s));
}

// X[0 .. 7] of a token row at any 2-byte alignment, zeros from element `left` on
// (left >= 1). A whole chunk takes two loads that need 4-byte alignment and four
// funnel shifts; only dwords that hold some of it are read. (Eight 2-byte loads
// took the ragged 4999 x 4093 layer at 21 tokens 21.8 us on the four-wavefront
// kernel.)
__device__ inline v4u32 load_x8(const uint16_t *__restrict__ x, int64_t left) {
    typedef v4u32 __attribute__((aligned(4))) v4u32_a4;
    if (left >= 8) {
        const uint32_t sh = (uint32_t)(reinterpret_cast<uintptr_t>(x) & 2);
        const uint32_t *p = reinterpret_cast<const uint32_t *>(reinterpret_cast<uintptr_t>(x) - sh);
        const v4u32 v = *reinterpret_cast<const v4u32_a4 *>(p);
        const uint32_t e = p[sh ? 4 : 3];
        return v4u32{__builtin_amdgcn_alignbyte(v[1], v[0], sh), __builtin_amdgcn_alignbyte(v[2], v[1], sh),
                     __builtin_amdgcn_alignbyte(v[3], v[2], sh), __builtin_amdgcn_alignbyte(e, v[3], sh)};
    }
    v4u32 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t lo = 2 * i < left ? x[2 * i] : 0, hi = 2 * i + 1 < left ? x[2 * i + 1] : 0;
        v[i] = lo | (hi << 16);
    }
    return v;
}

// Workgroup holding unit x when G workgroups split U units evenly: the largest
// w with floor(w U / G) <= x.
__host__ __device__ inline int64_t unit_owner(int64_t x, int64_t U, int64_t G) { return ((x + 1) * G - 1) / U; }

struct WaveArgs {
    int64_t M, K, RB, KT;
    int64_t sets, units, maxseg;  // row sets; sets * KT; partial slots per row set (wide kernel: per workgroup)
    const uint16_t *X;
    int64_t ldx;
    uint32_t x_bytes;             // readable bytes of X from its base
    uint16_t *Y;
    int64_t ldy;
    int N;
    float *ws;                    // partials [set][slot][token][16 R rows], or null
    uint32_t *cnt;                // arrival counters per row set and token group (zero between calls)
    int y_vec;
    int x_vec;                    // column-chunk kernel: X is 16-byte aligned, ldx and K multiples of 8
    int tg;                       // token groups: wavefronts that stream the same units
    const uint16_t *bias;         // fused epilogue (Epilogue): fp16 [M] or null
    const uint16_t *res;          // fp16 residual, token n at res + n * ldr, or null
    int64_t ldr;
    int act;                      // usp_activation
    int e_flags;                  // EpilogueFlags
    const uint8_t *xp;            // X packed in product order (pack_x_kernel), or null
    uint32_t xp_bytes;
    int tb;                       // blocks of 16 tokens in xp: ceil(N / 16) (wide kernel: of 32 tokens)
    // Wide kernel: the part of a plan that a launch runs. Workgroup b is the
    // plan's workgroup w0 + b of G and takes what units [u_lo, u_hi) have of its
    // range, for tokens [n_lo, N).
    int64_t w0, G, u_lo, u_hi;
    int n_lo;
};

typedef void (*WaveKernelFn)(WaveArgs, const uint32_t *, const uint8_t *);

// Stores row blocks set * R .. of the NB blocks of 16 tokens from tok0 (a lane's
// MFMA outputs).
template <int R, int NB, EpilogueMode EPI>
__device__ inline void store_set(const WaveArgs &a, int64_t set, int tok0, int lane, const floatx4 (&acc)[R][NB]) {
    const int64_t m = set * R * kTileRows + 4 * (lane >> 4);
    uint2 bq[R], rq[R];
    if (EPI == kEpiAhead) {
#pragma unroll
        for (int r = 0; r < R; ++r) bq[r] = bias_quad(a, m + r * kTileRows);
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int n = tok0 + 16 * nb + (lane & 15);
        if (n < a.N) {
            if (EPI == kEpiAhead) {
#pragma unroll
                for (int r = 0; r < R; ++r) rq[r] = residual_quad(a, n, m + r * kTileRows);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (EPI == kEpiAhead)
                    store_rows4(a, n, m + r * kTileRows, acc[r][nb], bq[r], rq[r]);
                else if (EPI == kEpiInline)
                    store_rows4(a, n, m + r * kTileRows, acc[r][nb]);
                else
                    store_rounded4(a, n, m + r * kTileRows, acc[r][nb]);
            }
        }
    }
}

// Counts this wavefront's arrival at row set `set` for token group g (its
// partial must already be acknowledged); returns the counter's previous value
// (in lane 0).
__device__ inline uint32_t arrive_count(const WaveArgs &a, int64_t set, int lane, int g = 0) {
    uint32_t old = 0;
    if (lane == 0)
        old = __hip_atomic_fetch_add(a.cnt + set * a.tg + g, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return old;
}

// Sums the nseg slots of row set `set` in order for token group g's NB blocks of
// 16 tokens and stores Y.
template <int R, int NB, EpilogueMode EPI>
__device__ inline void sum_slots(const WaveArgs &a, int64_t set, int64_t nseg, int lane, int g) {
    const int64_t slot_floats = (int64_t)a.N * kTileRows * R;
    float *slot0 = a.ws + set * a.maxseg * slot_floats;
    const __amdgpu_buffer_rsrc_t part =
        __builtin_amdgcn_make_buffer_rsrc(slot0, (short)0, (int)(nseg * slot_floats * 4), kBufferRsrcWord3);
    const int g4 = 4 * (lane >> 4);
    uint2 bq[R], rq[R];
    if (EPI == kEpiAhead) {
#pragma unroll
        for (int r = 0; r < R; ++r) bq[r] = bias_quad(a, (set * R + r) * kTileRows + g4);
    }
#pragma unroll 1
    for (int nb = 0; nb < NB; ++nb) {
        const int n = 16 * (NB * g + nb) + (lane & 15);
        if (n < a.N) {
            if (EPI == kEpiAhead) {
#pragma unroll
                for (int r = 0; r < R; ++r) rq[r] = residual_quad(a, n, (set * R + r) * kTileRows + g4);
            }
            // Batches of B slots x R row blocks (16 loads), issued together, then
            // added in slot order per row block: one round trip for up to B slots.
            constexpr int B = R >= 16 ? 1 : 16 / R;
            floatx4 sum[R];
#pragma unroll
            for (int r = 0; r < R; ++r) sum[r] = floatx4{0.f, 0.f, 0.f, 0.f};
            const int lofs = (n * kTileRows * R + g4) * 4;
            for (int64_t j0 = 0; j0 < nseg; j0 += B) {
                v4u32 v[B][R];
#pragma unroll
                for (int jj = 0; jj < B; ++jj)
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        v[jj][r] = j0 + jj < nseg ? __builtin_amdgcn_raw_buffer_load_b128(
                                                        part, (int)((j0 + jj) * slot_floats * 4) + lofs + 64 * r, 0,
                                                        kCachePolicyDevice)
                                                  : v4u32{0u, 0u, 0u, 0u};
#pragma unroll
                for (int jj = 0; jj < B; ++jj)
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        if (j0 + jj < nseg) sum[r] += __builtin_bit_cast(floatx4, v[jj][r]);
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int64_t m = (set * R + r) * kTileRows + g4;
                if (EPI == kEpiAhead && NB == 1)  // arrive_finish has tested that there is one
                    store_rounded4(a, n, m, epilogue(a, sum[r], bq[r], rq[r]));
                else if (EPI == kEpiAhead)
                    store_rows4(a, n, m, sum[r], bq[r], rq[r]);
                else if (EPI == kEpiInline)
                    store_rows4(a, n, m, sum[r]);
                else
                    store_rounded4(a, n, m, sum[r]);
            }
        }
    }
}

// With the counter's previous value: the last of the nseg arrivals sums the
// slots, stores Y and resets the counter. Calls without an epilogue sum in code
// that requests no operands: testing for them there cost 13B attention at 32
// tokens 0.3 us of 15.3. At one token block that code lies out of line, and the
// stores of the other test nothing: else calls with an epilogue lost 0.1 us of 12.8
// (13B attention at 16 tokens); at two blocks the same cost 0.3 of 17.6 (4999 x 4093
// at 21 tokens).
template <int R, int NB, EpilogueMode EPI>
__device__ inline void arrive_finish(const WaveArgs &a, int64_t set, int64_t nseg, uint32_t old, int lane,
                                     int g = 0) {
    old = __builtin_amdgcn_readfirstlane(old);
    if (old != (uint32_t)nseg - 1u) return;
    if (NB == 1 && EPI == kEpiAhead) {
        if (__builtin_expect(has_epilogue(a), 1))
            sum_slots<R, NB, EPI>(a, set, nseg, lane, g);
        else
            sum_slots<R, NB, kEpiNone>(a, set, nseg, lane, g);
    } else if (EPI == kEpiAhead && !has_epilogue(a))
        sum_slots<R, NB, kEpiNone>(a, set, nseg, lane, g);
    else
        sum_slots<R, NB, EPI>(a, set, nseg, lane, g);
    if (lane == 0) __hip_atomic_store(a.cnt + set * a.tg + g, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int R, int NB, EpilogueMode EPI>
__device__ inline void arrive_row_set(const WaveArgs &a, int64_t set, int64_t nseg, int lane, int g = 0) {
    arrive_finish<R, NB, EPI>(a, set, nseg, arrive_count(a, set, lane, g), lane, g);
}

// Encoding of s_waitcnt that waits until at most n vector memory operations
// are outstanding and ignores the other counters.
__device__ constexpr int vmcnt_only(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }

// This lane's mask word of the record staged in `slot`.
__device__ inline uint2 slot_mask(const uint8_t *slot, int lane) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    typedef const __attribute__((address_space(3))) u32x2 lds_u32x2;
    const u32x2 m = ((lds_u32x2 *)(const __attribute__((address_space(3))) void *)slot)[lane];
    return make_uint2(m.x, m.y);
}


// Workgroup barrier ordering LDS reads and writes only. __syncthreads() is a
// workgroup fence, and a fence that covers LDS also waits for every
// direct-to-LDS transfer in flight, which would drain the record ring at every
// barrier; here this wavefront's LDS instructions complete (lgkmcnt) before
// the barrier, and the clobber keeps the compiler from moving memory accesses
// across it. Transfers into a ring slot are only ever read by the wavefront
// that issued them, behind its own hand-counted wait.
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Loads the whole record at 16-byte units [o0, o1) into LDS at byte address
// `lds` (L transfers of 16 bytes per lane, non-temporal), issued from inline
// assembly: the compiler neither sees these loads nor waits for them, so the
// caller waits for them itself (s_waitcnt vmcnt, counting every vector memory
// instruction issued after them). The compiler's own waits for transfers into
// LDS arrays it can tell apart are exact only while at most 8 such arrays are in
// play and their index is a constant; a ring shared by the wavefronts of a
// workgroup, indexed by wavefront, made it wait for every transfer in flight.
typedef int v4i32 __attribute__((ext_vector_type(4)));
template <int L>
__device__ inline void dma_rec_asm(const uint8_t *__restrict__ stream, uint32_t o0, uint32_t o1, int lane,
                                   uint32_t lds) {
    const uint64_t base = reinterpret_cast<uint64_t>(stream) + (uint64_t)o0 * 16;
    const v4i32 rsrc = {(int)(uint32_t)base, (int)((uint32_t)(base >> 32) & 0xFFFFu), (int)((o1 - o0) * 16),
                        kBufferRsrcWord3};
#pragma unroll
    for (int i = 0; i < L; ++i)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds"
                     :
                     : "s"(lds + 1024u * i), "v"(1024 * i + lane * 16), "s"(rsrc)
                     : "memory", "m0");
}

// Calls f(std::integral_constant<int, P>{}) for P = 0, 1, ...: an unrolled loop
// whose index is a constant in every copy, however large the body.
template <class F, int... P>
__device__ __attribute__((always_inline)) inline void static_for(F &&f, std::integer_sequence<int, P...>) {
    (f(std::integral_constant<int, P>{}), ...);
}

}  // namespace
}  // namespace usp
