// usp_wide.hip -- the wide kernel: products over many tokens (X packed in
// product order first), and its launcher.
#include "usp_device.h"
#include "usp_internal.h"

#include <algorithm>

namespace usp {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kWideRows = 8;                    // row blocks per unit (128 rows) = wavefronts per workgroup
constexpr int kWidePairs = kWideRows / 2;       // 32-row A operands per 16 columns
constexpr int kWideStepBytes = kWideRows * kLanes * 16;  // decoded A operands of one 32-column step
constexpr int kWideTokens = 32;                 // tokens of a B operand
constexpr size_t kWideBlockBytes = 1024;        // packed B operand: 32 tokens x 16 columns

// ---------------------------------------------------------------------------
// X packed for v_mfma_f32_32x32x16_f16: block (((kt * 8 + st) * 2 + h) * TB + tb)
// of 1 KB, lane l = 32 g + n, holds X[32 tb + n][256 kt + 32 st + 16 h + 8 g ..
// + 7] (zeros past N and K). One wavefront per (column tile, token block).
// VEC: X is 16-byte aligned with ldx and K multiples of 8.
// ---------------------------------------------------------------------------
template <bool VEC>
__global__ __launch_bounds__(kLanes) void pack_wide_kernel(const uint16_t *__restrict__ X, int64_t ldx, int N,
                                                          int64_t K, int TB, uint8_t *__restrict__ xp) {
    const int lane = threadIdx.x;
    const int64_t kt = blockIdx.x / TB, tb = blockIdx.x % TB;
    const int64_t n = kWideTokens * tb + (lane & 31);
    const int64_t k0 = kt * kTileK + 8 * (lane >> 5);
    v4u32 v[2 * kSteps];
#pragma unroll
    for (int i = 0; i < 2 * kSteps; ++i) {
        const int64_t k = k0 + 16 * i;
        if (VEC) {
            v[i] = n < N && k < K ? *reinterpret_cast<const v4u32 *>(X + n * ldx + k) : v4u32{0u, 0u, 0u, 0u};
        } else {
            v[i] = n < N && k < K ? load_x8(X + n * ldx + k, K - k) : v4u32{0u, 0u, 0u, 0u};
        }
    }
#pragma unroll
    for (int i = 0; i < 2 * kSteps; ++i)
        reinterpret_cast<v4u32 *>(xp + ((kt * 2 * kSteps + i) * TB + tb) * kWideBlockBytes)[lane] = v[i];
}

// Partial slots. Where every workgroup's range lies inside one tile (a.maxseg =
// 1) workgroup w has slot w; otherwise it keeps the partial of a tile it starts in
// the middle of in slot 2 w and that of a tile it starts at the beginning of
// (and does not finish) in slot 2 w + 1. A slot holds the workgroup's
// accumulators as they sit in the registers:
// [wavefront][pair][token block][quad][lane] x 16 bytes.
__device__ inline int64_t wide_slot(const WaveArgs &a, int64_t w, int64_t w_first) {
    return a.maxseg == 1 ? w : 2 * w + (w == w_first);
}

// Stores the 32 x 32 product whose rows start at m and tokens at n0: lane l
// holds token l % 32 and rows 8 q + 4 (l / 32) .. + 3 in elements 4 q .. + 3. The
// epilogue's operands are requested for all of them first (one at a time, before
// each use, cost the 13B FFN up at 1024 tokens with bias and ReLU 18 us).
__device__ inline void store_block(const WaveArgs &a, int n0, int64_t m, int lane, const floatx16 &v) {
    const int n = n0 + (lane & 31);
    if (n >= a.N) return;
    const int64_t m0 = m + 4 * (lane >> 5);
    uint2 bq[4], rq[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) bq[q] = bias_quad(a, m0 + 8 * q);
#pragma unroll
    for (int q = 0; q < 4; ++q) rq[q] = residual_quad(a, n, m0 + 8 * q);
#pragma unroll
    for (int q = 0; q < 4; ++q)
        store_rows4(a, n, m0 + 8 * q, floatx4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]}, bq[q], rq[q]);
}

template <int NB>
__device__ inline void wide_finish(const WaveArgs &a, int64_t tile, int64_t w_first, int64_t nseg, uint32_t old,
                                   int j, int lane, int64_t m0, int tok0) {
    constexpr int P = kWidePairs;
    old = __builtin_amdgcn_readfirstlane(old);
    if (old != (uint32_t)nseg - 1u) return;
    constexpr int kWaveBytes = P * NB * 4096;  // one wavefront's share of a slot
    constexpr int64_t kSlotBytes = (int64_t)kWideRows * kWaveBytes;
#pragma unroll 1
    for (int i = 0; i < P * NB; ++i) {
        floatx4 sum[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) sum[q] = floatx4{0.f, 0.f, 0.f, 0.f};
        constexpr int B = 2;  // slots per round trip
        for (int64_t s0 = 0; s0 < nseg; s0 += B) {
            v4u32 v[B][4];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int64_t w = w_first + (s0 + b < nseg ? s0 + b : nseg - 1);
                const __amdgpu_buffer_rsrc_t part = __builtin_amdgcn_make_buffer_rsrc(
                    reinterpret_cast<uint8_t *>(a.ws) + wide_slot(a, w, w_first) * kSlotBytes + j * kWaveBytes, (short)0,
                    kWaveBytes, kBufferRsrcWord3);
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    v[b][q] = __builtin_amdgcn_raw_buffer_load_b128(part, i * 4096 + q * 1024 + lane * 16, 0,
                                                                    kCachePolicyDevice);
            }
#pragma unroll
            for (int b = 0; b < B; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (s0 + b < nseg) sum[q] += __builtin_bit_cast(floatx4, v[b][q]);
        }
        floatx16 v;
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = sum[e / 4][e % 4];
        store_block(a, tok0 + kWideTokens * (i % NB), m0 + 32 * (i / NB), lane, v);
    }
    if (lane == 0) __hip_atomic_store(a.cnt + tile * kWideRows + j, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------
// Wide kernel (193 to 256 tokens on large layers, from 320 tokens on all).
//
// A workgroup of eight wavefronts streams a contiguous range of units (8 row
// blocks x 1 column tile). Wavefront j owns row block j: it moves that record
// into its own LDS ring slots, decodes it once per unit and writes the A operands
// to a shared LDS buffer; every wavefront multiplies all 128 rows by its own NB
// blocks of 32 tokens, X read from the packed copy. What bounds it is the sum
// of the SIMD's VALU (decode, about 265 instructions per record) and matrix
// time, which two wavefronts per SIMD overlap in part, so a record has to serve
// many tokens: 7.3 us per unit and CU at 512 tokens per workgroup, 4.7 at 256,
// 3.4 at 128 (70B FFN, 50%). Each choice below was measured against its
// alternatives at 512 tokens per workgroup on the 13B FFN up at 1024 tokens
// (160 us; 665 in passes of 64 tokens on the four-wavefront kernel):
//   * 32 x 32 x 16 products: half the instructions of 16 x 16 x 32 for the same
//     work, and an A operand read from LDS serves 32 tokens;
//   * 8 wavefronts of 128 rows x 64 tokens: 4 wavefronts of 128 x 64 (256 tokens,
//     one wavefront per SIMD) took 233 us, 8 of 64 x 64 (256 tokens, every block
//     of X loaded by two wavefronts) 200, 8 of 64 x 128 168;
//   * the decode of a step is spread over the products of the step before it, the
//     record's prefix scan included; A operands are double-buffered by groups
//     of kWideGroup steps with one barrier per group, and read from LDS one
//     half step before their products, so no product waits for a barrier's
//     other side. Groups of 2 or 4 steps, 2 or 3 ring slots: within 1%.
// ---------------------------------------------------------------------------

// Ring slots per row block, and steps per group (the decoded A operands are
// double-buffered by groups of GS steps): what fits 160 KB of LDS.
constexpr int kWideGroup = 2;
constexpr int wide_slots(int L) { return L <= 5 ? 3 : 2; }
constexpr int kMaxWideLoads = 7;

template <int L, int NB>
__global__ __launch_bounds__(kWideRows *kLanes, 2) void spmm_wide_kernel(WaveArgs a, const uint32_t *__restrict__ off,
                                                                         const uint8_t *__restrict__ stream) {
    constexpr int P = kWidePairs;            // A operands (32 rows) per half step
    constexpr int GS = kWideGroup;           // steps per group
    constexpr int S = wide_slots(L);         // ring slots per row block
    constexpr int D0 = kSteps - GS;          // step during which the next unit's decode begins
    constexpr int XS = NB == 1 ? 4 : 2;      // steps of X in registers (256 registers per wavefront)
    constexpr int kRec = 1024 * L;
    constexpr int kAbuf = GS * kWideStepBytes;
    constexpr int kLut = 2 * kAbuf;
    constexpr int kRing = kLut + 128;
    __shared__ __attribute__((aligned(1024))) uint8_t smem[kRing + S * kWideRows * kRec + 16];
    uint8_t *const lut = smem + kLut;
    const int lane = threadIdx.x & (kLanes - 1);
    const int j = __builtin_amdgcn_readfirstlane(threadIdx.x / kLanes);
    const int64_t w = a.w0 + blockIdx.x, G = a.G;
    const int64_t ua = w * a.units / G, ub = (w + 1) * a.units / G;
    const int u0 = (int)(ua > a.u_lo ? ua : a.u_lo), u1 = (int)(ub < a.u_hi ? ub : a.u_hi);
    if (u0 >= u1) return;  // the whole workgroup
    if (threadIdx.x < 16) reinterpret_cast<uint2 *>(lut)[threadIdx.x] = nibble_selectors((uint32_t)threadIdx.x);

    const __amdgpu_buffer_rsrc_t xr =
        __builtin_amdgcn_make_buffer_rsrc((void *)a.xp, (short)0, (int)a.xp_bytes, kBufferRsrcWord3);
    const __amdgpu_buffer_rsrc_t offr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)off, (short)0, (int)((a.RB * a.KT + 1) * 4), kBufferRsrcWord3);

    struct Pos {
        int set, kt, tt;
    };
    const int KT = (int)a.KT, sets = (int)a.sets, RB = (int)a.RB;
    auto advance = [&](Pos &p) {
        if (++p.kt == KT) {
            p.kt = 0;
            if (++p.set == sets) {
                p.set = 0;
                ++p.tt;
            }
        }
    };
    // Extents of this wavefront's record of a unit: lane 0 its start, lane 1 its
    // end; empty past the range (real false) or the matrix.
    auto rec_offsets = [&](const Pos &p, bool real) -> uint32_t {
        const int rb = p.set * kWideRows + j;
        const bool ok = real && lane < 2 && rb < RB;
        return __builtin_amdgcn_raw_buffer_load_b32(offr, ok ? (rb * KT + p.kt + lane) * 4 : 0x7FFFFFF0, 0, 0);
    };
    const uint32_t smem_lds =
        (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t *)smem);
    auto slot_of = [&](int sl) -> int { return kRing + (sl * kWideRows + j) * kRec; };
    auto dma = [&](int sl, uint32_t o) {
        dma_rec_asm<L>(stream, __builtin_amdgcn_readlane(o, 0), __builtin_amdgcn_readlane(o, 1), lane,
                       smem_lds + slot_of(sl));
    };
    // X: the wavefront's blocks of (kt, step, half) start at a uniform offset.
    auto x_base = [&](const Pos &p) -> int {
        return (p.kt * 2 * kSteps * a.tb + (p.tt * kWideRows + j) * NB) * (int)kWideBlockBytes;
    };
    auto load_x = [&](int base, int st, int h, int nb) -> v4u32 {
        return __builtin_amdgcn_raw_buffer_load_b128(xr, lane * 16 + nb * (int)kWideBlockBytes,
                                                     base + (2 * st + h) * a.tb * (int)kWideBlockBytes, 0);
    };
    // Where this wavefront's decoded operand goes within a step of the A buffer:
    // lane l of the decode holds row l % 16 and columns 8 (l / 16) .. + 7 of the
    // step; the product reads row l % 32, columns 8 (l / 32) .. + 7 of each half.
    const int aw = j / 2 * 2048 + (lane >> 5) * 1024 + ((lane & 15) + 16 * (j & 1) + 32 * ((lane >> 4) & 1)) * 16;

    // Vector memory instructions issued after the transfer of the record that
    // the mask read of step D0 - 3 needs (issued S - 1 units before, at step D0):
    // X of 8 (S - 2) + 5 steps and the S - 2 transfers between; in the first
    // unit what follows it in the prologue and X of the steps since, in the
    // second (S = 3) likewise. Loads complete in order.
    constexpr int kMaskStep = D0 - 3;
    constexpr int kSteady = 8 * (S - 2) + 5 < XS + 8 + kMaskStep ? 8 * (S - 2) + 5 : XS + 8 + kMaskStep;
    constexpr int kRecOps = 2 * NB * kSteady - NB + (S - 2) * L;
    constexpr int kFirstOps = 2 * NB * (XS + kMaskStep) - NB + (S - 2) * L;
    constexpr int kRecWait = kRecOps < 63 ? kRecOps : 63;
    constexpr int kFirstUnitWait = kFirstOps < 63 ? kFirstOps : 63;
    constexpr int kStartOps = 2 * NB * XS + (S - 1) * L;
    constexpr int kStartWait = kStartOps < 63 ? kStartOps : 63;

    floatx16 acc[P][NB];
    auto clear = [&]() {
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[p][nb][i] = 0.f;
    };
    clear();
    Pos cur = {u0 / KT % sets, u0 % KT, u0 / KT / sets};
    Pos la = cur;  // the unit whose offsets are loaded next
    {
        uint32_t o[S];
#pragma unroll
        for (int i = 0; i < S; ++i) {
            o[i] = rec_offsets(la, u0 + i < u1);
            advance(la);
        }
#pragma unroll
        for (int i = 0; i < S; ++i) dma(i, o[i]);
    }
    uint32_t onext = rec_offsets(la, u0 + S < u1);  // the unit requested at step D0
    advance(la);
    v4u32 xb[XS][2][NB];
    {
        const int xc = x_base(cur);
#pragma unroll
        for (int st = 0; st < XS; ++st)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) xb[st][h][nb] = load_x(xc, st, h, nb);
    }
    lds_barrier();  // the selector table
    lds_u32 *const region = as_lds(smem);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kStartWait) : "memory");
    RecState rs = rec_state(slot_mask(smem + slot_of(0), lane), (uint32_t)(slot_of(0) + kMaskBytes));
#pragma unroll
    for (int st = 0; st < GS; ++st)
        *reinterpret_cast<uint4 *>(smem + st * kWideStepBytes + aw) =
            __builtin_bit_cast(uint4, decode_step(region, lut, rs, st));
    StepWords sw = read_step(region, lut, rs, GS);
    lds_barrier();  // the first group's operands

    int sl = 0;  // the current unit's ring slot
    for (int u = u0; u < u1; ++u) {
        const uint32_t onn = rec_offsets(la, u + S + 1 < u1);
        advance(la);
        Pos nx = cur;
        advance(nx);
        const bool more = u + 1 < u1;
        const int sn = sl + 1 == S ? 0 : sl + 1;
        const int xc = x_base(cur), xn = more ? x_base(nx) : xc;  // past the range: this unit's, unused
        half8 av[2][P];
        uint2 msk;
        RecState rn;
        // Products of half i = 2 st + h of the unit, then its X for later.
        auto products = [&](auto ic) __attribute__((always_inline)) {
            constexpr int st = decltype(ic)::value / 2, h = decltype(ic)::value % 2;
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[p][nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                        av[h][p], __builtin_bit_cast(half8, xb[st % XS][h][nb]), acc[p][nb], 0, 0, 0);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                xb[st % XS][h][nb] =
                    st + XS < kSteps ? load_x(xc, st + XS, h, nb) : load_x(xn, st + XS - kSteps, h, nb);
        };
        static_for(
            [&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value, st = i / 2, h = i % 2;
                constexpr int d = st + GS < kSteps ? st + GS : st + GS - kSteps;  // step decoded meanwhile
                constexpr int dn = st + 1 + GS < kSteps ? st + 1 + GS : st + 1 + GS - kSteps;
                __builtin_amdgcn_sched_barrier(0);
                if (st == kMaskStep && h == 0) {  // the next unit's record must have arrived
                    if (u == u0)
                        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kFirstUnitWait) : "memory");
                    else
                        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kRecWait) : "memory");
                    msk = slot_mask(smem + slot_of(sn), lane);
                }
#pragma unroll
                for (int p = 0; p < P; ++p)
                    av[h][p] = *reinterpret_cast<const half8 *>(smem + st % (2 * GS) * kWideStepBytes + p * 2048 +
                                                                h * 1024 + lane * 16);
                // A step's LDS words are read a step before they are expanded.
                StepWords now;
                if (h == 1) {
                    now = sw;
                    sw = read_step(region, lut, st + 1 < D0 ? rs : rn, dn);
                }
                if (st == D0 - 2 && h == 0) rn = rec_state(msk, (uint32_t)(slot_of(sn) + kMaskBytes));
                if (i > 0) products(std::integral_constant<int, (i > 0 ? i - 1 : 0)>{});
                if (h == 1)
                    *reinterpret_cast<uint4 *>(smem + d % (2 * GS) * kWideStepBytes + aw) =
                        __builtin_bit_cast(uint4, finish_step(now));
                if (st % GS == GS - 1 && h == 1) {
                    lds_barrier();  // the next group's operands are complete, this group's free
                    if (st + 1 == D0) {  // the unit's records are decoded: their slots take unit u + S
                        dma(sl, onext);
                        onext = onn;
                    }
                }
            },
            std::make_integer_sequence<int, 2 * kSteps>{});
        products(std::integral_constant<int, 2 * kSteps - 1>{});
        rs = rn;
        if (!more || nx.kt == 0) {  // end of this workgroup's part of the tile
            const int tok0 = (cur.tt * kWideRows + j) * NB * kWideTokens;
            const int64_t m0 = (int64_t)cur.set * kWideRows * kTileRows;
            if (tok0 < a.N && tok0 >= a.n_lo) {
                const int64_t tile = (int64_t)cur.tt * sets + cur.set;
                const int64_t w_first = unit_owner(tile * a.KT, a.units, G);
                const int64_t w_last = unit_owner(tile * a.KT + a.KT - 1, a.units, G);
                if (w_first == w_last) {
#pragma unroll 1
                    for (int i = 0; i < P * NB; ++i) {
                        floatx16 v = acc[0][0];
                        static_for(
                            [&](auto c) {
                                if (c.value > 0 && i == c.value) v = acc[c.value / NB][c.value % NB];
                            },
                            std::make_integer_sequence<int, P * NB>{});
                        store_block(a, tok0 + kWideTokens * (i % NB), m0 + 32 * (i / NB), lane, v);
                    }
                } else {
                    constexpr int kWaveBytes = P * NB * 4096;
                    const __amdgpu_buffer_rsrc_t part = __builtin_amdgcn_make_buffer_rsrc(
                        reinterpret_cast<uint8_t *>(a.ws) +
                            (wide_slot(a, w, w_first) * kWideRows + j) * (int64_t)kWaveBytes,
                        (short)0, kWaveBytes, kBufferRsrcWord3);
#pragma unroll
                    for (int p = 0; p < P; ++p)
#pragma unroll
                        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                __builtin_amdgcn_raw_buffer_store_b128(
                                    __builtin_bit_cast(v4u32, floatx4{acc[p][nb][4 * q], acc[p][nb][4 * q + 1],
                                                                      acc[p][nb][4 * q + 2], acc[p][nb][4 * q + 3]}),
                                    part, ((p * NB + nb) * 4 + q) * 1024 + lane * 16, 0, kCachePolicyDevice);
                    // Acknowledged before the arrival counts. The wait also covers the
                    // records and X in flight, which are the next ones needed.
                    __builtin_amdgcn_s_waitcnt(0);
                    uint32_t old = 0;
                    if (lane == 0)
                        old = __hip_atomic_fetch_add(a.cnt + tile * kWideRows + j, 1u, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT);
                    wide_finish<NB>(a, tile, w_first, w_last - w_first + 1, old, j, lane, m0, tok0);
                }
            }
            clear();
        }
        cur = nx;
        sl = sn;
    }
    __builtin_amdgcn_s_waitcnt(0);  // the transfers past the range's end
}


WaveKernelFn wide_kernel(int loads, int nb) {
#define USP_WIDE(NB)                               \
    switch (loads) {                               \
        case 2: return spmm_wide_kernel<2, NB>;    \
        case 3: return spmm_wide_kernel<3, NB>;    \
        case 4: return spmm_wide_kernel<4, NB>;    \
        case 5: return spmm_wide_kernel<5, NB>;    \
        case 6: return spmm_wide_kernel<6, NB>;    \
        default: return spmm_wide_kernel<7, NB>;   \
    }
    if (nb == 1) {
        USP_WIDE(1)
    }
    USP_WIDE(2)
#undef USP_WIDE
}

int wide_loads(const usp_matrix *A) {
    return std::max<int>(2, (int)ceil_div(kMaskChunks + A->max_chunks, kLanes));
}

// Tokens of one launch: calls of more are cut into equal passes (packed X then
// takes 4 KB x K at most).
constexpr int64_t kMaxWidePass = 2048;

int64_t wide_pass_tokens(int64_t N) {
    return ceil_div(ceil_div(N, ceil_div(N, kMaxWidePass)), kWideTokens) * kWideTokens;
}

}  // namespace

bool wide_serves(const usp_matrix *A, int64_t N) {
    const int64_t n = std::min(N, wide_pass_tokens(N));
    return wide_loads(A) <= kMaxWideLoads && (A->RB * A->KT + 1) * 4 < ((int64_t)1 << 31) &&
           (int64_t)A->KT * 2 * kSteps * ceil_div(n, kWideTokens) * (int64_t)kWideBlockBytes < ((int64_t)1 << 31);
}

// Bytes of X packed for `blocks` blocks of 32 tokens. A wavefront past the last
// tokens loads blocks past the last one.
static size_t wide_pack_bytes(int64_t KT, int64_t blocks) {
    return ((size_t)KT * 2 * kSteps * blocks + 2 * kWideRows) * kWideBlockBytes;
}

// Bytes of one workgroup's partial slots.
static size_t wide_slot_bytes(int nb, int slots) { return (size_t)slots * nb * kWideRows * kWideRows * 2048; }

// A plan can run in parts, one tile and one wavefront's token slice at the least
// (launch_wide); twice the larger of that slice's packed X and that tile's partials
// holds both.
static size_t wide_min_bytes(const usp_matrix *A, int nb, int64_t tile_segs, int slots) {
    return 2 * std::max(wide_pack_bytes(A->KT, nb), (size_t)tile_segs * wide_slot_bytes(nb, slots));
}

// The token blocks per wavefront and the workgroup ranges that cost least by
// what a unit takes on a CU (us, measured on the 70B FFN at 50%), a workgroup's
// start, and the partials of split tiles (us per byte). Ranges that cross tiles
// flush twice, and whole or evenly cut tiles win unless they leave many CUs idle:
// 70B FFN at 256 tokens 160 us on 224 workgroups against 164 on 256, 13B FFN up at
// 512 99 on 216 against 109 on 256.
// max_bytes: what a plan may take; min_bytes: what its smallest part may take.
WidePlan plan_wide(const usp_matrix *A, int64_t N, size_t max_bytes, size_t min_bytes) {
    WidePlan p;
    const int64_t cus = A->num_cus > 0 ? A->num_cus : 256;
    p.passes = ceil_div(N, wide_pass_tokens(N));
    const int64_t n = std::min(N, wide_pass_tokens(N));
    p.loads = wide_loads(A);
    p.tb = ceil_div(n, kWideTokens);
    p.sets = ceil_div(A->RB, kWideRows);
    p.pack_bytes = wide_pack_bytes(A->KT, p.tb);
    double best = 0;
    for (int nb = 1; nb <= 2; ++nb) {
        const int64_t tt = ceil_div(p.tb, (int64_t)nb * kWideRows), tiles = p.sets * tt, units = tiles * A->KT;
        const double unit = nb == 1 ? 4.7 : 7.3;
        auto consider = [&](int64_t G) {
            const bool split = units % G != 0 || (units / G) % A->KT != 0;
            // One slot per workgroup where no range crosses a tile's end, else two.
            const int slots = G % tiles == 0 ? 1 : 2;
            const size_t part = split ? (size_t)G * wide_slot_bytes(nb, slots) : 0;
            // The most workgroups that share a tile.
            const int64_t segs = !split ? 0 : slots == 1 ? G / tiles : ceil_div(G, tiles) + 1;
            const size_t least = wide_min_bytes(A, nb, segs, slots);
            if ((split && tiles * kWideRows > kMaxCounters) || part + p.pack_bytes > max_bytes || least > min_bytes)
                return;
            const double cost = (double)ceil_div(G, cus) * ((double)ceil_div(units, G) * unit + 3.0) +
                                (split ? 4.0 + (double)part * (slots == 1 ? 3e-7 : 2.5e-7) : 0.0);
            if (p.grid && cost >= best) return;
            best = cost;
            p.nb = nb;
            p.tt = tt;
            p.tiles = tiles;
            p.units = units;
            p.grid = G;
            p.split = split;
            p.slots = slots;
            p.part_bytes = part;
            p.min_bytes = std::min(least, part + p.pack_bytes);
        };
        consider(tiles);
        for (int64_t S = 2; S <= A->KT && tiles * S <= cus; ++S) consider(tiles * S);
        if (units > cus) consider(cus);
    }
    return p;
}

// A plan whose partials and packed X do not fit the workspace runs in parts that
// do, one after another: over token slices (whole token tiles while half the
// space holds their packed X), and over as many tiles as the rest holds partials
// of. The workgroups' ranges, and with them the order of every sum, are the
// plan's.
int launch_wide(const usp_matrix *A, const WidePlan &p, const void *X, int64_t ldx, void *Y, int64_t ldy, int64_t N,
                const Epilogue &ep, void *workspace, size_t ws_bytes, void *stream) {
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    static_assert(kMaxWidePass / kWideTokens * kWideBlockBytes <= kCounterRegionBytes,
                  "a part's packed X is addressed from up to this far before it");
    uint8_t *const ws = reinterpret_cast<uint8_t *>(workspace) + kCounterRegionBytes;
    const size_t room = ws_bytes - kCounterRegionBytes, slot_bytes = wide_slot_bytes(p.nb, p.slots);
    // Slices of nb blocks of 32 tokens of a part, 8 to a tile, and workgroups of a launch.
    int64_t slices = p.tt * kWideRows, max_wgs = p.grid;
    size_t part_bytes = p.part_bytes;
    if (p.part_bytes + p.pack_bytes > room) {
        while (slices > 1 && wide_pack_bytes(A->KT, slices * p.nb) > room / 2)
            slices = slices > kWideRows ? ceil_div(slices / kWideRows, 2) * kWideRows : slices / 2;
        if (p.split) {
            max_wgs = std::min(p.grid, (int64_t)((room - wide_pack_bytes(A->KT, slices * p.nb)) / slot_bytes));
            part_bytes = (size_t)max_wgs * slot_bytes;
        }
    }
    uint8_t *const xp = ws + part_bytes;
    WaveArgs a = {};
    a.M = A->M;
    a.K = A->K;
    a.RB = A->RB;
    a.KT = A->KT;
    a.sets = p.sets;
    a.units = p.units;
    a.maxseg = p.slots;
    a.ldy = ldy;
    a.cnt = reinterpret_cast<uint32_t *>(workspace);
    a.G = p.grid;
    a.bias = ep.bias;
    a.ldr = ep.ldr;
    a.act = ep.act;
    a.e_flags = epilogue_flags(ep);
    const int64_t P = wide_pass_tokens(N);
    const bool vec = (reinterpret_cast<uintptr_t>(X) & 15) == 0 && ldx % 8 == 0 && A->K % 8 == 0;
    for (int64_t n0 = 0; n0 < N; n0 += P) {
        const uint16_t *const x = reinterpret_cast<const uint16_t *>(X) + n0 * ldx;
        const int64_t n = std::min(P, N - n0);
        a.Y = reinterpret_cast<uint16_t *>(Y) + n0 * ldy;
        a.y_vec = ((reinterpret_cast<uintptr_t>(a.Y) & 7) == 0) && (ldy % 4 == 0);
        a.res = ep.res ? ep.res + n0 * ep.ldr : nullptr;
        for (int64_t s0 = 0; s0 * p.nb * kWideTokens < n; s0 += slices) {
            a.n_lo = (int)(s0 * p.nb * kWideTokens);
            a.N = (int)std::min(n, (s0 + slices) * p.nb * kWideTokens);
            a.tb = (int)std::min(slices * p.nb, p.tb - s0 * p.nb);
            // The kernel counts blocks from the pass's first token.
            const size_t before = (size_t)s0 * p.nb * kWideBlockBytes;
            a.xp = xp - before;
            a.xp_bytes = (uint32_t)(wide_pack_bytes(A->KT, a.tb) + before);
            hipLaunchKernelGGL(vec ? pack_wide_kernel<true> : pack_wide_kernel<false>, dim3((unsigned)(A->KT * a.tb)),
                               dim3(kLanes), 0, st, x + a.n_lo * ldx, ldx, a.N - a.n_lo, A->K, a.tb, xp);
            const int64_t end = std::min(p.tt, ceil_div(s0 + slices, (int64_t)kWideRows)) * p.sets;
            for (int64_t t = s0 / kWideRows * p.sets, t1; t < end; t = t1) {
                a.w0 = unit_owner(t * A->KT, p.units, p.grid);
                const int64_t w1 = std::min(a.w0 + max_wgs, p.grid);  // past the last workgroup
                t1 = std::min(end, w1 * p.units / p.grid / A->KT);
                a.u_lo = t * A->KT;
                a.u_hi = t1 * A->KT;
                a.ws = reinterpret_cast<float *>(ws - (size_t)a.w0 * slot_bytes);
                const int64_t wgs = unit_owner(a.u_hi - 1, p.units, p.grid) + 1 - a.w0;
                hipLaunchKernelGGL(wide_kernel(p.loads, p.nb), dim3((unsigned)wgs), dim3(kWideRows * kLanes), 0, st, a,
                                   A->d_off, reinterpret_cast<const uint8_t *>(A->d_stream));
            }
        }
    }
    return (int)hipGetLastError();
}

}  // namespace usp
