// usp_encode.cpp -- one-time host conversion of (W, mask) into tile records,
// and its inverse. This plays the role of the paper's dense-to-format
// conversion (Section 5.3, "Storage Format Conversion"), for the bitmap-class
// format described in usp_format.h.
#include <algorithm>
#include <cstring>
#include <thread>

#if defined(__SSE2__)
#include <emmintrin.h>
#endif

#include "usp_internal.h"

namespace usp {
namespace {

template <class F>
void parallel_rows(int64_t n, F &&fn) {
    unsigned hw = std::thread::hardware_concurrency();
    int64_t nt = std::max<int64_t>(1, std::min<int64_t>(hw ? hw : 1, 64));
    nt = std::min(nt, n);
    if (nt <= 1) {
        for (int64_t i = 0; i < n; ++i) fn(i);
        return;
    }
    std::vector<std::thread> th;
    th.reserve(nt);
    for (int64_t t = 0; t < nt; ++t) {
        th.emplace_back([&, t] {
            for (int64_t i = t; i < n; i += nt) fn(i);
        });
    }
    for (auto &x : th) x.join();
}

// Bit i of the result: byte i of p is nonzero. n bytes are readable (the others
// count as zero).
inline uint8_t nonzero_bits(const uint8_t *p, int64_t n) {
    uint64_t x = 0;
    if (n >= 8) {
        std::memcpy(&x, p, 8);
    } else {
        for (int64_t i = 0; i < n; ++i) x |= (uint64_t)p[i] << (8 * i);
    }
    // The top bit of every nonzero byte, then the eight top bits gathered.
    const uint64_t low = 0x7F7F7F7F7F7F7F7Full;
    const uint64_t t = (((x & low) + low) | x) & ~low;
    return (uint8_t)(((t >> 7) * 0x0102040810204080ull) >> 56);
}

}  // namespace

void encode_host(const uint16_t *W, int64_t ldw, const uint8_t *mask, int64_t ldm,
                 int64_t M, int64_t K, HostEncoding &out) {
    out.M = M;
    out.K = K;
    out.RB = ceil_div(M, kTileRows);
    out.KT = ceil_div(K, kTileK);
    const int64_t T = out.RB * out.KT;

    // Pass 1: the mask bytes of every record, in their final order, and its kept
    // count. Eight mask bytes become one byte of bits at a time, and pass 2 needs
    // the mask no more.
    std::vector<uint8_t, NoInit<uint8_t>> masks((size_t)T * kMaskBytes);
    std::vector<int64_t> tile_nnz(T, 0);
    parallel_rows(out.RB, [&](int64_t rb) {
        for (int64_t kt = 0; kt < out.KT; ++kt) {
            const int64_t t = rb * out.KT + kt;
            uint8_t *m = masks.data() + (size_t)t * kMaskBytes;
            for (int r = 0; r < kTileRows; ++r) {
                const int64_t row = rb * kTileRows + r;
                const uint8_t *mr = mask + row * ldm;
#if defined(__SSE2__)
                if (row < M && (kt + 1) * kTileK <= K) {  // 16 mask bytes at a time
                    for (int i = 0; i < kTileK / 16; ++i) {
                        const __m128i x = _mm_loadu_si128(reinterpret_cast<const __m128i *>(mr + kt * kTileK + 16 * i));
                        const int z = _mm_movemask_epi8(_mm_cmpeq_epi8(x, _mm_setzero_si128()));
                        const int s = i / 2, g = 2 * (i % 2);
                        m[8 * (g * kTileRows + r) + s] = (uint8_t)~z;
                        m[8 * ((g + 1) * kTileRows + r) + s] = (uint8_t)(~z >> 8);
                    }
                    continue;
                }
#endif
                for (int s = 0; s < kSteps; ++s)
                    for (int g = 0; g < kLanes / kTileRows; ++g) {
                        const int64_t c = kt * kTileK + tile_col(g, s, 0);
                        m[8 * (g * kTileRows + r) + s] = row < M && c < K ? nonzero_bits(mr + c, K - c) : 0;
                    }
            }
            int64_t cnt = 0;
            for (int l = 0; l < kLanes; ++l) {
                uint64_t x;
                std::memcpy(&x, m + 8 * l, 8);
                cnt += __builtin_popcountll(x);
            }
            tile_nnz[t] = cnt;
        }
    });
    out.off.assign(T + 1, 0);
    int64_t total = 0, nnz = 0, max_chunks = 0;
    for (int64_t t = 0; t < T; ++t) {
        out.off[t] = (uint32_t)total;
        const int64_t chunks = ceil_div(2 * tile_nnz[t], 16);
        total += kMaskChunks + chunks;
        max_chunks = std::max(max_chunks, chunks);
        nnz += tile_nnz[t];
        if (total >= (int64_t(1) << 32)) throw std::bad_alloc();
    }
    out.off[T] = (uint32_t)total;
    out.nnz = nnz;
    out.max_chunks = max_chunks;
    out.stream.resize((size_t)total * 16);  // every byte is written below

    // Pass 2: fill records. Each position writes its value at the record's current
    // end and advances it if it is kept: no branch on the mask.
    parallel_rows(out.RB, [&](int64_t rb) {
        uint16_t vals[kMaxValBytes / 2 + 8];
        for (int64_t kt = 0; kt < out.KT; ++kt) {
            const int64_t t = rb * out.KT + kt;
            const uint8_t *m = masks.data() + (size_t)t * kMaskBytes;
            const bool inside = (rb + 1) * kTileRows <= M && (kt + 1) * kTileK <= K;
            int64_t v = 0;
            for (int s = 0; s < kSteps; ++s) {
                // Values of step s: block (s, low nibble), then block (s, high nibble);
                // within a block lane 0's values first, in column order.
                for (int h = 0; h < 2; ++h) {
                    for (int l = 0; l < kLanes; ++l) {
                        const int r = l % kTileRows, g = l / kTileRows;
                        const uint32_t n = (uint32_t)(m[8 * l + s] >> (4 * h)) & 15u;
                        const uint16_t *w =
                            W + (rb * kTileRows + r) * ldw + kt * kTileK + tile_col(g, s, 0) + 4 * h;
                        if (inside) {
                            vals[v] = w[0];
                            v += n & 1;
                            vals[v] = w[1];
                            v += (n >> 1) & 1;
                            vals[v] = w[2];
                            v += (n >> 2) & 1;
                            vals[v] = w[3];
                            v += n >> 3;
                        } else {  // positions outside W are never kept
                            for (int j = 0; j < 4; ++j)
                                if (n & (1u << j)) vals[v++] = w[j];
                        }
                    }
                }
            }
            uint8_t *rec = out.stream.data() + (size_t)out.off[t] * 16;
            const size_t bytes = (size_t)v * 2, room = (size_t)(out.off[t + 1] - out.off[t]) * 16 - kMaskBytes;
            std::memcpy(rec, m, kMaskBytes);
            std::memcpy(rec + kMaskBytes, vals, bytes);
            std::memset(rec + kMaskBytes + bytes, 0, room - bytes);
        }
    });
}

bool decode_host(const HostEncoding &enc, uint16_t *W_out, uint8_t *mask_out) {
    const int64_t M = enc.M, K = enc.K;
    const int64_t T = enc.RB * enc.KT;
    if ((int64_t)enc.off.size() != T + 1) return false;
    if ((size_t)enc.off[T] * 16 != enc.stream.size()) return false;
    std::memset(W_out, 0, sizeof(uint16_t) * (size_t)(M * K));
    std::memset(mask_out, 0, (size_t)(M * K));
    bool ok = true;
    for (int64_t rb = 0; rb < enc.RB && ok; ++rb) {
        for (int64_t kt = 0; kt < enc.KT && ok; ++kt) {
            const int64_t t = rb * enc.KT + kt;
            const uint8_t *rec = enc.stream.data() + (size_t)enc.off[t] * 16;
            const int64_t cap = ((int64_t)enc.off[t + 1] - enc.off[t] - kMaskChunks) * 8;  // halfs
            const uint16_t *vals = reinterpret_cast<const uint16_t *>(rec + kMaskBytes);
            int64_t v = 0;
            for (int sh = 0; sh < 2 * kSteps && ok; ++sh) {
                const int s = sh / 2, h = sh % 2;  // block (step s, nibble half h)
                for (int l = 0; l < kLanes; ++l) {
                    const int r = l % kTileRows, g = l / kTileRows;
                    const int64_t row = rb * kTileRows + r;
                    const uint8_t b = rec[8 * l + s];
                    for (int j = 4 * h; j < 4 * h + 4; ++j) {
                        if (!(b & (1u << j))) continue;
                        const int64_t col = kt * kTileK + tile_col(g, s, j);
                        if (row >= M || col >= K || v >= cap) { ok = false; break; }
                        W_out[row * K + col] = vals[v++];
                        mask_out[row * K + col] = 1;
                    }
                }
            }
        }
    }
    return ok;
}

}  // namespace usp
