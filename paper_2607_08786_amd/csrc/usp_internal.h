// usp_internal.h -- handle layout and helpers shared by the library's sources.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <memory>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "usp.h"
#include "usp_format.h"

struct usp_matrix {
    int device;
    int64_t M, K;            // logical shape
    int64_t RB, KT;          // row blocks (16 rows) and column tiles (256 columns)
    int64_t nnz;
    int64_t max_chunks;      // most 16-byte value chunks in one tile record
    size_t stream_bytes;     // bytes of all tile records
    void *d_stream;          // device: tile records
    uint32_t *d_off;         // device: RB*KT + 1 offsets in 16-byte units
    int num_cus;             // compute units of the device
};

namespace usp {

// Most rows an encoding may have: the workspace's arrival counters (one
// 32-bit word per row block, rounded up to sets of 4) occupy a fixed 256 KB
// region at its start whatever the handle.
constexpr int64_t kMaxRows = int64_t(1) << 20;

// Allocator whose vectors leave new elements uninitialized: for buffers that are
// written whole (zeroing a layer's records first took as long as filling them).
template <class T>
struct NoInit : std::allocator<T> {
    template <class U>
    struct rebind {
        using other = NoInit<U>;
    };
    template <class U>
    void construct(U *p) noexcept {
        ::new ((void *)p) U;
    }
    template <class U, class... A>
    void construct(U *p, A &&...a) {
        ::new ((void *)p) U(std::forward<A>(a)...);
    }
};

// Host-side encoding result (before upload).
struct HostEncoding {
    int64_t M = 0, K = 0, RB = 0, KT = 0, nnz = 0;
    int64_t max_chunks = 0;        // most 16-byte value chunks in one record
    std::vector<uint32_t> off;     // RB*KT + 1 entries, 16-byte units
    std::vector<uint8_t, NoInit<uint8_t>> stream;  // 16 * off.back() bytes
};

// Encoder / decoder (usp_encode.cpp). encode_host throws std::bad_alloc on OOM.
void encode_host(const uint16_t *W, int64_t ldw, const uint8_t *mask, int64_t ldm,
                 int64_t M, int64_t K, HostEncoding &out);
// Returns false when the records are inconsistent with the shape.
bool decode_host(const HostEncoding &enc, uint16_t *W_out, uint8_t *mask_out);

// Error reporting (usp_abi.cpp).
usp_status fail(usp_status st, const std::string &msg);

// Launchers (usp_kernels.hip). They return hipSuccess or the launch error code.
struct SpmmPlan {
    int64_t row_groups;  // groups of 4 row blocks
    int64_t units;       // row groups * column tiles
    int64_t grid;        // persistent workgroups
    int64_t maxseg;      // most workgroups sharing one row group
    bool split;          // some row group is shared by several workgroups
};
SpmmPlan plan_spmm(const usp_matrix *A, int64_t N);
// The workspace of a product, and the least with which it runs (in parts, on the
// wide kernel above 256 tokens).
size_t spmm_workspace_bytes(const usp_matrix *A, int64_t N);
size_t spmm_workspace_min_bytes(const usp_matrix *A, int64_t N);
// The kernel usp_spmm runs for A and N (X 16-byte aligned, ldx = K), as text.
std::string describe_plan(const usp_matrix *A, int64_t N);
// Fused output epilogue: Y = act(W X + bias) + residual (all optional).
struct Epilogue {
    const uint16_t *bias = nullptr;  // fp16 [M]
    const uint16_t *res = nullptr;   // fp16, column n at res + n * ldr
    int64_t ldr = 0;
    int act = 0;                     // usp_activation
};
// What the kernels test of an epilogue: whether there is one, and which operands
// rows m .. m + 3 (m a multiple of 4) of a token may be read from as one 8-byte
// vector.
enum EpilogueFlags { kEpiBiasVec = 1, kEpiResVec = 2, kEpiAny = 4 };
inline int epilogue_flags(const Epilogue &ep) {
    return ((reinterpret_cast<uintptr_t>(ep.bias) & 7) == 0 ? kEpiBiasVec : 0) |
           ((reinterpret_cast<uintptr_t>(ep.res) & 7) == 0 && ep.ldr % 4 == 0 ? kEpiResVec : 0) |
           (ep.bias || ep.res || ep.act ? kEpiAny : 0);
}
int launch_spmm(const usp_matrix *A, const void *X, int64_t ldx, void *Y, int64_t ldy, int64_t N,
                const Epilogue &ep, void *workspace, size_t ws_bytes, void *stream);
// Arrival counters of a workspace: its first kCounterRegionBytes.
constexpr size_t kCounterRegionBytes = 256 * 1024;
constexpr int64_t kMaxCounters = kCounterRegionBytes / sizeof(uint32_t);

// The wide kernel (usp_wide.hip): whether it can run A at N tokens; its plan,
// with partials and packed X of at most max_bytes, those of its smallest part of
// at most min_bytes (grid 0: none fits); and the launch of that plan in a
// workspace that holds the counters and at least its smallest part.
struct WidePlan {
    int loads = 0, nb = 0;               // record load groups; blocks of 32 tokens per wavefront
    int64_t passes = 0;                  // launches over equal parts of the tokens
    int64_t tb = 0, sets = 0, tt = 0;    // blocks of 32 tokens of a pass; sets of 128 rows; token tiles
    int64_t tiles = 0, units = 0, grid = 0;
    bool split = false;                  // some tile is shared by several workgroups
    int slots = 1;                       // partial slots per workgroup
    size_t part_bytes = 0, pack_bytes = 0;
    size_t min_bytes = 0;                // partials and packed X of the smallest part
};
bool wide_serves(const usp_matrix *A, int64_t N);
WidePlan plan_wide(const usp_matrix *A, int64_t N, size_t max_bytes, size_t min_bytes);
int launch_wide(const usp_matrix *A, const WidePlan &plan, const void *X, int64_t ldx, void *Y, int64_t ldy,
                int64_t N, const Epilogue &ep, void *workspace, size_t ws_bytes, void *stream);
int launch_densify(const usp_matrix *A, void *Wd, int64_t ldw, void *stream);
// Device scratch of usp_spmm_noalloc: noalloc_setup looks up and clears the
// calling thread's current device's copy once (returns a HIP error code);
// noalloc_scratch returns its device address, or null before the set-up.
int noalloc_setup(int device);
void *noalloc_scratch(int device);

}  // namespace usp
