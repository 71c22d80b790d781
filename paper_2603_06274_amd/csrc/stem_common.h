// Internal declarations shared by the host API and the gfx950 kernels of libstem_hip.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>

#include "stem.h"

namespace stem {

// Packed-sequence table, passed to kernels by value (no device-side cu_seqlens read, no sync).
// A call covers, of every sequence, the query blocks of one chunk [chunk_start, chunk_end) (the
// whole sequence unless the shape says otherwise) and the keys before chunk_end.
struct SeqTable {
    int32_t batch;
    int32_t tok_start[STEM_MAX_BATCH + 1];      // cu_seqlens: token rows of K and V
    int32_t row_start[STEM_MAX_BATCH + 1];      // prefix sums of the call's query-block rows
    int32_t q_tok_start[STEM_MAX_BATCH + 1];    // prefix sums of the call's query tokens (rows of Q, O, lse)
    int32_t key_row_start[STEM_MAX_BATCH + 1];  // prefix sums of all blocks per sequence (rows of k_bar, m_v)
    int32_t first_block[STEM_MAX_BATCH];        // index in its sequence of the first query block of the call
    int32_t kv_end[STEM_MAX_BATCH];             // token row of K/V one past the last key of the call
};

// Everything the host derives from a stem_shape.
struct Problem {
    int32_t Hq, Hkv, G, B, batch;
    int32_t d;        // head size: 64, 128 or 256
    int32_t T;        // query tokens of the call (rows of Q, O, lse)
    int32_t R;        // query-block rows of the call
    int32_t Rk;       // blocks of all sequences (rows of k_bar, m_v)
    int32_t NBmax;    // most key blocks any row of the call can see
    int64_t q_st, q_sh, kv_st, kv_sh;
    SeqTable seq;
};

int make_problem(const stem_shape* shape, Problem* out);

struct WorkspaceLayout {
    size_t q_bar, k_bar, m_v, total;
};
WorkspaceLayout workspace_layout(const Problem& p, int ad_stride);
// STEM_OK if S is a supported anti-diagonal stride for this block size.
int check_ad_stride(const Problem& p, int ad_stride);

// Kernel launchers (one per translation unit); each returns a STEM_* status.
int launch_pool(const Problem& p, int ad_stride, const void* q, const void* k, const void* v,
                float* q_bar, float* k_bar, float* m_v, hipStream_t stream);
int launch_block_scores(const Problem& p, int ad_stride, const float* q_bar, const float* k_bar,
                        const float* m_v, float beta, float route_scale, bool fill_non_causal,
                        float* scores, hipStream_t stream);
int launch_group_scores(const Problem& p, const float* scores, int reduce, float* group_scores,
                        hipStream_t stream);
// heads = number of lists per row: Hq, or Hkv for group-shared lists
int launch_select(const Problem& p, int heads, const float* scores, const int32_t* budget,
                  int32_t n_sink, int32_t n_local, int32_t* counts, int32_t* indices, int32_t kmax,
                  hipStream_t stream);
int launch_score_select(const Problem& p, int ad_stride, const float* q_bar, const float* k_bar,
                        const float* m_v, float beta, float route_scale, const int32_t* budget,
                        int32_t n_sink, int32_t n_local, int32_t* counts, int32_t* indices,
                        int32_t kmax, float* debug_scores, hipStream_t stream);
int launch_sparse_attn(const Problem& p, const void* q, const void* k, const void* v,
                       const int32_t* counts, const int32_t* indices, int32_t kmax,
                       bool lists_per_kv_head, float softmax_scale, void* out, float* lse,
                       int32_t* queue, hipStream_t stream);
// Compute units of the current device, 0 on failure.  A constant of the device, kept after the first call
// (several threads may store the same value): the query costs a call that has 30 us in all about 1 %.
inline int compute_units() {
    constexpr int kDevices = 64;
    static std::atomic<int> known[kDevices];           // zero at start
    int device = 0, cus = 0;
    if (hipGetDevice(&device) != hipSuccess || device < 0) return 0;
    if (device < kDevices && (cus = known[device].load(std::memory_order_relaxed)) > 0) return cus;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || cus <= 0) return 0;
    if (device < kDevices) known[device].store(cus, std::memory_order_relaxed);
    return cus;
}

// How launch_sparse_attn hands its rows (head, query block) out to the workgroups: XCD x has slots 0 .. slots - 1, of which
// those before claim_from are rows by their number and the others claim one.
struct AttentionGrid {
    int32_t xcds_per_kv_head;   // XCDs that share one KV head's rows; 0: contiguous ranges of all rows instead
    int32_t items_per_xcd;      // most rows of one XCD
    int32_t claim_from;         // 0x7fffffff: no row is claimed
    int64_t slots;              // per XCD
};
constexpr int64_t kMaxWorkgroups = 0x7fffffff;         // of a launch
// units: where the number of compute units comes from (asked for long calls only)
bool attention_claims_rows(const Problem& p, int32_t kmax, int (*units)() = compute_units);
AttentionGrid attention_grid(const Problem& p, int32_t kmax, bool queue, int (*units)() = compute_units);
// rows of XCD x (0 and less: none)
__host__ __device__ inline int rows_of_xcd(int x, int Hq, int R, int G, int items_per_xcd, int xcds_per_kv_head) {
    if (xcds_per_kv_head > 0) return (R - x % xcds_per_kv_head + xcds_per_kv_head - 1) / xcds_per_kv_head * G;
    const int64_t left = (int64_t)Hq * R - (int64_t)x * items_per_xcd;
    return left < items_per_xcd ? (int)left : items_per_xcd;
}

inline int check_launch() {
    return hipGetLastError() == hipSuccess ? STEM_OK : STEM_ERR_HIP;
}

#if defined(__HIPCC__)
// Place of x in the n ascending prefix sums `start` (start[0] = 0, n <= 64, entries n .. 63 beyond every x): the last
// s < n with start[s] <= x.  Three sums and fewer are looked at one after the other.  For more, every lane
// loads one and a ballot counts: a scalar loop waits for one load after the other, which every workgroup of a
// packed batch paid before its first load of data (64 prompts of 100 tokens, 8 / 1 heads, all stages
// 44.6 -> 31.4 us; equal at four prompts, and at two the one scalar load is 0.1 us a kernel shorter than a load
// per lane).  Called by whole waves with one x per wave.
__device__ __forceinline__ int place_in(const int32_t* start, int n, int x) {
    static_assert(STEM_MAX_BATCH <= 64, "one lane per sequence");
    if (n > 3) return (int)__popcll(__builtin_amdgcn_ballot_w64(start[threadIdx.x & 63] <= x)) - 1;
    int s = 0;
    for (int y = 1; y < n; ++y) s = x >= start[y] ? y : s;
    return s;
}

// Sequence of a global query-block row.  Wave-uniform.
__device__ __forceinline__ int seq_of_row(const SeqTable& t, int r) { return place_in(t.row_start, t.batch, r); }

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
#endif

}  // namespace stem
